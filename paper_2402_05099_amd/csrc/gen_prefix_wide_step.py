#!/usr/bin/env python3
"""Writes prefix_wide_step.inc (D = 128) and prefix_wide_step_d64.inc (D = 64): the body of one pipeline step of the
256-row shared-block attention kernel (prefix_wide_impl.h) as straight-line C++.

Step j is 16 MFMAs in a fixed order: the first half of P*V of stage j (4), the scores of stage j + 2 (8), the second half of P*V
(4); a stage is 32 keys at D = 128 and 64 keys, two score tiles, at D = 64.  Between them go, in fixed places: the step's vector-ALU
work on stage j + 1, whose scores the step before has left (exponentials, packing to bf16, fp32 row sums), its two
HBM->LDS copy instructions (addressed by the kernel's copy cursor `cur`, which runs AHEAD stages ahead of the piece
`pc` being computed) and its 24 LDS fragment reads.  Every gap ends in a scheduling barrier so that the compiler keeps
this order: a wavefront then always has a matrix instruction in flight while it issues vector-ALU instructions,
instead of running the two kinds back to back.  The exponentials need no result of their own step and their own step needs
none of them, so they go evenly into all the gaps, and the row sum is there before the weights are multiplied with anything: it
says whether they have to be taken again against a larger maximum, which spares every step the search for it.

usage: gen_prefix_wide_step.py [D [out.inc [vector-ALU cycles per gap]]]     (no arguments: both files)
"""
import os
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
DEFAULT_OUT = {128: os.path.join(HERE, "prefix_wide_step.inc"), 64: os.path.join(HERE, "prefix_wide_step_d64.inc")}
DEFAULT_CAP = {128: 22.0, 64: 44.0}     # a 32x32x16 MFMA occupies the matrix pipe for 32 cycles
XYZW = "xyzw"
# measured issue cost of one wave64 instruction, cycles
C_FMA, C_EXP, C_CVT, C_ADD = 5.2, 8.8, 5.2, 4.9


def build(D=128, CAP=None):
    CAP = DEFAULT_CAP[D] if CAP is None else CAP
    wide = D == 128
    # score tile(s) of a stage as the kernel names them
    cur_t = ["Scur"] if wide else ["Scur.a", "Scur.b"]
    nxt_t = ["Snext"] if wide else ["Snext.a", "Snext.b"]
    # Only half a stage of K and of V fragments is held in registers (two wavefronts share a SIMD's register file):
    # each fragment register is reloaded twice per step, four gaps before its next use.  Fragment f of a stage's K is
    # (score tile f / KS, k-step f % KS); V fragments are (16-key group tt, 32-column block db).
    KS, DB = D // 16, D // 32
    mf = []         # [MFMA statement, statements before the gap's ALU work, statements after it]

    def value(i):
        return f"mfma_acc(Oacc[{i % DB}], vf[{i & 3}], pb[{i // DB}]);"

    def v_load(i, slot):      # fragment i (0 .. 7) of a stage's V
        return f"vf[{i & 3}] = lds_v({slot}, {i // DB}, {i % DB});"

    for i in range(4):           # gaps 0 .. 3; first half of the K fragments of stage j+2
        mf.append([value(i), [], [f"kf[{i}] = lds_k(slot2, {i});"]])
    for q in range(8):           # gaps 4 .. 11; second half of K, then second half of the V fragments of stage j
        tile, ks = (0, q) if wide else (q // 4, q % 4)
        f = "mfma_first" if ks == 0 else "mfma_acc"
        mf.append([f"{f}({nxt_t[tile]}, kf[{q & 3}], qf[{ks}]);", [], [f"kf[{q}] = lds_k(slot2, {q + 4});" if q < 4 else v_load(q, "slot")]])
    for i in range(4, 8):        # gaps 12 .. 15; first half of the V fragments of stage j+1, for the next step
        mf.append([value(i), [], [v_load(i - 4, "slot1")]])
    # the copy that keeps the ring AHEAD stages ahead (the copy cursor may already be in a later piece): scalar address
    # arithmetic in gap 0, the two copy instructions in gaps 1 and 3
    mf[0][1].extend(["const int64_t cp_off = (int64_t)min(cur.ks + cur.t * KT, cur.kwin) * rstride_b;",
                     "const unsigned cp_dst = ldsw + (unsigned)((slot + AHEAD) & (NS - 1)) * STB;"])
    mf[1][1].append("copy16(cur.Kg + cp_off, cur.voffK, cp_dst);")
    mf[3][1].append("copy16(cur.Vg + cp_off, cur.voffV, cp_dst + VRING);")

    work = []     # (cycles, statement)
    n = 0
    NPB = (32 if wide else 64) // 16        # packed operands pn[h]: the exponentials of keys 16 h .. 16 h + 15 of the stage
    pending = []
    for h in range(NPB):
        src = cur_t[h // 2]
        ids = list(range(n, n + 4))
        # all multiply-adds of a block of 8 scores, then its exponentials, then the packs and sums of the block: no instruction
        # uses the result of the one just before it
        for p, k in enumerate(ids):
            i0 = 8 * (h % 2) + 2 * p
            work.append((C_FMA, f"const float xa{k} = fmaf({src}[{i0}], c2, -mc);"))
            work.append((C_FMA, f"const float xb{k} = fmaf({src}[{i0 + 1}], c2, -mc);"))
        for p, k in enumerate(ids):
            work.append((C_EXP, f"const float ea{k} = __builtin_amdgcn_exp2f(xa{k});"))
            work.append((C_EXP, f"const float eb{k} = __builtin_amdgcn_exp2f(xb{k});"))
        for p, k in enumerate(ids):
            work.append((C_CVT, f"pn[{h}].{XYZW[p]} = pack_bf16_pair(ea{k}, eb{k});"))
            if k == 0:
                pending += ["ea0", "eb0"]
            elif k == 1:
                work.append((C_ADD, "float sa = ea0 + ea1;"))
                work.append((C_ADD, "float sb = eb0 + eb1;"))
            else:
                work.append((C_ADD, f"sa += ea{k};"))
                work.append((C_ADD, f"sb += eb{k};"))
        n += 4
    work.append((C_ADD, "ssum = sa + sb;"))
    out = []
    wi = 0
    budget = 0.0
    for g, (stmt, pre, post) in enumerate(mf):
        out.append(f"// gap {g}")
        out.append(stmt)
        out.extend(pre)
        if g == 0:
            out.append("if (kMasked) mask_stage(Scur, j + 1);")
        budget += CAP
        while wi < len(work) and budget > 0:
            out.append(work[wi][1])
            budget -= work[wi][0]
            wi += 1
        out.extend(post)
        out.append("__builtin_amdgcn_sched_barrier(0);")
    assert wi == len(work), ("work left over", wi, len(work))
    return "\n".join("        " + l for l in out) + "\n"


def write(D, out=None, cap=None):
    with open(out or DEFAULT_OUT[D], "w") as f:
        f.write(f"// Generated by gen_prefix_wide_step.py (one pipeline step of prefix_wide_impl.h, D = {D}); do not edit by hand.\n" + build(D, cap))


if __name__ == "__main__":
    if len(sys.argv) > 1:
        write(int(sys.argv[1]), sys.argv[2] if len(sys.argv) > 2 else None, float(sys.argv[3]) if len(sys.argv) > 3 else None)
    else:
        write(128)
        write(64)
