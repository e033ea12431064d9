// One wavefront's tile of query rows on the matrix cores, multiplied with stages of 32 K/V rows in LDS: fragment
// addresses, scores, online softmax, value product and results.  Used by the matrix-core suffix kernel (decode_mfma.hip)
// and by the combined launch (combined_impl.h).
#pragma once
#include "hg_internal.h"
#include "prefix_common.h"

namespace hg {
namespace dm {

constexpr int KT = 32;                  // keys per stage
constexpr float TAU = 8.0f;             // lazy-rescale threshold, log2 units

// Sizes that follow from the head dimension, and the XOR swizzles of the 16-byte chunks of a bf16 row in LDS (applied
// on the global side of the copies).  D = 128: a row is 256 bytes, one period of the 64 banks: K (and Q) chunk ^ row % 16
// makes the 16 rows of a ds_read_b128 pass distinct, V chunk ^ 4 (row % 4) separates the 4 rows of a transposing read.
// D = 64: a row is half a period, so consecutive rows already differ; K chunk ^ (row / 2) % 8, V chunk ^ 4 ((row / 2) % 2).
template <int D>
struct Geo {
    static_assert(D == 64 || D == 128, "head dimension");
    static constexpr int KS = D / 16;              // MFMA k-steps of the score product
    static constexpr int DB = D / 32;              // 32-row blocks of O^T
    static constexpr int CPR = D / 8;              // 16-byte chunks per bf16 row
    static constexpr int RPI = 64 / CPR;           // rows one copy instruction covers
    static constexpr int CPS = KT / RPI;           // copy instructions per stage and tensor
    static constexpr int ROWB = D * 2;             // bytes per bf16 row
    static constexpr int STB = KT * ROWB;          // bytes per stage and tensor
    static __device__ __forceinline__ int kswz(int row) { return D == 128 ? row % 16 : (row >> 1) & 7; }
    static __device__ __forceinline__ int vswz(int row) { return D == 128 ? 4 * (row % 4) : 4 * ((row >> 1) & 1); }
};

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pack_pair(float lo, float hi) {
    floatx2 f = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}

// s_waitcnt vmcnt(n) alone (lgkmcnt and expcnt untouched): vmcnt is split over bits [3:0] and [15:14]
template <int N>
__device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// A tile of TR query rows (32, or 16: see decode_mfma.hip) and the fragment addresses of its stages, relative to the K or V
// part of a stage.  FP8: K and V rows are E4M3 codes.
template <int D, bool FP8, int TR>
struct MfmaTile {
    using G_ = Geo<D>;
    static constexpr int KS = G_::KS, DB = G_::DB, CPR = G_::CPR, RPI = G_::RPI, CPS = G_::CPS, ROWB = G_::ROWB, STB = G_::STB;
    static constexpr int KS16 = D / 32, DB16 = D / 16;
    static constexpr int ES = FP8 ? 1 : 2;                // bytes per cache element
    static constexpr int CPRG = D * ES / 16;              // 16-byte chunks per cache row
    static constexpr int RPIG = 64 / CPRG;                // cache rows one copy instruction covers
    static constexpr int CPSG = KT / RPIG;                // copy instructions per stage and tensor
    static constexpr int QOPS = TR / RPI;                 // copy instructions of a query tile
    typedef float floatx4 __attribute__((ext_vector_type(4)));

    int l, lq, hl;         // lane; 32-row tiles: row of the tile, half of the keys
    int ln, lg;            // 16-row tiles: row of the tile and lane group (quarter of the keys)
    unsigned kaddr[KS], qaddr[KS];     // K fragments of a stage, Q fragments of a tile (bf16: the same addresses)
    unsigned kaddr16[2][KS16], qaddr16[KS16], vaddr16[DB16];
    unsigned vaddr8[DB], vaddr[DB];
    bf16x8 qf[KS], qf16[KS16];
    floatx16 Oacc[DB];
    floatx4 Oacc16[DB16];
    float c2, tau_raw, kscale;
    float m_used;          // raw-score maximum the exponentials are taken against (-inf: no key seen yet)
    float mc;              // m_used * c2, 0 while no key has been seen
    float lsum;            // this lane's share of the row sum (unrounded exponentials)
    struct Scores { floatx16 S; floatx4 S4[2]; };

    __device__ __forceinline__ explicit MfmaTile(float scale, int lane) {
        l = lane; lq = l & 31; hl = l >> 5; ln = l & 15; lg = l >> 4;
        kscale = scale;                // raw scores are in units of the codes
        c2 = kscale * kLog2e;
        tau_raw = TAU / c2;
        // ---- LDS fragment addresses (relative to the slot), as in prefix_wide.hip ------------------------------------------
#pragma unroll
        for (int s = 0; s < KS; ++s) kaddr[s] = qaddr[s] = (unsigned)(lq * ROWB + (((2 * s + hl) ^ G_::kswz(lq)) * 16));
        // FP8: the 8 codes of K row lq, columns 16 s + 8 hl .. +7: rows lie in copy order (row r at (r/8) KiB + (r%8) 128 B),
        // their 16-byte chunks XOR-swizzled by (r/2) % 8 on the global side so that 16 consecutive lanes hit 32 different banks
        if constexpr (FP8) {
#pragma unroll
            for (int s = 0; s < KS; ++s)
                kaddr[s] = (unsigned)((lq >> 3) * 1024 + (lq & 7) * 128 + ((s ^ ((lq >> 1) & 7)) * 16) + 8 * hl);
        }
        // 16-row tiles.  K (A operand, 16 keys x 32 columns per MFMA) and Q (B operand, 32 columns x 16 rows): lane (lg, ln)
        // holds row ln of the 16-key group (of the tile), columns 32 s + 8 lg .. +7: 16-byte chunk 4 s + lg of that row.
        // V^T (A operand, 16 columns x 32 keys): k-slot e of lane group lg stands for key 16 (e / 4) + 4 lg + e % 4, the key
        // whose score this lane holds as element e % 4 of score tile e / 4; lane s of a group points ds_read_b64_tr_b16 at
        // key 4 lg + s / 4, columns 16 db + 4 (s % 4) .. +3, and receives column 16 db + s of the group's four keys.
        if constexpr (TR == 16) {
#pragma unroll
            for (int s = 0; s < KS16; ++s) {
                qaddr16[s] = (unsigned)(ln * ROWB + (((4 * s + lg) ^ G_::kswz(ln)) * 16));
#pragma unroll
                for (int kg = 0; kg < 2; ++kg)
                    kaddr16[kg][s] = (unsigned)((16 * kg + ln) * ROWB + (((4 * s + lg) ^ G_::kswz(16 * kg + ln)) * 16));
            }
            const int vrow = 4 * lg + (ln >> 2), q4 = ln & 3;
#pragma unroll
            for (int db = 0; db < DB16; ++db)
                vaddr16[db] = (unsigned)(vrow * ROWB + (((2 * db + (q4 >> 1)) ^ G_::vswz(vrow)) * 16) + (q4 & 1) * 8);
            if constexpr (FP8) {
                // codes, rows in copy order: K row ln of key group kg, columns 32 s + 8 lg .. +7 (8 bytes); V^T through
                // ds_read_b64_tr_b8 as for 32-row tiles, lane s of a group pointing at the key of k-slot s / 2
                // (16 (j / 4) + 4 lg + j % 4) and columns 16 db + 8 (s % 2) .. +7; V chunks swizzled by (r/2) % 2 + 2 ((r/16) % 2)
#pragma unroll
                for (int s = 0; s < KS16; ++s)
#pragma unroll
                    for (int kg = 0; kg < 2; ++kg) {
                        const int row = 16 * kg + ln;
                        kaddr16[kg][s] = (unsigned)((row >> 3) * 1024 + (row & 7) * 128 + (((2 * s + (lg >> 1)) ^ ((row >> 1) & 7)) * 16) + 8 * (lg & 1));
                    }
                const int j = ln >> 1, pp = ln & 1;
                const int row = 16 * (j >> 2) + 4 * lg + (j & 3);
                const int fsw = ((row >> 1) & 1) | (((row >> 4) & 1) << 1);
#pragma unroll
                for (int db = 0; db < DB16; ++db)
                    vaddr16[db] = (unsigned)((row >> 3) * 1024 + (row & 7) * 128 + ((db ^ fsw) * 16) + 8 * pp);
            }
        }
        // FP8, V^T: ds_read_b64_tr_b8 works on groups of 16 lanes: every lane supplies the address of 8 bytes, and lane i
        // of the group receives, as byte j, byte i % 8 of the piece that lane 2 j + i / 8 of the group pointed at.  So
        // lane s of a group points at the V codes of key 8 (j / 4) + 4 hl + j % 4 (j = s / 2, the key of k-slot j), columns
        // 16 g1 + 8 (s % 2) .. +7 of the 32-column block: lane i then holds column 16 g1 + i of the 8 keys in k-slot order.
        // Rows lie in copy order (row r at (r / 8) KiB + (r % 8) 128 B); 16-byte chunks are XOR-swizzled on the global
        // side by (r / 2) % 2 + 2 ((r / 8) % 2), which spreads the 8 rows of a read over all banks.
        if constexpr (FP8) {
            const int sg = l & 15, g1 = (l >> 4) & 1;
            const int j = sg >> 1, pp = sg & 1;
            const int row = 8 * (j >> 2) + 4 * hl + (j & 3);        // + 16 tt
            const int fsw = ((row >> 1) & 1) | (((row >> 3) & 1) << 1);
#pragma unroll
            for (int db = 0; db < DB; ++db)
                vaddr8[db] = (unsigned)((row >> 3) * 1024 + (row & 7) * 128 + (((2 * db + g1) ^ fsw) * 16) + 8 * pp);
        }
        {
            const int i16 = l & 15, g1 = (l >> 4) & 1;
            const int keyq = 4 * hl + (i16 >> 2);
            const int fv = G_::vswz(keyq);
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int chunk = 4 * db + 2 * g1 + ((i16 & 3) >> 1);
                vaddr[db] = (unsigned)(keyq * ROWB + ((chunk ^ fv) * 16) + (i16 & 1) * 8);   // relative to the V stage
            }
        }
        clear();
        for (int s = 0; s < KS; ++s) qf[s] = __builtin_bit_cast(bf16x8, uintx4{0, 0, 0, 0});
        for (int s = 0; s < KS16; ++s) qf16[s] = __builtin_bit_cast(bf16x8, uintx4{0, 0, 0, 0});
    }

    __device__ __forceinline__ int row() const { return TR == 16 ? ln : lq; }      // this lane's row of the tile

    // fresh softmax state
    __device__ __forceinline__ void clear() {
        if constexpr (TR == 16) {
#pragma unroll
            for (int i = 0; i < DB16; ++i) Oacc16[i] = floatx4{0.f, 0.f, 0.f, 0.f};
        } else {
#pragma unroll
            for (int i = 0; i < DB; ++i)
#pragma unroll
                for (int k = 0; k < 16; ++k) Oacc[i][k] = 0.f;
        }
        m_used = -INFINITY;
        mc = 0.f;
        lsum = 0.f;
    }

    // Q tile at sb (LDS) -> registers; the reads have completed when this returns, sb may be overwritten
    __device__ __forceinline__ void load_q(const unsigned char* sb) {
        if constexpr (TR == 16) {
#pragma unroll
            for (int s = 0; s < KS16; ++s) qf16[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(sb + qaddr16[s]));
#pragma unroll
            for (int s = 0; s < KS16; ++s) asm volatile("" : "+v"(qf16[s]));
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) qf[s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4*>(sb + qaddr[s]));
#pragma unroll
            for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qf[s]));
        }
        asm volatile("" ::: "memory");
    }

    static __device__ __forceinline__ uintx4 expand8(unsigned c0, unsigned c1) {      // eight codes -> bf16, exactly
        uintx4 v;
        v[0] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c0, 1.0f, false));
        v[1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c0, 1.0f, true));
        v[2] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c1, 1.0f, false));
        v[3] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(c1, 1.0f, true));
        return v;
    }
    static __device__ __forceinline__ uintx4 k_fragment(const unsigned char* p) {
        if constexpr (FP8) {
            typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
            const uintx2 kc = *reinterpret_cast<const uintx2*>(p);
            return expand8(kc[0], kc[1]);
        } else {
            return *reinterpret_cast<const uintx4*>(p);
        }
    }

    // S^T = K Q^T for the K rows at sb.  16-row tiles: element i of tile kg is the score of stage row 16 kg + 4 lg + i;
    // 32-row tiles: element i that of row 8 (i / 4) + i % 4 + 4 hl
    __device__ __forceinline__ void scores(const unsigned char* sb, Scores& r) const {
        if constexpr (TR == 16) {
#pragma unroll
            for (int kg = 0; kg < 2; ++kg) r.S4[kg] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS16; ++s)
#pragma unroll
                for (int kg = 0; kg < 2; ++kg)
                    r.S4[kg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k_fragment(sb + kaddr16[kg][s])), qf16[s], r.S4[kg], 0, 0, 0);
            // (the wait states between a product and a read of its result: the compiler leaves them out where a branch lies
            // between, as the one around the mask does)
            asm volatile("s_nop 7" : "+v"(r.S4[0]), "+v"(r.S4[1]));
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) r.S[i] = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s)
                r.S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, k_fragment(sb + kaddr[s])), qf[s], r.S, 0, 0, 0);
            asm volatile("s_nop 11" : "+v"(r.S));
        }
    }

    // stage rows outside [lo, hi) get the score -inf (hi may differ from lane to lane)
    __device__ __forceinline__ void mask(Scores& r, int lo, int hi) const {
        if constexpr (TR == 16) {
            const int lo_i = lo - 4 * lg, hi_i = hi - 4 * lg;
#pragma unroll
            for (int kg = 0; kg < 2; ++kg)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int ri = 16 * kg + i;
                    if (ri < lo_i || ri >= hi_i) r.S4[kg][i] = -INFINITY;
                }
        } else {
            const int lo_i = lo - 4 * hl, hi_i = hi - 4 * hl;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int ri = 8 * (i >> 2) + (i & 3);
                if (ri < lo_i || ri >= hi_i) r.S[i] = -INFINITY;
            }
        }
    }

    // online softmax: scores -> weights as B operand of the value product (k-slot order), row sums, lazy rescaling
    __device__ __forceinline__ void softmax(const Scores& r, uintx4 (&pb)[2]) {
        float tmax;
        if constexpr (TR == 16) {
            tmax = fmaxf(fmaxf(fmaxf(r.S4[0][0], r.S4[0][1]), fmaxf(r.S4[0][2], r.S4[0][3])),
                         fmaxf(fmaxf(r.S4[1][0], r.S4[1][1]), fmaxf(r.S4[1][2], r.S4[1][3])));
            tmax = fmaxf(tmax, __shfl_xor(tmax, 16));      // the four lanes that share a row
        } else {
            tmax = fmaxf(r.S[0], r.S[1]);
#pragma unroll
            for (int i = 2; i < 16; i += 2) tmax = fmaxf(fmaxf(tmax, r.S[i]), r.S[i + 1]);
        }
        tmax = half_max(tmax);
        if (__any(tmax > m_used + tau_raw)) {
            const float m_new = fmaxf(m_used, tmax);
            // equal maxima (also -inf and -inf: a row that has seen no key yet) keep the accumulators
            const float alpha = (m_new == m_used) ? 1.0f : __builtin_amdgcn_exp2f((m_used - m_new) * c2);
            m_used = m_new;
            mc = (m_new == -INFINITY) ? 0.f : m_new * c2;
            lsum *= alpha;
            if constexpr (TR == 16) {
#pragma unroll
                for (int i = 0; i < DB16; ++i)
#pragma unroll
                    for (int k = 0; k < 4; ++k) Oacc16[i][k] *= alpha;
            } else {
#pragma unroll
                for (int i = 0; i < DB; ++i)
#pragma unroll
                    for (int k = 0; k < 16; ++k) Oacc[i][k] *= alpha;
            }
        }
#pragma unroll
        for (int tt = 0; tt < (TR == 16 ? 1 : 2); ++tt) {
            float p[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                p[i] = __builtin_amdgcn_exp2f(fmaf(TR == 16 ? r.S4[i >> 2][i & 3] : r.S[8 * tt + i], c2, -mc));
                lsum += p[i];
            }
            pb[tt] = uintx4{pack_pair(p[0], p[1]), pack_pair(p[2], p[3]), pack_pair(p[4], p[5]), pack_pair(p[6], p[7])};
        }
    }

    // O^T += V^T P^T for the V rows at vs.  The fragment reads have completed when this returns.
    __device__ __forceinline__ void values(const unsigned char* vs, const uintx4 (&pb)[2]) {
        typedef int intx2 __attribute__((ext_vector_type(2)));
        if constexpr (TR == 16) {
#pragma unroll
            for (int db = 0; db < DB16; ++db) {
                const unsigned char* vp = vs + vaddr16[db];
                if constexpr (FP8) {
                    const intx2 vc = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) intx2*)HG_LDS(vp));
                    const uintx4 vv = expand8((unsigned)vc[0], (unsigned)vc[1]);
                    Oacc16[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vv), __builtin_bit_cast(bf16x8, pb[0]), Oacc16[db], 0, 0, 0);
                } else {
                    const shortx4 vlo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp));
                    const shortx4 vhi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp + 16 * ROWB));
                    const shortx8 vv = __builtin_shufflevector(vlo, vhi, 0, 1, 2, 3, 4, 5, 6, 7);
                    Oacc16[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vv), __builtin_bit_cast(bf16x8, pb[0]), Oacc16[db], 0, 0, 0);
                }
            }
#pragma unroll
            for (int db = 0; db < DB16; ++db) asm volatile("" : "+v"(Oacc16[db]));
        } else {
#pragma unroll
            for (int tt = 0; tt < 2; ++tt)
#pragma unroll
                for (int db = 0; db < DB; ++db) {
                    if constexpr (FP8) {
                        const unsigned char* vp = vs + vaddr8[db] + tt * 2048;     // keys 16 tt ..: two copy blocks further
                        const intx2 vc = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) intx2*)HG_LDS(vp));
                        const uintx4 vv = expand8((unsigned)vc[0], (unsigned)vc[1]);
                        Oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv), __builtin_bit_cast(bf16x8, pb[tt]), Oacc[db], 0, 0, 0);
                    } else {
                        const unsigned char* vp = vs + vaddr[db] + tt * 16 * ROWB;
                        const shortx4 vlo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp));
                        const shortx4 vhi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp + 8 * ROWB));
                        const shortx8 vv = __builtin_shufflevector(vlo, vhi, 0, 1, 2, 3, 4, 5, 6, 7);
                        Oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vv), __builtin_bit_cast(bf16x8, pb[tt]), Oacc[db], 0, 0, 0);
                    }
                }
            // the accumulators depend on every fragment read of the stage: once they are pinned here the reads have
            // completed, and a later copy may overwrite the rows
#pragma unroll
            for (int db = 0; db < DB; ++db) asm volatile("" : "+v"(Oacc[db]));
        }
        asm volatile("" ::: "memory");
    }

    // V rows below lo / from hi on of the stage at vs -> 0 (they may hold anything; their weights are zero, but 0 * NaN is
    // NaN).  Lane l of copy instruction i holds cache row RPIG i + l / CPRG.  (Two functions: as one with both bounds it cost
    // the paged and comparison forms of decode_mfma.hip 11 to 13 spilled scalar registers, and the paged one 2 %.)
    __device__ __forceinline__ void clear_v_below(unsigned char* vs, int lo) const {
#pragma unroll
        for (int i = 0; i < CPSG; ++i)
            if (i * RPIG + l / CPRG < lo) *reinterpret_cast<uintx4*>(vs + i * 1024 + l * 16) = uintx4{0u, 0u, 0u, 0u};
    }
    __device__ __forceinline__ void clear_v_from(unsigned char* vs, int hi) const {
#pragma unroll
        for (int i = 0; i < CPSG; ++i)
            if (i * RPIG + l / CPRG >= hi) *reinterpret_cast<uintx4*>(vs + i * 1024 + l * 16) = uintx4{0u, 0u, 0u, 0u};
    }

    // (O, LSE) of this lane's row to part `c`; rv: the row exists; vscale: scale of the values (1 for bf16 rows)
    __device__ __forceinline__ void store(const OutDev& out, int c, int64_t qidx, bool rv, float vscale) const {
        float lsub = lsum;
        if constexpr (TR == 16) lsub += __shfl_xor(lsub, 16);
        const float ltot = half_sum(lsub);
        if (!rv) return;
        float* const Of = static_cast<float*>(out.O) + (int64_t)c * out.part_stride_O + qidx * D;
        uint16_t* const Ob = static_cast<uint16_t*>(out.O) + (int64_t)c * out.part_stride_O + qidx * D;
        const float inv = ltot > 0.f ? (FP8 ? vscale / ltot : 1.0f / ltot) : 0.f;    // a row that sees no key of this chunk: O = 0, LSE = -inf
        auto put = [&](int d, float o0, float o1, float o2, float o3) {
            if (out.bf16) *reinterpret_cast<uint2*>(Ob + d) = make_uint2(pack_bf16(o0, o1), pack_bf16(o2, o3));
            else *reinterpret_cast<float4*>(Of + d) = make_float4(o0, o1, o2, o3);
        };
        if constexpr (TR == 16) {
#pragma unroll
            for (int db = 0; db < DB16; ++db)     // element i of block db is column 16 db + 4 lg + i of this lane's row
                put(16 * db + 4 * lg, Oacc16[db][0] * inv, Oacc16[db][1] * inv, Oacc16[db][2] * inv, Oacc16[db][3] * inv);
        } else {
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
                    put(32 * db + 8 * q4 + 4 * hl, Oacc[db][4 * q4] * inv, Oacc[db][4 * q4 + 1] * inv, Oacc[db][4 * q4 + 2] * inv,
                        Oacc[db][4 * q4 + 3] * inv);
        }
        if ((TR == 16 ? lg : hl) == 0)
            out.LSE[(int64_t)c * out.part_stride_L + qidx] = ltot > 0.f ? m_used * kscale + __logf(ltot) : -INFINITY;
    }
};

}  // namespace dm
}  // namespace hg
