// Inter-sequence batched attention over one shared KV block (Sec. 3.2 of the paper), persistent 256-row kernel: the
// body shared by prefix_wide.hip (D = 128, HG_WIDE_D = 128) and prefix_wide_d64.hip (D = 64), which define HG_WIDE_D and
// HG_WIDE_KERNEL and include this file; the head dimension is a macro, not a template parameter, so that each
// translation unit sees exactly one kernel.  The B*G query rows that use a KV head are stacked into one matrix and multiplied against that
// head's keys/values on the matrix cores with an online softmax in registers, returning (O, LSE) per part
// (Eq. 1, Eq. 4); the parts are combined by the LSE merge (Eq. 5).
//
// Same mathematics and LDS layout as prefix.hip (transposed products S^T = K Q^T and O^T += V^T P^T with
// v_mfma_f32_32x32x16_bf16, K/V tiles in their HBM layout with XOR-swizzled 16-byte chunks, transposing LDS
// reads for V).  What differs, and why:
//   * One workgroup per CU, 8 wavefronts x 32 query rows = 256 rows: a workgroup amortises each K/V byte it
//     copies from L2 over 256 rows.  On this chip the copies cost power rather than time, and the kernel runs
//     against the power limit (a register-only MFMA loop on random data holds 1.85 GHz, not 2.4).
//   * Persistent: 256 workgroups.  Teams of T workgroups (one per 256-row tile of the query rows) walk the same
//     contiguous range of the flattened (column, stage) space, column = (block, KV head, row group) and stage =
//     KT keys (32 at D = 128, 64 at D = 64: 8 KiB of K and of V either way), so a team shares its K/V reads in one XCD's L2 and every team gets the same number of stages: no
//     tail round.  A column that is cut by a range boundary yields several partial results (part index = piece
//     index inside the column); the workgroup that finishes a column marks the unused parts empty.
//   * Ring of 8 stages (K and V, 16 KiB together) in 128 KiB of dynamic LDS, filled by direct HBM->LDS copies that
//     are issued from inline asm and waited for with counted s_waitcnt vmcnt: two to four stages are in flight while
//     two are consumed.  The wavefronts meet once in two steps (in every step, with seven stages ahead instead of six, before: where the shared block
//     has 8 CUs per XCD and the clock is high, 1024 x 40 heads, 16K keys 764 -> 748 us; 1024 x 8/1, 16K keys 81.5 -> 80.7; calls at the power limit equal).
//   * Software pipeline over stages, written out by gen_prefix_wide_step.py: in one step the scores of stage j+2 are
//     produced, the weights of stage j+1 are taken and the P*V product of stage j runs; fragments are loaded
//     from LDS four MFMAs before their use; the vector-ALU work is spread evenly over the gaps between the MFMAs.  At D = 64 a
//     stage has two 32-key score tiles: the same 16 MFMAs per step with twice the softmax work between them.
//   * No search for the row maximum: weights are taken against the maximum of the piece's first stage, and their sum, which is needed
//     anyway and is there a step before their product, says whether a stage has to be taken again against its own (add_sum).
//     Before, with exponentials and product of a stage in one step and the maximum of every stage: 73 instead of 59 vector-ALU instructions per
//     16 MFMAs (D = 64: 147 / 116).  The kernel runs at the board's power limit, so what counts is the energy of what it issues: 1024 x 40 heads,
//     16K keys 310.8 -> 302.2 us with its merge, 512 x 64/8, 4K keys 74.9 -> 73.7, D = 64, 1024 x 40, 4K keys 63.2 -> 61.6; in the
//     combined launch 256 x 64/8, four queries, 4K keys 179 -> 174, 1024 x 8/1, 16K keys 83.0 -> 81.6, 1024 x 40, 16K keys 480 -> 474.
#include <algorithm>
#include <numeric>
#include <type_traits>

#include "hg_internal.h"
#include "prefix_common.h"

// the copy helper names m0 as clobbered on purpose (it writes it)
#pragma clang diagnostic ignored "-Winline-asm"

namespace hg {

namespace {

constexpr int D = HG_WIDE_D;
constexpr int KT = D == 128 ? 32 : 64;  // keys per stage: 8 KiB of K and 8 KiB of V at either head dimension
constexpr int KB = KT / 32;             // 32-key score tiles per stage
constexpr int NS = 8;                   // ring slots
constexpr int NW = 8;                   // wavefronts per workgroup
constexpr int KS = D / 16;              // MFMA k-steps of the score product
constexpr int DB = D / 32;              // 32-row blocks of O^T
constexpr int NKF = 4, NVF = 4;         // K and V fragment registers a wavefront holds (half a stage's worth each)
constexpr int CPR = D / 8;              // 16-byte chunks per K/V row
constexpr int RPI = 64 / CPR;           // rows one wavefront copies per direct-to-LDS instruction
constexpr int ROWB = D * 2;             // bytes per row
constexpr int STB = KT * ROWB;          // bytes per stage and tensor
constexpr int VRING = NS * STB;         // byte offset of the V ring
constexpr int LDS_RING_BYTES = 2 * NS * STB;        // 128 KiB
constexpr int kStageBytes = 32 * 32 * 4;              // staging area of one wavefront for its results: 32 columns of its 32 rows, fp32
constexpr int LDS_BYTES = LDS_RING_BYTES + NW * kStageBytes;   // 160 KiB, all of a CU's LDS
constexpr int AHEAD = NS - 2;           // stages that the copies run ahead of the steps
constexpr int INFLIGHT = AHEAD - 4;     // stages that may still be in flight at a barrier (one before every second step)
// Largest sum of a lane's weights of one stage that is left as it is.  bf16 weights are the more exact the closer the largest is to 1: with scores of
// 4 nats' deviation, 4096 keys, error of O 1.49e-3 at 65536, 8.2e-4 at 256 (8.2e-4 with a search that let maxima grow by 2^8); of 1 nat's
// 1.61e-3 either way, in the same time: hardly a stage is taken again.  At 64, 256 x 64/8 heads, four queries, 4K keys 169.7 -> 170.7 us.
constexpr float kMostWeight = 256.f;
constexpr float kRoom = 16.f;           // log2 units, see add_sum
static_assert(KT == NW * RPI, "one copy instruction per wavefront, stage and tensor");
static_assert(kPrefixRowsWide == 32 * NW, "one 32-row query block per wavefront");

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// XOR swizzle of the 16-byte chunks of LDS row `row` (applied on the global side of the copies).  256-byte rows: K
// chunk ^ row % 16 makes the 16 rows of a ds_read_b128 pass distinct, V chunk ^ 4 (row % 4) separates the 4 rows of a
// transposing read.  128-byte rows are half a bank period, so consecutive rows already differ: K chunk ^ (row / 2) % 8,
// V chunk ^ 4 ((row / 2) % 2).
__device__ __forceinline__ int kswz(int row) { return D == 128 ? row % 16 : (row >> 1) & 7; }
__device__ __forceinline__ int vswz(int row) { return D == 128 ? 4 * (row % 4) : 4 * ((row >> 1) & 1); }

// The scores of one stage as this lane holds them: one 32-key tile at D = 128, two at D = 64.
#if HG_WIDE_D == 128
typedef floatx16 STile;
#else
struct STile { floatx16 a, b; };
#endif

__device__ __forceinline__ void mfma_first(floatx16& S, const uintx4& a, const bf16x8& b) {
    floatx16 z;
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = 0.f;
    S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), b, z, 0, 0, 0);
}
__device__ __forceinline__ void mfma_acc(floatx16& S, const uintx4& a, const bf16x8& b) {
    S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), b, S, 0, 0, 0);
}
__device__ __forceinline__ void mfma_acc(floatx16& O, const shortx8& a, const uintx4& b) {
    O = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), O, 0, 0, 0);
}
// Two floats to a packed bf16 pair (RNE).
__device__ __forceinline__ unsigned pack_bf16_pair(float lo, float hi) {
    floatx2 f = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}
extern __shared__ __attribute__((aligned(1024))) unsigned char wide_smem[];

// Phase time stamps of a -DHG_TRACE build (a measurement aid, compiled out otherwise): thread 0 of every workgroup
// stores the 100 MHz real-time counter at kernel entry (slot 0) and exit (slot 15) and, for its first three pieces
// p, at 1 + 4p + {0 piece entry, 1 first scores done, 2 main loop done, 3 results stored}; slots 16 + p hold the
// shader-clock cycles of piece p's main loop; slots 19 .. 22 split the boundary between pieces 0 and 1 (next piece
// looked up, its Q requested, Q landed, barrier passed); slots 13, 14 and 23 hold the number of stages of pieces 0, 1
// and 2 (a count, not a time); slots 24 .. 27 split the start of the kernel (first piece looked up, copy cursor set,
// two stages' copies issued, Q requested); slot 28 holds the id of the XCD the workgroup ran on.  hg_debug_read_wide_trace copies the table to the host.
#ifdef HG_TRACE
constexpr int kTraceSlots = 32;
__device__ unsigned long long hg_wide_trace[256 * kTraceSlots];
#define HG_T(slot) do { if (threadIdx.x == 0) hg_wide_trace[blockIdx.x * kTraceSlots + (slot)] = __builtin_amdgcn_s_memrealtime(); } while (0)
#define HG_TP(piece, k) do { if ((piece) < 3) HG_T(1 + 4 * (piece) + (k)); } while (0)
#define HG_TN(piece, n) do { if (threadIdx.x == 0 && (piece) < 3) hg_wide_trace[blockIdx.x * kTraceSlots + ((piece) == 2 ? 23 : 13 + (piece))] = (unsigned long long)(n); } while (0)
#define HG_TC_BEGIN() const unsigned long long hg_tc0 = __builtin_amdgcn_s_memtime()
#define HG_TC_END(piece) do { if (threadIdx.x == 0 && (piece) < 3) hg_wide_trace[blockIdx.x * kTraceSlots + 16 + (piece)] = __builtin_amdgcn_s_memtime() - hg_tc0; } while (0)
#else
#define HG_T(slot) do { } while (0)
#define HG_TP(piece, k) do { } while (0)
#define HG_TN(piece, n) do { } while (0)
#define HG_TC_BEGIN() do { } while (0)
#define HG_TC_END(piece) do { } while (0)
#endif

}  // namespace

// A piece of work: 256-row tile row0/256 of the query rows [seq0*rps, seq0*rps + nrows) of KV head kvh against keys
// [ks, ke) of the level's K/V rows, result to part sp.  Everything here is uniform over the workgroup.
struct WidePiece {
    int seq0, nrows, row0, kvh, sp;
    int ks, ke, kwin;    // kwin = max(ke - 32, 0): first row of the last full window of the range
    int nst, nfull;      // stages with at least one key (0: nothing to multiply), stages with KT keys
    int last_in_col;     // the piece ends its column: the parts above sp are marked empty
    int has_rows;        // row0 < nrows
};

// What one workgroup of the persistent kernel does with one level: the first 8 * wide.slots workgroups of the launch call
// this.  `ka` points at the level's arguments in the kernarg segment (without the tables at its end unless they are used).
typedef const __attribute__((address_space(4))) PrefixArgs* wide_args_ptr;
__device__ __forceinline__ unsigned div_by(unsigned n, const __attribute__((address_space(4))) Divider& d) { return Divider{d.mul, d.shift}.of(n); }
__device__ __forceinline__ void wide_role(const wide_args_ptr ka) {
    HG_T(0);
#ifdef HG_TRACE
    if (threadIdx.x == 0) hg_wide_trace[blockIdx.x * kTraceSlots + 28] = __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15u;   // XCC_ID
#endif
    if (ka->lv.seq_off) {
        UncoveredArgs u;
        u.lv.kv_off = ka->lv.kv_off; u.lv.seq_off = ka->lv.seq_off;
        u.lv.n_blocks = ka->lv.n_blocks; u.lv.max_rows = ka->lv.max_rows; u.lv.max_seqs = ka->lv.max_seqs;
        u.lv.K = ka->lv.K; u.lv.V = ka->lv.V;
        u.B = ka->B; u.Hq = ka->Hq; u.nq = ka->nq;
        u.out.O = ka->out.O; u.out.LSE = ka->out.LSE; u.out.bf16 = ka->out.bf16;
        u.out.part_stride_O = ka->out.part_stride_O; u.out.part_stride_L = ka->out.part_stride_L;
        mark_uncovered(u, D, ka->wide.nparts, blockIdx.x, 8 * ka->wide.slots);
    }
    unsigned char* const smem = wide_smem;
    const auto& p = ka->wide;
    const int pid = blockIdx.x;
    const int xcd = pid & 7, cu_slot = pid >> 3;         // workgroups whose ids are equal modulo 8 run on one XCD (which one varies by launch)
    const int team_local = (int)div_by((unsigned)cu_slot, p.by_T), member = cu_slot - team_local * p.T;
    if (team_local >= p.tpx) return;
    const int team = xcd * p.tpx + team_local;

    // ---- this team's range [f0, f1) of the flattened (column, stage) space; sp0 = part index of its first piece ----
    // (Divisions, here, in the look-up of a piece and in the lanes' row numbers, are multiplications by numbers from the host: on this
    // chip one by a run-time divisor takes some 30 instructions that wait for each other, one of 64 bits a loop.  With the order of the sequences
    // in combined_impl.h: 256 x 64/8 heads, 4K keys, four queries 185.4 -> 184.5 us, 512 x 64/8, 4K keys 135.0 -> 134.2; eleven drawn combined calls 1.008 in the mean.)
    int f0, f1, sp0;
    if (!wide_team_range(p, team, f0, f1, sp0)) return;

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 63, lq = l & 31, hl = l >> 5;
    const unsigned rstride_b = (unsigned)ka->Hkv * D * 2u;

    // block offsets are read through the constant address space: nothing writes them while the kernel runs, and the
    // loads then stay on the scalar unit (a vector load would make the compiler wait for vmcnt(0) and drain the ring)
    typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

    // Everything that happens once per piece reads the kernel's arguments again from the kernarg segment (through a
    // pointer the compiler cannot see through) instead of keeping them in scalar registers across the pipeline
    // steps: the steps need those registers themselves, and what does not fit is parked in vector-register lanes.
    typedef wide_args_ptr kargs_ptr;
    auto kargs = [&]() -> kargs_ptr {
        kargs_ptr k = ka;
        asm volatile("" : "+s"(k));
        return k;
    };

    // piece at flattened position f = (column c, stage k0) with part index sp; returns its length in stages
    auto load_piece = [&](kargs_ptr k, int f, int c, int k0, int sp, WidePiece& q) -> int {
        const int n_c = k->wide.n_c, rowgroups = k->wide.rowgroups, Hkv = k->Hkv;
        const int len = min(n_c - k0, f1 - f);
        const int head = (int)div_by((unsigned)c, k->wide.by_rowgroups), rg = c - head * rowgroups;
        const int g = (int)div_by((unsigned)head, k->by_heads), kvh = head - g * Hkv;
        int seq0 = 0, seq1 = k->B, kv0 = 0, kv1 = k->lv.max_rows;
        const const_i32_ptr seq_off_c = (const_i32_ptr)(uintptr_t)k->lv.seq_off;
        if (seq_off_c) {
            const const_i32_ptr kv_off_c = (const_i32_ptr)(uintptr_t)k->lv.kv_off;
            seq0 = seq_off_c[g];
            seq1 = min(seq_off_c[g + 1], seq0 + k->lv.max_seqs);
            kv0 = kv_off_c[g];
            kv1 = min(kv_off_c[g + 1], kv0 + k->lv.max_rows);
        }
        q.seq0 = seq0;
        q.nrows = (seq1 - seq0) * (k->nq * k->G);
        q.row0 = (rg * k->wide.T + member) * kPrefixRowsWide;
        q.kvh = kvh;
        q.sp = sp;
        q.ks = kv0 + k0 * KT;
        q.ke = min(q.ks + len * KT, kv1);
        q.kwin = max(q.ke - KT, 0);
        q.has_rows = q.row0 < q.nrows;
        const int n = q.ke - q.ks;
        q.nst = (q.has_rows && n > 0) ? (n + KT - 1) / KT : 0;
        q.nfull = n > 0 ? n / KT : 0;
        q.last_in_col = (k0 + len == n_c);
        return len;
    };

    // ---- HBM -> LDS copies -----------------------------------------------------------------------------------------
    // The ring is one stream of stages across all of this workgroup's pieces: global stage g lives in slot g % NS, and
    // the copy side (the cursor below) stays AHEAD stages ahead of the compute side, also across a piece boundary, so
    // that a piece after the first finds its first stages in LDS already.  Stage t of a piece holds keys
    // [k0c, k0c + 32) with k0c = min(ks + 32 t, kwin): a stage that is partial or past the range re-reads the last 32
    // rows of the range, so every stage is copied by the same uniform instruction (wavefront w copies rows 4w .. 4w+3,
    // 1 KiB); row i of a stage is a key of that stage iff ks + 32 t <= k0c + i < ke.  The XOR swizzle of the 16-byte
    // chunks is applied on the global side.  The copies are issued from inline asm so that the compiler's wait-count
    // pass does not see them: it would otherwise force vmcnt(0) before every LDS read that follows a copy.
    const int srow = w * RPI + l / CPR;     // row of the stage this lane copies
    const int sch = l % CPR;
    const unsigned ldsw = (unsigned)(uintptr_t)HG_LDS(smem) + (unsigned)w * (RPI * ROWB);
    struct Cursor {
        const unsigned char* Kg;     // the piece's KV head in the level's K / V tensors
        const unsigned char* Vg;
        int ks, kwin, t, left;       // t: next stage of the piece to copy; left: stages of the piece not yet copied
        unsigned voffK, voffV;       // this lane's byte offset inside a stage (row, swizzled chunk)
        int valid;
    } cur{};
    int cf = f0;                     // position of the piece after the cursor's
    int cc = (int)div_by((unsigned)f0, p.by_n_c), ck0 = f0 - cc * p.n_c;
    auto cursor_set = [&](kargs_ptr k, const WidePiece& q) {      // points the cursor at the first stage of piece q (q.nst > 0)
        // (everything but the lane offsets is uniform; saying so keeps it in scalar registers, where the copy
        // instructions take their base address from)
        auto uniform_ptr = [](const uint16_t* ptr) {
            const uint64_t v = reinterpret_cast<uint64_t>(ptr);
            const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
            return reinterpret_cast<const unsigned char*>(((uint64_t)hi << 32) | lo);
        };
        cur.Kg = uniform_ptr(k->lv.K + (int64_t)q.kvh * D);
        cur.Vg = uniform_ptr(k->lv.V + (int64_t)q.kvh * D);
        cur.ks = __builtin_amdgcn_readfirstlane(q.ks);
        cur.kwin = __builtin_amdgcn_readfirstlane(q.kwin);
        cur.t = 0;
        cur.left = __builtin_amdgcn_readfirstlane((q.nst + NS - 1) & ~(NS - 1));     // the stream pads every piece to whole groups of NS stages
        const int row = min(srow, q.ke - 1 - q.kwin);    // binds only when the range ends before row KT of the tensor
        cur.voffK = (unsigned)row * rstride_b + (unsigned)((sch ^ kswz(srow)) * 16);
        cur.voffV = (unsigned)row * rstride_b + (unsigned)((sch ^ vswz(srow)) * 16);
        cur.valid = 1;
    };
    auto cursor_next_piece = [&](kargs_ptr k) {          // moves the cursor to the next piece that has stages, if there is one
        while (cf < f1) {
            WidePiece q;
            const int len = load_piece(k, cf, cc, ck0, 0, q);
            cf += len;
            ++cc;
            ck0 = 0;
            if (q.nst > 0) {
                cursor_set(k, q);
                return;
            }
        }
    };
    auto copy16 = [&](const unsigned char* sbase, unsigned voff, unsigned lds_dst) {
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_dst) : "memory", "m0");
    };
    // after a stage has been issued: one stage further; past the end of its last piece the cursor stays where it is
    // and keeps re-reading that piece's last window (stages nobody consumes)
    auto cursor_advance = [&]() {
        ++cur.t;
        if (--cur.left == 0) cursor_next_piece(kargs());
    };
    auto cursor_step = [&]() {      // inside a group of NS steps, which is entered only with NS stages left in the cursor's piece
        ++cur.t;
        --cur.left;
    };
    auto issue_stage = [&](int slot) {
        const int64_t off = (int64_t)min(cur.ks + cur.t * KT, cur.kwin) * rstride_b;
        const unsigned dst = ldsw + (unsigned)slot * STB;
        copy16(cur.Kg + off, cur.voffK, dst);
        copy16(cur.Vg + off, cur.voffV, dst + VRING);
        cursor_advance();
    };

    // ---- LDS fragment reads (addresses relative to the slot) ---------------------------------------------------
    // K operand for fragment f = (32-key tile f / KS, k-step q = f % KS): row lq of the tile, chunk 2q+hl (rows 32 apart
    // share their swizzle).  V^T operand for d-block db and 16-key group tt:
    // within each 16-lane group lane i addresses key (i/4) of the 4 keys being transposed and columns
    // 4*(i%4) .. +3; group (l/16)&1 selects the lower/upper 16 columns, hl the key quad.
    unsigned kaddr[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) kaddr[s] = (unsigned)(lq * ROWB + (((2 * s + hl) ^ kswz(lq)) * 16));
    unsigned vaddr[DB];
    {
        const int i16 = l & 15, g1 = (l >> 4) & 1;
        const int keyq = 4 * hl + (i16 >> 2);
        const int fv = vswz(keyq);      // (rows 8 and 16 apart share their swizzle)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int chunk = 4 * db + 2 * g1 + ((i16 & 3) >> 1);
            vaddr[db] = (unsigned)(VRING + keyq * ROWB + ((chunk ^ fv) * 16) + (i16 & 1) * 8);
        }
    }
    auto lds_k = [&](int slot, int f) -> uintx4 {
        return *reinterpret_cast<const uintx4*>(smem + slot * STB + (f / KS) * 32 * ROWB + kaddr[f % KS]);
    };
    auto lds_v = [&](int slot, int tt, int db) -> shortx8 {
        const unsigned char* vp = smem + slot * STB + vaddr[db] + tt * 16 * ROWB;
        const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp));
        const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp + 8 * ROWB));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };

    // ---- per-lane view of a piece: this lane's query row and where its result goes ------------------------------------
    struct RowCtx { bool rv; int64_t qidx; };
    // a sequence contributes nq * G rows per KV head: (query t, head g) at t*G + g
    auto row_index = [&](kargs_ptr k, const WidePiece& q, int r) -> int64_t {     // (b*nq + t)*Hq + h of row r of the block
        const int G = k->G, nq = k->nq;
        const int b = (int)div_by((unsigned)r, k->by_seq), in_seq = r - b * (nq * G), t = (int)div_by((unsigned)in_seq, k->by_group);
        return ((int64_t)(q.seq0 + b) * nq + t) * k->Hq + q.kvh * G + (in_seq - t * G);
    };
    auto row_ctx = [&](kargs_ptr k, const WidePiece& q) -> RowCtx {
        const int r = q.row0 + w * 32 + lq;     // this lane's query row inside the block
        RowCtx rc;
        rc.rv = r < q.nrows;
        rc.qidx = row_index(k, q, rc.rv ? r : 0);
        return rc;
    };
    // Q operand (registers, whole piece).  The KS loads are issued from inline asm, like the copies, and waited for
    // with a counted s_waitcnt: the compiler would answer a load it can see with vmcnt(0) before the first product,
    // which waits for every copy in flight and every result store of the piece before.  Until that wait the registers
    // are only named, never read: the compiler takes them for loaded when the asm statement ends.  Lanes past the
    // block's last row read row 0 of the block (their results are never stored).
    uintx4 qraw[KS];
    auto load_q = [&](kargs_ptr k, const RowCtx& rc) {
        const uint16_t* qp = k->Q + rc.qidx * D + 8 * hl;
#if HG_WIDE_D == 64
        static_assert(KS == 4, "load_q names four registers");
        asm volatile(
            "global_load_dwordx4 %0, %4, off\n\t"
            "global_load_dwordx4 %1, %4, off offset:32\n\t"
            "global_load_dwordx4 %2, %4, off offset:64\n\t"
            "global_load_dwordx4 %3, %4, off offset:96"
            : "=&v"(qraw[0]), "=&v"(qraw[1]), "=&v"(qraw[2]), "=&v"(qraw[3])
            : "v"(qp)
            : "memory");
#else
        static_assert(KS == 8, "load_q names eight registers");
        asm volatile(
            "global_load_dwordx4 %0, %8, off\n\t"
            "global_load_dwordx4 %1, %8, off offset:32\n\t"
            "global_load_dwordx4 %2, %8, off offset:64\n\t"
            "global_load_dwordx4 %3, %8, off offset:96\n\t"
            "global_load_dwordx4 %4, %8, off offset:128\n\t"
            "global_load_dwordx4 %5, %8, off offset:160\n\t"
            "global_load_dwordx4 %6, %8, off offset:192\n\t"
            "global_load_dwordx4 %7, %8, off offset:224"
            : "=&v"(qraw[0]), "=&v"(qraw[1]), "=&v"(qraw[2]), "=&v"(qraw[3]), "=&v"(qraw[4]), "=&v"(qraw[5]), "=&v"(qraw[6]),
              "=&v"(qraw[7])
            : "v"(qp)
            : "memory");
#endif
    };
    // Memory operations of a wavefront complete in the order they were issued.  Waiting until at most `younger`
    // operations are outstanding, where `younger` operations were issued after the Q loads, therefore waits for Q and
    // for every copy issued before it, and for nothing issued after it.
    constexpr int kStoresPerPiece = D / 8 + 1;     // result stores of a wavefront whose 32 rows all exist: 16 of O, 1 of LSE
    enum { kQFirst = 0, kQAfterStores = 1, kQDrain = 2 };
    auto wait_q = [&](int kind) {
        constexpr int kFirst = (AHEAD - 2) * 2;       // kernel start: two stages, Q, then AHEAD-2 stages more, which may stay in flight
        if (kind == kQFirst) __builtin_amdgcn_s_waitcnt(0x0F70 | (kFirst & 15) | ((kFirst >> 4) << 14));
        else if (kind == kQAfterStores) __builtin_amdgcn_s_waitcnt(0x0F70 | (kStoresPerPiece & 15) | ((kStoresPerPiece >> 4) << 14));
        else __builtin_amdgcn_s_waitcnt(0x0F70);
    };
    auto mark_rest_empty = [&](kargs_ptr k, const WidePiece& q) {
        // last piece of a column: the remaining parts of these rows hold no keys
        const int r = q.row0 + tid;
        if (tid < kPrefixRowsWide && r < q.nrows) {
            const int64_t qidx = row_index(k, q, r);
            for (int i = q.sp + 1; i < k->wide.nparts; ++i) k->out.LSE[i * k->out.part_stride_L + qidx] = -INFINITY;
        }
    };
    auto store_empty = [&](kargs_ptr k, const WidePiece& q, const RowCtx& rc) {    // a piece without keys: O = 0, LSE = -inf
        if (rc.rv) {
            float* const Of = static_cast<float*>(k->out.O) + q.sp * k->out.part_stride_O + rc.qidx * D;
            uint16_t* const Ob = static_cast<uint16_t*>(k->out.O) + q.sp * k->out.part_stride_O + rc.qidx * D;
#pragma unroll
            for (int i = 0; i < D / 8; ++i) {
                const int d = 8 * i + 4 * hl;
                if (k->out.bf16) *reinterpret_cast<uint2*>(Ob + d) = make_uint2(0u, 0u);
                else *reinterpret_cast<float4*>(Of + d) = make_float4(0.f, 0.f, 0.f, 0.f);
            }
            if (hl == 0) k->out.LSE[q.sp * k->out.part_stride_L + rc.qidx] = -INFINITY;
        }
    };

    // ---- compute-side piece iterator: skips pieces with nothing to multiply (after writing what they owe) -------------
    int pf = f0;
    int pcol = cc, pk0 = ck0, psp = sp0;
    WidePiece pc{};
    auto next_piece = [&](kargs_ptr k) -> bool {     // false: the range is exhausted
        while (pf < f1) {
            const int len = load_piece(k, pf, pcol, pk0, psp, pc);
            pf += len;
            ++pcol;
            pk0 = 0;
            psp = 0;
            if (pc.nst > 0) return true;
            if (pc.has_rows) {
                store_empty(k, pc, row_ctx(k, pc));
                if (pc.last_in_col) mark_rest_empty(k, pc);
            }
        }
        return false;
    };

    // ---- online softmax state ------------------------------------------------------------------------------------
    floatx16 Oacc[DB];
    float lsum;                 // this lane's share of the row sum (of the unrounded exponentials)
    float mc;                   // what the exponents are taken against, log2 units
    const float c2 = ka->scale * kLog2e;
    // the weights of one stage (its scores against the present maximum), packed for the second product; returns this lane's sum of them
    auto weights = [&](const STile& S, uintx4 (&p)[KT / 16]) -> float {
        float sa = 0.f, sb = 0.f;
#pragma unroll
        for (int h = 0; h < KT / 16; ++h)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = 8 * (h & 1) + 2 * i;
#if HG_WIDE_D == 128
                const float x0 = S[e], x1 = S[e + 1];
#else
                const float x0 = h < 2 ? S.a[e] : S.b[e], x1 = h < 2 ? S.a[e + 1] : S.b[e + 1];
#endif
                const float ea = __builtin_amdgcn_exp2f(fmaf(x0, c2, -mc)), eb = __builtin_amdgcn_exp2f(fmaf(x1, c2, -mc));
                p[h][i] = pack_bf16_pair(ea, eb);
                sa += ea;
                sb += eb;
            }
        return sa + sb;
    };
    auto tile_max = [&](const STile& S) -> float {
#if HG_WIDE_D == 128
        float t = fmaxf(S[0], S[1]);
#pragma unroll
        for (int i = 2; i < 16; i += 2) t = fmaxf(fmaxf(t, S[i]), S[i + 1]);
#else
        float t = fmaxf(S.a[0], S.b[0]);
#pragma unroll
        for (int i = 1; i < 16; ++i) t = fmaxf(fmaxf(t, S.a[i]), S.b[i]);
#endif
        return half_max(t);
    };

    constexpr int kStepOutstanding = INFLIGHT * 2;
    constexpr int kStepWait = 0x0F70 | (kStepOutstanding & 15) | ((kStepOutstanding >> 4) << 14);

    // ---- results of a finished piece (its accumulators are still in registers when this runs) -------------------------
    // A lane holds half of one row of O^T (64 values, every other group of four columns), and consecutive lanes hold
    // rows that lie Hq * D elements apart in memory: stored from there, every lane of a store instruction would touch
    // a cache line of its own, and the store unit takes the lanes' addresses one at a time.  The rows therefore go
    // through a 4 KiB staging area per wavefront (in the 32 KiB of LDS behind the ring, which no copy touches), 32
    // columns of all 32 rows at a time, and leave it as whole 128-byte lines, eight rows per store instruction.
    // 16-byte chunk c of staged row r lives at chunk c ^ (r % 8): writes and reads are free of bank conflicts.
    // A wavefront whose 32 rows all exist issues exactly kStoresPerPiece store instructions; one with fewer rows, fewer.
    // fp32 results are parts, for the merge to read once, and written past the caches (those that hg_prefix_attn leaves in the caller's memory too: they are for hg_merge).  What
    // that saves is not the launch's traffic, which stays the same (2048 x 40 heads, two levels 3.10 -> 3.09 GB); why it is faster has not been measured.  Median us with the merge's
    // loads the same way: 2048 x 40 heads, two levels 549.5 -> 524.7, D = 64, 4K keys 181.9 -> 173.8, 8-bit rows, 4K keys 225.8 -> 217.1, 256 x 40, 2K keys 122.1 -> 120.8,
    // 1024 x 40, 16K keys 475.7 -> 470.7; this store alone, the same inputs every time, six drawn calls of one query row 2.9 % in the mean, 373.7 -> 353.3 at most.  hg_prefix_attn to fp32, 1024 x 40, 512 keys 23.9 ->
    // 22.7, with hg_suffix_attn and hg_merge 257.6 -> 257.5, D = 64, 1K keys 147.6 -> 146.8, 512 x 64/8, 1K keys 78.2 -> 77.9, 2048 x 40, 1K keys 529.6 -> 530.8.
    // Beside the tiles of several query rows they are stored the ordinary way, which is as good in the calls that the choice was made on, not in all: past the caches, inputs
    // changing from call to call, 512 x 64/8 heads, 4K keys 133.9 -> 134.4, 256 x 64/8, four queries 170.5 -> 170.8, 128 x 32/8, paged 41.2 -> 41.2; 16 drawn calls 0.8 % faster in the
    // mean, from 58.5 -> 59.7 (1416 x 4/4, four queries, 1850 keys, codes) and 37.4 -> 37.8 (272 x 64/8, 164 keys) over 81.5 -> 81.0 to 129.6 -> 124.8 (318 x 64/8, 379 keys, codes) and 572 -> 553.
    auto store_part = [](float* p, const float4& v) {
#ifdef HG_COMBINED_TILES
        *reinterpret_cast<float4*>(p) = v;
#else
        __builtin_nontemporal_store(__builtin_bit_cast(uintx4, v), reinterpret_cast<uintx4*>(p));
#endif
    };
    auto store_piece = [&](kargs_ptr k, const WidePiece& q, bool q_idle) {
        if (q_idle) return;
        // (the lane id is taken through an empty asm statement: the compiler would otherwise compute the staging
        // addresses once, before the first piece, and keep them in registers the pipeline steps need)
        int l = tid & 63;
        asm volatile("" : "+v"(l));
        const int lq = l & 31, hl = l >> 5;
        const RowCtx qrc = row_ctx(k, q);
        const float ltot = half_sum(lsum);
        const float inv = 1.0f / ltot;
        const int my_row = qrc.rv ? (int)qrc.qidx : -1;            // query row index (b*nq + t)*Hq + h, below 2^31 / D
        if (qrc.rv && hl == 0) k->out.LSE[q.sp * k->out.part_stride_L + qrc.qidx] = (mc + __log2f(ltot)) * kLn2;
        const int nvalid = min(q.nrows - (q.row0 + w * 32), 32);   // rows of this wavefront that exist (>= 1)
        unsigned char* const stg = smem + LDS_RING_BYTES + w * kStageBytes;
        float* const Of = static_cast<float*>(k->out.O) + q.sp * k->out.part_stride_O;
        uint16_t* const Ob = static_cast<uint16_t*>(k->out.O) + q.sp * k->out.part_stride_O;
        const bool out_bf16 = k->out.bf16 != 0;
        int row_of[4];       // the query row this lane forwards in the kk-th store of a pass: row 8 kk + l / 8 of the wavefront
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) row_of[kk] = __shfl(my_row, 8 * kk + (l >> 3));
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4)
                *reinterpret_cast<float4*>(stg + lq * 128 + (((2 * q4 + hl) ^ (lq & 7)) * 16)) =
                    make_float4(Oacc[db][4 * q4] * inv, Oacc[db][4 * q4 + 1] * inv, Oacc[db][4 * q4 + 2] * inv, Oacc[db][4 * q4 + 3] * inv);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                if (8 * kk < nvalid) {                             // (uniform: the instruction is issued or not as a whole)
                    const int r = 8 * kk + (l >> 3), c = l & 7;
                    const float4 v = *reinterpret_cast<const float4*>(stg + r * 128 + ((c ^ (r & 7)) * 16));
                    const int row = row_of[kk];
                    if (row >= 0) {
                        if (out_bf16)
                            *reinterpret_cast<uint2*>(Ob + (int64_t)row * D + 32 * db + 4 * c) = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
                        else
                            store_part(Of + (int64_t)row * D + 32 * db + 4 * c, v);
                    }
                }
            }
        }
    };

    // ---- the pieces of this workgroup, one per iteration ------------------------------------------------------------------
    {
        const kargs_ptr k = kargs();       // one look at the arguments for everything up to the first copies
        if (!next_piece(k)) return;
        HG_T(24);
        // the copy cursor starts at the piece the compute side has just found (the pieces before it have no stages); its
        // first two stages are requested before Q, which the first products need together with them
        cf = pf;
        cc = pcol;
        ck0 = pk0;
        cursor_set(k, pc);
        HG_T(25);
        issue_stage(0);
        issue_stage(1);
        HG_T(26);
        load_q(k, row_ctx(k, pc));
        HG_T(27);
    }
    int qkind = kQFirst;
#pragma unroll
    for (int s = 2; s < AHEAD; ++s) issue_stage(s);
    int piece_no = 0;

    for (;;) {
        HG_TP(piece_no, 0);
        HG_TN(piece_no, pc.nst);
        // ---- piece prologue ---------------------------------------------------------------------------------------------
        // Q and the stream's next stages have landed, for everyone
        wait_q(qkind);
        if (piece_no == 1) HG_T(21);
        __builtin_amdgcn_s_barrier();
        if (piece_no == 1) HG_T(22);
        bf16x8 qf[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            asm volatile("" : "+v"(qraw[s]));      // the products below stay behind the wait above
            qf[s] = __builtin_bit_cast(bf16x8, qraw[s]);
        }
        const int ks = pc.ks, ke = pc.ke, kwin = pc.kwin;
        const bool idle = pc.row0 + w * 32 >= pc.nrows;    // blocks of <= 224 rows: this wavefront has nothing to multiply

        // rows of a partial stage that are nobody's keys may hold anything: their scores are masked, and their V rows
        // are cleared in LDS before the second product reads them (0 * NaN would be NaN).  The partial stage is the
        // piece's last; it is cleared at the top of the step before the one that first reads its V rows.
        const int zstep = pc.nst > pc.nfull ? pc.nst - 2 : -8;
        auto clear_partial_v = [&]() {
            const int t = pc.nst - 1;
            const int key0 = ks + t * KT, k0c = min(key0, kwin);
            const int lo = key0 - k0c, hi = ke - k0c;
            const int row = tid / CPR;          // 64 * NW threads = KT rows x CPR chunks
            if (row < lo || row >= hi)
                *reinterpret_cast<uint4*>(smem + VRING + (t & (NS - 1)) * STB + row * ROWB + (tid % CPR) * 16) = make_uint4(0, 0, 0, 0);
            __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): the writes are done
            __builtin_amdgcn_s_barrier();
        };
        if (zstep == -1) clear_partial_v();

        auto mask_stage = [&](STile& S, int tstage) {
            const int key0 = ks + tstage * KT;
            const int k0c = min(key0, kwin);
            const int lo = key0 - k0c - 4 * hl, hi = ke - k0c - 4 * hl;   // row i of this lane is 8*(i/4) + i%4 + 4*hl (+ 32 in the second tile)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int ri = 8 * (i >> 2) + (i & 3);
#if HG_WIDE_D == 128
                if (ri < lo || ri >= hi) S[i] = -INFINITY;
#else
                if (ri < lo || ri >= hi) S.a[i] = -INFINITY;
                if (ri + 32 < lo || ri + 32 >= hi) S.b[i] = -INFINITY;
#endif
            }
        };

#pragma unroll
        for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int k = 0; k < 16; ++k) Oacc[i][k] = 0.f;
        lsum = 0.f;
        mc = 0.f;

        uintx4 kf[NKF];
        shortx8 vf[NVF];
        STile SA, SB;
        uintx4 PA[KT / 16], PB[KT / 16];
        // the scores of the stage in `slot` of the ring, all fragments loaded here
        auto scores = [&](int slot, STile& S) {
            uintx4 k0[KB * KS];
#pragma unroll
            for (int q = 0; q < KB * KS; ++q) k0[q] = lds_k(slot, q);
#if HG_WIDE_D == 128
            mfma_first(S, k0[0], qf[0]);
#pragma unroll
            for (int q = 1; q < KS; ++q) mfma_acc(S, k0[q], qf[q]);
            __builtin_amdgcn_sched_barrier(0);      // (what follows does not fit the registers beside the fragments)
#else
            mfma_first(S.a, k0[0], qf[0]);
            mfma_first(S.b, k0[KS], qf[0]);
#pragma unroll
            for (int q = 1; q < KS; ++q) {
                mfma_acc(S.a, k0[q], qf[q]);
                mfma_acc(S.b, k0[KS + q], qf[q]);
            }
#endif
        };
        if (!idle) {
            // what the first step expects (a piece starts at slot 0): weights of stage 0, scores of stage 1, V fragments of the first half of stage 0
            scores(0, SB);
            scores(1, SA);
            if (pc.nfull == 0) mask_stage(SB, 0);
            // (a finite number for a row with nothing but -inf, so that -inf has weight 0 and any finite score one that is infinite, which add_sum sees;
            // clamped behind the product: with c2 > 1 the product of a finite number may be -inf)
            mc = fmaxf(tile_max(SB) * c2, -3.4028234e38f);
            lsum = weights(SB, PA);
#pragma unroll
            for (int i = 0; i < NVF; ++i) vf[i] = lds_v(0, i / DB, i % DB);
        }
        HG_TP(piece_no, 1);
        HG_TC_BEGIN();

        // One pipeline step.  On entry: pb = weights of stage j, Scur = scores of stage j+1, vf = the first half of stage j's V
        // fragments.  On exit the same with j+1: pn = weights of stage j+1, Snext = scores of stage j+2 (of whatever follows in
        // the ring when there are no such stages in the piece).  The step's copy goes into the slot
        // whose stage was consumed two steps before.  slot = (g0 + j) % NS.  Returns this lane's sum of the new weights.
        // `plain` steps (the groups of NS) take the weights of full stages only and never reach the end of a piece: no mask, no
        // clearing, no look-up of a piece, no branch that would let the compiler move work out of its gap.
        // The body of a step is one basic block (a branch inside it lets the compiler move work out of its gap): the
        // steps outside the groups of NS apply the mask to every stage whose weights they take (it changes nothing on a full one; a
        // stage behind the piece's last gets weights of zero).
        auto step_body = [&](int j, int slot, const uintx4 (&pb)[KT / 16], uintx4 (&pn)[KT / 16], STile& Scur, STile& Snext, auto masked) -> float {
            constexpr bool kMasked = decltype(masked)::value;
            float ssum;
            const int slot1 = (slot + 1) & (NS - 1), slot2 = (slot + 2) & (NS - 1);
#if HG_WIDE_D == 128
#include "prefix_wide_step.inc"
#else
#include "prefix_wide_step_d64.inc"
#endif
            return ssum;
        };
        // The weights just taken are not too large for what they are summed with, or infinite, as long as their sum (at least as large as the
        // largest of them) is small.  Otherwise they are taken again against the larger maximum, from the scores, whose registers the next step
        // is the first to write; nothing has been multiplied with them yet.  (Exact: the stale maximum cancels in O/l and LSE.)
        // Where most rows have moved, scores rise along the keys, and the maxima are set kRoom too large so that the next few stages are not taken again
        // as well (a whole number: the largest weight stays a power of two, which bf16 holds exactly).  Single rows' outliers get no room: their largest
        // weights would be rounded for the rest of the piece (error of O at 4 nats 1.19e-3 -> 1.5e-3 with room at every second one).
        // us with a search for every stage's maximum / with the scores computed once more here and no room / now: 256 x 64/8 heads, four queries, 4K
        // keys, scores of 1, 2, 4 nats' deviation 176.5 / 170.7 / 170.5, 178.3 / 174.6 / 173.7, 185.8 / 193.2 / 185.0, of 1 nat and rising by 40 and 400 nats 182.3 / 192.0 / 172.6,
        // 197.1 / 251.6 / 188.4; D = 64, 1024 x 40, 4K keys, 1 and 4 nats 179.5 / 171.1 / 170.7, 180.6 / 175.8 / 174.6, rising by 40 and 400 180.4 / 177.2 / 171.1, 181.0 / 228.5 / 172.7.
        // The block alone, 1024 x 40, 16K keys, 1 and 4 nats 310.8 / 298.4 / 302.2, 327.1 / 333.8 / 324.6, D = 64, 4K keys 62.4 / 59.6 / 59.3, 64.7 / 69.6 / 67.2.
        // Error of O the same at 1 to 4 nats and up to 2^3 a stage; where scores rise by 2^9 a stage 1.1e-3 -> 1.6e-3 (1.65e-3 without a rise).
        auto add_sum = [&](const STile& S, float ssum, uintx4 (&pn)[KT / 16]) {
            if (__builtin_expect(__any(!(ssum <= kMostWeight)), 0)) {
                float top = tile_max(S) * c2;
                if (__builtin_popcountll(__ballot(top > mc + 2.0f)) >= 48) top += kRoom;
                const float mc_new = fmaxf(mc, top);
                const float alpha = __builtin_amdgcn_exp2f(mc - mc_new);
                mc = mc_new;
                lsum *= alpha;
#pragma unroll
                for (int i = 0; i < DB; ++i) {
                    Oacc[i] *= alpha;
                    __builtin_amdgcn_sched_barrier(0);      // (block by block: all in flight at once do not fit the registers)
                }
                ssum = weights(S, pn);
            }
            lsum += ssum;
        };
        // kind 1: a step of a group of NS that is not the piece's last; 0: a step of the last group.
        auto step = [&](int j, int slot, auto even, auto kind) {
            constexpr bool kPlain = decltype(kind)::value == 1, kEven = decltype(even)::value;
            STile &Scur = kEven ? SA : SB, &Snext = kEven ? SB : SA;
            uintx4 (&pb)[KT / 16] = kEven ? PA : PB, (&pn)[KT / 16] = kEven ? PB : PA;
            typedef std::integral_constant<bool, !kPlain> Masked;
            if constexpr (kEven) {                        // (a piece starts at slot 0: even steps are those at even slots)
                __builtin_amdgcn_s_waitcnt(kStepWait);    // own copies of the next three stages have landed
                __builtin_amdgcn_s_barrier();             // ... everyone's, and everyone has finished the step before
            } else {
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!kPlain && j == zstep) clear_partial_v();
            add_sum(Scur, step_body(j, slot, pb, pn, Scur, Snext, Masked{}), pn);
            if (kPlain) cursor_step();
            else cursor_advance();
        };

        if (idle) {
            // nothing to multiply (blocks of <= 224 rows): this wavefront keeps its share of the copies going and meets
            // the others at every barrier
            for (int j = 0; j < pc.nst; ++j) {
                if (j % 2 == 0) {
                    __builtin_amdgcn_s_waitcnt(kStepWait);
                    __builtin_amdgcn_s_barrier();
                }
                if (j == zstep) clear_partial_v();
                issue_stage((j + AHEAD) & (NS - 1));
            }
        } else {
            // Whole groups of NS steps at compile-time slots (a piece starts at slot 0: the stream pads every piece to
            // a multiple of NS stages) as long as every stage they score is a full one, which leaves at least the
            // piece's last group to the steps below; the copy cursor reaches the end of its piece only in a piece's
            // last group, so these steps never have to look a piece up.
            int j = 0;
            for (; j + NS < pc.nfull; j += NS) {
#pragma unroll
                for (int u = 0; u < NS; u += 2) {
                    step(j + u, u, std::true_type{}, std::integral_constant<int, 1>{});
                    step(j + u + 1, u + 1, std::false_type{}, std::integral_constant<int, 1>{});
                }
            }
            // The rest of the piece (1 .. NS + 1 steps: its last group, and one step more when the stage after a complete
            // group is the partial one), at compile-time slots too: a chain that ends at the first step beyond the
            // piece.  These steps mask every stage they score (it changes nothing on a full one) and may move the copy
            // cursor to the next piece.
            const int rest = pc.nst - j;
            auto tail = [&](auto self, auto uc) -> void {
                constexpr int u = decltype(uc)::value;
                if constexpr (u < NS + 1) {
                    if (u < rest) {
                        step(j + u, u & (NS - 1), std::integral_constant<bool, u % 2 == 0>{}, std::integral_constant<int, 0>{});
                        self(self, std::integral_constant<int, u + 1>{});
                    }
                }
            };
            tail(tail, std::integral_constant<int, 0>{});
        }
        // ... and its padding: steps that only keep the stream going (the slots of the padding stay unused)
        for (int j = pc.nst; j & (NS - 1); ++j) {
            if (j % 2 == 0) __builtin_amdgcn_s_barrier();
            issue_stage((j + AHEAD) & (NS - 1));
        }
        HG_TC_END(piece_no);
        HG_TP(piece_no, 2);

        // ---- the next piece's Q is requested before this piece's results are stored ---------------------------------------
        // (what is stored after the request is counted, see store_piece; the marks of empty parts and the results of
        // pieces without keys go out before it)
        const WidePiece done = pc;
        const kargs_ptr k = kargs();       // one look at the arguments for the whole boundary
        if (done.last_in_col) mark_rest_empty(k, done);
        const bool more = next_piece(k);
        if (piece_no == 0) HG_T(19);
        if (more) load_q(k, row_ctx(k, pc));
        if (piece_no == 0) HG_T(20);
        // a wavefront whose 32 rows all exist issues exactly kStoresPerPiece stores below; any other drains everything
        qkind = (!idle && done.row0 + w * 32 + 32 <= done.nrows) ? kQAfterStores : kQDrain;
        store_piece(k, done, idle);
        HG_TP(piece_no, 3);
        ++piece_no;
        if (!more) break;
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);   // the copies still in flight land before the ring is released
    HG_T(15);
}

#ifdef HG_WIDE_KERNEL
__global__ __launch_bounds__(64 * NW, 1) void HG_WIDE_KERNEL(PrefixArgs) { wide_role((wide_args_ptr)__builtin_amdgcn_kernarg_segment_ptr()); }

#if defined(HG_TRACE) && HG_WIDE_D == 128
}  // namespace hg
// Copies the phase time stamps of the most recent prefix_kernel_wide launches to `out` (HOST, 256 * 32 values) after
// synchronising the device; present only in a -DHG_TRACE build.
extern "C" int hg_debug_read_wide_trace(unsigned long long* out) {
    if (hipDeviceSynchronize() != hipSuccess) return HG_ERR_HIP;
    return hipMemcpyFromSymbol(out, HIP_SYMBOL(hg::hg_wide_trace), sizeof(unsigned long long) * 256 * hg::kTraceSlots) == hipSuccess
               ? HG_OK : HG_ERR_HIP;
}
namespace hg {
#endif

#if HG_WIDE_D == 128
// Work partition of the persistent kernel for a level (host side).  Returns false when the level does not fit
// (more than max_parts partial results per row would be needed).  table: the plan may use mode 2.  A stage is 32 keys at D = 128 and 64 keys at D = 64.
bool plan_prefix_wide(const LevelDev& lv, int Hkv, int G, int D, int max_parts, int slots_per_xcd, WidePlan* out,
                      bool table) {
    if (D != 128 && D != 64) return false;
    const int KT = D == 128 ? 32 : 64;
    // G here is the number of query rows per sequence and KV head (queries per sequence x heads per group)
    WidePlan p{};
    const long long rows = (long long)lv.max_seqs * G;
    const int mtiles = (int)((rows + kPrefixRowsWide - 1) / kPrefixRowsWide);
    if (mtiles < 1 || lv.max_rows < 1) return false;
    if (slots_per_xcd < 1 || slots_per_xcd > 32) return false;
    p.slots = slots_per_xcd;
    // Row groups: the workgroups of a team run on one XCD, so T <= slots, and slots % T CUs stay idle.  More, smaller
    // groups can fill them at the price of reading the block once more per group.  Both in units of the products' time on
    // all of the slots (a K/V row of 4 D bytes costs as much as multiplying it with 190 query rows: 4 D / 6 TB/s against
    // 4 D / 1.14 PFLOP/s per row): 4096 query rows on 24 CUs per XCD run as two teams of 8 tiles on 24 of them, not 16 on 16.
    // That leaves out what a group costs where blocks are short or teams many: the column ends that fall inside a team's
    // range, and the partial results, which every piece writes for its rows and the merge reads again (0.08 stages per piece
    // and tile).  Where the price in stages with these finds a choice better by a twentieth, it is taken: 563 x 16/2
    // heads, 395 keys, 4 queries 56.2 -> 41.9 us (18 tiles on 28 CUs instead of 9 three times), 614 x 64/8, 1892 keys 86.1 -> 73.4,
    // 1024 x 8/1, 16K keys 86.5 -> 83.0 (8 columns of 4 tiles, cut evenly, instead of 5 of 7).  22 of 1500 drawn calls change, by
    // 1.09 in the mean, none slower by more than 2 %; without the margin 58, some of them 7 % slower.  On fewer than 16 CUs per XCD the suffix
    // decides, and these terms only disturb (267 x 64/8, 253 keys, 8-bit rows: 50.9 -> 53.7).
    {
        const int r0 = (mtiles + p.slots - 1) / p.slots;
        const int r_end = mtiles >= 8 ? std::min(mtiles, 8 * r0) : r0;      // (few tiles: nothing to gain)
        const auto tiles_of = [&](int r) { return (mtiles + r - 1) / r; };
        const double row = (double)mtiles * kPrefixRowsWide, even = (double)lv.n_blocks * Hkv * mtiles * ((lv.max_rows + KT - 1) / KT) / (8.0 * p.slots);
        // the price of r groups in stages; `idle`: their products' time.  (The divisors last: they decide only where the rest is not too much.)
        const auto stages = [&](int r, int T, double idle, double limit) {
            const long long teams = 8 * (p.slots / T), cols = (long long)lv.n_blocks * Hkv * r;
            const double piece = (D == 128 ? 0.08 : 0.02) * T, most = (double)std::max(teams, cols), read = (idle + 100.0 * r / row) * even;
            if (read + piece * most >= limit) return limit;
            const double cuts = (double)(cols - std::gcd((int)(cols % teams), (int)teams));
            return read + kWideBoundaryCost * cuts / teams + piece * (most + std::min(cuts, (double)teams));
        };
        const bool priced = p.slots >= 16;
        int r1 = r0, r2 = r0;
        double best1 = 1e300, best2 = 1e300, price1 = 1e300;      // (price1: of r1, by stages)
        for (int r = r0; r <= r_end; ++r) {
            const int T = tiles_of(r);
            if ((r - 1) * T >= mtiles) continue;      // the last group would be empty
            const double idle = (double)r * T / mtiles * p.slots / (p.slots / T * T), cost = idle + 190.0 * r / row;
            const bool better = cost < 0.97 * best1;
            if (better) { r1 = r; best1 = cost; }
            if (!priced || r_end == r0) continue;
            const double price = stages(r, T, idle, better ? 1e300 : 0.97 * best2);
            if (better) price1 = price;
            if (price < 0.97 * best2) { r2 = r; best2 = price; }
        }
        p.rowgroups = best2 < 0.95 * price1 ? r2 : r1;
        p.T = tiles_of(p.rowgroups);
    }
    p.tpx = p.slots / p.T;
    p.n_c = (lv.max_rows + KT - 1) / KT;
    const long long ncols = (long long)lv.n_blocks * Hkv * p.rowgroups;
    if (ncols >= (1LL << 20) || ncols * p.n_c >= (1LL << 31)) return false;    // the kernel walks the space with 32-bit indices
    p.ncols = (int)ncols;
    const long long total = ncols * p.n_c;
    const int nteams = 8 * p.tpx;
    long long q = (total + nteams - 1) / nteams;
    if (q >= 64) q = (q + NS - 1) / NS * NS;                // long ranges: whole groups of NS stages
    if (q < 1) q = 1;
    auto parts_needed = [&](long long quota) {     // most pieces any column is cut into
        int np = 1;
        for (long long c = 0; c < ncols; ++c) {
            const long long lo = c * p.n_c, hi = lo + p.n_c - 1;
            const int n = (int)(hi / quota - lo / quota) + 1;
            if (n > np) np = n;
        }
        return np;
    };
    if (max_parts < 1) return false;
    int np = parts_needed(q);
    if (np > max_parts) {
        // Longer ranges per team (some teams then stay idle) until the parts fit, as long as the teams still cover
        // the whole space; otherwise whole columns per team, which always fits in one part.
        const long long qa = max_parts >= 2 ? (p.n_c + max_parts - 2) / (max_parts - 1) : 0;
        if (qa >= 1 && qa * nteams >= total && parts_needed(qa) <= max_parts) {
            q = qa;
            np = parts_needed(qa);
        } else {
            q = (ncols + nteams - 1) / nteams * p.n_c;
            np = 1;
        }
    }
    p.mode = 0;
    // Equal ranges give every team the same number of stages but may cut a team's range at a column boundary, and a
    // workgroup pays a fixed price per piece (its Q tile, the first products outside the pipeline, the result stores:
    // about kPieceCost stages).  When pieces are short that price decides: then ranges aligned to the columns win.
    // cost = most (stages + kPieceCost * pieces) any team has.
    {
        constexpr long long kPieceCost = 4;
        long long pieces0 = 1;
        for (int t = 0; t < nteams; ++t) {                   // exact: columns touched by [t q, (t+1) q)
            const long long lo = (long long)t * q, hi = std::min<long long>(lo + q, total);
            if (lo >= hi) break;
            pieces0 = std::max<long long>(pieces0, (hi - 1) / p.n_c - lo / p.n_c + 1);
        }
        const long long cost0 = q + kPieceCost * pieces0;
        long long cost1, np1;
        if (ncols <= nteams) {
            const long long nt_min = nteams / ncols;                      // teams of the column with the fewest
            np1 = (nteams + ncols - 1) / ncols;
            cost1 = (p.n_c + nt_min - 1) / nt_min + kPieceCost;
        } else {
            const long long cols = (ncols + nteams - 1) / nteams;
            np1 = 1;
            cost1 = cols * (p.n_c + kPieceCost);
        }
        if (cost1 < cost0 && np1 <= max_parts && np1 <= p.n_c) {   // (a column has at least one stage per team)
            p.mode = 1;
            np = (int)np1;
        }
    }
    if (q >= (1LL << 30)) return false;
    p.quota = (int)q;
    p.nparts = np;
    // Equal ranges, some with a column boundary inside and some without: the teams with a boundary finish later by what
    // a second piece costs.  Ranges of equal cost instead (cost = stages + kWideBoundaryCost per boundary inside): the
    // smallest cost C for which the teams, each taking the longest range that costs at most C, cover the space.
    if (table && p.mode == 0 && nteams <= kWideMaxTeams) {
        const long long nc = p.n_c, kappa = kWideBoundaryCost;
        auto end_of = [&](long long a, long long C) {      // the largest b <= total with (b - a) + kappa * boundaries inside (a, b) <= C
            long long best = a + 1;
            const long long m0 = a / nc * nc;
            for (long long k = 0; C - kappa * k >= 1; ++k) {
                const long long mk = k == 0 ? a : m0 + k * nc;            // k boundaries lie inside when b > m_k
                const long long b = std::min({m0 + (k + 1) * nc, a + C - kappa * k, total});
                if (b > mk) best = std::max(best, b);
                if (mk >= total) break;
            }
            return std::min(best, total);
        };
        auto covers = [&](long long C) {
            long long a = 0;
            for (int t = 0; t < nteams && a < total; ++t) a = end_of(a, C);
            return a >= total;
        };
        int with = 0, without = 0;
        long long cost0 = 0;
        for (int t = 0; t < nteams; ++t) {
            const long long lo = (long long)t * q, hi = std::min<long long>(lo + q, total);
            if (lo >= hi) break;
            const long long inner = (hi - 1) / nc - lo / nc;
            (inner ? with : without) += 1;
            cost0 = std::max(cost0, hi - lo + kappa * inner);
        }
        if (with && without) {
            long long lo = (total + nteams - 1) / nteams, hi = cost0;       // covers(hi) holds: equal ranges cost at most cost0
            while (lo < hi) {
                const long long mid = (lo + hi) / 2;
                if (covers(mid)) hi = mid;
                else lo = mid + 1;
            }
            if (hi < cost0) {
                WidePlan w = p;
                long long a = 0;
                int col = -1, in_col = 0, np2 = 1;
                for (int t = 0; t <= nteams; ++t) w.starts[t] = (int)total;
                for (int t = 0; t < nteams && a < total; ++t) {
                    const long long b = end_of(a, hi);
                    w.starts[t] = (int)a;
                    for (long long c = a / nc; c <= (b - 1) / nc; ++c) {       // the pieces of this team, column by column
                        if ((int)c != col) { col = (int)c; in_col = 0; }
                        if (c == a / nc) w.first_part[t] = in_col;
                        ++in_col;
                        np2 = std::max(np2, in_col);
                    }
                    a = b;
                }
                if (np2 <= max_parts) {
                    w.mode = 2;
                    w.nparts = np2;
                    w.quota = (int)hi;      // (the cost bound; not a length in this mode)
                    p = w;
                }
            }
        }
    }
    p.by_T = divider((unsigned)p.T);
    p.by_n_c = divider((unsigned)p.n_c);
    p.by_rowgroups = divider((unsigned)p.rowgroups);
    p.by_quota = divider((unsigned)p.quota);
    p.by_cols = divider((unsigned)p.ncols);
    p.by_teams = divider((unsigned)nteams);
    const int cut = std::max(1, nteams / p.ncols);
    p.by_cut[0] = divider((unsigned)cut);
    p.by_cut[1] = divider((unsigned)cut + 1);
    *out = p;
    return true;
}

#endif

#if HG_WIDE_D == 128
hipError_t launch_prefix_wide(const PrefixArgs& a, int D, hipStream_t s) {
    if (D == 64) return launch_prefix_wide_d64(a, s);
#else
hipError_t launch_prefix_wide_d64(const PrefixArgs& a, hipStream_t s) {
#endif
    static bool attr_set[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64 && !attr_set[dev]) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&HG_WIDE_KERNEL), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    HG_WIDE_KERNEL<<<8 * a.wide.slots, 64 * NW, LDS_BYTES, s>>>(a);
    return hipGetLastError();
}
#endif   // HG_WIDE_KERNEL

}  // namespace hg
