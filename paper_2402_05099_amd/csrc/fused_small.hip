// The whole of Hydragen's attention (App. B's top-level routine: attention over every shared block, attention over each
// sequence's own suffix, and the merge of the parts by their log-sum-exp, Eq. 5) in ONE launch, for calls with so
// little work that several launches and a pass over partial results cost more than the arithmetic.
//
// A column is 32 or 16 consecutive rows (TR) of the query rows of one KV head (Sec. 3.2's inter-sequence batching: row
// r = sequence * nq * G + query * G + head-in-group).  Its keys are a list of segments: the block of every shared
// level that covers its sequences (all rows of the tile attend to it, or those of the covered sequences when a
// block boundary falls inside the tile), then the suffix of each of the tile's sequences (only that sequence's rows
// attend).  Softmax over the union of all segments is one online softmax: a row that does not attend to a segment has
// its scores masked.  The decomposition of Eq. 5 appears twice: the 32-key stages of the list are dealt out to the
// wavefronts of the column's workgroups one by one (or in runs, see below), each with its own running maximum, sum and accumulator; the partial
// results of a workgroup's wavefronts meet in LDS and are combined with the weights exp(LSE_i - max LSE).
//
// 16 rows: products of 16 x 16 instead of 32 x 32, half the exponentials per lane, and fewer sequences whose suffixes a column
// has to walk; twice as many columns, which a small call has CUs for (the rule is in plan_fused).
//
// A column is worked on by `splits` workgroups (as many as leave the chip full: a small call has few columns, and one
// workgroup per column would leave most CUs idle; calls that must not share the workspace keep one, see plan_fused).  With more than one, each writes its combined result to the
// workspace and counts itself in at the column's arrival counter; the last to arrive combines the column's
// results, and the counter wraps to zero for the next call.  No workgroup ever waits for another.
// That meeting is a chain too: results stored and acknowledged 0.4 - 0.9 us, the counter 0.5, the results read 1.1 and up.  The reading
// lane asks for all results of its row at once, 16 bytes at a time (before: 8 at a time, repeated when there were fewer, 8 bytes each: 2.8
// and 3.3 us instead of 1.4 and 1.5 with nine workgroups of 16 rows and four of 32).  76 sequences x 4 heads, 1496 keys (nine
// workgroups per column) 10.9 -> 8.9 us, 32 x 64/8, 4752 keys (four, 32 rows) 21.4 -> 17.5; 26 drawn calls with split columns 1.076.
//
// Workgroups of four wavefronts (NWS), for calls with more columns than CUs: half the LDS, so that two of them share a CU and one's way to its
// first product and its combination, 5 us of a column that has few stages, run beside the other's stages.  Eight / four wavefronts: 683 x 64/8 heads, 549
// keys, four queries 222 / 167 us; 57 x 64/8, 342 + 3 x 297 keys, four queries 21.7 / 15.7.  A column with many stages, or a CU of its
// own, is the faster with eight: 1024 x 8/1, 16K keys 96 / 125.  The rule is in plan_fused.
//
// A wavefront streams its stages through one K slot and one V slot of 8 KiB of its own (HBM -> LDS copies issued from
// inline asm, counted s_waitcnt): the next stage's K rows are requested as soon as this stage's scores are done, its V
// rows after the second product.  With eight wavefronts per workgroup (two per SIMD) that keeps as many bytes in
// flight as four wavefronts with two slots for each, and the second wavefront fills the first one's waits.
// Products, XOR swizzles and lazy rescaling are those of the other kernels (prefix_wide.hip, decode_mfma.hip).
//
// What bounds it: latency.  By time stamps (16 rows, D = 128): arguments 0.4 us after the start, lengths, Q and the first stages' rows 1.7 later (128 KiB
// through the CU's 64 bytes a cycle), the first product 0.4 after them, 1.05 us per shared stage (products, exponentials and the
// 16 KiB of every one of eight wavefronts), 1.45 per suffix stage (masks, another segment each time), 1.2 for the combination
// and output.  What needs no loaded value (LDS addresses, index arithmetic) is therefore done while the first loads are on their way, the
// divisions are multiplications by numbers from the host, the prefix sum of the lengths stays in the vector ALU, and copies whose
// rows need no clamp run without a branch: before, lengths to first product 0.95 us, arguments to first request 0.1 longer;
// 45 x 16/2 heads, 515 keys, ragged up to 150 rows 9.86 -> 8.56 us, 256 x 8/1, 1K keys, 128 rows 12.2 -> 11.4, 40 drawn calls 1.046 in the mean.
// Stages dealt out one by one, 16-row columns and early requests (with one workgroup per column, runs of consecutive stages and 32 rows before): 256 sequences x 8 heads on one KV head, 1024
// shared keys, 128 suffix rows 16.2 -> 12.1 us; 45 x 16 heads on two KV heads, 515 keys, ragged up to 150 rows 13.9 -> 10.0;
// 57 calls of this kind drawn at random 1.19 times as fast in the mean (stages dealt out one by one and the first requested early
// alone: 1.05).
//
// PAGED: the suffix rows are found through a page table; CODES: they are E4M3 codes with one scale per tensor, expanded
// in registers (exactly: every E4M3 value is a bf16 value); the K scale multiplies the scores of those stages, the V
// scale finished sums: a wavefront whose run goes on from shared rows to codes divides its accumulators by it once and
// goes on in units of it, and multiplies them by it at its end (on the weights it would be rounded to bf16 with them:
// one key per sequence, whose weight is 1, came out 1.9e-3 off instead of exact).  Rows that the vector-ALU kernel would
// read with fp32 weights keep that precision (CODES = 2): a weight is taken as the sum of three bf16 values, which hold
// all 24 bits of it, in three products.  Error of O without a shared block 1.0e-7 (vector-ALU kernel 1.3e-7, one bf16 value
// per weight 1.1e-3); 5 x 40 heads, 269 keys, 1..37 codes: 11.0 us (10.3 with one value; separate kernels 19.8).
#include <type_traits>

#include "hg_internal.h"
#include "prefix_common.h"

#pragma clang diagnostic ignored "-Winline-asm"

namespace hg {

namespace {

constexpr int KT = 32;                  // keys per stage
constexpr float TAU = 8.0f;             // lazy-rescale threshold, log2 units

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef int intx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ unsigned pack_pair(float lo, float hi) {
    floatx2 f = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16x2));
}

template <int N>
__device__ __forceinline__ void wait_vm() {
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

extern __shared__ __attribute__((aligned(1024))) unsigned char fs_smem[];

typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;
typedef const __attribute__((address_space(4))) SmallArgs* kargs_ptr;

// One segment of a tile's key list (uniform over the workgroup).
struct Seg {
    const unsigned char* K;   // the segment's tensor at this KV head (bytes; a page pool's first row for paged suffixes)
    const unsigned char* V;
    int ks, ke;               // key rows [ks, ke) of that tensor (of the sequence when the suffix is paged)
    int rlo, rhi;             // rows [rlo, rhi) of the tile attend to it
    int vis_base;             // suffix: query t of the sequence sees rows below vis_base + t; shared block: INT_MAX / 2
    int nst;                  // stages of 32 keys
    int sfx;                  // index of the suffix's sequence among the tile's (-1: shared block)
};

// 8 E4M3 codes to 8 bf16 values (exact)
__device__ __forceinline__ uintx4 expand8(unsigned lo, unsigned hi) {
    uintx4 v;
    v[0] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false));
    v[1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true));
    v[2] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false));
    v[3] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true));
    return v;
}

// elements 8 tt .. 8 tt + 7 of a stage's weights, rounded to bf16
template <class V>
__device__ __forceinline__ uintx4 pack8(const V& p, int tt) {
    return uintx4{pack_pair(p[8 * tt], p[8 * tt + 1]), pack_pair(p[8 * tt + 2], p[8 * tt + 3]),
                  pack_pair(p[8 * tt + 4], p[8 * tt + 5]), pack_pair(p[8 * tt + 6], p[8 * tt + 7])};
}

// Results that another workgroup of the same launch will read: stores and loads at agent scope (the cache policy's bit SC1) go past
// the caches that the XCDs do not share, so that nothing has to be flushed before the arrival is counted.  Buffer
// instructions take 16 bytes at that scope, where an atomic access takes 8.
constexpr int kAgentScope = 16;
struct AgentBuffer {                        // `bytes` (less than 4 GiB) from p on
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ AgentBuffer(float* p, unsigned bytes) : rsrc(__builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000)) {}
    __device__ __forceinline__ void store4(unsigned off, const float4& v) const {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uintx4, v), rsrc, (int)off, 0, kAgentScope);
    }
    __device__ __forceinline__ void store1(unsigned off, float v) const {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rsrc, (int)off, 0, kAgentScope);
    }
    __device__ __forceinline__ float4 load4(unsigned off) const {
        return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)off, 0, kAgentScope));
    }
    __device__ __forceinline__ float load1(unsigned off) const {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)off, 0, kAgentScope));
    }
};

template <int D, int TR, int NWS>
struct SmallGeo {
    static constexpr int KS = D / 16, DB = D / 32;      // 32-row columns: k-steps of the scores, 32-row blocks of O^T
    static constexpr int KS16 = D / 32, DB16 = D / 16;  // 16-row columns: 32-column steps, 16-row blocks
    static constexpr int CPR = D / 8, RPI = 64 / CPR, CPS = KT / RPI, ROWB = D * 2, STB = KT * ROWB;   // bf16 rows
    static constexpr int CPR8 = D / 16, RPI8 = 64 / CPR8, CPS8 = KT / RPI8;                            // E4M3 rows
    static constexpr int OW = TR * D * 4;                // combined result of a wavefront (fp32)
    static constexpr int LDS = NWS * 2 * STB + NWS * TR * 8 + 16;   // rings or results, maxima and sums, the "last" flag
    static_assert(OW <= 2 * STB, "a wavefront's result takes the place of its ring");
    static constexpr int RPW = NWS == 4 ? TR / 4 : TR == 32 || D == 64 ? 4 : 2;         // rows a wavefront finishes (16 rows of D = 64: half of eight wavefronts do)
    static constexpr int LPR = 64 / RPW, CH = D / 4, CPL = CH / LPR;   // lanes of such a row, its 16-byte chunks, chunks per lane
    static_assert(CPL * LPR == CH && TR % RPW == 0 && TR / RPW <= NWS, "");
};

}  // namespace

// CODES: the suffix rows are bf16 (0), E4M3 codes (1), E4M3 codes whose weights keep fp32 precision (2).  TR: rows of a column.
// NWS: wavefronts of a workgroup.
template <int D, bool PAGED, int CODES, int TR, int NWS>
__global__ __launch_bounds__(64 * NWS, 2) void fused_small_kernel(SmallArgs a) {
    constexpr bool FP8 = CODES != 0, NARROW = TR == 16;
    using G_ = SmallGeo<D, TR, NWS>;
    constexpr int KS16 = G_::KS16, DB16 = G_::DB16;
    constexpr int KS = G_::KS, DB = G_::DB, CPR = G_::CPR, RPI = G_::RPI, CPS = G_::CPS, ROWB = G_::ROWB, STB = G_::STB;
    constexpr int CPR8 = G_::CPR8, RPI8 = G_::RPI8, CPS8 = G_::CPS8;
    constexpr int NP = CODES == 2 ? 3 : 1;          // bf16 pieces of a code's weight
    unsigned char* const smem_all = fs_smem;
    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l = tid & 63, lq = l & (TR - 1), hl = l >> 5, lg = l >> 4;     // lq: this lane's row of the column
    unsigned char* const smem = smem_all + w * (2 * STB);      // this wavefront's K slot, then its V slot
    const kargs_ptr k = (kargs_ptr)__builtin_amdgcn_kernarg_segment_ptr();

    // Workgroups whose ids are equal modulo 8 run on one XCD: each XCD takes an eighth of the list (KV head, tile, split), so that
    // the shared rows of a head are read into one L2 or few instead of all, whatever the number of heads.  Numbers of KV heads
    // that neither divide 8 nor are a multiple of it, dealt out over all XCDs before: 64 sequences x 40/10 heads, 8K keys, paged
    // 59.8 -> 33.6 us; 34 x 40/10, 10.5K keys, paged 50.3 -> 28.4; 56 x 24/12, 8574 keys, codes 45.9 -> 30.1.  The others, which had
    // an order of their own to the same end: 1.005 in the mean over 117 calls.
    int kvh, tile, split;
    // (loaded at once with the rest, not behind the way out or where they are first used: the first K rows are requested after one wait for
    // arguments, before after three, the second of them for lines that no cache held.  4 x 4 heads, D = 64, 128 keys 5.5 -> 5.0 us; 119 x 64/8, D = 64, 150
    // keys 5.6 -> 5.1; 256 x 8/1, D = 128, 1K keys, where the rows' way into the CU sets the time, 11.24 -> 11.14; 100 drawn calls 1.016 in the mean.  Keys
    // requested before the queries: D = 64 as fast, D = 128 slower by 2 %, the queries then come behind eight wavefronts' rows.)
    asm volatile("" ::"s"(a.nq), "s"(a.G), "s"(a.B), "s"(a.Q), "s"(a.lengths), "s"(a.offsets), "s"(a.by_seq.mul), "s"(a.by_group.mul), "s"(a.n_levels));
    asm volatile("" ::"s"(a.lv[0].K), "s"(a.lv[0].V), "s"(a.lv[0].seq_off), "s"(a.lv[0].max_rows), "s"(a.Ks), "s"(a.Vs), "s"(a.max_len), "s"(a.dealt), "s"(a.c2));
    if constexpr (PAGED) asm volatile("" ::"s"(a.pg.table), "s"(a.pg.shift), "s"(a.pg.stride), "s"(a.pg.n_pages));
    if (!small_work(blockIdx.x, a.tiles, a.splits, a.Hkv, a.by_head, a.by_split, kvh, tile, split)) return;
    const int col = kvh * a.tiles + tile;
    const int rps = a.nq * a.G;                     // query rows of one sequence for this KV head
    const int R = a.B * rps;
    const int r0 = tile * TR;
    const int b0 = (int)a.by_seq.of((unsigned)r0), b1 = min((int)a.by_seq.of((unsigned)(r0 + TR - 1)), a.B - 1);
    const int r = r0 + lq;                          // this lane's row
    const bool rv = r < R;
    const int rr = rv ? r : r0;
    const int b_lane = (int)a.by_seq.of((unsigned)rr), in_seq = rr - b_lane * rps, t_lane = (int)a.by_group.of((unsigned)in_seq), g_lane = in_seq - t_lane * a.G;
    const int64_t qidx = ((int64_t)b_lane * a.nq + t_lane) * a.Hq + kvh * a.G + g_lane;   // (b*nq + t)*Hq + h

    // ---- Q operand (registers) and the tile's suffix lengths / offsets (lane i: sequence b0 + i), loaded before any copy ----
    int len_v = 0, off_v = 0;
    if (a.lengths != nullptr && b0 + l <= b1) {
        len_v = a.lengths[b0 + l];
        if (!PAGED) off_v = a.offsets[b0 + l];
    }
    constexpr int QN = NARROW ? KS16 : KS;
    bf16x8 qf[QN];
    {
        const uint16_t* qp = a.Q + qidx * D;
#pragma unroll
        for (int s = 0; s < QN; ++s) {
            uint4 v = make_uint4(0, 0, 0, 0);
            if (rv) v = *reinterpret_cast<const uint4*>(qp + 8 * (NARROW ? 4 * s + lg : 2 * s + hl));
            qf[s] = __builtin_bit_cast(bf16x8, v);
        }
    }
    // ---- segment enumeration: shared blocks one by one, suffixes through a prefix sum over the lanes --------------------------
    const unsigned rstride_b = (unsigned)a.Hkv * D * 2u;
    const unsigned rstride_s = (unsigned)a.Hkv * D * (FP8 ? 1u : 2u);     // suffix rows
    struct Walk { int level, block; };              // the next shared block (block -1: not looked up yet)
    auto next_shared = [&](Walk& it, Seg& s) -> bool {        // the next shared block with keys and rows, if there is one
        for (;;) {
            if (it.level >= a.n_levels) return false;
            const int L = it.level;
            const const_i32_ptr seq_off = (const_i32_ptr)(uintptr_t)k->lv[L].seq_off;
            const const_i32_ptr kv_off = (const_i32_ptr)(uintptr_t)k->lv[L].kv_off;
            int sa = 0, sb = a.B, kv0 = 0, kv1 = k->lv[L].max_rows;
            if (seq_off != nullptr) {
                const int nb = k->lv[L].n_blocks;
                if (it.block < 0) {
                    // first block whose sequences end after b0
                    int lo = 0, hi = nb;
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (seq_off[mid + 1] <= b0) lo = mid + 1;
                        else hi = mid;
                    }
                    it.block = lo;
                }
                if (it.block >= nb || seq_off[it.block] > b1) {   // no further block of this level touches the tile
                    ++it.level;
                    it.block = -1;
                    continue;
                }
                sa = seq_off[it.block];
                sb = min(seq_off[it.block + 1], sa + k->lv[L].max_seqs);
                kv0 = kv_off[it.block];
                kv1 = min(kv_off[it.block + 1], kv0 + k->lv[L].max_rows);
                ++it.block;
            } else {
                ++it.level;
                it.block = -1;
            }
            s.K = reinterpret_cast<const unsigned char*>(k->lv[L].K + (int64_t)kvh * D);
            s.V = reinterpret_cast<const unsigned char*>(k->lv[L].V + (int64_t)kvh * D);
            s.ks = kv0;
            s.ke = kv1;
            s.rlo = max(max(sa, b0) * rps - r0, 0);
            s.rhi = min(min(sb, b1 + 1) * rps - r0, TR);
            s.vis_base = 0x3fffffff;
            s.sfx = -1;
            s.nst = (s.ke > s.ks && s.rhi > s.rlo) ? (s.ke - s.ks + KT - 1) / KT : 0;
            if (s.nst > 0) return true;
        }
    };
    // ---- HBM -> LDS copies -----------------------------------------------------------------------------------------------------
    // Stage t of a segment holds rows [k0c, k0c + 32), k0c = min(ks + 32 t, kwin), kwin = max(ke - 32, 0): a partial last
    // stage re-reads the 32 rows that end the range; row i of a stage is a key of it iff ks + 32 t <= k0c + i < ke.
    // Paged suffixes: a stage is 32 aligned logical rows and is never shifted; its two halves lie in one page each.
    // 16-byte chunks are XOR-swizzled on the global side (bf16 rows: K chunk ^ row % 16, V chunk ^ 4 (row % 4) at D = 128, see
    // decode_mfma.hip; codes: rows of 8 or 4 chunks, spread so that the reads below are free of bank conflicts).
    const unsigned ldsb = (unsigned)(uintptr_t)HG_LDS(smem);
    auto kswz = [](int row) { return D == 128 ? row % 16 : (row >> 1) & 7; };
    auto vswz = [](int row) { return D == 128 ? 4 * (row % 4) : 4 * ((row >> 1) & 1); };
    auto kswz8 = [](int row) { return D == 128 ? (row >> 1) & 7 : (row >> 2) & 3; };
    auto vswz8 = [](int row) { return D == 128 ? ((row >> 1) & 1) | (((row >> (NARROW ? 4 : 3)) & 1) << 1) : (row >> 2) & 3; };
    auto scalar_ptr = [&](const unsigned char* vbase) -> const unsigned char* {
        const uint64_t pv = reinterpret_cast<uint64_t>(vbase);
        const uint32_t plo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)pv);
        const uint32_t phi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(pv >> 32));
        return reinterpret_cast<const unsigned char*>(((uint64_t)phi << 32) | (uint64_t)plo);
    };
    auto copy16 = [&](const unsigned char* sbase, unsigned voff, unsigned lds_dst) {
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase), "s"(lds_dst) : "memory", "m0");
    };
    const int lrow = l / CPR, sch = l % CPR, lrow8 = l / CPR8, sch8 = l % CPR8;
    unsigned voffK[CPS], voffV[CPS];                // this lane's byte offset in a bf16 stage (whole stages)
#pragma unroll
    for (int i = 0; i < CPS; ++i) {
        const int srow = i * RPI + lrow;
        voffK[i] = (unsigned)srow * rstride_b + (unsigned)((sch ^ kswz(srow)) * 16);
        voffV[i] = (unsigned)srow * rstride_b + (unsigned)((sch ^ vswz(srow)) * 16);
    }
    unsigned voffK8[FP8 ? CPS8 : 1], voffV8[FP8 ? CPS8 : 1];
    if constexpr (FP8) {
#pragma unroll
        for (int i = 0; i < CPS8; ++i) {
            const int srow = i * RPI8 + lrow8;
            voffK8[i] = (unsigned)srow * rstride_s + (unsigned)((sch8 ^ kswz8(srow)) * 16);
            voffV8[i] = (unsigned)srow * rstride_s + (unsigned)((sch8 ^ vswz8(srow)) * 16);
        }
    }
    auto copies_of = [&](const Seg& s) { return FP8 && s.sfx >= 0 ? CPS8 : CPS; };     // copy instructions per stage and tensor
    // first row of stage t of segment s as it lies in LDS
    auto row0_of = [&](const Seg& s, int t) { return PAGED && s.sfx >= 0 ? t * KT : min(s.ks + t * KT, max(s.ke - KT, 0)); };
    // Paged suffixes: the table's entries for the two halves of stage t of segment s.  They are looked up when the stage becomes the next one and first
    // used behind the scores of the one before, so that the look-up lies under those.  (Looked up where the rows are requested, before: 82 x 64/8 heads, 340 keys,
    // codes 29.5 -> 28.5 us, 298 x 64/8, four queries, 15 x 171 keys, codes 98.3 -> 95.5; 49 drawn paged calls 1.005 in the mean.)
    struct Pages { int p0, p1; };
    auto pages_of = [&](const Seg& s, int t) -> Pages {
        Pages pg{0, 0};
        if (PAGED && s.sfx >= 0) {
            const const_i32_ptr table = (const_i32_ptr)(uintptr_t)a.pg.table + (int64_t)(b0 + s.sfx) * a.pg.stride;
            const int last = a.pg.stride - 1;
            pg.p0 = table[min((t * KT) >> a.pg.shift, last)];
            pg.p1 = table[min((t * KT + KT / 2) >> a.pg.shift, last)];
        }
        return pg;
    };
    auto issue = [&](const Seg& s, int t, const Pages& pg, auto is_v) {      // requests the K (or V) rows of stage t of segment s
        constexpr bool V = decltype(is_v)::value;
        const unsigned dst = (unsigned)__builtin_amdgcn_readfirstlane(ldsb + (V ? (unsigned)STB : 0u));
        const bool codes = FP8 && s.sfx >= 0;
        const unsigned rs = s.sfx >= 0 ? rstride_s : rstride_b;
        const unsigned char* const tensor = V ? s.V : s.K;
        const unsigned char *base0, *base1;         // of rows 0 .. 15 and 16 .. 31 (both relative to row 0)
        int rowclamp = KT - 1;                      // < 31 only when the range ends before row 32 of the tensor
        if (PAGED && s.sfx >= 0) {
            const int shift = a.pg.shift, mask = (1 << shift) - 1, n_pages = a.pg.n_pages;
            const int j0 = t * KT, j1 = j0 + KT / 2;
            const int p0 = min(max(pg.p0, 0), n_pages - 1);
            const int p1 = min(max(pg.p1, 0), n_pages - 1);
            base0 = scalar_ptr(tensor + (((int64_t)p0 << shift) + (j0 & mask)) * rs);
            base1 = scalar_ptr(tensor + (((int64_t)p1 << shift) + (j1 & mask) - KT / 2) * rs);
        } else {
            const int k0c = row0_of(s, t);
            rowclamp = min(s.ke - 1 - k0c, KT - 1);
            base0 = base1 = scalar_ptr(tensor + (int64_t)k0c * rs);
        }
        if (codes) {
            if constexpr (FP8) {
                if (__builtin_expect(rowclamp < KT - 1, 0)) {
#pragma unroll
                    for (int i = 0; i < CPS8; ++i) {
                        const int srow = i * RPI8 + lrow8;
                        copy16(base0, (V ? voffV8[i] : voffK8[i]) - (unsigned)(srow - min(srow, rowclamp)) * rs, dst + i * 1024);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < CPS8; ++i) copy16(i < CPS8 / 2 ? base0 : base1, V ? voffV8[i] : voffK8[i], dst + i * 1024);
                }
            }
        } else if (__builtin_expect(rowclamp < KT - 1, 0)) {
#pragma unroll
            for (int i = 0; i < CPS; ++i) {
                const int srow = i * RPI + lrow;
                copy16(base0, (V ? voffV[i] : voffK[i]) - (unsigned)(srow - min(srow, rowclamp)) * rs, dst + i * 1024);
            }
        } else {
#pragma unroll
            for (int i = 0; i < CPS; ++i) copy16(i < CPS / 2 ? base0 : base1, V ? voffV[i] : voffK[i], dst + i * 1024);
        }
    };
    // wait until at most `younger` copy instructions are outstanding (those of one tensor of one stage, or none)
    auto wait_for = [&](int younger) {
        if (younger == CPS) wait_vm<CPS>();
        else if (FP8 && younger == CPS8) wait_vm<CPS8>();
        else wait_vm<0>();
        asm volatile("" ::: "memory");
    };
    typedef std::integral_constant<bool, false> IsK;
    typedef std::integral_constant<bool, true> IsV;

    // ---- this wavefront's stages.  Dealt out one by one (positions run, run + runs, ... of the list): the stages of the shared blocks
    // come first, so that the first one, where there is one, is found and requested while the lengths are on their way, and every
    // wavefront gets its share of both kinds: with runs of consecutive stages those of suffix stages, which take longer, hold up the rest.
    // In runs where the suffix rows keep the HBM busy (see the rule in plan_fused): some wavefronts then stream them from the start, while
    // others multiply shared rows.
    const int runs = a.splits * NWS, run = split * NWS + w;
    Walk walk{0, -1};
    Seg cs{};
    int ct = 0, base = 0;                           // current stage of segment cs; shared stages before cs
    bool requested = false;
    auto reached = [&]() -> bool {                  // segment cs holds this wavefront's first stage (dealt out); else it is passed over
        if (a.dealt && base + cs.nst > run) return true;
        base += cs.nst;
        return false;
    };
    // (the only block of a first level without a list of blocks, which is most calls' only shared block, from arguments that are there already)
    if (a.n_levels > 0 && a.lv[0].seq_off == nullptr) {
        cs.K = reinterpret_cast<const unsigned char*>(a.lv[0].K + (int64_t)kvh * D);
        cs.V = reinterpret_cast<const unsigned char*>(a.lv[0].V + (int64_t)kvh * D);
        cs.ks = 0;
        cs.ke = a.lv[0].max_rows;
        cs.rlo = 0;
        cs.rhi = min((b1 + 1) * rps - r0, TR);
        cs.vis_base = 0x3fffffff;
        cs.sfx = -1;
        cs.nst = (cs.ke + KT - 1) / KT;
        walk.level = 1;
        requested = reached();
    }
    while (!requested && next_shared(walk, cs)) requested = reached();
    int shared_total = base;
    if (requested) {
        ct = run - base;
        issue(cs, ct, Pages{0, 0}, IsK{});
        Walk rest = walk;
        Seg s{};
        shared_total += cs.nst;
        while (next_shared(rest, s)) shared_total += s.nst;
    }
    shared_total = __builtin_amdgcn_readfirstlane(shared_total);
    // ---- LDS fragment addresses (relative to the slot), as in decode_mfma.hip ---------------------------------------------------
    constexpr int KA = NARROW ? 2 * KS16 : KS, VA = NARROW ? DB16 : DB;
    unsigned kaddr[KA], vaddr[VA], kaddr8[FP8 ? KA : 1], vaddr8[FP8 ? VA : 1];
    if constexpr (NARROW) {
        // K of 16-key group kg, 32-column step q: row 16 kg + lq, columns 32 q + 8 lg .. +7.  V^T of 16 columns: k-slot e of lane
        // group lg stands for key 16 (e / 4) + 4 lg + e % 4
#pragma unroll
        for (int q = 0; q < KS16; ++q)
#pragma unroll
            for (int kg = 0; kg < 2; ++kg) {
                const int row = 16 * kg + lq;
                kaddr[2 * q + kg] = (unsigned)(row * ROWB + (((4 * q + lg) ^ kswz(row)) * 16));
                if constexpr (FP8) kaddr8[2 * q + kg] = (unsigned)(row * D + (((2 * q + (lg >> 1)) ^ kswz8(row)) * 16) + 8 * (lg & 1));
            }
        const int vrow = 4 * lg + (lq >> 2), q4 = lq & 3;
        const int j = lq >> 1, row8 = 16 * (j >> 2) + 4 * lg + (j & 3);
#pragma unroll
        for (int db = 0; db < DB16; ++db) {
            vaddr[db] = (unsigned)(STB + vrow * ROWB + (((2 * db + (q4 >> 1)) ^ vswz(vrow)) * 16) + (q4 & 1) * 8);
            if constexpr (FP8) vaddr8[db] = (unsigned)(STB + row8 * D + ((db ^ vswz8(row8)) * 16) + 8 * (lq & 1));
        }
    } else {
#pragma unroll
        for (int s = 0; s < KS; ++s) kaddr[s] = (unsigned)(lq * ROWB + (((2 * s + hl) ^ kswz(lq)) * 16));
        const int i16 = l & 15, g1 = (l >> 4) & 1;
        const int keyq = 4 * hl + (i16 >> 2);
        const int fv = vswz(keyq);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
            const int chunk = 4 * db + 2 * g1 + ((i16 & 3) >> 1);
            vaddr[db] = (unsigned)(STB + keyq * ROWB + ((chunk ^ fv) * 16) + (i16 & 1) * 8);
        }
        if constexpr (FP8) {
            // codes: the 8 of K row lq, columns 16 s + 8 hl .. +7; V^T through ds_read_b64_tr_b8 (lane s of a group of 16 points
            // at the key of k-slot s / 2 and columns 8 (s % 2) .. +7 of its 16-column block)
#pragma unroll
            for (int s = 0; s < KS; ++s) kaddr8[s] = (unsigned)(lq * D + ((s ^ kswz8(lq)) * 16) + 8 * hl);
            const int j = i16 >> 1, pp = i16 & 1;
            const int row = 8 * (j >> 2) + 4 * hl + (j & 3);        // + 16 tt: the same swizzle
#pragma unroll
            for (int db = 0; db < DB; ++db) vaddr8[db] = (unsigned)(STB + row * D + (((2 * db + g1) ^ vswz8(row)) * 16) + 8 * pp);
        }
    }
    // (computed while lengths, queries and first rows are on their way)
#pragma unroll
    for (int i = 0; i < KA; ++i) asm volatile("" : "+v"(kaddr[i]));
#pragma unroll
    for (int i = 0; i < VA; ++i) asm volatile("" : "+v"(vaddr[i]));

    // (the loads above are the only ones the compiler sees; it waits for them, and with them for the first copies, here)
    asm volatile("" : "+v"(len_v), "+v"(off_v));
#pragma unroll
    for (int s = 0; s < QN; ++s) asm volatile("" : "+v"(qf[s]));
    // (the first V rows only now: the K rows of eight wavefronts, which the first products wait for, come through the CU's load path by themselves, and
    // the V rows while those are multiplied.  256 x 8/1 heads, 1K keys 11.35 -> 10.95 us, 45 x 16/2, 515 keys 8.60 -> 8.42, 29 drawn calls 1.004.)
    if (requested) issue(cs, ct, Pages{0, 0}, IsV{});
    len_v = max(min(len_v, a.max_len), 0);
    const int nst_v = (len_v + KT - 1) / KT;        // stages of the suffix of sequence b0 + l
    // ... of the suffixes of b0 .. b0 + l: a prefix sum over the TR lanes that can hold a sequence (within rows of 16 lanes, then the first row's total
    // into the second)
    int incl_v = nst_v;
    incl_v += __builtin_amdgcn_update_dpp(0, incl_v, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8
    incl_v += __builtin_amdgcn_update_dpp(0, incl_v, 0x112, 0xf, 0xf, false);
    incl_v += __builtin_amdgcn_update_dpp(0, incl_v, 0x114, 0xf, 0xf, false);
    incl_v += __builtin_amdgcn_update_dpp(0, incl_v, 0x118, 0xf, 0xf, false);
    if constexpr (TR == 32) incl_v += __builtin_amdgcn_update_dpp(0, incl_v, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
    constexpr uint64_t kSeqLanes = TR == 32 ? 0xffffffffull : 0xffffull;
    auto load_suffix = [&](int i, Seg& s) {         // the suffix of sequence b0 + i (which has rows)
        const int cnt = __builtin_amdgcn_readlane(len_v, i), off = PAGED ? 0 : __builtin_amdgcn_readlane(off_v, i);
        s.K = reinterpret_cast<const unsigned char*>(k->Ks) + (int64_t)kvh * D * (FP8 ? 1 : 2);
        s.V = reinterpret_cast<const unsigned char*>(k->Vs) + (int64_t)kvh * D * (FP8 ? 1 : 2);
        s.ks = off;
        s.ke = off + cnt;
        s.rlo = max((b0 + i) * rps - r0, 0);
        s.rhi = min((b0 + i + 1) * rps - r0, TR);
        s.vis_base = off + cnt - (a.nq - 1);        // query t sees rows below off + cnt - (nq-1-t)
        s.nst = (cnt + KT - 1) / KT;
        s.sfx = i;
    };
    const int total = shared_total + __builtin_amdgcn_readlane(incl_v, TR - 1);
    auto seek = [&](int pos, Seg& s, int& t) {      // the stage at position pos < total, behind the current one
        if (pos < shared_total) {
            t = pos - base;
            while (t >= s.nst) {
                base += s.nst;
                t -= s.nst;
                next_shared(walk, s);
            }
            return;
        }
        const int p = pos - shared_total;
        const int i = __builtin_popcountll(__ballot(incl_v <= p) & kSeqLanes);      // the first sequence whose stages reach past p
        load_suffix(i, s);
        t = p - (__builtin_amdgcn_readlane(incl_v, i) - s.nst);
    };
    const int step = a.dealt ? runs : 1;
    // (runs: the host gives a column one workgroup then; NWS * total stays below 2^31, a block's rows being fewer than 2^24)
    const int first = a.dealt ? run : (int)((unsigned)(run * total) / NWS), end = a.dealt ? total : (int)((unsigned)((run + 1) * total) / NWS);
    if (!requested && first < end) {
        if (!a.dealt && first < shared_total) {     // (the walk has counted the shared stages: once more from the beginning)
            walk = Walk{0, -1};
            base = 0;
            next_shared(walk, cs);
        }
        seek(first, cs, ct);
        const Pages pg = pages_of(cs, ct);
        issue(cs, ct, pg, IsK{});
        issue(cs, ct, pg, IsV{});
    }

    // ---- this wavefront's share of the softmax ------------------------------------------------------------------------------
    const float c2 = a.c2, tau_raw = a.tau_raw;
    // scores and accumulators: one 32 x 32 product per block of O^T, or two 16-key groups and 16 x 16 products
    typedef float floatx4 __attribute__((ext_vector_type(4)));
    using OBlock = std::conditional_t<NARROW, floatx4, floatx16>;
    constexpr int OE = NARROW ? 4 : 16, NE = NARROW ? 8 : 16;      // values of a block, scores of a stage, per lane
    OBlock Oacc[VA];
#pragma unroll
    for (int i = 0; i < VA; ++i)
#pragma unroll
        for (int j = 0; j < OE; ++j) Oacc[i][j] = 0.f;
    float m_used = -INFINITY;   // raw-score maximum the exponentials are taken against (-inf: no key seen yet)
    float mc = 0.f;             // m_used * c2, 0 while no key has been seen
    float lsum = 0.f;           // this lane's share of the row sum (unrounded exponentials)
    bool code_units = false;    // the accumulators hold sums of codes, to be multiplied by the V scale

    for (int pos = first; pos < end; pos += step) {
        const bool more = pos + step < end;
        Seg ns = cs;
        int nt = ct;
        if (more) {
            if (ct + step < cs.nst) nt = ct + step;
            else seek(pos + step, ns, nt);
        }
        const Pages npg = more ? pages_of(ns, nt) : Pages{0, 0};
        const bool codes = FP8 && cs.sfx >= 0;
        wait_for(copies_of(cs));                    // this stage's K rows are here, its V rows may still be on their way
        // S^T = K Q^T.  Element i: stage row 8 (i / 4) + i % 4 + 4 hl; 16-row columns: 16 (i / 4) + i % 4 + 4 lg
        using SVec = std::conditional_t<NARROW, floatx8, floatx16>;
        SVec S;
        if constexpr (NARROW) {
            floatx4 s4[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            if (codes) {
                if constexpr (FP8) {
#pragma unroll
                    for (int q = 0; q < KA; ++q) {
                        const uintx2 kc = *reinterpret_cast<const uintx2*>(smem + kaddr8[q]);
                        s4[q & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, expand8(kc[0], kc[1])), qf[q >> 1], s4[q & 1], 0, 0, 0);
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i) { s4[0][i] *= a.k_scale; s4[1][i] *= a.k_scale; }
                }
            } else {
#pragma unroll
                for (int q = 0; q < KA; ++q) {
                    const uintx4 kv = *reinterpret_cast<const uintx4*>(smem + kaddr[q]);
                    s4[q & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kv), qf[q >> 1], s4[q & 1], 0, 0, 0);
                }
            }
            S = __builtin_shufflevector(s4[0], s4[1], 0, 1, 2, 3, 4, 5, 6, 7);
        } else {
#pragma unroll
            for (int i = 0; i < 16; ++i) S[i] = 0.f;
            if (codes) {
                if constexpr (FP8) {
#pragma unroll
                    for (int q = 0; q < KS; ++q) {
                        const uintx2 kc = *reinterpret_cast<const uintx2*>(smem + kaddr8[q]);
                        S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, expand8(kc[0], kc[1])), qf[q], S, 0, 0, 0);
                    }
#pragma unroll
                    for (int i = 0; i < 16; ++i) S[i] *= a.k_scale;
                }
            } else {
#pragma unroll
                for (int q = 0; q < KS; ++q) {
                    const uintx4 kv = *reinterpret_cast<const uintx4*>(smem + kaddr[q]);
                    S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kv), qf[q], S, 0, 0, 0);
                }
            }
        }
        // the scores depend on every fragment read: once they are pinned here the K slot may be overwritten.  (The wait states
        // are those between a product and a read of its result, which the compiler does not count across a branch.)
        asm volatile("s_nop 11" : "+v"(S));
        asm volatile("" ::: "memory");
        if (more) issue(ns, nt, npg, IsK{});
        const int key0 = cs.ks + ct * KT;
        const int k0c = row0_of(cs, ct);
        const bool partial = k0c != key0 || cs.ke - k0c < KT;      // some stage rows are not keys of this stage
        // masks: keys outside the stage's range, keys this lane's query does not see yet, rows that do not attend
        constexpr int kGroup = NARROW ? 16 : 8;                     // stage rows between two groups of four scores
        if (partial || cs.rlo > 0 || cs.rhi < TR || key0 + KT > cs.vis_base) {
            const bool attends = lq >= cs.rlo && lq < cs.rhi;
            const int vis_end = min(cs.ke, cs.vis_base + t_lane);
            const int first = k0c + 4 * (NARROW ? lg : hl);         // stage row of element i is kGroup (i / 4) + i % 4 behind it
            const int lo_i = key0 - first, hi_i = (attends ? vis_end : k0c) - first;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int ri = kGroup * (i >> 2) + (i & 3);
                if (ri < lo_i || ri >= hi_i) S[i] = -INFINITY;
            }
        }
        float tmax = fmaxf(S[0], S[1]);
#pragma unroll
        for (int i = 2; i < NE; i += 2) tmax = fmaxf(fmaxf(tmax, S[i]), S[i + 1]);
        if (__any(tmax > m_used + tau_raw)) {       // (m_used is the same in all lanes of a row)
            if constexpr (NARROW) tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
            const float m_new = fmaxf(m_used, half_max(tmax));
            // equal maxima (also -inf and -inf: a row that has seen no key yet) keep the accumulators
            const float alpha = (m_new == m_used) ? 1.0f : __builtin_amdgcn_exp2f((m_used - m_new) * c2);
            m_used = m_new;
            mc = (m_new == -INFINITY) ? 0.f : m_new * c2;
            lsum *= alpha;
#pragma unroll
            for (int i = 0; i < VA; ++i)
#pragma unroll
                for (int j = 0; j < OE; ++j) Oacc[i][j] *= alpha;
        }
        constexpr int NT = NE / 8;
        uintx4 pb[NP][NT];
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            S[i] = __builtin_amdgcn_exp2f(fmaf(S[i], c2, -mc));
            lsum += S[i];
        }
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) pb[0][tt] = pack8(S, tt);
        if constexpr (NP > 1) {
            if (codes) {                            // what the first piece left out, and what the second one did (both differences are exact)
#pragma unroll
                for (int n = 1; n < NP; ++n)
#pragma unroll
                    for (int tt = 0; tt < NT; ++tt) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            S[8 * tt + 2 * i] -= bf16_lo(pb[n - 1][tt][i]);
                            S[8 * tt + 2 * i + 1] -= bf16_hi(pb[n - 1][tt][i]);
                        }
                        pb[n][tt] = pack8(S, tt);
                    }
            }
        }
        wait_for(more ? copies_of(ns) : 0);         // this stage's V rows are here, the next K rows may still be on their way
        if (partial) {
            // stage rows that are not keys of this stage (re-read from below the range, or past a range that ends before
            // row 32 of the tensor, or a page's unwritten tail) may hold anything: their probabilities are zero, but 0 * NaN
            // is NaN in the second product, so their V rows are cleared in LDS
            const int nlo = key0 - k0c, nhi = cs.ke - k0c;
            if (codes) {
#pragma unroll
                for (int i = 0; i < CPS8; ++i) {
                    const int row = i * RPI8 + lrow8;
                    if (row < nlo || row >= nhi) *reinterpret_cast<uintx4*>(smem + STB + i * 1024 + l * 16) = uintx4{0u, 0u, 0u, 0u};
                }
            } else {
#pragma unroll
                for (int i = 0; i < CPS; ++i) {
                    const int row = i * RPI + lrow;
                    if (row < nlo || row >= nhi) *reinterpret_cast<uintx4*>(smem + STB + i * 1024 + l * 16) = uintx4{0u, 0u, 0u, 0u};
                }
            }
        }
        if constexpr (FP8) {
            if (codes && !code_units) {             // (once per wavefront: the shared blocks come first; the host bounds the scale)
                const float rs = 1.0f / a.v_scale;
#pragma unroll
                for (int i = 0; i < VA; ++i)
#pragma unroll
                    for (int j = 0; j < OE; ++j) Oacc[i][j] *= rs;
                code_units = true;
            }
        }
        // O^T += V^T P^T
        auto product = [&](const bf16x8& vv, const uintx4& p, OBlock& o) {
            if constexpr (NARROW) o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, __builtin_bit_cast(bf16x8, p), o, 0, 0, 0);
            else o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vv, __builtin_bit_cast(bf16x8, p), o, 0, 0, 0);
        };
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
#pragma unroll
            for (int db = 0; db < VA; ++db) {
                bf16x8 vv;
                if (codes) {
                    if constexpr (FP8) {
                        const intx2 vc = __builtin_amdgcn_ds_read_tr8_b64_v2i32((__attribute__((address_space(3))) intx2*)HG_LDS(smem + vaddr8[db] + tt * 16 * D));
                        vv = __builtin_bit_cast(bf16x8, expand8((unsigned)vc[0], (unsigned)vc[1]));
                    }
                } else {
                    const unsigned char* vp = smem + vaddr[db] + tt * 16 * ROWB;
                    const shortx4 vlo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp));
                    const shortx4 vhi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)HG_LDS(vp + (NARROW ? 16 : 8) * ROWB));
                    vv = __builtin_bit_cast(bf16x8, __builtin_shufflevector(vlo, vhi, 0, 1, 2, 3, 4, 5, 6, 7));
                }
                if constexpr (NP > 1) {
                    if (codes) {
#pragma unroll
                        for (int n = NP - 1; n > 0; --n) product(vv, pb[n][tt], Oacc[db]);
                    }
                }
                product(vv, pb[0][tt], Oacc[db]);
            }
        }
        // the accumulators depend on every fragment read of this stage: once they are pinned here the V slot may be overwritten
#pragma unroll
        for (int db = 0; db < VA; ++db) asm volatile("" : "+v"(Oacc[db]));
        asm volatile("s_nop 11" ::: "memory");
        if (more) issue(ns, nt, npg, IsV{});
        cs = ns;
        ct = nt;
    }

    // ---- the workgroup's partial results meet in LDS (Eq. 5) -------------------------------------------------------------------------
    // O of wavefront v takes the place of its ring: row-major [TR][D] fp32 with the 16-byte chunk c of row r at chunk
    // c ^ (r % (D / 4)); behind all of them the maxima and sums [NWS][TR].
    constexpr int CH = G_::CH, RPW = G_::RPW, LPR = G_::LPR, CPL = G_::CPL;      // CH: 16-byte chunks per row
    float* const Mw = reinterpret_cast<float*>(smem_all + NWS * 2 * STB);
    float* const Lw = Mw + NWS * TR;
    int* const last_flag = reinterpret_cast<int*>(Lw + NWS * TR);
    if constexpr (NARROW) lsum += __shfl_xor(lsum, 16);
    const float ltot = half_sum(lsum);
    if constexpr (FP8) {
        if (code_units) {
#pragma unroll
            for (int i = 0; i < VA; ++i)
#pragma unroll
                for (int j = 0; j < OE; ++j) Oacc[i][j] *= a.v_scale;
        }
    }
    {                                               // (own ring only: nothing to wait for)
        unsigned char* const ow = smem_all + w * (2 * STB);
#pragma unroll
        for (int db = 0; db < VA; ++db)
#pragma unroll
            for (int q4 = 0; q4 < OE / 4; ++q4) {
                const int chunk = NARROW ? 4 * db + lg : 8 * db + 2 * q4 + hl;
                *reinterpret_cast<float4*>(ow + lq * (D * 4) + ((chunk ^ (lq & (CH - 1))) * 16)) =
                    make_float4(Oacc[db][4 * q4], Oacc[db][4 * q4 + 1], Oacc[db][4 * q4 + 2], Oacc[db][4 * q4 + 3]);
            }
        if (l < TR) {
            Mw[w * TR + lq] = m_used;
            Lw[w * TR + lq] = ltot;
        }
    }
    __syncthreads();
    // wavefront w finishes rows RPW w .. + RPW - 1: lane -> row RPW w + l / LPR, 16-byte chunks (l % LPR) * CPL .. + CPL - 1
    const int row = RPW * w + l / LPR, c0 = (l % LPR) * CPL;
    const bool finishes = row < TR && r0 + row < R;
    float4 acc[CPL];
    float M = -INFINITY, Lsum = 0.f;
    if (row < TR) {
        float mv[NWS];
#pragma unroll
        for (int v = 0; v < NWS; ++v) {
            mv[v] = Mw[v * TR + row];
            M = fmaxf(M, mv[v]);
        }
        float f[NWS];
#pragma unroll
        for (int v = 0; v < NWS; ++v) {
            f[v] = (mv[v] == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f((mv[v] - M) * c2);
            Lsum += f[v] * Lw[v * TR + row];
        }
        const float inv = Lsum > 0.f ? 1.0f / Lsum : 0.f;     // a row without any key: O = 0, LSE = -inf
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int v = 0; v < NWS; ++v) {
                const float4 o = *reinterpret_cast<const float4*>(smem_all + v * (2 * STB) + row * (D * 4) + (((c0 + c) ^ (row & (CH - 1))) * 16));
                acc[c].x += f[v] * o.x; acc[c].y += f[v] * o.y; acc[c].z += f[v] * o.z; acc[c].w += f[v] * o.w;
            }
            acc[c].x *= inv; acc[c].y *= inv; acc[c].z *= inv; acc[c].w *= inv;
        }
    }
    float lse = Lsum > 0.f ? M * a.scale + __logf(Lsum) : -INFINITY;

    if (NWS == 8 && a.splits > 1) {      // (four wavefronts: one workgroup per column)
        // ---- the column's results meet in the workspace ----------------------------------------------------------------------------------
        // (a column's [S][TR][D] results and, behind them, [S][TR] LSEs; every access below is at a row < TR of a split < S)
        const int S = a.splits;
        constexpr unsigned OB = TR * D * 4, LB = TR * 4;      // bytes of one split's
        const AgentBuffer part(a.part + (int64_t)col * S * (TR * (D + 1)), (unsigned)S * (OB + LB));
        const unsigned at = (unsigned)(row * D + 4 * c0) * 4u, lse_at = (unsigned)S * OB + (unsigned)row * 4u;
        if (finishes) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) part.store4((unsigned)split * OB + at + 16 * c, acc[c]);
            if (l % LPR == 0) part.store1((unsigned)split * LB + lse_at, lse);
        }
        wait_vm<0>();                               // this wavefront's results are where every XCD sees them
        __syncthreads();
        if (tid == 0) {
            // (the counter wraps to zero by itself and is used with this S only: whatever happens, S arrivals per launch leave it at zero)
            const unsigned before = atomicInc(a.arrivals + col, (unsigned)(S - 1));
            const int last = before == (unsigned)(S - 1);
            *last_flag = last;
        }
        __syncthreads();
        if (!*last_flag || !finishes) return;
        M = -INFINITY;
        Lsum = 0.f;
#pragma unroll
        for (int c = 0; c < CPL; ++c) acc[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        constexpr int U = 16 / CPL;                 // results in flight per lane: all of them, mostly
        for (int i0 = 0; i0 < S; i0 += U) {
            float li[U], gm = M;
            float4 ow[U][CPL];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                li[u] = -INFINITY;
#pragma unroll
                for (int c = 0; c < CPL; ++c) ow[u][c] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (i0 + u < S) {
                    li[u] = part.load1((unsigned)(i0 + u) * LB + lse_at);
#pragma unroll
                    for (int c = 0; c < CPL; ++c) ow[u][c] = part.load4((unsigned)(i0 + u) * OB + at + 16 * c);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) gm = fmaxf(gm, li[u]);
            const float gs = gm == -INFINITY ? 0.f : gm;        // nothing but empty results so far: every weight is 0
            const float re = __builtin_amdgcn_exp2f((M - gs) * kLog2e);
            M = gm;
            Lsum *= re;
#pragma unroll
            for (int c = 0; c < CPL; ++c) { acc[c].x *= re; acc[c].y *= re; acc[c].z *= re; acc[c].w *= re; }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float f = __builtin_amdgcn_exp2f((li[u] - gs) * kLog2e);
                Lsum += f;
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    acc[c].x = fmaf(f, ow[u][c].x, acc[c].x);
                    acc[c].y = fmaf(f, ow[u][c].y, acc[c].y);
                    acc[c].z = fmaf(f, ow[u][c].z, acc[c].z);
                    acc[c].w = fmaf(f, ow[u][c].w, acc[c].w);
                }
            }
        }
        const float inv = Lsum > 0.f ? 1.0f / Lsum : 0.f;
#pragma unroll
        for (int c = 0; c < CPL; ++c) { acc[c].x *= inv; acc[c].y *= inv; acc[c].z *= inv; acc[c].w *= inv; }
        lse = Lsum > 0.f ? M + __logf(Lsum) : -INFINITY;
    }

    const int rg = r0 + row;                        // the row this lane finishes
    if (finishes) {
        const int ob = (int)a.by_seq.of((unsigned)rg), of_seq = rg - ob * rps, ot = (int)a.by_group.of((unsigned)of_seq);
        const int64_t oidx = ((int64_t)ob * a.nq + ot) * a.Hq + kvh * a.G + (of_seq - ot * a.G);
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            const int d = 4 * (c0 + c);
            if (a.bf16) *reinterpret_cast<uint2*>(static_cast<uint16_t*>(a.O) + oidx * D + d) = make_uint2(pack_bf16(acc[c].x, acc[c].y), pack_bf16(acc[c].z, acc[c].w));
            else *reinterpret_cast<float4*>(static_cast<float*>(a.O) + oidx * D + d) = acc[c];
        }
        if (l % LPR == 0 && a.LSE != nullptr) a.LSE[oidx] = lse;
    }
}

template <int D, bool PAGED, int CODES, int TR, int NWS>
static hipError_t launch_small_t(const SmallArgs& a, hipStream_t s) {
    constexpr int lds = SmallGeo<D, TR, NWS>::LDS;
    static bool attr_set[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64 && !attr_set[dev]) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&fused_small_kernel<D, PAGED, CODES, TR, NWS>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    const unsigned grid = small_grid(a.cols * a.splits);
    fused_small_kernel<D, PAGED, CODES, TR, NWS><<<grid, 64 * NWS, lds, s>>>(a);
    return hipGetLastError();
}

template <int D, int TR, int NWS>
static hipError_t launch_small_d(const SmallArgs& a, hipStream_t s) {
    if constexpr (D == 128)      // (at D = 64 the vector-ALU kernel reads all 8-bit rows)
        if (a.fp8 && !a.fp32_weights) return a.pg.table ? launch_small_t<D, true, 1, TR, NWS>(a, s) : launch_small_t<D, false, 1, TR, NWS>(a, s);
    if (a.fp8) return a.pg.table ? launch_small_t<D, true, 2, TR, NWS>(a, s) : launch_small_t<D, false, 2, TR, NWS>(a, s);
    return a.pg.table ? launch_small_t<D, true, 0, TR, NWS>(a, s) : launch_small_t<D, false, 0, TR, NWS>(a, s);
}

// Workspace floats the splits of a call need: per column [splits][rows][D] results and [splits][rows] LSEs (and as many left over, which
// earlier layouts used: what fits a workspace does not change)
size_t small_part_floats(int cols, int splits, int rows, int D) { return (size_t)cols * splits * rows * (D + 2); }

hipError_t launch_fused_small(const SmallArgs& args, int D, hipStream_t s) {
    SmallArgs a = args;
    a.c2 = a.scale * kLog2e;
    a.tau_raw = TAU / a.c2;
    if (!a.dealt && a.splits != 1) return hipErrorInvalidValue;
    if (a.tiles < 1 || a.Hkv < 1 || a.splits < 1 || (D != 64 && D != 128)) return hipErrorInvalidValue;
    if ((long long)a.tiles * a.Hkv != a.cols || (long long)a.cols * a.splits >= (1LL << 31)) return hipErrorInvalidValue;
    if (a.splits > 1 && (!a.part || !a.arrivals)) return hipErrorInvalidValue;
    if (a.pg.table && (a.pg.shift < 4 || a.pg.stride < 1 || a.pg.n_pages < 1)) return hipErrorInvalidValue;
    if (a.rows != 16 && a.rows != 32) return hipErrorInvalidValue;
    if (a.wavefronts == 4) {
        if (a.splits != 1) return hipErrorInvalidValue;
        if (a.rows == 16) return D == 128 ? launch_small_d<128, 16, 4>(a, s) : launch_small_d<64, 16, 4>(a, s);
        return D == 128 ? launch_small_d<128, 32, 4>(a, s) : launch_small_d<64, 32, 4>(a, s);
    }
    if (a.wavefronts != 8) return hipErrorInvalidValue;
    if (a.rows == 16) return D == 128 ? launch_small_d<128, 16, 8>(a, s) : launch_small_d<64, 16, 8>(a, s);
    return D == 128 ? launch_small_d<128, 32, 8>(a, s) : launch_small_d<64, 32, 8>(a, s);
}

}  // namespace hg
