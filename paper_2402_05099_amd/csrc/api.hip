// Host side of libhydragen: argument checks, work partitioning, kernel sequencing.  No device allocation,
// no host synchronisation, no copies: every entry point only enqueues kernels on the context's stream.
#include <math.h>
#include <string.h>
#include <algorithm>
#include <mutex>
#include <new>

#include "hg_internal.h"
#include "hydragen_debug.h"

struct hg_ctx {
    int device;
    hipStream_t stream;
    unsigned char* ws;
    size_t ws_bytes;
    int opt_prefix_splits;
    int opt_suffix_chunk;
    int opt_overlap;
    int opt_naive_chunk;
    int opt_prefix_kernel;
    int opt_wide_slots;
    int opt_nq;            // queries per sequence (1 = decode)
    int opt_suffix_kernel; // 0 automatic, 1 vector-ALU kernel, 2 matrix-core kernel wherever it applies
    int opt_suffix_ipw;    // matrix-core suffix kernel: work items per wavefront (0 automatic)
    int opt_suffix_tile;   // matrix-core suffix kernel: query rows per tile (0 automatic, 16, 32)
    int opt_fused_kernel;  // fused call: 0 automatic, 1 separate kernels, 2 single launch whenever it applies
    unsigned* counters;    // kContextCounters device counters, zero between calls (null: none left)
    int counter_slot;      // (-1: none, or not to be given back)
    bool counters_used, counters_in_graph;
    hipStream_t counter_stream;      // the stream that used them last
    hipStream_t aux;       // second stream for the overlap option
    hipEvent_t ev_fork, ev_join;
    // stage timing ring: slot = call % HG_TIMING_RING, 2 events (begin, end) per stage
    int opt_timing;
    hipEvent_t* tev;       // [HG_TIMING_RING][HG_MAX_STAGES][2], created when timing is first enabled
    unsigned char* tused;  // [HG_TIMING_RING][HG_MAX_STAGES]
    long long tcalls;      // fused calls recorded since timing was enabled
};

// Partial-result memory of hg_hydragen_attn_static, the fused call for callers that cannot provide a workspace from an
// allocator: a fixed array in the library's device image (every GPU the library is loaded on holds its own copy until
// the process ends).  In host code the array's name is only a handle for hipGetSymbolAddress: the address a kernel may
// use is looked up once per device in hg_create and kept in g_scratch_ptr.
static __device__ __align__(256) unsigned char scratch[HG_STATIC_SCRATCH_BYTES];
static unsigned char* g_scratch_ptr[64];   // per device, set by hg_create on that device
static std::mutex g_scratch_mu;

// The contexts' device counters (work counter of combined_impl.h, meeting counters of fused_small.hip): a fixed array in the
// device image (zero when the library is loaded, and every call leaves its counters at zero), handed out to contexts
// in slots.  A slot is given back with the context, behind an event on the stream that used it last, and is handed
// out again once that event has happened: nothing ever waits for it.  Slots whose calls were captured stay out, for the
// graph may be replayed at any time, and so do those whose last use cannot be marked.  A context that finds no slot works
// without: separate kernels, one workgroup per column.
constexpr int kCounterSlots = 1024;
static __device__ unsigned context_counters[kCounterSlots * hg::kContextCounters];
struct CounterPool {
    unsigned* base = nullptr;
    int fresh = 0;                   // slots never handed out start here
    int n_back = 0;                  // slots given back, oldest first
    struct { int slot; hipEvent_t done; } back[kCounterSlots];      // done: null if the slot was never used
};
static CounterPool* g_counters[64];   // per device, guarded by g_scratch_mu

namespace {

using namespace hg;

inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
inline int round_up(int a, int b) { return ceil_div(a, b) * b; }

struct Parts {   // fp32 partial results carved out of the workspace
    float* O;    // [cap][rows][D]
    float* L;    // [cap][rows]
    int cap;
    int64_t rows;
    int D;
    float* o(int p) const { return O + (int64_t)p * rows * D; }
    float* l(int p) const { return L + (int64_t)p * rows; }
};

struct Ws { unsigned char* p; size_t bytes; };   // device memory that holds the partial results of one call

// partial results that fit `bytes` of such memory
int parts_cap(size_t bytes, int64_t rows, int D) {
    const size_t per = (size_t)rows * (D + 1) * sizeof(float);
    const size_t cap = per ? bytes / per : 0;
    return cap > HG_MAX_PARTS ? HG_MAX_PARTS : (int)cap;
}

Parts carve(const Ws& ws, int64_t rows, int D) {
    Parts p{};
    p.rows = rows;
    p.D = D;
    p.cap = ws.p ? parts_cap(ws.bytes, rows, D) : 0;
    p.O = reinterpret_cast<float*>(ws.p);
    p.L = p.O + (int64_t)p.cap * rows * D;
    return p;
}

int check_shape(int B, int Hq, int Hkv, int D, int nq) {
    if (B < 0 || Hq <= 0 || Hkv <= 0 || nq < 1) return HG_ERR_INVALID_ARG;
    if (D != 64 && D != 128) return HG_ERR_UNSUPPORTED;
    if (Hq % Hkv != 0) return HG_ERR_UNSUPPORTED;
    if ((int64_t)B * nq * Hq * D >= (1LL << 31)) return HG_ERR_UNSUPPORTED;
    return HG_OK;
}

// Byte offsets inside one sequence's suffix rows are 32-bit in the kernels: max_len * Hkv * D elements must stay below 2^31.
int check_suffix_span(int max_len, int Hkv, int D) {
    return (int64_t)max_len * Hkv * D >= (1LL << 31) ? HG_ERR_UNSUPPORTED : HG_OK;
}

int check_level(const hg_level* lv, int Hkv, int D) {
    if (!lv) return HG_ERR_INVALID_ARG;
    if (lv->n_blocks < 1 || lv->max_rows < 0 || lv->max_seqs < 0) return HG_ERR_INVALID_ARG;
    if ((lv->kv_off == nullptr) != (lv->seq_off == nullptr)) return HG_ERR_INVALID_ARG;
    if (lv->n_blocks > 1 && !lv->kv_off) return HG_ERR_INVALID_ARG;
    if (lv->max_rows > 0 && (!lv->K || !lv->V)) return HG_ERR_INVALID_ARG;
    if ((int64_t)lv->n_blocks * lv->max_rows * Hkv * D >= (1LL << 31)) return HG_ERR_UNSUPPORTED;
    return HG_OK;
}

LevelDev to_dev(const hg_level& lv, int B) {
    LevelDev d{};
    d.K = static_cast<const uint16_t*>(lv.K);
    d.V = static_cast<const uint16_t*>(lv.V);
    d.kv_off = lv.kv_off;
    d.seq_off = lv.seq_off;
    d.n_blocks = lv.n_blocks;
    d.max_rows = lv.max_rows;
    d.max_seqs = lv.kv_off ? lv.max_seqs : B;
    return d;
}

int pick_gt(int G) {
    for (int gt : {8, 4, 2}) if (G % gt == 0) return gt;
    return 1;
}

int hip_rc(hipError_t e) { return e == hipSuccess ? HG_OK : HG_ERR_HIP; }

// which shared-block kernel runs a level, and how many partial results per row it writes
struct LevelPlan { bool wide; int ns; WidePlan wp; };

// The persistent 256-row kernel runs a level whose blocks have more than 128 query rows; the 128-row
// kernel runs the rest.  (At D = 128, 16 blocks of 128 rows x 512 keys x 40 heads alone: 55 us on the
// persistent kernel against 63 us; but inside the fused call its workgroups take whole CUs from the suffix kernel, where
// 128-row workgroups share them: 0.646 against 0.591 ms on the two-level tree.)
// At D = 64 the same rule holds (fused call on 1024 x 40 heads x 16K keys: 0.351 against 0.377 ms; on the two-level
// tree the automatic choice gives 0.310 ms against 0.321 with 128-row workgroups only and 0.392 with 256-row only).
// HG_OPT_PREFIX_KERNEL = 1 forces the 128-row kernel, 2 the 256-row kernel.  max_parts bounds the
// partial results the plan may use.
// G: query rows per sequence and KV head (queries per sequence x query heads per KV head).
LevelPlan plan_level(const hg_ctx* c, const LevelDev& lv, int Hkv, int G, int D, int max_parts, int wide_slots = 32,
                     int wide_above = kPrefixRowsNarrow, bool table = true) {
    LevelPlan p{};
    const long long rows = (long long)lv.max_seqs * G;
    p.wide = false;
    p.ns = 1;
    if (lv.max_rows <= 0) return p;
    if (max_parts < 1) max_parts = 1;
    if (max_parts > HG_MAX_PARTS) max_parts = HG_MAX_PARTS;
    const bool want_wide = c->opt_prefix_kernel != 1 && (c->opt_prefix_kernel == 2 || rows > wide_above);
    if (want_wide && plan_prefix_wide(lv, Hkv, G, D, max_parts, c->opt_wide_slots > 0 ? c->opt_wide_slots : wide_slots, &p.wp, table)) {
        p.wide = true;
        p.ns = p.wp.nparts;
        return p;
    }
    const int slots = 512;   // 128-row workgroups resident on the 256 CUs (two per CU)
    const int64_t base = (int64_t)lv.n_blocks * ceil_div((int)rows, kPrefixRowsNarrow) * Hkv;
    const int max_ns = ceil_div(lv.max_rows, kPrefixKeys);
    int ns;
    if (c->opt_prefix_splits > 0) {
        ns = c->opt_prefix_splits;
    } else {
        // enough workgroups for about two full rounds of the resident slots, in chunks of at least 512 keys;
        // every extra split adds a partial result for the merge to read
        ns = (int)((2 * slots + base - 1) / (base > 0 ? base : 1));
        const int by_len = lv.max_rows / 512;
        if (ns > by_len) ns = by_len;
        if (ns > 16) ns = 16;
    }
    if (ns > max_ns) ns = max_ns;
    if (ns > max_parts) ns = max_parts;
    if (ns < 1) ns = 1;
    p.ns = ns;
    return p;
}

PrefixArgs level_args(const void* Q, const LevelDev& lv, const LevelPlan& plan, int B, int nq, int Hq, int Hkv, float scale, const OutDev& out) {
    PrefixArgs a{};
    a.Q = static_cast<const uint16_t*>(Q);
    a.lv = lv;
    a.B = B; a.Hq = Hq; a.Hkv = Hkv; a.G = Hq / Hkv;
    a.nq = nq;
    a.by_heads = divider((unsigned)Hkv);
    a.by_seq = divider((unsigned)(nq * a.G));
    a.by_group = divider((unsigned)a.G);
    a.scale = scale;
    a.out = out;
    if (plan.wide) a.wide = plan.wp;
    return a;
}

// enqueue the shared-block kernel for one level with `ns` splits writing to `out` (part = split)
int run_level(const void* Q, const LevelDev& lv, const LevelPlan& plan, int B, int nq, int Hq, int Hkv, int D, float scale,
              const OutDev& out, hipStream_t s) {
    PrefixArgs a = level_args(Q, lv, plan, B, nq, Hq, Hkv, scale, out);
    if (plan.wide) return hip_rc(launch_prefix_wide(a, D, s));
    a.mtiles = ceil_div(lv.max_seqs * a.G * nq, kPrefixRowsNarrow);
    a.nsplit = plan.ns;
    a.chunk = round_up(ceil_div(lv.max_rows > 0 ? lv.max_rows : 1, plan.ns), kPrefixKeys);
    const int64_t total = (int64_t)lv.n_blocks * plan.ns * Hkv * a.mtiles;
    if (total >= (1LL << 28)) return HG_ERR_UNSUPPORTED;
    a.total_tiles = (int)total;
    a.per_xcd = ceil_div(a.total_tiles, 8);
    return hip_rc(launch_prefix_narrow(a, D, s));
}

struct SuffixPlan { int chunk, nchunks, gt; bool mfma; int ipw; };

// Storage format of the suffix cache: bf16 rows, or E4M3 codes with one scale per tensor (value = code * scale).
struct KvFmt { int fp8 = 0; float k_scale = 1.f, v_scale = 1.f; };

// Automatic choice between the two per-sequence kernels (thresholds measured at D = 128).  The matrix-core kernel reads every K/V row
// once for all nq * G query rows that a KV head serves; the vector-ALU kernel pays one dot product per row and key
// and, across queries, re-reads the suffix.  Measured (B = 512, lengths up to 512, matrix-core against vector-ALU):
// nq = 2: 184 against 368 us; G = 3: 96 against 211 us; G = 2: 94 against 114 us, but 178 against 153 us when no
// sequence has more than 128 rows (the per-item cost of the matrix-core kernel).  One row per KV head: the
// matrix-core kernel streams long rows better (6.4 against 5.8-6.0 TB/s from a few hundred rows per sequence on:
// lengths 64..384: 794 against 841 us; 256..1024: 824 against 915 us) and loses on short ones (lengths up to 256:
// 121 against 116 us; 32..128: 328 against 285 us).  At D = 64 that last gain is not consistent (402 against 440 us at
// 64..384 rows, 462 against 427 us at 1024..4096) and the clause is left out.
bool auto_mfma(int nq, int G, int max_len, int D) {
    return nq >= 2 || G >= 3 || (G == 2 && max_len >= 256) || (D == 128 && max_len >= 384);
}

// Work items of the suffix kernel are (sequence, query, KV head, group of query heads, key chunk), one wavefront
// each, in the vector-ALU kernel, and (sequence, KV head, 32-row tile of the nq * G rows, key chunk) in the
// matrix-core kernel (chosen by auto_mfma, HG_OPT_SUFFIX_KERNEL forces either; an 8-bit cache at D = 64 stays on the
// vector ALU).
// 256 keys per chunk by default; when that leaves fewer than eight wavefronts per CU (few sequences or KV heads)
// the chunks shrink, down to 64 keys, so that enough loads are in flight to cover HBM latency.
// max_chunk bounds the keys per work item (a paged cache allows 32 pages per work item).
SuffixPlan plan_suffix(const hg_ctx* c, int max_len, int G, int B, int nq, int Hkv, int D, bool paged, int max_chunk = 1 << 30,
                       bool fp8 = false) {
    SuffixPlan p;
    p.gt = pick_gt(G);
    const int R = nq * G;
    p.ipw = c->opt_suffix_ipw;
    (void)paged;
    p.mfma = (D == 128 || !fp8) && c->opt_suffix_kernel != 1 && (c->opt_suffix_kernel == 2 || auto_mfma(nq, G, max_len, D));   // 8-bit rows on the matrix cores: D = 128 only
    if (p.mfma) max_chunk = 1 << 30;   // the matrix-core kernel looks pages up per stage: no limit on pages per item
    if (c->opt_suffix_chunk > 0) {
        p.chunk = round_up(c->opt_suffix_chunk, 32);
        if (p.chunk > max_chunk) p.chunk = max_chunk;
    } else if (p.mfma) {
        // a wavefront pays a fixed price per work item (its query tile, the first stage's latency, the result's
        // stores): long items, cut only when there would be fewer than three per CU
        p.chunk = 1024;
        const long long per_chunk = (long long)B * Hkv * ceil_div(R, 32);
        while (p.chunk > 128 && per_chunk * ceil_div(max_len > 0 ? max_len : 1, p.chunk) < 768) p.chunk /= 2;
    } else {
        p.chunk = 256;
        const long long per_chunk = (long long)B * nq * Hkv * (G / p.gt);
        while (p.chunk > 64 && per_chunk * ceil_div(max_len > 0 ? max_len : 1, p.chunk) < 2048) p.chunk /= 2;
    }
    if (p.chunk > max_chunk) p.chunk = max_chunk;
    p.nchunks = max_len > 0 ? ceil_div(max_len, p.chunk) : 1;
    return p;
}

DecodeArgs suffix_args(const void* Q, const void* Ks, const void* Vs, const int32_t* offsets, const int32_t* lengths, int max_len, int B,
                       int nq, int Hq, int Hkv, float scale, int chunk, int nchunks, int gt, const OutDev& out, const PagedDev& pg,
                       const KvFmt& fmt) {
    DecodeArgs a{};
    a.pg = pg;
    a.fp8 = fmt.fp8;
    a.k_scale = fmt.k_scale;
    a.v_scale = fmt.v_scale;
    a.Q = static_cast<const uint16_t*>(Q);
    a.Ks = static_cast<const uint16_t*>(Ks);
    a.Vs = static_cast<const uint16_t*>(Vs);
    a.offsets = offsets;
    a.lengths = lengths;
    a.max_len = max_len;
    a.B = B; a.Hq = Hq; a.Hkv = Hkv; a.G = Hq / Hkv;
    a.nq = nq;
    a.chunk = chunk;
    a.nchunks = nchunks;
    a.units = (int64_t)B * nq * nchunks * Hkv * (a.G / gt);
    a.scale = scale;
    a.out = out;
    return a;
}

int run_decode(const void* Q, int n_levels, const LevelDev* lv, const void* Ks, const void* Vs, const int32_t* offsets,
               const int32_t* lengths, int max_len, int B, int nq, int Hq, int Hkv, int D, float scale, int chunk, int nchunks,
               int gt, const OutDev& out, hipStream_t s, const PagedDev& pg = PagedDev{}, bool mfma = false, int mfma_ipw = 0, bool seg = false,
               const KvFmt& fmt = KvFmt{}, int mfma_tile = 0) {
    DecodeArgs a = suffix_args(Q, Ks, Vs, offsets, lengths, max_len, B, nq, Hq, Hkv, scale, chunk, nchunks, gt, out, pg, fmt);
    a.n_levels = n_levels;
    for (int i = 0; i < n_levels; ++i) a.lv[i] = lv[i];
    if (mfma) {
        a.seg = seg ? 1 : 0;
        // up to 16 rows per KV head and sequence fit a 16-row tile: half the matrix and softmax work per stage
        a.tile_rows = (nq * a.G <= 16 && mfma_tile != 32) ? 16 : 32;
        const int64_t items = (int64_t)B * nchunks * ceil_div(nq * a.G, a.tile_rows) * Hkv;
        if (items >= (1LL << 31)) return HG_ERR_UNSUPPORTED;
        a.items = (int)items;
        // consecutive items per wavefront: the copies of the next item are in flight while one is finished; few
        // enough per wavefront that the hardware still balances ragged lengths (>= 8 workgroups per resident slot)
        a.ipw = mfma_ipw > 0 ? mfma_ipw : (int)std::min<int64_t>(4, std::max<int64_t>(1, items / (1280 * 8)));
        return hip_rc(launch_decode_mfma(a, D, s));
    }
    return hip_rc(launch_decode(a, D, gt, s));
}

int run_merge(int n, const Parts& parts, int first, int D, void* O_out, int o_dtype, float* LSE_out, hipStream_t s, unsigned* clear = nullptr) {
    MergeArgs m{};
    m.clear = clear;
    m.n = n;
    for (int i = 0; i < n; ++i) {
        m.O[i] = parts.o(first + i);
        m.L[i] = parts.l(first + i);
    }
    m.rows = parts.rows;
    m.O_out = O_out;
    m.L_out = LSE_out;
    return hip_rc(launch_merge(m, D, false, o_dtype == HG_BF16, s));
}

float eff_scale(float scale, int D) { return scale > 0.f ? scale : 1.0f / sqrtf((float)D); }

OutDev direct_out(void* O, int o_dtype, float* LSE) {
    OutDev o{};
    o.O = O; o.LSE = LSE; o.bf16 = (o_dtype == HG_BF16); o.part_stride_O = 0; o.part_stride_L = 0;
    return o;
}

OutDev parts_out(const Parts& p, int first) {
    OutDev o{};
    o.O = p.o(first); o.LSE = p.l(first); o.bf16 = 0;
    o.part_stride_O = p.rows * p.D; o.part_stride_L = p.rows;
    return o;
}

// CUs per XCD for the persistent shared-block kernel when it overlaps the suffix kernel in the fused call.
// The shared-block kernel runs against the chip's power limit, so it loses little on fewer CUs (measured on
// config 3: 0.96 / 0.90 / 0.82 / 0.69 / 0.54 of its full-chip rate on 28 / 24 / 20 / 16 / 12 CUs per XCD), while
// the memory-bound suffix kernel takes the CUs that are left.  Model: while the shared-block kernel runs the
// suffix kernel streams at 0.7 x 6 TB/s x (its share of the CUs) (measured 0.92 / 1.77 / 2.06 TB/s on 64 / 96 /
// 128 CUs), afterwards at 6 TB/s; pick the count with the smallest finish time.  flops: shared-block work; bytes: suffix KV traffic (estimated from max_len).
int pick_wide_slots(double flops, double bytes, int T) {
    // relative rate of the shared-block kernel on 4, 8, .., 32 CUs per XCD (measured down to 12, scaled below)
    static const double rate[] = {0.18, 0.36, 0.543, 0.693, 0.823, 0.895, 0.964, 1.0};
    const double full_rate = 1.14e15, bw = 6.0e12;
    if (T < 1) T = 1;
    auto rate_at = [&](int eff) { return rate[eff / 4 - 1] + (rate[(eff + 3) / 4 - 1] - rate[eff / 4 - 1]) * (eff % 4) / 4.0; };
    const double ts = bytes / bw, tp32 = flops / full_rate;
    if (ts >= 2.0 * tp32) {
        // the suffix kernel dominates: the fewest CUs on which the shared blocks still finish in half its time
        // (when teams are so wide that no smaller count does, the general model below decides)
        for (int s = 4; s < 32; s += 4) {
            const int eff = s / T * T;
            if (eff >= 4 && flops / (full_rate * rate_at(eff)) <= 0.5 * ts) return eff;
        }
    }
    int best = 32;
    double best_t = 1e30;
    for (int s = 32; s >= 4; s -= 4) {
        const int eff = s / T * T;                 // CUs per XCD that hold whole teams (no workgroup is launched on the others)
        if (eff < 4) break;
        const double tp = flops / (full_rate * rate_at(eff));
        const double conc = 0.7 * bw * (256 - 8 * eff) / 256.0;
        const double t = bytes <= conc * tp ? tp : tp + (bytes - conc * tp) / bw;
        if (t < best_t * 0.995) { best_t = t; best = eff; }
    }
    return best;
}

// The same choice for the combined launch, where every CU goes on with suffix work when its shared-block pieces are done:
// the fewest CUs per XCD that finish the shared block before the end of the call.  Fewer CUs pay the persistent kernel's
// start-up and write its partial results; but the end of the launch must not wait for them.  Fitted (us): the launch
// takes ts + 0.65 (tp + 13), ts = the suffix alone, tp = the shared block alone on the whole chip; beside the suffix the shared
// block takes 1.2 times as long as alone on the same CUs, plus its start-up and 7 for every further 256-row tile (pieces)
// a CU has.  The tile role (tiles) gets a margin of a
// tenth: it is the slower to catch up.  Measured calls at 4 / 8 / 12 / 16 / 20 / 24 CUs: 1024 x 40 heads, 16K keys:
// - / 819 / 599 / 516 / 484 / 510; 4K keys, 8-bit cache: 433 / 245 / 219 / 223 / 229 / 246; 256 x 40 heads, 2K keys:
// 132 / 138 / 139 / 141 / 147 / 150; 512 x 64/8 heads, 4K keys: 349 / 186 / 153 / 134 / 157 / 166; 128 x 32/8 heads, 2K keys, paged:
// 46 / 52 / 55 / 60 / 64 / 69.  Where 4 would do, 5 are taken: the shared blocks end a fifth
// earlier for the start-up of eight more workgroups, and 40 teams hold the columns of 40 KV heads whole.  4 / 5 CUs, us: 256 x 40 heads, 2K keys
// 128.3 / 124.3; 267 x 64/8, 253 keys, 8-bit 51.4 / 41.9; 191 x 40, 699 keys, 8-bit 85.0 / 81.5; 1050 x 40, 78 keys, 8-bit paged 382.5 / 378.6; 32/8 heads, 515 keys 51.7 / 51.4; over 41 drawn calls
// that had 4: 1.015 in the mean, the worst 0.8 % slower.
int pick_combined_slots(double flops, double bytes, double pieces, int D, bool tiles) {
    static const double rate[] = {0.18, 0.36, 0.543, 0.693, 0.823, 0.895, 0.964, 1.0};      // on 4, 8, .., 32 CUs per XCD
    const double tp = flops / (D == 128 ? 1.14e15 : 0.63e15) * 1e6, ts = bytes / 6.0e12 * 1e6;
    const double end = ts + 0.65 * (tp + 13.0);
    auto shared_us = [&](int s) { return 1.2 * tp / rate[s / 4 - 1] + 13.0 + 7.0 * std::max(0.0, pieces / (8.0 * s) - 1.0); };
    for (int s = 4; s < 32; s += 4)
        if (shared_us(s) <= (tiles ? 0.9 * end + 5.0 : end)) return std::max(s, 5);
    // the shared block decides: the most CUs that leave enough for the suffix meanwhile
    for (int s = 28; s > 16; s -= 4)
        if (ts <= 1.3 * (32 - s) / 32.0 * shared_us(s)) return s;
    return 16;
}

// Gives context c its counters on its device (current), if there are any left.
void take_counters(hg_ctx* c) {
    c->counters = nullptr;
    c->counter_slot = -1;
    if (c->device < 0 || c->device >= 64) return;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    CounterPool*& pool = g_counters[c->device];
    if (!pool) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(context_counters)) != hipSuccess || !p) return;
        pool = new (std::nothrow) CounterPool();
        if (!pool) return;
        pool->base = static_cast<unsigned*>(p);
    }
    if (pool->fresh < kCounterSlots) {
        c->counter_slot = pool->fresh++;
    } else {
        // (an event query is allowed while some stream of the process is being captured, but not in the strictest mode)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        for (int i = 0; i < pool->n_back && c->counter_slot < 0; ++i) {
            const hipEvent_t done = pool->back[i].done;
            if (done) {
                if (hipEventQuery(done) != hipSuccess) {
                    (void)hipGetLastError();      // not ready: not an error of anybody's
                    continue;
                }
                (void)hipEventDestroy(done);
            }
            c->counter_slot = pool->back[i].slot;
            --pool->n_back;
            for (int k = i; k < pool->n_back; ++k) pool->back[k] = pool->back[k + 1];
        }
        (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
    if (c->counter_slot >= 0) c->counters = pool->base + (size_t)c->counter_slot * kContextCounters;
}

bool is_capturing(hipStream_t s) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return true;
}

// To be called for every call that uses the counters, before its launch.
void use_counters(hg_ctx* c) {
    c->counters_used = true;
    c->counter_stream = c->stream;
    if (!c->counters_in_graph && is_capturing(c->stream)) c->counters_in_graph = true;
}

void give_back_counters(hg_ctx* c) {
    if (c->counter_slot < 0 || c->counters_in_graph) return;
    hipEvent_t done = nullptr;
    if (c->counters_used) {
        if (!c->ev_fork || is_capturing(c->counter_stream) || hipEventRecord(c->ev_fork, c->counter_stream) != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        done = c->ev_fork;
        c->ev_fork = nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    CounterPool* const pool = g_counters[c->device];
    pool->back[pool->n_back].slot = c->counter_slot;
    pool->back[pool->n_back++].done = done;
}

int fill_empty(void* O, int o_dtype, float* LSE, int64_t rows, int D, hipStream_t s) {
    FillArgs f{};
    f.O = O; f.LSE = LSE; f.bf16 = (o_dtype == HG_BF16); f.rows = rows; f.D = D;
    return hip_rc(launch_fill_empty(f, s));
}

}  // namespace

extern "C" {

int hg_create(hg_ctx** out, int device, void* hip_stream, void* workspace, size_t workspace_bytes) {
    if (!out) return HG_ERR_INVALID_ARG;
    *out = nullptr;
    if (workspace_bytes && !workspace) return HG_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return HG_ERR_INVALID_ARG;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || device < 0 || device >= ndev) return HG_ERR_HIP;
    if (hipSetDevice(device) != hipSuccess) return HG_ERR_HIP;
    if (device < 64) {
        // this device's copy of the static scratch array (hg_hydragen_attn_static); the device is current here
        std::lock_guard<std::mutex> lock(g_scratch_mu);
        if (!g_scratch_ptr[device]) {
            void* p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return HG_ERR_HIP;
            g_scratch_ptr[device] = static_cast<unsigned char*>(p);
        }
    }
    hg_ctx* c = new (std::nothrow) hg_ctx();
    if (!c) return HG_ERR_HIP;
    c->counter_slot = -1;
    c->device = device;
    c->stream = static_cast<hipStream_t>(hip_stream);
    c->ws = static_cast<unsigned char*>(workspace);
    c->ws_bytes = workspace_bytes;
    c->opt_prefix_splits = c->opt_suffix_chunk = c->opt_overlap = c->opt_naive_chunk = c->opt_prefix_kernel = c->opt_wide_slots = 0;
    c->opt_nq = 1;
    c->opt_suffix_kernel = 0;
    c->opt_suffix_ipw = 0;
    c->opt_suffix_tile = 0;
    c->opt_fused_kernel = 0;
    c->aux = nullptr;
    c->ev_fork = c->ev_join = nullptr;
    c->opt_timing = 0;
    c->tev = nullptr;
    c->tused = nullptr;
    c->tcalls = 0;
    if (hipStreamCreateWithFlags(&c->aux, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming) != hipSuccess) {
        hg_destroy(c);
        return HG_ERR_HIP;
    }
    take_counters(c);
    *out = c;
    return HG_OK;
}

void hg_destroy(hg_ctx* c) {
    if (!c) return;
    give_back_counters(c);
    if (c->ev_fork) (void)hipEventDestroy(c->ev_fork);
    if (c->ev_join) (void)hipEventDestroy(c->ev_join);
    if (c->aux) (void)hipStreamDestroy(c->aux);
    if (c->tev) {
        for (int i = 0; i < HG_TIMING_RING * HG_MAX_STAGES * 2; ++i)
            if (c->tev[i]) (void)hipEventDestroy(c->tev[i]);
        delete[] c->tev;
    }
    delete[] c->tused;
    delete c;
}

int hg_set_stream(hg_ctx* c, void* hip_stream) {
    if (!c) return HG_ERR_INVALID_ARG;
    c->stream = static_cast<hipStream_t>(hip_stream);
    return HG_OK;
}

int hg_set_option(hg_ctx* c, int option, int value) {
    if (!c || value < 0) return HG_ERR_INVALID_ARG;
    switch (option) {
        case HG_OPT_PREFIX_SPLITS: c->opt_prefix_splits = value; return HG_OK;
        case HG_OPT_SUFFIX_CHUNK: c->opt_suffix_chunk = value; return HG_OK;
        case HG_OPT_OVERLAP:
            if (value > 2) return HG_ERR_INVALID_ARG;
            c->opt_overlap = value;
            return HG_OK;
        case HG_OPT_NAIVE_CHUNK: c->opt_naive_chunk = value; return HG_OK;
        case HG_OPT_PREFIX_KERNEL:
            if (value > 2) return HG_ERR_INVALID_ARG;
            c->opt_prefix_kernel = value;
            return HG_OK;
        case HG_OPT_NUM_QUERIES:
            if (value < 1 || value > 64) return HG_ERR_INVALID_ARG;
            c->opt_nq = value;
            return HG_OK;
        case HG_OPT_SUFFIX_KERNEL:
            if (value > 2) return HG_ERR_INVALID_ARG;
            c->opt_suffix_kernel = value;
            return HG_OK;
        case HG_OPT_SUFFIX_ITEMS_PER_WAVE:
            if (value > 1024) return HG_ERR_INVALID_ARG;
            c->opt_suffix_ipw = value;
            return HG_OK;
        case HG_OPT_SUFFIX_TILE_ROWS:
            if (value != 0 && value != 16 && value != 32) return HG_ERR_INVALID_ARG;
            c->opt_suffix_tile = value;
            return HG_OK;
        case HG_OPT_FUSED_KERNEL:
            if (value > 2) return HG_ERR_INVALID_ARG;
            c->opt_fused_kernel = value;
            return HG_OK;
        case HG_OPT_WIDE_SLOTS:
            if (value > 32) return HG_ERR_INVALID_ARG;
            c->opt_wide_slots = value;
            return HG_OK;
        case HG_OPT_STAGE_TIMING:
            if (value && !c->tev) {
                if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
                const int n = HG_TIMING_RING * HG_MAX_STAGES * 2;
                c->tev = new (std::nothrow) hipEvent_t[n]();
                c->tused = new (std::nothrow) unsigned char[HG_TIMING_RING * HG_MAX_STAGES]();
                if (!c->tev || !c->tused) return HG_ERR_HIP;
                for (int i = 0; i < n; ++i)
                    if (hipEventCreate(&c->tev[i]) != hipSuccess) return HG_ERR_HIP;
            }
            c->opt_timing = value ? 1 : 0;
            c->tcalls = 0;
            return HG_OK;
    }
    return HG_ERR_INVALID_ARG;
}

size_t hg_workspace_bytes(int B, int Hq, int D, int parts) {
    if (B <= 0 || Hq <= 0 || D <= 0 || parts <= 0) return 0;
    const size_t n = (size_t)parts * (size_t)B * Hq * (size_t)(D + 1) * sizeof(float);
    return (n + 255) / 256 * 256;
}

int hg_prefix_attn_grouped(hg_ctx* c, const void* Q, const hg_level* level, int B, int Hq, int Hkv, int D, float scale,
                           void* O, int o_dtype, float* LSE) {
    if (!c || !O || !LSE || (o_dtype != HG_F32 && o_dtype != HG_BF16)) return HG_ERR_INVALID_ARG;
    int rc = check_shape(B, Hq, Hkv, D, c ? c->opt_nq : 1);
    if (rc) return rc;
    rc = check_level(level, Hkv, D);
    if (rc) return rc;
    if (B == 0) return HG_OK;
    if (!Q) return HG_ERR_INVALID_ARG;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    scale = eff_scale(scale, D);
    const int nq = c->opt_nq;
    const int64_t rows = (int64_t)B * nq * Hq;
    const LevelDev lv = to_dev(*level, B);
    const Parts parts = carve(Ws{c->ws, c->ws_bytes}, rows, D);
    const LevelPlan plan = plan_level(c, lv, Hkv, nq * (Hq / Hkv), D, parts.cap);
    const int ns = plan.ns;
    hipStream_t s = c->stream;
    if (lv.max_rows == 0 || lv.max_seqs == 0) return fill_empty(O, o_dtype, LSE, rows, D, s);
    if (!plan.wide && (int64_t)lv.n_blocks * ns * Hkv * ceil_div(lv.max_seqs * nq * (Hq / Hkv), kPrefixRowsNarrow) >= (1LL << 28))
        return HG_ERR_UNSUPPORTED;      // (checked before anything is enqueued)
    // (sequences that no block covers are given their empty result by the level's kernel itself)
    if (ns == 1) return run_level(Q, lv, plan, B, nq, Hq, Hkv, D, scale, direct_out(O, o_dtype, LSE), s);
    rc = run_level(Q, lv, plan, B, nq, Hq, Hkv, D, scale, parts_out(parts, 0), s);
    if (rc) return rc;
    return run_merge(ns, parts, 0, D, O, o_dtype, LSE, s);
}

int hg_prefix_attn(hg_ctx* c, const void* Q, const void* Kp, const void* Vp, int B, int Hq, int Hkv, int D, int P,
                   float scale, void* O, int o_dtype, float* LSE) {
    if (P < 0) return HG_ERR_INVALID_ARG;
    hg_level lv{};
    lv.K = Kp; lv.V = Vp; lv.n_blocks = 1; lv.kv_off = nullptr; lv.seq_off = nullptr; lv.max_rows = P; lv.max_seqs = B;
    return hg_prefix_attn_grouped(c, Q, &lv, B, Hq, Hkv, D, scale, O, o_dtype, LSE);
}

// hg_suffix_attn and hg_suffix_attn_paged (pg.table set, offsets unused)
static int suffix_impl(hg_ctx* c, const void* Q, const void* Ks, const void* Vs, const int32_t* offsets,
                       const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D, float scale, void* O, int o_dtype,
                       float* LSE, const hg::PagedDev& pg, bool paged, const KvFmt& fmt = KvFmt{}) {
    if (!c || !O || !LSE || (o_dtype != HG_F32 && o_dtype != HG_BF16) || max_len < 0) return HG_ERR_INVALID_ARG;
    int rc = check_shape(B, Hq, Hkv, D, c ? c->opt_nq : 1);
    if (rc) return rc;
    rc = check_suffix_span(max_len, Hkv, D);
    if (rc) return rc;
    if (B == 0) return HG_OK;
    if (!Q || (!offsets && !paged) || !lengths) return HG_ERR_INVALID_ARG;
    if (max_len > 0 && (!Ks || !Vs)) return HG_ERR_INVALID_ARG;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    scale = eff_scale(scale, D);
    const int nq = c->opt_nq;
    const int64_t rows = (int64_t)B * nq * Hq;
    hipStream_t s = c->stream;
    if (max_len == 0) return fill_empty(O, o_dtype, LSE, rows, D, s);
    const Parts parts = carve(Ws{c->ws, c->ws_bytes}, rows, D);
    const int max_chunk = pg.table ? 32 << pg.shift : 1 << 30;
    SuffixPlan p = plan_suffix(c, max_len, Hq / Hkv, B, nq, Hkv, D, pg.table != nullptr, max_chunk, fmt.fp8 != 0);
    if (p.nchunks > parts.cap) {  // not enough room for partials: fewer, longer chunks
        p.nchunks = parts.cap > 1 ? parts.cap : 1;
        p.chunk = round_up(ceil_div(max_len, p.nchunks), 32);
        p.nchunks = ceil_div(max_len, p.chunk);
    }
    if (!p.mfma && p.chunk > max_chunk) return HG_ERR_WORKSPACE;
    if (p.nchunks == 1)
        return run_decode(Q, 0, nullptr, Ks, Vs, offsets, lengths, max_len, B, nq, Hq, Hkv, D, scale, p.chunk, 1, p.gt,
                          direct_out(O, o_dtype, LSE), s, pg, p.mfma, p.ipw, false, fmt, c->opt_suffix_tile);
    rc = run_decode(Q, 0, nullptr, Ks, Vs, offsets, lengths, max_len, B, nq, Hq, Hkv, D, scale, p.chunk, p.nchunks, p.gt,
                    parts_out(parts, 0), s, pg, p.mfma, p.ipw, false, fmt, c->opt_suffix_tile);
    if (rc) return rc;
    return run_merge(p.nchunks, parts, 0, D, O, o_dtype, LSE, s);
}

// scales of an 8-bit cache: finite and positive
static bool fp8_fmt(float k_scale, float v_scale, KvFmt* out) {
    if (!(k_scale > 0.f) || !(v_scale > 0.f) || k_scale > 3.0e38f || v_scale > 3.0e38f) return false;
    out->fp8 = 1;
    out->k_scale = k_scale;
    out->v_scale = v_scale;
    return true;
}

// checks an hg_paged_kv against the rows it must be able to address and translates it
static int paged_dev(const hg_paged_kv* kv, int rows_per_seq, int Hkv, int D, hg::PagedDev* out, KvFmt* fmt) {
    if (!kv || !out || !fmt) return HG_ERR_INVALID_ARG;
    *fmt = KvFmt{};
    if (kv->kv_format == HG_KV_E4M3) {
        if (!fp8_fmt(kv->k_scale, kv->v_scale, fmt)) return HG_ERR_INVALID_ARG;
    } else if (kv->kv_format != HG_KV_BF16) {
        return HG_ERR_INVALID_ARG;
    }
    int shift = 0;
    while ((1 << shift) < kv->page_size && shift < 11) ++shift;
    if (kv->page_size < 16 || kv->page_size > 1024 || (1 << shift) != kv->page_size) return HG_ERR_INVALID_ARG;
    if (kv->n_pages < 0 || kv->table_stride < 0) return HG_ERR_INVALID_ARG;
    if ((int64_t)kv->n_pages * kv->page_size * Hkv * D >= (1LL << 31)) return HG_ERR_UNSUPPORTED;
    if (rows_per_seq > 0) {
        if (!kv->K || !kv->V || !kv->page_table || kv->n_pages < 1) return HG_ERR_INVALID_ARG;
        if ((int64_t)kv->table_stride * kv->page_size < rows_per_seq) return HG_ERR_INVALID_ARG;
    }
    out->table = kv->page_table;
    out->shift = shift;
    out->stride = kv->table_stride;
    out->n_pages = kv->n_pages;
    return HG_OK;
}

int hg_suffix_attn(hg_ctx* c, const void* Q, const void* Ks, const void* Vs, const int32_t* offsets,
                   const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D, float scale, void* O, int o_dtype,
                   float* LSE) {
    return suffix_impl(c, Q, Ks, Vs, offsets, lengths, max_len, B, Hq, Hkv, D, scale, O, o_dtype, LSE, hg::PagedDev{}, false);
}

int hg_suffix_attn_paged(hg_ctx* c, const void* Q, const hg_paged_kv* kv, const int32_t* lengths, int max_len, int B,
                         int Hq, int Hkv, int D, float scale, void* O, int o_dtype, float* LSE) {
    if (max_len < 0 || Hkv <= 0 || (D != 64 && D != 128)) return HG_ERR_INVALID_ARG;
    hg::PagedDev pg{};
    KvFmt fmt;
    const int rc = paged_dev(kv, max_len, Hkv, D, &pg, &fmt);
    if (rc) return rc;
    return suffix_impl(c, Q, kv->K, kv->V, nullptr, lengths, max_len, B, Hq, Hkv, D, scale, O, o_dtype, LSE, pg, true, fmt);
}

int hg_merge(hg_ctx* c, int n, const void* const* O_parts, const float* const* LSE_parts, int o_dtype_in, int64_t rows,
             int D, void* O_out, int o_dtype_out, float* LSE_out) {
    if (!c || n < 1 || n > HG_MAX_PARTS || !O_parts || !LSE_parts || rows < 0 || !O_out) return HG_ERR_INVALID_ARG;
    if ((o_dtype_in != HG_F32 && o_dtype_in != HG_BF16) || (o_dtype_out != HG_F32 && o_dtype_out != HG_BF16))
        return HG_ERR_INVALID_ARG;
    if (D != 64 && D != 128) return HG_ERR_UNSUPPORTED;
    for (int i = 0; i < n; ++i)
        if (!O_parts[i] || !LSE_parts[i]) return HG_ERR_INVALID_ARG;
    if (rows == 0) return HG_OK;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    hg::MergeArgs m{};
    m.n = n;
    for (int i = 0; i < n; ++i) {
        m.O[i] = O_parts[i];
        m.L[i] = LSE_parts[i];
    }
    m.rows = rows;
    m.O_out = O_out;
    m.L_out = LSE_out;
    return hip_rc(hg::launch_merge(m, D, o_dtype_in == HG_BF16, o_dtype_out == HG_BF16, c->stream));
}

static int check_fused(hg_ctx* c, const void* Q, int n_levels, const hg_level* levels, const void* Ks, const void* Vs,
                       const int32_t* offsets, const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D,
                       void* O_out, int o_dtype, bool paged = false) {
    if (!c || !O_out || (o_dtype != HG_F32 && o_dtype != HG_BF16) || max_len < 0) return HG_ERR_INVALID_ARG;
    if (n_levels < 0 || n_levels > HG_MAX_LEVELS || (n_levels > 0 && !levels)) return HG_ERR_INVALID_ARG;
    int rc = check_shape(B, Hq, Hkv, D, c ? c->opt_nq : 1);
    if (rc) return rc;
    for (int i = 0; i < n_levels; ++i) {
        rc = check_level(&levels[i], Hkv, D);
        if (rc) return rc;
    }
    if (B > 0 && !Q) return HG_ERR_INVALID_ARG;
    if (Ks && max_len > 0 && (!Vs || (!offsets && !paged) || !lengths)) return HG_ERR_INVALID_ARG;
    if (Ks) {
        rc = check_suffix_span(max_len, Hkv, D);
        if (rc) return rc;
    }
    return HG_OK;
}

// How a fused call runs: everything that is decided from host values (shapes, options, room for partial results).
enum { kWaySingle = 0, kWayCombined = 1, kWayOneStream = 2, kWayTwoStreams = 3, kWayFill = 4 };
struct FusedPlan {
    int way;
    int splits;                     // single launch: workgroups per column
    int column_rows;                // and query rows
    int wavefronts;                 // of a workgroup
    bool dealt;                     // its stages go to the wavefronts one by one
    bool sfx_mfma;                  // the suffix kernel's choice for these rows is the matrix cores
    int nlev;                       // levels that hold keys
    LevelDev lv[HG_MAX_LEVELS];
    LevelPlan plan[HG_MAX_LEVELS];
    int ns[HG_MAX_LEVELS], index[HG_MAX_LEVELS];      // partial results of a level, its place in the caller's list
    int main_level, joint;          // the level with the most work (caller's list); combined launch: the level it is launched for
    SuffixPlan sp;
    int np;                         // partial results altogether
    bool tiny;                      // so little work that the event edges between two streams cost more than overlap can gain
};
// What a fused call is asked to do, as far as the host knows it.
struct FusedShape {
    int n_levels;
    const hg_level* levels;
    bool has_suffix;
    int max_len;
    int page_shift;                 // -1: packed rows
    bool fp8;
    float v_scale;
    bool wants_lse;
    int B, Hq, Hkv, D;
    size_t ws_bytes;                // room for partial results
    bool counters;                  // the context has its device counters
};

constexpr int kCombinedRows = 64;      // in the combined launch levels of more query rows run on the persistent kernel

// Parts per level and for the suffix, shrunk to fit the workspace: for the combined launch, or for separate kernels.
static int plan_parts(const hg_ctx* c, const FusedShape& f, bool combine, FusedPlan& p) {
    const int n_levels = f.n_levels, max_len = f.max_len, B = f.B, Hq = f.Hq, Hkv = f.Hkv, D = f.D, nq = c->opt_nq, G = Hq / Hkv;
    const hg_level* const levels = f.levels;
    const bool has_suffix = f.has_suffix, paged = f.page_shift >= 0, sfx_mfma = p.sfx_mfma;
    const int cap = parts_cap(f.ws_bytes, (int64_t)B * nq * Hq, D);
    LevelDev* const lv = p.lv;
    LevelPlan* const plan = p.plan;
    int *const ns = p.ns, *const index = p.index;
    int &nlev = p.nlev, &main_level = p.main_level;
    nlev = 0;
    main_level = -1;
    for (int i = 0; i < n_levels; ++i) {
        const double seqs = levels[i].kv_off ? levels[i].max_seqs : B;
        if (main_level < 0 || (double)levels[i].max_rows * levels[i].n_blocks * seqs >
                                  (double)levels[main_level].max_rows * levels[main_level].n_blocks * (levels[main_level].kv_off ? levels[main_level].max_seqs : B))
            main_level = i;
    }
    // In the combined launch levels of more than 64 query rows run on the persistent kernel as well: it costs no launch of its
    // own there.  Only the level with the most work may use the plan with a table.
    // (A number of splits is asked of the 128-row kernel.)
    const int wide_above = combine && c->opt_prefix_splits == 0 ? kCombinedRows : kPrefixRowsNarrow;
    int wide_slots = 32;
    bool& tiny = p.tiny;
    tiny = false;
    if (has_suffix && c->opt_overlap != 1) {
        double flops = 0.0;
        int T = 1;
        double pieces = 0.0, padded = 0.0;     // 256-row tiles of all levels, blocks and KV heads; flops with whole tiles
        for (int i = 0; i < n_levels; ++i) {
            const long long seqs = levels[i].kv_off ? levels[i].max_seqs : B;
            flops += 4.0 * levels[i].n_blocks * (double)levels[i].max_rows * seqs * nq * Hq * D;
            const long long tiles = (seqs * nq * G + kPrefixRowsWide - 1) / kPrefixRowsWide;
            if (seqs * nq * G > kPrefixRowsNarrow && tiles <= 32 && tiles > T) T = (int)tiles;
            if (levels[i].max_rows > 0 && seqs * nq * G > wide_above) {
                pieces += (double)tiles * levels[i].n_blocks * Hkv;
                padded += 4.0 * levels[i].n_blocks * (double)levels[i].max_rows * tiles * kPrefixRowsWide * Hkv * D;
            }
        }
        // K and V, bf16 (or 8-bit codes; on the matrix cores their expansion costs about a third of the saving); the
        // vector-ALU kernel reads them once per query; mean length taken as 0.75 max_len
        const double per_elem = f.fp8 ? (sfx_mfma ? 2.6 : 2.0) : 4.0;
        const double bytes = per_elem * B * (sfx_mfma ? 1 : nq) * (0.75 * max_len) * Hkv * D;
        wide_slots = pick_wide_slots(flops, bytes, T);
        tiny = c->opt_overlap == 0 && flops / 1.14e15 + bytes / 6.0e12 < 60e-6;
        if (tiny) wide_slots = 32;
        if (combine) wide_slots = pick_combined_slots(padded, 0.8 * bytes, pieces, D, sfx_mfma);     // (here the mean is taken as 0.6 max_len)
    }
    for (int i = 0; i < n_levels; ++i) {
        LevelDev d = to_dev(levels[i], B);
        if (d.max_rows == 0 || d.max_seqs == 0) continue;  // empty level contributes nothing
        lv[nlev] = d;
        index[nlev] = i;
        plan[nlev] = plan_level(c, d, Hkv, nq * G, D, cap, wide_slots, wide_above, !combine || i == main_level);
        ns[nlev] = plan[nlev].ns;
        ++nlev;
    }
    const int max_chunk = paged ? 32 << f.page_shift : 1 << 30;
    SuffixPlan& sp = p.sp;
    sp = plan_suffix(c, max_len, G, B, nq, Hkv, D, paged, max_chunk, f.fp8);
    // (the combined launch has 2048 wavefronts: items for all of them, equal shares of the longest suffix)
    if (combine && sp.mfma && c->opt_suffix_chunk == 0) {
        const long long whole = (long long)B * Hkv * ceil_div(nq * G, 32);
        const int n = (int)std::min<long long>({(2047 + whole) / whole, 4, std::max(1, max_len / 128)});
        if (n > sp.nchunks) {
            sp.chunk = round_up(ceil_div(max_len, n), 32);
            sp.nchunks = ceil_div(max_len, sp.chunk);
        }
    }
    if (!has_suffix) sp.nchunks = 0;
    auto total_parts = [&]() { int t = sp.nchunks; for (int i = 0; i < nlev; ++i) t += ns[i]; return t; };
    if (nlev + (has_suffix ? 1 : 0) > cap) return HG_ERR_WORKSPACE;
    while (total_parts() > cap) {  // shrink the largest split count first
        int big = -1, bigv = 1;
        for (int i = 0; i < nlev; ++i) if (ns[i] > bigv) { bigv = ns[i]; big = i; }
        if (sp.nchunks > bigv) {
            sp.nchunks -= 1;
            sp.chunk = round_up(ceil_div(max_len, sp.nchunks), 32);
            sp.nchunks = ceil_div(max_len, sp.chunk);
        } else if (big >= 0) {
            plan[big] = plan_level(c, lv[big], Hkv, nq * G, D, ns[big] - 1, wide_slots, wide_above, !combine || index[big] == main_level);
            ns[big] = plan[big].ns;
        } else {
            return HG_ERR_WORKSPACE;
        }
    }
    if (has_suffix && !sp.mfma && sp.chunk > max_chunk) return HG_ERR_WORKSPACE;
    // every size limit of the launches below is checked here, before anything is enqueued
    for (int i = 0; i < nlev; ++i) {
        if (plan[i].wide) continue;
        const int64_t tiles = (int64_t)lv[i].n_blocks * ns[i] * Hkv * ceil_div(lv[i].max_seqs * nq * G, kPrefixRowsNarrow);
        if (tiles >= (1LL << 28)) return HG_ERR_UNSUPPORTED;
    }
    if (has_suffix && sp.mfma) {
        const int tile_rows = (nq * G <= 16 && c->opt_suffix_tile != 32) ? 16 : 32;
        if ((int64_t)B * sp.nchunks * ceil_div(nq * G, tile_rows) * Hkv >= (1LL << 31)) return HG_ERR_UNSUPPORTED;
    }
    p.np = total_parts();
    return HG_OK;
}

static int plan_fused(const hg_ctx* c, const FusedShape& f, FusedPlan* out) {
    FusedPlan& p = *out;
    p.way = kWaySingle;
    p.splits = 1;
    p.column_rows = 32;
    p.wavefronts = 8;
    p.dealt = true;
    p.nlev = 0;
    p.main_level = p.joint = -1;
    const int n_levels = f.n_levels, max_len = f.max_len, B = f.B, Hq = f.Hq, Hkv = f.Hkv, D = f.D, nq = c->opt_nq, G = Hq / Hkv;
    const hg_level* const levels = f.levels;
    const bool has_suffix = f.has_suffix, paged = f.page_shift >= 0;

    const SuffixPlan alone = plan_suffix(c, max_len, G, B, nq, Hkv, D, paged, 1 << 30, f.fp8);      // the suffix on a kernel of its own
    const bool sfx_mfma = p.sfx_mfma = alone.mfma;

    // One row per KV head on the vector ALU: an item that short is over before the eight wavefronts of a CU have covered its
    // fixed price (its query, its result, the next item's look-up), where the suffix kernel has twenty.  Combined / separate, us:
    // 179 x 40 heads, 11K keys, 23 rows 106 / 98; 1554 x 40, D = 64, 4521 keys, 29 rows 188 / 210; 286 x 40, 6168 keys, 46 rows
    // 103 / 125; 8-bit: 832 x 40, D = 64, 71 rows 86 / 72; 1802 x 40, 2268 keys, 36 rows 240 / 216; 130 x 40, 4307 keys, 104 rows
    // 67 / 72.  Over some 120 drawn calls, separate / combined in the mean: packed bf16 0.94 (D = 64) and 1.02 at 16 to 23 rows, 1.04 and
    // 1.07 from 24 on; codes 0.80 below 24 rows, 0.93 at 40 to 47, level from 48 on; at D = 64 0.85 to 0.97 up to 79.
    // A caller that sets the CUs of the shared block has asked for the two side by side.
    const int combine_rows = !f.fp8 ? 24 : D == 128 ? 48 : 80;

    // Shared block and suffix in one launch (combined_impl.h): calls with a level on the persistent kernel and a suffix on the
    // matrix cores or with one query row per KV head.  The stage timings need separate kernels, items per wavefront the suffix kernel.
    // (8-bit codes in 32-row tiles stay on separate kernels: half the bytes in flight per wavefront do not cover the longer
    // stage; 215 sequences, 64/8 heads, 4 queries: 83 against 76 us.)
    const bool long_enough = sfx_mfma || c->opt_wide_slots > 0 || max_len >= combine_rows;
    const bool may_join = c->opt_overlap == 0 && c->opt_suffix_ipw == 0 && !c->opt_timing && has_suffix && f.counters && !(f.fp8 && (nq * G > 16 || c->opt_suffix_tile == 32)) &&
                          (sfx_mfma || (nq == 1 && G == 1));
    const bool may_combine = may_join && long_enough;

    // One launch for everything when that is the faster way (fused_small.hip): `splits` workgroups of eight wavefronts, or one of four, per
    // column of 32 or 16 query rows walk every shared block and the column's suffixes and merge, against one launch per part or for both,
    // two event edges and a round trip of the partial results through HBM for the other ways.  Both durations are
    // estimated, in microseconds, from fits to 2070 drawn calls of up to 260 us (B = 4 .. 2048, 0 .. 16K shared keys, every cache, each timed in
    // both ways, with 16 and 32 rows, with up to 30 workgroups per column and with four wavefronts; error of an estimate 13 %, of 4 wavefronts
    // and of the other ways 17 %); constants below:
    //   single launch, eight wavefronts: rounds x (b + c x stages per wavefront), where workgroups share a CU longer, and more for 8-bit rows with
    //                  fp32 weights; m0 + m1 x splits when a column's workgroups have to meet.
    //   four:          (columns per place + tail) x (b + c x stages per wavefront), shared and suffix stages by their own.
    //                  Both with the time in which the suffix rows stream in: the third root of the sum of cubes.
    //   the other way: a launch price for each shared level, the longer of suffix and shared blocks and a part of the shorter, partial results.
    // 16 rows: half the products and exponentials per stage and fewer sequences' suffixes per column, but twice the columns, each
    // reading the shared rows for itself: they win while there are CUs for them.  Measured 32 / 16 rows: 13.2 / 10.0 us (45 x 16/2
    // heads, 515 keys), 15.9 / 12.0 (256 x 8/1, 1K keys), 11.3 / 8.8 (95 x 16/2, two queries), 44.5 / 61 (139 x 64/8, four queries),
    // 27.2 / 31 (60 x 16/2, 3K keys, three workgroups per column).
    // Four wavefronts: half the LDS, so two columns share a CU (at D = 64 four, of 32 rows with fp32 weights three, by their registers; the price takes three) and one's prologue and combination run beside
    // the other's stages.  A column takes longer: for calls with more columns than CUs and few stages to a column.  Eight / four wavefronts, and the other
    // way, us: 683 x 64/8 heads, 549 keys, four queries 222 / 167, 199; 1965 x 64/8, 1294 + 16 x 115 keys 223 / 193, 225; 215 x 64/8, 553 keys, four
    // queries, codes 79 / 62, 76; 57 x 64/8, 342 + 3 x 297 keys, four queries 21.7 / 15.7, 22; 256 x 64/8, 4K keys, four queries 247 / 232, 185 (not taken).
    // The host knows only an upper bound of the suffix lengths; both estimates take 0.75 of it as the mean.  The single launch is
    // taken below 1.2 of the other estimate up to 36 us, beyond with a tenth of the suffix time to spare (long rows are where it disappoints); a suffix alone up to 15 us,
    // and below 0.8 where one row per KV head goes straight from its kernel to the outputs (414 x 4 heads, 47 rows 20 against 15 us), or by the price of its work items.
    // The estimates' errors are as large as most differences between the ways: of 14000 drawn calls 1168 go another way than with the constants of before (fitted when a
    // column's workgroups met in 2 us more and its prologue took 1) and without four wavefronts; of 1000 of these, timed, 695 are by more than a tenth faster, 43 slower, 1.24
    // times as fast in the mean.  Finer estimates (the suffix at its true mean, every part priced, errors of 8 to 11 %) chose no better with the mean unknown.
    // (the single launch divides sums by the V scale and multiplies them again: not with scales near the ends of fp32)
    const bool odd_scale = f.fp8 && has_suffix && !(f.v_scale >= 0x1p-60f && f.v_scale <= 0x1p60f);
    bool take_single = false;
    if (c->opt_fused_kernel != 1 && !c->opt_timing && !odd_scale) {
        const int rps = nq * G;
        const bool fp32_weights = f.fp8 && has_suffix && !sfx_mfma;
        long long shared_keys = 0;
        double flops = 0.0, padded = 0.0, shared_bytes = 0.0;      // padded: flops with whole 256-row tiles
        // wide: a level runs on the persistent kernel otherwise
        bool any = has_suffix, wide = false;
        int nonempty = 0;
        for (int i = 0; i < n_levels; ++i) {
            const long long seqs = levels[i].kv_off ? levels[i].max_seqs : B;
            if (levels[i].max_rows > 0 && seqs > 0) {
                shared_keys += levels[i].max_rows;
                flops += 4.0 * levels[i].n_blocks * (double)levels[i].max_rows * seqs * nq * Hq * D;
                padded += 4.0 * levels[i].n_blocks * (double)levels[i].max_rows * ((seqs * rps + kPrefixRowsWide - 1) / kPrefixRowsWide * kPrefixRowsWide) * Hkv * D;
                shared_bytes += 4.0 * levels[i].n_blocks * (double)levels[i].max_rows * Hkv * D;
                any = true;
                wide = wide || seqs * rps > kPrefixRowsNarrow;
                ++nonempty;
            }
        }
        // Shared rows that neither their XCD's L2 (4 MB) nor, with the suffix rows and another layer's, the 256 MB behind all of them hold: a stage takes
        // half as long again (from five workgroups per column on the waits overlap).  109 x 40/40 heads, D = 64, 7168 keys, 160 columns: 32 suffix rows 45.8 us, 68 rows 76 (separate kernels 48); 64 keys only 11.7
        // and 22; 32 x 40/40, 4K / 8K keys 1.9 / 3.0 us a stage.
        const bool far = shared_bytes / std::min(8, Hkv) > 4.0e6 && shared_bytes + (has_suffix ? (f.fp8 ? 2.0 : 4.0) * B * (0.75 * max_len) * Hkv * D : 0.0) > 1.25e8;
        struct Shape { int seqs_per_tile; long long cols; double stages, shared; };      // of columns of so many rows
        auto shape_of = [&](int rows) {
            Shape x;
            x.seqs_per_tile = rps >= rows ? 1 : (rows + rps - 1) / rps + (rows % rps ? 1 : 0);
            x.cols = ((long long)B * rps + rows - 1) / rows * Hkv;
            double shared_stages = 0.0;
            for (int i = 0; i < n_levels; ++i) {
                const long long seqs = levels[i].kv_off ? levels[i].max_seqs : B;
                if (levels[i].max_rows <= 0 || seqs <= 0) continue;
                // blocks that a column meets: all of a small block's neighbours as well
                const double met = std::min((double)levels[i].n_blocks, levels[i].n_blocks > 1 ? 1.0 + (rows - 1.0) / (double)(seqs * rps) : 1.0);
                shared_stages += met * ((levels[i].max_rows + 31) / 32);
            }
            x.shared = shared_stages;
            x.stages = shared_stages + (has_suffix ? std::min(x.seqs_per_tile, B) * ((0.75 * max_len + 16.0) / 32.0) : 0.0);
            return x;
        };
        const Shape shape32 = shape_of(32), shape16 = shape_of(16);
        const long long cols = shape32.cols;
        const int seqs_per_tile = shape32.seqs_per_tile;
        // Workgroups of eight wavefronts that run at a time: one per CU, at D = 64 two (LDS; of 32 rows with fp32 weights one, by their registers, which the constants below have taken in), which take longer then: 112 x 40/40 heads, 8K keys: 48 us with 160
        // columns of 32 rows, 66 with 280 of 16 rows (45 with 160 of them).
        auto rounds_of = [&](double wgs) { return ceil(wgs / (D == 128 ? 256.0 : 512.0)); };
        struct Eight { double b, c, m0, m1, fp32_weights, sharing, rounds, paged, packed; };      // (paged, packed: of the suffix rows' time at 5 TB/s)
        struct Four { double b, c, more, c_suffix, fp32_weights, tail, paged, packed; };
        static const Eight eight[2][2] = {      // [D = 64][16 rows]
            {{4.9, 1.58, 1.64, 0.35, 1.40, 1.0, 1.0, 1.04, 0.80}, {3.2, 1.43, 1.81, 0.09, 1.30, 1.0, 1.0, 0.92, 0.74}},
            {{3.2, 1.04, 1.58, 0.09, 1.70, 1.74, 1.51, 1.25, 0.83}, {2.6, 0.88, 1.37, 0.07, 1.54, 1.43, 1.19, 1.07, 0.83}}};
        static const Four four[2][2] = {
            {{5.5, 1.01, 0.48, 1.53, 1.26, 0.44, 0.83, 0.67}, {3.5, 0.91, 0.50, 1.72, 1.17, 0.25, 0.80, 0.65}},
            {{3.3, 0.84, 0.35, 1.09, 1.42, 0.38, 1.29, 0.93}, {2.2, 0.69, 0.29, 0.90, 1.41, 0.39, 1.22, 0.94}}};
        auto chain_at = [&](int rows, int S) {
            const Eight& k = eight[D == 64][rows == 16];
            const Shape& x = rows == 16 ? shape16 : shape32;
            const double wgs = (double)x.cols * S;
            const double per_stage = (wgs <= 256.0 ? 1.0 : wgs <= 512.0 ? k.sharing : k.rounds) * (fp32_weights ? k.fp32_weights : 1.0) * k.c;
            return rounds_of(wgs) * (k.b + per_stage * ceil((x.stages + (far && S <= 4 ? 0.5 * x.shared : 0.0)) / (8.0 * S))) + (S > 1 ? k.m0 + k.m1 * S : 0.0);
        };
        auto chain_of_four = [&](int rows) {
            const Four& k = four[D == 64][rows == 16];
            const Shape& x = rows == 16 ? shape16 : shape32;
            const double stages = (fp32_weights ? k.fp32_weights : 1.0) * (k.c * x.shared + k.c_suffix * (x.stages - x.shared));
            const double column = k.b + (1.0 + k.more * std::min(1.0, std::max(0.0, (x.cols - 128.0) / 384.0))) * stages / 4.0;
            return column * std::max(1.0, x.cols / (D == 128 ? 512.0 : 768.0) + k.tail);
        };
        // Small calls on packed rows touch nothing but their inputs and outputs: one workgroup per column, no workspace, no
        // counters.  A program may have several in flight for one context (streams, graph replays, branches of a graph) or run
        // them without a workspace, so which calls these are is fixed here and does not follow the estimates.  (Splitting their
        // columns too gained 1 % over 200 drawn calls of this kind, 30 % where few columns meet 2K shared keys.)
        bool own_memory = false;
        if (any && !paged && !f.fp8 && cols < (1LL << 31)) {
            const double suffix = has_suffix ? 4.0 * B * (double)max_len * Hkv * D / 5.0e6 : 0.0;
            const long long walked = (shared_keys + 31) / 32 + (has_suffix ? (long long)seqs_per_tile * ((max_len + 31) / 32) : 0);
            const double walk = 9.0 + (cols <= 128 ? 1.24 : 1.6) * (double)((walked + 3) / 4) * std::max(1.0, cols / 256.0);
            const double one = std::max(walk, suffix * (5.0 / 5.5) + 4.0);
            const double other = 24.0 + 0.75 * suffix + (shared_keys >= 1024 ? 8.0 : 0.0) + flops / 1.1e9;
            own_memory = c->opt_fused_kernel == 2 || (one <= 130.0 && one <= (one <= 40.0 ? 1.0 : 0.9) * other);
        }
        int &splits = p.splits, &rows = p.column_rows;
        // (columns that only the option splits have 32 rows unless 16 are asked for)
        const int asked = c->opt_fused_kernel != 2 ? 0 : c->opt_suffix_tile || own_memory ? c->opt_suffix_tile : 32;
        if (asked == 16 || (asked == 0 && chain_at(16, 1) < chain_at(32, 1))) rows = 16;
        if (!own_memory && f.counters) {
            for (int r : {32, 16}) {
                const Shape& x = r == 16 ? shape16 : shape32;
                if (x.cols * 2 > kSplitWorkgroups || (asked && asked != r)) continue;
                // (more workgroups than one stage per wavefront asks for only meet later)
                const int most = (int)std::min<long long>({kSplitWorkgroups / x.cols, kSmallMaxSplits, (long long)ceil(x.stages / 8.0)});
                for (int S = 2; S <= most; ++S)
                    if (chain_at(r, S) < 0.98 * chain_at(rows, splits) && small_part_floats((int)x.cols, S, r, D) * sizeof(float) <= f.ws_bytes) {
                        rows = r;
                        splits = S;
                    }
            }
        }
        int& wavefronts = p.wavefronts;
        for (int r : {32, 16}) {
            const Shape& x = r == 16 ? shape16 : shape32;
            // (columns that run at once in workgroups of eight are the faster so, but for those with fewer stages than a workgroup has wavefronts.  Eight / four, us: 290 x 4
            // heads, D = 64, four queries, 11 x 883 keys, codes (292 columns) 18.9 / 24.2; 35 x 64/8, D = 64, two queries, 977 keys, codes 10.9 / 14.2; 890 x 8/1, D = 64, 19 codes 6.4 / 5.9.)
            if (x.cols < 128 || (x.stages >= 6.0 && x.cols <= (D == 64 && r == 16 ? 512 : 256)) || (asked && asked != r) || chain_of_four(r) >= (wavefronts == 4 ? chain_of_four(rows) : chain_at(rows, splits))) continue;
            rows = r;
            splits = 1;
            wavefronts = 4;
        }
        const double suffix_us = has_suffix ? (f.fp8 ? 2.0 : 4.0) * B * (0.75 * max_len) * Hkv * D / 5.0e6 : 0.0;      // at 5 TB/s
        const double shared_us = shared_bytes / 5.0e6, part_us = 4.0 * B * nq * Hq * (double)D / 5.0e6;      // (one partial result of every row)
        const Eight& k8 = eight[D == 64][rows == 16];
        const Four& k4 = four[D == 64][rows == 16];
        const double streamed = wavefronts == 4 ? (paged ? k4.paged : k4.packed) : paged ? k8.paged : k8.packed;
        const double chain = wavefronts == 4 ? chain_of_four(rows) : chain_at(rows, splits), stream = streamed * suffix_us + shared_us + 6.0;
        const double est_single = cbrt(chain * chain * chain + stream * stream * stream);
        // Stages in runs where a round or two of workgroups fill the chip and the suffix rows are two fifths of the call: dealt out one by
        // one, all wavefronts multiply shared rows first and wait for the HBM together afterwards.  Dealt / runs, us: 1024 x 8/1 heads, 1K keys, 128 rows
        // 21.5 / 18.6; 512 rows 57.9 / 51.6; 2048 x 8/1, 1K keys, 512 rows 118 / 103; 456 x 16/2, 532 keys, up to 184 rows 17.8 / 16.4; 482 x 16/2, two
        // queries, 1359 keys, up to 996 rows 73.7 / 76.9 (the worst of 39, 0.955 in the mean).  Elsewhere dealing is the better by 6 %: fewer or more
        // columns (1.00 / 1.01 at this share), 16 rows (the phases are shorter), D = 64 (two workgroups per CU overlap), codes, several KV heads.
        p.dealt = f.fp8 || D == 64 || rows == 16 || splits > 1 || Hkv > 2 || cols < 200 || cols > 512 || suffix_us < 0.4 * est_single;
        const double sfx_alone = suffix_us * (sfx_mfma || rps == 1 ? 1.0 : 0.6 * rps), tiles_us = padded / 1.1e9;
        double est_other;
        const bool direct = nonempty == 0 && sfx_mfma && rps > 1 && alone.nchunks == 1;
        if (direct) {
            // The matrix-core suffix kernel straight to the outputs: what it takes goes by its work items, not by the bytes, where suffixes are short: a
            // wavefront of its own for each (its start, query tile, first rows, stores), 1280 at a time, more where they are smaller; and not below the
            // suffix rows' stream or the chain of one item.  Error 9 % over 410 drawn calls (by bytes and outputs alone 27 %: 607 x 8/1 heads, four queries, 26 rows
            // priced at 12.3 us take 8.6, on the single launch 12.0; 197 x 40/40, four queries, 25 rows at 24.5 take 43, on the single launch 21.6;
            // 547 x 64/8, two queries, up to 383 rows, paged at 129 take 102, on the single launch 110).
            const bool wide_tile = rps > 16;
            const double stages = (0.75 * max_len + 16.0) / 32.0, items = (double)B * Hkv * ceil_div(rps, wide_tile ? 32 : 16);
            const double places = 1280.0 * (D == 64 ? 2.4 : 1.0) * (f.fp8 ? 1.9 : 1.0);
            const double of_items = items / places * (wide_tile ? 5.5 + 3.4 * stages : 5.3 + 1.4 * stages);
            const double of_rows = suffix_us * (paged ? 0.99 : 0.86) * (f.fp8 ? 1.16 : 1.0);
            const double of_one = wide_tile ? 2.6 + 1.2 * stages : 1.8 + 0.9 * stages;
            est_other = 3.5 + cbrt(of_items * of_items * of_items + of_rows * of_rows * of_rows + of_one * of_one * of_one);
        } else if (nonempty == 0) {      // the suffix kernel alone: no event edges, hardly a merge
            est_other = 7.3 + 0.69 * (f.fp8 ? 1.2 : 1.0) * (paged ? 1.2 : 1.0) * (sfx_mfma || rps == 1 ? 1.0 : 1.5) * sfx_alone + 2.1 * part_us;
        } else if (may_combine && wide) {
            const double sfx = 0.55 * sfx_alone, sh = 0.9 * std::max((D == 128 ? 1.0 : 1.26) * tiles_us, shared_us);
            est_other = 12.9 + 8.1 * nonempty + std::max(sfx, sh) + 0.9 * std::min(sfx, sh) + 4.95 * part_us;
        } else {
            const double sfx = 0.61 * (f.fp8 ? 1.47 : 1.0) * sfx_alone, sh = 0.88 * std::max((D == 128 ? 1.0 : 0.91) * tiles_us, shared_us);
            est_other = 10.1 + 11.4 * nonempty + std::max(sfx, sh) + 1.32 * std::min(sfx, sh) + 5.83 * part_us;
        }
        // Trees, whose columns differ: between 256 and 512 columns of four wavefronts a launch lasts as long as the CUs that hold two of them, and stages of codes on
        // the matrix cores take longer than their bytes.  Single / other way, us: 286 x 32/8 heads, 3804 + 7 x 41 keys, 102 rows (288 columns) 68 / 56; 72 x 40/40, four queries,
        // 7199 + 14 x 102 keys 145 / 102; 100 x 40/40, 4542 + 16 x 922, 105 codes, paged 214 / 134; 331 x 32/8, 814 + 2 x 142, up to 482 codes 73 / 50.
        // (Calls with one level, and with more columns, lose by the same terms as often as they gain.)
        const long long single_cols = (rows == 16 ? shape16 : shape32).cols;
        const bool uneven = nonempty > 1 && wavefronts == 4 && D == 128 && single_cols > 256 && single_cols < 512;
        const double single_us = est_single * (f.fp8 && sfx_mfma && (direct || (nonempty > 1 && single_cols <= 768)) ? 1.06 : 1.0) * (uneven ? 1.0 + 0.25 * (512.0 / single_cols - 1.0) : 1.0);
        auto faster_than = [&](double other) {      // (calls with a shared block)
            return other <= 36.0 ? single_us <= 1.2 * other
                                 : single_us + 0.1 * suffix_us <= (f.fp8 && may_combine && wide && nonempty == 1 ? 0.91 : 1.0) * other;      // (codes: overestimated there)
        };
        bool small = direct ? single_us <= (est_other < 6.1 ? 1.26 : est_other < 36.0 ? 1.12 : 0.85) * est_other      // (a few items: 5 us are estimated at 7; rows by the thousand: it streams them slower)
                     : nonempty == 0 ? est_single <= (rps == 1 && alone.nchunks == 1 ? 0.8 : est_other <= 15.0 ? 1.2 : 1.0) * est_other
                     : faster_than(est_other);
        // The combined launch cuts a few columns with many keys into many parts, 0.6 us each beyond eight in its pieces' boundaries and in the merge: calls
        // with 19 and more parts took 20 % longer than the estimate, with 5 to 13 5 % less.  Counted from the teams and columns that its plan will have: within
        // 0.7 over 2430 drawn calls.
        // Combined / single, us: 185 x 16/2 heads, 9973 keys, 386 rows (20 parts) 49.3 / 40.5; 432 x 8/1, 9224 keys, up to 319 rows (14) 41.3 / 34.9.
        if (!small && nonempty > 0 && !own_memory && may_combine && wide) {
            double pieces = 0.0, tiled = 0.0;
            for (int i = 0; i < n_levels; ++i) {
                const long long seqs = levels[i].kv_off ? levels[i].max_seqs : B, tiles = (seqs * rps + kPrefixRowsWide - 1) / kPrefixRowsWide;
                if (levels[i].max_rows <= 0 || seqs * rps <= kCombinedRows) continue;
                pieces += (double)tiles * levels[i].n_blocks * Hkv;
                tiled += 4.0 * levels[i].n_blocks * (double)levels[i].max_rows * tiles * kPrefixRowsWide * Hkv * D;
            }
            const double suffix_bytes = (f.fp8 ? (sfx_mfma ? 2.6 : 2.0) : 4.0) * B * (sfx_mfma ? 1 : nq) * (0.75 * max_len) * Hkv * D;
            const int slots = pick_combined_slots(tiled, 0.8 * suffix_bytes, pieces, D, sfx_mfma);
            int parts = alone.nchunks;
            for (int i = 0; i < n_levels; ++i) {
                const long long seqs = levels[i].kv_off ? levels[i].max_seqs : B, tiles = (seqs * rps + kPrefixRowsWide - 1) / kPrefixRowsWide;
                if (levels[i].max_rows <= 0 || seqs <= 0) continue;
                if (seqs * rps <= kCombinedRows) { parts += 2; continue; }
                const long long T = std::min<long long>(tiles, slots), teams = 8 * (slots / T), columns = (long long)levels[i].n_blocks * Hkv * ((tiles + T - 1) / T);
                const long long cut = teams > columns ? (teams + columns - 1) / columns : 2;
                parts += (int)std::min<long long>(cut, std::max(1, levels[i].max_rows / (D == 128 ? 32 : 64)));
            }
            // (parts that have to be shrunk to the workspace: the single launch's check of it takes as long on the host as the gain)
            constexpr int kFreeParts = 8;
            if (parts > parts_cap(f.ws_bytes, (int64_t)B * nq * Hq, D)) parts = 0;
            small = faster_than(est_other + 0.6 * std::max(0, parts - kFreeParts));
        }
        if (own_memory) {
            // (a suffix alone, in one work item per row, goes from its kernel straight to the outputs: 782 x 4 heads, 21 rows
            // 14 us against 18 for the single launch)
            if (small || c->opt_fused_kernel == 2 || nonempty > 0 || !f.wants_lse) return HG_OK;
            p.sp = plan_suffix(c, max_len, G, B, nq, Hkv, D, false);
            if (p.sp.nchunks > 1) return HG_OK;
            p.way = kWayOneStream;
            p.np = 1;
            return HG_OK;
        }
        if (any && (rows == 16 ? shape16 : shape32).cols * splits < (1LL << 31)) {
            if (c->opt_fused_kernel == 2) return HG_OK;
            // (an option of the separate kernels asks for them)
            take_single = small && !c->opt_prefix_splits && !c->opt_prefix_kernel && !c->opt_wide_slots && !c->opt_overlap && !c->opt_suffix_kernel &&
                          !c->opt_suffix_chunk && !c->opt_suffix_ipw && !c->opt_suffix_tile;
        }
    }

    // The levels on the persistent kernel share the suffix's launch, provided that one has more than 128 query rows; the
    // others, and more than a few, go before it.
    if (may_combine && !take_single && c->opt_prefix_kernel != 1) {
        bool large = false;
        for (int i = 0; i < n_levels; ++i)
            large = large || (levels[i].max_rows > 0 && (double)(levels[i].kv_off ? levels[i].max_seqs : B) * nq * G > kPrefixRowsNarrow);
        if (large && plan_parts(c, f, true, p) == HG_OK && (int64_t)B * nq * G * p.sp.nchunks * Hkv < (1LL << 30)) {
            for (int i = 0; i < p.nlev; ++i)
                if (p.plan[i].wide && (p.joint < 0 || p.index[i] == p.main_level)) p.joint = i;
            if (p.joint >= 0) {
                p.way = kWayCombined;
                return HG_OK;
            }
        }
    }
    const int rc = plan_parts(c, f, false, p);
    if (rc) return rc;
    // (planned for the single launch too: a call is refused for its shape and workspace, not for what the estimates say)
    if (take_single) return HG_OK;
    if (p.np == 0) {
        p.way = kWayFill;
        return HG_OK;
    }

    // Two streams unless asked for one.  In automatic mode a call whose levels all run in the persistent kernel on
    // the whole chip stays on one stream (there is no CU left for the suffix kernel to run beside it), and so does a
    // call with less than about 60 us of work (forking and joining streams costs more than it can gain).
    bool all_wide_full = p.nlev > 0;
    for (int i = 0; i < p.nlev; ++i) all_wide_full = all_wide_full && p.plan[i].wide && p.plan[i].wp.slots == 32;
    const bool two = c->opt_overlap != 1 && has_suffix && p.nlev > 0 && !(c->opt_overlap == 0 && (all_wide_full || p.tiny));
    p.way = two ? kWayTwoStreams : kWayOneStream;
    return HG_OK;
}

// hg_hydragen_attn and hg_hydragen_attn_paged (pg.table set, offsets unused)
static int fused_impl(hg_ctx* c, const void* Q, int n_levels, const hg_level* levels, const void* Ks, const void* Vs,
                      const int32_t* offsets, const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D,
                      float scale, void* O_out, int o_dtype, float* LSE_out, const hg::PagedDev& pg, const KvFmt& fmt = KvFmt{},
                      const Ws* ws_override = nullptr) {
    int rc = check_fused(c, Q, n_levels, levels, Ks, Vs, offsets, lengths, max_len, B, Hq, Hkv, D, O_out, o_dtype,
                         pg.table != nullptr);
    if (rc) return rc;
    if (B == 0) return HG_OK;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    scale = eff_scale(scale, D);
    const int nq = c->opt_nq;
    const int64_t rows = (int64_t)B * nq * Hq;
    const int G = Hq / Hkv;
    const bool has_suffix = Ks != nullptr && max_len > 0;
    const Ws ws = ws_override ? *ws_override : Ws{c->ws, c->ws_bytes};

    FusedPlan p;
    rc = plan_fused(c, FusedShape{n_levels, levels, has_suffix, max_len, pg.table ? pg.shift : -1, fmt.fp8 != 0, fmt.v_scale, LSE_out != nullptr, B, Hq, Hkv, D,
                                  ws.p ? ws.bytes : 0, c->counters != nullptr}, &p);
    if (rc) return rc;
    hipStream_t s = c->stream;
    if (p.way == kWayFill) return fill_empty(O_out, o_dtype, LSE_out, rows, D, s);
    if (p.way == kWayCombined || (p.way == kWaySingle && p.splits > 1)) use_counters(c);
    if (p.way == kWaySingle) {
        SmallArgs sa{};
        sa.Q = static_cast<const uint16_t*>(Q);
        sa.n_levels = 0;
        for (int i = 0; i < n_levels; ++i) {
            const LevelDev d = to_dev(levels[i], B);
            if (d.max_rows == 0 || d.max_seqs == 0) continue;
            sa.lv[sa.n_levels++] = d;
        }
        sa.Ks = static_cast<const uint16_t*>(Ks);
        sa.Vs = static_cast<const uint16_t*>(Vs);
        sa.offsets = offsets;
        sa.lengths = has_suffix ? lengths : nullptr;
        sa.pg = has_suffix ? pg : PagedDev{};
        sa.fp8 = has_suffix ? fmt.fp8 : 0;
        sa.k_scale = fmt.k_scale; sa.v_scale = fmt.v_scale;
        sa.fp32_weights = sa.fp8 && !p.sfx_mfma;
        sa.max_len = max_len;
        sa.B = B; sa.Hq = Hq; sa.Hkv = Hkv; sa.G = G; sa.nq = nq;
        sa.rows = p.column_rows;
        sa.tiles = (B * nq * G + sa.rows - 1) / sa.rows;
        sa.cols = sa.tiles * Hkv;
        sa.splits = p.splits;
        sa.wavefronts = p.wavefronts;
        sa.by_head = divider((unsigned)(sa.tiles * sa.splits));
        sa.by_split = divider((unsigned)sa.splits);
        sa.by_seq = divider((unsigned)(nq * G));
        sa.by_group = divider((unsigned)G);
        sa.dealt = p.dealt;
        sa.part = reinterpret_cast<float*>(ws.p);
        sa.arrivals = p.splits > 1 ? c->counters + meeting_counter(p.splits) : nullptr;
        sa.scale = scale;
        sa.O = O_out; sa.LSE = LSE_out; sa.bf16 = (o_dtype == HG_BF16);
        return hip_rc(launch_fused_small(sa, D, c->stream));
    }
    const Parts parts = carve(ws, rows, D);
    const LevelDev* const lv = p.lv;
    const LevelPlan* const plan = p.plan;
    const int *const ns = p.ns;
    const int nlev = p.nlev, np = p.np;
    const SuffixPlan& sp = p.sp;

    // (grouped levels may leave sequences uncovered: the level's kernel marks their partial results empty)
    if (p.way == kWayCombined) {
        const int joint = p.joint;
        CombinedArgs ca{};
        int part = 0;
        for (int i = 0; i < nlev; ++i) {
            const OutDev out = parts_out(parts, part);
            if (i == joint) {
                ca.p = level_args(Q, lv[i], plan[i], B, nq, Hq, Hkv, scale, out);
            } else if (plan[i].wide && plan[i].wp.mode != 2 && plan[i].wp.slots == plan[joint].wp.slots && ca.n_more < kMoreLevels) {
                const PrefixArgs pa = level_args(Q, lv[i], plan[i], B, nq, Hq, Hkv, scale, out);
                memcpy(ca.more[ca.n_more++].args, &pa, kShortPrefixArgs);
            } else {
                rc = run_level(Q, lv[i], plan[i], B, nq, Hq, Hkv, D, scale, out, s);
                if (rc) return rc;
            }
            part += ns[i];
        }
        ca.d = suffix_args(Q, Ks, Vs, offsets, lengths, max_len, B, nq, Hq, Hkv, scale, sp.chunk, sp.nchunks, 1, parts_out(parts, part), pg, fmt);
        ca.tickets = c->counters;
        if (sp.mfma) {
            ca.d.tile_rows = (nq * G <= 16 && c->opt_suffix_tile != 32) ? 16 : 32;
            ca.d.units = (int64_t)B * sp.nchunks * ceil_div(nq * G, ca.d.tile_rows) * Hkv;
        }
        ca.d.by_heads = divider((unsigned)Hkv);
        ca.d.by_chunks = divider((unsigned)sp.nchunks);
        ca.d.by_tiles = divider((unsigned)(sp.mfma ? ceil_div(nq * G, ca.d.tile_rows) : 1));
        ca.d.by_group = divider((unsigned)G);
        const int units = (int)ca.d.units, wide = 8 * ca.p.wide.slots, starters = wide == 256 ? 256 : 256 - wide;
        const ItemRuns runs = item_runs(units, starters);
        ca.long_runs = runs.long_runs;
        ca.long_run = runs.long_run;
        ca.tail_run = runs.tail_run;
        ca.n_tickets = runs.n_tickets;
        if (sp.mfma) rc = hip_rc(D == 128 ? launch_combined_tiles(ca, s) : launch_combined_tiles_d64(ca, s));
        else rc = hip_rc(D == 128 ? launch_combined_vector(ca, s) : launch_combined_vector_d64(ca, s));
        if (rc) return rc;
        // The merge sets the work counter back.  (Set back by the launch itself it could be lost when two calls of a context are
        // in flight: wrong results for those two, which share the workspace, but also for every later call.)
        rc = run_merge(np, parts, 0, D, O_out, o_dtype, LSE_out, s, ca.tickets);
        if (rc) {      // nobody will: no further use of these counters, by whomever
            c->counters = nullptr;
            c->counter_slot = -1;
        }
        return rc;
    }

    // one part, no timing events to place: straight to the outputs
    if (nlev == 0 && np == 1 && LSE_out && !c->opt_timing)
        return run_decode(Q, 0, nullptr, Ks, Vs, offsets, lengths, max_len, B, nq, Hq, Hkv, D, scale, sp.chunk, 1, sp.gt,
                          direct_out(O_out, o_dtype, LSE_out), s, pg, sp.mfma, sp.ipw, false, fmt, c->opt_suffix_tile);

    const bool overlap = p.way == kWayTwoStreams;
    hipStream_t ssfx = s;
    if (overlap) {
        if (hipEventRecord(c->ev_fork, s) != hipSuccess) return HG_ERR_HIP;
        if (hipStreamWaitEvent(c->aux, c->ev_fork, 0) != hipSuccess) return HG_ERR_HIP;
        ssfx = c->aux;
    }
    // optional stage timing: events bracket each kernel on the stream it runs on
    const int slot = c->opt_timing ? (int)(c->tcalls % HG_TIMING_RING) : -1;
    if (slot >= 0)
        for (int i = 0; i < HG_MAX_STAGES; ++i) c->tused[slot * HG_MAX_STAGES + i] = 0;
    auto mark = [&](int stage, int which, hipStream_t st) -> bool {
        if (slot < 0) return true;
        c->tused[slot * HG_MAX_STAGES + stage] = 1;
        return hipEventRecord(c->tev[(slot * HG_MAX_STAGES + stage) * 2 + which], st) == hipSuccess;
    };
    int suffix_first = 0;
    for (int i = 0; i < nlev; ++i) suffix_first += ns[i];
    auto enqueue_suffix = [&]() -> int {
        if (!has_suffix) return HG_OK;
        if (!mark(0, 0, ssfx)) return HG_ERR_HIP;
        const int r = run_decode(Q, 0, nullptr, Ks, Vs, offsets, lengths, max_len, B, nq, Hq, Hkv, D, scale, sp.chunk,
                                 sp.nchunks, sp.gt, parts_out(parts, suffix_first), ssfx, pg, sp.mfma, sp.ipw, false, fmt, c->opt_suffix_tile);
        if (r) return r;
        if (!mark(0, 1, ssfx)) return HG_ERR_HIP;
        if (overlap && hipEventRecord(c->ev_join, c->aux) != hipSuccess) return HG_ERR_HIP;
        return HG_OK;
    };
    auto enqueue_levels = [&]() -> int {
        int part = 0;
        for (int i = 0; i < nlev; ++i) {
            if (!mark(1 + i, 0, s)) return HG_ERR_HIP;
            const int r = run_level(Q, lv[i], plan[i], B, nq, Hq, Hkv, D, scale, parts_out(parts, part), s);
            if (r) return r;
            if (!mark(1 + i, 1, s)) return HG_ERR_HIP;
            part += ns[i];
        }
        return HG_OK;
    };
    // Two streams: the memory-bound suffix kernel and the power-bound shared-block kernels run side by side.  The
    // persistent 256-row kernel takes whole CUs (wide_slots per XCD, chosen above) and is enqueued first so that
    // its workgroups are placed before the suffix kernel fills the chip; 128-row workgroups leave register space
    // for suffix wavefronts on their CUs and go second unless HG_OPT_OVERLAP = 2 asks for them first.
    bool any_wide = false;
    for (int i = 0; i < nlev; ++i) any_wide = any_wide || plan[i].wide;
    // A launch that fails here (a HIP runtime error: the sizes were checked above) leaves work enqueued and the
    // second stream forked: the fork is still joined before the error is returned, so that a stream capture in
    // progress stays valid and nothing runs behind the caller's back on the second stream.
    auto fail = [&](int code) -> int {
        if (overlap) {
            (void)hipEventRecord(c->ev_join, c->aux);
            (void)hipStreamWaitEvent(s, c->ev_join, 0);
        }
        return code;
    };
    if (c->opt_overlap == 2 || (c->opt_overlap == 0 && any_wide)) {
        rc = enqueue_levels();
        if (rc) return fail(rc);
        rc = enqueue_suffix();
        if (rc) return fail(rc);
    } else {
        rc = enqueue_suffix();
        if (rc) return fail(rc);
        rc = enqueue_levels();
        if (rc) return fail(rc);
    }
    if (overlap && hipStreamWaitEvent(s, c->ev_join, 0) != hipSuccess) return HG_ERR_HIP;
    if (!mark(nlev + 1, 0, s)) return HG_ERR_HIP;
    rc = run_merge(np, parts, 0, D, O_out, o_dtype, LSE_out, s);
    if (rc) return rc;
    if (!mark(nlev + 1, 1, s)) return HG_ERR_HIP;
    if (slot >= 0) c->tcalls += 1;
    return HG_OK;
}

int hg_hydragen_attn(hg_ctx* c, const void* Q, int n_levels, const hg_level* levels, const void* Ks, const void* Vs,
                     const int32_t* offsets, const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D,
                     float scale, void* O_out, int o_dtype, float* LSE_out) {
    return fused_impl(c, Q, n_levels, levels, Ks, Vs, offsets, lengths, max_len, B, Hq, Hkv, D, scale, O_out, o_dtype,
                      LSE_out, hg::PagedDev{});
}

int hg_hydragen_attn_static(hg_ctx* c, const void* Q, int n_levels, const hg_level* levels, const void* Ks, const void* Vs,
                            const int32_t* offsets, const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D,
                            float scale, void* O_out, int o_dtype, float* LSE_out) {
    if (!c) return HG_ERR_INVALID_ARG;
    if (c->device < 0 || c->device >= 64 || !g_scratch_ptr[c->device]) return HG_ERR_UNSUPPORTED;
    int rc = check_fused(c, Q, n_levels, levels, Ks, Vs, offsets, lengths, max_len, B, Hq, Hkv, D, O_out, o_dtype);
    if (rc) return rc;
    // one fp32 partial result per non-empty shared level and one for the suffix must fit the array
    int need = (Ks != nullptr && max_len > 0) ? 1 : 0;
    for (int i = 0; i < n_levels; ++i)
        if (levels[i].max_rows > 0 && (levels[i].kv_off ? levels[i].max_seqs : B) > 0) ++need;
    const unsigned long long per = (unsigned long long)B * c->opt_nq * Hq * (D + 1) * sizeof(float);
    if ((unsigned long long)need * per > (unsigned long long)HG_STATIC_SCRATCH_BYTES) return HG_ERR_STATIC_LIMIT;
    const Ws ws{g_scratch_ptr[c->device], (size_t)HG_STATIC_SCRATCH_BYTES};
    return fused_impl(c, Q, n_levels, levels, Ks, Vs, offsets, lengths, max_len, B, Hq, Hkv, D, scale, O_out, o_dtype,
                      LSE_out, hg::PagedDev{}, KvFmt{}, &ws);
}

int hg_hydragen_attn_paged(hg_ctx* c, const void* Q, int n_levels, const hg_level* levels, const hg_paged_kv* kv,
                           const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D, float scale, void* O_out,
                           int o_dtype, float* LSE_out) {
    if (max_len < 0 || Hkv <= 0 || (D != 64 && D != 128)) return HG_ERR_INVALID_ARG;
    hg::PagedDev pg{};
    KvFmt fmt;
    const int rc = paged_dev(kv, max_len, Hkv, D, &pg, &fmt);
    if (rc) return rc;
    if (max_len == 0) pg.table = nullptr;   // no suffix rows: the call reduces to the shared levels
    return fused_impl(c, Q, n_levels, levels, max_len > 0 ? kv->K : nullptr, kv->V, nullptr, lengths, max_len, B, Hq, Hkv, D,
                      scale, O_out, o_dtype, LSE_out, pg, fmt);
}

// hg_kv_append and hg_kv_append_paged
static int append_impl(hg_ctx* c, const void* Knew, const void* Vnew, void* Ks, void* Vs, const int32_t* offsets,
                       int32_t* lengths, int capacity, int B, int Hkv, int D, const hg::PagedDev& pg, const KvFmt& fmt = KvFmt{}) {
    if (!c || B < 0 || Hkv <= 0 || capacity < 0) return HG_ERR_INVALID_ARG;
    if (D != 64 && D != 128) return HG_ERR_UNSUPPORTED;
    if ((int64_t)B * c->opt_nq * Hkv * D >= (1LL << 31)) return HG_ERR_UNSUPPORTED;
    if (B == 0) return HG_OK;
    if (!Knew || !Vnew || !lengths || (!offsets && !pg.table)) return HG_ERR_INVALID_ARG;
    if (capacity > 0 && (!Ks || !Vs)) return HG_ERR_INVALID_ARG;
    if (capacity == 0) return HG_OK;   // no room anywhere: every new row is dropped, lengths stay
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    hg::AppendArgs a{};
    a.Knew = static_cast<const uint16_t*>(Knew);
    a.Vnew = static_cast<const uint16_t*>(Vnew);
    a.Ks = static_cast<uint16_t*>(Ks);
    a.Vs = static_cast<uint16_t*>(Vs);
    a.offsets = offsets;
    a.lengths = lengths;
    a.pg = pg;
    a.capacity = capacity;
    a.B = B;
    a.nq = c->opt_nq;
    a.row_elems = Hkv * D;
    a.fp8 = fmt.fp8;
    a.k_scale = fmt.k_scale;
    a.v_scale = fmt.v_scale;
    return hip_rc(hg::launch_kv_append(a, c->stream));
}

int hg_kv_append(hg_ctx* c, const void* Knew, const void* Vnew, void* Ks, void* Vs, const int32_t* offsets,
                 int32_t* lengths, int capacity, int B, int Hkv, int D) {
    return append_impl(c, Knew, Vnew, Ks, Vs, offsets, lengths, capacity, B, Hkv, D, hg::PagedDev{});
}

int hg_kv_append_paged(hg_ctx* c, const void* Knew, const void* Vnew, const hg_paged_kv* kv, int32_t* lengths,
                       int capacity, int B, int Hkv, int D) {
    if (capacity < 0 || Hkv <= 0 || (D != 64 && D != 128)) return HG_ERR_INVALID_ARG;
    hg::PagedDev pg{};
    KvFmt fmt;
    const int rc = paged_dev(kv, capacity, Hkv, D, &pg, &fmt);
    if (rc) return rc;
    if (capacity == 0) return HG_OK;
    return append_impl(c, Knew, Vnew, kv->K, kv->V, nullptr, lengths, capacity, B, Hkv, D, pg, fmt);
}

int hg_suffix_attn_fp8(hg_ctx* c, const void* Q, const void* Ks8, const void* Vs8, float k_scale, float v_scale,
                       const int32_t* offsets, const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D, float scale,
                       void* O, int o_dtype, float* LSE) {
    KvFmt fmt;
    if (!fp8_fmt(k_scale, v_scale, &fmt)) return HG_ERR_INVALID_ARG;
    return suffix_impl(c, Q, Ks8, Vs8, offsets, lengths, max_len, B, Hq, Hkv, D, scale, O, o_dtype, LSE, hg::PagedDev{}, false, fmt);
}

int hg_hydragen_attn_fp8(hg_ctx* c, const void* Q, int n_levels, const hg_level* levels, const void* Ks8, const void* Vs8,
                         float k_scale, float v_scale, const int32_t* offsets, const int32_t* lengths, int max_len, int B,
                         int Hq, int Hkv, int D, float scale, void* O_out, int o_dtype, float* LSE_out) {
    KvFmt fmt;
    if (!fp8_fmt(k_scale, v_scale, &fmt)) return HG_ERR_INVALID_ARG;
    return fused_impl(c, Q, n_levels, levels, Ks8, Vs8, offsets, lengths, max_len, B, Hq, Hkv, D, scale, O_out, o_dtype,
                      LSE_out, hg::PagedDev{}, fmt);
}

int hg_kv_append_fp8(hg_ctx* c, const void* Knew, const void* Vnew, void* Ks8, void* Vs8, float k_scale, float v_scale,
                     const int32_t* offsets, int32_t* lengths, int capacity, int B, int Hkv, int D) {
    KvFmt fmt;
    if (!fp8_fmt(k_scale, v_scale, &fmt)) return HG_ERR_INVALID_ARG;
    return append_impl(c, Knew, Vnew, Ks8, Vs8, offsets, lengths, capacity, B, Hkv, D, hg::PagedDev{}, fmt);
}

int hg_naive_attn(hg_ctx* c, const void* Q, int n_levels, const hg_level* levels, const void* Ks, const void* Vs,
                  const int32_t* offsets, const int32_t* lengths, int max_len, int B, int Hq, int Hkv, int D, float scale,
                  void* O_out, int o_dtype, float* LSE_out) {
    int rc = check_fused(c, Q, n_levels, levels, Ks, Vs, offsets, lengths, max_len, B, Hq, Hkv, D, O_out, o_dtype);
    if (rc) return rc;
    if (B == 0) return HG_OK;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    scale = eff_scale(scale, D);
    const int nq = c->opt_nq;
    const int64_t rows = (int64_t)B * nq * Hq;
    const int G = Hq / Hkv;
    const bool has_suffix = Ks != nullptr && max_len > 0;
    const Parts parts = carve(Ws{c->ws, c->ws_bytes}, rows, D);
    LevelDev lv[HG_MAX_LEVELS];
    int64_t nmax = has_suffix ? max_len : 0;
    for (int i = 0; i < n_levels; ++i) {
        lv[i] = to_dev(levels[i], B);
        nmax += lv[i].max_rows;
    }
    hipStream_t s = c->stream;
    if (parts.cap < 1) return HG_ERR_WORKSPACE;
    if (nmax == 0) return fill_empty(O_out, o_dtype, LSE_out, rows, D, s);
    if (nmax >= (1LL << 30)) return HG_ERR_UNSUPPORTED;
    // (with one row per KV head the vector-ALU kernel is the faster comparison: 38 against 49 ms on config 3)
    if (c->opt_suffix_kernel != 1 && (c->opt_suffix_kernel == 2 || (nq * G >= 2 && auto_mfma(nq, G, (int)nmax, D)))) {
        // Several query rows per KV head: the per-sequence kernel on the matrix cores, once per level (every sequence
        // walks the block that covers it by itself) and once for the suffix, each writing its own partial results.
        int chunk = c->opt_naive_chunk > 0 ? round_up(c->opt_naive_chunk, 32) : 1024;
        const int cap = parts.cap < HG_MAX_PARTS ? parts.cap : HG_MAX_PARTS;
        auto parts_for = [&](int ch) {
            int n = has_suffix ? ceil_div(max_len, ch) : 0;
            for (int i = 0; i < n_levels; ++i) if (lv[i].max_rows > 0) n += ceil_div(lv[i].max_rows, ch);
            return n;
        };
        while (parts_for(chunk) > cap && chunk < (1 << 29)) chunk *= 2;
        if (parts_for(chunk) > cap) return HG_ERR_WORKSPACE;
        {   // item counts of every launch below, checked before anything is enqueued
            const int tile_rows = (nq * G <= 16 && c->opt_suffix_tile != 32) ? 16 : 32;
            const int64_t per = (int64_t)B * ceil_div(nq * G, tile_rows) * Hkv;
            if (per * parts_for(chunk) >= (1LL << 31)) return HG_ERR_UNSUPPORTED;
        }
        int first = 0;
        for (int i = 0; i < n_levels; ++i) {
            if (lv[i].max_rows <= 0) continue;
            const int n = ceil_div(lv[i].max_rows, chunk);
            rc = run_decode(Q, 1, &lv[i], lv[i].K, lv[i].V, nullptr, nullptr, lv[i].max_rows, B, nq, Hq, Hkv, D, scale, chunk, n, 1,
                            parts_out(parts, first), s, PagedDev{}, true, c->opt_suffix_ipw, true, KvFmt{}, c->opt_suffix_tile);
            if (rc) return rc;
            first += n;
        }
        if (has_suffix) {
            const int n = ceil_div(max_len, chunk);
            rc = run_decode(Q, 0, nullptr, Ks, Vs, offsets, lengths, max_len, B, nq, Hq, Hkv, D, scale, chunk, n, 1,
                            parts_out(parts, first), s, PagedDev{}, true, c->opt_suffix_ipw, false, KvFmt{}, c->opt_suffix_tile);
            if (rc) return rc;
            first += n;
        }
        return run_merge(first, parts, 0, D, O_out, o_dtype, LSE_out, s);
    }
    int chunk = c->opt_naive_chunk > 0 ? round_up(c->opt_naive_chunk, 32) : 512;
    int nchunks = ceil_div((int)nmax, chunk);
    const int cap = parts.cap < 32 ? parts.cap : 32;
    if (nchunks > cap) {
        chunk = round_up(ceil_div((int)nmax, cap), 32);
        nchunks = ceil_div((int)nmax, chunk);
    }
    rc = run_decode(Q, n_levels, lv, has_suffix ? Ks : nullptr, Vs, offsets, has_suffix ? lengths : nullptr, max_len, B, nq, Hq,
                    Hkv, D, scale, chunk, nchunks, pick_gt(G), parts_out(parts, 0), s);
    if (rc) return rc;
    return run_merge(nchunks, parts, 0, D, O_out, o_dtype, LSE_out, s);
}

int hg_read_stage_timings(hg_ctx* c, float* ms, int n_calls) {
    if (!c || !ms || n_calls < 0) return -HG_ERR_INVALID_ARG;
    if (!c->tev) return 0;
    if (hipSetDevice(c->device) != hipSuccess) return -HG_ERR_HIP;
    long long avail = c->tcalls < HG_TIMING_RING ? c->tcalls : HG_TIMING_RING;
    const int n = (int)(n_calls < avail ? n_calls : avail);
    for (int k = 0; k < n; ++k) {
        const int slot = (int)((c->tcalls - 1 - k) % HG_TIMING_RING);
        for (int st = 0; st < HG_MAX_STAGES; ++st) {
            float t = 0.f;
            if (c->tused[slot * HG_MAX_STAGES + st]) {
                hipEvent_t e0 = c->tev[(slot * HG_MAX_STAGES + st) * 2], e1 = c->tev[(slot * HG_MAX_STAGES + st) * 2 + 1];
                if (hipEventSynchronize(e1) != hipSuccess) return -HG_ERR_HIP;
                if (hipEventElapsedTime(&t, e0, e1) != hipSuccess) return -HG_ERR_HIP;
            }
            ms[k * HG_MAX_STAGES + st] = t;
        }
    }
    return n;
}

int hg_debug_wide_plan(int n_blocks, int max_rows, int max_seqs, int Hkv, int rows_per_seq, int max_parts, int slots_per_xcd,
                       int D, int out[9]) {
    if (!out || n_blocks < 1 || max_rows < 0 || max_seqs < 0 || Hkv < 1 || rows_per_seq < 1 || (D != 64 && D != 128)) return 0;
    hg::LevelDev lv{};
    lv.n_blocks = n_blocks;
    lv.max_rows = max_rows;
    lv.max_seqs = max_seqs;
    hg::WidePlan p{};
    if (!hg::plan_prefix_wide(lv, Hkv, rows_per_seq, D, max_parts, slots_per_xcd, &p)) return 0;
    out[0] = p.n_c; out[1] = p.ncols; out[2] = p.rowgroups; out[3] = p.T;
    out[4] = p.slots; out[5] = p.tpx; out[6] = p.quota; out[7] = p.nparts; out[8] = p.mode;
    return 1;
}

int hg_debug_wide_ranges(int n_blocks, int max_rows, int max_seqs, int Hkv, int rows_per_seq, int max_parts, int slots_per_xcd,
                         int D, int starts[257], int first_part[256]) {
    if (!starts || !first_part || n_blocks < 1 || max_rows < 0 || max_seqs < 0 || Hkv < 1 || rows_per_seq < 1 || (D != 64 && D != 128)) return 0;
    hg::LevelDev lv{};
    lv.n_blocks = n_blocks;
    lv.max_rows = max_rows;
    lv.max_seqs = max_seqs;
    hg::WidePlan p{};
    if (!hg::plan_prefix_wide(lv, Hkv, rows_per_seq, D, max_parts, slots_per_xcd, &p) || p.mode != 2) return 0;
    const int nteams = 8 * p.tpx;
    for (int t = 0; t <= nteams; ++t) starts[t] = p.starts[t];
    for (int t = 0; t < nteams; ++t) first_part[t] = p.first_part[t];
    return nteams;
}

int hg_debug_wide_team(int n_blocks, int max_rows, int max_seqs, int Hkv, int rows_per_seq, int max_parts, int slots_per_xcd,
                       int D, int team, int out[3]) {
    if (!out || team < 0 || n_blocks < 1 || max_rows < 0 || max_seqs < 0 || Hkv < 1 || rows_per_seq < 1 || (D != 64 && D != 128)) return 0;
    hg::LevelDev lv{};
    lv.n_blocks = n_blocks;
    lv.max_rows = max_rows;
    lv.max_seqs = max_seqs;
    hg::WidePlan p{};
    if (!hg::plan_prefix_wide(lv, Hkv, rows_per_seq, D, max_parts, slots_per_xcd, &p) || team >= 8 * p.tpx) return 0;
    return hg::wide_team_range(p, team, out[0], out[1], out[2]) ? 1 : 0;
}

int hg_debug_item_runs(int items, int slots_per_xcd, int out[5]) {
    if (!out || items < 1 || items >= (1 << 30) || slots_per_xcd < 1 || slots_per_xcd > 32) return 0;
    const int starters = slots_per_xcd == 32 ? 256 : 256 - 8 * slots_per_xcd;
    const hg::ItemRuns r = hg::item_runs(items, starters);
    out[0] = r.long_runs; out[1] = r.long_run; out[2] = r.tail_run; out[3] = r.n_tickets; out[4] = starters;
    return 1;
}

int hg_debug_suffix_plan(int B, int nq, int Hq, int Hkv, int D, int max_len, int page_size, int out[4]) {
    if (!out || B < 1 || nq < 1 || Hkv < 1 || Hq < Hkv || Hq % Hkv != 0 || (D != 64 && D != 128) || max_len < 0 || page_size < 0) return 0;
    hg_ctx c{};   // default options
    c.opt_nq = nq;
    const SuffixPlan p = plan_suffix(&c, max_len, Hq / Hkv, B, nq, Hkv, D, page_size > 0, page_size > 0 ? 32 * page_size : 1 << 30);
    out[0] = p.chunk; out[1] = p.nchunks; out[2] = p.mfma ? 1 : 0; out[3] = p.gt;
    return 1;
}

int hg_debug_fused_plan(const int* options, int n_options, int n_levels, const hg_level* levels, int B, int nq, int Hq, int Hkv, int D,
                        int max_len, int page_size, int fp8, size_t workspace_bytes, int out[8]) {
    if (!out || n_options < 0 || (n_options > 0 && !options) || n_levels < 0 || n_levels > HG_MAX_LEVELS || (n_levels > 0 && !levels)) return HG_ERR_INVALID_ARG;
    if (B < 1 || nq < 1 || nq > 64 || max_len < 0 || page_size < 0 || page_size > 1024) return HG_ERR_INVALID_ARG;
    const int rc = check_shape(B, Hq, Hkv, D, nq);
    if (rc) return rc;
    hg_ctx c{};
    for (int i = 0; i < n_options; ++i) {
        const int set = options[2 * i] == HG_OPT_STAGE_TIMING ? HG_ERR_INVALID_ARG : hg_set_option(&c, options[2 * i], options[2 * i + 1]);
        if (set) return set;
    }
    c.opt_nq = nq;
    int shift = -1;
    if (page_size > 0)
        for (shift = 0; (1 << shift) < page_size;) ++shift;
    FusedPlan p;
    const int r = plan_fused(&c, FusedShape{n_levels, levels, max_len > 0, max_len, shift, fp8 != 0, 1.0f, true, B, Hq, Hkv, D, workspace_bytes, true}, &p);
    if (r) return r;
    const bool single = p.way == kWaySingle;
    out[0] = p.way;
    out[1] = single ? p.splits : 0;
    out[2] = single ? 0 : p.np;
    out[3] = single ? p.column_rows : p.sp.chunk;
    out[4] = single ? p.dealt : p.sp.nchunks;
    out[5] = !single && p.sp.nchunks > 0 && p.sp.mfma ? 1 : 0;
    out[6] = 0;
    out[7] = single ? p.wavefronts : 0;
    for (int i = 0; !single && i < p.nlev; ++i) {
        if (!p.plan[i].wide) continue;
        out[6] |= 1 << p.index[i];
        if (p.index[i] == p.main_level || !out[7]) out[7] = p.plan[i].wp.slots;
    }
    return HG_OK;
}

int hg_debug_single_work(int workgroup, int tiles, int splits, int Hkv, int out[3]) {
    if (workgroup < 0 || tiles < 1 || splits < 1 || Hkv < 1 || !out || (long long)tiles * splits * Hkv >= (1LL << 31) - 8) return 0;
    if ((unsigned)workgroup >= hg::small_grid(tiles * splits * Hkv)) return 0;
    return hg::small_work((unsigned)workgroup, tiles, splits, Hkv, hg::divider((unsigned)(tiles * splits)), hg::divider((unsigned)splits), out[0], out[1], out[2]) ? 1 : 0;
}

int hg_debug_mfma_loop(hg_ctx* c, int random_operands, int iters, unsigned long long* clocks, float* sink) {
    if (!c || iters < 1 || !clocks || !sink) return HG_ERR_INVALID_ARG;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    return hip_rc(hg::launch_mfma_loop(iters, random_operands ? 1 : 0, clocks, sink, c->stream));
}

int hg_debug_stream_read(hg_ctx* c, const void* src, size_t bytes, float* sink) {
    if (!c || !src || !sink || bytes < 16 || reinterpret_cast<uintptr_t>(src) % 16 != 0) return HG_ERR_INVALID_ARG;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    return hip_rc(hg::launch_stream_read(src, bytes, sink, c->stream));
}

int hg_debug_xcd_of_workgroups(hg_ctx* c, int n_workgroups, int* out) {
    if (!c || !out || n_workgroups < 1 || n_workgroups > 4096) return HG_ERR_INVALID_ARG;
    if (hipSetDevice(c->device) != hipSuccess) return HG_ERR_HIP;
    return hip_rc(hg::launch_xcd_probe(n_workgroups, out, c->stream));
}

const char* hg_strerror(int code) {
    switch (code) {
        case HG_OK: return "ok";
        case HG_ERR_INVALID_ARG: return "invalid argument";
        case HG_ERR_UNSUPPORTED: return "unsupported shape or dtype";
        case HG_ERR_WORKSPACE: return "workspace too small";
        case HG_ERR_HIP: return "HIP runtime error";
        case HG_ERR_STATIC_LIMIT: return "too many query rows for the static scratch array of hg_hydragen_attn_static";
    }
    return "unknown error";
}

}  // extern "C"
