// Internal declarations shared by the HIP translation units of libhydragen (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "hydragen.h"

namespace hg {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Division by a number that the host knows, without one: q = n / d for n < 2^31 (Granlund and Montgomery, "Division by invariant
// integers using multiplication": with s = ceil(log2 d) and mul = ceil(2^(31 + s) / d) < 2^32, q = floor(n mul / 2^(31 + s))).
struct Divider {
    unsigned mul, shift;
    __host__ __device__ unsigned of(unsigned n) const { return (unsigned)(((uint64_t)(2u * n) * mul) >> 32) >> shift; }
};
inline Divider divider(unsigned d) {      // 1 <= d < 2^31
    unsigned s = 0;
    while ((1u << s) < d) ++s;
    return Divider{(unsigned)(((1ull << (31 + s)) + d - 1) / d), s};
}

// ---- device-side descriptions --------------------------------------------------------------------

struct LevelDev {
    const uint16_t* K;
    const uint16_t* V;
    const int32_t* kv_off;   // may be null when n_blocks == 1
    const int32_t* seq_off;  // may be null when n_blocks == 1
    int n_blocks;
    int max_rows;
    int max_seqs;
};

// Where a kernel puts a partial (or final) result for query row idx = (b*nq + t)*Hq + h.
struct OutDev {
    void* O;          // [rows, D] fp32 or bf16
    float* LSE;       // [rows]
    int bf16;         // 1: O is bf16
    int64_t part_stride_O;    // elements between consecutive parts (0 when a single part)
    int64_t part_stride_L;
};

constexpr int kWideMaxTeams = 256;        // one team per CU at most
constexpr int kWideBoundaryCost = 9;      // stages a piece boundary costs a workgroup (measured: 8 us at 0.85 us per stage)

// Work partition of the persistent 256-row shared-block kernel (prefix_wide_impl.h).
struct WidePlan {
    int n_c;        // stages per column (32 keys each at D = 128, 64 at D = 64), from the host's bound on rows per block
    int ncols;      // columns = n_blocks * Hkv * rowgroups
    int rowgroups;  // groups of at most 32 query-row tiles
    int T;          // workgroups per team = query-row tiles per row group
    int slots;      // workgroups (CUs) per XCD that the kernel occupies
    int tpx;        // teams per XCD (slots / T)
    int quota;      // stages per team (mode 0)
    int nparts;     // partial results per query row
    int mode;       // how the flattened (column, stage) space is cut into one contiguous range per team:
                    // 0: equal ranges of `quota` stages; 1: ranges that never straddle a column boundary (each column
                    // cut evenly among its own teams, or whole columns per team when there are more columns than teams);
                    // 2: ranges of equal cost from the table below (a column boundary inside a range counts as
                    // kWideBoundaryCost stages: the team's workgroups store a result and load a Q tile there)
    Divider by_T, by_n_c, by_rowgroups;          // divisions that a workgroup makes on its way to a piece
    Divider by_quota, by_cols, by_teams;         // (quota, ncols, 8 * tpx)
    Divider by_cut[2];                           // mode 1: by the teams of a column, nteams / ncols and one more
    int starts[kWideMaxTeams + 1];      // mode 2: team t walks [starts[t], starts[t + 1])
    int first_part[kWideMaxTeams];      // mode 2: part index of team t's first piece (pieces of its column before it)
};

// The range [f0, f1) of the flattened (column, stage) space that a team walks, and the part index of its first piece; false: none.
// `p`: a WidePlan, on the device in the kernarg segment.
template <class Plan>
__host__ __device__ inline bool wide_team_range(const Plan& p, int team, int& f0, int& f1, int& sp0) {
    const auto div = [](unsigned n, const auto& d) { return Divider{d.mul, d.shift}.of(n); };
    const int nteams = 8 * p.tpx;
    const int total = p.ncols * p.n_c;      // the planner keeps this below 2^31 (and the columns below 2^20)
    if (p.mode == 0) {            // equal contiguous ranges
        const long long lo = (long long)team * p.quota;
        if (lo >= total) return false;
        f0 = (int)lo;
        f1 = (int)(lo + p.quota < total ? lo + p.quota : total);
        sp0 = team - (int)div(div((unsigned)f0, p.by_n_c) * (unsigned)p.n_c, p.by_quota);
    } else if (p.mode == 2) {     // ranges of equal cost, from the planner's table
        f0 = p.starts[team];
        f1 = p.starts[team + 1];
        sp0 = p.first_part[team];
    } else if (p.ncols <= nteams) {   // every column is cut evenly among its own teams
        const int c = (int)div((unsigned)(team * p.ncols), p.by_teams);
        const int tf = (int)div((unsigned)(c * nteams + p.ncols - 1), p.by_cols);
        const int nt = (int)div((unsigned)((c + 1) * nteams + p.ncols - 1), p.by_cols) - tf;
        const int more = nt * p.ncols > nteams;      // nteams / ncols teams, or one more
        sp0 = team - tf;
        f0 = c * p.n_c + (int)div((unsigned)(sp0 * p.n_c), p.by_cut[more]);
        f1 = c * p.n_c + (int)div((unsigned)((sp0 + 1) * p.n_c), p.by_cut[more]);
    } else {                      // whole columns per team
        f0 = (int)div((unsigned)(team * p.ncols), p.by_teams) * p.n_c;
        f1 = (int)div((unsigned)((team + 1) * p.ncols), p.by_teams) * p.n_c;
        sp0 = 0;
    }
    return f0 < f1;
}

struct PrefixArgs {
    const uint16_t* Q;
    LevelDev lv;
    int B, Hq, Hkv, G;
    int nq;           // queries per sequence: a sequence contributes nq*G rows per KV head, row = t*G + g
    Divider by_heads, by_seq, by_group;      // division by Hkv, nq * G, G
    int mtiles;       // query-row tiles per (block, KV head)
    int nsplit;       // key-range splits per block
    int chunk;        // keys per split (multiple of the key tile)
    int total_tiles;  // n_blocks * nsplit * Hkv * mtiles
    int per_xcd;      // ceil(total_tiles / 8)
    float scale;      // softmax scale
    OutDev out;       // part index = split
    WidePlan wide;    // persistent kernel only
};

// Page table of a paged suffix cache: suffix row j of sequence b is pool row
// (table[b*stride + (j >> shift)] << shift) + (j & ((1 << shift) - 1)); page ids are clamped to [0, n_pages).
struct PagedDev {
    const int32_t* table;   // null: the suffix is addressed by offsets[b] + j
    int shift;              // log2(rows per page), 4..10
    int stride;             // table entries per sequence
    int n_pages;
};

struct DecodeArgs {
    const uint16_t* Q;
    int n_levels;
    LevelDev lv[HG_MAX_LEVELS];
    const uint16_t* Ks;
    const uint16_t* Vs;
    const int32_t* offsets;
    const int32_t* lengths;   // null: no suffix
    PagedDev pg;              // suffix read through a page table when pg.table != null (then offsets is unused)
    int max_len;
    int B, Hq, Hkv, G;
    int nq;           // queries per sequence; query t sees suffix rows [0, length - (nq-1-t))
    int chunk;        // keys per work item
    int nchunks;      // work items per (sequence, KV head, query-head group)
    int64_t units;    // B * nq * nchunks * Hkv * (G / GT)
    Divider by_heads, by_chunks, by_tiles, by_group;      // combined launch: division by Hkv, nchunks, tiles of nq * G rows, G
    int tile_rows;    // matrix-core kernel: query rows per tile, 32 or 16 (16: at most 16 rows per KV head and sequence)
    int items;        // matrix-core kernel: B * nchunks * ceil(nq*G / tile_rows) * Hkv work items
    int ipw;          // matrix-core kernel: consecutive work items per wavefront
    int seg;          // matrix-core kernel: 1 = the keys of sequence b are the rows of the block of lv[0] that covers b
                      // (Ks/Vs then point at that level's tensors; offsets/lengths are unused, no causal bound)
    float scale;
    int fp8;          // vector-ALU kernel, suffix only: Ks/Vs hold E4M3 codes (one byte per element)
    float k_scale, v_scale;   // value = code * scale (fp8 only)
    OutDev out;       // part index = chunk
};

// Shared block and suffix in one launch (combined_impl.h): `p` (first: the shared-block role reads it from the kernarg
// segment) for the largest level on the persistent kernel, `d` for the suffix; d.units counts its work items.
constexpr int kMoreLevels = 3;
constexpr size_t kShortPrefixArgs = offsetof(PrefixArgs, wide) + offsetof(WidePlan, starts);      // a level without its tables
struct alignas(16) MoreLevel { unsigned char args[(kShortPrefixArgs + 15) / 16 * 16]; };
struct CombinedArgs {
    PrefixArgs p;
    DecodeArgs d;
    int n_more;                     // further levels, one after another on the same workgroups
    MoreLevel more[kMoreLevels];
    unsigned* tickets;    // work counter, zero at the start (the merge that follows sets it back)
    int long_runs;        // (item_runs below)
    int long_run;
    int tail_run;
    int n_tickets;
};
// Work items go out in runs (tickets).  The first runs, one for every workgroup that starts with one, have an item for each of its wavefronts where there are
// as many: those without would wait for the draws of all the others (128 x 32/8 heads, 2K keys, paged: 216 workgroups start with 1728 of 2048
// items; with runs of 2 some wavefronts had their first item at 11 of 34 us).  Long runs until kTailItems are left, then short ones so that the workgroups
// end together: a run of eight 256-row items keeps a CU busy for 45 us.  (256 x 40 heads with suffixes of 1..256 rows: runs of 32 and 8
// 150 us, 32 / 8 / 2 150, 16 / 4 / 2 134, 8 / 2 135, 4 138.)  Calls whose first runs leave fewer than kTailItems, or none (2048 items on 256 starting
// workgroups), have that much less of a tail; of 700 drawn calls with these runs none is slower than with the short runs by more than 3 %.
constexpr int kLongRun = 8, kTailItems = 1024;
struct ItemRuns { int long_runs, long_run, tail_run, n_tickets; };      // tickets below long_runs stand for long_run items, the others for tail_run
inline ItemRuns item_runs(int units, int starters) {
    ItemRuns r;
    r.long_run = units / starters < 1 ? 1 : units / starters < kLongRun ? units / starters : kLongRun;
    const int full = units > kTailItems ? (units - kTailItems) / kLongRun : 0, most = units / r.long_run;
    r.long_runs = full > starters ? full : starters;
    if (r.long_runs > most) r.long_runs = most;
    r.tail_run = r.long_run < 4 ? 1 : 2;
    r.n_tickets = r.long_runs + (units - r.long_runs * r.long_run + r.tail_run - 1) / r.tail_run;
    return r;
}

// The single-launch fused kernel (fused_small.hip): every level, the suffix and the merge for columns of 32 or 16 query rows.
constexpr int kSmallMaxSplits = 32;           // workgroups per column at most
constexpr int kSplitWorkgroups = 256;         // workgroups of a call whose columns are split, at most
// Device counters of a context: the combined launch's work counter, from kMeetingCounters on those of split columns: one for
// every number of workgroups per column (S) and column, so that a counter always counts to the same S.
constexpr int kContextCounters = 1024, kMeetingCounters = 32;
constexpr int meeting_counter(int S) {        // the first counter for S workgroups per column
    int at = kMeetingCounters;
    for (int s = 2; s < S; ++s) at += kSplitWorkgroups / s;
    return at;
}
static_assert(meeting_counter(kSmallMaxSplits + 1) <= kContextCounters, "");
// Workgroups of a single launch: XCD x (ids equal to x modulo 8) takes the x-th eighth of the list (KV head, tile, split), splits
// fastest (those of a column share its suffix rows and meet: 64 sequences x 8/1 heads, 4K keys, 512 rows, seven workgroups per column 14.8 us
// with the tiles fastest, 13.9 so).  false: nothing for this one.
__host__ __device__ inline unsigned small_grid(int n) { return 8u * (((unsigned)n + 7u) / 8u); }      // n: entries of the list
// by_head, by_split: division by tiles * splits and by splits
__host__ __device__ inline bool small_work(unsigned id, int tiles, int splits, int Hkv, Divider by_head, Divider by_split, int& kvh, int& tile, int& split) {
    const unsigned of_head = (unsigned)(tiles * splits), n = of_head * (unsigned)Hkv, x = id & 7u;
    const unsigned eighth = n >> 3, rest = n & 7u;       // x n / 8 without its 64 bits
    const unsigned first = x * eighth + (x * rest >> 3), count = eighth + (((x + 1) * rest >> 3) - (x * rest >> 3));
    if (id >> 3 >= count) return false;
    const unsigned at = first + (id >> 3);
    kvh = (int)by_head.of(at);
    const unsigned in_head = at - (unsigned)kvh * of_head;
    tile = (int)by_split.of(in_head);
    split = (int)(in_head - (unsigned)tile * (unsigned)splits);
    return true;
}
struct SmallArgs {
    // Everything but the further levels lies side by side: a wavefront reads it at its start with loads that wait for each other nowhere.
    const uint16_t* Q;
    const int32_t* lengths;   // null: no suffix
    const int32_t* offsets;
    Divider by_head, by_split, by_seq, by_group;      // division by tiles * splits, splits, nq * G, G
    int B, Hq, Hkv, G;
    int nq;
    int tiles;                // `rows` at a time of the B * nq * G query rows of one KV head
    int splits;               // workgroups per column
    int dealt;                // stages go to the wavefronts one by one (else in runs)
    int n_levels;
    int max_len;
    const uint16_t* Ks;
    const uint16_t* Vs;
    PagedDev pg;              // suffix read through a page table when pg.table != null
    float c2, tau_raw;        // scale * log2(e); by how much a raw score may pass the maximum before sums are rescaled (set by launch_fused_small)
    LevelDev lv[HG_MAX_LEVELS];
    int fp8;                  // suffix rows are E4M3 codes: value = code * scale
    float k_scale, v_scale;
    int fp32_weights;         // the weights of codes are not rounded to bf16
    int rows;                 // query rows of a column: 32 or 16
    int cols;                 // tiles * Hkv columns
    int wavefronts;           // of a workgroup: 8 or 4
    float* part;              // splits > 1: partial results (small_part_floats)
    unsigned* arrivals;       // splits > 1: [cols] counters that only ever count to `splits`, zero between calls
    float scale;
    void* O;                  // final results: [B, nq, Hq, D] bf16 or fp32, LSE [B, nq, Hq] (may be null)
    float* LSE;
    int bf16;
};

struct MergeArgs {
    int64_t rows;     // (first what a wavefront needs whatever the parts; the kernel reads it with the first parts' pointers at its start)
    void* O_out;
    float* L_out;     // may be null
    unsigned* clear;  // a counter to set to zero, or null
    int n;
    const float* L[HG_MAX_PARTS];
    const void* O[HG_MAX_PARTS];
};

// KV-cache update of a decode step: nq new rows per sequence appended to the suffix cache, lengths advanced.
struct AppendArgs {
    const uint16_t* Knew;     // [B, nq, Hkv, D]
    const uint16_t* Vnew;
    uint16_t* Ks;             // suffix cache (packed rows or page pool)
    uint16_t* Vs;
    const int32_t* offsets;   // unused when pg.table != null
    int32_t* lengths;
    PagedDev pg;
    int capacity;             // rows reserved per sequence
    int B, nq;
    int row_elems;            // Hkv * D
    int fp8;                  // the cache holds E4M3 codes: code = nearest(value / scale), saturating
    float k_scale, v_scale;
};

struct FillArgs {
    void* O; float* LSE; int bf16; int64_t rows; int D;
};

// ---- launchers (defined next to their kernels) ------------------------------------------------------
hipError_t launch_prefix_narrow(const PrefixArgs& a, int D, hipStream_t s);
hipError_t launch_prefix_wide(const PrefixArgs& a, int D, hipStream_t s);   // a.wide from plan_prefix_wide with the same D
hipError_t launch_prefix_wide_d64(const PrefixArgs& a, hipStream_t s);      // (the D = 64 kernel lives in its own translation unit)
hipError_t launch_combined_vector(const CombinedArgs& c, hipStream_t s);      // 256 workgroups; one query row per KV head
hipError_t launch_combined_vector_d64(const CombinedArgs& c, hipStream_t s);
hipError_t launch_combined_tiles(const CombinedArgs& c, hipStream_t s);       // several query rows per KV head, tiles of d.tile_rows
hipError_t launch_combined_tiles_d64(const CombinedArgs& c, hipStream_t s);   // (bf16 rows only)
bool plan_prefix_wide(const LevelDev& lv, int Hkv, int G, int D, int max_parts, int slots_per_xcd, WidePlan* out,
                      bool table = true);
hipError_t launch_decode(const DecodeArgs& a, int D, int GT, hipStream_t s);
hipError_t launch_decode_mfma(const DecodeArgs& a, int D, hipStream_t s);   // matrix-core per-sequence kernel (8-bit rows: D = 128 only)
hipError_t launch_merge(const MergeArgs& a, int D, bool in_bf16, bool out_bf16, hipStream_t s);
hipError_t launch_fused_small(const SmallArgs& a, int D, hipStream_t s);
size_t small_part_floats(int cols, int splits, int rows, int D);   // workspace floats of a split single launch
hipError_t launch_mfma_loop(int iters, int random_operands, unsigned long long* clocks, float* sink, hipStream_t s);
hipError_t launch_stream_read(const void* src, size_t bytes, float* sink, hipStream_t s);
hipError_t launch_xcd_probe(int n_workgroups, int* out, hipStream_t s);
hipError_t launch_fill_empty(const FillArgs& a, hipStream_t s);
hipError_t launch_kv_append(const AppendArgs& a, hipStream_t s);

constexpr int kPrefixRowsNarrow = 128;  // query rows per workgroup of the 128-row kernel (4 wavefronts x 32 rows)
constexpr int kPrefixRowsWide = 256;    // query rows per workgroup of the persistent kernel (8 wavefronts x 32 rows)
constexpr int kPrefixKeys = 64;         // keys per prefix LDS tile

// ---- small device helpers -------------------------------------------------------------------------
#ifdef __HIPCC__
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

// round-to-nearest-even fp32 -> bf16 bits (finite inputs; NaN stays NaN)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}
#endif

}  // namespace hg
