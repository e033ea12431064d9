// Shared block and suffix in ONE launch for calls with much work in both: the persistent shared-block kernel and the
// suffix kernel as two roles of the workgroups of one grid, one per CU.  The first 8 * wide.slots workgroups walk their
// pieces of the shared block (wide_role, prefix_wide_impl.h); every workgroup then takes suffix work items from a common
// counter until there are none left.  Compiled for D = 128 and D = 64 by combined.hip and combined_d64.hip.
//
// Why one launch: side by side on two streams the same two kernels pay for the event edges between the streams.  The
// second stream's kernel starts 6 us after the first, the merge 11 us after the last kernel's end and the next call 5 us
// later; kernels that follow each other on one stream are 1.2 us apart.  And a CU that is done with the shared block
// goes on with suffix rows at once, without a workgroup launch between any two work items.  Measured, two streams -> one
// launch: 256 x 40 heads, 2K keys, suffixes 1..256 153 -> 135 us; 1024 x 40 heads, suffixes 32..128: 16K keys 505 -> 485,
// 4K keys with an 8-bit cache 258 -> 233, 4K keys at D = 64 205 -> 183.  What bounds it: HBM and the board's power while the
// shared block runs, HBM afterwards (5.6 TB/s over the launch at 2K keys).
//
// Suffix role, one query row per KV head (SuffixStream; vector ALU, the arithmetic of decode.hip): a CU holds eight wavefronts here where
// decode.hip runs about twenty, so each has to keep more bytes in flight: a wavefront streams the batches (16 keys; 32 at
// D = 64) of its work items as one sequence, NB - 1 batches ahead of the one it multiplies, across the ends of work
// items.  Every batch is loaded by the same unconditional instructions (lanes past an item's last key re-read its
// first; a wavefront without further work re-reads its last batch's first key), so that the compiler's wait counts stay
// exact, and carries the item's query row along.
//
// Suffix role, several query rows per KV head (SuffixTiles; matrix cores, the arithmetic of decode_mfma.hip): decode_mfma.hip
// runs four wavefronts with two 16 KiB slots each on a CU; eight here have one K and one V slot of 8 KiB: the next stage's K
// rows are requested as soon as this stage's scores are done, its V rows after the value product, and across items the
// next item's first K rows during the last stage, its query tile (through the V slot) while the results are stored.
#include "decode_core.h"
#include "decode_mfma_core.h"
#include "prefix_wide_impl.h"

#pragma clang diagnostic ignored "-Winline-asm"

namespace hg {

namespace {

typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

// The workgroup's other LDS, behind the ring: the queue, the sequences per length class, and the order of the sequences.
constexpr int kQueueOffset = LDS_RING_BYTES, kCountsOffset = kQueueOffset + 64;
constexpr int kOrderOffset = kQueueOffset + 512, kMaxOrdered = (LDS_BYTES - kOrderOffset) / 2 / 1024 * 1024;
constexpr int kLengthClasses = 8;
static_assert(offsetof(CombinedArgs, p) == 0 && sizeof(CombinedArgs) <= 4096, "the kernarg segment");
static_assert(kLengthClasses * NW == 64, "one lane per class and wavefront");

// order[0 .. B): the sequences in descending order of their length class (eighths of max_len), by number within a class, so
// that the last items handed out are the short ones.  Every workgroup computes it for itself (512 lengths per round, read once if
// that is all; the prefix sum stays in the vector ALU) and all come to the same order.  Longest first against order of the sequences: 512 x 64/8 heads with suffixes of 1..512
// rows 148 -> 131 us, 256 x 40 heads, 1..256 rows 135 -> 127.
__device__ __forceinline__ void order_by_length(const DecodeArgs& a, unsigned char* smem) {
    uint16_t* const order = reinterpret_cast<uint16_t*>(smem + kOrderOffset);
    unsigned* const counts = reinterpret_cast<unsigned*>(smem + kCountsOffset);      // [class][wavefront]
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int seg = (a.B + 64 * NW - 1) / (64 * NW) * 64;           // sequences of one wavefront, a contiguous range
    const int b0 = min(w * seg, a.B), b1 = min(b0 + seg, a.B);
    const float per = (float)kLengthClasses / (float)(a.max_len + 1);
    auto class_of = [&](int b) -> int {
        const int n = b < b1 ? max(min(a.lengths[b], a.max_len), 0) : 0;
        return b < b1 ? kLengthClasses - 1 - min((int)((float)n * per), kLengthClasses - 1) : kLengthClasses;
    };
    int cnt[kLengthClasses] = {};
    const int k0 = class_of(b0 + lane);         // (up to 512 sequences: all there is, and its length is read once)
    for (int b = b0; b < b1; b += 64) {
        const int k = b == b0 ? k0 : class_of(b + lane);
#pragma unroll
        for (int i = 0; i < kLengthClasses; ++i) cnt[i] += __popcll(__ballot(k == i));
    }
    if (lane == 0)
#pragma unroll
        for (int i = 0; i < kLengthClasses; ++i) counts[i * NW + w] = cnt[i];
    __syncthreads();
    int at = (int)counts[lane];
    const int own = at;
    // exclusive prefix sum over (class, wavefront): within rows of 16 lanes, then the rows' totals
    at += __builtin_amdgcn_update_dpp(0, at, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8
    at += __builtin_amdgcn_update_dpp(0, at, 0x112, 0xf, 0xf, false);
    at += __builtin_amdgcn_update_dpp(0, at, 0x114, 0xf, 0xf, false);
    at += __builtin_amdgcn_update_dpp(0, at, 0x118, 0xf, 0xf, false);
    at += __builtin_amdgcn_update_dpp(0, at, 0x142, 0xa, 0xf, false);      // row_bcast:15 into rows 1 and 3
    at += __builtin_amdgcn_update_dpp(0, at, 0x143, 0xc, 0xf, false);      // row_bcast:31 into rows 2 and 3
    at -= own;
    int base[kLengthClasses];
#pragma unroll
    for (int i = 0; i < kLengthClasses; ++i) base[i] = __builtin_amdgcn_readlane(at, i * NW + w);
    for (int b = b0; b < b1; b += 64) {
        const int k = b == b0 ? k0 : class_of(b + lane);
#pragma unroll
        for (int i = 0; i < kLengthClasses; ++i) {
            const unsigned long long m = __ballot(k == i);
            if (k == i) order[base[i] + __popcll(m & ((1ull << lane) - 1))] = (uint16_t)(b + lane);
            base[i] += __popcll(m);
        }
    }
    __syncthreads();
}
// the sequence at position p of that order
__device__ __forceinline__ int sequence_at(const DecodeArgs& a, const unsigned char* smem, int p) {
    if (a.B > kMaxOrdered) return p;
    return __builtin_amdgcn_readfirstlane((int)reinterpret_cast<const uint16_t*>(smem + kOrderOffset)[p]);
}

// A workgroup's queue of work items, in LDS: items [pos, end) are left of the run it holds, pos in the low word.  pos
// beyond end: the run is used up and a wavefront is fetching the next one; end = 0: there are no more.
typedef unsigned long long queue_word;
constexpr queue_word kQueueEmpty = (1ull << 32) | 1u;
constexpr queue_word kQueueFinished = 0x40000000u;

// The items of ticket t: [base, stop), stop not beyond the last item.
__device__ __forceinline__ unsigned run_of(const CombinedArgs& ca, unsigned t, unsigned& stop) {
    const unsigned nl = (unsigned)ca.long_runs;
    const unsigned size = t < nl ? (unsigned)ca.long_run : (unsigned)ca.tail_run;
    const unsigned base = t < nl ? t * size : nl * (unsigned)ca.long_run + (t - nl) * size;
    stop = min(base + size, (unsigned)ca.d.units);
    return base;
}

// Tickets handed out without a draw (256 draws at one address take 3 us): a workgroup without shared-block work starts with
// ticket blockIdx.x - 8 * wide.slots; where every workgroup has shared-block work, so that all would draw at the same time
// after it, each starts with ticket blockIdx.x.
__device__ __forceinline__ unsigned first_ticket(const CombinedArgs& ca, unsigned& given) {
    const unsigned wide = 8 * ca.p.wide.slots;
    given = wide == gridDim.x ? wide : gridDim.x - wide;
    return wide == gridDim.x ? blockIdx.x : blockIdx.x - wide;      // (beyond `given` for a workgroup that starts without one)
}

// Next work item for this wavefront (-1: none left).  The wavefront that finds the run just used up draws the next
// ticket; the others look again until it has stored the new run (it depends on nobody).  Draws are few because all
// wavefronts of the chip make them at one address, 13 ns apart: with every wavefront drawing its items one by one, 40960
// of them took 557 us where this takes 300.
__device__ __forceinline__ int take_item(const CombinedArgs& ca, queue_word* queue) {
    const bool lane0 = (threadIdx.x & 63) == 0;
    for (;;) {
        queue_word old = 0;
        if (lane0) old = __hip_atomic_fetch_add(queue, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        const unsigned pos = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)old);
        const unsigned end = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(old >> 32));
        if (end == 0) return -1;
        if (pos < end) return (int)pos;
        if (pos == end) {
            unsigned given;
            first_ticket(ca, given);
            unsigned t = (unsigned)ca.n_tickets;
            if (given < t) {
                t = 0;
                if (lane0) t = __hip_atomic_fetch_add(ca.tickets, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                t = (unsigned)__builtin_amdgcn_readfirstlane((int)t) + given;
            }
            const bool any = t < (unsigned)ca.n_tickets;
            unsigned stop;
            const unsigned base = run_of(ca, t, stop);
            if (lane0)
                __hip_atomic_store(queue, any ? ((queue_word)stop << 32) | (base + 1) : kQueueFinished, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            return any ? (int)base : -1;
        }
        __builtin_amdgcn_s_sleep(2);
    }
}

template <bool PAGED, bool FP8>
struct SuffixStream {
    static constexpr int EPL = epl_of<D, 1, FP8>();
    static constexpr int LPR = D / EPL;
    static constexpr int KPW = 64 / LPR;             // keys per wave-wide load
    static constexpr int U = 4 / (EPL / 8);          // loads per tensor and batch
    static constexpr int STEP = KPW * U;             // keys per batch: 16 (D = 64: 32)
    static constexpr int NB = FP8 ? 6 : 4;           // batches a wavefront holds: 20 and 24 KiB in flight
    static constexpr int QW = EPL / 2;               // query words of this lane's columns
    static constexpr unsigned ES = FP8 ? 1u : 2u;

    struct Batch {
        KVBatch<D, U, FP8, EPL> kv;
        unsigned q[QW];
        int left;      // keys of the item from this batch on (0: no batch)
        int unit;      // the item's index in the results (query row * nchunks + chunk), and bit 31: this is its first batch
    };

    const CombinedArgs& ca;
    const DecodeArgs& a;
    const int lane, sub;
    const unsigned rstride_b, colb, subrow;
    // the item whose batches are being loaded
    unsigned char* const smem;
    queue_word* const queue;
    int no_more;              // the queue has been seen empty for good
    int left, first;          // keys not yet requested; the next batch is the item's first
    int cur_unit, cur_kvh;
    int pos, brow;            // paged: logical row of the next batch, its sequence
    const unsigned char* kb;  // the next batch's first row
    const unsigned char* vb;
    const unsigned char* qp;  // the item's query row
    // results that are kept (see below)
    unsigned char *ring_rows, *more_rows;
    int n_kept, kept_max;

    __device__ __forceinline__ SuffixStream(const CombinedArgs& c, unsigned char* sm, int l)
        : ca(c), a(c.d), lane(l), sub(l / LPR), rstride_b((unsigned)c.d.Hkv * D * ES), colb((unsigned)(l % LPR) * EPL * ES),
          subrow((unsigned)(l / LPR) * ((unsigned)c.d.Hkv * D * ES) + (unsigned)(l % LPR) * EPL * ES), smem(sm), queue(reinterpret_cast<queue_word*>(sm + kQueueOffset)) {
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int used = (kOrderOffset + (a.B <= kMaxOrdered ? 2 * a.B : 0) + 15) & ~15, more = (LDS_BYTES - used) / (NW * kRowBytes);
        ring_rows = smem + w * (LDS_RING_BYTES / NW);
        more_rows = smem + used + w * more * kRowBytes;
        kept_max = kInRing + more;
        n_kept = 0;
        no_more = 0;
        left = 0;
        first = 0;
        cur_unit = cur_kvh = 0;
        pos = brow = 0;
        kb = reinterpret_cast<const unsigned char*>(a.Q);     // a valid row of D elements, should there be no item at all
        vb = kb;
        qp = kb;
    }

    __device__ __forceinline__ void page_base() {     // paged: points kb / vb at logical row `pos` of sequence brow
        const const_i32_ptr table = (const_i32_ptr)(uintptr_t)a.pg.table;
        const int shift = a.pg.shift;
        int page = table[(int64_t)brow * a.pg.stride + min(pos >> shift, a.pg.stride - 1)];
        page = min(max(page, 0), a.pg.n_pages - 1);
        const int64_t off = (int64_t)((page << shift) + (pos & ((1 << shift) - 1))) * rstride_b + (int64_t)cur_kvh * (D * ES);
        kb = uniform_ptr(reinterpret_cast<const unsigned char*>(a.Ks) + off);
        vb = uniform_ptr(reinterpret_cast<const unsigned char*>(a.Vs) + off);
    }

    // moves on to the next item with keys; items without keys get their empty result on the way
    __device__ __forceinline__ void next_item() {
        const const_i32_ptr lengths = (const_i32_ptr)(uintptr_t)a.lengths;
        const const_i32_ptr offsets = (const_i32_ptr)(uintptr_t)a.offsets;
        for (;;) {
            if (no_more) return;
            const int u = take_item(ca, queue);
            if (u < 0) { no_more = 1; return; }
            const int bc = (int)a.by_heads.of((unsigned)u), kvh = __builtin_amdgcn_readfirstlane(u - bc * a.Hkv);
            const int p = (int)a.by_chunks.of((unsigned)bc), c = __builtin_amdgcn_readfirstlane(bc - p * a.nchunks), b = sequence_at(a, smem, __builtin_amdgcn_readfirstlane(p));
            const int count = min(lengths[b], a.max_len);
            const int lo = c * a.chunk;
            const int n = __builtin_amdgcn_readfirstlane(min(count - lo, a.chunk));
            if (n <= 0) {
                if (lane == 0) a.out.LSE[(int64_t)c * a.out.part_stride_L + (int64_t)b * a.Hq + kvh] = -INFINITY;
                continue;
            }
            cur_unit = (b * a.Hq + kvh) * a.nchunks + c;
            cur_kvh = kvh;
            left = n;
            first = 1;
            qp = uniform_ptr(reinterpret_cast<const unsigned char*>(a.Q + ((int64_t)b * a.Hq + kvh) * D));
            if constexpr (PAGED) {
                brow = b;
                pos = lo;
                page_base();
            } else {
                const int64_t off = (((int64_t)offsets[b] + lo) * a.Hkv + kvh) * (int64_t)(D * ES);
                kb = uniform_ptr(reinterpret_cast<const unsigned char*>(a.Ks) + off);
                vb = uniform_ptr(reinterpret_cast<const unsigned char*>(a.Vs) + off);
            }
            return;
        }
    }

    __device__ __forceinline__ void produce(Batch& bt) {
        if (left <= 0) next_item();
        left = __builtin_amdgcn_readfirstlane(left);
        bt.left = left;
        bt.unit = __builtin_amdgcn_readfirstlane(cur_unit | (first << 31));
        first = 0;
        const unsigned char* const kp = kb;
        const unsigned char* const vp = vb;
        {
            const unsigned qo = (unsigned)(lane % LPR) * EPL * 2u;
#pragma unroll
            for (int i = 0; i < QW / 4; ++i) {
                const uint4 v = ldg128<false>(qp, qo + 16 * i);
                bt.q[4 * i] = v.x; bt.q[4 * i + 1] = v.y; bt.q[4 * i + 2] = v.z; bt.q[4 * i + 3] = v.w;
            }
        }
        if (PAGED && STEP > 16) {
            // a batch of 32 rows may span two pages of 16: its second half is addressed from a page of its own
            const int half_pos = pos;
            const unsigned char* const k0 = kp;
            const unsigned char* const v0 = vp;
            const unsigned char* k1 = kp + (size_t)16 * rstride_b;
            const unsigned char* v1 = vp + (size_t)16 * rstride_b;
            if (left > 16) {
                pos += 16;
                page_base();
                k1 = kb;
                v1 = vb;
                pos = half_pos;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = u * KPW + sub < left;
                const unsigned off = in ? (unsigned)((u * KPW) % 16) * rstride_b + subrow : colb;
                const unsigned char* const ku = u * KPW < 16 || left <= 16 ? k0 : k1;
                const unsigned char* const vu = u * KPW < 16 || left <= 16 ? v0 : v1;
                bt.kv.k[u] = ldg_row<true, FP8 && EPL == 8>(ku, off);
                bt.kv.v[u] = ldg_row<true, FP8 && EPL == 8>(vu, off);
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = u * KPW + sub < left;
                const unsigned off = in ? (unsigned)(u * KPW) * rstride_b + subrow : colb;
                bt.kv.k[u] = ldg_row<true, FP8 && EPL == 8>(kp, off);
                bt.kv.v[u] = ldg_row<true, FP8 && EPL == 8>(vp, off);
            }
        }
        left -= STEP;
        if (left > 0) {
            if constexpr (PAGED) {
                pos += STEP;
                page_base();
            } else {
                kb += (size_t)STEP * rstride_b;
                vb += (size_t)STEP * rstride_b;
            }
        }
    }

    __device__ __forceinline__ void run() {
        Batch bt[NB];
        DecodeState<D, 1, EPL> st;
        st.m[0] = -INFINITY;
        st.l[0] = 0.f;
        st.qs = (FP8 ? a.scale * a.k_scale : a.scale) * kLog2e;
#pragma unroll
        for (int j = 0; j < EPL; ++j) st.acc[0][j] = 0.f;
#pragma unroll
        for (int i = 0; i < NB - 1; ++i) produce(bt[i]);
        // (no way out of the middle of the loop: past the last item the batches are empty)
        do {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                produce(bt[(i + NB - 1) % NB]);
                __builtin_amdgcn_sched_barrier(0);      // keep the loads ahead of the arithmetic that hides their latency
                Batch& cb = bt[i];
                if (cb.left > 0) {
                    if (cb.unit < 0) {
#pragma unroll
                        for (int j = 0; j < QW; ++j) st.qp[0][j] = cb.q[j];
                        st.m[0] = -INFINITY;
                        st.l[0] = 0.f;
#pragma unroll
                        for (int j = 0; j < EPL; ++j) st.acc[0][j] = 0.f;
                    }
                    consume_batch<D, 1, U, FP8, EPL>(st, cb.kv, sub, cb.left);
                    if (cb.left <= STEP) {
                        const int u = cb.unit & 0x7fffffff;
                        if (n_kept < kept_max) keep(st, u);
                        else {
                            const int row = (int)a.by_chunks.of((unsigned)u);
                            decode_finish<D, 1, FP8, EPL>(st, a, 0, row, u - row * a.nchunks, lane);
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } while (bt[NB - 1].left > 0);
        write_kept();
    }

    // ---- results ------------------------------------------------------------------------------------------------------------
    // Written one by one while the rows stream in, results cost the HBM far more time than their bytes: 8-bit suffixes of 32..128
    // rows, 1024 x 40 heads, hardly a shared block: the last rows are read at 171 us, and at 147 without the writes, which
    // are 2.5 % of the bytes.  So a wavefront keeps its results in LDS (the ring's, which this role does not need, and what is
    // left behind the order of the sequences) and writes them when it has no more rows to read; one that finds no room is written at once.
    // (Merging them right there with the parts of the shared levels, and passing over such rows in the merge kernel, was no
    // faster: those parts have to come past the XCD's caches, in a phase as long as the merge kernel.)
    // Measured, us: 1024 x 40 heads, 16K keys 494 -> 484; D = 64, 4K keys 187.8 -> 184.6; 2048 x 40, two levels 562 -> 549; 256 x 40, 2K keys 128.6 ->
    // 127.3; 8-bit rows, 4K keys, where the shared block ends last, 233.4 -> 233.1 (hardly a shared block: 183 -> 170).
    static constexpr int kRowBytes = D * 4 + 16;                          // O, LSE, index in the results
    static constexpr int kInRing = LDS_RING_BYTES / NW / kRowBytes;       // results of a wavefront in the ring's memory
    __device__ __forceinline__ unsigned char* kept_row(int i) const {
        return i < kInRing ? ring_rows + i * kRowBytes : more_rows + (i - kInRing) * kRowBytes;
    }

    __device__ __forceinline__ void keep(const DecodeState<D, 1, EPL>& st, int unit) {
        constexpr int N = EPL / 4;
        float M, l, o[N];
        decode_combine<D, 1, EPL>(st, 0, M, l, o);
        unsigned char* const p = kept_row(n_kept);
        const float inv = l > 0.f ? (FP8 ? a.v_scale / l : 1.0f / l) : 0.f;
        if (LPR == 16 || !(lane & 8)) {
            float* const op = reinterpret_cast<float*>(p) + combined_col<D, EPL>(lane);
            if constexpr (N == 4) *reinterpret_cast<float4*>(op) = make_float4(o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
            else *reinterpret_cast<float2*>(op) = make_float2(o[0] * inv, o[1] * inv);
        }
        if (lane == 0) *reinterpret_cast<float2*>(p + D * 4) = make_float2(l > 0.f ? (M + __log2f(l)) * kLn2 : -INFINITY, __builtin_bit_cast(float, unit));
        n_kept = __builtin_amdgcn_readfirstlane(n_kept + 1);
    }

    __device__ __forceinline__ void write_kept() const {
        constexpr int LR = D / 4;                     // lanes per row
        const int col = 4 * (lane % LR);
        for (int i = lane / LR; i < n_kept; i += 64 / LR) {
            const unsigned char* const p = kept_row(i);
            const float2 info = *reinterpret_cast<const float2*>(p + D * 4);
            const int unit = __builtin_bit_cast(int, info.y), row = (int)a.by_chunks.of((unsigned)unit), c = unit - row * a.nchunks;
            // (past the caches: the merge reads them once, see store_part)
            __builtin_nontemporal_store(*reinterpret_cast<const uintx4*>(p + col * 4),
                                        reinterpret_cast<uintx4*>(static_cast<float*>(a.out.O) + (int64_t)c * a.out.part_stride_O + (int64_t)row * D + col));
            if (col == 0) a.out.LSE[(int64_t)c * a.out.part_stride_L + row] = info.x;
        }
    }
};

// Several query rows per KV head: a work item is (sequence, KV head, tile of TR query rows, key chunk), as in decode_mfma.hip.
template <bool PAGED, bool FP8, int TR>
struct SuffixTiles {
    using Tile = dm::MfmaTile<D, FP8, TR>;
    using G_ = dm::Geo<D>;
    static constexpr int KEYS = dm::KT, CPSG = Tile::CPSG, RPIG = Tile::RPIG, CPRG = Tile::CPRG, QOPS = Tile::QOPS, ES = Tile::ES;
    static constexpr int kSlot = 8192;               // K slot, then V slot, per wavefront
    static_assert(KEYS * D * ES <= kSlot && TR * D * 2 <= kSlot, "a stage's rows and a query tile fit a slot");
    static_assert(NW * 2 * kSlot <= LDS_RING_BYTES, "the slots lie in the ring's memory");

    struct Item {
        int b, c, rt, kvh;
        int off, count;      // first suffix row of the sequence in Ks/Vs; suffix rows the newest query sees
        int ks, ke;          // absolute rows [ks, ke) of this item's keys
        int kwin, nst;       // first row of the last full window of the range (packed rows); stages
    };

    const CombinedArgs& ca;
    const DecodeArgs& a;
    unsigned char* const smem;
    queue_word* const queue;
    const int l, R, RT;
    const unsigned rstride_b;
    unsigned char* const lds;
    unsigned ldsb;
    int no_more;
    unsigned voffK[CPSG], voffV[CPSG], voffQ[QOPS];      // lane offsets of the copies: K/V stage rows, query tile rows
    int voff_clamp, voff_rt;                             // the row clamp / row tile they were computed for
    int pg0, pg1;                                        // paged: pages of the stage whose K rows were requested last
    int lane_rt, lane_tq, lane_g;                        // this lane's row of tile lane_rt: query, head in the group
    bool rv;

    __device__ __forceinline__ SuffixTiles(const CombinedArgs& c, unsigned char* sm)
        : ca(c), a(c.d), smem(sm), queue(reinterpret_cast<queue_word*>(sm + kQueueOffset)), l(threadIdx.x & 63), R(c.d.nq * c.d.G), RT((c.d.nq * c.d.G + TR - 1) / TR),
          rstride_b((unsigned)c.d.Hkv * D * ES), lds(sm + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * (2 * kSlot)) {
        ldsb = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(uintptr_t)HG_LDS(lds));
        no_more = 0;
        voff_clamp = voff_rt = lane_rt = -1;
        pg0 = pg1 = 0;
        lane_tq = lane_g = 0;
        rv = false;
    }

    __device__ __forceinline__ void lane_of(const Item& it) {
        if (it.rt != lane_rt) {
            lane_rt = it.rt;
            const int r = it.rt * TR + (TR == 16 ? (l & 15) : (l & 31));
            rv = r < R;
            const int rr = rv ? r : 0;
            lane_tq = (int)a.by_group.of((unsigned)rr);
            lane_g = rr - lane_tq * a.G;
        }
    }
    __device__ __forceinline__ int64_t row_of(const Item& it) const { return ((int64_t)it.b * a.nq + lane_tq) * a.Hq + it.kvh * a.G + lane_g; }

    // the next item with keys (false: none left) and the lane offsets of its copies; items without keys get their empty result
    __device__ __forceinline__ bool next_item(Item& it) {
        const const_i32_ptr lengths = (const_i32_ptr)(uintptr_t)a.lengths;
        const const_i32_ptr offsets = (const_i32_ptr)(uintptr_t)a.offsets;
        for (;;) {
            if (no_more) return false;
            const int u = take_item(ca, queue);
            if (u < 0) { no_more = 1; return false; }
            const int by_head = (int)a.by_heads.of((unsigned)u), by_tile = (int)a.by_tiles.of((unsigned)by_head), p = (int)a.by_chunks.of((unsigned)by_tile);
            it.kvh = __builtin_amdgcn_readfirstlane(u - by_head * a.Hkv);
            it.rt = __builtin_amdgcn_readfirstlane(by_head - by_tile * RT);
            it.c = __builtin_amdgcn_readfirstlane(by_tile - p * a.nchunks);
            it.b = sequence_at(a, smem, __builtin_amdgcn_readfirstlane(p));
            it.count = __builtin_amdgcn_readfirstlane(max(min(lengths[it.b], a.max_len), 0));
            it.off = PAGED ? 0 : __builtin_amdgcn_readfirstlane(offsets[it.b]);
            const int lo = it.c * a.chunk, hi = min(lo + a.chunk, it.count);
            if (lo < hi) {
                it.ks = __builtin_amdgcn_readfirstlane(it.off + lo);
                it.ke = __builtin_amdgcn_readfirstlane(it.off + hi);
                break;
            }
            lane_of(it);
            if (rv && l < TR) a.out.LSE[(int64_t)it.c * a.out.part_stride_L + row_of(it)] = -INFINITY;
        }
        it.kwin = PAGED ? 0x3fffffff : max(it.ke - KEYS, 0);     // paged: stages stay where they are, rows past ke are masked
        it.nst = (it.ke - it.ks + KEYS - 1) / KEYS;
        const int rowclamp = PAGED ? KEYS - 1 : min(it.ke - 1 - it.kwin, KEYS - 1);   // < 31 only when the range ends before row 32 of the tensor
        if (rowclamp != voff_clamp) {
            voff_clamp = rowclamp;
#pragma unroll
            for (int i = 0; i < CPSG; ++i) {
                const int srow = i * RPIG + l / CPRG, ch = l % CPRG;
                const unsigned ro = (unsigned)min(srow, rowclamp) * rstride_b;
                if (FP8) {
                    voffK[i] = ro + (unsigned)((ch ^ ((srow >> 1) & 7)) * 16);
                    voffV[i] = ro + (unsigned)((ch ^ (((srow >> 1) & 1) | (((srow >> (TR == 16 ? 4 : 3)) & 1) << 1))) * 16);
                } else {
                    voffK[i] = ro + (unsigned)((ch ^ G_::kswz(srow)) * 16);
                    voffV[i] = ro + (unsigned)((ch ^ G_::vswz(srow)) * 16);
                }
            }
        }
        if (it.rt != voff_rt) {
            voff_rt = it.rt;
#pragma unroll
            for (int i = 0; i < QOPS; ++i) {
                const int srow = i * G_::RPI + l / G_::CPR;
                int r = it.rt * TR + srow;
                if (r >= R) r = 0;
                const int tq = (int)a.by_group.of((unsigned)r);
                voffQ[i] = (unsigned)(tq * a.Hq + r - tq * a.G) * G_::ROWB + (unsigned)(((l % G_::CPR) ^ G_::kswz(srow)) * 16);
            }
        }
        return true;
    }

    // ---- copies, issued from inline asm and waited for with counted s_waitcnt (see decode_mfma.hip) ----
    __device__ __forceinline__ void copy16(const unsigned char* sbase, unsigned voff, unsigned lds_dst) const {
        asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(voff), "s"(sbase), "s"(lds_dst) : "memory", "m0");
    }
    __device__ __forceinline__ void issue_rows(const Item& it, int t, const uint16_t* base, const unsigned (&voff)[CPSG], unsigned dst) const {
        const unsigned char* const bp = reinterpret_cast<const unsigned char*>(base);
        if constexpr (PAGED) {
            const int r0 = it.ks + t * KEYS, ps_mask = (1 << a.pg.shift) - 1;
#pragma unroll
            for (int i = 0; i < CPSG; ++i) {
                const int jr = r0 + i * RPIG;
                const int64_t prow = ((int64_t)(i < CPSG / 2 ? pg0 : pg1) << a.pg.shift) + (jr & ps_mask);
                copy16(uniform_ptr(bp + prow * rstride_b + (int64_t)it.kvh * (D * ES)), voff[i] - (unsigned)(i * RPIG) * rstride_b, dst + i * 1024);
            }
        } else {
            const int k0c = min(it.ks + t * KEYS, it.kwin);
            const unsigned char* const g = uniform_ptr(bp + (int64_t)k0c * rstride_b + (int64_t)it.kvh * (D * ES));
#pragma unroll
            for (int i = 0; i < CPSG; ++i) copy16(g, voff[i], dst + i * 1024);
        }
    }
    __device__ __forceinline__ void issue_k(const Item& it, int t) {
        if constexpr (PAGED) {     // the four or eight rows of one copy lie in one page (pages hold a power of two >= 16 rows)
            const const_i32_ptr table = (const_i32_ptr)(uintptr_t)a.pg.table;
            const int64_t trow = (int64_t)it.b * a.pg.stride;
            const int r0 = it.ks + t * KEYS;
            pg0 = __builtin_amdgcn_readfirstlane(min(max(table[trow + min(r0 >> a.pg.shift, a.pg.stride - 1)], 0), a.pg.n_pages - 1));
            pg1 = __builtin_amdgcn_readfirstlane(min(max(table[trow + min((r0 + KEYS / 2) >> a.pg.shift, a.pg.stride - 1)], 0), a.pg.n_pages - 1));
        }
        issue_rows(it, t, a.Ks, voffK, ldsb);
    }
    __device__ __forceinline__ void issue_v(const Item& it, int t) const { issue_rows(it, t, a.Vs, voffV, ldsb + kSlot); }
    __device__ __forceinline__ void issue_q(const Item& it) const {
        const unsigned char* const q = uniform_ptr(reinterpret_cast<const unsigned char*>(a.Q + ((int64_t)it.b * a.nq * a.Hq + it.kvh * a.G) * D));
#pragma unroll
        for (int i = 0; i < QOPS; ++i) copy16(q, voffQ[i], ldsb + kSlot + i * (G_::RPI * G_::ROWB));
    }

    __device__ __forceinline__ void run() {
        Item nx{};
        if (!next_item(nx)) return;
        Tile tile(FP8 ? a.scale * a.k_scale : a.scale, l);
        unsigned char* const vslot = lds + kSlot;
        // K rows of the first stage, query tile (through the V slot), V rows of the first stage
        auto begin = [&]() {
            dm::wait_vm<0>();                     // the query tile, and the K rows requested before it
            asm volatile("" ::: "memory");
            tile.load_q(vslot);
            issue_v(nx, 0);
        };
        issue_k(nx, 0);
        issue_q(nx);
        begin();
        for (bool more = true; more;) {
            const Item it = nx;
            lane_of(it);
            const int vis_end = it.off + it.count - (a.nq - 1 - lane_tq);     // this lane's query sees absolute rows below vis_end
            const int causal_from = it.off + it.count - (a.nq - 1);           // below this row every query sees every key
            tile.clear();
            for (int t = 0; t < it.nst; ++t) {
                const bool last = t + 1 == it.nst;
                if (t > 0) {
                    dm::wait_vm<CPSG>();          // at most this stage's V rows are outstanding: its K rows are there
                    asm volatile("" ::: "memory");
                }
                typename Tile::Scores S;
                uintx4 pb[2];
                tile.scores(lds, S);
                if constexpr (TR == 16) asm volatile("" : "+v"(S.S4[0]), "+v"(S.S4[1]));     // the K rows have been read
                else asm volatile("" : "+v"(S.S));
                asm volatile("" ::: "memory");
                if (!last) {
                    issue_k(it, t + 1);
                } else {
                    more = next_item(nx);
                    if (more) issue_k(nx, 0);
                }
                const int key0 = it.ks + t * KEYS, k0c = min(key0, it.kwin);
                // stage rows before the stage's first key (window clamp), past the range, and not visible to this lane's query yet
                if (k0c != key0 || key0 + KEYS > it.ke || key0 + KEYS > causal_from) tile.mask(S, key0 - k0c, min(it.ke, vis_end) - k0c);
                tile.softmax(S, pb);
                if (!last || more) dm::wait_vm<CPSG>();     // at most the K rows just requested are outstanding
                else dm::wait_vm<0>();
                asm volatile("" ::: "memory");
                // rows that are nobody's keys may hold anything
                if (PAGED && key0 + KEYS > it.ke) tile.clear_v_from(vslot, it.ke - key0);
                if (k0c != key0) tile.clear_v_below(vslot, key0 - k0c);
                tile.values(vslot, pb);
                if (!last) issue_v(it, t + 1);
            }
            if (more) {
                issue_q(nx);
                begin();
            }
            // (the stores follow the next item's first V rows: nothing waits for them before those have landed)
            lane_of(it);
            tile.store(a.out, it.c, row_of(it), rv, a.v_scale);
        }
    }
};

template <bool PAGED, bool FP8>
struct VectorRole {
    static __device__ __forceinline__ void run(const CombinedArgs& c, unsigned char* smem) {
        SuffixStream<PAGED, FP8> s(c, smem, threadIdx.x & 63);
        s.run();
    }
};
template <bool PAGED, bool FP8, int TR>
struct TileRole {
    static __device__ __forceinline__ void run(const CombinedArgs& c, unsigned char* smem) {
        SuffixTiles<PAGED, FP8, TR> s(c, smem);
        s.run();
    }
};

template <class Role>
__global__ __launch_bounds__(64 * NW, 1) void combined_kernel(CombinedArgs c) {
    unsigned char* const smem = wide_smem;
    // The arguments that either role reads on its way to the first request: their lines, which no cache holds at the start of a launch (0.4 us each), are
    // loaded at once instead of one behind the other.  1024 x 8/1 heads, 16K keys 79.5 -> 79.1 us, others equal.
    asm volatile("" ::"s"(c.p.lv.K), "s"(c.p.Hkv), "s"(c.p.by_heads.mul), "s"(c.p.scale), "s"(c.p.out.O), "s"(c.p.out.part_stride_L), "s"(c.p.wide.n_c),
                 "s"(c.p.wide.mode), "s"(c.p.wide.by_teams.mul), "s"(c.p.wide.by_cut[1].mul));
    asm volatile("" ::"s"(c.d.Q), "s"(c.d.Ks), "s"(c.d.lengths), "s"(c.d.pg.table), "s"(c.d.max_len), "s"(c.d.nchunks), "s"(c.d.by_heads.mul),
                 "s"(c.d.by_group.mul), "s"(c.d.scale), "s"(c.d.out.O), "s"(c.d.out.part_stride_L), "s"(c.n_more), "s"(c.tickets), "s"(c.n_tickets));
    if (blockIdx.x < 8 * c.p.wide.slots) {
        const wide_args_ptr first = (wide_args_ptr)__builtin_amdgcn_kernarg_segment_ptr();
        for (int i = 0; i <= c.n_more; ++i) {
            const size_t at = i == 0 ? 0 : offsetof(CombinedArgs, more) + (i - 1) * sizeof(MoreLevel);
            wide_role((wide_args_ptr)((const __attribute__((address_space(4))) unsigned char*)first + at));
            __builtin_amdgcn_s_waitcnt(0x0F70);      // copies that nobody consumed have landed
            __syncthreads();
        }
    }
    queue_word* const queue = reinterpret_cast<queue_word*>(smem + kQueueOffset);
    if (threadIdx.x == 0) {
        queue_word first = kQueueEmpty;
        unsigned given;
        const unsigned t = first_ticket(c, given);
        if (t < given && t < (unsigned)c.n_tickets) {
            unsigned stop;
            const unsigned base = run_of(c, t, stop);
            first = ((queue_word)stop << 32) | base;
        }
        *queue = first;
    }
    if (c.d.B <= kMaxOrdered) order_by_length(c.d, smem);
    __syncthreads();
    Role::run(c, smem);
}

template <class Role>
hipError_t launch_role(const CombinedArgs& c, hipStream_t s) {
    static bool attr_set[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64 && !attr_set[dev]) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&combined_kernel<Role>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    combined_kernel<Role><<<256, 64 * NW, LDS_BYTES, s>>>(c);
    return hipGetLastError();
}

}  // namespace

// One translation unit per head dimension and kind of suffix role.
#if HG_WIDE_D == 128 && defined(HG_COMBINED_TILES)
hipError_t launch_combined_tiles(const CombinedArgs& c, hipStream_t s) {
#elif HG_WIDE_D == 128
hipError_t launch_combined_vector(const CombinedArgs& c, hipStream_t s) {
#elif defined(HG_COMBINED_TILES)
hipError_t launch_combined_tiles_d64(const CombinedArgs& c, hipStream_t s) {
#else
hipError_t launch_combined_vector_d64(const CombinedArgs& c, hipStream_t s) {
#endif
    const bool paged = c.d.pg.table != nullptr;
#ifndef HG_COMBINED_TILES
    if (paged) return c.d.fp8 ? launch_role<VectorRole<true, true>>(c, s) : launch_role<VectorRole<true, false>>(c, s);
    return c.d.fp8 ? launch_role<VectorRole<false, true>>(c, s) : launch_role<VectorRole<false, false>>(c, s);
#else
#if HG_WIDE_D == 128
    if (c.d.fp8 && c.d.tile_rows == 16) return paged ? launch_role<TileRole<true, true, 16>>(c, s) : launch_role<TileRole<false, true, 16>>(c, s);
    if (c.d.fp8) return hipErrorInvalidValue;      // (the caller keeps 8-bit codes in 32-row tiles on the separate kernels)
#else
    if (c.d.fp8) return hipErrorInvalidValue;      // 8-bit rows on the matrix cores: D = 128 only
#endif
    if (c.d.tile_rows == 16) return paged ? launch_role<TileRole<true, false, 16>>(c, s) : launch_role<TileRole<false, false, 16>>(c, s);
    return paged ? launch_role<TileRole<true, false, 32>>(c, s) : launch_role<TileRole<false, false, 32>>(c, s);
#endif
}

}  // namespace hg
