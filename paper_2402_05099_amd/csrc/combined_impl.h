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
// Suffix role (one query row per KV head, vector ALU, the arithmetic of decode.hip): a CU holds eight wavefronts here where
// decode.hip runs about twenty, so each has to keep more bytes in flight: a wavefront streams the batches (16 keys; 32 at
// D = 64) of its work items as one sequence, NB - 1 batches ahead of the one it multiplies, across the ends of work
// items.  Every batch is loaded by the same unconditional instructions (lanes past an item's last key re-read its
// first; a wavefront without further work re-reads its last batch's first key), so that the compiler's wait counts stay
// exact, and carries the item's query row along.
#include "decode_core.h"
#include "prefix_wide_impl.h"

namespace hg {

namespace {

typedef const __attribute__((address_space(4))) int32_t* const_i32_ptr;

// A workgroup's queue of work items, in LDS: items [pos, end) are left of the run it holds, pos in the low word.  pos
// beyond end: the run is used up and a wavefront is fetching the next one; end = 0: there are no more.
typedef unsigned long long queue_word;
constexpr queue_word kQueueEmpty = (1ull << 32) | 1u;
constexpr queue_word kQueueFinished = 0x40000000u;

// The items of ticket t: [base, stop), stop not beyond the last item.
__device__ __forceinline__ unsigned run_of(const CombinedArgs& ca, unsigned t, unsigned& stop) {
    const unsigned nl = (unsigned)ca.long_runs;
    const unsigned base = t < nl ? t * kLongRun : nl * kLongRun + (t - nl) * kTailRun;
    stop = min(base + (t < nl ? kLongRun : kTailRun), (unsigned)ca.d.units);
    return base;
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
            unsigned t = 0;
            if (lane0) t = __hip_atomic_fetch_add(ca.tickets, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            t = (unsigned)__builtin_amdgcn_readfirstlane((int)t);
            t += (unsigned)(gridDim.x - 8 * ca.p.wide.slots);      // tickets handed out in advance, see the kernel
            unsigned stop;
            const unsigned base = run_of(ca, t, stop);
            const unsigned units = (unsigned)ca.d.units;
            const bool any = base < units;
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
        int unit;      // the item, and bit 31: this is its first batch
    };

    const CombinedArgs& ca;
    const DecodeArgs& a;
    const int lane, sub;
    const unsigned rstride_b, colb, subrow;
    // the item whose batches are being loaded
    queue_word* const queue;
    int no_more;              // the queue has been seen empty for good
    int left, first;          // keys not yet requested; the next batch is the item's first
    int cur_unit, cur_kvh;
    int pos, brow;            // paged: logical row of the next batch, its sequence
    const unsigned char* kb;  // the next batch's first row
    const unsigned char* vb;
    const unsigned char* qp;  // the item's query row

    __device__ __forceinline__ SuffixStream(const CombinedArgs& c, queue_word* qu, int l)
        : ca(c), a(c.d), lane(l), sub(l / LPR), rstride_b((unsigned)c.d.Hkv * D * ES), colb((unsigned)(l % LPR) * EPL * ES),
          subrow((unsigned)(l / LPR) * ((unsigned)c.d.Hkv * D * ES) + (unsigned)(l % LPR) * EPL * ES), queue(qu) {
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
            const int kvh = __builtin_amdgcn_readfirstlane(u % a.Hkv), bc = __builtin_amdgcn_readfirstlane(u / a.Hkv);
            const int c = __builtin_amdgcn_readfirstlane(bc % a.nchunks), b = __builtin_amdgcn_readfirstlane(bc / a.nchunks);
            const int count = min(lengths[b], a.max_len);
            const int lo = c * a.chunk;
            const int n = __builtin_amdgcn_readfirstlane(min(count - lo, a.chunk));
            if (n <= 0) {
                if (lane == 0) a.out.LSE[(int64_t)c * a.out.part_stride_L + (int64_t)b * a.Hq + kvh] = -INFINITY;
                continue;
            }
            cur_unit = u;
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
                        for (int j = 0; j < QW; ++j) {
                            st.qp[0][j] = cb.q[j];
                            st.q[0][2 * j] = bf16_lo(cb.q[j]) * st.qs;
                            st.q[0][2 * j + 1] = bf16_hi(cb.q[j]) * st.qs;
                        }
                        st.m[0] = -INFINITY;
                        st.l[0] = 0.f;
#pragma unroll
                        for (int j = 0; j < EPL; ++j) st.acc[0][j] = 0.f;
                    }
                    consume_batch<D, 1, U, FP8, EPL>(st, cb.kv, sub, cb.left);
                    if (cb.left <= STEP) {
                        const int u = cb.unit & 0x7fffffff;
                        const int kvh = u % a.Hkv, bc = u / a.Hkv;
                        decode_finish<D, 1, FP8, EPL>(st, a, bc / a.nchunks, kvh, bc % a.nchunks, lane);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } while (bt[NB - 1].left > 0);
    }
};

template <bool PAGED, bool FP8>
__global__ __launch_bounds__(64 * NW, 1) void combined_kernel(CombinedArgs c) {
    unsigned char* const smem = wide_smem;
    if (blockIdx.x < 8 * c.p.wide.slots) {
        wide_role(c.p);
        __builtin_amdgcn_s_waitcnt(0x0F70);      // copies that nobody consumed have landed
        __syncthreads();
    }
    queue_word* const queue = reinterpret_cast<queue_word*>(smem);
    unsigned* const done = reinterpret_cast<unsigned*>(smem + 16);     // wavefronts of this workgroup that are done
    if (threadIdx.x == 0) {
        // a workgroup without shared-block work has its first ticket without a draw (256 draws at once take 3 us)
        queue_word first = kQueueEmpty;
        if (blockIdx.x >= 8 * c.p.wide.slots) {
            unsigned stop;
            const unsigned base = run_of(c, blockIdx.x - 8 * c.p.wide.slots, stop);
            if (base < stop) first = ((queue_word)stop << 32) | base;
        }
        *queue = first;
        *done = 0;
    }
    __syncthreads();
    {
        SuffixStream<PAGED, FP8> s(c, queue, threadIdx.x & 63);
        s.run();
    }
    // no wavefront of this workgroup draws any more once all eight are here: the last workgroup of the launch sets the
    // counters back to zero for the next call
    if ((threadIdx.x & 63) == 0) {
        __builtin_amdgcn_s_waitcnt(0x0F70);
        if (__hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) == NW - 1) {
            unsigned* const wgs = c.tickets + 32;
            if (__hip_atomic_fetch_add(wgs, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1) {
                __hip_atomic_store(c.tickets, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(wgs, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

template <bool PAGED, bool FP8>
hipError_t launch_combined_t(const CombinedArgs& c, hipStream_t s) {
    static bool attr_set[64] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < 64 && !attr_set[dev]) {
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(&combined_kernel<PAGED, FP8>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        if (e != hipSuccess) return e;
        attr_set[dev] = true;
    }
    combined_kernel<PAGED, FP8><<<256, 64 * NW, LDS_BYTES, s>>>(c);
    return hipGetLastError();
}

}  // namespace

#if HG_WIDE_D == 128
hipError_t launch_combined(const CombinedArgs& c, int head_dim, hipStream_t s) {
    if (head_dim == 64) return launch_combined_d64(c, s);
#else
hipError_t launch_combined_d64(const CombinedArgs& c, hipStream_t s) {
#endif
    if (c.d.pg.table) return c.d.fp8 ? launch_combined_t<true, true>(c, s) : launch_combined_t<true, false>(c, s);
    return c.d.fp8 ? launch_combined_t<false, true>(c, s) : launch_combined_t<false, false>(c, s);
}

}  // namespace hg
