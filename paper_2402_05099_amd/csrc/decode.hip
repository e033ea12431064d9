// Per-sequence decode attention over a list of key spans: the suffix part of Hydragen (Sec. 3.2, last
// paragraph: one query per sequence, no batching across sequences) and, with the shared blocks added to
// the span list, the non-decomposed per-sequence comparison (what Sec. 1 / Sec. 2.3 say existing decode
// kernels do: every sequence re-reads the shared rows).  Memory-bound: one wavefront per work item
// (sequence, KV head, group of GT query heads, key chunk), 16-byte bf16 loads, fp32 arithmetic on the
// vector ALU, DPP reductions inside the 16-lane row that holds one key.
// FP8 = true (suffix rows only, packed or paged): the cache holds 8-bit E4M3 codes with one fp32 scale per tensor (not in the
// paper: half the bytes for the part of the method that is bound by them).  The same lanes own the same 8 columns,
// fetched with 8-byte loads and converted two at a time by the hardware; the K scale is folded into the query, the
// V scale into the final normalisation.
#include "decode_core.h"

namespace hg {

// SHARED = false: suffix rows only (the Hydragen suffix part).  SHARED = true: the shared blocks of every level
// are walked too (the non-decomposed comparison); a separate instantiation so that profiles tell them apart.
// PAGED (only without SHARED): the suffix rows are read through a page table.
// FP8 (only without SHARED): the suffix rows are E4M3 codes; a key is code * a.k_scale, a value code * a.v_scale.
template <int D, int GT, bool SHARED, bool PAGED, bool FP8 = false>
__global__ __launch_bounds__(256) void decode_kernel(DecodeArgs a) {
    constexpr int EPL = epl_of<D, GT, FP8>();   // columns per lane
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int64_t u = (int64_t)blockIdx.x * 4 + wave;
    if (u >= a.units) return;
    const int GB = a.G / GT;
    const int gb = (int)(u % GB); u /= GB;
    const int kvh = (int)(u % a.Hkv); u /= a.Hkv;
    const int c = (int)(u % a.nchunks);
    const int bq = (int)(u / a.nchunks);     // (sequence, query) pair: b*nq + t
    const int b = bq / a.nq;
    const int tq = bq % a.nq;
    const int h0 = kvh * a.G + gb * GT;  // first query head of this work item

    // Fresh state: query elements loaded and scaled, nothing seen yet.  (Here and not in a function: as one, paged 8-bit rows
    // got 90 registers instead of 108 and took 1 to 2 % longer.)
    DecodeState<D, GT, EPL> st;
    {
        constexpr int LPR = D / EPL;
        const int col = (lane % LPR) * EPL;
#pragma unroll
        for (int g = 0; g < GT; ++g) {
#pragma unroll
            for (int h8 = 0; h8 < EPL / 8; ++h8) {
                const uint4 qv = *reinterpret_cast<const uint4*>(a.Q + ((int64_t)bq * a.Hq + h0 + g) * D + col + 8 * h8);
                st.qp[g][4 * h8] = qv.x; st.qp[g][4 * h8 + 1] = qv.y; st.qp[g][4 * h8 + 2] = qv.z; st.qp[g][4 * h8 + 3] = qv.w;
            }
            st.m[g] = -INFINITY;
            st.l[g] = 0.f;
#pragma unroll
            for (int j = 0; j < EPL; ++j) st.acc[g][j] = 0.f;
        }
        st.qs = FP8 ? a.scale * kLog2e * a.k_scale : a.scale * kLog2e;
    }

    // walk the concatenated key list (shared blocks root first, then the suffix), clipped to this chunk
    const int64_t lo = (int64_t)c * a.chunk, hi = lo + a.chunk;
    int64_t pos = 0;
    if constexpr (SHARED)
        for (int li = 0; li < a.n_levels; ++li) {
            int begin, count;
            block_of(a.lv[li], b, a.B, begin, count);
            const int64_t s0 = max(lo, pos), s1 = min(hi, pos + count);
            if (s0 < s1) decode_span<D, GT, false, false, EPL>(st, a.lv[li].K, a.lv[li].V, begin + (s0 - pos), (int)(s1 - s0), a.Hkv, kvh, lane);
            pos += count;
        }
    if (a.lengths) {
        // the nq queries of a sequence are its last nq suffix tokens: query t does not see the later ones
        int count = min(a.lengths[b], a.max_len) - (a.nq - 1 - tq);
        if (count < 0) count = 0;
        const int64_t s0 = max(lo, pos), s1 = min(hi, pos + count);
        if (s0 < s1) {
            if constexpr (PAGED) decode_span_paged<D, GT, FP8, EPL>(st, a.Ks, a.Vs, a.pg, b, (int)s0, (int)(s1 - s0), a.Hkv, kvh, lane);
            else decode_span<D, GT, true, FP8, EPL>(st, a.Ks, a.Vs, a.offsets[b] + (s0 - pos), (int)(s1 - s0), a.Hkv, kvh, lane);
        }
    }

    decode_finish<D, GT, FP8, EPL>(st, a, bq, h0, c, lane);
}

template <int D, int GT>
static hipError_t launch_decode_t(const DecodeArgs& a, hipStream_t s) {
    if (a.units == 0) return hipSuccess;
    const int64_t grid = (a.units + 3) / 4;
    if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
    if (a.fp8) {
        if (a.n_levels > 0) return hipErrorInvalidValue;   // 8-bit rows: suffix only
        if (a.pg.table) decode_kernel<D, GT, false, true, true><<<(unsigned)grid, 256, 0, s>>>(a);
        else decode_kernel<D, GT, false, false, true><<<(unsigned)grid, 256, 0, s>>>(a);
    } else if (a.pg.table) {
        if (a.n_levels > 0) return hipErrorInvalidValue;   // the comparison kernel has no paged form
        decode_kernel<D, GT, false, true><<<(unsigned)grid, 256, 0, s>>>(a);
    } else if (a.n_levels > 0) {
        decode_kernel<D, GT, true, false><<<(unsigned)grid, 256, 0, s>>>(a);
    } else {
        decode_kernel<D, GT, false, false><<<(unsigned)grid, 256, 0, s>>>(a);
    }
    return hipGetLastError();
}

hipError_t launch_decode(const DecodeArgs& a, int D, int GT, hipStream_t s) {
    if (D == 128) {
        switch (GT) {
            case 1: return launch_decode_t<128, 1>(a, s);
            case 2: return launch_decode_t<128, 2>(a, s);
            case 4: return launch_decode_t<128, 4>(a, s);
            case 8: return launch_decode_t<128, 8>(a, s);
        }
    } else if (D == 64) {
        switch (GT) {
            case 1: return launch_decode_t<64, 1>(a, s);
            case 2: return launch_decode_t<64, 2>(a, s);
            case 4: return launch_decode_t<64, 4>(a, s);
            case 8: return launch_decode_t<64, 8>(a, s);
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace hg
