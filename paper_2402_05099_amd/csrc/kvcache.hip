// KV-cache update of a decode step (Sec. 2.2: the cache holds the keys and values of all earlier tokens and every
// step adds the newest token's; Sec. 3.5: suffix lengths change from step to step while the launch sequence stays
// the same, so lengths live on the device and are advanced there).  Pure data movement: one workgroup per sequence
// copies the nq new K and V rows behind the sequence's last suffix row, then its first thread advances the length.
#include <algorithm>
#include <type_traits>

#include "hg_internal.h"

namespace hg {

// E4M3 codes of eight bf16 values divided by `scale`: the fp32 quotient (correctly rounded division), magnitudes
// above 448 saturated, then the hardware's round-to-nearest-even conversion; NaN stays NaN.
__device__ __forceinline__ uint2 quantize8(const uint4& r, float scale) {
    const float f[8] = {bf16_lo(r.x), bf16_hi(r.x), bf16_lo(r.y), bf16_hi(r.y), bf16_lo(r.z), bf16_hi(r.z), bf16_lo(r.w), bf16_hi(r.w)};
    float q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float x = f[i] / scale;
        q[i] = x != x ? x : fminf(fmaxf(x, -448.0f), 448.0f);
    }
    int lo = 0, hi = 0;
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], lo, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], lo, true);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(q[4], q[5], hi, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(q[6], q[7], hi, true);
    return make_uint2((unsigned)lo, (unsigned)hi);
}

// What bounds it: a chain of loads (arguments, length, page, each 0.4 - 0.8 us), so whatever does not depend on the length is requested
// with it: a thread's first piece of the new rows, the sequence's offset.  One thread per 16-byte piece of K and V, up to
// 1024: a workgroup must cover its sequence, for the length may only be advanced when all have read it.
// (256 threads, rows requested behind the length and the page before.)  Steps with codes: 10 x 40 heads 18.2 -> 16.0 us, 6 x 40 34.7 -> 31.5;
// 6 x 40, D = 64, four new rows 13.3 -> 11.7; 128 x 32/8, paged 44.4 -> 44.2; 17 drawn steps 1.039 in the mean.
// FP8: the cache holds E4M3 codes, the rows are quantised on the way in.
template <bool FP8>
__global__ __launch_bounds__(1024) void kv_append_kernel(AppendArgs a) {
    using Piece = std::conditional_t<FP8, uint2, uint4>;
    const int b = blockIdx.x, n = blockDim.x;
    const int vec = a.row_elems / 8;       // 8-element groups per row (Hkv * D is a multiple of 64): 16 bytes of bf16
    const int most = a.nq * vec;
    const uint4* const Kn = reinterpret_cast<const uint4*>(a.Knew) + (int64_t)b * most;
    const uint4* const Vn = reinterpret_cast<const uint4*>(a.Vnew) + (int64_t)b * most;
    int i = threadIdx.x;
    const int len = a.lengths[b];          // every thread reads the old length before thread 0 replaces it
    const int off = a.pg.table ? 0 : a.offsets[b];
    uint4 k = Kn[min(i, most - 1)], v = Vn[min(i, most - 1)];
    __syncthreads();
    const int room = a.capacity - len;
    const int take = len < 0 ? 0 : room < a.nq ? (room > 0 ? room : 0) : a.nq;   // rows that fit below the capacity
    const int end = take * vec;
    while (i < end) {
        const int t = i / vec, c = i - t * vec;
        const int j = len + t;             // suffix row that token t becomes
        int64_t row;
        if (a.pg.table) {
            int page = a.pg.table[(int64_t)b * a.pg.stride + (j >> a.pg.shift)];
            page = min(max(page, 0), a.pg.n_pages - 1);
            row = ((int64_t)page << a.pg.shift) + (j & ((1 << a.pg.shift) - 1));
        } else {
            row = (int64_t)off + j;
        }
        const int64_t dst = row * vec + c;
        Piece kp, vp;
        if constexpr (FP8) {
            kp = quantize8(k, a.k_scale);
            vp = quantize8(v, a.v_scale);
        } else {
            kp = k;
            vp = v;
        }
        i += n;
        if (i < end) {
            k = Kn[i];
            v = Vn[i];
        }
        reinterpret_cast<Piece*>(a.Ks)[dst] = kp;
        reinterpret_cast<Piece*>(a.Vs)[dst] = vp;
    }
    if (threadIdx.x == 0 && take > 0) a.lengths[b] = len + take;
}

hipError_t launch_kv_append(const AppendArgs& a, hipStream_t s) {
    if (a.B == 0) return hipSuccess;
    const int64_t pieces = (int64_t)a.nq * (a.row_elems / 8);
    const unsigned threads = (unsigned)std::min<int64_t>(1024, (pieces + 63) / 64 * 64);
    if (a.fp8) kv_append_kernel<true><<<(unsigned)a.B, threads, 0, s>>>(a);
    else kv_append_kernel<false><<<(unsigned)a.B, threads, 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace hg
