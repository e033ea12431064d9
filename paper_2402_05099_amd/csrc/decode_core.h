// The wavefront-level pieces of the vector-ALU suffix kernel (decode.hip), used by it and by the combined launch
// (combined_impl.h): loads, scores, online softmax and value sums of one work item, and its result's way out.
#pragma once
#include <type_traits>

#include "hg_internal.h"

namespace hg {

template <int CTRL>
__device__ __forceinline__ float dpp_f32(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

// sum over the LPR (8 or 16) lanes that share one key row; every lane of the row gets the total
template <int LPR>
__device__ __forceinline__ float row_allreduce_sum(float x) {
    x += dpp_f32<0xB1>(x);   // quad_perm [1,0,3,2]
    x += dpp_f32<0x4E>(x);   // quad_perm [2,3,0,1]
    x += dpp_f32<0x141>(x);  // row_half_mirror: pairs the two quads of each 8 lanes
    if constexpr (LPR == 16) x += dpp_f32<0x140>(x);  // row_mirror: pairs the two halves of 16 lanes
    return x;
}

// tells the compiler that a pointer is the same in every lane of the wavefront (it then lives in scalar registers)
__device__ __forceinline__ const unsigned char* uniform_ptr(const unsigned char* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<const unsigned char*>(((uint64_t)hi << 32) | lo);
}

// Columns of a row that one lane owns: 8 (one 16-byte load of bf16, one 8-byte load of codes), or 16 codes (one
// 16-byte load) where registers allow: an 8-bit row of D = 128 is then covered by 8 lanes, a wave-wide load brings 8
// keys instead of 4, and the per-key overhead (cross-lane sum, exponential, masks) halves per byte.
template <int D, int GT, bool FP8>
constexpr int epl_of() { return (FP8 && D == 128 && GT <= 2) ? 16 : 8; }

// Rows are multiplied two elements at a time with v_dot2_f32_bf16 (products of bf16 values are exact in fp32, the
// sums are taken in fp32): the score of a bf16 row is four such instructions on the packed words of K and Q as they come from memory
// (codes are expanded to packed bf16 values first, exactly, two to an instruction), and the value sums of bf16 rows take the rounded weights of two
// keys against those keys' values of one column.  The values of codes are multiplied with fp32 weights.
typedef __bf16 bf16pair __attribute__((ext_vector_type(2)));
typedef float f32pair __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned pack_pair_bf16(float lo, float hi) {      // v_cvt_pk_bf16_f32, round to nearest even
    f32pair f = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f, bf16pair));
}
__device__ __forceinline__ float dot2_bf16(unsigned a, unsigned b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16pair, a), __builtin_bit_cast(bf16pair, b), c, false);
}

constexpr float kLazy = 8.f;      // log2 units

template <int D, int GT, int EPL = 8>
struct DecodeState {
    unsigned qp[GT][EPL / 2];   // query elements of this lane's column slice, packed bf16 pairs
    float qs;            // scale*log2(e) (codes: times their K scale), applied to a score after its sum
    float m[GT];         // running max (log2 domain); codes: a score that no score has passed by more than kLazy
    float l[GT];         // running sum of 2^(s-m)
    float acc[GT][EPL];  // running sum of 2^(s-m) * v
};

// One batch of U wave-wide loads: KPW keys each, K and V rows of this lane's 8-column slice.
template <int D, int U, bool FP8, int EPL = 8>
struct KVBatch {
    using Row = std::conditional_t<FP8 && EPL == 8, uint2, uint4>;   // this lane's EPL elements of a row
    Row k[U], v[U];
};

// 16-byte load from global memory at uniform base + 32-bit lane offset (scalar base register + vector offset form)
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// STREAM: rows read exactly once (suffix KV) bypass the caches' retention; shared rows are loaded normally so that
// the re-reads of other sequences can hit in L2 / Infinity Cache
template <bool STREAM>
__device__ __forceinline__ uint4 ldg128(const unsigned char* base, unsigned off) {
    const auto* p = reinterpret_cast<const __attribute__((address_space(1))) u32x4*>(
        (const __attribute__((address_space(1))) unsigned char*)base + off);
    const u32x4 v = STREAM ? __builtin_nontemporal_load(p) : *p;
    return make_uint4(v.x, v.y, v.z, v.w);
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <bool STREAM>
__device__ __forceinline__ uint2 ldg64(const unsigned char* base, unsigned off) {
    const auto* p = reinterpret_cast<const __attribute__((address_space(1))) u32x2*>(
        (const __attribute__((address_space(1))) unsigned char*)base + off);
    const u32x2 v = STREAM ? __builtin_nontemporal_load(p) : *p;
    return make_uint2(v.x, v.y);
}
template <bool STREAM, bool HALF>
__device__ __forceinline__ auto ldg_row(const unsigned char* base, unsigned off) {
    if constexpr (HALF) return ldg64<STREAM>(base, off);
    else return ldg128<STREAM>(base, off);
}

// this lane's 16 or 8 codes of a row as fp32
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void unpack_codes(const uint4& r, float (&f)[16]) {
    const unsigned w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[j], false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)w[j], true);
        f[4 * j] = a.x; f[4 * j + 1] = a.y; f[4 * j + 2] = b.x; f[4 * j + 3] = b.y;
    }
}
__device__ __forceinline__ void unpack_codes(const uint2& r, float (&f)[8]) {
    const f32x2 a = __builtin_amdgcn_cvt_pk_f32_fp8((int)r.x, false), b = __builtin_amdgcn_cvt_pk_f32_fp8((int)r.x, true);
    const f32x2 c = __builtin_amdgcn_cvt_pk_f32_fp8((int)r.y, false), d = __builtin_amdgcn_cvt_pk_f32_fp8((int)r.y, true);
    f[0] = a.x; f[1] = a.y; f[2] = b.x; f[3] = b.y; f[4] = c.x; f[5] = c.y; f[6] = d.x; f[7] = d.y;
}

// this lane's elements of a row as packed bf16 pairs
__device__ __forceinline__ void pairs_of(const uint4& r, unsigned (&p)[4]) { p[0] = r.x; p[1] = r.y; p[2] = r.z; p[3] = r.w; }
template <int N, class Row>
__device__ __forceinline__ void pairs_of_codes(const Row& r, unsigned (&p)[N]) {
    const unsigned* const w = reinterpret_cast<const unsigned*>(&r);
#pragma unroll
    for (int j = 0; j < N / 2; ++j) {
        p[2 * j] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[j], 1.0f, false));
        p[2 * j + 1] = __builtin_bit_cast(unsigned, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w[j], 1.0f, true));
    }
}

// kb/vb: wavefront-uniform byte pointers to the span's first row of this KV head; rowoff: this lane's byte offset
// of its key in load 0 of the batch (sub-row, column slice and batch start); colb: the column part alone.  Lanes
// whose key lies past the span read the span's first row instead (always valid; their score is masked), so no
// load is predicated and a batch may be requested past the end of the span.
template <int D, int U, bool STREAM, bool FP8, int EPL>
__device__ __forceinline__ void load_batch(KVBatch<D, U, FP8, EPL>& bt, const unsigned char* __restrict__ kb,
                                           const unsigned char* __restrict__ vb, unsigned rstride_b, unsigned rowoff,
                                           unsigned colb, int first, int n) {
    constexpr int KPW = 64 / (D / EPL);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = first + u * KPW;   // `first` already includes this lane's sub-row
        const unsigned off = i < n ? (unsigned)(u * KPW) * rstride_b + rowoff : colb;
        bt.k[u] = ldg_row<STREAM, FP8 && EPL == 8>(kb, off);
        bt.v[u] = ldg_row<STREAM, FP8 && EPL == 8>(vb, off);
    }
}

// online-softmax update of the state with one batch (keys first + u*KPW, masked beyond n)
template <int D, int GT, int U, bool FP8, int EPL>
__device__ __forceinline__ void consume_batch(DecodeState<D, GT, EPL>& st, const KVBatch<D, U, FP8, EPL>& bt, int first, int n) {
    constexpr int LPR = D / EPL;
    constexpr int KPW = 64 / LPR;
    float s[U][GT];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool ok = first + u * KPW < n;
        unsigned kw[EPL / 2];
        if constexpr (FP8) pairs_of_codes(bt.k[u], kw);
        else pairs_of(bt.k[u], kw);
#pragma unroll
        for (int g = 0; g < GT; ++g) {
            float d0 = 0.f, d1 = 0.f;       // two chains
#pragma unroll
            for (int j = 0; j < EPL / 2; j += 2) {
                d0 = dot2_bf16(kw[j], st.qp[g][j], d0);
                d1 = dot2_bf16(kw[j + 1], st.qp[g][j + 1], d1);
            }
            const float d = row_allreduce_sum<LPR>(d0 + d1) * st.qs;
            s[u][g] = ok ? d : -INFINITY;
        }
    }
#pragma unroll
    for (int g = 0; g < GT; ++g) {
        float mx = st.m[g];
#pragma unroll
        for (int u = 0; u < U; ++u) mx = fmaxf(mx, s[u][g]);
        // (fp32 weights lose nothing when the largest is not 1: sums are rescaled only when a score passes the maximum by kLazy.  bf16
        // weights do: the largest would be rounded)
        float alpha = 1.0f;
        if (!FP8 || __any(mx > st.m[g] + kLazy)) {
            alpha = __builtin_amdgcn_exp2f(st.m[g] - ((mx == -INFINITY) ? 0.f : mx));
            st.m[g] = mx;
            if constexpr (FP8) {
                st.l[g] *= alpha;
#pragma unroll
                for (int j = 0; j < EPL; ++j) st.acc[g][j] *= alpha;
            }
        }
        const float ms = (st.m[g] == -INFINITY) ? 0.f : st.m[g];
        float p[U];
        float ps = 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            p[u] = __builtin_amdgcn_exp2f(s[u][g] - ms);
            ps += p[u];
        }
        if constexpr (FP8) {
            st.l[g] += ps;
        } else {
            st.l[g] = fmaf(st.l[g], alpha, ps);
#pragma unroll
            for (int j = 0; j < EPL; ++j) st.acc[g][j] *= alpha;
        }
        if constexpr (!FP8) {
            static_assert(FP8 || U % 2 == 0, "keys are taken in pairs");
            // weights of two keys, rounded to bf16 (as the matrix-core kernels round theirs; the row sum above keeps
            // the unrounded ones), against the two keys' values of one column: v_perm_b32 gathers the column's pair
#pragma unroll
            for (int u = 0; u < U; u += 2) {
                const unsigned pp = pack_pair_bf16(p[u], p[u + 1]);
                const unsigned va[4] = {bt.v[u].x, bt.v[u].y, bt.v[u].z, bt.v[u].w};
                const unsigned vb[4] = {bt.v[u + 1].x, bt.v[u + 1].y, bt.v[u + 1].z, bt.v[u + 1].w};
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const unsigned lo = __builtin_amdgcn_perm(vb[w], va[w], 0x05040100u);   // (va.lo, vb.lo)
                    const unsigned hi = __builtin_amdgcn_perm(vb[w], va[w], 0x07060302u);   // (va.hi, vb.hi)
                    st.acc[g][2 * w] = dot2_bf16(lo, pp, st.acc[g][2 * w]);
                    st.acc[g][2 * w + 1] = dot2_bf16(hi, pp, st.acc[g][2 * w + 1]);
                }
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float v[EPL];
                unpack_codes(bt.v[u], v);
#pragma unroll
                for (int j = 0; j < EPL; ++j) st.acc[g][j] = fmaf(p[u], v[j], st.acc[g][j]);
            }
        }
    }
}

// Online-softmax pass over `n` consecutive KV rows starting at row0, KV head kvh.  Software pipelined: the
// loads of the next batch are issued before the current batch is consumed, so a wavefront always has a
// batch in flight while it computes.
template <int D, int GT, bool STREAM, bool FP8 = false, int EPL = 8>
__device__ __forceinline__ void decode_span(DecodeState<D, GT, EPL>& st, const uint16_t* __restrict__ K,
                                            const uint16_t* __restrict__ V, int64_t row0, int n, int Hkv, int kvh,
                                            int lane) {
    constexpr int LPR = D / EPL;
    constexpr int KPW = 64 / LPR;
    constexpr int U = (GT >= 8 ? 2 : 4) / (EPL / 8);   // the same keys per batch whatever a lane owns of a row
    constexpr int STEP = KPW * U;
    constexpr unsigned ES = FP8 ? 1u : 2u;     // bytes per element
    const int sub = lane / LPR;
    const unsigned rstride_b = (unsigned)Hkv * D * ES;
    const unsigned colb = (unsigned)(lane % LPR) * EPL * ES;
    unsigned rowoff = (unsigned)sub * rstride_b + colb;
    const int64_t first_b = (row0 * Hkv + kvh) * (int64_t)D * ES;
    const unsigned char* kb = uniform_ptr(reinterpret_cast<const unsigned char*>(K) + first_b);
    const unsigned char* vb = uniform_ptr(reinterpret_cast<const unsigned char*>(V) + first_b);
    const unsigned step_b = (unsigned)STEP * rstride_b;

    // every load is issued unconditionally (see load_batch), so the wait counts the compiler derives are exact
    KVBatch<D, U, FP8, EPL> ba, bb;
    load_batch<D, U, STREAM, FP8, EPL>(ba, kb, vb, rstride_b, rowoff, colb, sub, n);
    for (int it = 0; it < n; it += 2 * STEP) {
        rowoff += step_b;
        load_batch<D, U, STREAM, FP8, EPL>(bb, kb, vb, rstride_b, rowoff, colb, it + STEP + sub, n);
        __builtin_amdgcn_sched_barrier(0);   // keep the loads ahead of the arithmetic that hides their latency
        consume_batch<D, GT, U, FP8, EPL>(st, ba, it + sub, n);
        rowoff += step_b;
        __builtin_amdgcn_sched_barrier(0);
        load_batch<D, U, STREAM, FP8, EPL>(ba, kb, vb, rstride_b, rowoff, colb, it + 2 * STEP + sub, n);
        __builtin_amdgcn_sched_barrier(0);
        if (it + STEP < n) consume_batch<D, GT, U, FP8, EPL>(st, bb, it + STEP + sub, n);
    }
}

// The same pass over rows [start, start+n) of sequence b's suffix when the rows live in a paged pool (`start` is a
// multiple of 32, the span touches at most 64 pages: the host bounds the chunk by 32 pages).  Lane i of the
// wavefront holds the physical page of the span's i-th logical page; the 4 or 8 keys of one wave-wide load (64 lanes / lanes per row) never
// straddle a page (pages hold at least 16 rows), so the page of a load is wavefront-uniform: one v_readlane and
// a few scalar instructions per load, the same unpredicated vector loads and the same pipeline as above.
template <int D, int GT, bool FP8 = false, int EPL = 8>
__device__ __forceinline__ void decode_span_paged(DecodeState<D, GT, EPL>& st, const uint16_t* __restrict__ K,
                                                  const uint16_t* __restrict__ V, const PagedDev& pg, int b, int start,
                                                  int n, int Hkv, int kvh, int lane) {
    constexpr int LPR = D / EPL;
    constexpr int KPW = 64 / LPR;
    constexpr int U = (GT >= 8 ? 2 : 4) / (EPL / 8);
    constexpr int STEP = KPW * U;
    constexpr unsigned ES = FP8 ? 1u : 2u;     // bytes per element
    const int sub = lane / LPR;
    const unsigned rstride_b = (unsigned)Hkv * D * ES;
    const unsigned colb = (unsigned)(lane % LPR) * EPL * ES;
    const unsigned subrow = (unsigned)sub * rstride_b + colb;
    const unsigned char* kb = uniform_ptr(reinterpret_cast<const unsigned char*>(K) + (int64_t)kvh * D * ES);
    const unsigned char* vb = uniform_ptr(reinterpret_cast<const unsigned char*>(V) + (int64_t)kvh * D * ES);
    const int shift = pg.shift;
    const int lp0 = start >> shift;
    const int lpn = ((start + n - 1) >> shift) - lp0 + 1;
    int pages = 0;
    if (lane < lpn) pages = pg.table[(int64_t)b * pg.stride + lp0 + lane];
    pages = min(max(pages, 0), pg.n_pages - 1);
    // byte offset of the pool row that holds the span's key i0 (i0: wavefront-uniform multiple of KPW)
    auto row_base = [&](int i0) -> unsigned {
        const int pos = start + i0;
        const int page = __builtin_amdgcn_readlane(pages, ((pos >> shift) - lp0) & 63);
        return ((unsigned)(page << shift) + (unsigned)(pos & ((1 << shift) - 1))) * rstride_b;
    };
    const unsigned safe = row_base(0) + colb;   // lanes past the span read its first row (their scores are masked)
    auto load = [&](KVBatch<D, U, FP8, EPL>& bt, int i0) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int iu = i0 + u * KPW;
            const unsigned off = iu + sub < n ? row_base(iu) + subrow : safe;
            bt.k[u] = ldg_row<true, FP8 && EPL == 8>(kb, off);
            bt.v[u] = ldg_row<true, FP8 && EPL == 8>(vb, off);
        }
    };

    KVBatch<D, U, FP8, EPL> ba, bb;
    load(ba, 0);
    for (int it = 0; it < n; it += 2 * STEP) {
        load(bb, it + STEP);
        __builtin_amdgcn_sched_barrier(0);
        consume_batch<D, GT, U, FP8, EPL>(st, ba, it + sub, n);
        __builtin_amdgcn_sched_barrier(0);
        load(ba, it + 2 * STEP);
        __builtin_amdgcn_sched_barrier(0);
        if (it + STEP < n) consume_batch<D, GT, U, FP8, EPL>(st, bb, it + STEP + sub, n);
    }
}

// rows [begin, begin+count) of the block of level `lv` that covers sequence b (count = 0 if none)
__device__ __forceinline__ void block_of(const LevelDev& lv, int b, int B, int& begin, int& count) {
    if (lv.n_blocks == 1 && lv.seq_off == nullptr) {
        begin = 0;
        count = lv.max_rows;
        return;
    }
    int lo = 0, hi = lv.n_blocks;  // find g with seq_off[g] <= b < seq_off[g+1]
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (lv.seq_off[mid + 1] <= b) lo = mid + 1;
        else hi = mid;
    }
    begin = 0;
    count = 0;
    if (lo < lv.n_blocks && lv.seq_off[lo] <= b) {
        begin = lv.kv_off[lo];
        count = min(lv.kv_off[lo + 1] - begin, lv.max_rows);
        if (count < 0) count = 0;
    }
}

// Combines the 64/LPR key sub-streams of the wavefront for query head g: maximum (0 if there is none) and sum in every lane; of the value
// sums a lane keeps EPL / 4, those of columns combined_col(lane) and up (with 8 lanes to a row, lanes 8 apart keep the same ones).
// The lanes that hold parts of a column are 8, 16 and 32 apart: a swap of 32-lane halves (rows of 16 lanes) between two registers and an
// addition sum two columns at once, each in the half (row) that keeps it, in place of an exchange through LDS for every column (16 columns of
// codes, maximum and sum: 54 exchanges before, 16 swaps and 6 rotations within rows of 16 lanes now).  With scores of codes by dot products (24 -> 16 instructions a key) and sums that are rescaled
// past kLazy only: 1024 x 40 heads, 4K keys, suffixes of 32..128 codes 226.7 -> 223.6 us, error of O on the suffixes alone 1.17e-7 -> 1.00e-7;
// bf16 rows, 256 x 40, 2K keys 122.0 -> 121.8, 1024 x 40, 16K keys 470.5 -> 469.7, 2048 x 40, two levels 548.7 -> 549.4.
template <int D, int EPL>
__device__ __forceinline__ int combined_col(int lane) {
    return lane % (D / EPL) * EPL + (lane & 32 ? EPL / 2 : 0) + (lane & 16 ? EPL / 4 : 0);
}
template <int LPR, class F>
__device__ __forceinline__ float over_substreams(float x, F f) {
    // (the value of the lane 32 or 16 away, picked by lane: taking both results of a swap of a register with itself for the pair is folded away)
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    x = f(x, __builtin_bit_cast(float, threadIdx.x & 32 ? r[0] : r[1]));
    const auto t = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
    x = f(x, __builtin_bit_cast(float, threadIdx.x & 16 ? t[0] : t[1]));
    if constexpr (LPR == 8) x = f(x, dpp_f32<0x128>(x));      // row_ror:8
    return x;
}
template <int D, int GT, int EPL>
__device__ __forceinline__ void decode_combine(const DecodeState<D, GT, EPL>& st, int g, float& Ms, float& l, float (&o)[EPL / 4]) {
    constexpr int LPR = D / EPL;
    static_assert(LPR == 8 || LPR == 16, "");
    const auto sum = [](float a, float b) { return a + b; };
    const auto bits = [](float v) { return __builtin_bit_cast(unsigned, v); };
    const auto value = [](unsigned v) { return __builtin_bit_cast(float, v); };
    const float M = over_substreams<LPR>(st.m[g], [](float a, float b) { return fmaxf(a, b); });
    Ms = (M == -INFINITY) ? 0.f : M;
    const float f = __builtin_amdgcn_exp2f(st.m[g] - Ms);
    l = over_substreams<LPR>(st.l[g] * f, sum);
    float h[EPL / 2];
#pragma unroll
    for (int j = 0; j < EPL / 2; ++j) {
        const auto r = __builtin_amdgcn_permlane32_swap(bits(st.acc[g][j] * f), bits(st.acc[g][j + EPL / 2] * f), false, false);
        h[j] = value(r[0]) + value(r[1]);
    }
#pragma unroll
    for (int j = 0; j < EPL / 4; ++j) {
        const auto r = __builtin_amdgcn_permlane16_swap(bits(h[j]), bits(h[j + EPL / 4]), false, false);
        o[j] = value(r[0]) + value(r[1]);
        if constexpr (LPR == 8) o[j] += dpp_f32<0x128>(o[j]);
    }
}

// Combines the sub-streams and writes (O, LSE) of chunk c.
template <int D, int GT, bool FP8, int EPL>
__device__ __forceinline__ void decode_finish(const DecodeState<D, GT, EPL>& st, const DecodeArgs& a, int bq, int h0, int c, int lane) {
    constexpr int LPR = D / EPL, N = EPL / 4;
#pragma unroll
    for (int g = 0; g < GT; ++g) {
        float Ms, l, o[N];
        decode_combine<D, GT, EPL>(st, g, Ms, l, o);
        const float inv = l > 0.f ? (FP8 ? a.v_scale / l : 1.0f / l) : 0.f;
        const int64_t idx = (int64_t)bq * a.Hq + h0 + g;
        if (LPR == 16 || !(lane & 8)) {
            const int64_t e = (int64_t)c * a.out.part_stride_O + idx * D + combined_col<D, EPL>(lane);
            if (a.out.bf16) {
                unsigned* const op = reinterpret_cast<unsigned*>(static_cast<uint16_t*>(a.out.O) + e);
                if constexpr (N == 4) *reinterpret_cast<uint2*>(op) = make_uint2(pack_bf16(o[0] * inv, o[1] * inv), pack_bf16(o[2] * inv, o[3] * inv));
                else *op = pack_bf16(o[0] * inv, o[1] * inv);
            } else {
                float* const op = static_cast<float*>(a.out.O) + e;
                if constexpr (N == 4) *reinterpret_cast<float4*>(op) = make_float4(o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
                else *reinterpret_cast<float2*>(op) = make_float2(o[0] * inv, o[1] * inv);
            }
        }
        if (lane == 0) a.out.LSE[(int64_t)c * a.out.part_stride_L + idx] = l > 0.f ? (Ms + __log2f(l)) * kLn2 : -INFINITY;
    }
}

}  // namespace hg
