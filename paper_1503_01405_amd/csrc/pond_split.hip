// Split middle pass for blocks of 2^25 .. 2^27 samples: the row transform
// of length n1 = m2 m1 (m1 = 2^13, m2 = 4 .. 16), too long for one
// workgroup's LDS, is done in four steps of its own (Sec. 3.7 computes the
// whole block's spectrum; this only changes how the transform is cut):
//   split_cols (forward): per row k2 and column c < m1, the m2 values at
//     c + m1 i times the block twiddle exp(-2 pi i k2 (c + m1 i) / N),
//     transformed over i, times exp(-2 pi i c k / n1), stored at c + m1 k;
//   K2 kRowChirp: each sub-row k (m1 contiguous values) transformed, times
//     the chirp at frequency k2 + n2 (k + m2 c'), transformed back;
//   split_cols (inverse): the first step conjugated, in reverse order.
// One thread holds the m2 values of two adjacent columns of a row k2: the
// accesses of a wave are 128 consecutive columns and the transform is in
// registers.  Bound: memory (one read and write of the block per pass).  It
// was bound by its twiddle lookups, 3 m2 scattered 8-byte loads per column
// from tables in L2; the loads left scattered are one or two per column, the
// rest are in order (values unchanged).  2^26 in float32: 508 us a pass ->
// about 250 (1.07 GB, 4.3 TB/s; a large copy reaches 5.4).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cmath>

#include "pond_device.hpp"

namespace pond {

namespace {

__device__ __forceinline__ float2 ld_f2(const float2* p) { return *p; }
__device__ __forceinline__ float2 ld_f2(const __half2* p) { return to_f2(__builtin_bit_cast(h2, *p)); }
__device__ __forceinline__ void st_f2(float2* p, float2 v) { *p = v; }
__device__ __forceinline__ void st_f2(__half2* p, float2 v) { *p = __builtin_bit_cast(__half2, to_h2(v)); }
__device__ __forceinline__ float2 ld_f2(const bf16x2* p) { return Elem<bf16x2>::load(p); }
__device__ __forceinline__ void st_f2(bf16x2* p, float2 v) { Elem<bf16x2>::store(p, v); }

// Two adjacent columns of a row: one access per value pair.
template <class T>
struct Pair2;
template <>
struct Pair2<float2> {
    float4 u;
    __device__ __forceinline__ float2 get(int i) const { return i ? make_float2(u.z, u.w) : make_float2(u.x, u.y); }
    __device__ __forceinline__ static Pair2 make(float2 a, float2 b) { return {make_float4(a.x, a.y, b.x, b.y)}; }
};
template <class T>
struct Pair2 {
    static_assert(sizeof(T) == 4, "16-bit pairs");
    uint2 u;
    __device__ __forceinline__ float2 get(int i) const {
        const T t = __builtin_bit_cast(T, i ? u.y : u.x);
        return ld_f2(&t);
    }
    __device__ __forceinline__ static Pair2 make(float2 a, float2 b) {
        T ta, tb;
        st_f2(&ta, a);
        st_f2(&tb, b);
        return {make_uint2(__builtin_bit_cast(uint32_t, ta), __builtin_bit_cast(uint32_t, tb))};
    }
};

// log2 of the entries of the low level of the block twiddle table
constexpr int split_log2s(int log2m2) { return log2m2 == 4 ? 14 : 13; }

template <int LOG2M2, bool INV, class T>
__global__ void __launch_bounds__(256) split_cols(SplitColArgs a) {
    constexpr int M2 = 1 << LOG2M2;
    constexpr int LOG2M1 = kSplitLog2M1;
    constexpr int M1 = 1 << LOG2M1;
    constexpr int LOG2S = split_log2s(LOG2M2);
    constexpr int LOG2WG = LOG2M1 - 9;  // workgroups per row: 512 columns each
    const uint32_t c = ((blockIdx.x & ((1u << LOG2WG) - 1u)) << 9) + 2 * threadIdx.x;
    const int64_t row_index = blockIdx.x >> LOG2WG;                    // b n2 + k2
    const uint32_t k2 = (uint32_t)row_index & ((1u << a.log2n2) - 1u);  // the same for the whole workgroup
    const uint32_t nmask = (1u << (a.log2n1 + a.log2n2)) - 1u;
    Pair2<T>* row = reinterpret_cast<Pair2<T>*>(reinterpret_cast<T*>(a.work) + (row_index << a.log2n1) + c);
    Pair2<T> x[M2];
#pragma unroll
    for (int i = 0; i < M2; ++i) x[i] = row[(int64_t)i * (M1 / 2)];
    // Block twiddles exp(-2 pi i r / N), r = k2 (c + M1 i), from the two-level
    // table: r >> LOG2S moves by at most 8 over a wave's columns (the loads of
    // a wave fall in one or two lines), and r mod 2^LOG2S is the same for every
    // i (or, for 2^14 low entries, one of two by the parity of k2 i), so each
    // column costs one or two scattered loads instead of M2.
    float2 lo[2][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t r = k2 * (c + h);
        lo[h][0] = a.tw_lo[r & ((1u << LOG2S) - 1u)];
        lo[h][1] = LOG2S > LOG2M1 ? a.tw_lo[(r + M1) & ((1u << LOG2S) - 1u)] : lo[h][0];
    }
    auto block_twiddle = [&](int h, int i) {
        const uint32_t r = (k2 * (c + h + (uint32_t)i * M1)) & nmask;
        return cmul(a.tw_hi[r >> LOG2S], (k2 * i) & 1 ? lo[h][1] : lo[h][0]);
    };
    float2 v[2][M2];
    if constexpr (!INV) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int i = 0; i < M2; ++i) v[h][i] = cmul(x[i].get(h), block_twiddle(h, i));
            Dft<M2, -1, float2>::run(v[h]);
        }
#pragma unroll
        for (int k = 0; k < M2; ++k) {
            const float4 w = *reinterpret_cast<const float4*>(a.tw_ck + k * M1 + c);
            row[(int64_t)k * (M1 / 2)] =
                Pair2<T>::make(cscale(cmul(v[0][k], make_float2(w.x, w.y)), a.scale),
                               cscale(cmul(v[1][k], make_float2(w.z, w.w)), a.scale));
        }
    } else {
#pragma unroll
        for (int k = 0; k < M2; ++k) {
            const float4 w = *reinterpret_cast<const float4*>(a.tw_ck + k * M1 + c);
            v[0][k] = cmulc(x[k].get(0), make_float2(w.x, w.y));
            v[1][k] = cmulc(x[k].get(1), make_float2(w.z, w.w));
        }
        Dft<M2, +1, float2>::run(v[0]);
        Dft<M2, +1, float2>::run(v[1]);
#pragma unroll
        for (int i = 0; i < M2; ++i)
            row[(int64_t)i * (M1 / 2)] = Pair2<T>::make(cscale(cmulc(v[0][i], block_twiddle(0, i)), a.scale),
                                                        cscale(cmulc(v[1][i], block_twiddle(1, i)), a.scale));
    }
}

// tw[k m1 + c] = exp(-2 pi i c k / n1), c < m1, k < n1 / m1.
__global__ void __launch_bounds__(256) build_split_twiddles(float2* tw, int log2n1) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 1ll << log2n1) return;
    const int64_t t = (i & ((1ll << kSplitLog2M1) - 1)) * (i >> kSplitLog2M1);
    double sn, cs;
    sincospi(2.0 * (double)t / (double)(1ll << log2n1), &sn, &cs);
    tw[i] = make_float2((float)cs, (float)-sn);
}

// Chirp of the split middle pass in sub-row order (see the header).
template <bool F16>
__global__ void __launch_bounds__(256) build_split_chirp(void* tab, int log2n1, int log2n2, double chirp_a, double f0,
                                                         double df, double chirp_scale, double taper) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int log2n = log2n1 + log2n2;
    const int64_t n = 1ll << log2n;
    if (i >= n) return;
    const int log2m2 = log2n1 - kSplitLog2M1;
    const int64_t cp = i & ((1ll << kSplitLog2M1) - 1);
    const int64_t k = (i >> kSplitLog2M1) & ((1ll << log2m2) - 1);
    const int64_t k2 = i >> log2n1;
    const int64_t kf = k2 + ((k + (cp << log2m2)) << log2n2);
    const int64_t kk = kf < (n >> 1) ? kf : kf - n;
    const double f = (double)kk * df;
    const double turns = chirp_a * (f * f) / (f0 + f);
    const double frac = turns - rint(turns);
    double cs, cc;
    sincospi(2.0 * frac, &cs, &cc);
    const double w = taper_w(f, df * (double)n, taper);
    if constexpr (F16) {
        const double m = chirp_scale * w;
        reinterpret_cast<h2*>(tab)[i] = f16_unit(cc * m, -cs * m, m);
    } else {
        reinterpret_cast<float2*>(tab)[i] = make_float2((float)(cc * w), (float)(-cs * w));
    }
}

template <int LOG2M2, class T>
hipError_t split_one(bool inverse, const SplitColArgs& a, hipStream_t s) {
    const dim3 grid((unsigned)((int64_t)a.nblocks << (a.log2n2 + kSplitLog2M1 - 9)));
    if (inverse) hipLaunchKernelGGL((split_cols<LOG2M2, true, T>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((split_cols<LOG2M2, false, T>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <class T>
hipError_t split_dispatch(bool inverse, const SplitColArgs& a, hipStream_t s) {
    switch (a.log2n1 - kSplitLog2M1) {
        case 2: return split_one<2, T>(inverse, a, s);
        case 3: return split_one<3, T>(inverse, a, s);
        case 4: return split_one<4, T>(inverse, a, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_split_cols(int prec, bool inverse, const SplitColArgs& a, hipStream_t s) {
    if (a.log2n1 + a.log2n2 > 31 || a.log2s != split_log2s(a.log2n1 - kSplitLog2M1)) return hipErrorInvalidValue;
    if (prec == kFp32) return split_dispatch<float2>(inverse, a, s);
    if (prec == kBf16) return split_dispatch<bf16x2>(inverse, a, s);
    return split_dispatch<__half2>(inverse, a, s);
}

hipError_t launch_build_split_twiddles(float2* tw, int log2n1, hipStream_t s) {
    hipLaunchKernelGGL(build_split_twiddles, dim3((unsigned)(((1ll << log2n1) + 255) / 256)), dim3(256), 0, s, tw,
                       log2n1);
    return hipGetLastError();
}

hipError_t launch_build_split_chirp(void* tab, bool f16, int log2n1, int log2n2, double chirp_a, double f0, double df,
                                    double taper, hipStream_t s) {
    if (log2n1 <= kSplitLog2M1 || log2n1 > kSplitLog2M1 + 4) return hipErrorInvalidValue;
    const int64_t n = 1ll << (log2n1 + log2n2);
    const dim3 grid((unsigned)((n + 255) / 256));
    const double chirp_scale = std::ldexp(1.0, -half_row_rem(kSplitLog2M1));
    if (f16)
        hipLaunchKernelGGL(build_split_chirp<true>, grid, dim3(256), 0, s, tab, log2n1, log2n2, chirp_a, f0, df,
                           chirp_scale, taper);
    else
        hipLaunchKernelGGL(build_split_chirp<false>, grid, dim3(256), 0, s, tab, log2n1, log2n2, chirp_a, f0, df,
                           chirp_scale, taper);
    return hipGetLastError();
}

}  // namespace pond
