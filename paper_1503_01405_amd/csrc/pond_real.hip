// The real two-channel input path (channels added in phase, packed
// real-to-complex transforms).
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "pond_device.hpp"

namespace pond {

// ----------------------------------------------------- real input path
// Z = FFT_N(z) of z[m] = x[2m] + i x[2m+1] (x real, 2N samples).  With the
// partner value G[k] = conj Z[N-k], the bins 0..N of the real 2N-point
// transform are X[k] = E + W^k O, E = (Z + G) / 2, O = -i (Z - G) / 2, W =
// exp(-i pi / N); Y = X M is filtered (DC and Nyquist factors real), and the
// filtered real signal's packed spectrum is Z' = e + i o, e = (Y[k] + conj
// Y[N-k]) / 2, o = conj(W^k) (Y[k] - conj Y[N-k]) / 2.  All of that is linear
// in (Z, G): with P = (M[k] + conj M[N-k]) / 2, Q = (M[k] - conj M[N-k]) / 2
// and W^k = exp(-i t),
//   Z'[k] = a Z + b G,   G'[k] = conj Z'[N-k] = d G - b Z,
//   a = P - sin(t) Q,   d = P + sin(t) Q,   b = i cos(t) Q,
// evaluated in float64 once per plan: two complex products per bin.
//
// Bin k = k2 + n2 k1 lies in row k2, its partner in row n2 - k2 at column
// n1 - 1 - k1 (row 0: in row 0 at column -k1 mod n1).  Conjugating turns that
// reversal into the forward transform itself: G[k1] over row k2 is the row
// transform of conj(c[n]) W_N^(k2 n), c the partner row's column-pass output,
// with the four-step twiddle of row k2.  So a thread that transforms both
// rows holds Z and G of the same bins in the same registers, and the partner
// needs no exchange.
//
// One workgroup takes row pairs {k2, n2 - k2}; rows 0 and n2/2 are their own
// partners (the same work, the partner's result not stored).  The block
// crosses memory once.  Bound: VALU and exchanges, as the float32 row pass.
// Rows up to 2^kRealPairMaxLog2N1: the two rows in different threads, which
// swap their spectra through LDS for the 2 x 2 step.
template <int LOG2N1>
struct K2PairShape {
    static constexpr int L = 1 << LOG2N1;
    static constexpr int TPV = L / 16;
    static constexpr int ROWS = TPV >= 256 ? 2 : 256 / TPV;  // even: whole pairs
    static constexpr int THREADS = ROWS * TPV;
    static constexpr int STRIDE = L + L / 16;
};

template <int LOG2N1, class T>
__global__ void __launch_bounds__(K2PairShape<LOG2N1>::THREADS) __attribute__((amdgpu_waves_per_eu(4)))
k2_real_pair(RealPairArgs a) {
    using Sh = K2PairShape<LOG2N1>;
    constexpr int TPV = Sh::TPV;
    constexpr int PAIRS = Sh::ROWS / 2;
    __shared__ float2 lds[Sh::ROWS * Sh::STRIDE];

    const int logical = xcd_logical(blockIdx.x, gridDim.x);
    const int n2 = 1 << a.log2n2;
    const int npairs = n2 / 2 + 1;
    const int pair_groups = (npairs + PAIRS - 1) / PAIRS;
    if (logical >= pair_groups * a.nblocks) return;
    const int pg = logical / a.nblocks;
    const int b = logical - pg * a.nblocks;

    const int r = threadIdx.x / TPV;  // LDS row slot
    const int j = threadIdx.x - r * TPV;
    const bool partner = r & 1;       // this thread holds the partner row, conjugated
    const int pr = pg * PAIRS + (r >> 1);
    const int ra = min(pr, npairs - 1);
    const int rb = ra == 0 ? 0 : n2 - ra;
    // pairs past the last re-run it and never store, nor does the partner
    // side of a row that is its own partner
    const bool stores = pr < npairs && !(partner && ra == rb);
    const PadLds<float2> lrow{lds + r * Sh::STRIDE};
    const PadLds<float2> prow{lds + (r ^ 1) * Sh::STRIDE};

    StageBases<LOG2N1> tb;
    tb.load(j, a.tw1);
    T* data = reinterpret_cast<T*>(a.data) + (((int64_t)b << a.log2n2) << LOG2N1);
    const uint32_t ot = ((uint32_t)ra << LOG2N1) + (uint32_t)j;                    // in the tables
    const uint32_t od = ((uint32_t)(partner ? rb : ra) << LOG2N1) + (uint32_t)j;  // in the block
    auto conj_if = [&](float2 v) { return make_float2(v.x, partner ? -v.y : v.y); };

    float2 v[16];
    {
        const uint32_t o = opaque(od), t = opaque(ot);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float2 x = Elem<T>::load(at(data, (o + TPV * e) * (uint32_t)sizeof(T)));
            v[e] = cmul(conj_if(x), *at(a.tw4, (t + TPV * e) * 8u));
        }
    }
    // this row's coefficient, a or d, fetched during the last exchange
    float2 own[16];
    auto fetch_own = [&] {
        const uint32_t t = opaque(ot * 16u + (partner ? 8u : 0u));
#pragma unroll
        for (int e = 0; e < 16; ++e) own[e] = *reinterpret_cast<const float2*>(at(a.ad, t + TPV * e * 16u));
    };
    fft_wg<LOG2N1, -1, false, 0, false>(v, j, tb, lrow, nullptr, fetch_own);  // first LDS use
    __syncthreads();
    static_for<16>([&](auto ei) {
        constexpr int e = decltype(ei)::value;
        lrow.template put<TPV * e>(j, v[e]);
    });
    __syncthreads();
    {
        const uint32_t t = opaque(ot);
        static_for<16>([&](auto ei) {
            constexpr int e = decltype(ei)::value;
            const float2 c = *at(a.b, (t + TPV * e) * 8u);
            const float2 x = cmul(c, prow.template get<TPV * e>(j));
            v[e] = cadd(cmul(own[e], v[e]), partner ? cneg(x) : x);
        });
    }
    // the partner has read this row (rows of one wave have no barrier of their own)
    if constexpr (kWaveRow<LOG2N1>) __syncthreads();
    // output twiddles fetched during the last exchange
    float2 wo[16];
    auto fetch_tw = [&] {
        const uint32_t t = opaque(ot);
#pragma unroll
        for (int e = 0; e < 16; ++e) wo[e] = *at(a.tw4, (t + TPV * e) * 8u);
    };
    fft_wg<LOG2N1, +1>(v, j, tb, lrow, nullptr, fetch_tw);
    asm volatile("" ::: "memory");
    if (stores) {
        const uint32_t o = opaque(od);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            Elem<T>::store(at(data, (o + TPV * e) * (uint32_t)sizeof(T)), conj_if(cmulc(v[e], wo[e])));
    }
}

// Longer rows: a thread holds 16 values of each row and takes the rows
// through one LDS row in turn (forward, forward, 2 x 2 step, inverse,
// inverse), so that two workgroups of 512 threads (2^13: 68 KB of LDS, 128
// registers) share a CU; both rows at once, in 1,024 threads and 136 KB, with
// the partner read in reverse order and the split, filter and recombination
// done in turn, took 800 us per 14 blocks of 2^23 in the float16-storage form
// where this takes 520.
template <int LOG2N1>
struct K2SeqShape {
    static constexpr int L = 1 << LOG2N1;
    static constexpr int TPV = L / 16;
    static constexpr int PAIRS = TPV >= 256 ? 1 : 256 / TPV;
    static constexpr int THREADS = PAIRS * TPV;
    static constexpr int STRIDE = L + L / 16;
};

template <int LOG2N1, class T>
__global__ void __launch_bounds__(K2SeqShape<LOG2N1>::THREADS) __attribute__((amdgpu_waves_per_eu(4)))
k2_real_rows(RealPairArgs a) {
    using Sh = K2SeqShape<LOG2N1>;
    constexpr int TPV = Sh::TPV;
    __shared__ float2 lds[Sh::PAIRS * Sh::STRIDE];

    const int logical = xcd_logical(blockIdx.x, gridDim.x);
    const int n2 = 1 << a.log2n2;
    const int npairs = n2 / 2 + 1;
    const int pair_groups = (npairs + Sh::PAIRS - 1) / Sh::PAIRS;
    if (logical >= pair_groups * a.nblocks) return;
    const int pg = logical / a.nblocks;
    const int b = logical - pg * a.nblocks;

    const int slot = threadIdx.x / TPV;
    const int j = threadIdx.x - slot * TPV;
    const bool valid = pg * Sh::PAIRS + slot < npairs;  // pairs past the last re-run it and never store
    const int ra = min(pg * Sh::PAIRS + slot, npairs - 1);
    const int rb = ra == 0 ? 0 : n2 - ra;
    const PadLds<float2> lrow{lds + slot * Sh::STRIDE};

    StageBases<LOG2N1> tb;
    tb.load(j, a.tw1);
    T* data = reinterpret_cast<T*>(a.data) + (((int64_t)b << a.log2n2) << LOG2N1);
    // element offsets of the thread's first value: rows a and b of the
    // block, and row a of the tables
    const uint32_t oa = ((uint32_t)ra << LOG2N1) + (uint32_t)j;
    const uint32_t ob = ((uint32_t)rb << LOG2N1) + (uint32_t)j;

    float2 z[16], g[16];
    {
        const uint32_t o = opaque(oa);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float2 x = Elem<T>::load(at(data, (o + TPV * e) * (uint32_t)sizeof(T)));
            z[e] = cmul(x, *at(a.tw4, (o + TPV * e) * 8u));
        }
    }
    // the partner row, fetched during the last exchange of the first row
    T gr[16];
    auto fetch_g = [&] {
        const uint32_t o = opaque(ob);
#pragma unroll
        for (int e = 0; e < 16; ++e) gr[e] = *at(data, (o + TPV * e) * (uint32_t)sizeof(T));
    };
    fft_wg<LOG2N1, -1, false, 0, false>(z, j, tb, lrow, nullptr, fetch_g);  // first LDS use
    {
        const uint32_t o = opaque(oa);
#pragma unroll
        for (int e = 0; e < 16; ++e) g[e] = cmulc(*at(a.tw4, (o + TPV * e) * 8u), Elem<T>::load(&gr[e]));
    }
    fft_wg<LOG2N1, -1>(g, j, tb, lrow);
    {
        const uint32_t o = opaque(oa);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float4 ad = *at(a.ad, (o + TPV * e) * 16u);
            const float2 cb = *at(a.b, (o + TPV * e) * 8u);
            const float2 ca = make_float2(ad.x, ad.y), cd = make_float2(ad.z, ad.w);
            const float2 zz = z[e], gg = g[e];
            z[e] = cadd(cmul(ca, zz), cmul(cb, gg));
            g[e] = csub(cmul(cd, gg), cmul(cb, zz));
        }
    }
    fft_wg<LOG2N1, +1>(g, j, tb, lrow);
    asm volatile("" ::: "memory");
    if (valid && ra != rb) {
        const uint32_t o = opaque(oa), os = opaque(ob);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            Elem<T>::store(at(data, (os + TPV * e) * (uint32_t)sizeof(T)),
                           cmulc(*at(a.tw4, (o + TPV * e) * 8u), g[e]));
    }
    // output twiddles fetched during the last exchange (there are no
    // registers for that while both rows are held)
    float2 wo[16];
    auto fetch_tw = [&] {
        const uint32_t o = opaque(oa);
#pragma unroll
        for (int e = 0; e < 16; ++e) wo[e] = *at(a.tw4, (o + TPV * e) * 8u);
    };
    fft_wg<LOG2N1, +1>(z, j, tb, lrow, nullptr, fetch_tw);
    asm volatile("" ::: "memory");
    if (valid) {
        const uint32_t o = opaque(oa);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            Elem<T>::store(at(data, (o + TPV * e) * (uint32_t)sizeof(T)), cmulc(z[e], wo[e]));
    }
}

// Tables of k2_real_pair, entry i = k2 n1 + k1 for rows k2 = 0..n2/2 (bin k =
// k2 + n2 k1): tw4 the four-step twiddle W_N^(k1 k2), (a, d) and b the 2 x 2
// step, times `scale`.  M[k] is the filter of real-transform bin k (baseband
// k bw / N): upper sideband exp(-2 pi i turns(f)), f = k bw/N - bw/2; lower
// sideband exp(+2 pi i turns(f)), f = bw/2 - k bw/N; times the taper; real
// part only at k = 0 and k = N.  Float64, phases reduced mod 1 turn.
struct RealBin {
    double re, im;
};
__device__ __forceinline__ RealBin real_filter(int64_t k, int64_t N, double chirp_a, double f0, double bw, int lsb,
                                               double taper) {
    const double fb = (double)k * bw / (double)N;
    const double f = lsb ? bw * 0.5 - fb : fb - bw * 0.5;
    const double turns = chirp_a * (f * f) / (f0 + f);
    const double frac = turns - rint(turns);
    double sm, cm;
    sincospi(2.0 * frac, &sm, &cm);
    const double wt = taper_w(f, bw, taper);
    RealBin m{cm * wt, (lsb ? sm : -sm) * wt};
    if (k == 0 || k == N) m.im = 0.0;
    return m;
}

__global__ void __launch_bounds__(256) real_build_pair_table(float2* __restrict__ tw4, float4* __restrict__ ad,
                                                              float2* __restrict__ b, int log2n1, int log2n2,
                                                              double chirp_a, double f0, double bw, int lsb,
                                                              double taper, double scale) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int log2n = log2n1 + log2n2;
    const int64_t N = 1ll << log2n, n1 = 1ll << log2n1, n2 = 1ll << log2n2;
    if (i >= (n2 / 2 + 1) << log2n1) return;
    const int64_t k2 = i >> log2n1, k1 = i & (n1 - 1);
    const int64_t k = k2 + (k1 << log2n2);
    const RealBin m = real_filter(k, N, chirp_a, f0, bw, lsb, taper);
    const RealBin mn = real_filter(N - k, N, chirp_a, f0, bw, lsb, taper);
    const double px = 0.5 * scale * (m.re + mn.re), py = 0.5 * scale * (m.im - mn.im);
    const double qx = 0.5 * scale * (m.re - mn.re), qy = 0.5 * scale * (m.im + mn.im);
    double s, c;
    sincospi((double)k / (double)N, &s, &c);
    ad[i] = make_float4((float)(px - s * qx), (float)(py - s * qy), (float)(px + s * qx), (float)(py + s * qy));
    b[i] = make_float2((float)(-c * qy), (float)(c * qx));
    double st, ct;
    sincospi(2.0 * (double)((k1 * k2) & (N - 1)) / (double)N, &st, &ct);
    tw4[i] = make_float2((float)ct, (float)-st);
}

// Rows up to here have a thread group per row: a workgroup that takes two
// short rows in turn is a chain of four transforms with too little beside it
// (24 packed blocks of 2^17: 148.9 us a call against 111.2).  From 2^12 on two
// such workgroups fill a CU and the pair needs half the LDS (packed 2^22:
// 1,502 us against 1,588).
constexpr int kRealPairMaxLog2N1 = 11;
template <class T, int LOG2N1>
static hipError_t real_pair_one(const RealPairArgs& a, hipStream_t s) {
    constexpr bool kSeq = LOG2N1 > kRealPairMaxLog2N1;
    const int npairs = (1 << a.log2n2) / 2 + 1;
    constexpr int kPairs = kSeq ? K2SeqShape<LOG2N1>::PAIRS : K2PairShape<LOG2N1>::ROWS / 2;
    const int groups = (npairs + kPairs - 1) / kPairs * a.nblocks;
    const int grid = (groups + 7) & ~7;
    if constexpr (kSeq)
        hipLaunchKernelGGL((k2_real_rows<LOG2N1, T>), dim3(grid), dim3(K2SeqShape<LOG2N1>::THREADS), 0, s, a);
    else
        hipLaunchKernelGGL((k2_real_pair<LOG2N1, T>), dim3(grid), dim3(K2PairShape<LOG2N1>::THREADS), 0, s, a);
    return hipGetLastError();
}

template <class T>
static hipError_t real_pair_dispatch(int log2n1, const RealPairArgs& a, hipStream_t s) {
    switch (log2n1) {
        case 5: return real_pair_one<T, 5>(a, s);
        case 6: return real_pair_one<T, 6>(a, s);
        case 7: return real_pair_one<T, 7>(a, s);
        case 8: return real_pair_one<T, 8>(a, s);
        case 9: return real_pair_one<T, 9>(a, s);
        case 10: return real_pair_one<T, 10>(a, s);
        case 11: return real_pair_one<T, 11>(a, s);
        case 12: return real_pair_one<T, 12>(a, s);
        case 13: return real_pair_one<T, 13>(a, s);
        case 14:
            // float32 only (see real_split)
            if constexpr (std::is_same<T, float2>::value) return real_pair_one<T, 14>(a, s);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_real_pair(int prec, int log2n1, const RealPairArgs& a, hipStream_t s) {
    switch (prec) {
        case kFp32: return real_pair_dispatch<float2>(log2n1, a, s);
        case kMixedValu: return real_pair_dispatch<__half2>(log2n1, a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_real_build_pair_table(float2* tw4, float4* ad, float2* b, int log2n1, int log2n2, double chirp_a,
                                        double f0, double bw, int lsb, double taper, hipStream_t s) {
    const int64_t n = ((int64_t)(1 << log2n2) / 2 + 1) << log2n1;
    // the forward rows' 1/n1
    const double scale = std::ldexp(1.0, -log2n1);
    hipLaunchKernelGGL(real_build_pair_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, tw4, ad, b, log2n1,
                       log2n2, chirp_a, f0, bw, lsb, taper, scale);
    return hipGetLastError();
}

// Float16 storage, rows of 2^14 (packed blocks of 2^24): forward rows, this
// step over the stored spectrum, inverse rows.  The form's spectrum is
// float16 there, and keeping both rows in float32 (as the shorter ones are)
// changes its series by 1.4e-4, so the three passes stay.  One thread per
// pair {k, N-k} (rows 0..n2/2; on the two rows that pair with themselves, the
// thread of the lower index) reads and writes both bins in place; tab[i] =
// (W^k, M[k]) of the bin at position i of the block, tab[N] = (-1, M[N]).
__global__ void __launch_bounds__(256) real_split(RealSplitArgs a) {
    const int64_t gi = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int log2n = a.log2n1 + a.log2n2;
    const int n1 = 1 << a.log2n1, n2 = 1 << a.log2n2, N = 1 << log2n;
    const int per_block = (n2 / 2 + 1) << a.log2n1;  // rows 0..n2/2
    if (gi >= (int64_t)a.nblocks * per_block) return;
    const int64_t b = gi / per_block;
    const int i = (int)(gi - b * per_block);
    const int k2 = i >> a.log2n1, k1 = i & (n1 - 1);
    const int ip = k2 == 0 ? ((n1 - k1) & (n1 - 1)) : (((n2 - k2) << a.log2n1) + (n1 - 1 - k1));
    if (ip < i) return;  // the pair belongs to the thread of index ip
    using T = __half2;
    T* z = reinterpret_cast<T*>(a.data) + (b << log2n);
    const float2 A = Elem<T>::load(z + i), B = Elem<T>::load(z + ip);
    const float4 tk = a.tab[i], tn = a.tab[i == 0 ? N : ip];
    const float2 w = make_float2(tk.x, tk.y), mk = make_float2(tk.z, tk.w), mn = make_float2(tn.z, tn.w);
    const float2 E = make_float2(0.5f * (A.x + B.x), 0.5f * (A.y - B.y));
    const float2 D = make_float2(0.5f * (A.x - B.x), 0.5f * (A.y + B.y));  // (Z[k] - conj Z[N-k]) / 2
    const float2 O = make_float2(D.y, -D.x);                                // -i D
    const float2 wo = cmul(w, O);
    const float2 yk = cmul(cadd(E, wo), mk);
    const float2 en = csub(E, wo);
    const float2 yn = cmul(make_float2(en.x, -en.y), mn);                    // Y[N-k]
    const float2 ync = make_float2(yn.x, -yn.y);
    const float2 e2 = cscale(cadd(yk, ync), 0.5f);
    const float2 o2 = cmulc(cscale(csub(yk, ync), 0.5f), w);
    Elem<T>::store(z + i, make_float2(e2.x - o2.y, e2.y + o2.x));
    if (ip != i) Elem<T>::store(z + ip, make_float2(e2.x + o2.y, o2.x - e2.y));
}

__global__ void __launch_bounds__(256) real_build_table(float4* __restrict__ tab, int log2n1, int log2n2,
                                                         double chirp_a, double f0, double bw, int lsb,
                                                         double taper) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int log2n = log2n1 + log2n2;
    const int64_t N = 1ll << log2n;
    if (i > N) return;
    const int64_t k = i == N ? N : (i >> log2n1) + ((i & ((1ll << log2n1) - 1)) << log2n2);
    double sw, cw;
    sincospi((double)k / (double)N, &sw, &cw);
    const RealBin m = real_filter(k, N, chirp_a, f0, bw, lsb, taper);
    tab[i] = make_float4((float)cw, (float)-sw, (float)m.re, (float)m.im);
}

hipError_t launch_real_split(const RealSplitArgs& a, hipStream_t s) {
    const int64_t n = (int64_t)a.nblocks * (((1 << a.log2n2) / 2 + 1) << a.log2n1);
    hipLaunchKernelGGL(real_split, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_real_build_table(float4* tab, int log2n1, int log2n2, double chirp_a, double f0, double bw,
                                   int lsb, double taper, hipStream_t s) {
    const int64_t n = (1ll << (log2n1 + log2n2)) + 1;
    hipLaunchKernelGGL(real_build_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, tab, log2n1, log2n2,
                       chirp_a, f0, bw, lsb, taper);
    return hipGetLastError();
}

}  // namespace pond
