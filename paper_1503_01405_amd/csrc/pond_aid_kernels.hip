// Incoherent (AID) mode kernels: filterbank, channel shift-and-sum, fold.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "pond_device.hpp"

namespace pond {

// ------------------------------------------------- incoherent (AID) mode
// Filterbank: spectra of consecutive nchan-sample blocks (square window, no
// overlap), |X|^2 summed over nint spectra per output time.  One FFT group
// of nchan/16 threads per row of the workgroup (as K2's short rows); each
// group takes AID_TS consecutive output times and keeps their powers in
// registers; the workgroup then writes them channel-major, F[c][t], through
// an LDS transpose (rows of ROWS*AID_TS consecutive times per channel).
// Bound: VALU (about 50 instructions per sample).  512 threads and two times
// per group (LDS 68 KB, at most 128 registers) give 16 waves per CU; with 256
// threads and four times 64 of 150 registers held powers and 8 waves ran.  The
// next spectrum's samples are read during a transform.
constexpr int AID_TS = 2;
template <int LOG2C>
struct AidShape {
    static constexpr int TPV = (1 << LOG2C) / 16;
    static constexpr int THREADS = 512;
    static constexpr int ROWS = THREADS / TPV;
    static constexpr int STRIDE = (1 << LOG2C) + (1 << LOG2C) / 16;
};

template <int LOG2C>
__global__ void __launch_bounds__(AidShape<LOG2C>::THREADS) __attribute__((amdgpu_waves_per_eu(4)))
aid_filterbank(AidArgs a) {
    using Sh = AidShape<LOG2C>;
    constexpr int C = 1 << LOG2C;
    constexpr int TPV = Sh::TPV;
    constexpr int ROWS = Sh::ROWS;
    constexpr int COLS = ROWS * AID_TS;  // output times per workgroup
    constexpr int FFT_LDS = ROWS * Sh::STRIDE * 8;
    constexpr int TILE_LDS = C * COLS * 4;
    __shared__ __align__(16) char lds_raw[FFT_LDS > TILE_LDS ? FFT_LDS : TILE_LDS];
    float2* lds = reinterpret_cast<float2*>(lds_raw);
    float* tile = reinterpret_cast<float*>(lds_raw);

    const int g = threadIdx.x / TPV;
    const int j = threadIdx.x - g * TPV;
    const PadLds<float2> lrow{lds + g * Sh::STRIDE};
    StageBases<LOG2C> tb;
    tb.load(j, a.tw);
    const int64_t tbase = (int64_t)blockIdx.x * COLS;
    // the group's spectra are consecutive blocks of C samples; output times
    // past the last re-read its blocks and are not stored
    const int64_t t0 = tbase + g * AID_TS;
    const int nspec = AID_TS * a.nint;
    const int64_t last = a.nspec * a.nint - 1;  // last block of the input
    uint32_t raw[16];
    auto load = [&](int k) {
        const int64_t blk = min(t0 * a.nint + k, last);
        const int8_t* p = a.iq + 2 * blk * (int64_t)C;
        const uint32_t o = opaque((uint32_t)j);
#pragma unroll
        for (int e = 0; e < 16; ++e) raw[e] = *at(reinterpret_cast<const uint16_t*>(p), (o + TPV * e) * 2u);
    };
    load(0);
    float acc[AID_TS][16];
#pragma unroll
    for (int ts = 0; ts < AID_TS; ++ts) {
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[ts][e] = 0.f;
        for (int i = 0; i < a.nint; ++i) {
            float2 v[16];
#pragma unroll
            for (int e = 0; e < 16; ++e)
                v[e] = make_float2((float)(int8_t)(raw[e] & 0xff), (float)(int8_t)((raw[e] >> 8) & 0xff));
            const int next = ts * a.nint + i + 1;
            if (next < nspec) load(next);
            fft_wg<LOG2C, -1>(v, j, tb, lrow);
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[ts][e] = fmaf(v[e].x, v[e].x, fmaf(v[e].y, v[e].y, acc[ts][e]));
        }
    }
    __syncthreads();  // the FFT scratch becomes the transpose tile
#pragma unroll
    for (int e = 0; e < 16; ++e)
        *reinterpret_cast<float2*>(tile + (j + TPV * e) * COLS + g * AID_TS) = make_float2(acc[0][e], acc[1][e]);
    __syncthreads();
    const int64_t ncols = a.nspec - tbase < COLS ? a.nspec - tbase : COLS;
    for (int idx = threadIdx.x; idx < C * COLS; idx += Sh::THREADS) {
        const int c = idx / COLS, col = idx - c * COLS;
        if (col < ncols) a.F[(int64_t)c * a.nspec + tbase + col] = tile[idx];
    }
}

// Channel shift-and-sum and fold: output m = sum_c F[c][m + dd_c], with
// dd_c = d_c - d_min >= 0 (Eq. (3) delays in integrated samples); the
// series value and its fold into integer (sub-integration-free) histograms
// as K3 does, fold phase x = (m - d_min) * nchan * nint * inv_pfs.
// A wave takes 64 consecutive outputs and 1 / 2^log2split of the channels; the
// waves of a workgroup that share outputs meet in LDS.  Bound: reading F (60 s of
// 1024 channels: 960 MB).  One output per thread over all channels left the chip
// idle on short segments of many channels.  Whole calls, before and now: 4,882
// outputs of 4,096 channels 476 and 121 us (16 ways); 7,812 of 512, 73 and 32
// (16); 117,187 of 128, 83.5 and 80.7 (4); 468,750 of 64, 82.5 and 79.7 (none:
// the barriers of 16 ways cost it 116); 234,375 of 1,024, 1,385 and 1,356 (2).
constexpr int AID_SUM_THREADS = 1024;
__global__ void __launch_bounds__(AID_SUM_THREADS) aid_dedisperse_fold(AidArgs a) {
    constexpr int WAVES = AID_SUM_THREADS / 64;
    extern __shared__ uint64_t dyn_u64[];
    float* part = reinterpret_cast<float*>(dyn_u64);  // [WAVES][64], with a split only
    uint64_t* hsum = dyn_u64 + (a.log2split > 0 ? WAVES * 32 : 0);
    uint32_t* hcnt = reinterpret_cast<uint32_t*>(hsum + a.nbins);
    int32_t* dd = reinterpret_cast<int32_t*>(hcnt + a.nbins);
    for (int i = threadIdx.x; i < a.nbins; i += blockDim.x) {
        hsum[i] = 0;
        hcnt[i] = 0;
    }
    for (int c = threadIdx.x; c < a.nchan; c += blockDim.x) dd[c] = a.dd[c];
    __syncthreads();
    uint32_t flags = 0;
    const double spec = (double)a.nchan * (double)a.nint;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int share = wave & ((1 << a.log2split) - 1);  // which of the channels
    const int per_wave = a.nchan >> a.log2split;
    const int64_t step = (int64_t)64 * (WAVES >> a.log2split);  // outputs per workgroup at a time
    for (int64_t base = (int64_t)blockIdx.x * step; base < a.nout; base += (int64_t)gridDim.x * step) {
        const int64_t m = base + 64 * (wave >> a.log2split) + lane;
        float s = 0.f;
        if (m < a.nout) {
            const float* f = a.F + m;
#pragma unroll 8
            for (int c = share * per_wave; c < (share + 1) * per_wave; ++c) s += f[(int64_t)c * a.nspec + dd[c]];
        }
        if (a.log2split > 0) {
            __syncthreads();  // the previous outputs' sums have been read
            part[wave * 64 + lane] = s;
            __syncthreads();
        }
        if (share == 0 && m < a.nout) {
            for (int w = 1; w < 1 << a.log2split; ++w) s += part[(wave + w) * 64 + lane];
            if (a.series) a.series[m] = s;
            const double x = (double)(m - a.d_min) * spec * a.inv_pfs;
            int bin = (int)((x - floor(x)) * (double)a.nbins);
            bin = bin < a.nbins - 1 ? bin : a.nbins - 1;
            const double dv = (double)s * kFoldScale;
            if (!(dv < kFoldRangeLimit * kFoldScale)) flags |= 2u;
            if (!isfinite(s)) flags |= 1u;
            const uint64_t fx = isfinite(s) ? (uint64_t)__double2ull_rn(dv) : 0ull;
            atomicAdd((unsigned long long*)&hsum[bin], (unsigned long long)fx);
            atomicAdd(&hcnt[bin], 1u);
        }
    }
    if (flags) atomicOr(a.status, flags);
    __syncthreads();
    uint64_t* ps = a.part_sum + (int64_t)blockIdx.x * a.nbins;
    uint32_t* pc = a.part_cnt + (int64_t)blockIdx.x * a.nbins;
    for (int i = threadIdx.x; i < a.nbins; i += blockDim.x) {
        ps[i] = hsum[i];
        pc[i] = hcnt[i];
    }
}

template <int LOG2C>
static hipError_t aid_fb_one(const AidArgs& a, hipStream_t s) {
    using Sh = AidShape<LOG2C>;
    const int64_t cols = Sh::ROWS * AID_TS;
    const int64_t grid = (a.nspec + cols - 1) / cols;
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(aid_filterbank<LOG2C>, dim3((unsigned)grid), dim3(Sh::THREADS), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_aid_filterbank(int log2c, const AidArgs& a, hipStream_t s) {
    switch (log2c) {
        case 6: return aid_fb_one<6>(a, s);
        case 7: return aid_fb_one<7>(a, s);
        case 8: return aid_fb_one<8>(a, s);
        case 9: return aid_fb_one<9>(a, s);
        case 10: return aid_fb_one<10>(a, s);
        case 11: return aid_fb_one<11>(a, s);
        case 12: return aid_fb_one<12>(a, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_aid_dedisperse_fold(const AidArgs& a, int grid, hipStream_t s) {
    const size_t dyn = aid_sum_lds(a.nbins, a.nchan, a.log2split);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&aid_dedisperse_fold),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kAidSumLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(aid_dedisperse_fold, dim3(grid), dim3(AID_SUM_THREADS), dyn, s, a);
    return hipGetLastError();
}

}  // namespace pond
