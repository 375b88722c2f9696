// Fold reduction and finalisation, the streaming copy and small fills.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pond_device.hpp"

namespace pond {

// ------------------------------------------------------ fold reduction
// Sum the per-workgroup partial histograms (integer, so order-free) of up to
// kReduceSlots queued launches and add them to the accumulators.  Grid: x over
// entries, y over part chunks, z the launch; each has its own partials,
// accumulators and sizes.  The partials were just written and sit in cache: a
// full chunk issues all its loads at once, so a call costs about one load
// latency, not a chain.
constexpr int kReduceChunk = 8;
__global__ void __launch_bounds__(256) fold_reduce_batch(ReduceBatch b) {
    const ReduceJob& j = b.job[blockIdx.z];
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= j.entries) return;
    const int p0 = blockIdx.y * kReduceChunk;
    if (p0 >= j.nparts) return;
    const int p1 = min(j.nparts, p0 + kReduceChunk);
    const uint64_t* ps = j.part_sum;
    const uint32_t* pc = j.part_cnt;
    const int entries = j.entries;
    uint64_t s = 0, n = 0;
    if (p1 - p0 == kReduceChunk) {
        uint64_t sv[kReduceChunk];
        uint32_t nv[kReduceChunk];
#pragma unroll
        for (int k = 0; k < kReduceChunk; ++k) {
            sv[k] = ps[(int64_t)(p0 + k) * entries + i];
            nv[k] = pc[(int64_t)(p0 + k) * entries + i];
        }
#pragma unroll
        for (int k = 0; k < kReduceChunk; ++k) {
            s += sv[k];
            n += nv[k];
        }
    } else {
        for (int q = p0; q < p1; ++q) {
            s += ps[(int64_t)q * entries + i];
            n += pc[(int64_t)q * entries + i];
        }
    }
    if (n) {
        atomicAdd((unsigned long long*)&j.acc_sum[j.acc_off + i], (unsigned long long)s);
        atomicAdd((unsigned long long*)&j.acc_cnt[j.acc_off + i], (unsigned long long)n);
    }
}

// The partials of the only launch of a call, summed straight into its profile
// (a call that accumulates over launches goes through fold_reduce_batch).  A
// workgroup takes 16 bins (128 bytes of a partial's sums) and reads 64 partials
// at once: the bound is the latency of these loads (7,812 filterbank outputs,
// whole call: 31.4 us with the four launches that cleared two accumulators, added
// to them and divided, 28.2 with this one).
constexpr int kProfileBins = 16;
__global__ void __launch_bounds__(1024) fold_reduce_profile(const uint64_t* __restrict__ ps,
                                                            const uint32_t* __restrict__ pc, int nparts, int nbins,
                                                            float* profile) {
    constexpr int PARTS = 1024 / kProfileBins;
    __shared__ uint64_t sum[PARTS][kProfileBins], cnt[PARTS][kProfileBins];
    const int lane = threadIdx.x % kProfileBins, part = threadIdx.x / kProfileBins;
    const int bin = blockIdx.x * kProfileBins + lane;
    uint64_t s = 0, n = 0;
    if (bin < nbins) {
#pragma unroll 8
        for (int q = part; q < nparts; q += PARTS) {
            s += ps[(int64_t)q * nbins + bin];
            n += pc[(int64_t)q * nbins + bin];
        }
    }
    sum[part][lane] = s;
    cnt[part][lane] = n;
    __syncthreads();
    if (part > 0 || bin >= nbins) return;
    for (int w = 1; w < PARTS; ++w) {
        s += sum[w][lane];
        n += cnt[w][lane];
    }
    profile[bin] = n ? (float)(((double)s / kFoldScale) / (double)n) : 0.f;
}

// Write the profiles of the first n_complete slots, then move slot
// n_complete (the still-open sub-integration, if any) to slot 0 and clear
// the rest of the n_touched slots.  One thread per bin.  A status word is
// cleared beside it (the end of a stream: not a launch of its own).
__global__ void __launch_bounds__(256) fold_finalize(uint64_t* acc_sum, uint64_t* acc_cnt, int nbins, int n_complete,
                                                     int n_touched, float* profiles, uint64_t* status) {
    const int bin = blockIdx.x * blockDim.x + threadIdx.x;
    if (status && bin == 0) *status = 0;
    if (bin >= nbins) return;
    for (int k = 0; k < n_complete; ++k) {
        const uint64_t s = acc_sum[(int64_t)k * nbins + bin];
        const uint64_t n = acc_cnt[(int64_t)k * nbins + bin];
        profiles[(int64_t)k * nbins + bin] = n ? (float)(((double)s / kFoldScale) / (double)n) : 0.f;
    }
    if (n_complete > 0) {
        uint64_t cs = 0, cn = 0;
        if (n_complete < n_touched) {
            cs = acc_sum[(int64_t)n_complete * nbins + bin];
            cn = acc_cnt[(int64_t)n_complete * nbins + bin];
        }
        acc_sum[bin] = cs;
        acc_cnt[bin] = cn;
        for (int k = 1; k < n_touched; ++k) {
            acc_sum[(int64_t)k * nbins + bin] = 0;
            acc_cnt[(int64_t)k * nbins + bin] = 0;
        }
    }
}

// Mean power per (trial, bin): sum / count, 0 for an empty bin.
__global__ void __launch_bounds__(256) fold_profiles(const uint64_t* acc_sum, const uint64_t* acc_cnt, int64_t n,
                                                     float* profiles) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t c = acc_cnt[i];
    profiles[i] = c ? (float)(((double)acc_sum[i] / kFoldScale) / (double)c) : 0.f;
}

// The na bytes at a, then the nb at b, to dst: the samples that the next blocks
// need, from the previous carry and from this call's input.  dst is 16-byte
// aligned, the sources need not be.  Bound: the launch on short calls (300,007
// samples and the flush: 61.9 us with two copy commands and a launch that only
// cleared the status word, 60.2 without).
__global__ void __launch_bounds__(256) carry_tail(int8_t* __restrict__ dst, const int8_t* __restrict__ a, int64_t na,
                                                  const int8_t* __restrict__ b, int64_t nb) {
    const int64_t o = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * 16;
    const int64_t total = na + nb;
    if (o >= total) return;
    if (o + 16 <= total && (o + 16 <= na || o >= na)) {
        struct Word { uint32_t w[4]; } v;
        __builtin_memcpy(&v, o >= na ? b + (o - na) : a + o, 16);
        *reinterpret_cast<uint4*>(dst + o) = make_uint4(v.w[0], v.w[1], v.w[2], v.w[3]);
    } else {
        const int64_t end = o + 16 < total ? o + 16 : total;
        for (int64_t k = o; k < end; ++k) dst[k] = k < na ? a[k] : b[k - na];
    }
}

// Streaming copy of n16 16-byte words (measurement of the achievable HBM
// bandwidth): each workgroup moves contiguous 16 KB chunks, a thread's four
// loads of a chunk in flight before its stores.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__global__ void __launch_bounds__(256) copy_u128(u32x4* __restrict__ dst, const u32x4* __restrict__ src,
                                                 int64_t n16) {
    constexpr int U = 4;
    constexpr int64_t kChunk = 256 * U;
    for (int64_t base = (int64_t)blockIdx.x * kChunk; base < n16; base += (int64_t)gridDim.x * kChunk) {
        u32x4 v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = base + u * 256 + threadIdx.x;
            v[u] = k < n16 ? src[k] : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = base + u * 256 + threadIdx.x;
            if (k < n16) dst[k] = v[u];
        }
    }
}

// Stage twiddles of a length-n transform for t < count.
__global__ void __launch_bounds__(256) stage_twiddles(float2* w, int64_t count, int64_t n) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    w[t] = stage_twiddle(t, n);
}

// splitmix64 (Steele, Lea & Flood 2014).
__device__ __forceinline__ uint64_t splitmix64(uint64_t x) {
    x += 0x9e3779b97f4a7c15ull;
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    return x ^ (x >> 31);
}

// Pseudo-random bytes (splitmix64 of the word index and a seed): timing input
// for the autotuner, not part of the method.
__global__ void __launch_bounds__(256) fill_noise_u64(uint64_t* p, int64_t n, uint64_t seed) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    p[i] = splitmix64(seed + 0x9e3779b97f4a7c15ull * (uint64_t)i);
}

// One word is 4 complex samples.  Integer sums: the energy is exact in any
// order.  With this noise made on the host (8 MB and its copy; 16 MB at 2^23) a
// packed float16 plan of 2^20 points was created in 4.1 ms, now in 0.5; 2^23 8.0
// and 0.8.
__global__ void __launch_bounds__(256) calibration_noise(uint64_t* __restrict__ iq, int64_t words, uint64_t* energy) {
    uint64_t sum = 0;
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < words; w += (int64_t)gridDim.x * blockDim.x) {
        const uint64_t h = splitmix64((uint64_t)(4 * w));
        iq[w] = h;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int v = (int8_t)((h >> (8 * k)) & 0xff);
            sum += (uint64_t)(v * v);
        }
    }
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    if ((threadIdx.x & 63) == 0) atomicAdd((unsigned long long*)energy, (unsigned long long)sum);
}

__global__ void __launch_bounds__(256) zero_u64(uint64_t* p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

hipError_t launch_fold_reduce_profile(const uint64_t* ps, const uint32_t* pc, int nparts, int nbins, float* profile,
                                      hipStream_t s) {
    hipLaunchKernelGGL(fold_reduce_profile, dim3((nbins + kProfileBins - 1) / kProfileBins), dim3(1024), 0, s,
                       ps, pc, nparts, nbins, profile);
    return hipGetLastError();
}

hipError_t launch_fold_reduce_batch(const ReduceBatch& b, hipStream_t s) {
    if (b.n < 1 || b.n > kReduceSlots) return hipErrorInvalidValue;
    int entries = 0, nparts = 0;
    for (int k = 0; k < b.n; ++k) {
        entries = std::max(entries, (int)b.job[k].entries);
        nparts = std::max(nparts, (int)b.job[k].nparts);
    }
    if (entries <= 0 || nparts <= 0) return hipSuccess;
    const dim3 grid((entries + 255) / 256, (nparts + kReduceChunk - 1) / kReduceChunk, b.n);
    hipLaunchKernelGGL(fold_reduce_batch, grid, dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_fold_finalize(uint64_t* acc_sum, uint64_t* acc_cnt, int nbins, int n_complete, int n_touched,
                                float* profiles, uint64_t* status, hipStream_t s) {
    hipLaunchKernelGGL(fold_finalize, dim3((nbins + 255) / 256), dim3(256), 0, s, acc_sum, acc_cnt, nbins,
                       n_complete, n_touched, profiles, status);
    return hipGetLastError();
}

hipError_t launch_carry_tail(int8_t* dst, const int8_t* a, int64_t na, const int8_t* b, int64_t nb, hipStream_t s) {
    if (na + nb <= 0) return hipSuccess;
    const int64_t words = (na + nb + 15) / 16;
    hipLaunchKernelGGL(carry_tail, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, dst, a, na, b, nb);
    return hipGetLastError();
}

hipError_t launch_copy_u128(void* dst, const void* src, int64_t n16, hipStream_t s) {
    if (n16 <= 0) return hipSuccess;
    const int64_t chunks = (n16 + 1023) / 1024;
    const unsigned grid = (unsigned)(chunks < 16384 ? chunks : 16384);
    hipLaunchKernelGGL(copy_u128, dim3(grid), dim3(256), 0, s, reinterpret_cast<u32x4*>(dst),
                       reinterpret_cast<const u32x4*>(src), n16);
    return hipGetLastError();
}

hipError_t launch_stage_twiddles(float2* w, int64_t n, hipStream_t s) { return launch_partial_twiddles(w, n, n, s); }

hipError_t launch_partial_twiddles(float2* w, int64_t count, int64_t n, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    if (count > n) return hipErrorInvalidValue;
    hipLaunchKernelGGL(stage_twiddles, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, w, count, n);
    return hipGetLastError();
}

hipError_t launch_fill_noise_u64(uint64_t* p, int64_t n, uint64_t seed, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_noise_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, seed);
    return hipGetLastError();
}

hipError_t launch_calibration_noise(uint64_t* iq, int64_t words, uint64_t* energy, hipStream_t s) {
    if (words <= 0) return hipSuccess;
    const int64_t groups = (words + 255) / 256;
    hipLaunchKernelGGL(calibration_noise, dim3((unsigned)(groups < 1024 ? groups : 1024)), dim3(256), 0, s, iq, words,
                       energy);
    return hipGetLastError();
}

hipError_t launch_zero_u64(uint64_t* p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_u64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_fold_profiles(const uint64_t* acc_sum, const uint64_t* acc_cnt, int64_t n, float* profiles,
                                hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fold_profiles, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, acc_sum, acc_cnt, n,
                       profiles);
    return hipGetLastError();
}

}  // namespace pond
