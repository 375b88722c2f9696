// K3: inverse column FFTs, square-law detection, the integrated series
// and the fold into per-workgroup integer histograms.
#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "pond_device.hpp"

namespace pond {

// Power buffer: row-major, 16 floats per row, the four float4 quarters of a
// row rotated by (row / 4) mod 4, so that the epilogue's float4 reads of 16
// consecutive rows (one per lane) and the detection's writes of four rows per
// wave use every bank once.
__device__ __forceinline__ int k3_pidx(int row, int col) {
    return row * 16 + ((((col >> 2) + (row >> 2)) & 3) << 2) + (col & 3);
}
// The same with 32 floats per row, rotated by 4 (row mod 8) floats.
__device__ __forceinline__ int k3_pidx32(int row, int x) { return row * 32 + ((x + 4 * (row & 7)) & 31); }

// A power in fixed point: round(val 2^16) to nearest even, 0 for a value that
// is not finite (the product is exact in float32, and so are its two halves).
__device__ __forceinline__ uint64_t fold_fixed(float val) {
    float x = rintf(val * 65536.0f);
    x = fabsf(x) < 18446744073709551616.0f ? x : 0.0f;
    const float hi = floorf(x * 2.3283064365386963e-10f);
    const float lo = fmaf(hi, -4294967296.0f, x);
    return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// The kernel's own arguments where the launch left them.  The epilogue of an
// item reads what it needs from there, through a pointer the compiler cannot
// see through: kept over the transform, its 40 or so scalars would be spilled
// into vector registers.
using K3Kernarg = const __attribute__((address_space(4))) K3Args;
__device__ __forceinline__ K3Kernarg& k3_kernarg() {
    K3Kernarg* p = (K3Kernarg*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *p;
}

// Add fx, the fixed-point sum of `cnt` powers, to the histogram: entry `bin` of
// sub-integration s_base + sub_rel.
__device__ __forceinline__ void k3_fold_add(K3Kernarg& a, uint64_t* hsum, uint32_t* hcnt, int sub_rel, int bin,
                                            uint64_t fx, uint32_t cnt) {
    if (a.global_mode) {
        const int64_t gk = ((int64_t)sub_rel + a.s_base - a.acc_s0) * a.nbins + bin;
        atomicAdd((unsigned long long*)&a.acc_sum[gk], (unsigned long long)fx);
        atomicAdd((unsigned long long*)&a.acc_cnt[gk], (unsigned long long)cnt);
    } else {
        const int key = sub_rel * a.nbins + bin;
        atomicAdd((unsigned long long*)&hsum[key], (unsigned long long)fx);
        atomicAdd(&hcnt[key], cnt);
    }
}

// REAL (real input path, float32 arithmetic): element m of the output is
// y[2m] + i y[2m+1] of the real dedispersed voltage, detected per real
// sample (y^2); the group of 16 elements is 32 real outputs, the series
// (sums over decim elements = 2 decim real samples) is unchanged, and the
// fold takes real sample r = 2 m + j with phase (r + 2 n_front) inv_pfs
// (inv_pfs of the real sample rate).
//
// An item is 16 columns of a block: thread (c, j) transforms column c, holding
// rows j + TPV e, and leaves the detected powers in LDS, in the tile the
// transform has left; thread q then takes the 16 consecutive outputs of row q.
// Bound: the exchanges' barriers and the strided tile reads in turn (2^23,
// packed float16, per block: 14.4 us; 13.8 without the transform, 10.6 with
// every tile in L2, 12.2 without the series, whose 4-byte stores fall in one
// cache line each).  So the powers take no LDS of their own (68 KB instead of
// 133) and the epilogue's scalars and float64 constants no registers (k3_kernarg,
// K3Args), which lets two workgroups share a CU in packed float16 (TWO); the fold
// phase of a group is one float64 product and the second one only near a bin's
// edge.  2^23, per block, before and now: packed float16 in launches of 4 / 8
// 13.5 / 14.3 and 12.1 / 13.1 us; float32 in launches of 3 / 8 18.8 / 22.7 and
// 18.4 / 22.5.
// WIDE (matrix-core form): tiles of 32 columns, two adjacent ones per thread,
// one workgroup per CU (it needs more than 64 registers): 14.2 / 15.3 and 13.7 /
// 13.9 in launches of 4 / 8; packed float16 gains nothing from it.  A reduction of
// the powers across lanes in place of the LDS buffer (four DPP steps) cost 25%
// more VALU instructions and 8% more time.
template <int LOG2N2, class T, int FORM, bool REAL, bool TWO, bool WIDE, bool AHEAD>
__global__ void __launch_bounds__(1 << LOG2N2) __attribute__((amdgpu_waves_per_eu(TWO ? 8 : 4)))
k3_colinv_detect_fold(K3Args args) {
    using Sh = K3Shape<LOG2N2>;
    constexpr int L = Sh::L;
    constexpr int TPV = Sh::TPV;
    __shared__ __align__(16) char lds_raw[Sh::lds(FORM, WIDE)];
    extern __shared__ uint64_t dyn_u64[];
    uint64_t* hsum = dyn_u64;
    uint32_t* hcnt = reinterpret_cast<uint32_t*>(dyn_u64 + (args.global_mode ? 0 : args.entries));
    constexpr bool H16 = FORM == kFormF16 || FORM == kFormMfma;  // float16 arithmetic
    constexpr bool MX = FORM == kFormMfma && kMxShape<LOG2N2, true>;  // radix-16 sums on matrix cores
    static_assert(!WIDE || (MX && !REAL), "32-column tiles: matrix-core form");
    constexpr int W = WIDE ? 2 : 1;  // adjacent columns per thread, groups of 16 outputs per row
    using V = std::conditional_t<WIDE, hh2, std::conditional_t<H16, h2, float2>>;
    V* const tile = reinterpret_cast<V*>(lds_raw);
    float* const pf = reinterpret_cast<float*>(lds_raw);

    // The arguments lie in host memory: fetch all of their cache lines now, in
    // one round trip, for the epilogue's reads (k3_kernarg) to find them.
    asm volatile("" ::"s"(args.work), "s"(args.inv_pfs), "s"(args.acc_sum), "s"(args.inv_subint));

    const int c = threadIdx.x & 15;
    const int j = threadIdx.x >> 4;
    const int n1 = 1 << args.log2n1;
    const int log2tiles = args.log2n1 - (WIDE ? 5 : 4);  // tiles of 16 W columns per block
    const int items = args.nblocks << log2tiles;
    const int r0 = (int)(args.n_front & 15);

    if (!args.global_mode) {
        for (int i = threadIdx.x; i < args.entries; i += blockDim.x) {
            hsum[i] = 0;
            hcnt[i] = 0;
        }
    }
    // Items are split into 8 contiguous chunks, one per XCD, so that the
    // workgroups running together on one XCD handle neighbouring tiles.
    const int per_xcd = gridDim.x >> 3;
    const int xcd = blockIdx.x & 7;
    const int local = blockIdx.x >> 3;
    const int chunk = (items + 7) >> 3;
    const int it_end = min(items, (xcd + 1) * chunk);
    uint32_t flags = 0;
    StageBases<LOG2N2, V> tb;
    tb.load(j, args.tw2);
    // packed float16: the twiddle tables follow the tile
    h2* ttab = reinterpret_cast<h2*>(lds_raw + W * Sh::kHalfTile);
    if constexpr (H16) if (threadIdx.x < 64) fill_twiddle_tables<LOG2N2, 64>(ttab, args.tw2, threadIdx.x);

    // The column tile of an item, as stored.  Where one workgroup has the CU
    // (TWO: two share it and hide each other's loads), the next item's tile
    // is loaded while this one is transformed and folded (AHEAD), if it is 64 bytes
    // a thread: the 128 of float32 and of WIDE cost more than they hide where the
    // launch's work area is cached (2^23, per block in launches of 1 / 3 / 8:
    // float32 28.9 / 19.5 / 21.8 us with the read-ahead, 24.7 / 18.4 / 22.5
    // without; matrix-core form of 1 / 4 / 8: 19.7 / 15.0 / 14.6 and 19.1 / 13.7 /
    // 13.9).  Float32 reads ahead where it is not (kAheadBytes).  WIDE: a thread's two
    // columns are one 8-byte access (4-byte aligned), but for the pair that
    // crosses n1 (r0 odd), whose second column is column 0.
    constexpr bool kPrefetch = AHEAD && !TWO && !WIDE && LOG2N2 >= 9;
    using Raw = std::conditional_t<WIDE, hh2, std::conditional_t<H16, h2, T>>;
    auto load_tile = [&](int it, Raw(&dst)[16]) {
        const int bb = it >> log2tiles;
        const int tt = it & ((1 << log2tiles) - 1);
        const uint32_t cc = opaque((uint32_t)((r0 + W * (16 * tt + c)) & (n1 - 1)));
        const T* const ib = uniform_ptr(reinterpret_cast<const T*>(args.work) + ((int64_t)bb << (args.log2n1 + LOG2N2)));
        // matrix-core layout: value e = 4b + t at position
        // 4 (j / 4) + b + (4 (j mod 4) + t) TPV
        const uint32_t ioff =
            (cc + ((uint32_t)(MX ? 4 * (j >> 2) + 4 * (j & 3) * TPV : j) << args.log2n1)) * (uint32_t)sizeof(T);
        auto row = [](int e) { return MX ? (e >> 2) + (e & 3) * TPV : TPV * e; };
        if constexpr (sizeof(T) == 4) {
            // the block through a buffer descriptor: the lane's offset in a
            // vector register, the row offset of value e in a scalar one
            const BufRes rb = buf_res(ib, (uint32_t)sizeof(T) << (args.log2n1 + LOG2N2));
            if constexpr (WIDE) {
                if ((r0 & 1) == 0 || 32 * tt + 32 + r0 <= n1) {
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        dst[e] = buf_ld<hh2>(rb, ioff, (int)(row(e) * sizeof(T)) << args.log2n1);
                } else {
                    // r0 odd, last tile: the second column of a pair may be column 0
                    const uint32_t ioff1 = ioff + (cc + 1 < (uint32_t)n1 ? 1u : 1u - (uint32_t)n1) * (uint32_t)sizeof(T);
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int so = (int)(row(e) * sizeof(T)) << args.log2n1;
                        dst[e] = hh2{buf_ld<h2>(rb, ioff, so), buf_ld<h2>(rb, ioff1, so)};
                    }
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) dst[e] = buf_ld<Raw>(rb, ioff, (int)(row(e) * sizeof(T)) << args.log2n1);
            }
        } else {
#pragma unroll
            for (int e = 0; e < 16; ++e) dst[e] = *at(ib + ((int64_t)(TPV * e) << args.log2n1), ioff);
        }
    };
    Raw nxt[16];
    if constexpr (kPrefetch) {
        if (xcd * chunk + local < it_end) load_tile(xcd * chunk + local, nxt);
    }
    constexpr int G = REAL ? 32 : 16;  // fold samples of a group
    constexpr int U = REAL ? 2 : 1;    // per element
    for (int item = xcd * chunk + local; item < it_end; item += per_xcd) {
        const int b = item >> log2tiles;
        const int t = item & ((1 << log2tiles) - 1);
        V v[16];
        if constexpr (!kPrefetch) load_tile(item, nxt);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if constexpr (H16) v[e] = nxt[e];
            else v[e] = Elem<T>::load(&nxt[e]);
        }
        if constexpr (kPrefetch) {
            if (item + per_xcd < it_end) load_tile(item + per_xcd, nxt);
        }
        if constexpr (MX && WIDE) {
            // one column at a time, each in its own tile
            h2* const t0 = reinterpret_cast<h2*>(lds_raw);
            h2 x[16], y[16];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                x[e] = v[e].a;
                y[e] = v[e].b;
            }
            fft_mx<LOG2N2, +1, false, true, true>(x, j, t0 + c, ttab);
            fft_mx<LOG2N2, +1, false, true, false>(y, j, t0 + 16 * L + c, ttab);
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = hh2{x[e], y[e]};
        } else if constexpr (MX) {
            fft_mx<LOG2N2, +1, false, true, true>(v, j, tile + c, ttab);
        } else if constexpr (H16) {
            fft_wg<LOG2N2, +1, false, 2>(v, j, tb, ColSwz<V>{tile + c}, ttab);
        } else {
            fft_wg<LOG2N2, +1>(v, j, tb, ColSwz<V>{tile + c});
        }

        // Detected powers to LDS once every thread has left the transform:
        // rows of 16 powers, or 32 (WIDE: of 32 columns; REAL: two per column).
        __syncthreads();
        K3Kernarg& a = k3_kernarg();
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = j + TPV * e;
            // float16: in float32 from the pair (exact products)
            auto power = [&](h2 y) {
                const float yx = (float)y.x, yy = (float)y.y;
                return fmaf(yx, yx, yy * yy) * a.pscale;
            };
            if constexpr (WIDE) {
                *reinterpret_cast<float2*>(pf + k3_pidx32(row, 2 * c)) = make_float2(power(v[e].a), power(v[e].b));
            } else if constexpr (H16) {
                pf[k3_pidx(row, c)] = power(v[e]);
            } else {
                const float2 y = cscale(v[e], a.scale);
                if constexpr (REAL)
                    *reinterpret_cast<float2*>(pf + k3_pidx32(row, 2 * c)) = make_float2(y.x * y.x, y.y * y.y);
                else
                    pf[k3_pidx(row, c)] = fmaf(y.x, y.x, y.y * y.y);
            }
        }
        __syncthreads();

        // Thread q takes row q: W groups of 16 consecutive kept outputs n = r0 +
        // 16 (W t + g) + n1 q + [0, 16) (columns that wrap past n1 hold them one
        // row further down).
        const int q = threadIdx.x;
#pragma unroll 1
        for (int g = 0; g < W; ++g) {
            const int col0 = r0 + 16 * (W * t + g);
            const int off0 = col0 - (int)a.n_front;
            const int off = off0 + (q << a.log2n1);
            if (off < 0 || off >= (int)a.hop) continue;
            auto pidx = [&](int row, int x) {
                return WIDE || REAL ? k3_pidx32(row, x + 16 * g) : k3_pidx(row, x);
            };
            float p[16];
            float pr[REAL ? 32 : 1];  // REAL: the 32 real-sample powers of the group
            if (col0 + 15 < n1) {
                if constexpr (REAL) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const float4 x4 = *reinterpret_cast<const float4*>(pf + pidx(q, 4 * i));
                        pr[4 * i] = x4.x;
                        pr[4 * i + 1] = x4.y;
                        pr[4 * i + 2] = x4.z;
                        pr[4 * i + 3] = x4.w;
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float4 x4 = *reinterpret_cast<const float4*>(pf + pidx(q, 4 * i));
                        p[4 * i] = x4.x;
                        p[4 * i + 1] = x4.y;
                        p[4 * i + 2] = x4.z;
                        p[4 * i + 3] = x4.w;
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = q + ((col0 + i) >> a.log2n1);
                    if constexpr (REAL) {
                        pr[2 * i] = row < L ? pf[pidx(row, 2 * i)] : 0.f;
                        pr[2 * i + 1] = row < L ? pf[pidx(row, 2 * i + 1)] : 0.f;
                    } else {
                        p[i] = row < L ? pf[pidx(row, i)] : 0.f;
                    }
                }
            }
            if constexpr (REAL) {
#pragma unroll
                for (int i = 0; i < 16; ++i) p[i] = pr[2 * i] + pr[2 * i + 1];
            }

            // Group sum and the decimated series (sums of `decim` consecutive
            // powers, pairwise).
            float s2[8], s4[4], s8[2];
#pragma unroll
            for (int i = 0; i < 8; ++i) s2[i] = p[2 * i] + p[2 * i + 1];
#pragma unroll
            for (int i = 0; i < 4; ++i) s4[i] = s2[2 * i] + s2[2 * i + 1];
            s8[0] = s4[0] + s4[1];
            s8[1] = s4[2] + s4[3];
            const float s16 = s8[0] + s8[1];
            const int64_t mb = (a.block0 + b) * a.hop + off0;  // a multiple of 16
            const int64_t m0 = mb + ((int64_t)q << a.log2n1);  // first output of the group
            if (a.series) {
                const int log2d = __builtin_ctz((unsigned)a.decim);  // decim is a power of two
                float* const sp = a.series + ((mb >> log2d) - a.series_base) + ((int64_t)q << (a.log2n1 - log2d));
                if (a.decim == 16) {
                    sp[0] = s16;
                } else if (a.decim == 8) {
                    sp[0] = s8[0];
                    sp[1] = s8[1];
                } else if (a.decim == 4) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) sp[i] = s4[i];
                } else if (a.decim == 2) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) sp[i] = s2[i];
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) sp[i] = p[i];
                }
            }
            if (!isfinite(s16)) flags |= 1u;
            // (the limit is on what is added at once, not on the group)
            auto range = [&](float v) { return v < (float)kFoldRangeLimit ? 0u : 2u; };

            // Fold: one contribution when all outputs of the group share pulse,
            // bin and sub-integration.  (The element indices are exact in
            // float64, so x0 is fold_bin's phase; a phase within fold_safe of
            // the next bin only fails the test.)
            const uint64_t fx = fold_fixed(s16);
            const double x0 = fma((double)(q << a.log2n1), (double)U, (double)(U * (mb + a.n_front))) * a.inv_pfs;
            const double fl = floor(x0);
            const double y0 = (x0 - fl) * a.nbins_d;
            const int bin0 = min((int)y0, a.nbins - 1);
            const double next = (double)(bin0 + 1);
            // Sub-integration of the group, if the launch spans more than one (in
            // global memory the entries may be more than an int32 counts); its 16
            // outputs share it unless it ends within them.
            int sub0 = 0;
            bool one_sub = true;
            const int64_t d0 = m0 - a.s_base * a.subint;
            if (a.subint > 0 && (a.global_mode || a.entries != a.nbins)) {
                sub0 = (int)subint_rel(d0, a.subint, a.inv_subint);
                one_sub = d0 - sub0 * a.subint + 15 < a.subint;
            }
            if (one_sub && y0 + fma(x0, a.fold_safe1, a.fold_safe0) < next) {
                flags |= range(s16);
                k3_fold_add(a, hsum, hcnt, sub0, bin0, fx, G);
                continue;
            }
            // Otherwise by the per-sample float64 evaluation itself.
            const int64_t f0i = U * m0, fnf = U * a.n_front;
            double t15;
            const int bin15 = fold_bin(f0i + G - 1, fnf, a.inv_pfs, a.nbins, &t15);
            if (one_sub && bin0 == bin15 && fl == t15) {
                flags |= range(s16);
                k3_fold_add(a, hsum, hcnt, sub0, bin0, fx, G);
                continue;
            }
            // Phase grows with the sample index, so each (pulse, bin) cell holds
            // consecutive samples.  Two cells (the bin is longer than the
            // group): the first ends before sample `hi`, estimated from the phase
            // and checked on both sides; two partial sums.
            if (one_sub) {
                // (where a bin is a whole number of samples, rounding decides
                // whose the boundary sample is: the estimate takes the lower one)
                int hi = max(1, min(G - 1, (int)ceil((next - y0) * a.samples_per_bin - 1e-3)));
                double ta, tb2;
                const int ba = fold_bin(f0i + hi - 1, fnf, a.inv_pfs, a.nbins, &ta);
                int bb = fold_bin(f0i + hi, fnf, a.inv_pfs, a.nbins, &tb2);
                if (bb == bin0 && tb2 == fl) {
                    ++hi;  // below G: the last sample is in another cell
                    bb = fold_bin(f0i + hi, fnf, a.inv_pfs, a.nbins, &tb2);
                }
                if (ba == bin0 && ta == fl && bb == bin15 && tb2 == t15) {
                    // (each from its own samples: the rest of s16 carries the
                    // rounding of both, either sign where the second is silent)
                    float sa = 0.f, sb = 0.f;
#pragma unroll
                    for (int i = 0; i < G; ++i) sa += i < hi ? (REAL ? pr[i] : p[i]) : 0.f;
                    const int hi2 = (int)opaque((uint32_t)hi);  // (16 comparisons made again, not kept)
#pragma unroll
                    for (int i = 0; i < G; ++i) sb += i < hi2 ? 0.f : (REAL ? pr[i] : p[i]);
                    flags |= range(sa) | range(sb);
                    k3_fold_add(a, hsum, hcnt, sub0, bin0, fold_fixed(sa), (uint32_t)hi);
                    k3_fold_add(a, hsum, hcnt, sub0, bin15, fold_fixed(sb), (uint32_t)(G - hi));
                    continue;
                }
            }
            // A bin shorter than the group, a sub-integration edge, or an
            // estimate further off: one add per sample (from LDS again: no
            // thread writes there before the next item's first barrier).
            for (int i = 0; i < G; ++i) {
                const int ci = REAL ? i >> 1 : i;
                const int row = q + ((col0 + ci) >> a.log2n1);
                const float pi = row >= L ? 0.f : pf[pidx(row, i)];
                double ti;
                const int bi = fold_bin(f0i + i, fnf, a.inv_pfs, a.nbins, &ti);
                const int si = a.subint > 0 ? (int)subint_rel(d0 + ci, a.subint, a.inv_subint) : 0;
                flags |= range(pi);
                k3_fold_add(a, hsum, hcnt, si, bi, fold_fixed(pi), 1);
            }
        }
    }
    K3Kernarg& a = k3_kernarg();
    if (flags) atomicOr(a.status, flags);
    if (!a.global_mode) {
        __syncthreads();
        uint64_t* ps = a.part_sum + (int64_t)blockIdx.x * a.entries;
        uint32_t* pc = a.part_cnt + (int64_t)blockIdx.x * a.entries;
        for (int i = threadIdx.x; i < a.entries; i += blockDim.x) {
            ps[i] = hsum[i];
            pc[i] = hcnt[i];
        }
    }
}

template <class T, int FORM, int LOG2N2, bool REAL, bool TWO, bool WIDE = false, bool AHEAD = sizeof(T) == 4>
static hipError_t k3_launch(const K3Args& a, int grid, size_t dyn, hipStream_t s) {
    static const hipError_t attr = hipFuncSetAttribute(
        reinterpret_cast<const void*>(&k3_colinv_detect_fold<LOG2N2, T, FORM, REAL, TWO, WIDE, AHEAD>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)(160 * 1024 - K3Shape<LOG2N2>::lds(FORM, WIDE)));
    if (attr != hipSuccess) return attr;
    K3Args c = a;
    const double per_sample = a.inv_pfs * (double)a.nbins;  // bins per sample
    c.nbins_d = (double)a.nbins;
    c.fold_safe0 = (REAL ? 31 : 15) * per_sample + 1e-9;
    c.fold_safe1 = 1e-15 * (double)a.nbins;
    c.samples_per_bin = 1.0 / per_sample;
    c.inv_subint = a.subint > 0 ? 1.0 / (double)a.subint : 0.0;
    hipLaunchKernelGGL((k3_colinv_detect_fold<LOG2N2, T, FORM, REAL, TWO, WIDE, AHEAD>), dim3(grid), dim3(1 << LOG2N2), dyn,
                       s, c);
    return hipGetLastError();
}

// 32-column tiles (items: of 16 columns): the matrix-core form's columns of 2^10,
// where they leave an item for every CU and the histogram fits beside them.
constexpr int64_t kWideItems = 256;
static bool k3_wide(bool mfma, int log2n2, int64_t items, size_t dyn) {
    return mfma && log2n2 == 10 && items / 2 >= kWideItems && K3Shape<10>::LDS_WIDE + dyn <= kLdsBytes;
}

constexpr int64_t kAheadBytes = 1ll << 28;  // of work area in a launch: the Infinity Cache

template <class T, int FORM, int LOG2N2>
static hipError_t k3_one(const K3Args& a, int grid, size_t dyn, hipStream_t s) {
    if constexpr (FORM == kFormMfma && LOG2N2 == 10) {
        if (k3_wide(true, LOG2N2, (int64_t)a.nblocks << (a.log2n1 - 4), dyn))
            return k3_launch<T, FORM, LOG2N2, false, false, true>(a, grid, dyn, s);
    }
    // Packed float16, columns of 2^9 and 2^10: two (four) workgroups share a CU
    // at 64 registers, unless the histogram leaves no room for two.  (Shorter
    // columns fit four to a CU either way, and the matrix-core form needs more
    // registers than that.)
    if constexpr (FORM == kFormF16 && LOG2N2 >= 9) {
        if (2 * (K3Shape<LOG2N2>::lds(FORM) + dyn) <= kLdsBytes)
            return k3_launch<T, FORM, LOG2N2, false, true>(a, grid, dyn, s);
    }
    // Float32: beyond the 256 MB Infinity Cache the work area comes from memory, and
    // the read-ahead pays (512 MB: 2^23 21.8 us a block against 22.5, 2^24 48.3 and
    // 48.8; 256 MB 21.9 and 21.8, 48.6 and 48.8; 2^26, DM 130, the call 4,793 and
    // 4,817 us).
    if constexpr (FORM == kFormF32 && LOG2N2 == 10 && sizeof(T) == 8) {
        if (((int64_t)a.nblocks << (a.log2n1 + LOG2N2)) * (int64_t)sizeof(T) > kAheadBytes)
            return k3_launch<T, FORM, LOG2N2, false, false, false, true>(a, grid, dyn, s);
    }
    return k3_launch<T, FORM, LOG2N2, false, false>(a, grid, dyn, s);
}

template <class T, int FORM>
static hipError_t k3_dispatch(int log2n2, const K3Args& a, int grid, size_t dyn, hipStream_t s) {
    switch (log2n2) {
        case 5: return k3_one<T, FORM, 5>(a, grid, dyn, s);
        case 6: return k3_one<T, FORM, 6>(a, grid, dyn, s);
        case 7: return k3_one<T, FORM, 7>(a, grid, dyn, s);
        case 8: return k3_one<T, FORM, 8>(a, grid, dyn, s);
        case 9: return k3_one<T, FORM, 9>(a, grid, dyn, s);
        case 10: return k3_one<T, FORM, 10>(a, grid, dyn, s);
        default: return hipErrorInvalidValue;
    }
}

template <class T>
static hipError_t k3_real_dispatch(int log2n2, const K3Args& a, int grid, size_t dyn, hipStream_t s) {
    switch (log2n2) {
        case 5: return k3_launch<T, kFormF32, 5, true, false>(a, grid, dyn, s);
        case 6: return k3_launch<T, kFormF32, 6, true, false>(a, grid, dyn, s);
        case 7: return k3_launch<T, kFormF32, 7, true, false>(a, grid, dyn, s);
        case 8: return k3_launch<T, kFormF32, 8, true, false>(a, grid, dyn, s);
        case 9: return k3_launch<T, kFormF32, 9, true, false>(a, grid, dyn, s);
        case 10: return k3_launch<T, kFormF32, 10, true, false>(a, grid, dyn, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_k3_real(int prec, int log2n2, const K3Args& a, int grid, size_t dyn, hipStream_t s) {
    switch (prec) {
        case kFp32: return k3_real_dispatch<float2>(log2n2, a, grid, dyn, s);
        case kMixedValu: return k3_real_dispatch<__half2>(log2n2, a, grid, dyn, s);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_k3(int prec, int log2n2, const K3Args& a, int grid, size_t dyn, hipStream_t s) {
    switch (prec) {
        case kMixed: return k3_dispatch<__half2, kFormMfma>(log2n2, a, grid, dyn, s);
        case kMixedValu: return k3_dispatch<__half2, kFormF32>(log2n2, a, grid, dyn, s);
        case kHalf: return k3_dispatch<__half2, kFormF16>(log2n2, a, grid, dyn, s);
        case kBf16: return k3_dispatch<bf16x2, kFormF32>(log2n2, a, grid, dyn, s);
        default: return k3_dispatch<float2, kFormF32>(log2n2, a, grid, dyn, s);
    }
}

int64_t hist_capacity(int log2n2, int prec) {
    const int64_t cap = (int64_t)((kLdsBytes - k3_static_lds(log2n2, prec)) / 12);
    return cap < kHistCapMax ? cap : kHistCapMax;
}

int k3_grid(int log2n2, int prec, size_t dyn_lds, int64_t items, int64_t entries, bool global_mode,
            int64_t part_entries) {
    const bool wide = k3_wide(prec == kMixed, log2n2, items, dyn_lds);
    if (wide) items /= 2;
    const size_t lds = (wide ? K3Shape<10>::LDS_WIDE : k3_static_lds(log2n2, prec)) + dyn_lds;
    int per_cu = (int)(kLdsBytes / lds);
    per_cu = per_cu < 1 ? 1 : (per_cu > 4 ? 4 : per_cu);
    int64_t grid = 256 * per_cu;
    if (!global_mode && grid * entries > part_entries) grid = part_entries / entries;
    const int64_t items8 = (items + 7) & ~int64_t(7);
    if (grid > items8) grid = items8;
    grid &= ~int64_t(7);
    if (grid < 8) grid = 8;
    return (int)grid;
}

size_t k3_static_lds(int log2n2, int prec) {
    if (prec != kHalf && prec != kMixed) return sizeof(float2) * 16 * ((size_t)1 << log2n2);
    switch (log2n2) {
        case 5: return K3Shape<5>::LDS_HALF;
        case 6: return K3Shape<6>::LDS_HALF;
        case 7: return K3Shape<7>::LDS_HALF;
        case 8: return K3Shape<8>::LDS_HALF;
        case 9: return K3Shape<9>::LDS_HALF;
        default: return K3Shape<10>::LDS_HALF;
    }
}
int k1_threads(int log2n2) { return 1 << log2n2; }
int k3_threads(int log2n2) { return 1 << log2n2; }
int k2_threads(int log2n1) {
    const int tpv = (1 << log2n1) / 16;
    return tpv >= 256 ? tpv : 256;
}

// The host-side table scale must match the device schedule.
static_assert(half_row_rem(5) == Sched<5>::kHalfRem && half_row_rem(6) == Sched<6>::kHalfRem &&
                  half_row_rem(7) == Sched<7>::kHalfRem && half_row_rem(8) == Sched<8>::kHalfRem &&
                  half_row_rem(9) == Sched<9>::kHalfRem && half_row_rem(10) == Sched<10>::kHalfRem &&
                  half_row_rem(11) == Sched<11>::kHalfRem && half_row_rem(12) == Sched<12>::kHalfRem &&
                  half_row_rem(13) == Sched<13>::kHalfRem && half_row_rem(14) == Sched<14>::kHalfRem,
              "row normalisation split");
}  // namespace pond
