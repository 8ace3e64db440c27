// Seismograms at R receivers and their ensemble statistics, from the state
// traces of a stepped chunk.
//
// Method: the velocity at a target point is reconstructed from a single row
// of the velocity basis, so a receiver is a row c_r of length Kv and its
// seismogram for sample m after step n is  Y[n][r][m] = c_r . V_m^(n+1)
// (Sec. 4.5).  Over the ensemble of M samples each (step, receiver) gets
// the mean, the population variance and the nearest-rank 5th / 50th / 95th
// percentiles (the ceil(p M / 100)-th smallest value), the statistics the
// paper plots for its ensemble.
//
// One workgroup per step of the chunk.  Thread t owns sample columns
// t, t + 256, ... and accumulates the dot products of kRcRows receivers at a
// time in FP64.  The trace comes through LDS in tiles of kRcTile entries of
// 256 columns, read in lines; the receiver rows, k-major in FP64, are scalar
// operands of the multiply-adds.  Then each wave takes receivers of its own:
// fixed-order sums, and the three percentiles by bisection, counting the
// values up to a pivot with a compare and a ballot per register of values.
//
// Bound by the FP64 multiply-adds and the trace's bytes.  Measured, 500 steps
// of K = 256, M = 256, R = 16: 300 us with one uncoalesced column per thread,
// receiver rows converted in LDS and a block-wide bitonic sort per receiver,
// now 120.
#include <math.h>

#include "k_common.h"
#include "k_lane.h"
#include "rom_internal.h"

namespace rom {
namespace {

constexpr int kRcThreads = 256;
constexpr int kRcWaves = kRcThreads / 64;
constexpr int kRcRows = 16;        // receivers per accumulation pass
constexpr int kRcTile = 32;        // trace entries per LDS tile
constexpr int kRcLd = kRcTile + 1;

// c64[k][r] = C[r][k], zero from row R on (rp rows).
__global__ void receiver_rows_kernel(const float *__restrict__ C, int R, int rp, int kv, double *__restrict__ c64) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= kv * rp) return;
    const int k = idx / rp, r = idx - k * rp;
    c64[idx] = r < R ? (double)C[(size_t)r * kv + k] : 0.0;
}

// The sum over the wave in each lane, as a tree over the lane's bits from
// the highest down (values that agree across bit 3 need row_ror:4 for bit 2).
__device__ __forceinline__ double tree_sum(double x) {
    x = lane::swap_sum64<true>(x);
    x = lane::swap_sum64<false>(x);
    x += lane::dpp_mov64<lane::kDppRor8>(x);
    x += lane::dpp_mov64<0x124>(x);
    x += lane::dpp_mov64<lane::kDppXor2>(x);
    x += lane::dpp_mov64<lane::kDppXor1>(x);
    return x;
}

__device__ __forceinline__ double wave_max(double x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x = fmax(x, __shfl_xor(x, o, 64));
    return x;
}

// Order-preserving integers of doubles (and back).
__device__ __forceinline__ long long key_of(double x) {
    const long long b = __builtin_bit_cast(long long, x);
    return b < 0 ? (long long)(0x8000000000000000ull - (unsigned long long)b) : b;
}
__device__ __forceinline__ double value_of(long long k) {
    return __builtin_bit_cast(double, k < 0 ? (long long)(0x8000000000000000ull - (unsigned long long)k) : k);
}

// The values of the wave (E per lane) up to v.
template <int E>
__device__ __forceinline__ int count_to(const double (&x)[E], double v) {
    int n = 0;
#pragma unroll
    for (int e = 0; e < E; ++e) n += __popcll(__ballot(x[e] <= v));
    return n;
}

// The value at 0-based sorted position k of the wave's values, all in [lo,
// hi].  Kept: count_to(below) <= k < count_to(hi).  The pivot halves the
// interval of values, after 24 rounds that of their integers, so the loop
// ends after 24 + 64 rounds at the latest (also with values that compare with
// nothing); one value left in the interval ends it at once.
template <int E>
__device__ __forceinline__ double select(const double (&x)[E], int k, double lo, double hi) {
    const int c0 = count_to(x, lo);
    if (k < c0) return lo;
    long long kl = key_of(lo), kh = key_of(hi);
    int nl = c0, nh = count_to(x, hi);
    for (int it = 0; it < 88 && kl + 1 < kh; ++it) {
        if (nh - nl == 1) {
            // the one value in (lo, hi]
            const double l = value_of(kl), h = value_of(kh);
            double v = h;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const unsigned long long m = __ballot(x[e] > l && x[e] <= h);
                if (m) v = __shfl(x[e], __ffsll((long long)m) - 1, 64);
            }
            return v;
        }
        long long km = kl + (long long)((unsigned long long)(kh - kl) >> 1);
        if (it < 24) {
            const long long t = key_of(0.5 * value_of(kl) + 0.5 * value_of(kh));
            if (t > kl && t < kh) km = t;
        }
        const int n = count_to(x, value_of(km));
        if (k < n) {
            kh = km;
            nh = n;
        } else {
            kl = km;
            nl = n;
        }
    }
    return value_of(kh);
}

// Mean, variance and percentiles of yr[0 .. M), by one wave (M <= 64 E).
// The sums: of yr[t], yr[t + 256], .. for t = 0 .. 255 in order, then a tree
// over t from its highest bit down.
template <int E>
__device__ __forceinline__ void wave_stats(const double *yr, int M, int lane, int i0, int i1, int i2, double *o) {
    double x[E], s[4];
#pragma unroll
    for (int e = 0; e < E; ++e) x[e] = 64 * e + lane < M ? yr[64 * e + lane] : HUGE_VAL;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        s[t] = 0.0;
#pragma unroll
        for (int e = t; e < E; e += 4)
            if (64 * e + lane < M) s[t] += x[e];
    }
    const double mean = tree_sum((s[0] + s[2]) + (s[1] + s[3])) / M;
    double hi = -HUGE_VAL, lo = -HUGE_VAL;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        s[t] = 0.0;
#pragma unroll
        for (int e = t; e < E; e += 4)
            if (64 * e + lane < M) {
                const double d = x[e] - mean;
                s[t] += d * d;
            }
    }
    const double var = tree_sum((s[0] + s[2]) + (s[1] + s[3])) / M;
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (64 * e + lane < M) {
            hi = fmax(hi, x[e]);
            lo = fmax(lo, -x[e]);
        }
    hi = wave_max(hi);
    lo = -wave_max(lo);
    // NaN sorts behind every number
    int nn = M;
#pragma unroll
    for (int e = 0; e < E; ++e) nn -= __popcll(__ballot(x[e] != x[e]));
    auto value = [&](int k) { return k < nn ? select(x, k, lo, hi) : __builtin_nan(""); };
    const double p0 = value(i0), p1 = value(i1), p2 = value(i2);
    if (lane == 0) {
        o[0] = mean;
        o[1] = var;
        o[2] = p0;
        o[3] = p1;
        o[4] = p2;
    }
}

// vtr: (L + 1) x M x Kv FP32 states, entry n + 1 = after step n of the
// chunk; c64: Kv x rp FP64 (receiver_rows_kernel); Y: L x R x M FP64 (or
// null); stats: L x R x 5 FP64 (or null): mean, variance, p0, p1, p2
// percentiles at the 0-based sorted positions i0, i1, i2.
template <int E>
__global__ __launch_bounds__(kRcThreads) void receivers_kernel(const float *__restrict__ vtr, int kv, int M,
                                                               const double *__restrict__ c64, int R, int rp,
                                                               double *__restrict__ Y, double *__restrict__ stats,
                                                               int i0, int i1, int i2) {
    extern __shared__ __align__(16) unsigned char smem[];
    float *vt = reinterpret_cast<float *>(smem);                     // [min(M, 256)][kRcLd]
    const int mt = min(M, kRcThreads);
    double *ys = reinterpret_cast<double *>(vt + (mt * kRcLd + 3) / 4 * 4);   // [R][M]
    const int n = blockIdx.x, tid = threadIdx.x;
    const float *V = vtr + (size_t)(n + 1) * M * kv;

    for (int m0 = 0; m0 < M; m0 += kRcThreads) {
        const int m = m0 + tid, nm = min(kRcThreads, M - m0);
        for (int r0 = 0; r0 < R; r0 += kRcRows) {
            double acc[kRcRows];
#pragma unroll
            for (int i = 0; i < kRcRows; ++i) acc[i] = 0.0;
            // the next tile's loads are in flight while a tile is used (behind
            // the last column the buffer's bound gives zeros)
            constexpr int kPer = kRcTile;      // entries per thread of 256 columns
            const int kk = tid & (kRcTile - 1), j0 = tid / kRcTile;
            float next[kPer];
            const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<float *>(V + (size_t)m0 * kv), (short)0, nm * kv * 4, 0x00020000);
            auto load = [&](int k0) {
#pragma unroll
                for (int i = 0; i < kPer; ++i)
                    next[i] = __builtin_bit_cast(
                        float, __builtin_amdgcn_raw_buffer_load_b32(
                                   rv, ((j0 + i * (kRcThreads / kRcTile)) * kv + kk + k0) * 4, 0, 0));
            };
            load(0);
            for (int k0 = 0; k0 < kv; k0 += kRcTile) {
                const int nk = min(kRcTile, kv - k0);
                __syncthreads();
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int j = j0 + i * (kRcThreads / kRcTile);
                    if (j < mt) vt[j * kRcLd + kk] = next[i];
                }
                __syncthreads();
                load(k0 + kRcTile);
                if (m < M) {
                    const double *ck = c64 + (size_t)k0 * rp + r0;
                    // (four entries' rows requested at once)
                    int k = 0;
                    for (; k + 4 <= nk; k += 4, ck += 4 * rp) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const double v = (double)vt[tid * kRcLd + k + j];
#pragma unroll
                            for (int i = 0; i < kRcRows; ++i) acc[i] = fma(ck[j * rp + i], v, acc[i]);
                        }
                    }
                    for (; k < nk; ++k, ck += rp) {
                        const double v = (double)vt[tid * kRcLd + k];
#pragma unroll
                        for (int i = 0; i < kRcRows; ++i) acc[i] = fma(ck[i], v, acc[i]);
                    }
                }
            }
            if (m < M) {
#pragma unroll
                for (int i = 0; i < kRcRows; ++i)
                    if (r0 + i < R) ys[(size_t)(r0 + i) * M + m] = acc[i];
            }
        }
    }
    __syncthreads();
    if (Y) {
        double *Yn = Y + (size_t)n * R * M;
        for (int idx = tid; idx < R * M; idx += kRcThreads) Yn[idx] = ys[idx];
    }
    if (!stats) return;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int r = w; r < R; r += kRcWaves)
        wave_stats<E>(ys + (size_t)r * M, M, tid & 63, i0, i1, i2, stats + ((size_t)n * R + r) * 5);
}

int pow2_at_least(int x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

int padded_rows(int R) { return (R + kRcRows - 1) / kRcRows * kRcRows; }

typedef void (*Receivers)(const float *, int, int, const double *, int, int, double *, double *, int, int, int);
constexpr Receivers kReceivers[5] = {receivers_kernel<1>, receivers_kernel<2>, receivers_kernel<4>,
                                     receivers_kernel<8>, receivers_kernel<16>};

}  // namespace

// The limit of what a run takes (one workgroup's receivers, samples and
// rows), not the LDS that it uses, which is less.
size_t receivers_lds_bytes(int kv, int M, int R) {
    const int P = pow2_at_least(M);
    return sizeof(double) * ((size_t)R * M + P + kRcThreads) + sizeof(float) * (size_t)kv * padded_rows(R);
}

size_t receivers_rows_bytes(int kv, int R) { return sizeof(double) * (size_t)kv * padded_rows(R); }

hipError_t launch_receiver_rows(const float *C, int R, int kv, double *c64, hipStream_t st) {
    const int rp = padded_rows(R);
    hipLaunchKernelGGL(receiver_rows_kernel, dim3((kv * rp + 255) / 256), dim3(256), 0, st, C, R, rp, kv, c64);
    return hipGetLastError();
}

static int pct_index(int p, int M) {
    const int k = (p * M + 99) / 100;
    return (k < 1 ? 1 : k) - 1;
}

hipError_t launch_receivers(const float *vtr, int kv, int M, int L, const double *c64, int R, double *Y,
                            double *stats, hipStream_t st) {
    if (L <= 0) return hipSuccess;
    if (M < 1 || M > 1024) return hipErrorInvalidValue;
    const int mt = M < kRcThreads ? M : kRcThreads;
    const size_t lds = sizeof(float) * (size_t)((mt * kRcLd + 3) / 4 * 4) + sizeof(double) * (size_t)R * M;
    int i = 0;
    while (64 << i < M) ++i;
    hipLaunchKernelGGL(kReceivers[i], dim3(L), dim3(kRcThreads), lds, st, vtr, kv, M, c64, R, padded_rows(R), Y,
                       stats, pct_index(5, M), pct_index(50, M), pct_index(95, M));
    return hipGetLastError();
}

hipError_t receivers_configure() {
    for (Receivers f : kReceivers) {
        const hipError_t e = hipFuncSetAttribute((const void *)f, hipFuncAttributeMaxDynamicSharedMemorySize,
                                                 160 * 1024);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rom
