// Support kernels of the discrete adjoint: the operator-gradient products
// dAvs += dt * W * S^T and dAsv += dt * Q * V^T over all (step, sample)
// pairs of a checkpoint segment, packing of the transposed operators for the
// reverse sweep, and the final FP64 -> FP32 conversion.
//
// The gradient product reduces over segment_length * M terms (~1.8e4 at the
// adjoint workload, ~1.3e6 over a whole run).  It runs on
// v_mfma_f32_16x16x4f32: the FP32 trace values multiply exactly, each MFMA
// chain sums kChainSteps * 4 = 64 terms in FP32, and every chain is folded
// into FP64 sums, so the result keeps ~1e-7 relative accuracy over any
// reduction length.  The reduction is split over waves and workgroups; the
// FP64 partials are summed in a fixed order by a second kernel, so the
// gradient is deterministic.
#include <algorithm>

#include "k_common.h"
#include "rom_internal.h"

namespace rom {
namespace {

using dev::f4;
constexpr int kTile = 64;         // output rows and columns per wave (and per workgroup)
constexpr int kChainSteps = 16;   // MFMA k-steps (4 terms each) per FP32 chain
constexpr int kDepth = 4;         // k-steps of operand loads in flight

// Four consecutive rows r .. r+3 of column k of a column-major matrix with
// `ld` rows, read at an address clamped into the matrix (column ke - 1 past
// the end of the reduction, row 0 past the last row), so the load is always
// in bounds and never has to be waited for before its use.  Values of rows
// past the end only reach output rows that are never stored; values past
// the end of the reduction are zeroed where they are used.  VEC: ld and r
// are multiples of 4 (one aligned float4).
template <bool VEC>
__device__ __forceinline__ f4 load_rows4(const float *__restrict__ A, int r, int ld, int64_t k, int64_t ke) {
    const float *col = A + (k < ke ? k : ke - 1) * ld;
    if (VEC) return *reinterpret_cast<const f4 *>(col + (r < ld ? r : 0));
    f4 v;
#pragma unroll
    for (int s = 0; s < 4; ++s) v[s] = col[r + s < ld ? r + s : ld - 1];
    return v;
}

__host__ __device__ __forceinline__ int tiles_of(int rows, int cols) {
    return ((rows + kTile - 1) / kTile) * ((cols + kTile - 1) / kTile);
}

// Up to two products X Y^T over one reduction, in one launch.
struct Products {
    const float *X[2], *Y[2];
    int rows[2], cols[2];
    int n0;                        // work items of the first
};

// part[split][col][row] = sum over k in split's range of X[row][k] Y[col][k]
// for a 64 x 64 output tile; wave w of the workgroup takes a quarter of the
// split.  Lane l loads rows r0 + 4 (l % 16) + s (s = 0..3) of reduction
// index k0 + l / 16, which makes s the row phase of four 16-row MFMA A
// fragments (and likewise four B fragments for the columns): 2 loads feed 16
// MFMAs.  MFMA output register r of fragment pair (s, s') in lane l is row
// r0 + 16 (l / 16) + 4 r + s, column c0 + 4 (l % 16) + s'.  The waves'
// quarters meet in LDS, added in order.
//
// Bound by the operands' bytes behind the L2 unless the workgroups of an XCD
// read the same columns at the same time: workgroup b runs on XCD b % 8, and
// an XCD takes consecutive work items, the tiles of a split next to each
// other.  Measured, a segment's two products (512 x 512, 7936 columns): 132
// us with a split's tiles spread over the XCDs, a launch and 16 partials per
// product, now 89, and the sum of the partials 4 instead of 27.
constexpr int kLdT = kTile + 2;
constexpr size_t kGemmLds = sizeof(double) * 4 * kTile * kLdT;

template <bool VEC>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void gemm_nt_mfma_kernel(Products pr, int items, int64_t R, int64_t kper, double *__restrict__ part) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int li = lane & 15, lk = lane >> 4;
    int it = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (it >= items) return;
    const int q = it >= pr.n0 ? 1 : 0;
    if (q) it -= pr.n0;
    const float *__restrict__ X = pr.X[q], *__restrict__ Y = pr.Y[q];
    const int rows = pr.rows[q], cols = pr.cols[q];
    const int tr = (rows + kTile - 1) / kTile, tc = (cols + kTile - 1) / kTile;
    const int split = it / (tr * tc), tile = it % (tr * tc);
    const int r0 = tile % tr * kTile, c0 = tile / tr * kTile;
    const int64_t kb = min((int64_t)(4 * split + w) * kper, R);
    const int64_t ke = kb + kper < R ? kb + kper : R;
    const int rr = r0 + 4 * li, cc = c0 + 4 * li;
    double acc[4][4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[s][t][r] = 0.0;
    // operands of k-step j sit in ring slot j % kDepth, loaded kDepth steps
    // before their MFMAs
    f4 ra[kDepth], rb[kDepth];
#pragma unroll
    for (int d = 0; d < kDepth; ++d) {
        ra[d] = load_rows4<VEC>(X, rr, rows, kb + 4 * d + lk, ke);
        rb[d] = load_rows4<VEC>(Y, cc, cols, kb + 4 * d + lk, ke);
    }
    for (int64_t k0 = kb; k0 < ke; k0 += 4 * kChainSteps) {
        f4 ch[4][4];
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t) ch[s][t] = f4{0.f, 0.f, 0.f, 0.f};
        // the ring is carried by this (rolled) loop, so the compiler cannot
        // sink a prefetch next to its use
#pragma unroll 1
        for (int g = 0; g < kChainSteps; g += kDepth) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                // k-step k0/4 + g + d; zero the A operand past the reduction
                const bool kin = k0 + 4 * (g + d) + lk < ke;
                f4 a;
#pragma unroll
                for (int s = 0; s < 4; ++s) a[s] = kin ? ra[d][s] : 0.f;
                const f4 b = rb[d];
                const int64_t kn = k0 + 4 * (g + d + kDepth) + lk;
                ra[d] = load_rows4<VEC>(X, rr, rows, kn, ke);
                rb[d] = load_rows4<VEC>(Y, cc, cols, kn, ke);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int t = 0; t < 4; ++t)
                        ch[s][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[t], ch[s][t], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[s][t][r] += (double)ch[s][t][r];
    }
    double *sm = reinterpret_cast<double *>(smem);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                sm[(size_t)(w * kTile + 4 * li + t) * kLdT + 16 * lk + 4 * r + s] = acc[s][t][r];
    __syncthreads();
    double *P = part + (q ? (size_t)(pr.n0 / tiles_of(pr.rows[0], pr.cols[0])) * pr.rows[0] * pr.cols[0] : 0) +
                (size_t)split * rows * cols;
    for (int i = threadIdx.x; i < kTile * kTile; i += 256) {
        const int r = i % kTile, c = i / kTile;
        const double *d = sm + (size_t)c * kLdT + r;
        if (r0 + r < rows && c0 + c < cols)
            P[r0 + r + (size_t)(c0 + c) * rows] = ((d[0] + d[kTile * kLdT]) + d[2 * kTile * kLdT]) + d[3 * kTile * kLdT];
    }
}

// dA[i] += alpha * sum_p part[p][i], p = 0 .. nsplit - 1 in order, for the
// launch's products (blockIdx.y).
__global__ void reduce_parts_kernel(const double *__restrict__ part0, int nsplit, int64_t n, double alpha,
                                    double *__restrict__ dA0, double *__restrict__ dA1) {
    const double *part = part0 + (size_t)blockIdx.y * nsplit * n;
    double *dA = blockIdx.y ? dA1 : dA0;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        double v = 0.0;
        for (int p = 0; p < nsplit; ++p) v += part[(size_t)p * n + i];
        dA[i] += alpha * v;
    }
}

// ytr[k M + m] = c . (state m at trace entry k + 1) for k < len: the forward
// probe trace of a segment recovered from its state traces (one wave per
// value, lanes striding over the rows, FP64 sums).
__global__ __launch_bounds__(256) void probe_trace_kernel(const float *__restrict__ vtr, const float *__restrict__ c,
                                                          int kv, int M, int64_t len, double *__restrict__ ytr) {
    const int lane = threadIdx.x & 63;
    const int64_t nval = len * M;
    for (int64_t idx = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); idx < nval; idx += (int64_t)gridDim.x * 4) {
        const float *v = vtr + (size_t)(idx + M) * kv;      // entry k + 1, column m: (k + 1) M + m = idx + M
        double acc = 0.0;
        for (int i = lane; i < kv; i += 64) acc += (double)c[i] * (double)v[i];
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if (lane == 0) ytr[idx] = acc;
    }
}

__global__ void f64_to_f32_kernel(const double *__restrict__ s, float *__restrict__ d, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        d[i] = (float)s[i];
}

// pk[t][k/4][lane][k%4] = T[64 t + lane][k], T = A or A^T (A column-major
// rows x cols), zero outside T; padded T sizes prow x pcol.
__global__ void pack_from_f32_kernel(const float *__restrict__ A, int rows, int cols, int tr,
                                     int prow, int pcol, float *__restrict__ pk) {
    const int tR = tr ? cols : rows, tC = tr ? rows : cols;
    const int64_t total = (int64_t)prow * pcol;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        int64_t r = idx;
        const int k4 = (int)(r % 4); r /= 4;
        const int lane = (int)(r % 64); r /= 64;
        const int kq = (int)(r % (pcol / 4)); r /= (pcol / 4);
        const int i = (int)r * kTileRows + lane, k = kq * 4 + k4;
        float v = 0.f;
        if (i < tR && k < tC) v = tr ? A[k + (int64_t)i * rows] : A[i + (int64_t)k * rows];
        pk[idx] = v;
    }
}

int grid_for(int64_t n, int cap) {
    int64_t b = (n + 255) / 256;
    return (int)(b < 1 ? 1 : (b > cap ? cap : b));
}

}  // namespace

// Splits of the reduction: enough tiles x splits to cover the CUs once (at
// most 8, at least 1).
static int gemm_nt_zsplit(int rows, int cols, int n) {
    const int tiles = n * tiles_of(rows, cols);
    const int z = (256 + tiles - 1) / tiles;
    return z < 1 ? 1 : (z > 8 ? 8 : z);
}

size_t gemm_nt_part_doubles(int rows, int cols) {
    const int z1 = gemm_nt_zsplit(rows, cols, 1), z2 = 2 * gemm_nt_zsplit(rows, cols, 2);
    return (size_t)(z1 > z2 ? z1 : z2) * rows * cols;
}

hipError_t launch_gemm_nt_acc64(const GemmNT *p, int n, int64_t R, double alpha, double *part, hipStream_t st) {
    if (R <= 0 || n <= 0) return hipSuccess;
    // (both products have the same rows x cols, perhaps transposed)
    if (n > 2 || (n == 2 && (int64_t)p[0].rows * p[0].cols != (int64_t)p[1].rows * p[1].cols))
        return hipErrorInvalidValue;
    const int z = gemm_nt_zsplit(p[0].rows, p[0].cols, n);
    const int64_t kper = ((R + 4 * z - 1) / (4 * z) + 3) / 4 * 4;
    Products pr{};
    bool vec = true;
    int items = 0;
    for (int i = 0; i < n; ++i) {
        pr.X[i] = p[i].X;
        pr.Y[i] = p[i].Y;
        pr.rows[i] = p[i].rows;
        pr.cols[i] = p[i].cols;
        if (tiles_of(p[i].rows, p[i].cols) != tiles_of(p[0].rows, p[0].cols)) return hipErrorInvalidValue;
        items += z * tiles_of(p[i].rows, p[i].cols);
        vec = vec && p[i].rows % 4 == 0 && p[i].cols % 4 == 0;
    }
    pr.n0 = items / n;
    const dim3 grid((items + 7) / 8 * 8);
    if (vec)
        hipLaunchKernelGGL(gemm_nt_mfma_kernel<true>, grid, dim3(256), kGemmLds, st, pr, items, R, kper, part);
    else
        hipLaunchKernelGGL(gemm_nt_mfma_kernel<false>, grid, dim3(256), kGemmLds, st, pr, items, R, kper, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nd = (int64_t)p[0].rows * p[0].cols;
    hipLaunchKernelGGL(reduce_parts_kernel, dim3(grid_for(nd, 4096), n), dim3(256), 0, st, part, z, nd, alpha, p[0].dA,
                       n > 1 ? p[1].dA : nullptr);
    return hipGetLastError();
}

hipError_t gemm_nt_configure() {
    const hipError_t e = hipFuncSetAttribute((const void *)gemm_nt_mfma_kernel<true>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGemmLds);
    return e != hipSuccess ? e : hipFuncSetAttribute((const void *)gemm_nt_mfma_kernel<false>,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)kGemmLds);
}

hipError_t launch_probe_trace(const float *vtr, const float *c, int kv, int M, int64_t len, double *ytr,
                              hipStream_t st) {
    const int64_t nval = len * M;
    if (nval <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((nval + 3) / 4, 16384);
    hipLaunchKernelGGL(probe_trace_kernel, dim3((unsigned)blocks), dim3(256), 0, st, vtr, c, kv, M, len, ytr);
    return hipGetLastError();
}

hipError_t launch_f64_to_f32(const double *src, float *dst, int64_t n, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(f64_to_f32_kernel, dim3(grid_for(n, 4096)), dim3(256), 0, st, src, dst, n);
    return hipGetLastError();
}

hipError_t launch_pack_f32_from_f32(const float *A, int rows, int cols, bool transpose, int prow,
                                    int pcol, float *pk, hipStream_t st) {
    const int64_t total = (int64_t)prow * pcol;
    hipLaunchKernelGGL(pack_from_f32_kernel, dim3(grid_for(total, 8192)), dim3(256), 0, st, A, rows,
                       cols, transpose ? 1 : 0, prow, pcol, pk);
    return hipGetLastError();
}

}  // namespace rom
