// What the FP32-state row-split kernels (k_rank2_split.hip: BF16 / FP8
// operators, k_rank2_split_f32.hip: FP32 operators) share: launch arguments,
// group placement and the per-step source windows.
#pragma once

#include "k_common.h"
#include "k_exchange.h"
#include "k_lane.h"
#include "rom_internal.h"

namespace rom {
namespace split {

typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
using dev::f4;
using xch::u64;

constexpr int kRows = 64;          // rows per workgroup tile
constexpr int kCols = 64;          // sample columns of the widest group
constexpr int kWaves = 4;
constexpr int kThreads = 256;
constexpr int kXcds = 8, kCusPerXcd = 32;

struct SplitArgs {
    const u4 *opv, *ops;        // packed fragments of Avs and Asv
    const float *b, *c;         // source (kv), probe (kv) or null
    const double *mu;
    float *V, *S;               // caller states, ld kv / ks
    double *J, *y;
    float *x;                   // exchange ring: xch::kRing buffers of xfloats words
    size_t xfloats;
    u64 *yp;                    // probe partials [group][xch::kRing][row tile][col]
    unsigned *flags;            // published phases [group][32 row tiles][wave]
    unsigned *slots;            // per-XCD slot counters (8)
    unsigned *done;             // repeatable runs: two words per group for its end (k_exchange.h); else null
    int *status;                // status[1] <- ROM_E_TIMEOUT, status[2] abort
    float *vtr, *str;           // FP32 traced runs: state traces (entry e, sample m, row: [e][m][row])
    const double *ytr;          // adjoint runs: forward probe trace [step][m]
    float *wtr, *qtr;           // adjoint runs: P after / Q before each step's P update
    double *dmu;                // adjoint runs: += dt (b^T P) du/dmu
    const SplitGroup *grp;      // grouped FP32 runs: per-group instance data, from grp[g0]
    const int *smap;            // grouped FP32 runs: slot map (see rank2_split_f32_kernel)
    int g0;
    int source;                 // source signal (dev::Source)
    long spin_max;              // poll budget of one wait
    int forced;                 // host-forced time-outs
    int kv, kp, M, G, R;
    int64_t n0, nsteps;
    double dt;
    float scale;
};

// This workgroup's slot code (xcd + 8 * slot on that XCD), from the launch's
// per-XCD slot counters.
__device__ __forceinline__ int take_slot(unsigned *slots) {
    __shared__ int sh_slot;
    if (threadIdx.x == 0) {
        const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 7u;   // HW_REG_XCC_ID
        const unsigned s = __hip_atomic_fetch_add(&slots[xcc], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_slot = (int)(xcc + 8u * s);
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(sh_slot);
}

// Forcing of a window of kUWin steps for the group's NC columns, in LDS:
// u[s][j] = u(t_{n + s}; mu of column col0 + j) (zero past M), evaluated by
// all threads together once per window, so each step reads its column's
// value instead of evaluating the source (whose exp constants would
// otherwise be held, and spilled, across the time loop).
constexpr int kUWin = 16;
template <int NC>
__device__ __forceinline__ void forcing_window(double *u, int src, int64_t n, double dt, const double *mu, int col0,
                                               int M) {
    for (int idx = threadIdx.x; idx < kUWin * NC; idx += kThreads) {
        const int s = idx / NC, j = idx - s * NC, m = col0 + j;
        u[idx] = m < M ? dev::forcing(src, (double)(n + s) * dt, mu[m]) : 0.0;
    }
}

// Adjoint amplitude window: u[s][j] = 2 y(step r0 - s, column col0 + j)
// for the kUWin iterations from r0 down (zero before the segment or past M):
// the reverse sweep's source amplitude, from the forward probe trace.
template <int NC>
__device__ __forceinline__ void adjoint_window(double *u, const double *ytr, int64_t r0, int col0, int M) {
    for (int idx = threadIdx.x; idx < kUWin * NC; idx += kThreads) {
        const int s = idx / NC, j = idx - s * NC, m = col0 + j;
        const int64_t r = r0 - s;
        u[idx] = (m < M && r >= 0) ? 2.0 * ytr[(size_t)r * M + m] : 0.0;
    }
}

// FP64 sum over the TPC (4, 8 or 16) consecutive lanes of a column, in each of them, as a binary tree over the
// lane's bits from the lowest up (once the lanes below agree, row_half_mirror
// and row_ror:8 are the partners p ^ 4 and p ^ 8), leaving out the first FROM
// bits.
template <int TPC, int FROM = 0>
__device__ __forceinline__ double column_sum(double y) {
    if constexpr (FROM < 1) y += lane::dpp_mov64<lane::kDppXor1>(y);
    if constexpr (FROM < 2) y += lane::dpp_mov64<lane::kDppXor2>(y);
    if constexpr (TPC >= 8 && FROM < 3) y += lane::dpp_mov64<lane::kDppHalfMirror>(y);
    if constexpr (TPC == 16 && FROM < 4) y += lane::dpp_mov64<lane::kDppRor8>(y);
    return y;
}

// Exchanged data, read with device-scope buffer loads (the vector L1 does
// not serve them from lines it kept from an earlier read).  The base is
// wave-uniform; offsets are in bytes, and one past the block reads zeros
// (the buffer's bound) instead of faulting.
constexpr int kDeviceScope = 16;             // cache-policy bit SC1
constexpr int kRawBufferWord3 = 0x00020000;  // untyped 32-bit data format
__device__ __forceinline__ __amdgpu_buffer_rsrc_t raw_buffer(const void *base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes, kRawBufferWord3);
}

// A 64-bit value that is the same in every lane, moved to scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Sum of one column's R <= 32 row-tile probe partials, p[q * stride], missing
// ones zero: SEQ = 0: a binary tree over q from its lowest bit up; SEQ > 0:
// such a tree over each SEQ neighbours (a power of two up to 4), and up to
// four of those sums in sequence (more: the tree).  The
// column's TPC consecutive threads take the partials q = fs, fs + TPC, ..;
// every one of them gets the total.  The partials of a step are loaded (load)
// ahead of the poll for the rows of the next half-step, so that they cost
// row tile 0 no trip of their own, and completed (wait) behind it.  All lanes
// of the wave must call each.
// NN: partials per thread (at least R / TPC).
template <int TPC, int SEQ = 0, int NN = 32 / TPC>
struct ProbeSum {
    static constexpr int N = NN;
    u64 v[N];
    __device__ __forceinline__ void load(const u64 *p, int stride, int R, int fs) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = xch::get64(p + (size_t)min(fs + i * TPC, R - 1) * stride);
    }
    __device__ __forceinline__ double sum(xch::Wait &wait, const u64 *p, int stride, int R, int fs) {
        long spins = 0;
        for (;;) {
            unsigned m = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) m = xch::max3u(m, m, (unsigned)(v[i] >> 32));
            if (wait.dead || __ballot(m == xch::kEmpty) == 0) break;
            if (wait.give_up(spins)) break;
            load(p, stride, R, fs);
        }
        double y[N];
#pragma unroll
        for (int i = 0; i < N; ++i)
            y[i] = fs + i * TPC < R ? __builtin_bit_cast(double, v[i]) : 0.0;
        if (SEQ > 0 && R <= 4 * SEQ) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = q * SEQ / TPC, l = q * SEQ % TPC;
                double x = y[i];
                if constexpr (SEQ >= 2) x += lane::dpp_mov64<lane::kDppXor1>(x);
                if constexpr (SEQ >= 4) x += lane::dpp_mov64<lane::kDppXor2>(x);
                t += __shfl(x, l, TPC);
            }
            return t;
        }
#pragma unroll
        for (int i = 0; i < N; ++i) y[i] = column_sum<TPC>(y[i]);
#pragma unroll
        for (int h = 1; h < N; h <<= 1)
#pragma unroll
            for (int i = 0; i + h < N; i += 2 * h) y[i] += y[i + h];
        return y[0];
    }
};

}  // namespace split

// Host side, shared by the launchers.
// Carve a workspace of rank2_split_ws_bytes(xfloats, ypd) into a's exchange
// ring, probe partials, flags and slot counters, and enqueue their clearing
// (empty partials and, for kernels that poll the rows themselves, exchange
// slots; zero flags, counters and abort word).
hipError_t split_workspace(split::SplitArgs &a, void *ws, size_t xfloats, size_t ypd, bool poll_rows, hipStream_t st);
void fill_split_args(split::SplitArgs &a, const void *opv, const void *ops, const Rank2Args &r2, float scale,
                     int *status);
// Width index (group width 16 << wi columns) of the narrowest group whose
// ceil(M / width) groups fit in one launch; the caller's check that the
// 64-column groups fit guarantees that one does.
int split_width_index(int M, int kvp);

}  // namespace rom
