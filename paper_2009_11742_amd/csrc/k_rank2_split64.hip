// Rank-2 leapfrog stepper with FP64 states, row-split schedule: operators
// between the FP64 resident kernel's sizes and the panel schedule's
// (128 < max(Kv_pad, Ks_pad) <= 512, or smaller pairs the resident kernel
// cannot hold).
//
// Method: Sec. 2.4 eq. (2.5) for the staggered system of Sec. 3.1 eq. (3.3),
//     V <- V + dt (Avs S + b u(t_n; mu))      then      S <- S + dt Asv V,
// with the probe QoI J += dt (c^T V)^2 on the new V of each step.
//
// Why this schedule.  At these sizes the operators (0.5 to 4 MB) fit neither
// one CU's registers nor its LDS, and a vector-ALU column block streams them
// through every CU each step (K = 300: 80 us per step).  Here a group of
// NC = 16 samples (the width of the FP64 matrix instruction) is stepped by R
// workgroups of one XCD, each of which keeps RT rows of both operators
// in registers for the whole run and moves only its 16 x RT new state
// entries per half-step, through the XCD's L2 (k_exchange.h: one store and
// one load of latency, no barrier).  Both operators are zero padded to
// KP x KP, KP = max(Kv_pad, Ks_pad), so Kv and Ks need not be equal.
//
// RT = 16 where the R = KP / 16 workgroups of every group then fit on the
// chip, else 32: the matrix-core time of a half-step is proportional to RT
// (KP RT 16 multiply-adds at one CU's 64 per clock), the exchange is not.
// More groups than fit are taken in rounds: a group slot steps one group of
// samples through the whole run, then the next.
//
// Products: v_mfma_f64_16x16x4f64 (A lane l: row l % 16, term l / 16; B lane
// l: term l / 16, column l % 16; D entry v of lane l: row l / 16 + 4 v,
// column l % 16).  Wave w sums the terms [w KP/4, (w+1) KP/4); terms come in
// groups of 8, lane l holding terms 2 (l / 16) and 2 (l / 16) + 1 of the
// group for two consecutive instructions, each in a chain of its own.  The four
// partials meet in LDS and one thread per RT / 16 rows of a column (one of each
// 16-row tile) adds them in a fixed order and updates its state entries, which
// live in its registers.  The probe is summed per 16-row tile, then over those.
// So a sample's bits do not depend on RT, hence not on its company.
//
// Bound: latency.  Per half-step the matrix time is 0.5 (RT = 16) or 1.1 us
// (RT = 32) at KP = 320; the exchange (store to L2, poll, load), about
// 0.8 us, and the LDS meeting of the waves are the rest.  Measured (us per
// step, this schedule / the vector-ALU column blocks): (300, 280) M = 128
// 3.6 / 80; (128, 128) non-skew M = 3 2.0 / 14.5; (192, 192) M = 700 7.3
// (two rounds); (320, 320) M = 900 14.7 (three rounds).  The probe costs
// nothing measurable: its sum runs while row tile 0 would wait for the next
// rows (read before the stress half-step, it took 0.8 us of the step).
#include "k_common.h"
#include "k_exchange.h"
#include "k_lane.h"
#include "rom_internal.h"

namespace rom {
namespace {

using xch::u64;

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int kT = 256, kW = 4, kNC = 16;
constexpr int kWin = 16;           // steps of forcing evaluated at a time
constexpr int kXcd = 8, kCuXcd = 32;
// one workgroup per CU, so that each XCD takes 32 of the 256
constexpr size_t kLds64 = 96 * 1024;

struct Args64 {
    const d2 *opv, *ops;        // packed fragments (see pack64_kernel)
    const double *b, *c, *mu;
    double *V, *S, *J, *y;
    u64 *x;                     // [slot][kRing][KP kNC] exchange, B-fragment order
    u64 *yp;                    // [slot][kRing][KP / 16][kNC] probe partials
    unsigned *slots;            // per-XCD slot counters
    unsigned *done;             // [slot] two words for the end of its rounds (k_exchange.h)
    int *status;
    long spin_max;
    int forced;
    int kv, ks, M, G, cap, R, source;
    int64_t n0, nsteps;
    double dt;
};

constexpr int ld64(int NT) { return 16 * NT + 2; }     // LDS column stride of the partials

// A wave's partials of its NT 16-row tiles, to LDS: the first and the second
// terms of its KG groups in a chain each.
template <int KG, int NT>
__device__ __forceinline__ void partials64(const d2 (&op)[KG][NT], const u64 (&x)[KG][2], int l, double *pw) {
    d4 acc[NT][2];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) acc[t][h] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t][e] = __builtin_amdgcn_mfma_f64_16x16x4f64(op[g][t][e], __builtin_bit_cast(double, x[g][e]),
                                                                 acc[t][e], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            pw[(l & 15) * ld64(NT) + 16 * t + (l >> 4) + 4 * v] = acc[t][0][v] + acc[t][1][v];
}

// The sum of the four waves' partials of one row.
template <int NT>
__device__ __forceinline__ double total64(const double *d) {
    constexpr int W = kNC * ld64(NT);
    return (d[0] + d[W]) + (d[2 * W] + d[3 * W]);
}

// The sum over a column's 16 threads (one 16-lane row).
__device__ __forceinline__ double tile_sum64(double y) {
    y += lane::dpp_mov64<lane::kDppRor8>(y);
    y += lane::dpp_mov64<lane::kDppHalfMirror>(y);
    y += lane::dpp_mov64<lane::kDppXor2>(y);
    y += lane::dpp_mov64<lane::kDppXor1>(y);
    return y;
}

// The sum over the four 16-lane rows.
__device__ __forceinline__ double rows_sum64(double y) { return lane::swap_sum64<true>(lane::swap_sum64<false>(y)); }

template <int KP, int RT>
__global__ __launch_bounds__(kT) __attribute__((amdgpu_waves_per_eu(1, 1)))
void rank2_split64_kernel(Args64 a) {
    constexpr int KG = KP / 32;                // 8-term groups per wave
    constexpr int NT = RT / 16;                // 16-row tiles, rows per finishing thread
    constexpr int NP = KP / 16;                // probe partials
    constexpr int LD = ld64(NT);
    __shared__ double part[2][kW][kNC * LD];
    __shared__ double uwin[kWin * kNC];
    __shared__ int sh_code;

    const int tid = threadIdx.x, l = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (tid == 0) {
        const unsigned xcc = __builtin_amdgcn_s_getreg((3 << 11) | (0 << 6) | 20) & 7u;   // HW_REG_XCC_ID
        const unsigned s = __hip_atomic_fetch_add(&a.slots[xcc], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        sh_code = (int)(xcc + 8u * s);
    }
    __syncthreads();
    const int code = __builtin_amdgcn_readfirstlane(sh_code);
    const int xcc = code & 7, s = code >> 3;
    const int R = a.R;
    const int r = s % R, slot = (s / R) * kXcd + xcc;
    if (slot >= a.cap) return;                 // idle workgroup

    xch::Wait wait{a.status, a.spin_max, a.forced, false};
    u64 *const xg = a.x + (size_t)slot * xch::kRing * KP * kNC;
    u64 *const yg = a.yp + (size_t)slot * xch::kRing * NP * kNC;

    // operator fragments of this wave's terms, registers for the whole run
    d2 ov[KG][NT], os[KG][NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int g = 0; g < KG; ++g) {
            const size_t i = ((size_t)((r * NT + t) * kW + w) * KG + g) * 64 + l;
            ov[g][t] = a.opv[i];
            os[g][t] = a.ops[i];
        }

    // finishing thread: column fj, rows fs, 16 + fs, .. of the tile
    const int fj = tid >> 4, fs = tid & 15;
    const int fr = r * RT + fs;
    double bb[NT], cc[NT];
#pragma unroll
    for (int e = 0; e < NT; ++e) {
        bb[e] = fr + 16 * e < a.kv ? a.b[fr + 16 * e] : 0.0;
        cc[e] = (a.c != nullptr && fr + 16 * e < a.kv) ? a.c[fr + 16 * e] : 0.0;
    }
    const bool probe = a.c != nullptr;
    // this thread's slots in an exchange buffer: row fr of column fj, and the
    // rows 16 on, kTileStep words further
    const size_t xo = (size_t)((fr >> 3) * 64 + 16 * ((fr & 7) >> 1) + fj) * 2 + (fr & 1);
    constexpr int kTileStep = 2 * 128;

    int64_t q = 0, ny = 0;                     // phase, probe row to publish next
    auto publish = [&](const double (&v)[NT]) {
        u64 *d = xg + (size_t)(q & 3) * KP * kNC + xo;
#pragma unroll
        for (int e = 0; e < NT; ++e) xch::put64(d + e * kTileStep, v[e]);
        u64 *z = xg + (size_t)((q + 2) & 3) * KP * kNC + xo;   // phase q - 2
#pragma unroll
        for (int e = 0; e < NT; ++e) xch::clear64(z + e * kTileStep);
        ++q;
    };
    // Probe partials, one per 16-row tile, have a ring of their own, one entry
    // per step: row tile 0 reads entry k before it publishes the velocity of
    // step k + 1, so whoever publishes that of step k + 2 may empty it.
    auto publish_y = [&](const double (&y)[NT]) {
        if (fs == 0) {
#pragma unroll
            for (int e = 0; e < NT; ++e) {
                xch::put64(yg + ((size_t)(ny & 3) * NP + NT * r + e) * kNC + fj, y[e]);
                xch::clear64(yg + ((size_t)((ny + 2) & 3) * NP + NT * r + e) * kNC + fj);
            }
        }
        ++ny;
    };

    // products of the field's rows with phase q - 1's states, partials to LDS
    auto products = [&](const d2 (&op)[KG][NT], double *pw) {
        const u64 *src = xg + (size_t)((q - 1) & 3) * KP * kNC + ((size_t)(w * KG) * 64 + l) * 2;
        u64 x[KG][2];
        long spins = 0;
        for (;;) {
            unsigned m = 0;
#pragma unroll
            for (int g = 0; g < KG; ++g) {
                x[g][0] = xch::get64(src + (size_t)g * 128);
                x[g][1] = xch::get64(src + (size_t)g * 128 + 1);
            }
#pragma unroll
            for (int g = 0; g < KG; ++g) m = xch::max3u(m, (unsigned)(x[g][0] >> 32), (unsigned)(x[g][1] >> 32));
            if (wait.dead || (!wait.forced && __ballot(m == xch::kEmpty) == 0)) break;
            if (wait.give_up(spins)) break;
        }
        // (the emptied slots of the last publication: before the next one)
        xch::publish_fence();
        partials64<KG, NT>(op, x, l, pw);
    };
    // sum of the four waves' partials of this thread's row e
    auto total = [&](const double *p, int e) {
        return total64<NT>(p + fj * LD + 16 * e + fs);
    };

    unsigned round = 0;
    for (int g = slot; g < xch::args_here<Args64>().G; g += xch::args_here<Args64>().cap) {
        const int col0 = g * kNC, fm = col0 + fj;
        const bool fok = fm < xch::args_here<Args64>().M;
        double sv[NT], ss[NT];
        const auto &in = xch::args_here<Args64>();       // (held, they cost 0.15 us per step)
#pragma unroll
        for (int e = 0; e < NT; ++e) {
            sv[e] = (fok && fr + 16 * e < in.kv) ? in.V[(size_t)fm * in.kv + fr + 16 * e] : 0.0;
            ss[e] = (fok && fr + 16 * e < in.ks) ? in.S[(size_t)fm * in.ks + fr + 16 * e] : 0.0;
        }
        xch::publish_fence();
        publish(ss);
        double Jacc = 0.0;
        for (int64_t k = 0; k < a.nsteps; ++k) {
            if (k % kWin == 0) {
                // read in the velocity update below, after its barrier; the
                // last reads of the previous window lie before the stress
                // update's barrier
                const int st = tid >> 4, j = tid & 15;
                uwin[tid] = col0 + j < a.M
                                ? dev::forcing(a.source, (double)(a.n0 + k + st) * a.dt, a.mu[col0 + j]) : 0.0;
            }
            // ---- velocity half-step
            products(ov, &part[0][w][0]);
            __syncthreads();
            const double u = uwin[(int)(k % kWin) * kNC + fj];
            double yt[NT];
#pragma unroll
            for (int e = 0; e < NT; ++e) {
                const double inc = fma(bb[e], u, total(&part[0][0][0], e));
                sv[e] = fr + 16 * e < a.kv ? fma(a.dt, inc, sv[e]) : 0.0;
                yt[e] = cc[e] * sv[e];
            }
            if (probe) {
#pragma unroll
                for (int e = 0; e < NT; ++e) yt[e] = tile_sum64(yt[e]);
            }
            publish(sv);
            if (probe) publish_y(yt);
            // ---- stress half-step
            products(os, &part[1][w][0]);
            __syncthreads();
#pragma unroll
            for (int e = 0; e < NT; ++e)
                ss[e] = fr + 16 * e < a.ks ? fma(a.dt, total(&part[1][0][0], e), ss[e]) : 0.0;
            // the last stress field is not read; a further group's first
            // publication takes its phase
            if (k + 1 < a.nsteps) {
                publish(ss);
            }
            // ---- probe: row tile 0 sums the group's partials of this step,
            // in the time it would wait for the stress rows
            if (probe && r == 0 && w == 0) {
                static_assert(NP % 4 == 0, "four quarters of the wave");
                const u64 *p = yg + ((size_t)((ny - 1) & 3) * NP + (l >> 4)) * kNC + (l & 15);
                u64 v[NP / 4];
                long spins = 0;
                for (;;) {
                    unsigned m = 0;
#pragma unroll
                    for (int i = 0; i < NP / 4; ++i) v[i] = xch::get64(p + (size_t)4 * i * kNC);
#pragma unroll
                    for (int i = 0; i < NP / 4; ++i) m = xch::max3u(m, m, (unsigned)(v[i] >> 32));
                    if (wait.dead || __ballot(m == xch::kEmpty) == 0) break;
                    if (wait.give_up(spins)) break;
                }
                double y = 0.0;
#pragma unroll
                for (int i = 0; i < NP / 4; ++i) y += __builtin_bit_cast(double, v[i]);
                y = rows_sum64(y);
                Jacc = fma(a.dt, y * y, Jacc);
                if (a.y && l < kNC && col0 + l < a.M) a.y[(size_t)k * a.M + col0 + l] = y;
            }
        }
        const auto &out = xch::args_here<Args64>();
        if (!xch::agree(out.done + 2 * slot, out.R, round++, wait)) return;
#pragma unroll
        for (int e = 0; e < NT; ++e) {
            if (fok && fr + 16 * e < out.kv) out.V[(size_t)fm * out.kv + fr + 16 * e] = sv[e];
            if (fok && fr + 16 * e < out.ks) out.S[(size_t)fm * out.ks + fr + 16 * e] = ss[e];
        }
        if (probe && out.J && r == 0 && w == 0 && l < kNC && col0 + l < out.M) out.J[col0 + l] += Jacc;
    }
}

// Runs of a few steps: a launch per half-step, which needs no exchange, no
// cleared slots and no launch that may repeat it, with the sums of the kernel
// above, so that a run cut into single steps gives the same bits.  Workgroup
// R g + r: rows 16 r .. of the field for group g, the other field's terms read
// from the caller's states.  Bound by its launches, 5 us a step at the small
// sizes.  Measured, us per call of one step, vector-ALU blocks / row-split
// kernel / here: (128, 128), M = 3 18 / 21 / 12, (192, 192), M = 500 32 / 27 / 13,
// (300, 280), M = 128 86 / 27 / 12.
struct Half64 {
    const d2 *op;
    const double *x;            // the other field's states, n entries a column
    double *f;                  // this field's, rows entries a column
    const double *b, *c, *mu;   // velocity half-step: source, probe (or null); b null in the other
    double *yp;                 // probe partials [group][16-row tile][kNC]
    int n, rows, M, source;
    double t, dt;
};

template <int KP>
__global__ __launch_bounds__(kT) void rank2_half64_kernel(Half64 a) {
    constexpr int KG = KP / 32, R = KP / 16;
    __shared__ double part[kW][kNC * ld64(1)];
    const int tid = threadIdx.x, l = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = blockIdx.x % R, g = blockIdx.x / R, col0 = g * kNC;
    d2 op[KG][1];
    u64 x[KG][2];
    const int m = col0 + (l & 15);
#pragma unroll
    for (int q = 0; q < KG; ++q) {
        op[q][0] = a.op[((size_t)(r * kW + w) * KG + q) * 64 + l];
        const int k = w * (KP / 4) + 8 * q + 2 * (l >> 4);
#pragma unroll
        for (int e = 0; e < 2; ++e)
            x[q][e] = __builtin_bit_cast(u64, m < a.M && k + e < a.n ? a.x[(size_t)m * a.n + k + e] : 0.0);
    }
    partials64<KG, 1>(op, x, l, part[w]);
    __syncthreads();
    const int fj = tid >> 4, fs = tid & 15, row = 16 * r + fs, fm = col0 + fj;
    const bool ok = fm < a.M && row < a.rows;
    double inc = total64<1>(&part[0][fj * ld64(1) + fs]), v = ok ? a.f[(size_t)fm * a.rows + row] : 0.0;
    if (a.b)
        inc = fma(row < a.rows ? a.b[row] : 0.0, fm < a.M ? dev::forcing(a.source, a.t, a.mu[fm]) : 0.0, inc);
    v = row < a.rows ? fma(a.dt, inc, v) : 0.0;
    if (ok) a.f[(size_t)fm * a.rows + row] = v;
    if (a.c) {
        const double y = tile_sum64((row < a.rows ? a.c[row] : 0.0) * v);
        if (fs == 0) a.yp[((size_t)g * R + r) * kNC + fj] = y;
    }
}

// The probe of such a run, a wave per group: yp [step][group][R][kNC].
__global__ __launch_bounds__(64) void rank2_half64_probe_kernel(const double *yp, int nsteps, int R, int M, double dt,
                                                                double *J, double *y) {
    const int l = threadIdx.x, g = blockIdx.x, m = g * kNC + l;
    double Jacc = 0.0;
    for (int k = 0; k < nsteps; ++k) {
        const double *p = yp + (((size_t)k * gridDim.x + g) * R + (l >> 4)) * kNC + (l & 15);
        double v = 0.0;
        for (int i = 0; i < R / 4; ++i) v += p[(size_t)4 * i * kNC];
        v = rows_sum64(v);
        Jacc = fma(dt, v * v, Jacc);
        if (y && l < kNC && m < M) y[(size_t)k * M + m] = v;
    }
    if (J && l < kNC && m < M) J[m] += Jacc;
}

// Fragments of a column-major rows x cols operator zero padded to KP x KP:
// dst[16-row tile][wave][8-term group][lane] = terms 2 (lane / 16), + 1 of
// the group, row lane % 16 of the tile.
__global__ void pack64_kernel(const double *__restrict__ A, int rows, int cols, int KP, d2 *__restrict__ dst) {
    const int KG = KP / 32;
    const int n = KP / 16 * kW * KG * 64;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
        const int l = i & 63;
        int t = i >> 6;
        const int g = t % KG;
        t /= KG;
        const int w = t % kW;
        t /= kW;
        const int row = 16 * t + (l & 15), k = w * (KP / 4) + 8 * g + 2 * (l >> 4);
        d2 v = {0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 2; ++e)
            if (row < rows && k + e < cols) v[e] = A[row + (size_t)(k + e) * rows];
        dst[i] = v;
    }
}

// Behind the probe partials: 8 slot counters, 8 words of status, the slots'
// words.
constexpr int kWords64 = 16 + 2 * kXcd * kCuXcd;

// Empty exchange slots, zero those words and the abort word.
__global__ void clear64_kernel(u64 *x, size_t n, unsigned *slots, int *status) {
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (size_t i = i0; i < n; i += (size_t)gridDim.x * blockDim.x) x[i] = xch::kEmpty64;
    if (i0 < kWords64) slots[i0] = 0u;
    if (i0 == 0) status[2] = 0;
}

struct Kern64 {
    int kp;
    const void *f[2];          // RT = 16, 32
    const void *half;
};
#define ROM_K64(KP)                                                                                     \
    {KP, {(const void *)rank2_split64_kernel<KP, 16>, (const void *)rank2_split64_kernel<KP, 32>},      \
     (const void *)rank2_half64_kernel<KP>}
const Kern64 kKern64[] = {ROM_K64(128), ROM_K64(192), ROM_K64(256), ROM_K64(320),
                          ROM_K64(384), ROM_K64(448), ROM_K64(512)};
#undef ROM_K64

const Kern64 *kern64(int kvp, int ksp) {
    const int kp = kvp > ksp ? kvp : ksp;
    for (const Kern64 &k : kKern64)
        if (k.kp == kp) return &k;
    return nullptr;
}

int slots64(int kp, int RT) { return kXcd * (kCuXcd / (kp / RT)); }

}  // namespace

bool rank2_split64_applies(int kvp, int ksp) { return kern64(kvp, ksp) != nullptr; }

size_t rank2_split64_op_bytes(int kvp, int ksp) {
    const size_t kp = kvp > ksp ? kvp : ksp;
    return kp * kp * sizeof(double);
}

size_t rank2_split64_ws_bytes(int kvp, int ksp) {
    const int kp = kvp > ksp ? kvp : ksp;
    size_t n = 0;
    for (int RT = 16; RT <= 32; RT += 16) {
        const size_t c = slots64(kp, RT);
        const size_t m = c * xch::kRing * kNC * ((size_t)kp + kp / 16);
        if (m > n) n = m;
    }
    return n * sizeof(u64) + kWords64 * sizeof(unsigned);
}

hipError_t launch_split64_pack(const double *A, int rows, int cols, int kvp, int ksp, void *dst, hipStream_t st) {
    const int kp = kvp > ksp ? kvp : ksp;
    hipLaunchKernelGGL(pack64_kernel, dim3(kp * kp / 2 / 256), dim3(256), 0, st, A, rows, cols, kp,
                       static_cast<d2 *>(dst));
    return hipGetLastError();
}

bool rank2_split64_device_ok() {
    for (const Kern64 &k : kKern64)
        for (const void *f : k.f) {
            int nb = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kT, kLds64) != hipSuccess || nb < 1) return false;
        }
    return true;
}

hipError_t rank2_split64_configure() {
    for (const Kern64 &k : kKern64)
        for (const void *f : k.f) {
            hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds64);
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

// opv, ops: launch_split64_pack of Avs and Asv; ws: rank2_split64_ws_bytes.
// The run is repeatable (rep: for the launch behind it); a time-out that was
// forced is recorded in status all the same, so that a test sees it happen.
hipError_t launch_rank2_split64(const void *opv, const void *ops, const Rank2Args &r2, void *ws, int *status,
                                hipStream_t st, Repeat &rep) {
    const Kern64 *k = kern64(r2.kvp, r2.ksp);
    if (!k || r2.M < 1 || r2.nsteps < 1) return hipErrorInvalidValue;
    Args64 a{};
    a.opv = static_cast<const d2 *>(opv);
    a.ops = static_cast<const d2 *>(ops);
    a.b = static_cast<const double *>(r2.b);
    a.c = static_cast<const double *>(r2.c);
    a.mu = r2.mu;
    a.V = static_cast<double *>(r2.V);
    a.S = static_cast<double *>(r2.S);
    a.J = r2.J;
    a.y = r2.y;
    a.spin_max = g_forced_timeout == 1 ? 256 : xch::kSpinMax;
    a.forced = g_forced_timeout == 1 ? 1 : 0;
    a.kv = r2.kv;
    a.ks = r2.ks;
    a.M = r2.M;
    a.G = (r2.M + kNC - 1) / kNC;
    a.source = r2.source;
    a.n0 = r2.n0;
    a.nsteps = r2.nsteps;
    a.dt = r2.dt;
    const int ri = a.G <= slots64(k->kp, 16) ? 0 : 1;      // RT = 16 if all groups then run at once
    const int RT = 16 << ri;
    a.R = k->kp / RT;
    const int cap = slots64(k->kp, RT);
    a.cap = a.G < cap ? a.G : cap;
    a.x = static_cast<u64 *>(ws);
    const size_t nx = (size_t)a.cap * xch::kRing * kNC * k->kp, ny = (size_t)a.cap * xch::kRing * kNC * (k->kp / 16);
    a.yp = a.x + nx;
    a.slots = reinterpret_cast<unsigned *>(a.yp + ny);
    a.status = g_forced_timeout == 1 ? status : reinterpret_cast<int *>(a.slots + 8);
    a.done = a.slots + 16;
    rep = Repeat{a.done, kNC, a.cap};
    hipLaunchKernelGGL(clear64_kernel, dim3(256), dim3(256), 0, st, a.x, nx + ny, a.slots, status);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && g_forced_timeout == 2) e = freeze_odd_groups(a.done, a.cap, st);
    if (e != hipSuccess) return e;
    void *args[] = {&a};
    static_assert(kT == 256 && kXcd * kCuXcd == 256, "launch_waiting");
    return launch_waiting(k->f[ri], args, kLds64, st, false);
}

// Whether a launch per half-step is faster than the exchanging kernel: three
// steps of as many samples as 16-row tiles hold at once ((128, 128), M = 3 21 us
// against 25, (64, 512), M = 33 32 against 38, (300, 280), M = 128 26 against 34;
// four 26, 42, 35 against 27, 43, 38), two of as many as 32-row tiles hold
// ((192, 192), M = 500 25 against 31, three 37 against 34).
bool rank2_split64_short(int kvp, int ksp, int M, int64_t nsteps) {
    const Kern64 *k = kern64(kvp, ksp);
    const int G = (M + kNC - 1) / kNC;
    return k && G <= slots64(k->kp, 32) && nsteps <= (G <= slots64(k->kp, 16) ? 3 : 2);
}

// Such a run; ws (rank2_split64_ws_bytes) only for a probe.
hipError_t launch_rank2_short64(const void *opv, const void *ops, const Rank2Args &r2, void *ws, hipStream_t st) {
    const Kern64 *k = kern64(r2.kvp, r2.ksp);
    if (!rank2_split64_short(r2.kvp, r2.ksp, r2.M, r2.nsteps) || r2.M < 1 || (r2.c && !ws)) return hipErrorInvalidValue;
    const int R = k->kp / 16, G = (r2.M + kNC - 1) / kNC;
    Half64 v{}, s{};
    v.op = static_cast<const d2 *>(opv);
    s.op = static_cast<const d2 *>(ops);
    v.f = static_cast<double *>(r2.V);
    s.f = static_cast<double *>(r2.S);
    v.x = s.f;
    s.x = v.f;
    v.rows = s.n = r2.kv;
    v.n = s.rows = r2.ks;
    v.b = static_cast<const double *>(r2.b);
    v.c = static_cast<const double *>(r2.c);
    v.mu = r2.mu;
    v.M = s.M = r2.M;
    v.dt = s.dt = r2.dt;
    v.source = r2.source;
    for (int64_t i = 0; i < r2.nsteps; ++i) {
        v.t = (double)(r2.n0 + i) * r2.dt;
        v.yp = static_cast<double *>(ws) + (size_t)i * G * R * kNC;
        for (Half64 *h : {&v, &s}) {
            void *args[] = {h};
            const hipError_t e = hipLaunchKernel(k->half, dim3(R * G), dim3(kT), args, 0, st);
            if (e != hipSuccess) return e;
        }
    }
    if (r2.c && (r2.J || r2.y))
        hipLaunchKernelGGL(rank2_half64_probe_kernel, dim3(G), dim3(64), 0, st, static_cast<const double *>(ws),
                           (int)r2.nsteps, R, r2.M, r2.dt, r2.J, r2.y);
    return hipGetLastError();
}

}  // namespace rom
