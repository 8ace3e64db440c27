// Rank-2 leapfrog stepper, row-split schedule: low-precision (BF16 /
// FP8-E4M3) operators, FP32 states.
//
// Method: Sec. 2.4 eq. (2.5) for the staggered system of Sec. 3.1 eq. (3.3),
// one step being  V <- V + dt (Avs S + b u(t_n; mu)^T),  S <- S + dt Asv V.
//
// Why a second schedule.  The column-block kernels give every workgroup a
// few sample columns and the whole operator, so each CU streams the full
// operator every step; with BF16 / FP8 operators at K = 1024 that stream
// (4 MB / 2 MB per step per CU) bounds the step far above the MFMA time.
// Here the operator rows are split instead: the workgroups of a column
// group (kRows = 64 rows each, R = K / 64 of them) cover K rows of both
// fields for a group of samples: 16, 32 or 64 columns (the narrowest whose
// workgroups all fit on the chip; kCols = 64 sizes the buffers).  Each keeps
// its operator rows in
// registers for the whole run (every wave holds a quarter of the reduction
// of both fields as BF16 MFMA fragments: 256 registers per lane at K =
// 1024), so no operator bytes move after the start.  The price is one
// exchange per half-step: a workgroup publishes its updated rows, as the
// BF16 (hi, lo) pair the products consume, and the others poll for them or
// wait for per-wave flags (k_exchange.h) before the other half-step.
//
// The exchange stays inside one XCD: a workgroup reads the XCD it runs on
// (HW_REG_XCC_ID) and takes a group slot on that XCD with an atomic, so a
// group's members share an L2 and the exchange needs no L2 write-back or
// invalidate: device-scope loads and stores meet there.  The
// launch is cooperative (all workgroups resident; one per CU); every wait
// is bounded, and a wait that runs out sets ROM_E_TIMEOUT in the status
// word and makes every later wait return at once, so the kernel always ends.
//
// Products: v_mfma_f32_16x16x32_bf16 (A lane l: row l % 16, terms
// 8 (l / 16) .. +7; B lane l: terms 8 (l / 16) .. +7, column l % 16;
// D register r of lane l: row 4 (l / 16) + r, column l % 16).  Wave w of a
// workgroup sums reduction terms [w kp/4, (w+1) kp/4) for all 64 x 64
// outputs, with the state operand fed as x_hi + x_lo (two MFMAs; x_hi alone,
// one MFMA, in the single-pass variant, which also publishes x_hi only); the four
// FP32 partials meet in LDS, where each thread finishes 16 outputs: their
// FP32 sum, then in FP64 the scale (FP8), forcing and the update of the
// FP32 (hi, lo) state.
//
// Bound by the exchange (about 0.8 us from one workgroup's store to the
// others' read, twice a step), then by the loads of the wide groups.  With
// the group barrier and invalidated caches that polled rows and flags
// replaced, K = 512, M = 256 took 3.6 us per step (now 2.7), K = 1024, M =
// 500 6.8 (now 6.3).
#include <mutex>
#include <string>
#include <type_traits>

#include "k_split.h"

namespace rom {
namespace {

using namespace split;

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2 __attribute__((ext_vector_type(2)));

constexpr int kLd = kRows + 4;     // LDS column stride (floats)

__device__ __forceinline__ bf8 as_bf8(u4 v) { return __builtin_bit_cast(bf8, v); }

// Products of one half-step for wave w: acc[rb][cb] (rows 16 rb.., columns
// 16 cb..) = sum over this wave's KB k-blocks of op fragments x (x_hi + x_lo).
// x points at the group's exchange block of the other field.  The B
// fragments of k-block kb are loaded kDepth k-blocks ahead into a register
// ring; the loop is fully unrolled (static fragment indices) and
// sched_barriers keep every load batch ahead of the MFMAs it must precede,
// which the scheduler would otherwise sink next to their use under this
// kernel's register pressure.
constexpr int kDepth = 2;

// Exchange layout: per group of NCB 16-column blocks, [k-block (kp/32)]
// [column block (NCB)][hi | lo][lane (64)][8 terms], lane = 16 ((k % 32) / 8)
// + column % 16 -- exactly the B fragments, so one wave load reads 1 KB
// contiguous.  Offset (in BF16 elements) of fragment (kb, cb, hl) within a
// group's block:
template <int NCB>
__device__ __forceinline__ size_t frag_offset(int kb, int cb, int hl) {
    return ((size_t)(kb * NCB + cb) * 2 + hl) * 512;
}

template <bool SINGLE, int NCB>
__device__ __forceinline__ void load_b(const __amdgpu_buffer_rsrc_t &xg, int kb, unsigned loff, u4 (&bh)[NCB], u4 (&bl)[NCB]) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
        bh[cb] = __builtin_amdgcn_raw_buffer_load_b128(xg, loff, 2 * (int)frag_offset<NCB>(kb, cb, 0), kDeviceScope);
        if constexpr (!SINGLE)
            bl[cb] = __builtin_amdgcn_raw_buffer_load_b128(xg, loff, 2 * (int)frag_offset<NCB>(kb, cb, 1), kDeviceScope);
    }
}

// Whether the kernel polls the rows themselves (a wave's fragments all in
// registers at once) or flags (see k_exchange.h).
template <int KB, int NCB>
constexpr bool polled() { return KB * NCB <= 8; }

// Ring depth in k-blocks (measured at K = 1024: the single-operand kernel
// with 64-column groups takes 7.2 us per step at depth 2, 7.5 at 3 and 7.7
// at 4; the pair 10.6 at 2 and 10.7 at 3 or 4), deeper only for the
// narrower pair groups; polled rows are all loaded at once.
template <int KB, bool SINGLE, int NCB>
constexpr int ring_depth() {
    constexpr int d = (SINGLE || NCB == 4) ? kDepth : 3;
    return polled<KB, NCB>() || KB < d ? KB : d;
}

template <int KB, bool SINGLE, int NCB, class F>
__device__ __forceinline__ void products(const u4 (&op)[4][KB], const float *x, unsigned xbytes, int w, int lane,
                                         const unsigned *flag, unsigned phase, xch::Wait &wait, F &&waited,
                                         f4 (&acc)[4][NCB]) {
    constexpr int D = ring_depth<KB, SINGLE, NCB>();
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) acc[rb][cb] = f4{0.f, 0.f, 0.f, 0.f};
    // The fragment addresses are the same every step; without this opaque
    // redefinition of the base the compiler hoists all of them out of the
    // time loop and spills them.
    uint64_t bits = reinterpret_cast<uint64_t>(x);
    asm volatile("" : "+s"(bits));
    const __amdgpu_buffer_rsrc_t xg = raw_buffer(reinterpret_cast<void *>(bits), xbytes);
    // this wave's k-blocks are w KB .. w KB + KB - 1 of the group's block
    const int kb0 = w * KB;
    const unsigned loff = 16u * (unsigned)lane;
    u4 rh[D][NCB], rl[D][NCB];
    if constexpr (polled<KB, NCB>()) {
        long spins = 0;
        for (;;) {
#pragma unroll
            for (int d = 0; d < D; ++d) load_b<SINGLE, NCB>(xg, kb0 + d, loff, rh[d], rl[d]);
            unsigned m = 0;
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) {
                    m = xch::max3u(xch::max3u(m, rh[d][cb][0], rh[d][cb][1]), rh[d][cb][2], rh[d][cb][3]);
                    if constexpr (!SINGLE)
                        m = xch::max3u(xch::max3u(m, rl[d][cb][0], rl[d][cb][1]), rl[d][cb][2], rl[d][cb][3]);
                }
            if (wait.dead || (!wait.forced && __ballot(m == xch::kEmpty) == 0)) break;
            if (wait.give_up(spins)) break;
        }
        // (the emptied slots of the last publication: before the next one)
        xch::publish_fence();
    } else {
        xch::wait_flags(wait, flag, phase);
        waited();
#pragma unroll
        for (int d = 0; d < D; ++d) load_b<SINGLE, NCB>(xg, kb0 + d, loff, rh[d], rl[d]);
    }
    __builtin_amdgcn_sched_barrier(0);
    // Column block by column block: the MFMAs of k-block kb that read a ring
    // slot's column-block fragments are issued, then that column block's
    // fragments of k-block kb + D are loaded into the same registers.  The
    // ring needs no copies of the fragments in use, and each load still has
    // the rest of this k-block and all of the next ahead of its use.
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        const int slot = kb % D;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) {
                const bf8 A = as_bf8(op[rb][kb]);
                acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, as_bf8(rh[slot][cb]), acc[rb][cb], 0, 0, 0);
                if constexpr (!SINGLE)
                    acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, as_bf8(rl[slot][cb]), acc[rb][cb], 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (kb + D < KB) {
                rh[slot][cb] = __builtin_amdgcn_raw_buffer_load_b128(
                    xg, loff, 2 * (int)frag_offset<NCB>(kb0 + kb + D, cb, 0), kDeviceScope);
                if constexpr (!SINGLE)
                    rl[slot][cb] = __builtin_amdgcn_raw_buffer_load_b128(
                        xg, loff, 2 * (int)frag_offset<NCB>(kb0 + kb + D, cb, 1), kDeviceScope);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// NCB: 16-column blocks per group (NC = 16 NCB samples).  Finishing
// threads: TPC = 256 / NC per column, each owning RPT = 4 NCB consecutive rows
// of the tile, published in runs of 8 rows (one lane's B fragment) or 4 (half
// of one).
template <int KB, bool SINGLE, int NCB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void rank2_split_kernel(SplitArgs a) {
    static_assert(NCB == 1 || NCB == 2 || NCB == 4, "16, 32 or 64 columns per group");
    constexpr int NC = 16 * NCB, TPC = kThreads / NC, RPT = 4 * NCB;
    extern __shared__ __align__(16) unsigned char smem[];
    float *sth = reinterpret_cast<float *>(smem);          // [field][col][kLd] hi
    float *stl = sth + 2 * NC * kLd;                     // lo
    float *part = stl + 2 * NC * kLd;                    // [wave][col][kLd]
    float *bl = part + kWaves * NC * kLd;                // own rows of b
    float *cl = bl + kRows;                                 // own rows of c
    __shared__ double uwin[kUWin * NC];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kp = a.kp, R = a.R;

    // ---- group slot on this workgroup's XCD
    const int code = take_slot(a.slots);
    const int xcc = code & 7, s = code >> 3;
    const int r = s % R;                       // row tile
    const int g = (s / R) * 8 + xcc;           // group, interleaved over the XCDs
    if (g >= a.G) return;                      // idle workgroup
    const int col0 = g * NC;
    xch::Wait wait{a.status, a.spin_max, a.forced, false};

    // ---- operator fragments (registers for the whole run)
    u4 opv[4][KB], ops[4][KB];
    {
        const u4 *pv = a.opv + ((size_t)(r * kWaves + w) * 4 * KB) * 64 + lane;
        const u4 *ps = a.ops + ((size_t)(r * kWaves + w) * 4 * KB) * 64 + lane;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                opv[rb][kb] = pv[(rb * KB + kb) * 64];
                ops[rb][kb] = ps[(rb * KB + kb) * 64];
            }
    }

    // ---- own tiles of V and S, b, c
    const int row0 = r * kRows;
    for (int idx = tid; idx < 2 * NC * kRows; idx += kThreads) {
        const int f = idx / (NC * kRows), rem = idx - f * NC * kRows;
        const int j = rem / kRows, i = rem - j * kRows;
        const int m = col0 + j, row = row0 + i;
        const float *src = f == 0 ? a.V : a.S;
        float v = 0.f;
        if (m < a.M && row < a.kv) v = src[(size_t)m * a.kv + row];
        sth[(f * NC + j) * kLd + i] = v;
        stl[(f * NC + j) * kLd + i] = 0.f;
    }
    for (int i = tid; i < kRows; i += kThreads) {
        const int row = row0 + i;
        bl[i] = row < a.kv ? a.b[row] : 0.f;
        cl[i] = (a.c != nullptr && row < a.kv) ? a.c[row] : 0.f;
    }
    __syncthreads();

    // finishing thread: column fj, rows RPT fs .. RPT fs + RPT - 1
    const int fj = tid / TPC, fs = tid % TPC;
    const int fm = col0 + fj;
    const bool fok = fm < a.M;

    const size_t xoff = (size_t)g * NC * kp;   // the group's exchange block (words)
    u64 *const yg = a.yp + (size_t)g * xch::kRing * R * NC;
    int64_t q = 0, ny = 0;                     // phase, probe row to publish next
    // flags: this lane's word of the row tiles its wave reads, its wave's own
    constexpr bool kPolled = polled<KB, NCB>();
    unsigned *const fg = a.flags + (size_t)g * 128;
    const int fb = w * KB / 2 + (lane >> 2);
    const unsigned *flag = fb <= (w * KB + KB - 1) / 2 ? fg + 4 * fb + (lane & 3) : nullptr;

    // publish this thread's rows (values hv(i)) as BF16 (hi, lo) in the
    // B-fragment order: tile row o of column fj is term o % 8 of lane
    // 16 ((o % 32) / 8) + fj % 16 of k-block (row0 + o) / 32, column block
    // fj / 16 (row0 is a multiple of 32); then empty its slots of two phases
    // ago (polled rows) or raise its wave's flag
    auto publish = [&](auto hv) {
        constexpr int CH = RPT < 8 ? RPT : 8;      // rows per store
        float *xg = a.x + (size_t)(q & 3) * a.xfloats + xoff, *zg = a.x + (size_t)((q + 2) & 3) * a.xfloats + xoff;
        const int cb = fj / 16;
#pragma unroll
        for (int c = 0; c < RPT / CH; ++c) {
            unsigned ph[CH / 2], pl[CH / 2];
#pragma unroll
            for (int i = 0; i < CH / 2; ++i) {
                // hardware round-to-nearest-even, two values per instruction
                const f2 v = {hv(CH * c + 2 * i), hv(CH * c + 2 * i + 1)};
                const bf2 hi = __builtin_convertvector(v, bf2);
                const f2 rest = v - __builtin_convertvector(hi, f2);
                const bf2 lo = __builtin_convertvector(rest, bf2);
                const unsigned uh = __builtin_bit_cast(unsigned, hi), ul = __builtin_bit_cast(unsigned, lo);
                ph[i] = uh == xch::kEmpty ? 0x7FFF7FFFu : uh;
                pl[i] = ul == xch::kEmpty ? 0x7FFF7FFFu : ul;
            }
            constexpr unsigned E = xch::kEmpty;
            const int o = RPT * fs + CH * c;
            const int kb = (row0 + o) / 32, ln = 16 * ((o % 32) / 8) + (fj & 15);
            const size_t oh = frag_offset<NCB>(kb, cb, 0) / 2 + 4 * ln + (o % 8) / 2;   // words
            const size_t ol = frag_offset<NCB>(kb, cb, 1) / 2 + 4 * ln + (o % 8) / 2;
            if constexpr (CH == 8) {
                *reinterpret_cast<u4 *>(xg + oh) = u4{ph[0], ph[1], ph[2], ph[3]};
                if constexpr (!SINGLE) *reinterpret_cast<u4 *>(xg + ol) = u4{pl[0], pl[1], pl[2], pl[3]};
                if constexpr (kPolled) *reinterpret_cast<u4 *>(zg + oh) = u4{E, E, E, E};
                if constexpr (kPolled && !SINGLE) *reinterpret_cast<u4 *>(zg + ol) = u4{E, E, E, E};
            } else {
                *reinterpret_cast<u2 *>(xg + oh) = u2{ph[0], ph[1]};
                if constexpr (!SINGLE) *reinterpret_cast<u2 *>(xg + ol) = u2{pl[0], pl[1]};
                if constexpr (kPolled) *reinterpret_cast<u2 *>(zg + oh) = u2{E, E};
                if constexpr (kPolled && !SINGLE) *reinterpret_cast<u2 *>(zg + ol) = u2{E, E};
            }
        }
        if constexpr (!kPolled) xch::raise_flag(fg + 4 * r + w, (unsigned)(q + 1));
        ++q;
    };

    // products -> LDS partials -> finished rows (FP64 update) -> published
    // (ysum: where the last step's probe sum goes (row tile 0), or null)
    auto half_step = [&](int f, const u4 (&op)[4][KB], const double *up, bool forced, bool last,
                         double *ysum) -> double {
        const u64 *yp = yg + (size_t)((ny - 1) & 3) * R * NC + fj;
        // (behind flags the sum follows the wait for them, whose first look
        // has waited for the partials too: the registers are the products')
        ProbeSum<TPC, 0, (2 * KB + TPC - 1) / TPC> ps;
        if (ysum) ps.load(yp, NC, R, fs);
        auto sum = [&] {
            if (ysum) *ysum = ps.sum(wait, yp, NC, R, fs);
        };
        f4 acc[4][NCB];
        products<KB, SINGLE, NCB>(op, a.x + (size_t)((q - 1) & 3) * a.xfloats + xoff, 4u * NC * kp, w, lane, flag,
                                  (unsigned)q, wait, sum, acc);
        if (kPolled) sum();
        float *pw = part + w * NC * kLd;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
                *reinterpret_cast<f4 *>(pw + (16 * cb + (lane & 15)) * kLd + 16 * rb + 4 * (lane >> 4)) = acc[rb][cb];
        __syncthreads();
        const double u = forced ? *up : 0.0;
        double ypart = 0.0;
        float *h = sth + (f * NC + fj) * kLd + RPT * fs;
        float *l = stl + (f * NC + fj) * kLd + RPT * fs;
        float hn[RPT];                             // the new hi words, published below
#pragma unroll
        for (int q = 0; q < RPT / 4; ++q) {
            f4 p0 = *reinterpret_cast<const f4 *>(part + (0 * NC + fj) * kLd + RPT * fs + 4 * q);
            f4 p1 = *reinterpret_cast<const f4 *>(part + (1 * NC + fj) * kLd + RPT * fs + 4 * q);
            f4 p2 = *reinterpret_cast<const f4 *>(part + (2 * NC + fj) * kLd + RPT * fs + 4 * q);
            f4 p3 = *reinterpret_cast<const f4 *>(part + (3 * NC + fj) * kLd + RPT * fs + 4 * q);
            f4 hh = *reinterpret_cast<const f4 *>(h + 4 * q);
            f4 ll = *reinterpret_cast<const f4 *>(l + 4 * q);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = RPT * fs + 4 * q + e;
                // the wave partials are FP32 chain sums; one more FP32 rounding is
                // far below the BF16 state operand's
                double inc = (double)((p0[e] + p1[e]) + (p2[e] + p3[e])) * (double)a.scale;
                if (forced) inc = fma((double)bl[i], u, inc);
                const double yv = fma(a.dt, inc, (double)hh[e] + (double)ll[e]);
                const float hv = (float)yv;
                hh[e] = hv;
                ll[e] = (float)(yv - (double)hv);
                if (forced) ypart += (double)cl[i] * yv;
            }
            *reinterpret_cast<f4 *>(h + 4 * q) = hh;
            *reinterpret_cast<f4 *>(l + 4 * q) = ll;
#pragma unroll
            for (int e = 0; e < 4; ++e) hn[4 * q + e] = hh[e];
        }
        if (!last) publish([&](int i) { return hn[i]; });
        __syncthreads();   // partials read before the next half-step writes them
        return ypart;
    };

    // ---- initial exchange: S rows (the first half-step reads S)
    {
        const float *h0 = sth + (1 * NC + fj) * kLd + RPT * fs;
        publish([&](int i) { return h0[i]; });
    }

    double Jacc = 0.0;
    const bool probe = a.c != nullptr, sums = probe && r == 0;
    // the probe sum of step k (row tile 0)
    auto probe_row = [&](int64_t k, double yv) {
        if (fs != 0 || !fok) return;
        Jacc += a.dt * (yv * yv);
        if (a.y) a.y[(size_t)k * a.M + fm] = yv;
    };
    for (int64_t k = 0; k < a.nsteps; ++k) {
        if (k % kUWin == 0) forcing_window<NC>(uwin, a.source, a.n0 + k, a.dt, a.mu, col0, a.M);
        // (read after the products' barrier inside half_step)
        double ysum = 0.0;
        double yp = half_step(0, opv, uwin + (k % kUWin) * NC + fj, true, false, sums && k > 0 ? &ysum : nullptr);
        if (sums && k > 0) probe_row(k - 1, ysum);
        if (probe) {
            // sum the TPC strips of column fj, then publish this tile's
            // partial (a ring entry per step: row tile 0 reads entry k before
            // it publishes the velocity of step k + 1, so whoever publishes
            // that of step k + 2 may empty it)
            yp = column_sum<TPC>(yp);
            if (fs == 0) {
                xch::put64(yg + ((size_t)(ny & 3) * R + r) * NC + fj, yp);
                xch::clear64(yg + ((size_t)((ny + 2) & 3) * R + r) * NC + fj);
            }
            ++ny;
        }
        half_step(1, ops, nullptr, false, k + 1 == a.nsteps, nullptr);
    }
    if (sums) {
        ProbeSum<TPC> ps;
        const u64 *yp = yg + (size_t)((ny - 1) & 3) * R * NC + fj;
        ps.load(yp, NC, R, fs);
        probe_row(a.nsteps - 1, ps.sum(wait, yp, NC, R, fs));
    }

    // ---- write back (hi + lo), J
    for (int idx = tid; idx < 2 * NC * kRows; idx += kThreads) {
        const int f = idx / (NC * kRows), rem = idx - f * NC * kRows;
        const int j = rem / kRows, i = rem - j * kRows;
        const int m = col0 + j, row = row0 + i;
        if (m < a.M && row < a.kv) {
            float *dst = f == 0 ? a.V : a.S;
            dst[(size_t)m * a.kv + row] = sth[(f * NC + j) * kLd + i] + stl[(f * NC + j) * kLd + i];
        }
    }
    if (probe && a.J && r == 0 && fs == 0 && fok) a.J[fm] += Jacc;
}

// Split-layout BF16 fragments from the low-precision packed operator:
// dst[t][w][rb][kb][lane][e] = op[64 t + 16 rb + lane % 16][w kp/4 + 32 kb +
// 8 (lane / 16) + e], read from the column-block layout
// (BF16: pk[t][k/8][row][8]; FP8: pk[t][k/16][row][16] E4M3 bytes, widened
// exactly to BF16).
__global__ void split_pack_kernel(const unsigned char *__restrict__ src, int fp8, int T, int kp,
                                  unsigned short *__restrict__ dst) {
    const int KB = kp / 128;
    const int64_t total = (int64_t)T * kWaves * 4 * KB * 64 * 8;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        int64_t q = idx;
        const int e = (int)(q % 8); q /= 8;
        const int lane = (int)(q % 64); q /= 64;
        const int kb = (int)(q % KB); q /= KB;
        const int rb = (int)(q % 4); q /= 4;
        const int w = (int)(q % kWaves); q /= kWaves;
        const int t = (int)q;
        const int i = 16 * rb + (lane & 15);                    // row within tile
        const int k = w * (kp / 4) + 32 * kb + 8 * (lane >> 4) + e;
        unsigned short v;
        if (!fp8) {
            const unsigned short *s16 = reinterpret_cast<const unsigned short *>(src);
            v = s16[(((int64_t)t * (kp / 8) + k / 8) * 64 + i) * 8 + k % 8];
        } else {
            const unsigned char byte = src[(((int64_t)t * (kp / 16) + k / 16) * 64 + i) * 16 + k % 16];
            typedef float f2 __attribute__((ext_vector_type(2)));
            const f2 wv = __builtin_amdgcn_cvt_pk_f32_fp8((int)byte, false);
            v = (unsigned short)(__float_as_uint(wv.x) >> 16);   // E4M3 values are exact in BF16
        }
        dst[idx] = v;
    }
}

// Empty n 16-byte words of exchange slots and partials, zero flags (or the
// words of repeatable groups), the 64 words behind them (slot counters, status
// of repeatable runs) and the abort word.
constexpr int kFlagWords = 128 * 128;      // 128 groups of 32 row tiles x 4 waves
__global__ void split_clear_kernel(u4 *__restrict__ x, size_t n, unsigned *__restrict__ flags, int *__restrict__ status) {
    constexpr unsigned E = xch::kEmpty;
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = i0; i < n; i += step) x[i] = u4{E, E, E, E};
    for (size_t i = i0; i < kFlagWords + 64; i += step) flags[i] = 0u;
    if (i0 == 0) status[2] = 0;
}

__global__ void freeze_odd_kernel(unsigned *done, int n) {
    const int g = 2 * (int)threadIdx.x + 1;
    if (g < n) done[2 * g + 1] = xch::kGivenUp;
}

}  // namespace

hipError_t freeze_odd_groups(unsigned *done, int n, hipStream_t st) {
    if (n > 2 * kThreads) return hipErrorInvalidValue;
    hipLaunchKernelGGL(freeze_odd_kernel, dim3(1), dim3(kThreads), 0, st, done, n);
    return hipGetLastError();
}

size_t rank2_split_lds_bytes() {
    return sizeof(float) * ((size_t)2 * 2 * kCols * kLd + (size_t)kWaves * kCols * kLd + 2 * kRows);
}

bool rank2_split_k_ok(int kvp, bool f32) {
    if (f32) return kvp % kRows == 0 && kvp >= 2 * kRows && kvp <= kMaxSplitK;
    return kvp % 128 == 0 && kvp >= 128 && kvp <= 1024;   // whole 32-term k-blocks per wave
}

// Groups of R = kvp / 64 workgroups one launch holds: a group's workgroups
// share an XCD, so each of the 8 XCDs (32 CUs) holds floor(32 / R) groups.
int rank2_split_groups_per_launch(int kvp) { return kXcds * (kCusPerXcd / (kvp / kRows)); }

// Supported shapes: Kv == Ks == K with K a multiple of 64 in [128, 2048]
// for FP32 operators, a multiple of 128 up to 1024 for BF16 / FP8 ones (register-
// resident fragments), and all 64-column groups in one launch (one
// workgroup per CU, all resident).  Returns the group count, or 0 if the
// row-split schedule does not apply.
int rank2_split_groups(int kv, int ks, int kvp, int ksp, int M, bool f32) {
    if (kv != ks || kvp != ksp || !rank2_split_k_ok(kvp, f32)) return 0;
    const int G = (M + kCols - 1) / kCols;
    if (G > rank2_split_groups_per_launch(kvp)) return 0;
    return G;
}

size_t rank2_split_workspace_bytes(int kvp, int G) {
    return rank2_split_ws_bytes((size_t)G * kCols * kvp, (size_t)G * (kvp / 16) * kCols);
}

size_t rank2_split_ws_bytes(size_t xfloats, size_t ypd) {
    return sizeof(float) * xch::kRing * xfloats                        // exchange ring
           + sizeof(u64) * xch::kRing * ypd                            // probe partials
           + sizeof(unsigned) * (kFlagWords + 64);                     // flags, slot counters
}

hipError_t launch_split_pack(const void *lp, bool fp8, int kvp, int ksp, void *dst, hipStream_t st) {
    const int T = kvp / kRows;
    const int64_t total = (int64_t)T * 64 * ksp;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(split_pack_kernel, dim3(blocks), dim3(256), 0, st,
                       static_cast<const unsigned char *>(lp), fp8 ? 1 : 0, T, ksp,
                       static_cast<unsigned short *>(dst));
    return hipGetLastError();
}

hipError_t split_workspace(SplitArgs &a, void *ws, size_t xfloats, size_t ypd, bool poll_rows, hipStream_t st) {
    if (xfloats % 4) return hipErrorInvalidValue;
    a.x = static_cast<float *>(ws);
    a.xfloats = xfloats;
    a.yp = reinterpret_cast<u64 *>(a.x + xch::kRing * xfloats);
    a.flags = reinterpret_cast<unsigned *>(a.yp + xch::kRing * ypd);
    a.slots = a.flags + kFlagWords;
    a.spin_max = g_forced_timeout == 1 ? 256 : xch::kSpinMax;
    a.forced = g_forced_timeout == 1 ? 1 : 0;
    const size_t n = (poll_rows ? xfloats : 0) + 2 * ypd;      // 16-byte words
    u4 *from = reinterpret_cast<u4 *>(poll_rows ? ws : static_cast<void *>(a.yp));
    const int blocks = (int)(n / 256 < 64 ? 64 : (n / 256 > 1024 ? 1024 : n / 256));
    hipLaunchKernelGGL(split_clear_kernel, dim3(blocks), dim3(256), 0, st, from, n, a.flags, a.status);
    return hipGetLastError();
}

void fill_split_args(SplitArgs &a, const void *opv, const void *ops, const Rank2Args &r2, float scale, int *status) {
    a = SplitArgs{};
    a.opv = static_cast<const u4 *>(opv);
    a.ops = static_cast<const u4 *>(ops);
    a.b = static_cast<const float *>(r2.b);
    a.c = static_cast<const float *>(r2.c);
    a.mu = r2.mu;
    a.V = static_cast<float *>(r2.V);
    a.S = static_cast<float *>(r2.S);
    a.J = r2.J;
    a.y = r2.y;
    a.kv = r2.kv;
    a.kp = r2.kvp;
    a.M = r2.M;
    a.R = r2.kvp / kRows;
    a.n0 = r2.n0;
    a.nsteps = r2.nsteps;
    a.dt = r2.dt;
    a.source = r2.source;
    a.scale = scale;
    a.status = status;
    a.vtr = r2.vtr;
    a.str = r2.str;
    a.ytr = r2.ytr;
    a.wtr = r2.wtr;
    a.qtr = r2.qtr;
    a.dmu = r2.dmu;
}

int split_width_index(int M, int kvp) {
    const int cap = rank2_split_groups_per_launch(kvp);
    int wi = 0;
    while (wi < 2 && (M + (16 << wi) - 1) / (16 << wi) > cap) ++wi;
    return wi;
}

namespace {

// Low-precision kernels by (K = 128 KB, KB = 1 .. 8) x (pair, single-pass) x
// (group width 16, 32, 64 columns).
#define ROM_LP_WIDTHS(KB, SG)                                                           \
    (const void *)rank2_split_kernel<KB, SG, 1>, (const void *)rank2_split_kernel<KB, SG, 2>, \
        (const void *)rank2_split_kernel<KB, SG, 4>
const void *const kSplitLpKernels[48] = {
    ROM_LP_WIDTHS(1, false), ROM_LP_WIDTHS(1, true), ROM_LP_WIDTHS(2, false), ROM_LP_WIDTHS(2, true),
    ROM_LP_WIDTHS(3, false), ROM_LP_WIDTHS(3, true), ROM_LP_WIDTHS(4, false), ROM_LP_WIDTHS(4, true),
    ROM_LP_WIDTHS(5, false), ROM_LP_WIDTHS(5, true), ROM_LP_WIDTHS(6, false), ROM_LP_WIDTHS(6, true),
    ROM_LP_WIDTHS(7, false), ROM_LP_WIDTHS(7, true), ROM_LP_WIDTHS(8, false), ROM_LP_WIDTHS(8, true)};
#undef ROM_LP_WIDTHS

// Scratch of the allocation-free row-split run (rom_run_rank2_noalloc):
// exchange ring, probe partials and slot counters of the largest launch
// the schedule makes (rank2_split_workspace_bytes over every eligible shape:
// 16 MiB of exchange at G K = 256 x 64, 2 MiB of probe partials (16-row
// tiles), 64 KiB of flags).  One copy per GPU, held until the process ends; every call on a
// GPU uses that GPU's copy.
constexpr size_t kStaticScratchBytes = (size_t)18560 * 1024;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

}  // namespace

size_t rank2_split_static_bytes() { return kStaticScratchBytes; }

// Device address of this GPU's static scratch, looked up once per device
// with that device current (the array's host-side name is not a device
// address).  Only the returned pointer is passed to kernels.
hipError_t rank2_split_static_scratch(int device, void **ptr) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[device]) {
        int cur = -1;
        hipError_t e = hipGetDevice(&cur);
        if (e != hipSuccess) return e;
        if (cur != device) return hipErrorInvalidDevice;
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *ptr = addr[device];
    return hipSuccess;
}

hipError_t launch_rank2_split(const void *opv, const void *ops, const Rank2Args &r2, float scale, void *ws,
                              int G, int *status, bool f32, hipStream_t st, int mode) {
    if (f32) return launch_rank2_split_f32(opv, ops, r2, ws, G, status, st, mode);
    if (mode != 0 || !rank2_split_k_ok(r2.kvp, false) || G > rank2_split_groups_per_launch(r2.kvp))
        return hipErrorInvalidValue;
    SplitArgs a;
    fill_split_args(a, opv, ops, r2, scale, status);
    // the narrowest column group (16, 32 or 64 columns) whose workgroups all
    // fit; the workspace, sized for G 64-column groups, covers it
    const int wi = split_width_index(a.M, a.kp), nc = 16 << wi;
    a.G = (a.M + nc - 1) / nc;
    hipError_t e = split_workspace(a, ws, (size_t)a.G * nc * a.kp, (size_t)a.G * a.R * nc,
                                   a.kp / 128 << wi <= 8, st);
    if (e != hipSuccess) return e;
    void *args[] = {&a};
    const int idx = a.kp / 128 - 1;   // k-blocks per wave - 1 (K a multiple of 128, checked above)
    return launch_waiting(kSplitLpKernels[6 * idx + 3 * (r2.single ? 1 : 0) + wi], args, rank2_split_lds_bytes(), st, true);
}

hipError_t launch_waiting(const void *f, void **args, size_t lds, hipStream_t st, bool together) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    // behind the device's last such launch; it orders kernels and hands no data
    // on (contexts guard their workspaces), so its record releases no caches
    static hipEvent_t last[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    // (held until the launch is recorded: the next one, of any thread, waits
    // for this one)
    std::lock_guard<std::mutex> lk(mu);
    e = last[dev] ? hipStreamWaitEvent(st, last[dev], 0)
                  : hipEventCreateWithFlags(&last[dev], hipEventDisableTiming | hipEventDisableSystemFence);
    if (e != hipSuccess) return e;
    const dim3 grid(kXcds * kCusPerXcd), block(kThreads);
    e = together ? hipLaunchCooperativeKernel(f, grid, block, args, lds, st) : hipLaunchKernel(f, grid, block, args, lds, st);
    return e == hipSuccess ? hipEventRecord(last[dev], st) : e;
}

// The schedule needs all 256 workgroups resident at once, one per CU, 32 on
// each of the 8 XCDs (the group-slot logic counts on it), and cooperative
// launch support.
bool split_chip_ok() {
    int dev = 0, ncu = 0, coop = 0;
    if (hipGetDevice(&dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return false;
    if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess) return false;
    if (ncu != 256 || !coop) return false;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return false;
    return std::string(prop.gcnArchName).rfind("gfx950", 0) == 0;
}

bool rank2_split_device_ok() {
    if (!split_chip_ok()) return false;
    const size_t lds = rank2_split_lds_bytes();
    for (const void *f : kSplitLpKernels) {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kThreads, lds) != hipSuccess || nb < 1) return false;
    }
    return rank2_split_f32_device_ok() && rank2_rsplit_device_ok();
}

hipError_t rank2_split_configure() {
    // exactly the dynamic LDS the launch asks for (the kernel also has a few
    // bytes of static LDS, so the 160 KB maximum would be refused)
    const int lds = (int)rank2_split_lds_bytes();
    hipError_t e;
    for (const void *f : kSplitLpKernels) {
        e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    hipError_t ef = rank2_split_f32_configure();
    return ef == hipSuccess ? rank2_rsplit_configure() : ef;
}

}  // namespace rom
