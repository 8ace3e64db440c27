// Rank-2 leapfrog stepper, row-split schedule, FP32 operators and states
// (method and placement: see k_rank2_split.hip).
//
// The FP32 operator rows of a workgroup are 512 KB at K = 1024; products on
// v_mfma_f32_16x16x4f32 (A lane l: row l % 16, term l / 16; B lane l: term
// l / 16, column l % 16; D register r of lane l: row 4 (l / 16) + r, column
// l % 16).  Operands come in k-groups of 16 terms (4 instructions): lane l
// holds terms 4 j + l / 16 (j = 0..3) as one float4, for the operator
//   opf[t][kgg][rb][lane] = op[64 t + 16 rb + l % 16][16 kgg + 4 j + l / 16]
// and for the exchanged state, per group of NC = 16 NCB columns,
//   xf[kgg][cb][lane] = x[16 kgg + 4 j + l / 16][16 cb + l % 16]   (cb < NCB),
// so every wave load is 1 KB contiguous.  Wave w of a workgroup sums the
// reduction terms [w kp/4, (w+1) kp/4) in FP32 chains of 64 terms (the last
// one of a wave shorter where kp / 64 is not a multiple of 4), each folded
// into FP64 sums; the four FP64 partials meet in LDS, and the state (hi, lo)
// of a finishing thread's 4 NCB entries per field lives in its registers.
//
// Group width: each workgroup reads its 64 operator rows whatever the width,
// while its products and exchanged reads scale with NC, so the host takes
// the narrowest group (16, 32 or 64 columns) that still fits all workgroups
// on the chip.  A column's state arithmetic does not depend on NC, so every
// width gives bitwise the same states; only the probe's FP64 row sum is
// associated differently.
//
// Operator rows: where a wave has two chains per field (K = 320 .. 512) and the
// group 32 columns they stay in registers for the run (64 per chain and field);
// else they are streamed from L2 every half-step.  Up to K = 1024 and the
// samples that its groups hold, k_rank2_rsplit.hip with smaller row tiles runs
// instead, bitwise the same.
#include <type_traits>

#include "k_lane.h"
#include "k_split.h"

namespace rom {
namespace {

using namespace split;

constexpr int kLdD = kRows + 2;    // LDS column stride of the FP64 partials (doubles)
constexpr int kCG = 4;             // k-groups per FP32 chain (64 terms)
constexpr int kFrag = 4 * kCG;     // operator fragments of a chain: [k-group][16-row tile]

__device__ __forceinline__ f4 as_f4(u4 v) { return __builtin_bit_cast(f4, v); }

// A lane offset past every buffer's bound: such loads return zeros and move
// nothing (k-groups behind a wave's last one).
constexpr unsigned kNowhere = 0xF0000000u;

// Kernel kinds.  KIND > 0: the wave's KIND chains per field are resident and
// the rows polled themselves (all in registers at once).  Else streamed rows
// behind flags: KIND = -KGT with the k-group count known at compile time,
// 0 with any.
typedef const __attribute__((address_space(1))) unsigned char gbyte;
typedef const __attribute__((address_space(1))) f4 gf4;
typedef const __attribute__((address_space(1))) unsigned long long gu64;

// Two relaxed device-scope 8-byte loads (global_load_dwordx2 ... sc1), which
// the unrolled k-group loop schedules better than 16-byte buffer loads
// (measured: 41 against 48 us per step at K = M = 1024).
__device__ __forceinline__ u4 ld_shared(gbyte *p) {
    const gu64 *q = reinterpret_cast<const gu64 *>(p);
    const unsigned long long lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return u4{(unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32)};
}

// Streamed products of one field for wave w: acc[rb][cb][r] = sum over the
// wave's KG k-groups of op rows 16 rb .. x state columns 16 cb ..
// KGT: k-groups per wave (K / 64) when fixed at compile time (fully
// unrolled; K = 1024 with 32 columns), 0 for any K that is a multiple of 64 (KG
// taken at run time).  Both forms issue the same MFMAs in the same order
// (FP32 chains of 4 k-groups, the last one shorter when KG % 4 != 0, each
// folded into FP64 at its end), so they give the same sums.  The group's
// rows are waited for by flag (k_exchange.h): streamed rows that carry their
// own arrival would put a branch and a wait into the loop.
template <int KGT, int NCB>
__device__ __forceinline__ void products_stream(const u4 *opw, const float *xgrp, int KG, int w, int lane,
                                                const unsigned *flag, unsigned phase, xch::Wait &wait,
                                                double (&acc)[4][NCB][4]) {
    xch::wait_flags(wait, flag, phase);
    constexpr int D = 2;     // ring depth in k-groups (K >= 128: KG >= 2)
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[rb][cb][r] = 0.0;
    // opaque per-step bases (see products): no hoisted, spilled addresses
    uint64_t ob = reinterpret_cast<uint64_t>(opw), xb = reinterpret_cast<uint64_t>(xgrp);
    asm volatile("" : "+s"(ob), "+s"(xb));
    const unsigned loff = 16u * (unsigned)lane;
    f4 ra[D][4], rbx[D][NCB];
    // one FP32 chain of NQ k-groups from kg0, folded into the FP64 sums at
    // its end; `load` refills ring slot kg % D with k-group kg + D
    auto chain = [&](auto nq, int kg0, auto &&load) {
        constexpr int NQ = decltype(nq)::value;
        f4 c[4][NCB];
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) c[rb][cb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int kg = kg0 + q;
            const int slot = q % D;   // kg0 is a multiple of kCG, itself one of D
            f4 a[4], b[NCB];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = ra[slot][i];
#pragma unroll
            for (int i = 0; i < NCB; ++i) b[i] = rbx[slot][i];
            load(kg + D, ra[slot], rbx[slot]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
                        c[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[rb][j], b[cb][j], c[rb][cb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[rb][cb][r] += (double)c[rb][cb][r];
        __builtin_amdgcn_sched_barrier(0);
    };
    using Q4 = std::integral_constant<int, kCG>;
    if constexpr (KGT > 0) {
        gbyte *opb = reinterpret_cast<gbyte *>(ob);
        gbyte *xbb = reinterpret_cast<gbyte *>(xb) + (size_t)w * KGT * NCB * 1024;   // this wave's k-groups
        auto load = [&](int kg, f4 (&a)[4], f4 (&b)[NCB]) {
            if (kg >= KGT) return;
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = *reinterpret_cast<gf4 *>(opb + (size_t)(kg * 4 + q) * 1024 + loff);
#pragma unroll
            for (int q = 0; q < NCB; ++q)
                b[q] = __builtin_bit_cast(f4, ld_shared(xbb + (size_t)(kg * NCB + q) * 1024 + loff));
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, ra[d], rbx[d]);
        __builtin_amdgcn_sched_barrier(0);
        static_assert(KGT % kCG == 0, "whole chains");
#pragma unroll
        for (int kg0 = 0; kg0 < KGT; kg0 += kCG) chain(Q4{}, kg0, load);
    } else {
        // Run-time KG: buffer loads whose k-group offset is a scalar
        // (soffset), so no per-load address arithmetic; a ring refill past
        // the wave's last k-group re-reads that k-group (straight-line code:
        // a branch around the refill would make the compiler wait for every
        // load in flight).  Exchange loads take the device-scope policy.
        const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<void *>(ob), (short)0, KG * 4 * 1024, kRawBufferWord3);
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
            reinterpret_cast<void *>(xb), (short)0, 4 * KG * NCB * 1024, kRawBufferWord3);
        const int xw = w * KG * NCB * 1024;
        auto load = [&](int kg, f4 (&a)[4], f4 (&b)[NCB]) {
            kg = min(kg, KG - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q)
                a[q] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(ro, loff, (kg * 4 + q) * 1024, 0));
#pragma unroll
            for (int q = 0; q < NCB; ++q)
                b[q] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rx, loff, xw + (kg * NCB + q) * 1024, kDeviceScope));
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(d, ra[d], rbx[d]);
        __builtin_amdgcn_sched_barrier(0);
        const int full = KG - KG % kCG;
        for (int kg0 = 0; kg0 < full; kg0 += kCG) chain(Q4{}, kg0, load);
        switch (KG % kCG) {
        case 1: chain(std::integral_constant<int, 1>{}, full, load); break;
        case 2: chain(std::integral_constant<int, 2>{}, full, load); break;
        case 3: chain(std::integral_constant<int, 3>{}, full, load); break;
        default: break;
        }
    }
}

// The same sums from resident operator chains.
template <int KIND, int NCB>
__device__ __forceinline__ void products_resident(const u4 (&res)[KIND][kFrag], int R, int w, int lane, const float *xb,
                                                  xch::Wait &wait, double (&acc)[4][NCB][4]) {
    constexpr int NC = 16 * NCB;
#pragma unroll
    for (int rb = 0; rb < 4; ++rb)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[rb][cb][r] = 0.0;
    // opaque per-step base: no hoisted, spilled addresses
    uint64_t xa = reinterpret_cast<uint64_t>(xb);
    asm volatile("" : "+s"(xa));
    const __amdgpu_buffer_rsrc_t rx = raw_buffer(reinterpret_cast<void *>(xa), (unsigned)R * (kRows * NC * 4));
    const unsigned loff = 16u * (unsigned)lane;
    u4 bx[KIND][NCB][kCG];
    long spins = 0;
    for (;;) {
#pragma unroll
        for (int i = 0; i < KIND; ++i)
#pragma unroll
            for (int q = 0; q < kCG; ++q) {
                const int kg = kCG * i + q;
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
                    bx[i][cb][q] = __builtin_amdgcn_raw_buffer_load_b128(rx, kg < R ? loff : kNowhere,
                                                                         ((w * R + kg) * NCB + cb) * 1024, kDeviceScope);
            }
        unsigned m = 0;
#pragma unroll
        for (int i = 0; i < KIND; ++i)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                for (int q = 0; q < kCG; ++q) {
                    const u4 &v = bx[i][cb][q];
                    m = xch::max3u(xch::max3u(m, v[0], v[1]), v[2], v[3]);
                }
        if (wait.dead || (!wait.forced && __ballot(m == xch::kEmpty) == 0)) break;
        if (wait.give_up(spins)) break;
    }
    // (the emptied slots of the last publication: before the next one)
    xch::publish_fence();
    auto chain = [&](int i, auto nq) {
        constexpr int NQ = decltype(nq)::value;
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
            f4 c[4];
#pragma unroll
            for (int rb = 0; rb < 4; ++rb) c[rb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int rb = 0; rb < 4; ++rb)
                        c[rb] = __builtin_amdgcn_mfma_f32_16x16x4f32(as_f4(res[i][4 * q + rb])[j],
                                                                     as_f4(bx[i][cb][q])[j], c[rb], 0, 0, 0);
#pragma unroll
            for (int rb = 0; rb < 4; ++rb)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[rb][cb][r] += (double)c[rb][r];
        }
    };
    if constexpr (KIND == 2) chain(0, std::integral_constant<int, 4>{});
    switch (R & 3) {                           // k-groups of the last chain
    case 0: chain(KIND - 1, std::integral_constant<int, 4>{}); break;
    case 1: chain(KIND - 1, std::integral_constant<int, 1>{}); break;
    case 2: chain(KIND - 1, std::integral_constant<int, 2>{}); break;
    default: chain(KIND - 1, std::integral_constant<int, 3>{}); break;
    }
}

// GR: grouped run of many instances (64-column groups, each with its own
// padded K).  A workgroup finds its group and row tile in the launch's slot
// map (a.smap[32 xcc + slot]: 32 lg + r, or -1 for an idle slot); group lg
// then takes its operators, source, mu, states, sizes, padded K, exchange
// offset, first sample column and dt from a.grp[a.g0 + lg] (the probe is
// off).  Otherwise they come from the arguments, the R = K / 64 row tiles of
// group g are R consecutive slots of one XCD, and group g owns columns NC g
// .. NC g + NC - 1.  The arithmetic of a column is the same either way.
//
// Finishing threads: TPC = 256 / NC threads per column; thread fs of column
// fj owns the rows 16 kgl + 4 j + q0 + qq (j = 0..3, qq < NCB) of the row
// tile, kgl = fs / (4 / NCB), q0 = NCB (fs % (4 / NCB)), as entry e = NCB j +
// qq of its registers: the entries of one qq are the 4 terms of one lane's
// fragment, published as one float4.
// MODE: kSplitPlain, kSplitTraced (also writes the state after every step to
// a.vtr / a.str, entry 0 the state given, and the probe trace to a.y), or
// kSplitAdjoint: the discrete adjoint of the step run backwards, with the
// fields (V, S) holding (P, Q), the operators packed as (Asv^T, Avs^T), the
// host passing c as the source vector and b as the probe, the amplitude 2 y
// read from a.ytr, iteration k taking step n = n0 + nsteps - 1 - k; it
// writes a.qtr[n - n0] = Q before and a.wtr[n - n0] = P after the P update
// and adds dt (b^T P) du/dmu(t_n) to a.dmu.
enum SplitMode { kSplitPlain = 0, kSplitTraced = 1, kSplitAdjoint = 2 };

// The run of row tile r of group g (see the kernels below).
template <int KIND, bool GR, int NCB, int MODE>
__device__ __forceinline__ void split_f32_run(const SplitArgs &a, int g, int r, double *uwin) {
    static_assert(NCB == 1 || NCB == 2 || NCB == 4, "16, 32 or 64 columns per group");
    static_assert(!GR || (NCB == 4 && KIND == 0 && MODE == kSplitPlain), "grouped runs: plain, 64-column groups");
    static_assert(KIND <= 0 || NCB <= 2, "polled rows of 64 columns do not fit in registers");
    constexpr bool kPolled = KIND > 0;
    constexpr int NC = 16 * NCB;               // columns per group
    constexpr int TPC = kThreads / NC;         // finishing threads per column
    constexpr int RPT = 4 * NCB;               // rows per finishing thread and field
    constexpr int PSZ = kWaves * NC * kLdD;    // doubles of the four partials
    constexpr bool kTwo = NCB <= 2;            // a partials buffer per field
    extern __shared__ __align__(16) unsigned char smem[];
    float *bl = reinterpret_cast<float *>(smem);               // own rows of b and c
    float *cl = bl + kRows;
    double *part = reinterpret_cast<double *>(cl + kRows);      // [field][wave][col][kLdD]

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int kp = a.kp, R = a.R;
    int kv = a.kv, M = a.M, col0 = g * NC, src = a.source;
    size_t xoff = (size_t)g * NC * kp;         // the group's exchange block (words)
    double dt = a.dt;
    const float *bsrc = a.b, *csrc = a.c;
    const double *mup = a.mu;
    float *Vp = a.V, *Sp = a.S;
    const void *opv = a.opv, *ops = a.ops;
    if constexpr (GR) {
        // the descriptor is the same for the whole workgroup: keep its
        // fields in scalar registers (the operator bases must be scalar)
        const SplitGroup &q = a.grp[a.g0 + g];
        kv = __builtin_amdgcn_readfirstlane(q.kv);
        kp = __builtin_amdgcn_readfirstlane(q.kp);
        R = kp / kRows;
        xoff = (size_t)uniform64((uint64_t)q.xoff);
        M = __builtin_amdgcn_readfirstlane(q.M);
        col0 = __builtin_amdgcn_readfirstlane(q.col0);
        src = __builtin_amdgcn_readfirstlane(q.source);
        dt = __builtin_bit_cast(double, uniform64(__builtin_bit_cast(uint64_t, q.dt)));
        bsrc = reinterpret_cast<const float *>(uniform64(reinterpret_cast<uint64_t>(q.b)));
        csrc = nullptr;
        mup = reinterpret_cast<const double *>(uniform64(reinterpret_cast<uint64_t>(q.mu)));
        Vp = reinterpret_cast<float *>(uniform64(reinterpret_cast<uint64_t>(q.V)));
        Sp = reinterpret_cast<float *>(uniform64(reinterpret_cast<uint64_t>(q.S)));
        opv = reinterpret_cast<const void *>(uniform64(reinterpret_cast<uint64_t>(q.opv)));
        ops = reinterpret_cast<const void *>(uniform64(reinterpret_cast<uint64_t>(q.ops)));
    }
    xch::Wait wait{a.status, a.spin_max, a.forced, false};
    const int row0 = r * kRows;
    for (int i = tid; i < kRows; i += kThreads) {
        const int row = row0 + i;
        bl[i] = row < kv ? bsrc[row] : 0.f;
        cl[i] = (csrc != nullptr && row < kv) ? csrc[row] : 0.f;
    }
    // finishing thread: column fj, RPT rows (see above); its state entries of
    // both fields stay in registers
    const int fj = tid / TPC, fs = tid % TPC;
    const int kgl = fs / (4 / NCB), q0 = NCB * (fs % (4 / NCB));
    auto frow = [&](int e) { return 16 * kgl + 4 * (e / NCB) + q0 + e % NCB; };   // row within the tile
    const int fm = col0 + fj;
    const bool fok = fm < M;
    float sh[2][RPT], sl[2][RPT];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int e = 0; e < RPT; ++e) {
            const int row = row0 + frow(e);
            const float *sp = f == 0 ? Vp : Sp;
            sh[f][e] = (fok && row < kv) ? sp[(size_t)fm * kv + row] : 0.f;
            sl[f][e] = 0.f;
        }
    // operator fragments of row tile r; this wave's resident chains
    const u4 *opvt = static_cast<const u4 *>(opv) + (size_t)r * R * kFrag * 64;
    const u4 *opst = static_cast<const u4 *>(ops) + (size_t)r * R * kFrag * 64;
    u4 rv[KIND > 0 ? KIND : 1][kFrag], rs[KIND > 0 ? KIND : 1][kFrag];
    if constexpr (KIND > 0) {
#pragma unroll
        for (int i = 0; i < KIND; ++i)
#pragma unroll
            for (int q = 0; q < kFrag; ++q) {
                const size_t o = ((size_t)(w * R + min(kCG * i + q / 4, R - 1)) * 4 + q % 4) * 64 + lane;
                rv[i][q] = opvt[o];
                rs[i][q] = opst[o];
            }
    }
    __syncthreads();

    u64 *const yg = a.yp + (size_t)g * xch::kRing * R * NC;
    const double muf = fok ? mup[fm] : 1.0;
    const bool probe = csrc != nullptr;
    int64_t q = 0, ny = 0;                     // phase, probe row to publish next

    // flags: this lane's word of the blocks its wave reads, its wave's own
    unsigned *const fg = a.flags + (size_t)g * 128;
    // (its k-groups w R .. w R + R - 1 are rows of the tiles w R / 4 ..)
    const int fb = w * R / 4 + (lane >> 2);
    const unsigned *flag = fb <= (w * R + R - 1) / 4 ? fg + 4 * fb + (lane & 3) : nullptr;

    // publish this thread's rows (hi words) of field f in fragment order: row
    // row0 + 16 kgl + 4 j + q of column fj is term j of lane 16 q + fj % 16 in
    // k-group (row0 + 16 kgl) / 16, column block fj / 16; then empty its slots
    // of two phases ago (polled rows) or raise its wave's flag
    auto publish = [&](int f) {
        float *xg = a.x + (size_t)(q & 3) * a.xfloats + xoff, *zg = a.x + (size_t)((q + 2) & 3) * a.xfloats + xoff;
        const size_t o = ((size_t)(((row0 + 16 * kgl) / 16) * NCB + fj / 16) * 64 + 16 * q0 + (fj & 15)) * 4;
#pragma unroll
        for (int qq = 0; qq < NCB; ++qq) {
            u4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned x = __builtin_bit_cast(unsigned, sh[f][NCB * j + qq]);
                v[j] = kPolled && x == xch::kEmpty ? 0x7FC00000u : x;
            }
            *reinterpret_cast<u4 *>(xg + o + 64 * qq) = v;
            constexpr unsigned E = xch::kEmpty;
            if constexpr (kPolled) *reinterpret_cast<u4 *>(zg + o + 64 * qq) = u4{E, E, E, E};
        }
        if constexpr (!kPolled) xch::raise_flag(fg + 4 * r + w, (unsigned)(q + 1));
        ++q;
    };

    // ysum: where the last step's probe sum goes (row tile 0), or null
    auto half_step = [&](int f, const u4 (&res)[KIND > 0 ? KIND : 1][kFrag], const u4 *opt, const double *up, bool forced,
                         bool last, double *ysum) -> double {
        const u64 *yp = yg + (size_t)((ny - 1) & 3) * R * NC + fj;
        // (behind flags the sum goes ahead of the wait for them: the partials
        // are a half-step old, and the registers are the products')
        ProbeSum<TPC> ps;
        if (ysum) ps.load(yp, NC, R, fs);
        auto sum = [&] {
            if (ysum) *ysum = ps.sum(wait, yp, NC, R, fs);
        };
        if (!kPolled) sum();
        double acc[4][NCB][4];
        const float *xb = a.x + (size_t)((q - 1) & 3) * a.xfloats + xoff;
        if constexpr (KIND > 0)
            products_resident<KIND, NCB>(res, R, w, lane, xb, wait, acc);
        else
            products_stream<-KIND, NCB>(opt + (size_t)w * R * kFrag / kCG * 64, xb, R, w, lane, flag, (unsigned)q, wait,
                                        acc);
        if (kPolled) sum();
        double *pf = part + (kTwo ? f * PSZ : 0), *pw = pf + w * NC * kLdD;
#pragma unroll
        for (int rb = 0; rb < 4; ++rb)
#pragma unroll
            for (int cb = 0; cb < NCB; ++cb) {
                double *d = pw + (16 * cb + (lane & 15)) * kLdD + 16 * rb + 4 * (lane >> 4);
#pragma unroll
                for (int rr = 0; rr < 4; ++rr) d[rr] = acc[rb][cb][rr];
            }
        __syncthreads();
        const double u = forced ? *up : 0.0;
        double ypart = 0.0;
#pragma unroll
        for (int e = 0; e < RPT; ++e) {
            const int i = frow(e);
            const double *d = pf + fj * kLdD + i;
            double inc = (d[0] + d[NC * kLdD]) + (d[2 * NC * kLdD] + d[3 * NC * kLdD]);
            if (forced) inc = fma((double)bl[i], u, inc);
            const double yv = fma(dt, inc, (double)sh[f][e] + (double)sl[f][e]);
            const float hv = (float)yv;
            sh[f][e] = hv;
            sl[f][e] = (float)(yv - (double)hv);
            if (forced) ypart += (double)cl[i] * yv;
        }
        if (!last) publish(f);
        if constexpr (!kTwo) __syncthreads();   // partials read before the next half-step writes them
        return ypart;
    };

    // this thread's rows of field f (hi + lo) into trace matrix tr (M x kv
    // per entry), entry e
    auto trace = [&](float *tr, int f, int64_t e) {
        float *d = tr + (size_t)e * M * kv + (size_t)fm * kv;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int row = row0 + frow(i);
            if (fok && row < kv) d[row] = sh[f][i] + sl[f][i];
        }
    };

    publish(1);
    if constexpr (MODE == kSplitTraced) {
        trace(a.vtr, 0, 0);
        trace(a.str, 1, 0);
    }

    double Jacc = 0.0;
    // the probe sum of iteration k (row tile 0)
    auto probe_row = [&](int64_t k, double yv) {
        if (fs != 0 || !fok) return;
        if constexpr (MODE == kSplitAdjoint) {
            Jacc += dt * yv * dev::forcing_dmu(src, (double)(a.n0 + a.nsteps - 1 - k) * dt, muf);
        } else {
            Jacc += dt * (yv * yv);
            if (a.y) a.y[(size_t)k * M + fm] = yv;
        }
    };
    const bool sums = probe && r == 0;
    for (int64_t k = 0; k < a.nsteps; ++k) {
        // step n of this iteration, its trace row
        const int64_t n = MODE == kSplitAdjoint ? a.n0 + a.nsteps - 1 - k : a.n0 + k;
        if (k % kUWin == 0) {
            if constexpr (MODE == kSplitAdjoint)
                adjoint_window<NC>(uwin, a.ytr, a.nsteps - 1 - k, col0, M);
            else
                forcing_window<NC>(uwin, src, a.n0 + k, dt, mup, col0, M);
        }
        if constexpr (MODE == kSplitAdjoint) trace(a.qtr, 1, n - a.n0);   // Q^{n+1}
        // (read after the products' barrier inside half_step)
        double ysum = 0.0;
        double yp = half_step(0, rv, opvt, uwin + (k % kUWin) * NC + fj, true, false, sums && k > 0 ? &ysum : nullptr);
        if (sums && k > 0) probe_row(k - 1, ysum);
        if constexpr (MODE == kSplitAdjoint) trace(a.wtr, 0, n - a.n0);   // w^n
        if constexpr (MODE == kSplitTraced) trace(a.vtr, 0, k + 1);
        if (probe) {
            // sum over the TPC consecutive threads of column fj.  The ring
            // of probe partials has an entry per step: row tile 0 reads
            // entry k before it publishes the velocity of step k + 1, so
            // whoever publishes that of step k + 2 may empty it.
            yp = column_sum<TPC>(yp);
            if (fs == 0) {
                xch::put64(yg + ((size_t)(ny & 3) * R + r) * NC + fj, yp);
                xch::clear64(yg + ((size_t)((ny + 2) & 3) * R + r) * NC + fj);
            }
            ++ny;
        }
        half_step(1, rs, opst, nullptr, false, k + 1 == a.nsteps, nullptr);
        if constexpr (MODE == kSplitTraced) trace(a.str, 1, k + 1);
    }
    if (sums) {
        ProbeSum<TPC> ps;
        const u64 *yp = yg + (size_t)((ny - 1) & 3) * R * NC + fj;
        ps.load(yp, NC, R, fs);
        probe_row(a.nsteps - 1, ps.sum(wait, yp, NC, R, fs));
    }

#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int e = 0; e < RPT; ++e) {
            const int row = row0 + frow(e);
            float *dst = f == 0 ? Vp : Sp;
            if (fok && row < kv) dst[(size_t)fm * kv + row] = sh[f][e] + sl[f][e];
        }
    if constexpr (MODE == kSplitAdjoint) {
        if (probe && a.dmu && r == 0 && fs == 0 && fok) a.dmu[fm] += Jacc;
    } else {
        if (probe && a.J && r == 0 && fs == 0 && fok) a.J[fm] += Jacc;
    }
}

template <int KIND, bool GR, int NCB, int MODE = kSplitPlain>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void rank2_split_f32_kernel(SplitArgs a) {
    __shared__ double uwin[kUWin * 16 * NCB];
    const int code = take_slot(a.slots);
    const int xcc = code & 7, s = code >> 3;
    int r, g;
    if constexpr (GR) {
        const int e = s < 32 ? a.smap[32 * xcc + s] : -1;
        if (e < 0) return;                     // idle workgroup
        g = __builtin_amdgcn_readfirstlane(e >> 5);
        r = __builtin_amdgcn_readfirstlane(e & 31);
    } else {
        r = s % a.R;
        g = (s / a.R) * 8 + xcc;
        if (g >= a.G) return;
    }
    split_f32_run<KIND, GR, NCB, MODE>(a, g, r, uwin);
}

// Two runs of one shape side by side in one launch, on disjoint workgroups:
// groups 0 .. G-1 run a0 traced (the adjoint's recompute of a segment),
// groups G .. 2G-1 run a1 in adjoint mode (the reverse sweep of the next
// segment).  Each run has its own workspace; the slot counters are a0's.
template <int KIND, int NCB>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void rank2_split_f32_dual_kernel(SplitArgs a0, SplitArgs a1) {
    __shared__ double uwin[kUWin * 16 * NCB];
    const int code = take_slot(a0.slots);
    const int xcc = code & 7, s = code >> 3;
    const int r = s % a0.R, g = (s / a0.R) * 8 + xcc;
    if (g >= 2 * a0.G) return;
    if (g < a0.G)
        split_f32_run<KIND, false, NCB, kSplitTraced>(a0, g, r, uwin);
    else
        split_f32_run<KIND, false, NCB, kSplitAdjoint>(a1, g - a0.G, r, uwin);
}

// FP32 split-layout operator (rows x cols) from a column-major FP32 matrix:
// A itself (ld rows), or with `trans` the transpose of a column-major
// cols x rows matrix (ld cols); zero padded: dst[t][kgg][rb][lane][j] (see
// above).
__global__ void split_pack_f32_kernel(const float *__restrict__ A, int rows, int cols, int T, int kp, int trans,
                                      float *__restrict__ dst) {
    const int KG = kp / 16;
    const int64_t total = (int64_t)T * KG * 4 * 64 * 4;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total;
         idx += (int64_t)gridDim.x * blockDim.x) {
        int64_t q = idx;
        const int j = (int)(q % 4); q /= 4;
        const int lane = (int)(q % 64); q /= 64;
        const int rb = (int)(q % 4); q /= 4;
        const int kg = (int)(q % KG); q /= KG;
        const int t = (int)q;
        const int row = 64 * t + 16 * rb + (lane & 15);
        const int k = 16 * kg + 4 * j + (lane >> 4);
        dst[idx] = (row < rows && k < cols) ? (trans ? A[k + (int64_t)row * cols] : A[row + (int64_t)k * rows]) : 0.f;
    }
}

// Streamed kernels by width index, and the resident ones, two chains per wave
// with 32 columns.  Runs take these only where k_rank2_rsplit.hip has no tile
// (more samples than its groups hold, K > 1024), where one chain per wave
// never occurs with 16 or 32 columns, nor two with 16; the compile-time k-group
// count pays at K = 1024 with 32 columns.
struct KernelSet {
    const void *streamed[3], *resident;
};
constexpr int kResidentWidth = 1;
const KernelSet kF32Plain = {{(const void *)rank2_split_f32_kernel<0, false, 1>,
                              (const void *)rank2_split_f32_kernel<0, false, 2>,
                              (const void *)rank2_split_f32_kernel<0, false, 4>},
                             (const void *)rank2_split_f32_kernel<2, false, 2>};
const void *const kF32Plain1024 = (const void *)rank2_split_f32_kernel<-16, false, 2>;
const KernelSet kF32Traced = {{(const void *)rank2_split_f32_kernel<0, false, 1, kSplitTraced>,
                               (const void *)rank2_split_f32_kernel<0, false, 2, kSplitTraced>,
                               (const void *)rank2_split_f32_kernel<0, false, 4, kSplitTraced>},
                              nullptr};
const KernelSet kF32Adjoint = {{(const void *)rank2_split_f32_kernel<0, false, 1, kSplitAdjoint>,
                                (const void *)rank2_split_f32_kernel<0, false, 2, kSplitAdjoint>,
                                (const void *)rank2_split_f32_kernel<0, false, 4, kSplitAdjoint>},
                               (const void *)rank2_split_f32_kernel<2, false, 2, kSplitAdjoint>};
const void *const kF32Grouped = (const void *)rank2_split_f32_kernel<0, true, 4>;
const KernelSet kF32Dual = {{(const void *)rank2_split_f32_dual_kernel<0, 1>,
                             (const void *)rank2_split_f32_dual_kernel<0, 2>,
                             (const void *)rank2_split_f32_dual_kernel<0, 4>},
                            (const void *)rank2_split_f32_dual_kernel<2, 2>};

// Whether the runs of a set at padded size kp and width 16 << wi have a
// resident kernel (two chains per wave: K in 320 .. 512).
bool resident(const KernelSet &s, int kp, int wi) {
    return s.resident && wi == kResidentWidth && (kp / kRows + kCG - 1) / kCG == 2;
}

template <class F>
hipError_t each_kernel(F f) {
    hipError_t e = f(kF32Grouped);
    if (e == hipSuccess) e = f(kF32Plain1024);
    for (const KernelSet *s : {&kF32Plain, &kF32Traced, &kF32Adjoint, &kF32Dual}) {
        for (const void *k : s->streamed)
            if (e == hipSuccess) e = f(k);
        if (e == hipSuccess && s->resident) e = f(s->resident);
    }
    return e;
}

// The four partials of 64 columns (narrower groups: of both fields), b and
// c; more than half a CU's LDS, so one workgroup per CU.
constexpr size_t kLdsF32 = sizeof(double) * (size_t)kWaves * kCols * kLdD + sizeof(float) * 2 * kRows;

}  // namespace

hipError_t launch_split_pack_f32(const float *A, int rows, int cols, int prow, int pcol, void *dst, hipStream_t st,
                                 bool trans) {
    const int T = prow / kRows;
    const int64_t total = (int64_t)T * 64 * pcol;
    int blocks = (int)((total + 255) / 256);
    if (blocks > 8192) blocks = 8192;
    hipLaunchKernelGGL(split_pack_f32_kernel, dim3(blocks), dim3(256), 0, st, A, rows, cols, T, pcol, trans ? 1 : 0,
                       static_cast<float *>(dst));
    return hipGetLastError();
}

hipError_t launch_grouped_split_f32(const SplitGroup *grp_dev, int g0, int G, const int *smap_dev, size_t xfloats,
                                    void *ws, int *status, int64_t n0, int64_t nsteps, hipStream_t st) {
    if (G <= 0 || nsteps <= 0) return hipSuccess;
    if (G > kXcds * kCusPerXcd / 2) return hipErrorInvalidValue;
    SplitArgs a{};
    a.grp = grp_dev;
    a.smap = smap_dev;
    a.g0 = g0;
    a.G = G;
    a.n0 = n0;
    a.nsteps = nsteps;
    a.scale = 1.0f;
    a.status = status;
    hipError_t e = split_workspace(a, ws, xfloats, 0, false, st);
    if (e != hipSuccess) return e;
    void *args[] = {&a};
    return launch_waiting(kF32Grouped, args, kLdsF32, st, true);
}

// mode: kSplitPlain, kSplitTraced, kSplitAdjoint.
hipError_t launch_rank2_split_f32(const void *opv, const void *ops, const Rank2Args &r2, void *ws, int G, int *status,
                                  hipStream_t st, int mode) {
    if (mode < 0 || mode > 2 || !rank2_split_k_ok(r2.kvp, true) || G > rank2_split_groups_per_launch(r2.kvp))
        return hipErrorInvalidValue;
    if (rank2_rsplit_applies(false, r2.kv, r2.ks, r2.kvp, r2.ksp, r2.M, 1))
        return launch_rank2_rsplit(false, opv, ops, r2, ws, status, st, mode);
    SplitArgs a;
    fill_split_args(a, opv, ops, r2, 1.0f, status);
    // the narrowest column group whose workgroups all fit; the workspace,
    // sized for G 64-column groups, covers it
    const int wi = split_width_index(a.M, a.kp), nc = 16 << wi;
    a.G = (a.M + nc - 1) / nc;
    const KernelSet &s = mode == kSplitPlain ? kF32Plain : (mode == kSplitTraced ? kF32Traced : kF32Adjoint);
    const bool res = resident(s, a.kp, wi);
    hipError_t e = split_workspace(a, ws, (size_t)a.G * nc * a.kp, (size_t)a.G * a.R * nc, res, st);
    if (e != hipSuccess) return e;
    void *args[] = {&a};
    const void *f = mode == kSplitPlain && a.kp == 1024 && wi == 1 ? kF32Plain1024 : res ? s.resident : s.streamed[wi];
    return launch_waiting(f, args, kLdsF32, st, true);
}

int rank2_split_dual_width(int kvp, int M) {
    if (!rank2_split_k_ok(kvp, true)) return -1;
    const int cap = rank2_split_groups_per_launch(kvp);
    for (int wi = 0; wi < 3; ++wi)
        if (2 * ((M + (16 << wi) - 1) / (16 << wi)) <= cap) return wi;
    return -1;
}

hipError_t launch_rank2_split_dual(const void *opv0, const void *ops0, const Rank2Args &r0, void *ws0,
                                   const void *opv1, const void *ops1, const Rank2Args &r1, void *ws1, int G,
                                   int *status, hipStream_t st) {
    const int wi = rank2_split_dual_width(r0.kvp, r0.M);
    if (wi < 0 || r1.kvp != r0.kvp || r1.M != r0.M || r1.nsteps <= 0 || r0.nsteps <= 0) return hipErrorInvalidValue;
    SplitArgs a0, a1;
    fill_split_args(a0, opv0, ops0, r0, 1.0f, status);
    fill_split_args(a1, opv1, ops1, r1, 1.0f, status);
    const int nc = 16 << wi;
    a0.G = a1.G = (r0.M + nc - 1) / nc;
    if (a0.G * nc > G * kCols) return hipErrorInvalidValue;    // the workspaces hold G 64-column groups
    const size_t nx = (size_t)a0.G * nc * a0.kp, ny = (size_t)a0.G * a0.R * nc;
    const bool res = resident(kF32Dual, a0.kp, wi);
    hipError_t e = split_workspace(a0, ws0, nx, ny, res, st);
    if (e == hipSuccess) e = split_workspace(a1, ws1, nx, ny, res, st);
    if (e != hipSuccess) return e;
    void *args[] = {&a0, &a1};
    return launch_waiting(res ? kF32Dual.resident : kF32Dual.streamed[wi], args, kLdsF32, st, true);
}

bool rank2_split_f32_device_ok() {
    return each_kernel([](const void *f) {
               int nb = 0;
               hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kThreads, kLdsF32);
               return e == hipSuccess && nb < 1 ? hipErrorLaunchOutOfResources : e;
           }) == hipSuccess;
}

hipError_t rank2_split_f32_configure() {
    return each_kernel([](const void *f) {
        return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsF32);
    });
}

}  // namespace rom
