// Rank-2 leapfrog stepper, FP32 operators and states: row-split groups whose
// operator rows stay in registers for the whole run (method and placement:
// see k_rank2_split.hip).
//
// A group of NC = 16 NCB samples is stepped by R workgroups of one XCD, each
// owning RT = 16 NRB rows of both fields; Kv and Ks need not be equal.  Up to
// K = 1024 those rows of both operators fit in a CU's registers (32 NCH NRB
// per lane, NCH = ceil(K / 256)), so a half-step moves only the group's state:
// every wave polls the exchange slots of its quarter of the terms
// (k_exchange.h), all in registers at once.
//
// Products on v_mfma_f32_16x16x4f32, fragments and operator pack as in
// k_rank2_split_f32.hip.  The instruction rounds like four fused multiply-
// adds in the order of its terms (checked bit by bit against fmaf, as is the
// 4x4x1 instruction), so the sums of two older schedules come out bit for
// bit from these kernels:
//  * POL = kQuarters: the row-split schedule's.  Wave w sums the terms
//    [w kp/4, (w+1) kp/4) in FP32 chains of 64 folded into FP64; the four
//    FP64 partials are added pairwise.
//  * POL = kPairs: the column blocks'.  Each 64 terms give two FP32 chains,
//    the even and the odd groups of 4 terms; all chains of a row are folded
//    into one FP64 sum in order.  Wave w computes the 64-term blocks w, w +
//    4, .. and leaves its FP32 chains in LDS for the fold.
//
// Tile: the smallest RT NC whose groups all fit on the chip at once; the
// matrix-core time of a half-step is proportional to it, the exchange is not.
//
// Bound by the exchange, 0.8 us twice a step, up to K = 300 or so and by the
// FP32 matrix cores beyond.  Measured, us per step without a probe (which
// adds 0.5: its sum over the row tiles), before on the streamed kernels ->
// here: row-split schedule K = 128 4.5 -> 1.6, 256 6.1 -> 1.9, 512 (M = 256)
// 8.2 -> 4.1, 1024 (M = 100) 12.9 -> 6.9; column blocks (256, 256), M = 64
// 4.4 -> 2.1, (300, 200), M = 100 7.1 -> 2.5, (500, 1000), M = 100 32.7 ->
// 8.2; adjoint of 1000 steps, K = 512, M = 256 26.6 -> 20.8 ms.
#pragma once

#include <type_traits>

#include "k_split.h"

namespace rom {
namespace rsplit {

using namespace split;

enum Pol { kQuarters = 0, kPairs = 1 };
// kPlain; kTraced: also writes V (and, with a.str, S) after every step to
// the traces, entry 0 the state given; kAdjoint: the discrete adjoint of the
// step run backwards, with the fields (V, S) holding (P, Q), the operators
// packed as (Asv^T, Avs^T), the host passing c as the source vector and b as
// the probe, the amplitude 2 y read from a.ytr, iteration k taking step n =
// n0 + nsteps - 1 - k; it writes a.qtr[n - n0] = Q before and a.wtr[n - n0] =
// P after the P update and adds dt (b^T P) du/dmu(t_n) to a.dmu; kDual: two
// runs of one shape side by side, groups 0 .. G-1 traced, G .. 2G-1 adjoint
// (the recompute of a segment beside the reverse sweep of the next one).
enum Mode { kPlain = 0, kTraced = 1, kAdjoint = 2, kDual = 3 };

// one workgroup per CU, so that each XCD takes 32 of the 256
constexpr size_t kLdsR = 150 * 1024;
constexpr unsigned kNowhere = 0xF0000000u;     // past every buffer: loads give zeros

__device__ __forceinline__ f4 as_f4(u4 v) { return __builtin_bit_cast(f4, v); }

struct RArgs {
    SplitArgs s;
    int ks, kgv, kgs;           // Ks; k-groups (16 terms) of the V and S updates' reductions
    int np;                     // exchange words per column and buffer
    int kgpub;                  // k-groups that some workgroup owns (the terms behind them are zero)
};

// The run of row tile r of group g.
template <int POL, int NCH, int NRB, int NCB, int MODE>
__device__ __forceinline__ void run_rsplit(const RArgs &ra, int g, int r, unsigned char *smem, double *uwin) {
    constexpr int NC = 16 * NCB, RT = 16 * NRB;
    constexpr int TPC = kThreads / NC, RPT = NRB * NCB;
    constexpr int JL = RPT < 4 ? RPT : 4, QL = RPT / JL, JB = 4 / JL, QB = 4 / QL;
    constexpr int LDQ = RT + 2, LDP = RT + 4;  // LDS column strides (doubles; floats)
    // chains of a field in LDS; with room for both fields' a half-step needs
    // one workgroup barrier, else a second one before the next one's chains
    constexpr size_t kPart = POL == kQuarters ? sizeof(double) * kWaves * NC * LDQ : sizeof(float) * 8 * NCH * NC * LDP;
    constexpr bool kTwo = 2 * kPart <= kLdsR;
    const SplitArgs &a = ra.s;
    const int R = a.R;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kv = a.kv, ks = ra.ks, M = a.M, col0 = g * NC;
    xch::Wait wait{a.status, a.spin_max, a.forced, false};
    float *const xg = a.x + (size_t)g * NC * ra.np;
    u64 *const yg = a.yp + (size_t)g * xch::kRing * R * NC;

    // k-group q of this wave's chain i in a reduction of kg k-groups, or -1
    auto kgroup = [&](int kg, int i, int q) {
        if constexpr (POL == kQuarters) {
            const int n = kg >> 2, o = 4 * i + q;
            return o < n ? w * n + o : -1;
        } else {
            const int o = 4 * (w + kWaves * i) + q;
            return o < kg ? o : -1;
        }
    };

    // operator rows (16-row tiles NRB r ..), registers for the whole run
    u4 ov[NCH][4][NRB], os[NCH][4][NRB];
#pragma unroll
    for (int i = 0; i < NCH; ++i)
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < NRB; ++t) {
                const int tile = NRB * r + t;
                const int kv_ = kgroup(ra.kgv, i, q), ks_ = kgroup(ra.kgs, i, q);
                const u4 z = {0u, 0u, 0u, 0u};
                ov[i][q][t] = kv_ >= 0 && 16 * tile < kv
                                  ? a.opv[(((size_t)(tile >> 2) * ra.kgv + kv_) * 4 + (tile & 3)) * 64 + lane] : z;
                os[i][q][t] = ks_ >= 0 && 16 * tile < ks
                                  ? a.ops[(((size_t)(tile >> 2) * ra.kgs + ks_) * 4 + (tile & 3)) * 64 + lane] : z;
            }

    // finishing thread: column fj, rows 16 kgl + 4 j + q' of the tile with
    // JL values of j and QL of q', so that the entries of one q' are
    // neighbouring terms of one lane's fragment
    const int fj = tid / TPC, fs = tid % TPC;
    const int kgl = fs / (JB * QB), jb = fs % JB, qb = (fs % (JB * QB)) / JB;
    const int fr = r * RT + 16 * kgl + 4 * jb * JL + qb * QL;      // row of entry 0
    auto frow = [&](int e) { return 4 * (e % JL) + e / JL; };       // further rows
    const int lrow = fr - r * RT;
    const int fm = col0 + fj;
    const bool fok = fm < M;
    const double dt = a.dt;
    const bool probe = a.c != nullptr;
    const int rp = (kv + RT - 1) / RT;         // row tiles with rows of V
    float sh[2][RPT], sl[2][RPT];
    double bb[RPT], cc[RPT];
#pragma unroll
    for (int e = 0; e < RPT; ++e) {
        const int row = fr + frow(e);
        sh[0][e] = (fok && row < kv) ? a.V[(size_t)fm * kv + row] : 0.f;
        sh[1][e] = (fok && row < ks) ? a.S[(size_t)fm * ks + row] : 0.f;
        sl[0][e] = sl[1][e] = 0.f;
        bb[e] = row < kv ? (double)a.b[row] : 0.0;
        cc[e] = (probe && row < kv) ? (double)a.c[row] : 0.0;
    }

    int64_t q = 0, ny = 0;                     // phase, probe row to publish next
    const size_t xo = ((size_t)((fr >> 4) * NCB + fj / 16) * 64 + 16 * qb * QL + (fj & 15)) * 4 + jb * JL;
    auto publish = [&](int f) {
        // a tile row past the padded rows of the other field's reduction is not read
        if ((fr >> 4) >= (f == 0 ? ra.kgs : ra.kgv)) {
            ++q;
            return;
        }
        float *d = xg + (size_t)(q & 3) * a.xfloats + xo, *z = xg + (size_t)((q + 2) & 3) * a.xfloats + xo;
        constexpr unsigned E = xch::kEmpty;
#pragma unroll
        for (int i = 0; i < QL; ++i) {
            unsigned v[4];
#pragma unroll
            for (int j = 0; j < JL; ++j) {
                const unsigned x = __builtin_bit_cast(unsigned, sh[f][i * JL + j]);
                v[j] = x == E ? 0x7FC00000u : x;
            }
            if constexpr (JL == 4) {
                *reinterpret_cast<u4 *>(d + 64 * i) = u4{v[0], v[1], v[2], v[3]};
                *reinterpret_cast<u4 *>(z + 64 * i) = u4{E, E, E, E};
            } else if constexpr (JL == 2) {
                *reinterpret_cast<u2 *>(d + 64 * i) = u2{v[0], v[1]};
                *reinterpret_cast<u2 *>(z + 64 * i) = u2{E, E};
            } else {
                *reinterpret_cast<unsigned *>(d + 64 * i) = v[0];
                *reinterpret_cast<unsigned *>(z + 64 * i) = E;
            }
        }
        ++q;
    };

    // ysum: where the last step's probe sum goes (row tile 0), or null
    auto half_step = [&](int f, const u4 (&op)[NCH][4][NRB], int kw, bool last, double *ysum) -> double {
        const u64 *yp = yg + (size_t)((ny - 1) & 3) * R * NC + fj;
        ProbeSum<TPC, POL == kPairs ? 4 / NRB : 0> ps;
        if (ysum) ps.load(yp, NC, rp, fs);
        const int kg = f == 0 ? ra.kgv : ra.kgs;
        // ---- the wave's terms of the other field, polled until complete
        uint64_t xa = reinterpret_cast<uint64_t>(xg + (size_t)((q - 1) & 3) * a.xfloats);
        asm volatile("" : "+s"(xa));
        const __amdgpu_buffer_rsrc_t rx = raw_buffer(reinterpret_cast<void *>(xa), (unsigned)kg * (NCB * 1024));
        const unsigned loff = 16u * (unsigned)lane;
        u4 bx[NCH][4][NCB];
        long spins = 0;
        for (;;) {
#pragma unroll
            for (int i = 0; i < NCH; ++i)
#pragma unroll
                for (int p = 0; p < 4; ++p) {
                    const int k = kgroup(kg, i, p);
                    const unsigned lo = k >= 0 && k < ra.kgpub ? loff : kNowhere;
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
                        bx[i][p][cb] = __builtin_amdgcn_raw_buffer_load_b128(rx, lo, (k * NCB + cb) * 1024, kDeviceScope);
                }
            unsigned m = 0;
#pragma unroll
            for (int i = 0; i < NCH; ++i)
#pragma unroll
                for (int p = 0; p < 4; ++p)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) {
                        const u4 &v = bx[i][p][cb];
                        m = xch::max3u(xch::max3u(m, v[0], v[1]), v[2], v[3]);
                    }
            if (wait.dead || (!wait.forced && __ballot(m == xch::kEmpty) == 0)) break;
            if (wait.give_up(spins)) break;
        }
        // (the emptied slots of the last publication: before the next one)
        xch::publish_fence();
        if (ysum) *ysum = ps.sum(wait, yp, NC, rp, fs);
        // ---- chains, to LDS
        unsigned char *part = smem + (kTwo ? f * kPart : 0);
        double *pq = reinterpret_cast<double *>(part);       // quarters: [wave][col][LDQ]
        float *pp = reinterpret_cast<float *>(part);         // pairs: [block][parity][col][LDP]
        double acc[NRB][NCB][4];
        if constexpr (POL == kQuarters) {
#pragma unroll
            for (int t = 0; t < NRB; ++t)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[t][cb][v] = 0.0;
        }
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            if (kgroup(kg, i, 0) < 0) continue;
            f4 c[POL == kPairs ? 2 : 1][NRB][NCB];
#pragma unroll
            for (int h = 0; h < (POL == kPairs ? 2 : 1); ++h)
#pragma unroll
                for (int t = 0; t < NRB; ++t)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb) c[h][t][cb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                // (a block of 64 terms is whole; a quarter may end inside one)
                if (POL == kQuarters && p > 0 && kgroup(kg, i, p) < 0) break;
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int t = 0; t < NRB; ++t)
#pragma unroll
                        for (int cb = 0; cb < NCB; ++cb) {
                            f4 &d = c[POL == kPairs ? (j & 1) : 0][t][cb];
                            d = __builtin_amdgcn_mfma_f32_16x16x4f32(as_f4(op[i][p][t])[j], as_f4(bx[i][p][cb])[j], d,
                                                                     0, 0, 0);
                        }
            }
            if constexpr (POL == kQuarters) {
#pragma unroll
                for (int t = 0; t < NRB; ++t)
#pragma unroll
                    for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[t][cb][v] += (double)c[0][t][cb][v];
            } else {
                float *d = pp + (size_t)(w + kWaves * i) * 2 * NC * LDP;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int t = 0; t < NRB; ++t)
#pragma unroll
                        for (int cb = 0; cb < NCB; ++cb)
                            *reinterpret_cast<f4 *>(d + (h * NC + 16 * cb + (lane & 15)) * LDP + 16 * t +
                                                    4 * (lane >> 4)) = c[h][t][cb];
            }
        }
        if constexpr (POL == kQuarters) {
#pragma unroll
            for (int t = 0; t < NRB; ++t)
#pragma unroll
                for (int cb = 0; cb < NCB; ++cb) {
                    double *d = pq + (size_t)(w * NC + 16 * cb + (lane & 15)) * LDQ + 16 * t + 4 * (lane >> 4);
#pragma unroll
                    for (int v = 0; v < 4; ++v) d[v] = acc[t][cb][v];
                }
        }
        __syncthreads();
        // ---- finish
        const double u = f == 0 ? uwin[kw * NC + fj] : 0.0;
        double yt[RPT];
#pragma unroll
        for (int e = 0; e < RPT; ++e) {
            const int i = lrow + frow(e);
            double inc = 0.0;
            if constexpr (POL == kQuarters) {
                const double *d = pq + (size_t)fj * LDQ + i;
                inc = (d[0] + d[NC * LDQ]) + (d[2 * NC * LDQ] + d[3 * NC * LDQ]);
            } else {
                const float *d = pp + (size_t)fj * LDP + i;
#pragma unroll
                for (int p = 0; p < 4 * NCH; ++p)
                    if (4 * p < kg) {
                        inc += (double)d[(size_t)(2 * p) * NC * LDP];
                        inc += (double)d[(size_t)(2 * p + 1) * NC * LDP];
                    }
            }
            if (f == 0) inc = fma(bb[e], u, inc);
            const double yv = fma(dt, inc, (double)sh[f][e] + (double)sl[f][e]);
            const float hv = (float)yv;
            sh[f][e] = hv;
            sl[f][e] = (float)(yv - (double)hv);
            yt[e] = f == 0 ? cc[e] * yv : 0.0;
        }
        if (!last) publish(f);
        if constexpr (!kTwo) __syncthreads();
        // the column's probe sum over this row tile, in the order of the
        // schedule (an adjoint's amplitude, hence its rounding, follows from
        // it), the row being 16 kgl + 4 j + q'.  kQuarters: per q' the four j
        // in sequence, then binary trees over q' and the 16-row tiles.
        // kPairs: per j the four q' in sequence, handed on from lane to
        // lane, then binary trees over j and the 16-row
        // tiles up to 64 rows; the sums of up to four 64-row tiles are added
        // in sequence (more, and a column-block wave chains through two
        // tiles: those sums agree to rounding only).  The total is in the
        // last of the column's threads.
        if (f != 0 || !probe) return 0.0;
        if constexpr (POL == kPairs) {
            double t[JL];
#pragma unroll
            for (int j = 0; j < JL; ++j) {
                auto chain = [&](double in) {
#pragma unroll
                    for (int i = 0; i < QL; ++i) in += yt[i * JL + j];
                    return in;
                };
                t[j] = chain(0.0);
#pragma unroll
                for (int i = 1; i < QB; ++i) {
                    const double in = lane::dpp_mov64<0x110 + JB>(t[j]);      // row_shr:JB
                    t[j] = chain(qb == 0 ? 0.0 : in);
                }
            }
            double y = t[0];
            if constexpr (JL == 2) y = t[0] + t[1];
            if constexpr (JL == 4) y = (t[0] + t[1]) + (t[2] + t[3]);
            if constexpr (JB >= 2) y += lane::dpp_mov64<lane::kDppXor1>(y);
            if constexpr (JB >= 4) y += lane::dpp_mov64<lane::kDppXor2>(y);
            if constexpr (JB == 1 && QB == 4) y = lane::dpp_mov64<0xFF>(y);   // quad_perm: lane 3
            if constexpr (JB == 1 && QB == 2) y = lane::dpp_mov64<0xF5>(y);   // quad_perm: lanes 1 1 3 3
            return column_sum<TPC, JB * QB == 16 ? 4 : JB * QB == 8 ? 3 : JB * QB == 4 ? 2 : JB * QB == 2 ? 1 : 0>(y);
        }
        double ypart = 0.0;
#pragma unroll
        for (int i = 0; i < QL; ++i) {
            double t;
            if constexpr (JL == 4) {
                t = ((yt[4 * i] + yt[4 * i + 1]) + yt[4 * i + 2]) + yt[4 * i + 3];
            } else if constexpr (JL == 2) {
                const double o0 = lane::dpp_mov64<lane::kDppXor1>(yt[0]), o1 = lane::dpp_mov64<lane::kDppXor1>(yt[1]);
                const bool hi = (fs & 1) != 0;
                t = (((hi ? o0 : yt[0]) + (hi ? o1 : yt[1])) + (hi ? yt[0] : o0)) + (hi ? yt[1] : o1);
            } else {
                t = ((lane::dpp_mov64<0x00>(yt[0]) + lane::dpp_mov64<0x55>(yt[0])) + lane::dpp_mov64<0xAA>(yt[0])) +
                    lane::dpp_mov64<0xFF>(yt[0]);                 // quad_perm: the quad's lanes 0, 1, 2, 3
            }
            ypart = i == 0 ? t : ypart + t;
        }
        return column_sum<TPC, JL == 4 ? 0 : (JL == 2 ? 1 : 2)>(ypart);
    };

    // this thread's rows of field f (hi + lo) into trace matrix tr (M x K per
    // entry), entry e
    auto trace = [&](float *tr, int f, int64_t e) {
        const int K = f == 0 ? kv : ks;
        float *d = tr + ((size_t)e * M + fm) * K;
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int row = fr + frow(i);
            if (fok && row < K) d[row] = sh[f][i] + sl[f][i];
        }
    };

    publish(1);
    if constexpr (MODE == kTraced) {
        trace(a.vtr, 0, 0);
        if (a.str) trace(a.str, 1, 0);
    }
    double Jacc = 0.0;
    const double muf = MODE == kAdjoint && fok ? a.mu[fm] : 1.0;
    // the probe sum of iteration k (row tile 0)
    auto probe_row = [&](int64_t k, double yv) {
        if (fs != 0 || !fok) return;
        if constexpr (MODE == kAdjoint) {
            Jacc += dt * yv * dev::forcing_dmu(a.source, (double)(a.n0 + a.nsteps - 1 - k) * dt, muf);
        } else {
            Jacc += dt * (yv * yv);
            if (a.y) a.y[(size_t)k * M + fm] = yv;
        }
    };
    const bool sums = probe && r == 0;
    for (int64_t k = 0; k < a.nsteps; ++k) {
        const int64_t n = MODE == kAdjoint ? a.n0 + a.nsteps - 1 - k : a.n0 + k;     // step
        // (read in the velocity half-step, after its barrier; the last reads
        // of the previous window lie before the stress half-step's)
        if (k % kUWin == 0) {
            if constexpr (MODE == kAdjoint)
                adjoint_window<NC>(uwin, a.ytr, a.nsteps - 1 - k, col0, M);
            else
                forcing_window<NC>(uwin, a.source, a.n0 + k, dt, a.mu, col0, M);
        }
        if constexpr (MODE == kAdjoint) trace(a.qtr, 1, n - a.n0);   // Q^{n+1}
        double ysum = 0.0;
        const double yp = half_step(0, ov, (int)(k % kUWin), false, sums && k > 0 ? &ysum : nullptr);
        if (sums && k > 0) probe_row(k - 1, ysum);
        if constexpr (MODE == kTraced) trace(a.vtr, 0, k + 1);
        if constexpr (MODE == kAdjoint) trace(a.wtr, 0, n - a.n0);   // w^n
        if (probe) {
            // a ring entry per step: row tile 0 reads entry k before it
            // publishes the velocity of step k + 1, so whoever publishes that
            // of step k + 2 may empty it
            if (fs == TPC - 1) {
                xch::put64(yg + ((size_t)(ny & 3) * R + r) * NC + fj, yp);
                xch::clear64(yg + ((size_t)((ny + 2) & 3) * R + r) * NC + fj);
            }
            ++ny;
        }
        half_step(1, os, 0, k + 1 == a.nsteps, nullptr);
        if constexpr (MODE == kTraced) {
            if (a.str) trace(a.str, 1, k + 1);
        }
    }
    if (sums) {
        ProbeSum<TPC, POL == kPairs ? 4 / NRB : 0> ps;
        const u64 *yp = yg + (size_t)((ny - 1) & 3) * R * NC + fj;
        ps.load(yp, NC, rp, fs);
        probe_row(a.nsteps - 1, ps.sum(wait, yp, NC, rp, fs));
    }
    auto finish = [&](const auto &z, int zkv, int zks) {
#pragma unroll
        for (int e = 0; e < RPT; ++e) {
            const int row = fr + frow(e);
            if (fok && row < zkv) z.V[(size_t)fm * zkv + row] = sh[0][e] + sl[0][e];
            if (fok && row < zks) z.S[(size_t)fm * zks + row] = sh[1][e] + sl[1][e];
        }
        double *sum = MODE == kAdjoint ? z.dmu : z.J;
        if (probe && sum && r == 0 && fs == 0 && fok) sum[fm] += Jacc;
    };
    if constexpr (POL == kPairs) {             // these runs can be repeated
        const auto &z = xch::args_here<RArgs>();
        if (!xch::agree(z.s.done + 2 * g, z.s.R, 0, wait)) return;
        finish(z.s, z.s.kv, z.ks);
    } else {
        finish(a, kv, ks);
    }
}

template <int POL, int NCH, int NRB, int NCB, int MODE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
void rank2_rsplit_kernel(RArgs a0, RArgs a1) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double uwin[kUWin * 16 * NCB];
    const int code = take_slot(a0.s.slots);
    const int xcc = code & 7, s = code >> 3;
    const int r = s % a0.s.R, g = (s / a0.s.R) * 8 + xcc;
    if constexpr (MODE == kDual) {
        if (g < a0.s.G)
            run_rsplit<POL, NCH, NRB, NCB, kTraced>(a0, g, r, smem, uwin);
        else if (g < 2 * a0.s.G)
            run_rsplit<POL, NCH, NRB, NCB, kAdjoint>(a1, g - a0.s.G, r, smem, uwin);
    } else {
        if (g < a0.s.G) run_rsplit<POL, NCH, NRB, NCB, MODE>(a0, g, r, smem, uwin);
    }
}

// Tiles (NCH, NRB, NCB).  NCH = 3, 4 take 32 rows (16 rows would need more
// than 32 workgroups per group, 64 more registers).
// us: a step of the largest K of the class with a probe, measured on kPairs
// (kQuarters, which folds its chains in registers, takes 0.2 to 1 less); 64
// rows less take 3 to 5 % less.
struct Tile {
    int nch, nrb, ncb;
    float us;
    const void *f[4];          // by Mode (kPairs: plain and traced runs only)
};
#define ROM_RK(P, C, B, N, MODE) (const void *)rank2_rsplit_kernel<P, C, B, N, MODE>
#define ROM_RT_kQuarters(C, B, N, US)                                                                               \
    {C, B, N, US, {ROM_RK(kQuarters, C, B, N, kPlain), ROM_RK(kQuarters, C, B, N, kTraced),                         \
                   ROM_RK(kQuarters, C, B, N, kAdjoint), ROM_RK(kQuarters, C, B, N, kDual)}}
#define ROM_RT_kPairs(C, B, N, US)                                                                                  \
    {C, B, N, US, {ROM_RK(kPairs, C, B, N, kPlain), ROM_RK(kPairs, C, B, N, kTraced), nullptr, nullptr}}
// Left out are tiles that no run takes: 64 x 16 and 16 x 32 where others of
// their area hold as many samples, and for kPairs those of one chain that are
// slower than the column blocks (32 x 32: 6.0 against 4.6).
constexpr int kQuarterCount = 12, kPairCount = 10;
#define ROM_RT_LONG(P)                                                                                              \
    ROM_RT_##P(2, 1, 1, 3.9f), ROM_RT_##P(2, 2, 1, 5.7f), ROM_RT_##P(2, 2, 2, 10.2f), ROM_RT_##P(2, 4, 1, 10.4f),    \
        ROM_RT_##P(3, 2, 1, 8.0f), ROM_RT_##P(3, 2, 2, 15.2f), ROM_RT_##P(4, 2, 1, 10.3f), ROM_RT_##P(4, 2, 2, 20.8f)
extern const Tile kQuarterTiles[kQuarterCount], kPairTiles[kPairCount];

}  // namespace rsplit
}  // namespace rom
