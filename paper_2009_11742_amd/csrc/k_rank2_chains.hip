// Rank-2 leapfrog stepper, FP32 operators and states, small models of any
// pair (Avs, Asv): one or four samples per workgroup, both operators in its
// registers for the whole run, the sums of the column blocks
// (k_rank2_f32.hip) bit for bit.
//
// The column blocks' sum of a row is, for each 64 terms, two FP32 chains of
// fused multiply-adds (the even and the odd groups of four terms), all chains
// folded in order into one FP64 sum.  Up to 256 terms and 4 samples they are
// bound by the length of those chains: one wave runs all of a 64-row tile's,
// the other waves of the workgroup idle.  Here
// every chain of 32 terms has its own lanes: a DPP row (16 lanes) takes one
// chain of 16 operator rows, its 32 state terms lie in two registers across
// the same lanes and reach the multiply-adds as DPP row broadcasts, so a
// half-step reads two LDS words per lane and chain.  The chains of a row meet
// in registers (v_permlane16_swap, v_permlane32_swap), every lane of the row
// finishes it in FP64, and one barrier ends the half-step.
//
// C = 2 or 4 DPP rows share 16 operator rows; each lane has L = 2 NB / C
// chains (NB blocks of 64 terms) of 32 operator registers.  C = 4 where that
// gives a workgroup at most 8 waves.  One more wave sums the probe of the
// step while the others are in the stress half-step (k_rank2_f32.hip's order:
// four rows in sequence, a tree over the 16 such groups of a 64-row tile, the
// tiles in sequence), except where the operators take too many registers for
// a ninth wave; there the last waves do it.
//
// Bound by the multiply-adds with a DPP broadcast, 8 cycles each (16 for the
// 4 x 4 matrix blocks), from K = 128 on, below by the half-step's serial path
// (LDS, 32 multiply-adds, swaps, FP64 sum, LDS, barrier: 0.2 us).  Measured,
// us per step, column blocks -> here: (30, 28), M = 1 1.7 -> 0.39; K = 64,
// M = 256 1.7 -> 0.46, M = 1000 1.7 -> 0.70; K = 128, M = 256 2.3 -> 0.74,
// M = 1000 2.4 -> 0.91; (150, 130), M = 256 3.1 -> 1.25; (128, 256), M =
// 1022 3.5 -> 1.75.
#include "k_common.h"
#include "k_lane.h"
#include "rom_internal.h"

namespace rom {
namespace {

using dev::f4;

enum Mode { kPlain = 0, kTraced = 1, kAdjoint = 2 };

constexpr int kMaxK = 256;
// Samples up to which each has a workgroup of its own: one per CU.  Four per
// workgroup take the matrix cores' 4 x 4 blocks, which do four samples in the
// time of two broadcast multiply-adds, so that a second workgroup on a CU
// never pays (K = 128: 0.75 us per step one sample each, 0.9 four; 512
// samples 1.2 one each).  Two launches side by side share the CUs.
constexpr int kOneSample = 256;
constexpr int kWin = 64;           // steps per source window
constexpr int kBlk = 80;           // LDS words per 64-term block (banks of two blocks' rows apart)

// DPP rows per 16 operator rows for a sum of nb blocks over rb 64-row tiles
constexpr int dpp_rows(int nb, int rb) { return (nb == 2 && rb <= 2) || nb == 4 ? 4 : 2; }
constexpr int waves_of(int nb, int rb) { return rb * dpp_rows(nb, rb); }

// A kernel for Kv_pad = 64 A, Ks_pad = 64 B.
template <int A, int B>
struct Shape {
    static constexpr int CV = dpp_rows(B, A), CS = dpp_rows(A, B);
    static constexpr int LV = 2 * B / CV, LS = 2 * A / CS;
    static constexpr int W = waves_of(B, A) > waves_of(A, B) ? waves_of(B, A) : waves_of(A, B);
    // a wave for the probe: 9 waves leave 168 registers per lane
    static constexpr bool kProbeWave = W < 8 || LV + LS <= 2;
    static constexpr int kThreads = 64 * (W + (kProbeWave ? 1 : 0));
};

// LDS word of term k of sample s.  One sample: a chain's 32 terms in order
// (word 16 t + i of a chain goes to lane i, register t); four: the chain's
// terms 4 g + e at 8 e + g, so that lane 4 e + s reads its eight words in two
// loads, and the samples' words in banks of their own.
template <int NS>
__device__ __forceinline__ int word_of(int k, int s, int ldx) {
    const int b = k >> 6, h = (k >> 2) & 1, g = (k >> 3) & 7, e = k & 3;
    return NS == 1 ? b * kBlk + 32 * h + 4 * g + e
                   : s * ldx + 32 * (s >> 1) + 4 * (s & 1) + 64 * b + 32 * h + 8 * e + g;
}

// acc = fma(op[base + n], lane n of the DPP row's x, acc), n = 0 .. 15.  (The
// compiler keeps broadcast and multiply-add apart, twice the instructions.
// The waits cover a DPP read of a register just written, ahead, and a lane
// swap of the result, behind.)
__device__ __forceinline__ void chain16(const float (&op)[32], int base, float x, float &acc) {
    asm("s_nop 1\n"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %10 row_newbcast:8 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %12 row_newbcast:10 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %13 row_newbcast:11 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %14 row_newbcast:12 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %15 row_newbcast:13 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %16 row_newbcast:14 row_mask:0xf bank_mask:0xf\n"
        "v_fmac_f32_dpp %0, %1, %17 row_newbcast:15 row_mask:0xf bank_mask:0xf\n"
        "s_nop 1"
        : "+v"(acc)
        : "v"(x), "v"(op[base + 0]), "v"(op[base + 1]), "v"(op[base + 2]), "v"(op[base + 3]), "v"(op[base + 4]), 
          "v"(op[base + 5]), "v"(op[base + 6]), "v"(op[base + 7]), "v"(op[base + 8]), "v"(op[base + 9]), "v"(op[base + 10]), 
          "v"(op[base + 11]), "v"(op[base + 12]), "v"(op[base + 13]), "v"(op[base + 14]), "v"(op[base + 15]));
}

// This lane's part of the operator (packed as launch_pack_f32): the chains l
// of row `row`, terms in order; zero behind the rows of the operator.
template <int C, int L>
__device__ __forceinline__ void load_op(float (&op)[L][32], const f4 *pk, int row, int rowsp, int kp, int q) {
    const f4 *p = pk + ((size_t)(row >> 6) * (kp >> 2)) * 64 + (row & 63);
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const int b = C == 2 ? l : (q >> 1) + 2 * l;
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const f4 v = row < rowsp ? p[(size_t)(16 * b + 2 * g + (q & 1)) * 64] : f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) op[l][4 * g + e] = v[e];
        }
    }
}

// x of the lower and the upper of two neighbouring DPP rows (halves of the
// wave), in both.
template <bool W32>
__device__ __forceinline__ void row_pair(float &x, float &hi) {
    const unsigned a = lane::fbits(x);
    const auto r = W32 ? __builtin_amdgcn_permlane32_swap(a, a, false, false)
                       : __builtin_amdgcn_permlane16_swap(a, a, false, false);
    x = lane::bitsf(r[0]);
    hi = lane::bitsf(r[1]);
}

// Row sum of one half-step: x the other field's LDS words, i the lane in its
// DPP row, q the DPP row's number among its C.
template <int C, int L>
__device__ __forceinline__ double row_sum(const float (&op)[L][32], const float *x, int i, int q) {
    float acc[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const int b = C == 2 ? l : (q >> 1) + 2 * l;
        const float *xp = x + b * kBlk + (q & 1) * 32 + i;
        const float x0 = xp[0], x1 = xp[16];
        acc[l] = 0.f;
        chain16(op[l], 0, x0, acc[l]);
        chain16(op[l], 16, x1, acc[l]);
    }
    double inc = 0.0;
#pragma unroll
    for (int l = 0; l < L; ++l) {
        float c0 = acc[l], c1;
        row_pair<false>(c0, c1);
        if constexpr (C == 2) {
            inc += (double)c0;
            inc += (double)c1;
        } else {
            float c2, c3;
            row_pair<true>(c0, c2);
            row_pair<true>(c1, c3);
            inc += (double)c0;
            inc += (double)c1;
            inc += (double)c2;
            inc += (double)c3;
        }
    }
    return inc;
}

// a, b: their lower and upper DPP rows (halves) exchanged, so that a lane of
// a lower row holds its a of both rows, one of an upper row its b.
template <bool W32>
__device__ __forceinline__ void exchange_rows(float &a, float &b) {
    const auto r = W32 ? __builtin_amdgcn_permlane32_swap(lane::fbits(a), lane::fbits(b), false, false)
                       : __builtin_amdgcn_permlane16_swap(lane::fbits(a), lane::fbits(b), false, false);
    a = lane::bitsf(r[0]);
    b = lane::bitsf(r[1]);
}

// The same for four samples on v_mfma_f32_4x4x1f32 (16 blocks of 4 x 4, one
// term; here rows the samples, columns four operator rows).  Its A operand
// can be one block's for all four blocks of a DPP row: lane 4 e + s holds
// term e of four of sample s, and four instructions take block 0, 1, 2, 3.
// Lane i then has operator row i's chain of sample r in register r; each lane
// keeps the sums inc[e], e < 4 / C, of samples (4 / C) q + e.
__device__ __forceinline__ f4 chain32(const float (&op)[32], const f4 &xa, const f4 &xb) {
    f4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int g = 0; g < 8; ++g) {
        const float x = g < 4 ? xa[g & 3] : xb[g & 3];
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, op[4 * g], acc, 2, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, op[4 * g + 1], acc, 2, 1, 0);
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, op[4 * g + 2], acc, 2, 2, 0);
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, op[4 * g + 3], acc, 2, 3, 0);
    }
    return acc;
}

template <int C, int L, int LDX>
__device__ __forceinline__ void row_sums4(const float (&op)[L][32], const float *x, int i, int q,
                                          double (&inc)[4 / C]) {
    const float *xp = x + word_of<4>(i >> 2, i & 3, LDX) + 32 * (q & 1);
    f4 xa[L], xb[L];
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const int b = C == 2 ? l : (q >> 1) + 2 * l;
        xa[l] = *reinterpret_cast<const f4 *>(xp + 64 * b);
        xb[l] = *reinterpret_cast<const f4 *>(xp + 64 * b + 4);
    }
#pragma unroll
    for (int e = 0; e < 4 / C; ++e) inc[e] = 0.0;
#pragma unroll
    for (int l = 0; l < L; ++l) {
        const f4 acc = chain32(op[l], xa[l], xb[l]);
        float r[4] = {acc[0], acc[1], acc[2], acc[3]};
        if constexpr (C == 2) {
            exchange_rows<false>(r[0], r[2]);
            exchange_rows<false>(r[1], r[3]);
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                inc[e] += (double)r[e];
                inc[e] += (double)r[e + 2];
            }
        } else {
            exchange_rows<false>(r[0], r[1]);
            exchange_rows<false>(r[2], r[3]);
            exchange_rows<true>(r[0], r[2]);
            exchange_rows<true>(r[1], r[3]);
#pragma unroll
            for (int c = 0; c < 4; ++c) inc[0] += (double)r[c];
        }
    }
}

// row_pair for FP64 values.
template <bool W32>
__device__ __forceinline__ void row_pair(double &x, double &hi) {
    const uint64_t b = __builtin_bit_cast(uint64_t, x);
    float l0 = lane::bitsf((unsigned)b), h0 = lane::bitsf((unsigned)(b >> 32)), l1, h1;
    row_pair<W32>(l0, l1);
    row_pair<W32>(h0, h1);
    x = __builtin_bit_cast(double, ((uint64_t)lane::fbits(h0) << 32) | lane::fbits(l0));
    hi = __builtin_bit_cast(double, ((uint64_t)lane::fbits(h1) << 32) | lane::fbits(l1));
}

// Probe sums of a step: pb the NS samples' products, tile rows in order.  A
// DPP row takes one 64-row tile of one sample, so a pass over the wave takes
// four samples of one tile, two of two or one of more.  DPP row dr keeps the
// sum of sample probe_sample(dr), taken in pass probe_pass(dr).
template <int A, int NS>
constexpr int kPasses = NS == 1 || A == 1 ? 1 : A == 2 ? 2 : 4;

template <int A, int NS>
__device__ __forceinline__ int probe_sample(int dr) {
    return NS == 1 ? 0 : A == 2 ? 2 * (dr & 1) + (dr >> 1) : dr;
}

template <int A, int NS>
__device__ __forceinline__ int probe_pass(int dr) {
    return kPasses<A, NS> == 1 ? 0 : A == 2 ? dr & 1 : dr;
}

template <int A, int NS>
__device__ __forceinline__ double probe_sum(const double (*pb)[64 * A], int pass, int i, int dr) {
    const int s = NS == 1 ? 0 : A == 1 ? dr : A == 2 ? 2 * pass + (dr >> 1) : pass;
    const int t = A == 1 ? 0 : A == 2 ? dr & 1 : min(dr, A - 1);
    const double *p = &pb[s][64 * t + 4 * i];
    double v = ((p[0] + p[1]) + p[2]) + p[3];
    v += lane::dpp_mov64<lane::kDppXor1>(v);
    v += lane::dpp_mov64<lane::kDppXor2>(v);
    v += lane::dpp_mov64<lane::kDppHalfMirror>(v);
    v += lane::dpp_mov64<lane::kDppRor8>(v);
    double y = 0.0;
    if constexpr (A == 1) {
        y += v;
    } else {
        double t1;
        row_pair<false>(v, t1);
        if constexpr (A == 2) {
            y += v;
            y += t1;
        } else {
            double t2, t3;
            row_pair<true>(v, t2);
            row_pair<true>(t1, t3);
            y += v;
            y += t1;
            y += t2;
            if constexpr (A == 4) y += t3;
        }
    }
    return y;
}

// (double)x, converted where it is used: held across the loop in 64 bits, the
// source and probe entries would spill.
__device__ __forceinline__ double widen(float x) {
    asm volatile("" : "+v"(x));
    return (double)x;
}

template <int A, int B, int NS, int MODE>
__global__ __launch_bounds__((Shape<A, B>::kThreads))
void rank2_chains_kernel(Rank2Args a) {
    using T = Shape<A, B>;
    constexpr int LDX = (NS == 4 ? 64 : kBlk) * (A > B ? A : B);
    constexpr int EV = NS == 4 ? 4 / T::CV : 1, ES = NS == 4 ? 4 / T::CS : 1;   // a lane's samples
    __shared__ __align__(16) float xs[2][NS * LDX + (NS == 4 ? 64 : 0)];   // V, S (rounded to FP32)
    __shared__ __align__(16) double pb[NS][64 * A];       // probe products of V's rows
    __shared__ double uw[NS][kWin], dw[MODE == kAdjoint ? NS : 1][kWin];   // source amplitude, du/dmu
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nt = blockDim.x, nw = nt >> 6;
    const int i = lane & 15, dr = lane >> 4;
    const int kv = a.kv, ks = a.ks, M = a.M, m0 = blockIdx.x * NS;
    const double dt = a.dt;
    const float *src = static_cast<const float *>(MODE == kAdjoint ? a.c : a.b);
    const float *prb = static_cast<const float *>(MODE == kAdjoint ? a.b : a.c);
    const bool probe = prb != nullptr;
    const int qv = dr % T::CV, qs = dr % T::CS;
    const int rv = w * (64 / T::CV) + (dr / T::CV) * 16 + i, rs = w * (64 / T::CS) + (dr / T::CS) * 16 + i;
    // (whole waves behind the last row skip its half-step)
    const bool wv = w * (64 / T::CV) < kv, ws = w * (64 / T::CS) < ks;
    // with one sample all C rows' lanes finish the same row
    const int sv = NS == 4 ? EV * qv : 0, ss = NS == 4 ? ES * qs : 0;
    const bool okv = rv < kv && (NS == 4 || qv == 0), oks = rs < ks && (NS == 4 || qs == 0);

    float opv[T::LV][32], ops[T::LS][32];
    load_op<T::CV, T::LV>(opv, static_cast<const f4 *>(a.avs), rv, a.kvp, a.ksp, qv);
    load_op<T::CS, T::LS>(ops, static_cast<const f4 *>(a.asv), rs, a.ksp, a.kvp, qs);
    for (int k = tid; k < (int)(sizeof(xs) / sizeof(float)); k += nt) xs[0][k] = 0.f;
    for (int k = tid; k < NS * 64 * A; k += nt) pb[0][k] = 0.0;
    const float bb = rv < kv && src ? src[rv] : 0.f, cc = rv < kv && prb ? prb[rv] : 0.f;
    // the states, hi + lo: (float)v64 is the rounded sum that is stored, not
    // always the hi of the pair
    double v64[EV], s64[ES];
    int xv[EV], xw[ES];                                   // LDS words
    __syncthreads();
#pragma unroll
    for (int e = 0; e < EV; ++e) {
        const int m = m0 + sv + e;
        const float h = rv < kv && m < M ? static_cast<const float *>(a.V)[(size_t)m * kv + rv] : 0.f;
        v64[e] = (double)h;
        xv[e] = word_of<NS>(rv, sv + e, LDX);
        if (okv) xs[0][xv[e]] = h;
    }
#pragma unroll
    for (int e = 0; e < ES; ++e) {
        const int m = m0 + ss + e;
        const float h = rs < ks && m < M ? static_cast<const float *>(a.S)[(size_t)m * ks + rs] : 0.f;
        s64[e] = (double)h;
        xw[e] = word_of<NS>(rs, ss + e, LDX);
        if (oks) xs[1][xw[e]] = h;
    }
    // (the operators' loads are waited for here, not in the loop)
    __builtin_amdgcn_s_waitcnt(dev::kWaitVm0);
    __syncthreads();
    // the probe: the last wave, or with no wave of its own the last ones, a
    // pass each
    constexpr int P = kPasses<A, NS>;
    const int pw = nw - 1 - w;
    const bool pwave = probe && pw < (T::kProbeWave ? 1 : P);
    const int pm = m0 + probe_sample<A, NS>(dr);          // the sample of this lane's J
    const bool pok = i == 0 && pm < M && (NS == 4 || dr == 0) && (T::kProbeWave || probe_pass<A, NS>(dr) == pw);
    double Jacc = 0.0;

    auto store_v = [&](float *d) {
#pragma unroll
        for (int e = 0; e < EV; ++e)
            if (okv && m0 + sv + e < M) d[(size_t)(m0 + sv + e) * kv + rv] = (float)v64[e];
    };
    auto store_s = [&](float *d) {
#pragma unroll
        for (int e = 0; e < ES; ++e)
            if (oks && m0 + ss + e < M) d[(size_t)(m0 + ss + e) * ks + rs] = (float)s64[e];
    };
    if constexpr (MODE == kTraced) {
        store_v(a.vtr);
        if (a.str) store_s(a.str);
    }

    double un[EV];                                        // the next step's amplitudes
    auto amplitudes = [&](int j) {
#pragma unroll
        for (int e = 0; e < EV; ++e) un[e] = uw[sv + e][j];
    };
    for (int64_t k = 0; k < a.nsteps; ++k) {
        const int64_t n = MODE == kAdjoint ? a.n0 + a.nsteps - 1 - k : a.n0 + k;
        const int kw = (int)(k % kWin);
        if (kw == 0) {
            // (the last reads of the window before lie in front of the last
            // barrier)
            for (int idx = tid; idx < NS * kWin; idx += nt) {
                const int s = idx / kWin, j = idx % kWin, q = m0 + s;
                double u = 0.0, d = 0.0;
                if (q < M && k + j < a.nsteps) {
                    if constexpr (MODE == kAdjoint) {
                        u = 2.0 * a.ytr[(size_t)(n - a.n0 - j) * M + q];
                        d = dev::forcing_dmu(a.source, (double)(n - j) * dt, a.mu[q]);
                    } else {
                        u = dev::forcing(a.source, (double)(n + j) * dt, a.mu[q]);
                    }
                }
                uw[s][j] = u;
                if constexpr (MODE == kAdjoint) dw[s][j] = d;
            }
            __syncthreads();
            amplitudes(0);
        }
        if constexpr (MODE == kAdjoint) store_s(a.qtr + (size_t)(n - a.n0) * M * ks);     // Q^{n+1}
        // ---- V += dt (Avs S + b u)
        if (wv) {
            double inc[EV];
            if constexpr (NS == 4)
                row_sums4<T::CV, T::LV, LDX>(opv, xs[1], i, qv, inc);
            else
                inc[0] = row_sum<T::CV, T::LV>(opv, xs[1], i, qv);
#pragma unroll
            for (int e = 0; e < EV; ++e) {
                const double y = fma(dt, fma(widen(bb), un[e], inc[e]), v64[e]);
                const float h = (float)y;
                if (okv) {
                    xs[0][xv[e]] = h;
                    if (probe) pb[sv + e][rv] = widen(cc) * y;
                }
                v64[e] = (double)h + (double)(float)(y - (double)h);
            }
        }
        if constexpr (MODE == kAdjoint) store_v(a.wtr + (size_t)(n - a.n0) * M * kv);     // w^n
        __syncthreads();
        amplitudes((kw + 1) % kWin);
        if constexpr (MODE == kTraced) store_v(a.vtr + (size_t)(k + 1) * M * kv);
        // ---- S += dt Asv V
        if (ws) {
            double inc[ES];
            if constexpr (NS == 4)
                row_sums4<T::CS, T::LS, LDX>(ops, xs[0], i, qs, inc);
            else
                inc[0] = row_sum<T::CS, T::LS>(ops, xs[0], i, qs);
#pragma unroll
            for (int e = 0; e < ES; ++e) {
                const double y = fma(dt, inc[e], s64[e]);
                const float h = (float)y;
                if (oks) xs[1][xw[e]] = h;
                s64[e] = (double)h + (double)(float)(y - (double)h);
            }
        }
        if (pwave) {
            double y;
            if constexpr (T::kProbeWave) {
                y = probe_sum<A, NS>(pb, 0, i, dr);
#pragma unroll
                for (int pass = 1; pass < P; ++pass) {
                    const double z = probe_sum<A, NS>(pb, pass, i, dr);
                    y = probe_pass<A, NS>(dr) == pass ? z : y;
                }
            } else {
                y = probe_sum<A, NS>(pb, pw, i, dr);
            }
            if constexpr (MODE == kAdjoint) {
                Jacc += dt * y * dw[NS == 1 ? 0 : pm - m0][kw];
            } else {
                Jacc += dt * (y * y);
                if (a.y && pok) a.y[(size_t)k * M + pm] = y;
            }
        }
        if constexpr (MODE == kTraced) {
            if (a.str) store_s(a.str + (size_t)(k + 1) * M * ks);
        }
        __syncthreads();
    }
    store_v(static_cast<float *>(a.V));
    store_s(static_cast<float *>(a.S));
    double *sum = MODE == kAdjoint ? a.dmu : a.J;
    if (pwave && sum && pok) sum[pm] += Jacc;
}

// A kernel's variants, DPP rows per 16 operator rows of its two sums, and
// whether it has a wave for the probe.
struct Kernel {
    const void *f[2][3];               // one, four samples; mode
    int cv, cs;
    bool probe_wave;
};

template <int A, int B>
Kernel make_kernel() {
    return {{{(const void *)rank2_chains_kernel<A, B, 1, kPlain>, (const void *)rank2_chains_kernel<A, B, 1, kTraced>,
              (const void *)rank2_chains_kernel<A, B, 1, kAdjoint>},
             {(const void *)rank2_chains_kernel<A, B, 4, kPlain>, (const void *)rank2_chains_kernel<A, B, 4, kTraced>,
              (const void *)rank2_chains_kernel<A, B, 4, kAdjoint>}},
            Shape<A, B>::CV, Shape<A, B>::CS, Shape<A, B>::kProbeWave};
}

const Kernel *find_kernel(int kvp, int ksp) {
    static const Kernel t[4][4] = {
        {make_kernel<1, 1>(), make_kernel<1, 2>(), make_kernel<1, 3>(), make_kernel<1, 4>()},
        {make_kernel<2, 1>(), make_kernel<2, 2>(), make_kernel<2, 3>(), make_kernel<2, 4>()},
        {make_kernel<3, 1>(), make_kernel<3, 2>(), make_kernel<3, 3>(), Kernel{}},
        {make_kernel<4, 1>(), make_kernel<4, 2>(), Kernel{}, Kernel{}}};
    if (kvp < 64 || ksp < 64 || kvp > kMaxK || ksp > kMaxK) return nullptr;
    const Kernel *k = &t[kvp / 64 - 1][ksp / 64 - 1];
    return k->f[0][0] ? k : nullptr;
}

}  // namespace

bool rank2_chains_applies(int kvp, int ksp, int M) { return M >= 1 && find_kernel(kvp, ksp) != nullptr; }

// (four samples per workgroup, both sums of three blocks: the other sizes
// are faster than any row-split tile)
float rank2_chains_us(int kvp, int ksp, int M) {
    return M <= kOneSample ? 1.3f : kvp == 192 && ksp == 192 ? 2.5f : 2.0f;
}

// Arguments as for launch_rank2_f32_mfma (mode 0, traced with a.vtr) and
// launch_adjoint_f32_mfma (adjoint), a.str and the
// probe of a traced run may be null; launches: how many such run side by side.
hipError_t launch_rank2_chains(const Rank2Args &a, bool adjoint, int launches, hipStream_t st) {
    const Kernel *k = find_kernel(a.kvp, a.ksp);
    if (!k) return hipErrorInvalidValue;
    const bool traced = a.vtr != nullptr;
    if (adjoint && !(a.b && a.c && a.ytr && a.qtr && a.wtr)) return hipErrorInvalidValue;
    const int ns = launches * a.M > kOneSample ? 4 : 1;
    const int rv = 64 / k->cv, rs = 64 / k->cs;
    const int wv = (a.kv + rv - 1) / rv, ws = (a.ks + rs - 1) / rs;
    const int waves = (wv > ws ? wv : ws) + (k->probe_wave && (adjoint || a.c) ? 1 : 0);
    Rank2Args c = a;
    void *args[] = {&c};
    return hipLaunchKernel(k->f[ns / 4][adjoint ? kAdjoint : traced ? kTraced : kPlain], dim3((a.M + ns - 1) / ns),
                           dim3(64 * waves), args, 0, st);
}

}  // namespace rom
