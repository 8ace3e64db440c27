// Launchers of the resident row-split kernels (k_rsplit.h).
#include "k_rsplit.h"

#include <cmath>

namespace rom {
namespace {

using namespace rsplit;

// The tile for a run (`runs` of them side by side), or null: of those whose
// groups fit in one launch the one with the smallest area (the first of
// equals).
const Tile *pick_tile(bool pairs, int kv, int ks, int kvp, int ksp, int M, int runs) {
    const int kp = kvp > ksp ? kvp : ksp, k = kv > ks ? kv : ks, nch = (kp + 255) / 256;
    const Tile *best = nullptr, *tiles = pairs ? kPairTiles : kQuarterTiles;
    for (int i = 0; i < (pairs ? kPairCount : kQuarterCount); ++i) {
        const Tile &t = tiles[i];
        if (t.nch != nch) continue;
        const int R = (k + 16 * t.nrb - 1) / (16 * t.nrb), G = (M + 16 * t.ncb - 1) / (16 * t.ncb);
        if (R > kCusPerXcd || runs * G > kXcds * (kCusPerXcd / R)) continue;
        if (!best || t.nrb * t.ncb < best->nrb * best->ncb) best = &t;
    }
    return best;
}

hipError_t fill(RArgs &a, const Tile *t, const void *opv, const void *ops, const Rank2Args &r2, void *ws, int *status,
                hipStream_t st) {
    fill_split_args(a.s, opv, ops, r2, 1.0f, status);
    const int kp = r2.kvp > r2.ksp ? r2.kvp : r2.ksp, k = r2.kv > r2.ks ? r2.kv : r2.ks, nc = 16 * t->ncb;
    a.ks = r2.ks;
    a.kgv = r2.ksp / 16;
    a.kgs = r2.kvp / 16;
    a.np = kp;
    a.s.R = (k + 16 * t->nrb - 1) / (16 * t->nrb);
    a.kgpub = a.s.R * t->nrb;
    a.s.G = (r2.M + nc - 1) / nc;
    return split_workspace(a.s, ws, (size_t)a.s.G * nc * kp, (size_t)a.s.G * nc * a.s.R, true, st);
}

// A repeatable run (rep): its groups' words are the flags, which these kernels
// do not use, its status words are its own, behind the slot counters.
hipError_t repeatable(RArgs &a, const Tile *t, Repeat *rep, hipStream_t st) {
    if (!rep) return hipSuccess;
    a.s.done = a.s.flags;
    a.s.status = reinterpret_cast<int *>(a.s.slots + 8);
    *rep = Repeat{a.s.done, 16 * t->ncb, a.s.G};
    return g_forced_timeout == 2 ? freeze_odd_groups(a.s.done, a.s.G, st) : hipSuccess;
}

hipError_t launch(const void *f, RArgs &a0, RArgs &a1, hipStream_t st) {
    void *args[] = {&a0, &a1};
    return launch_waiting(f, args, kLdsR, st, a0.s.done == nullptr);
}

template <class F>
hipError_t each_kernel(F f) {
    hipError_t e = hipSuccess;
    auto tile = [&](const Tile &t) {
        for (const void *k : t.f)
            if (k && e == hipSuccess) e = f(k);
    };
    for (const Tile &t : kQuarterTiles) tile(t);
    for (const Tile &t : kPairTiles) tile(t);
    return e;
}

}  // namespace

bool rank2_rsplit_applies(bool pairs, int kv, int ks, int kvp, int ksp, int M, int runs) {
    return M >= 1 && pick_tile(pairs, kv, ks, kvp, ksp, M, runs) != nullptr;
}

float rank2_rsplit_us(bool pairs, int kv, int ks, int kvp, int ksp, int M) {
    const Tile *t = M >= 1 ? pick_tile(pairs, kv, ks, kvp, ksp, M, 1) : nullptr;
    if (!t) return INFINITY;
    const int kp = kvp > ksp ? kvp : ksp;
    return t->us * (1.0f - 0.04f * (float)((256 * t->nch - kp) / 64));
}

// (rank2_split_workspace_bytes of the same padded size and 64-column groups
// covers it: the groups are at most 32 columns wide)
size_t rank2_rsplit_ws_bytes(int kvp, int ksp, int M) {
    return rank2_split_workspace_bytes(kvp > ksp ? kvp : ksp, (M + kCols - 1) / kCols);
}

hipError_t launch_rank2_rsplit(bool pairs, const void *opv, const void *ops, const Rank2Args &r2, void *ws, int *status,
                               hipStream_t st, int mode, Repeat *rep) {
    if (r2.M < 1 || r2.nsteps < 1 || mode < kPlain || mode > kAdjoint || pairs != (rep != nullptr))
        return hipErrorInvalidValue;
    const Tile *t = pick_tile(pairs, r2.kv, r2.ks, r2.kvp, r2.ksp, r2.M, 1);
    if (!t || !t->f[mode]) return hipErrorInvalidValue;
    RArgs a{}, none{};
    hipError_t e = fill(a, t, opv, ops, r2, ws, status, st);
    if (e == hipSuccess) e = repeatable(a, t, rep, st);
    return e == hipSuccess ? launch(t->f[mode], a, none, st) : e;
}

hipError_t launch_rank2_rsplit_dual(const void *opv0, const void *ops0, const Rank2Args &r0, void *ws0,
                                    const void *opv1, const void *ops1, const Rank2Args &r1, void *ws1, int *status,
                                    hipStream_t st) {
    if (r0.M < 1 || r0.nsteps < 1 || r1.nsteps < 1 || r1.M != r0.M || r1.kvp != r0.kvp || r1.ksp != r0.ksp)
        return hipErrorInvalidValue;
    const Tile *t = pick_tile(false, r0.kv, r0.ks, r0.kvp, r0.ksp, r0.M, 2);
    if (!t) return hipErrorInvalidValue;
    RArgs a0{}, a1{};
    hipError_t e = fill(a0, t, opv0, ops0, r0, ws0, status, st);
    if (e == hipSuccess) e = fill(a1, t, opv1, ops1, r1, ws1, status, st);
    return e == hipSuccess ? launch(t->f[kDual], a0, a1, st) : e;
}

bool rank2_rsplit_device_ok() {
    return each_kernel([](const void *f) {
               int nb = 0;
               hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kThreads, kLdsR);
               return e == hipSuccess && nb < 1 ? hipErrorLaunchOutOfResources : e;
           }) == hipSuccess;
}

hipError_t rank2_rsplit_configure() {
    return each_kernel([](const void *f) {
        return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsR);
    });
}

}  // namespace rom
