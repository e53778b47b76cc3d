// Forces of a small droplet in one launch: one-sided Coulomb tiles and, beside
// them, the Lennard-Jones groups.
//
// Bound by latency: a few thousand NPs are a few thousand 64 x 64 tiles for
// 1024 SIMDs, and a wavefront alone issues one operation per ~6 clocks, so
// what counts is how many wavefronts share the tiles and how many launches
// follow each other.  A workgroup takes one 64-slot i group against every
// j_split-th run of its wavefronts' j groups (a group per wavefront per turn,
// staged in the wavefront's own LDS slice, no barrier until the end, where
// the wavefronts' sums are added in order); the Lennard-Jones workgroups, the
// longest chains of dependent loads, come first in the grid.
// Measured against k_pair's two instances followed by k_lj and, after the
// update, a launch for the clock: a step of 1000 slots 45 -> 18 us, of 5000
// slots 64 -> 28 us.
//
// Positions are relative to the centre of the i group's box, (hi - c) + lo, so
// a difference carries the rounding of the distance rather than of |x|.  In a
// stretched box (NPs thrown out) they would lose too much: far groups then use
// the high words and near ones the exact (hi, lo) differences.  FP32 pair
// terms in blocks of 32, as everywhere (ld_pair_core.h).
#include "ld_pair_core.h"

namespace ld {
namespace {

using namespace pair;

struct DirectArgs {
    const float4* pos;
    const float4* lo;
    const int* typ;
    const Box* box;
    int n, ngroups, j_split;
    double* F;                             // [1 + j_split][3][n]
    DevState* st;                          // step clock to advance by adv_dt first
    double adv_dt;
    int lj_blocks;
    PairTable tab;
};

template <int WAVES>
struct CoulombShared {
    float4 sp[WAVES][kGroup], sl[WAVES][kGroup];
    double red[WAVES][3][kGroup];
};

template <int WAVES, int COMP, bool LONG>
__global__ __launch_bounds__(WAVES * kGroup) void k_direct(DirectArgs A) {
    __shared__ union U {
        CoulombShared<WAVES> c;
        LjBlock<WAVES, 3, LONG> lj;
        __device__ U() {}
    } sh;
    if (A.adv_dt > 0.0 && blockIdx.x == 0 && threadIdx.x == 0) {
        A.st->t = A.st->t + A.adv_dt;
        A.st->step = A.st->step + 1;
    }
    const size_t n = (size_t)A.n;
    if ((int)blockIdx.x < A.lj_blocks) {
        double sums[3];
        if (!lj_block<false, false, WAVES, LONG>(A.pos, A.lo, A.typ, A.box, A.n, blockIdx.x, A.tab,
                                                 sh.lj, sums))
            return;
        const size_t i = (size_t)blockIdx.x * kGroup + threadIdx.x;
        for (int c = 0; c < 3; ++c) A.F[c * n + i] = -sums[c];
        return;
    }
    const int t = (int)blockIdx.x - A.lj_blocks;
    const int gi = t % A.ngroups, split = t / A.ngroups;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kGroup);
    const int lane = threadIdx.x % kGroup;
    const int i = gi * kGroup + lane;
    const bool live = i < A.n;
    const float4 pi = A.pos[min(i, A.n - 1)], li = A.lo[min(i, A.n - 1)];
    const Box bi = A.box[gi];
    const bool rel = box_compact(bi);
    const float cull2 = A.tab.rc2max * 1.0001f;
    const float3 o = make_float3(0.5f * (bi.lo.x + bi.hi.x), 0.5f * (bi.lo.y + bi.hi.y),
                                 0.5f * (bi.lo.z + bi.hi.z));
    const float4 pr = rel ? make_float4((pi.x - o.x) + li.x, (pi.y - o.y) + li.y,
                                        (pi.z - o.z) + li.z, pi.w)
                          : pi;
    Acc a;
    if (bi.lo.w != 0.f) {                  // uncharged groups have no Coulomb terms
        for (int gj = split * WAVES + w; gj < A.ngroups; gj += A.j_split * WAVES) {
            const Box bj = A.box[gj];
            if (bj.lo.w == 0.f) continue;
            const int j = gj * kGroup + lane;
            const float4 h = A.pos[min(j, A.n - 1)], l = A.lo[min(j, A.n - 1)];
            const bool exact = !rel && __any(live && point_box_dist2(pi, bj) < cull2);
            float4 q = rel ? make_float4((h.x - o.x) + l.x, (h.y - o.y) + l.y, (h.z - o.z) + l.z,
                                         h.w)
                           : h;
            if (j >= A.n) q = make_float4(kFarAway, kFarAway, kFarAway, 0.f);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            sh.c.sp[w][lane] = q;
            if (exact) sh.c.sl[w][lane] = j < A.n ? l : make_float4(0.f, 0.f, 0.f, 0.f);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (exact)
                group_near<COMP, false>(sh.c.sp[w], sh.c.sl[w], gj * kGroup, i, pi, li, a);
            else
                group_rel<COMP>(sh.c.sp[w], pr, a);
        }
    }
    if constexpr (COMP == 1) {
        a.Fx = (double)a.sx - (double)a.cx;
        a.Fy = (double)a.sy - (double)a.cy;
        a.Fz = (double)a.sz - (double)a.cz;
    }
    sh.c.red[w][0][lane] = a.Fx;
    sh.c.red[w][1][lane] = a.Fy;
    sh.c.red[w][2][lane] = a.Fz;
    __syncthreads();
    if (w != 0 || !live) return;
    // F_i = -q_i sum_j q_j r^-3 (x_j - x_i)
    double* F = A.F + (size_t)(1 + split) * 3 * n;
    for (int c = 0; c < 3; ++c) {
        double f = 0.0;
        for (int v = 0; v < WAVES; ++v) f += sh.c.red[v][c][lane];
        F[c * n + i] = -(double)pi.w * f;
    }
}

template <int WAVES>
hipError_t launch_waves(const PairLaunch& L, const PairTable& tab, hipStream_t s,
                        hipEvent_t before_coulomb, hipEvent_t after_coulomb) {
    DirectArgs A{};
    A.pos = L.pos;
    A.lo = L.lo;
    A.typ = L.typ;
    A.box = L.box;
    A.n = L.n;
    A.ngroups = (L.n + kGroup - 1) / kGroup;
    A.j_split = L.j_split;
    A.F = L.Fpart;
    A.st = L.st;
    A.adv_dt = L.adv_dt;
    A.tab = tab;
    auto launch = [&](int lj, int coulomb) {
        A.lj_blocks = lj;
        const bool far = lj_long(tab);
        hipLaunchKernelGGL(L.comp == 0 ? (far ? k_direct<WAVES, 0, true> : k_direct<WAVES, 0, false>)
                                       : (far ? k_direct<WAVES, 1, true> : k_direct<WAVES, 1, false>),
                           dim3(lj + coulomb), dim3(WAVES * kGroup), 0, s, A);
        A.adv_dt = 0.0;
    };
    // A single wavefront is longer at a Lennard-Jones group than at a short run of
    // tiles, so blocks of 64 give the groups a launch of four wavefronts each.
    // Steps in 8 parts 59 -> 34 us (1000 slots), 121 -> 107 (11 000); in one part,
    // where the runs are the longer ones, 94 -> 118 (2500), and two groups or less
    // 20 -> 23 (100): those stay in one launch.
    const bool apart = WAVES == 1 && A.ngroups > 2 && A.ngroups <= 24 * A.j_split;
    auto groups = [&] {
        if (!apart) {
            launch(A.ngroups, 0);
        } else {
            A.lj_blocks = A.ngroups;
            hipLaunchKernelGGL((lj_long(tab) ? k_direct<4, 0, true> : k_direct<4, 0, false>),
                               dim3(A.ngroups), dim3(4 * kGroup), 0, s, A);
            A.adv_dt = 0.0;
        }
    };
    const int tiles = A.ngroups * A.j_split;
    if (!after_coulomb) {
        if (apart) groups();
        launch(apart ? 0 : A.ngroups, tiles);
        return hipGetLastError();
    }
    // timed: the Coulomb tiles by themselves
    groups();
    hipError_t e = hipEventRecord(before_coulomb, s);
    if (e != hipSuccess) return e;
    launch(0, tiles);
    e = hipEventRecord(after_coulomb, s);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace

hipError_t launch_direct(const PairLaunch& L, const PairTable& tab, hipStream_t s,
                         hipEvent_t before_coulomb, hipEvent_t after_coulomb) {
    switch (L.block) {
        case 64: return launch_waves<1>(L, tab, s, before_coulomb, after_coulomb);
        case 128: return launch_waves<2>(L, tab, s, before_coulomb, after_coulomb);
        case 256: return launch_waves<4>(L, tab, s, before_coulomb, after_coulomb);
        case 512: return launch_waves<8>(L, tab, s, before_coulomb, after_coulomb);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ld
