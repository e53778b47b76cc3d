// All-pairs force kernels: the O(N^2) part of each step (section 2.2, step
// (ii): Lennard-Jones and Coulomb forces, both unshifted; Coulomb here runs
// over all pairs).
//
// k_pair: the Coulomb sum.  One work-item owns one particle i (slot order).
// A workgroup of BLOCK work-items streams the j range of its split through
// LDS one tile of BLOCK particles at a time; every lane reads the same LDS
// word per j (a broadcast), so the j stream costs one ds_read per wavefront
// per j and the VALU does the rest.  Per pair: 12 FP32 VALU operations plus
// one v_rsq_f32 (three subtractions, r^2 as mul+fma+fma, q_j r^-3 as three
// multiplications, three fma into the block accumulators).  With tile
// culling on, a 64-particle j group whose bounding box is farther than the
// largest LJ range from the wavefront's own box takes the plain loop on the
// FP32 high words; a nearer group takes the loop on positions relative to
// the centre c of the workgroup's box, (hi - c) + lo, staged beside the high
// words (same instruction count, and the rounding of |x - c| instead of
// |x|), which also leaves out the self pair; a far
// pair of groups one of which is uncharged is skipped (no force at all).
//
// k_lj: the Lennard-Jones sum, which is short-ranged (lj_cut sigma_ij), in
// FP64: the groups whose boxes come within the largest LJ range, screened
// slot by slot.  It adds its result into the first force partial of each
// slot after k_pair has written it (same stream, one writer per slot).
//
// Precision.  The Coulomb pair terms are FP32.  Each lane sums KB = 32 of
// them in an FP32 block accumulator and then moves the block into FP64
// totals (COMP=0) or into a blocked Kahan pair (COMP=1, flushed to FP64 at
// the end).  The worst-case rounding of a 32-term FP32 block is
// 31 u sum|f| ~ 1.8e-6 of the conditioning scale S_i = sum_j |f_ij|.  The
// Lennard-Jones terms are FP64 throughout.
#include "ld_pair_core.h"

namespace ld {
namespace {

using namespace pair;

// Wavefronts per SIMD the register allocation must allow (block 64 keeps a
// whole j tile in registers whatever the bound; it is left unconstrained).
#ifndef LD_PAIR_MIN_WAVES
#define LD_PAIR_MIN_WAVES 6
#endif

constexpr float kRelReach = 255.f;         // sigma; see the near-loop choice in k_pair
#ifndef LD_PAIR_REL_GUARD
#define LD_PAIR_REL_GUARD 1
#endif

// Workgroup -> (i tile, j split) on a one-dimensional grid.  Workgroups go
// to the eight XCDs in turn (linear id mod 8), so XCD k takes i tiles k,
// k + 8, k + 16, ... for every split, split after split: the i tiles one
// XCD serves (about an eighth of them) stay in its L2 across the splits
// instead of every tile being fetched again for each split.  Workgroups
// past the last tile of an XCD's share leave at once.
constexpr int kXcds = 8;
__host__ __device__ inline int pair_grid(int tiles, int j_split) {
    return kXcds * ((tiles + kXcds - 1) / kXcds) * j_split;
}

template <int BLOCK, int COMP, bool DIAG, bool CULL, bool REL>
__global__ __launch_bounds__(BLOCK, BLOCK == 64 ? 1 : LD_PAIR_MIN_WAVES) void k_pair(const float4* __restrict__ pos,
                                                const float4* __restrict__ lo,
                                                const Box* __restrict__ box, int n,
                                                int j_per_split, float rc2max,
                                                double* __restrict__ Fpart,
                                                double* __restrict__ S_out,
                                                double* __restrict__ U_out) {
    __shared__ float4 sp[BLOCK];             // j tile, high words
    __shared__ float4 sr[BLOCK];             // near loop: positions relative to c, or low words

    const int tid = threadIdx.x;
    const int ngroups = (n + kGroup - 1) / kGroup;
    const int tiles = (n + BLOCK - 1) / BLOCK;
    const int per_xcd = (tiles + kXcds - 1) / kXcds;
    const int q = (int)blockIdx.x / kXcds;
    const int tx = (int)blockIdx.x % kXcds + kXcds * (q % per_xcd);   // i tile
    const int ty = q / per_xcd;                                         // j split
    if (tx >= tiles) return;                     // uniform per workgroup
    // A small margin covers FP32 rounding of box distances against r^2.
    const float cull2 = rc2max * 1.0001f;
    // Near loop on positions relative to c, the centre of the box of the
    // workgroup's BLOCK slots, when that box is compact (half-extent below
    // kRelReach: |x - c| < 256 sigma, so (hi - c) + lo carries at most two
    // FP32 roundings of 2^-17 sigma, 1.5e-5 sigma, and in practice a few
    // times less, most near pairs sitting tens of sigma from c); otherwise,
    // and without culling (no boxes), on exact (hi, lo) differences, e.g.
    // where a blown-up step has thrown NPs far out or the slots are not in
    // spatial order.  The choice is uniform per workgroup and made before
    // anything else is loaded.  The two loops are separate instances (REL),
    // so the common one keeps its own register allocation, launched on the
    // same grid: first the exact one, which leaves compact workgroups at
    // once and takes only the near group pairs of stretched ones; then the
    // relative one, which takes compact workgroups whole and the far group
    // pairs of stretched ones, adding them to what the exact one wrote.  A
    // stretched workgroup thus adds no long serial tail after the relative
    // launch.  Without culling, or in diagnostic mode, the exact instance
    // runs alone and takes everything.
    bool rel = false;
    float4 c = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (CULL && !DIAG) {
        float3 blo = make_float3(INFINITY, INFINITY, INFINITY);
        float3 bhi = make_float3(-INFINITY, -INFINITY, -INFINITY);
        for (int g4 = 0; g4 < BLOCK / kGroup; ++g4) {
            const int gq = tx * (BLOCK / kGroup) + g4;
            if (gq >= ngroups) break;
            const Box bq = box[gq];
            blo = make_float3(fminf(blo.x, bq.lo.x), fminf(blo.y, bq.lo.y), fminf(blo.z, bq.lo.z));
            bhi = make_float3(fmaxf(bhi.x, bq.hi.x), fmaxf(bhi.y, bq.hi.y), fmaxf(bhi.z, bq.hi.z));
        }
        c = make_float4(0.5f * (blo.x + bhi.x), 0.5f * (blo.y + bhi.y), 0.5f * (blo.z + bhi.z),
                        0.f);
        const float ext = fmaxf(fmaxf(bhi.x - blo.x, bhi.y - blo.y), bhi.z - blo.z);
        rel = !LD_PAIR_REL_GUARD || ext < 2.f * kRelReach;    // false for NaN or infinite boxes
    }
    constexpr bool SPLIT = CULL && !DIAG;
    if (!REL && rel) return;                     // uniform per workgroup

    const int i = tx * BLOCK + tid;
    const bool live = i < n;
    const float4 pi = live ? pos[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    const float4 li = live ? lo[i] : make_float4(0.f, 0.f, 0.f, 0.f);

    // This wavefront's bounding box (culling only).
    Box bi;
    if constexpr (CULL) {
        const int gi = (tx * BLOCK + (tid & ~(kGroup - 1))) / kGroup;
        if (gi < ngroups) {
            bi = box[gi];
        } else {
            bi.lo = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
            bi.hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.f);
        }
    }
    const float4 pr = make_float4((pi.x - c.x) + li.x, (pi.y - c.y) + li.y, (pi.z - c.z) + li.z,
                                  pi.w);

    const int j0 = ty * j_per_split;
    const int j1 = min(n, j0 + j_per_split);
    Acc a;
#pragma unroll 1
    for (int jt = j0; jt < j1; jt += BLOCK) {
        __syncthreads();
        const int j = jt + tid;
        {
            float4 h = make_float4(kFarAway, kFarAway, kFarAway, 0.f);
            float4 r = REL ? h : make_float4(0.f, 0.f, 0.f, 0.f);
            if (j < j1) {
                h = pos[j];
                const float4 l = lo[j];
                r = REL ? make_float4((h.x - c.x) + l.x, (h.y - c.y) + l.y, (h.z - c.z) + l.z, h.w)
                        : l;
            }
            sp[tid] = h;
            sr[tid] = r;
        }
        __syncthreads();
#pragma unroll 1
        for (int g = 0; g < BLOCK / kGroup; ++g) {
            const int jg = jt + g * kGroup;
            bool near = true;
            if constexpr (CULL) {
                const int gj = jg / kGroup;
                near = false;
                bool coulomb = false;
                if (jg < j1 && gj < ngroups) {
                    const Box bj = box[gj];
                    if (REL && rel) {
                        near = box_dist2(bi, bj) < cull2;
                    } else {
                        // the i group's own box may be stretched across the
                        // droplet by one NP thrown out: test each lane's i
                        near = __ballot(live && point_box_dist2(pi, bj) < cull2) != 0;
                    }
                    coulomb = bi.lo.w != 0.f && bj.lo.w != 0.f;
                }
                if (!near && !__builtin_amdgcn_readfirstlane((int)coulomb)) continue;
                // a stretched workgroup's near pairs go to the exact
                // instance, its far ones to the relative instance
                if constexpr (SPLIT) {
                    if (REL ? (!rel && near) : !near) continue;
                }
            }
            if constexpr (DIAG) near = true;
            if (__builtin_amdgcn_readfirstlane((int)near)) {
                if constexpr (REL)
                    group_near_rel<COMP, DIAG>(sr + g * kGroup, jg, i, pr, a);
                else
                    group_near<COMP, DIAG>(sp + g * kGroup, sr + g * kGroup, jg, i, pi, li, a);
            } else {
                group_far<COMP>(sp + g * kGroup, pi, a);
            }
        }
    }
    if constexpr (COMP == 1) {
        a.Fx = (double)a.sx - (double)a.cx;
        a.Fy = (double)a.sy - (double)a.cy;
        a.Fz = (double)a.sz - (double)a.cz;
    }
    if (live) {
        // F_i = -q_i sum_j q_j r^-3 (x_j - x_i)
        const double qi = (double)pi.w;
        double* F = Fpart + (size_t)ty * 3 * (size_t)n;
        if (REL && !rel) {                       // after the exact instance's near part
            F[i] += -qi * a.Fx;
            F[(size_t)n + i] += -qi * a.Fy;
            F[2 * (size_t)n + i] += -qi * a.Fz;
        } else {
            F[i] = -qi * a.Fx;
            F[(size_t)n + i] = -qi * a.Fy;
            F[2 * (size_t)n + i] = -qi * a.Fz;
        }
        if constexpr (DIAG) {
            S_out[i] = a.S;
            U_out[i] = 0.0;
            U_out[(size_t)n + i] = a.Uc;
        }
    }
}

// Lennard-Jones forces of every slot (and, with DIAG, S and the LJ energy row
// of U), added into partial 0 after k_pair.  One workgroup per 64-slot i
// group (lj_group).
template <bool DIAG, int WAVES, bool LONG>
__global__ __launch_bounds__(WAVES * kGroup) void k_lj(const float4* __restrict__ pos,
                                                        const float4* __restrict__ lo,
                                                        const int* __restrict__ typ,
                                                        const Box* __restrict__ box, int n,
                                                        double* __restrict__ F,
                                                        double* __restrict__ S_out,
                                                        double* __restrict__ U_out,
                                                        PairTable tab) {
    __shared__ LjBlock<WAVES, DIAG ? 5 : 3, LONG> sh;
    double sums[DIAG ? 5 : 3];
    const int i = blockIdx.x * kGroup + threadIdx.x;
    if (!lj_block<DIAG, false, WAVES, LONG>(pos, lo, typ, box, n, blockIdx.x, tab, sh, sums))
        return;
    for (int c = 0; c < 3; ++c) F[(size_t)c * (size_t)n + i] -= sums[c];
    if constexpr (DIAG) {
        S_out[i] += sums[3];
        U_out[i] += sums[4];
    }
}

// Wavefronts per i group: 16 while the groups are too few to fill the chip
// with four each.
template <bool DIAG, bool LONG>
void launch_lj(const PairLaunch& L, const PairTable& tab, hipStream_t s) {
    const dim3 grid((L.n + kGroup - 1) / kGroup);
    if (grid.x < 1024)
        hipLaunchKernelGGL((k_lj<DIAG, 16, LONG>), grid, dim3(16 * kGroup), 0, s, L.pos, L.lo,
                           L.typ, L.box, L.n, L.Fpart, L.S, L.U, tab);
    else
        hipLaunchKernelGGL((k_lj<DIAG, 4, LONG>), grid, dim3(4 * kGroup), 0, s, L.pos, L.lo,
                           L.typ, L.box, L.n, L.Fpart, L.S, L.U, tab);
}
template <bool DIAG>
void launch_lj(const PairLaunch& L, const PairTable& tab, hipStream_t s) {
    if (lj_long(tab))
        launch_lj<DIAG, true>(L, tab, s);
    else
        launch_lj<DIAG, false>(L, tab, s);
}

template <int BLOCK, int COMP, bool DIAG, bool CULL>
hipError_t launch_t(const PairLaunch& L, const PairTable& tab, hipStream_t s) {
    const int tiles = (L.n + BLOCK - 1) / BLOCK;
    const int per = (tiles + L.j_split - 1) / L.j_split;
    const dim3 grid(pair_grid(tiles, L.j_split));
    // with culling: the exact instance (stretched workgroups' near pairs)
    // first, then the relative one, which adds to it; otherwise the exact
    // instance alone
    if (!(CULL && !DIAG) || LD_PAIR_REL_GUARD)
        hipLaunchKernelGGL((k_pair<BLOCK, COMP, DIAG, CULL, false>), grid, dim3(BLOCK), 0, s,
                           L.pos, L.lo, L.box, L.n, per * BLOCK, tab.rc2max, L.Fpart, L.S, L.U);
    if constexpr (CULL && !DIAG)
        hipLaunchKernelGGL((k_pair<BLOCK, COMP, DIAG, CULL, true>), grid, dim3(BLOCK), 0, s,
                           L.pos, L.lo, L.box, L.n, per * BLOCK, tab.rc2max, L.Fpart, L.S, L.U);
    return hipGetLastError();
}

template <int BLOCK>
hipError_t launch_b(const PairLaunch& L, const PairTable& tab, hipStream_t s) {
    const bool diag = L.S != nullptr;
    if (diag) return launch_t<BLOCK, 0, true, false>(L, tab, s);
    if (L.comp == 0) {
        return L.cull ? launch_t<BLOCK, 0, false, true>(L, tab, s)
                      : launch_t<BLOCK, 0, false, false>(L, tab, s);
    }
    return L.cull ? launch_t<BLOCK, 1, false, true>(L, tab, s)
                  : launch_t<BLOCK, 1, false, false>(L, tab, s);
}

hipError_t launch_coulomb(const PairLaunch& L, const PairTable& tab, hipStream_t s) {
    switch (L.block) {
        case 64: return launch_b<64>(L, tab, s);
        case 128: return launch_b<128>(L, tab, s);
        case 256: return launch_b<256>(L, tab, s);
        case 512: return launch_b<512>(L, tab, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_pair(const PairLaunch& L, const PairTable& tab, hipStream_t s,
                       hipEvent_t before_coulomb, hipEvent_t after_coulomb) {
    if (L.sym) return launch_pair_sym(L, tab, s, before_coulomb, after_coulomb);
    if (L.direct) return launch_direct(L, tab, s, before_coulomb, after_coulomb);
    hipError_t e;
    if (before_coulomb && (e = hipEventRecord(before_coulomb, s)) != hipSuccess) return e;
    if ((e = launch_coulomb(L, tab, s)) != hipSuccess) return e;
    if (after_coulomb && (e = hipEventRecord(after_coulomb, s)) != hipSuccess) return e;
    if (L.S)
        launch_lj<true>(L, tab, s);
    else
        launch_lj<false>(L, tab, s);
    return hipGetLastError();
}

}  // namespace ld
