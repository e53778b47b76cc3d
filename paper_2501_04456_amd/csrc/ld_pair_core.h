// Inner loops of the one-sided all-pairs Coulomb sum (k_pair in ld_pair.hip,
// k_direct in ld_direct.hip), and the Lennard-Jones groups of all force kernels.
//
// Per pair the Coulomb path is 12 FP32 VALU operations plus one
// v_rsq_f32: three subtractions, r^2 as mul+fma+fma, q_j r^-3 as three
// multiplications and three fma into FP32 block accumulators.  Each lane sums
// KB = 32 pair terms in FP32 and then moves the block into FP64 totals
// (COMP=0) or into a blocked Kahan pair (COMP=1); LJ terms (near groups
// only) are computed and summed in FP64 by their own kernel.  The
// worst-case rounding of a 32-term FP32 block is 31 u sum|f| ~ 1.8e-6 of
// S_i = sum_j |f_ij|.
#pragma once

#include "ld_internal.h"

namespace ld {
namespace pair {

// Upper bound on the FP32 1/r of the near loops: 1/r of any two distinct
// particles is far below it (they never come within 1e-10 sigma), and
// |q_j| kInvRCap^3 stays finite, so the self pair (r = 0) adds w * 0 = 0.
// Two distinct particles at bitwise equal positions would get a zero
// Coulomb term here (their Lennard-Jones term is still infinite).
constexpr float kInvRCap = 1e10f;

constexpr int KB = 32;

struct Acc {
    double Fx = 0.0, Fy = 0.0, Fz = 0.0;   // sum_j q_j r^-3 (x_j - x_i), FP64
    float sx = 0.f, sy = 0.f, sz = 0.f;    // Kahan sums (COMP == 1)
    float cx = 0.f, cy = 0.f, cz = 0.f;    // Kahan compensations
    double S = 0.0, Uc = 0.0;              // diagnostic mode only (Coulomb part)
};

template <int COMP>
__device__ __forceinline__ void flush(Acc& a, float bx, float by, float bz) {
    if constexpr (COMP == 0) {
        a.Fx += (double)bx;
        a.Fy += (double)by;
        a.Fz += (double)bz;
    } else {
        float y, t;
        y = bx - a.cx; t = a.sx + y; a.cx = (t - a.sx) - y; a.sx = t;
        y = by - a.cy; t = a.sy + y; a.cy = (t - a.sy) - y; a.sy = t;
        y = bz - a.cz; t = a.sz + y; a.cz = (t - a.sz) - y; a.sz = t;
    }
}

// 64 j particles with no LJ partner in range and no self pair: Coulomb only.
template <int COMP>
__device__ __forceinline__ void group_far(const float4* __restrict__ sp, const float4 pi,
                                          Acc& a) {
#pragma unroll
    for (int kb = 0; kb < kGroup; kb += KB) {
        float bx = 0.f, by = 0.f, bz = 0.f;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const float4 pj = sp[kb + k];
            const float dx = pj.x - pi.x;
            const float dy = pj.y - pi.y;
            const float dz = pj.z - pi.z;
            const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            const float ri = __builtin_amdgcn_rsqf(r2);
            const float w = (pj.w * ri) * (ri * ri);
            bx = fmaf(w, dx, bx);
            by = fmaf(w, dy, by);
            bz = fmaf(w, dz, bz);
        }
        flush<COMP>(a, bx, by, bz);
    }
}

// 64 j particles at any distance, i itself among them or not, positions
// relative to one origin near i's group: the far loop, with kTiny added to
// r^2 so that the self pair's weight stays finite (its differences are 0; the
// r^2 of any two particles is far above it).
constexpr float kTiny = 1e-20f;
template <int COMP>
__device__ __forceinline__ void group_rel(const float4* __restrict__ sp, const float4 pi, Acc& a) {
#pragma unroll
    for (int kb = 0; kb < kGroup; kb += KB) {
        float bx = 0.f, by = 0.f, bz = 0.f;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const float4 pj = sp[kb + k];
            const float dx = pj.x - pi.x;
            const float dy = pj.y - pi.y;
            const float dz = pj.z - pi.z;
            const float r2 = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, kTiny)));
            const float ri = __builtin_amdgcn_rsqf(r2);
            const float w = (pj.w * ri) * (ri * ri);
            bx = fmaf(w, dx, bx);
            by = fmaf(w, dy, by);
            bz = fmaf(w, dz, bz);
        }
        flush<COMP>(a, bx, by, bz);
    }
}

// 64 j particles near i's group (within the largest LJ range of its box) or
// holding i itself: the Coulomb terms with the low words of the positions
// in the differences, the self pair left out.  The difference of the FP32
// high words of two nearby particles is exact, and adding the difference of
// their low words gives r_ij to FP32 rounding of r_ij itself.  Used where
// the relative positions below would lose too much (a workgroup whose box
// is stretched by NPs thrown far out).
template <int COMP, bool DIAG>
__device__ __forceinline__ void group_near(const float4* __restrict__ sp,
                                           const float4* __restrict__ sl, int jbase, int i,
                                           const float4 pi, const float4 li, Acc& a) {
#pragma unroll
    for (int kb = 0; kb < kGroup; kb += KB) {
        float bx = 0.f, by = 0.f, bz = 0.f;   // Coulomb, FP32 block
#pragma unroll 4
        for (int k = 0; k < KB; ++k) {
            const float4 pj = sp[kb + k];
            const float4 lj = sl[kb + k];
            const float dx = (pj.x - pi.x) + (lj.x - li.x);
            const float dy = (pj.y - pi.y) + (lj.y - li.y);
            const float dz = (pj.z - pi.z) + (lj.z - li.z);
            const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            // the self pair has dx = dy = dz = 0 exactly; capping 1/r keeps
            // its weight finite, so its term is 0 without a test
            const float ri = fminf(__builtin_amdgcn_rsqf(r2), kInvRCap);
            const float w = (pj.w * ri) * (ri * ri);
            if constexpr (DIAG) {
                if (jbase + kb + k != i) {
                    const float qq = pi.w * pj.w;
                    a.S += (double)(fabsf(qq) * ri * ri);
                    a.Uc += 0.5 * (double)(qq * ri);
                }
            }
            bx = fmaf(w, dx, bx);
            by = fmaf(w, dy, by);
            bz = fmaf(w, dz, bz);
        }
        flush<COMP>(a, bx, by, bz);
    }
}

// 64 j particles near i's group (within the largest LJ range of its box) or
// holding i itself: the Coulomb terms, the self pair left out, from
// positions taken relative to an origin c near both groups (the centre of
// the box of the workgroup's slots).  Each
// staged j and the lane's own i hold (hi - c) + lo rounded to FP32, so a
// difference carries the rounding of |x - c| (tens of sigma for the groups
// this loop sees) instead of |x|: near |x| = 300 sigma one ulp of a
// coordinate is 3e-5 sigma, which at contact distance would move a Coulomb
// term by ~1e-4 of itself; at |x - c| = 64 sigma it is 8e-6 sigma.  One LDS
// read and three subtractions per pair, as in the far loop.  The
// Lennard-Jones terms of these groups are added by a kernel of their own
// (k_lj), in FP64 from the exact (hi, lo) differences.
template <int COMP, bool DIAG>
__device__ __forceinline__ void group_near_rel(const float4* __restrict__ sr, int jbase, int i,
                                               const float4 ri4, Acc& a) {
#pragma unroll
    for (int kb = 0; kb < kGroup; kb += KB) {
        float bx = 0.f, by = 0.f, bz = 0.f;   // Coulomb, FP32 block
#pragma unroll 4
        for (int k = 0; k < KB; ++k) {
            const float4 pj = sr[kb + k];
            const float dx = pj.x - ri4.x, dy = pj.y - ri4.y, dz = pj.z - ri4.z;
            const float r2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
            // the self pair has dx = dy = dz = 0 exactly; capping 1/r keeps
            // its weight finite, so its term is 0 without a test
            const float ri = fminf(__builtin_amdgcn_rsqf(r2), kInvRCap);
            const float w = (pj.w * ri) * (ri * ri);
            if constexpr (DIAG) {
                if (jbase + kb + k != i) {
                    const float qq = ri4.w * pj.w;
                    a.S += (double)(fabsf(qq) * ri * ri);
                    a.Uc += 0.5 * (double)(qq * ri);
                }
            }
            bx = fmaf(w, dx, bx);
            by = fmaf(w, dy, by);
            bz = fmaf(w, dz, bz);
        }
        flush<COMP>(a, bx, by, bz);
    }
}

// One Lennard-Jones pair (section 2.1: truncated at lj_cut sigma_ij, not
// shifted) in FP64 from the exact difference of the (hi, lo) positions, if
// it is within the cutoff.  t64: sigma_ij^2, 24 eps_ij, 4 eps_ij and
// (lj_cut sigma_ij)^2, each kMaxTypes^2 long.  Near the minimum the force is
// a small difference of two large terms; FP32 operands would leave an error
// of ~1e-6 of 24 eps_ij / r there.  Accumulates sum_j g_ij (x_j - x_i) and,
// with DIAG, |f_ij| and half the pair energy.
template <bool DIAG>
__device__ __forceinline__ void lj_pair64(const float4 pj, const float4 lj, const float4 pi,
                                          const float4 li, const double* __restrict__ t64,
                                          int pidx, double L[3], double& S, double& U) {
    const double ex = ((double)pj.x - (double)pi.x) + ((double)lj.x - (double)li.x);
    const double ey = ((double)pj.y - (double)pi.y) + ((double)lj.y - (double)li.y);
    const double ez = ((double)pj.z - (double)pi.z) + ((double)lj.z - (double)li.z);
    const double q2 = ex * ex + ey * ey + ez * ez;
    if (!(q2 < t64[3 * kMaxTypes * kMaxTypes + pidx])) return;
    const double ir2 = 1.0 / q2;
    const double s2 = t64[pidx] * ir2;                         // sigma_ij^2 / r^2
    const double s6 = s2 * s2 * s2;
    const double g = t64[kMaxTypes * kMaxTypes + pidx] * s6 * (2.0 * s6 - 1.0) * ir2;
    L[0] += g * ex;
    L[1] += g * ey;
    L[2] += g * ez;
    if constexpr (DIAG) {
        S += fabs(g) * sqrt(q2);
        U += 0.5 * (t64[2 * kMaxTypes * kMaxTypes + pidx] * s6 * (s6 - 1.0));
    }
}

__device__ __forceinline__ float box_dist2(const Box& a, const Box& b) {
    const float gx = fmaxf(0.f, fmaxf(b.lo.x - a.hi.x, a.lo.x - b.hi.x));
    const float gy = fmaxf(0.f, fmaxf(b.lo.y - a.hi.y, a.lo.y - b.hi.y));
    const float gz = fmaxf(0.f, fmaxf(b.lo.z - a.hi.z, a.lo.z - b.hi.z));
    return gx * gx + gy * gy + gz * gz;
}

// A box whose half-extent is below 255 sigma: positions relative to its
// centre carry at most two FP32 roundings of 2^-17 sigma.  False for NaN or
// infinite boxes.
constexpr float kCompactExtent = 510.f;
__device__ __forceinline__ bool box_compact(const Box& b) {
    return fmaxf(fmaxf(b.hi.x - b.lo.x, b.hi.y - b.lo.y), b.hi.z - b.lo.z) < kCompactExtent;
}

// Coulomb pairs that the symmetric kernel leaves to k_lj: both groups
// charged, near, one of the boxes stretched.  (Whether any particle of the
// one comes near the other's box is tested by both kernels alike.)
__device__ __forceinline__ bool sym_leaves_out(const Box& a, const Box& b) {
    return (!box_compact(a) || !box_compact(b)) && a.lo.w != 0.f && b.lo.w != 0.f;
}

// Squared distance from point p to box b (0 inside; NaN coordinates give 0).
__device__ __forceinline__ float point_box_dist2(const float4& p, const Box& b) {
    const float gx = fmaxf(0.f, fmaxf(b.lo.x - p.x, p.x - b.hi.x));
    const float gy = fmaxf(0.f, fmaxf(b.lo.y - p.y, p.y - b.hi.y));
    const float gz = fmaxf(0.f, fmaxf(b.lo.z - p.z, p.z - b.hi.z));
    return gx * gx + gy * gy + gz * gz;
}

// Lennard-Jones sums of one 64-slot i group, by a workgroup of WAVES
// wavefronts, which share the tests of the boxes and then the near groups.
// Bound by latency and by the FP64
// pair arithmetic: a near group pair has a few hundred pairs in sight and a
// handful in range, so
//   - of a near group's slots only those within range of the i group's box
//     are paired with the 64 i (about an eighth in a dispersed droplet);
//   - those pairs are only screened, in FP32 with a margin; a lane notes its
//     partners in a short list (LDS) and the FP64 terms are evaluated for the
//     lists at once, so the FP64 code runs as often as the longest list is
//     long, not for every slot that some lane has in range.
// Measured against a loop over every slot of the near groups with the FP64
// terms inline: 5000 slots 27.5 -> 14.3 us a launch, 32768 slots 31.3 -> 26.8,
// 250 000 slots 127 -> 118, and the pair loops no longer flag the group pairs
// that hold a pair in range (one operation in fourteen of their near loops).
// Slots without spatial order have all groups near each other, which costs more
// than those flags did: the callers see to the order (order_slots).
// Partners come in the same order whatever the timing, and the wavefronts'
// sums are added in order.
//
// SYM: group pairs that the symmetric Coulomb kernel leaves out, near ones
// with a stretched box, get their Coulomb terms here, in FP64 from the exact
// (hi, lo) differences.
//
// pos .. box point at the droplet's first slot and group; t64 as for
// lj_pair64.  Returns true for the work-items that hold a slot's sums (the
// first wavefront's, lane = slot): sum_j g_ij (x_j - x_i) and, with DIAG, S
// and the energy.
constexpr int kLjList = 8;               // partners a lane holds between evaluations

constexpr int kLjScan = 4;               // boxes / 64 a wavefront tests per round

// LONG: where a type pair's range is beyond kLjLong lengths, most slots in sight
// are in range of many lanes.  Four slots that at least kLjInline of their 256
// lanes have in range are then evaluated where they are met, from LDS, instead of
// from the lists (the partners of a lane keep their order).  A step at 30
// sigma_ij of 11 000 slots 625 -> 501 us, 32 768 1076 -> 912, 64 droplets of 500 to
// 4000 473 -> 359; at 11 sigma_ij (the longest 22) 174 -> 164, 368 -> 350, 192 ->
// 188; at 8 (the longest 16) 110 and 113, 284 and 287, 160 and 170, for the 30
// registers more that it takes: so shorter ranges go without.
constexpr float kLjLong = 20.f;
constexpr int kLjInline = 16;
inline bool lj_long(const PairTable& tab) { return tab.rc2max > kLjLong * kLjLong; }

template <int WAVES, int SUMS, bool LONG>
struct LjShared {
    union {
        struct {
            float4 hi[WAVES][kGroup];            // .w: the slot
            float4 lo[LONG ? WAVES : 1][LONG ? kGroup : 1];   // .w: the type
            int list[WAVES][kLjList][kGroup];
        };
        double red[WAVES][SUMS][kGroup];         // after the last round
    };
    int near[WAVES][kLjScan * kGroup];
    int found[WAVES];
};

template <bool DIAG, bool SYM, int WAVES, bool LONG>
__device__ __forceinline__ bool lj_group(const float4* __restrict__ pos,
                                         const float4* __restrict__ lo,
                                         const int* __restrict__ typ, const Box* __restrict__ box,
                                         int n, int gi, int T, float rc2max,
                                         const double* __restrict__ t64,
                                         LjShared<WAVES, DIAG ? 5 : 3, LONG>& sh,
                                         double (&sums)[DIAG ? 5 : 3]) {
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kGroup);
    const int lane = threadIdx.x % kGroup;
    const int ngroups = (n + kGroup - 1) / kGroup;
    const int i = gi * kGroup + lane;
    const bool live = i < n;
    const float4 pi = live ? pos[i] : make_float4(kFarAway, kFarAway, kFarAway, 0.f);
    const float4 li = live ? lo[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    const int ti = live ? typ[i] : 0;
    const Box bi = box[gi];
    // Box tests, and the FP32 screen of the high words: the range widened by
    // what their rounding and that of the difference move a component at the
    // coordinates a partner of the lane's particle can have (not its box, which
    // one NP thrown far out may stretch); the cutoff itself is decided in FP64.
    // (With the low words in the screen too, a second LDS read for each
    // candidate, the groups of 8200 unsorted droplets of 1000 took 4.05 ms, 2.8
    // before the lists; so a step of them takes 6.3 ms, 6.9 then.)
    const float cull2 = rc2max * 1.0001f;
    const float reach = sqrtf(cull2);
    const float far = fmaxf(fabsf(pi.x), fmaxf(fabsf(pi.y), fabsf(pi.z)));
    const float wide = reach + (far + reach) * 0x1p-20f;
    const float screen = wide * wide;
    double L[3] = {0.0, 0.0, 0.0};
    double S = 0.0, U = 0.0;
    int cnt = 0;                                 // partners in this lane's list
    auto evaluate = [&]() {
        for (int t = 0; __any(t < cnt); ++t) {
            if (t < cnt) {
                const int j = sh.list[w][t][lane];
                lj_pair64<DIAG>(pos[j], lo[j], pi, li, t64, ti * T + typ[j], L, S, U);
            }
        }
        cnt = 0;
    };
    // one near group g: its slots (hj of lane), its box
    auto visit = [&](int g, float4 hj, const Box& bj) {
        if (!__any(live && point_box_dist2(pi, bj) < cull2)) return;
        const int j = g * kGroup + lane;
        const unsigned long long jclose = __ballot(j < n && point_box_dist2(hj, bi) < cull2);
        if (jclose == 0ull) return;
        // the close slots, packed; .w carries the slot; padded to a
        // multiple of four with filler (slot -1; its distance alone would not
        // keep it out of a range of 1e18 sigma or of none)
        const int at = __popcll(jclose & ((1ull << lane) - 1ull));
        const int m4 = (__popcll(jclose) + 3) & ~3;
        hj.w = __int_as_float(j);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if ((jclose >> lane) & 1ull) sh.hi[w][at] = hj;
        if (lane >= __popcll(jclose) && lane < m4)
            sh.hi[w][lane] = make_float4(kFarAway, kFarAway, kFarAway, __int_as_float(-1));
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        bool staged = false;                     // the low words and types too
        for (int k0 = 0; k0 < m4; k0 += 4) {
            // four slots in flight: the loop is bound by LDS latency
            float r2[4];
            int jj[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 pj = sh.hi[w][k0 + k];
                const float dx = pj.x - pi.x, dy = pj.y - pi.y, dz = pj.z - pi.z;
                r2[k] = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                jj[k] = __float_as_int(pj.w);
            }
            bool in[4], any = false;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                in[k] = live && !(r2[k] >= screen) && jj[k] != i && jj[k] >= 0;
                any = any || in[k];
            }
            if (!__any(any)) continue;
            if constexpr (LONG) {
                int pass = 0;
#pragma unroll
                for (int k = 0; k < 4; ++k) pass += __popcll(__ballot(in[k]));
                if (pass >= kLjInline) {
                    evaluate();                  // the partners met before
                    if (!staged) {
                        if ((jclose >> lane) & 1ull) {
                            float4 l = lo[j];
                            l.w = __int_as_float(typ[j]);
                            sh.lo[w][at] = l;
                        }
                        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                        __builtin_amdgcn_wave_barrier();
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                        staged = true;
                    }
                    float4 pj[4], qj[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        pj[k] = sh.hi[w][k0 + k];
                        qj[k] = sh.lo[w][k0 + k];
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (in[k])
                            lj_pair64<DIAG>(pj[k], qj[k], pi, li, t64,
                                            ti * T + __float_as_int(qj[k].w), L, S, U);
                    continue;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (in[k]) sh.list[w][cnt++][lane] = jj[k];
            if (__any(cnt > kLjList - 4)) evaluate();
        }
        if (SYM && sym_leaves_out(bi, bj)) {
            for (int k = 0; k < min(kGroup, n - g * kGroup); ++k) {
                const float4 pj = pos[g * kGroup + k];
                const float4 qj = lo[g * kGroup + k];
                const double ex = ((double)pj.x - (double)pi.x) + ((double)qj.x - (double)li.x);
                const double ey = ((double)pj.y - (double)pi.y) + ((double)qj.y - (double)li.y);
                const double ez = ((double)pj.z - (double)pi.z) + ((double)qj.z - (double)li.z);
                const double q2 = ex * ex + ey * ey + ez * ez;
                if (live && q2 > 0.0) {
                    const double f = (double)pi.w * (double)pj.w / (q2 * sqrt(q2));
                    L[0] += f * ex;
                    L[1] += f * ey;
                    L[2] += f * ez;
                }
            }
        }
    };
    // Rounds of kLjScan x 64 boxes per wavefront: each notes the near groups,
    // then all share the notes round-robin.
    for (int r0 = 0; r0 < ngroups; r0 += WAVES * kLjScan * kGroup) {
        int found = 0;
        for (int k = 0; k < kLjScan; ++k) {
            const int gc = r0 + (k * WAVES + w) * kGroup + lane;
            const bool near = gc < ngroups && box_dist2(bi, box[min(gc, ngroups - 1)]) < cull2;
            const unsigned long long m = __ballot(near);
            if (near) sh.near[w][found + __popcll(m & ((1ull << lane) - 1ull))] = gc;
            found += __popcll(m);
        }
        if (lane == 0) sh.found[w] = found;
        __syncthreads();
        int skip = w;                            // next of the notes that is this wavefront's
        for (int v = 0; v < WAVES; ++v) {
            const int cntv = __builtin_amdgcn_readfirstlane(sh.found[v]);
            int q = skip;
            if (q < cntv) {
                // a group's slots are loaded while the one before is screened
                int g = __builtin_amdgcn_readfirstlane(sh.near[v][q]);
                float4 h = pos[min(g * kGroup + lane, n - 1)];
                Box b = box[g];
                while (q < cntv) {
                    const int gc = g;
                    const float4 hc = h;
                    const Box bc = b;
                    q += WAVES;
                    if (q < cntv) {
                        g = __builtin_amdgcn_readfirstlane(sh.near[v][q]);
                        h = pos[min(g * kGroup + lane, n - 1)];
                        b = box[g];
                    }
                    visit(gc, hc, bc);
                }
            }
            skip = q - cntv;
        }
        __syncthreads();
    }
    evaluate();
    __syncthreads();
    sh.red[w][0][lane] = L[0];
    sh.red[w][1][lane] = L[1];
    sh.red[w][2][lane] = L[2];
    if constexpr (DIAG) {
        sh.red[w][3][lane] = S;
        sh.red[w][4][lane] = U;
    }
    __syncthreads();
    if (w != 0 || !live) return false;
    for (int c = 0; c < (DIAG ? 5 : 3); ++c) {
        sums[c] = 0.0;
        for (int v = 0; v < WAVES; ++v) sums[c] += sh.red[v][c][lane];
    }
    return true;
}

// lj_group with the type constants staged in LDS first (a whole workgroup).
template <int WAVES, int SUMS, bool LONG>
struct LjBlock {
    double t64[4 * kMaxTypes * kMaxTypes];
    LjShared<WAVES, SUMS, LONG> g;
};

template <bool DIAG, bool SYM, int WAVES, bool LONG>
__device__ __forceinline__ bool lj_block(const float4* __restrict__ pos,
                                         const float4* __restrict__ lo,
                                         const int* __restrict__ typ, const Box* __restrict__ box,
                                         int n, int gi, const PairTable& tab,
                                         LjBlock<WAVES, DIAG ? 5 : 3, LONG>& sh,
                                         double (&sums)[DIAG ? 5 : 3]) {
    for (int k = threadIdx.x; k < kMaxTypes * kMaxTypes; k += WAVES * kGroup) {
        sh.t64[k] = tab.sig2d[k];
        sh.t64[kMaxTypes * kMaxTypes + k] = tab.e24d[k];
        sh.t64[2 * kMaxTypes * kMaxTypes + k] = tab.e4d[k];
        sh.t64[3 * kMaxTypes * kMaxTypes + k] = tab.rc2d[k];
    }
    __syncthreads();
    return lj_group<DIAG, SYM, WAVES, LONG>(pos, lo, typ, box, n, gi, tab.T, tab.rc2max, sh.t64,
                                            sh.g, sums);
}

}  // namespace pair
}  // namespace ld
