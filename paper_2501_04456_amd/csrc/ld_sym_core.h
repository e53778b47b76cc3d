// The all-pairs Coulomb sum with every unordered pair evaluated once
// (Newton's third law), for droplets large enough to fill the chip with it.
//
// What bounds it: FP32 VALU issue.  A pair costs 3 differences, 3 for r^2,
// v_rsq_f32, 2 for r^-3, 2 for the two charge weights and 6 for the two
// sums -- 16 operations and a root for two forces, where the one-sided loop
// (k_pair) takes 12 and a root for each.
//
// Layout.  A wavefront holds the 64 rows of one slot group I, 16 rows in
// the registers of each of its four 16-lane groups (position relative to
// the centre of I's box, and charge: 64 VGPRs, with 48 for their sums), and
// streams column groups J past them, 16 columns at a time, one column per
// lane: a lane meets 16 rows per column, so each of the 64 x 16 pairs of a
// column tile is met by one lane.  Row sums stay in the lane until the end;
// a column's sum over the 64 rows is finished per column tile by adding the
// four lane groups (v_permlane32_swap, v_permlane16_swap: 6 operations per
// 16 pairs).  Rotating columns through the lanes by DPP instead costs a
// half-rate operation per value and measured no faster than k_pair.
// Measured, this kernel against k_pair (same box): 250 000 slots, 200 000 of
// them charged, 10.85 -> 8.05 ms a launch; 32768 charged slots, 331 -> 250 us.
// The loop alone runs at 29 clocks (2.4 GHz) per 64 ordered pairs per SIMD,
// k_pair's at 43, and no faster with two or four wavefronts per SIMD than
// with the three its 160 VGPRs leave.
//
// Blocks.  jb consecutive groups (4 or 8) make a block; a workgroup of
// kSymWaves wavefronts takes the rows of mA blocks against a run of column
// blocks.  In a column block its wavefronts start at different groups and
// go round, a barrier every jb / kSymWaves groups, so the FP64 column sums in
// LDS have one writer at a time and a fixed order.  Block pairs are shared out
// cyclically (a takes b = a + 1 .. a + nbc/2 mod nbc), so every row block
// has the same work and each unordered pair of blocks one owner.
//
// Sums.  A row's FP32 sum is 16 columns a lane (blocks of 4 groups) or 32 (of
// 8) and a tree of four levels over the 16 lanes, a column's 16 rows a lane and
// a tree of two levels; all go on in FP64.  The longest run of roundings is 36,
// 20 and 18, where the one-sided loops' blocks of 32 terms have 32; the error
// against FP64 is smaller, as the positions are relative to a near centre
// (Coulomb alone, rms of |dF| / S: 12 288 slots 3.10e-8 one-sided, 2.69e-8 so,
// 32 768 3.05 and 1.88, 81 919 4.05 and 2.20, 250 000 2.76 and 1.85; ensembles
// of 500 to 8000 6.31 and 6.27, 300 to 600 8.63 and 8.63).  The 16 lanes of
// blocks of 8 added in FP64: 1.84e-8 at 250 000, and 1.2 % of a step.  The
// partial sums a workgroup
// stores are FP64: one per column block and row super-block, one per row
// and chunk of column blocks; the update adds them in slot order, so the
// forces do not depend on timing.
//
// Near pairs take the same loop: positions relative to the centre of I's box
// carry the rounding of tens of sigma.  Where a box is stretched (half-extent
// of 255 sigma or more: NPs thrown out by a blown-up step), they would lose
// too much: pairs with a stretched I then use the high words, and pairs of
// groups near each other of which one is stretched are left to k_lj, which
// takes their Coulomb terms from the exact (hi, lo) differences in FP64.
// Groups without charge have no Coulomb terms and are not visited.
//
// Slots in no spatial order (kExact: ensembles of more droplets than the sort
// key holds) have boxes as wide as the droplet, where positions relative to a
// centre would lose up to 2^-17 sigma a component: every pair then takes the
// exact differences of the high and low words, the rows' low words from LDS
// (a lane's 64 row words and 48 sums leave no registers for them), and no
// pair is left to k_lj.
#pragma once

#include "ld_pair_core.h"

namespace ld {
namespace sym {

using namespace pair;

constexpr int kW = kSymWaves;
constexpr int kRows = 16;                  // rows per lane

// Every how many workgroups of a launch one takes a Lennard-Jones group while
// there are any.  An odd number: workgroups go to the 8 XCDs in turn and there
// to 4 shader engines in turn, so that groups every second or fourth workgroup
// leave half or a quarter of the engines without Coulomb tasks (65 536 charged
// slots stepped 1.02 ms so and step 0.97, 200 000 stepped 11.3 and step 8.3).
inline int lj_stride(int lj, int tasks) {
    const int k = lj > 0 ? (lj + tasks) / lj : 1;
    return k % 2 ? k : k - 1;
}

// What a workgroup works on: one droplet's slots and boxes, and its force
// partials F[slot][3][stride], already at the droplet's first slot.
struct View {
    const float4* pos;
    const float4* lo;
    const Box* box;
    int n, ngroups;
    float cull2;                           // (largest LJ range)^2 with a margin
    double* F;
    size_t stride;
    int nbc, mA, nA, nds;                  // as in SymPlan
};

constexpr int kLoPitch = kRows + 1;         // the four lane groups' rows in different banks

template <int kJB, bool kExact = false>
struct Shared {
    float4 sx[kW][kGroup];
    float sj[kW][4 * kGroup];
    double acc[kJB][3][kGroup];            // column sums of the current block
    float4 cl[kExact ? kW : 1][kExact ? kGroup : 1];          // columns' low words
    float4 rl[kExact ? kW : 1][kExact ? 4 * kLoPitch : 1];    // rows' low words
};

__device__ __forceinline__ void sync_wave() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ bool stretched(const Box& b) { return !box_compact(b); }

// Slot s relative to o, (hi - o) + lo, or its high words (words); filler past
// the last slot.
__device__ __forceinline__ float4 rel_slot(const View& A, int s, bool words, float3 o) {
    if (s >= A.n) return make_float4(kFarAway, kFarAway, kFarAway, 0.f);
    const float4 h = A.pos[s];
    if (words) return h;
    const float4 lw = A.lo[s];
    return make_float4((h.x - o.x) + lw.x, (h.y - o.y) + lw.y, (h.z - o.z) + lw.z, h.w);
}

__device__ __forceinline__ float4 low_words(const View& A, int s) {
    return s < A.n ? A.lo[s] : make_float4(0.f, 0.f, 0.f, 0.f);
}

// a.lo + a.hi in lanes 0..31, b.lo + b.hi in lanes 32..63.
__device__ __forceinline__ float fold32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// The same between the odd and even 16-lane rows.
__device__ __forceinline__ float fold16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}

// Sums over the 16 lanes of a row of 16 values each: lane c returns the sum
// of v[c].  A step keeps the half of the values that the lane's bit names and
// adds the partner's copy of it; the partners (c^15, c^7, c^2, c^1) differ
// in the step's bit and agree in the bits already used.
__device__ __forceinline__ float fold_rows(const float (&v)[kRows], int c) {
    const bool b3 = c & 8, b2 = c & 4, b1 = c & 2, b0 = c & 1;
    float p[8], q[4], r[2];
#pragma unroll
    for (int k = 0; k < 8; ++k)
        p[k] = (b3 ? v[k + 8] : v[k]) + dpp<0x140>(b3 ? v[k] : v[k + 8]);   // row_mirror
#pragma unroll
    for (int k = 0; k < 4; ++k)
        q[k] = (b2 ? p[k + 4] : p[k]) + dpp<0x141>(b2 ? p[k] : p[k + 4]);   // row_half_mirror
#pragma unroll
    for (int k = 0; k < 2; ++k)
        r[k] = (b1 ? q[k + 2] : q[k]) + dpp<0x4e>(b1 ? q[k] : q[k + 2]);    // lanes 2 3 0 1
    return (b0 ? r[1] : r[0]) + dpp<0xb1>(b0 ? r[0] : r[1]);                // lanes 1 0 3 2
}

// One 64 x 64 tile: rows in P (registers), columns in sx (LDS, lane order).
// Row sums go on in S; the column sums, 64 x {x, y, z}, into sj.  kTiny keeps
// the self pair's weight finite (its differences are 0) and is far below the
// r^2 of any two particles; one loop serves near and far tiles alike, as two
// would each want their own registers for the 48 row sums.  kExact: cl, rl
// hold the low words (rl in steps of kLoPitch a lane group).
template <bool kExact>
__device__ __forceinline__ void tile(const float4* __restrict__ sx, const float4* __restrict__ cl,
                                     const float4* __restrict__ rl, float* __restrict__ sj,
                                     const float4 (&P)[kRows], float (&Sx)[kRows],
                                     float (&Sy)[kRows], float (&Sz)[kRows], int g, int c) {
#pragma unroll 1
    for (int ct = 0; ct < 4; ++ct) {
        const float4 v = sx[16 * ct + c];
        float4 vl = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (kExact) vl = cl[16 * ct + c];
        float jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            float dx = v.x - P[r].x, dy = v.y - P[r].y, dz = v.z - P[r].z;
            if constexpr (kExact) {
                const float4 l = rl[g * kLoPitch + r];
                dx += vl.x - l.x;
                dy += vl.y - l.y;
                dz += vl.z - l.z;
            }
            const float r2 = fmaf(dz, dz, fmaf(dy, dy, fmaf(dx, dx, kTiny)));
            const float ri = __builtin_amdgcn_rsqf(r2);
            const float w = ri * (ri * ri);
            const float wi = w * v.w, wj = w * P[r].w;
            Sx[r] = fmaf(wi, dx, Sx[r]);
            Sy[r] = fmaf(wi, dy, Sy[r]);
            Sz[r] = fmaf(wi, dz, Sz[r]);
            jx = fmaf(wj, dx, jx);
            jy = fmaf(wj, dy, jy);
            jz = fmaf(wj, dz, jz);
        }
        // lane group 0: x, 1: y, 2: z of the 16 columns (3: nothing of use)
        sj[g * kGroup + 16 * ct + c] = fold16(fold32(jx, jz), fold32(jy, 0.f));
    }
}

// Does block pair (a, b), taken from row block a, belong to a?  (a != b)
__device__ __forceinline__ bool owns(int a, int b, int nbc) {
    int d = b - a;
    if (d < 0) d += nbc;
    return 2 * d < nbc || (2 * d == nbc && a < b);
}

// One task: the rows of super-block sa against the column super-blocks at
// distances s0 .. s1 - 1; row partials go to slot 1 + nds + chunk, column
// partials to slot 1 + distance.
template <int kJB, bool kExact = false>
__device__ __forceinline__ void task(const View& A, int sa, int chunk, int s0, int s1,
                                     Shared<kJB, kExact>& sh) {
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kGroup);
    const int l = threadIdx.x % kGroup, g = l >> 4, c = l & 15;
    const size_t n = A.stride;
    const float cull2 = A.cull2;
    const int a0 = sa * A.mA, a1 = min(a0 + A.mA, A.nbc);
    double* Fr = A.F + (size_t)(1 + A.nds + chunk) * 3 * n;    // the rows' partials
    for (int i = a0 * kJB * kGroup + (int)threadIdx.x; i < min(a1 * kJB * kGroup, A.n);
         i += 64 * kW)
        for (int k = 0; k < 3; ++k) Fr[k * n + i] = 0.0;
    for (int ds = s0; ds < s1; ++ds) {
        const int sb = (sa + ds) % A.nA;
        const int b0 = sb * A.mA, b1 = min(b0 + A.mA, A.nbc);
        for (int b = b0; b < b1; ++b) {
            __syncthreads();                     // the last block's sums are read
            for (int k = threadIdx.x; k < kJB * 3 * kGroup; k += 64 * kW) (&sh.acc[0][0][0])[k] = 0.0;
            __syncthreads();
            for (int a = a0; a < a1; ++a) {
                if (a != b && !owns(a, b, A.nbc)) continue;
#pragma unroll 1
                for (int ii = 0; ii < kJB / kW; ++ii) {
                    const int gl = ii * kW + w;           // group within the block
                    const int gi = a * kJB + gl;
                    const bool ilive = gi < A.ngroups;
                    Box bi;
                    bool ist = false;
                    float4 P[kRows];
                    float3 o = make_float3(0.f, 0.f, 0.f);
                    if (ilive) {
                        bi = A.box[gi];
                        ist = kExact || stretched(bi);
                        if (!ist)
                            o = make_float3(0.5f * (bi.lo.x + bi.hi.x), 0.5f * (bi.lo.y + bi.hi.y),
                                            0.5f * (bi.lo.z + bi.hi.z));
                    }
                    // rows through LDS: a lane's 16 rows are 16-lane broadcasts
                    sync_wave();
                    sh.sx[w][l] = rel_slot(A, gi * kGroup + l, ist, o);
                    if constexpr (kExact) sh.rl[w][g * kLoPitch + c] = low_words(A, gi * kGroup + l);
                    sync_wave();
                    float Sx[kRows], Sy[kRows], Sz[kRows];
#pragma unroll
                    for (int r = 0; r < kRows; ++r) {
                        P[r] = sh.sx[w][g * kRows + r];
                        Sx[r] = Sy[r] = Sz[r] = 0.f;
                    }
#pragma unroll 1
                    for (int k = 0; k < kJB; ++k) {
                        const int jl = (k + w * (kJB / kW)) % kJB;
                        const int gj = b * kJB + jl;
                        bool take = ilive && gj < A.ngroups;
                        if (a == b) {                     // within a block, cyclic too
                            const int d = (jl - gl + kJB) % kJB;
                            take = take && (2 * d < kJB || (2 * d == kJB && gl < jl));
                        }
                        Box bj;
                        if (take) {
                            bj = A.box[gj];
                            take = bi.lo.w != 0.f && bj.lo.w != 0.f;   // both charged
                        }
                        if (__builtin_amdgcn_readfirstlane((int)take)) {
                            const int j = gj * kGroup + l;
                            const float4 q = rel_slot(A, j, ist, o);
                            float4 ql = make_float4(0.f, 0.f, 0.f, 0.f);
                            if constexpr (kExact) ql = low_words(A, j);
                            // near pairs with a stretched box are left to k_lj, which
                            // decides by the same tests (such a box is near almost
                            // everything, so the particles are tested one by one)
                            bool exact = false;
                            if (!kExact && sym_leaves_out(bi, bj) && box_dist2(bi, bj) < cull2) {
                                const int i = gi * kGroup + l;
                                exact = __any(i < A.n && point_box_dist2(A.pos[min(i, A.n - 1)],
                                                                         bj) < cull2) &&
                                        __any(j < A.n && point_box_dist2(A.pos[min(j, A.n - 1)],
                                                                         bi) < cull2);
                            }
                            if (!exact) {
                                sync_wave();
                                sh.sx[w][l] = q;
                                if constexpr (kExact) sh.cl[w][l] = ql;
                                sync_wave();
                                tile<kExact>(sh.sx[w], sh.cl[kExact ? w : 0],
                                             sh.rl[kExact ? w : 0], sh.sj[w], P, Sx, Sy, Sz, g, c);
                                sync_wave();
                                if (gi != gj) {
                                    for (int d = 0; d < 3; ++d)
                                        sh.acc[jl][d][l] += (double)sh.sj[w][d * kGroup + l];
                                }
                            }
                        }
                        // the wavefronts are kJB / kW groups apart
                        if (k % (kJB / kW) == kJB / kW - 1) __syncthreads();
                    }
                    // rows: F_i -= q_i sum_j q_j r^-3 (x_j - x_i)
                    const float fx = fold_rows(Sx, c), fy = fold_rows(Sy, c),
                                fz = fold_rows(Sz, c);
                    const int i = gi * kGroup + l;         // lane (g, c) holds row 16 g + c
                    if (i < A.n) {
                        const double qi = (double)A.pos[i].w;
                        Fr[i] -= qi * (double)fx;
                        Fr[n + i] -= qi * (double)fy;
                        Fr[2 * n + i] -= qi * (double)fz;
                    }
                }
            }
            // columns: F_j += q_j sum_i q_i r^-3 (x_j - x_i)
            double* Fc = A.F + (size_t)(1 + ds) * 3 * n;
            for (int jl = w; jl < kJB; jl += kW) {
                const int j = (b * kJB + jl) * kGroup + l;
                if (j < A.n) {
                    const double qj = (double)A.pos[j].w;
                    for (int d = 0; d < 3; ++d) Fc[d * n + j] = qj * sh.acc[jl][d][l];
                }
            }
        }
    }
}

}  // namespace sym
}  // namespace ld
