// Cell lists by counting, shared by the truncated scheme and the statistics:
// count every slot into its cell, scan the counts, list the slots cell by
// cell, and order each cell's by slot number (the caller's placing kernel),
// so the result does not depend on the atomics' order.  And the walk over the
// 27 cells around a particle.
#pragma once

#include "ld_internal.h"

namespace ld {
namespace cells {

constexpr int kMaxCells = 64;           // per axis
constexpr int kNC = kMaxCells * kMaxCells * kMaxCells;
constexpr int kCoarse = 1024;           // cells of a coarse count (a scan workgroup's share)
constexpr int kWin = 4;                 // candidates loaded together
constexpr int kWide = 8;                // and in crowded cells

struct Grid {
    double L;                           // half width of the cube the cells divide
    double hc;                          // cell side (>= the largest pair range)
    int Gc;                             // cells per axis
};

// The integer workspace.  count and coarse are zero between sorts; mx holds
// bits of largest |coordinate|s (of three consecutive steps).
struct Work {
    int* count;                         // [kNC]
    int* coarse;                        // [kNC / kCoarse]
    int* first;                         // [kNC + 1] first slot of every cell
    unsigned* mx;                       // [3]
};
constexpr size_t kWorkInts = (size_t)kNC + kNC / kCoarse + kNC + 1 + 3;

inline Work work_at(int* b) {
    return Work{b, b + kNC, b + kNC + kNC / kCoarse,
                reinterpret_cast<unsigned*>(b + kNC + kNC / kCoarse + kNC + 1)};
}

// The grid of a largest coordinate m for pairs within range r.  Coordinates
// beyond L fall into the edge cells, which keeps any two particles closer
// than hc in adjacent cells, so the m of an earlier step is as right as the
// present one.
__device__ __forceinline__ Grid grid_of(float m, double r) {
    Grid g;
    m = fmaxf(m, 1e-3f);
    g.L = (double)(m * 1.0009765625f);
    int G = (int)floor(2.0 * g.L / r);
    G = G < 1 ? 1 : (G > kMaxCells ? kMaxCells : G);
    g.Gc = G;
    g.hc = 2.0 * g.L / G;
    return g;
}

__device__ __forceinline__ int cell1(double x, double L, double h, int G) {
    int c = (int)floor((x + L) / h);
    return c < 0 ? 0 : (c > G - 1 ? G - 1 : c);
}

// Squared FP32 screen from hi words for pairs within `range`: widened by the
// screen's worst rounding (coordinates within m: hi rounding and the FP32
// difference move each component by <= L 2^-22, the squared sum by a few
// ulp), so every pair the FP64 test keeps passes it.
__device__ __forceinline__ float screen2(double range, float m) {
    const double w = range + (double)(fmaxf(m, 1e-3f) * 1.0009765625f) * 0x1p-20;
    return (float)(w * w * (1.0 + 0x1p-18));
}

// Count slot s (live lanes of one wavefront) into its cell.  With COARSE, for
// slots in cell order, the coarse counts too: one atomic per distinct coarse
// cell of the wavefront.  (Slots in Hilbert order meet more of them: 250 000
// took 52 us to count that way, and take 15 with launch_coarse after it.)
template <bool COARSE>
__device__ __forceinline__ void bin(const Grid& g, bool live, int s, const double x[3],
                                    const Work& C, int* cell, int* rank) {
    const int c = live ? (cell1(x[2], g.L, g.hc, g.Gc) * g.Gc + cell1(x[1], g.L, g.hc, g.Gc)) *
                                 g.Gc + cell1(x[0], g.L, g.hc, g.Gc)
                       : -1;
    if (live) {
        cell[s] = c;
        rank[s] = atomicAdd(&C.count[c], 1);
    }
    unsigned long long left = COARSE ? __ballot(live) : 0ull;
    while (left) {
        const int k = __shfl(c, (int)__builtin_ctzll(left)) / kCoarse;
        const unsigned long long same = __ballot(live && c / kCoarse == k) & left;
        if ((int)(threadIdx.x % 64) == (int)__builtin_ctzll(left))
            atomicAdd(&C.coarse[k], __popcll(same));
        left &= ~same;
    }
}

// The largest coordinate of the 64 partial maxima of launch_absmax.
__device__ __forceinline__ float absmax_of(const float* __restrict__ part) {
    float m = part[threadIdx.x % 64];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    return m;
}

// Place of list entry s of cell c: the cell's first slot and the number of
// smaller slots listed there.
__device__ __forceinline__ int place(const int* __restrict__ first, const int* __restrict__ list,
                                     int c, int s) {
    const int f = first[c], e = first[c + 1];
    int d = f;
    for (int q = f; q < e; ++q) d += list[q] < s;
    return d;
}

// The candidates around particle i of cell c (all lanes of a wavefront call;
// LANES of them share a particle): the 27 cells around the cell, whose
// x-rows are runs of consecutive slots, so nine ranges cover them; with HALF
// those after i only.  A candidate whose hi word passes the FP32 screen is
// listed, and eval(j) is called for the listed ones when the walk is over or
// a list full: few pass, and evaluated where they are met nearly every
// candidate would cost a wavefront the body.
template <int LANES, bool HALF, int BLOCK, int LIST, class Eval>
__device__ __forceinline__ void walk(const float4* __restrict__ pos,
                                     const int* __restrict__ first, int G, bool live, int i, int c,
                                     const float4& hi, float screen, int (*list)[BLOCK],
                                     Eval eval) {
    const int t = threadIdx.x, sub = t % LANES;
    int r0[9], r1[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) r0[k] = r1[k] = 0;
    if (live) {
        const int cx = c % G, cy = (c / G) % G, cz = c / (G * G);
        const int x0 = cx > 0 ? cx - 1 : 0, x1 = cx < G - 1 ? cx + 1 : G - 1;
#pragma unroll
        for (int k = 0; k < 9; ++k) {                  // independent loads
            const int z = cz + k / 3 - 1, y = cy + k % 3 - 1;
            const bool in = z >= 0 && z < G && y >= 0 && y < G;
            const int row = (z * G + y) * G;
            r0[k] = in ? first[row + x0] : 0;
            r1[k] = in ? first[row + x1 + 1] : 0;
        }
    }
    int cnt = 0;                                       // the lane's listed partners
    auto flush = [&]() {
        for (int k = 0; __any(k < cnt); ++k)
            if (k < cnt) eval(list[k][t]);
        cnt = 0;
    };
    auto screened = [&](const float4& hj) {
        const float dx = hj.x - hi.x, dy = hj.y - hi.y, dz = hj.z - hi.z;
        return fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    };
    auto meet = [&](int j, bool valid, const float4& hj) {
        if (valid && j != i && screened(hj) < screen) list[cnt++][t] = j;
    };
#pragma unroll
    for (int k = 0; k < 9; ++k) r0[k] = (HALF ? max(r0[k], i + 1) : r0[k]) + sub;
    if constexpr (LANES > 1) {
        // every row's first LANES candidates in flight together, which few
        // rows outlast; a list has room for nine
        static_assert(LIST >= 9 + kWin, "room for the first candidates");
        float4 hq[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) hq[k] = pos[r0[k] < r1[k] ? r0[k] : 0];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            meet(r0[k], r0[k] < r1[k], hq[k]);
            r0[k] += LANES;
        }
        if (__any(cnt > LIST - kWin)) flush();
    }
    // Crowded cells (one particle thrown far out makes all cells wide) are bound
    // by the screen, which next to nobody passes: full windows of kWide candidates
    // at one address, looked at again only where the least distance passes.  A
    // step of 100 000 with a particle 3000 (1e6) sigma out: 5.5 (20) ms in windows
    // of kWin, 2.2 (8.6) so; of 60 000 4.3 and 1.5.
    const bool crowded = LANES == 1 && __any(r1[4] - r0[4] > 8 * kWide);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        if (crowded) {
            static_assert(LIST >= 2 * kWide, "room for a window");
            while (__any(r0[k] + kWide <= r1[k])) {
                const bool full = r0[k] + kWide <= r1[k];
                const float4* p = pos + (full ? r0[k] : 0);
                float4 hq[kWide];
#pragma unroll
                for (int u = 0; u < kWide; ++u) hq[u] = p[u];
                float least = INFINITY;
#pragma unroll
                for (int u = 0; u < kWide; ++u) least = fminf(least, screened(hq[u]));
                if (__any(full && least < screen)) {
#pragma unroll
                    for (int u = 0; u < kWide; ++u) meet(r0[k] + u, full, hq[u]);
                    if (__any(cnt > LIST - kWide)) flush();
                }
                if (full) r0[k] += kWide;
            }
        }
        for (int j = r0[k]; __any(j < r1[k]); j += kWin * LANES) {
            float4 hq[kWin];                           // in flight together
#pragma unroll
            for (int u = 0; u < kWin; ++u) hq[u] = pos[j + u * LANES < r1[k] ? j + u * LANES : 0];
#pragma unroll
            for (int u = 0; u < kWin; ++u) meet(j + u * LANES, j + u * LANES < r1[k], hq[u]);
            if (__any(cnt > LIST - kWin)) flush();
        }
    }
    flush();
}

// Largest |coordinate| as 64 partial maxima; also clears count.
hipError_t launch_absmax(const float4* pos, int n, float* part, const Work& C, hipStream_t s);
// Coarse counts from the counts.
hipError_t launch_coarse(const Work& C, hipStream_t s);
// First slots from the counts of the grid of mx[grid_mx] (counts and mx[next_mx]
// end zero); advances the step clock first by adv_dt > 0.
hipError_t launch_scan(const Work& C, int grid_mx, int next_mx, double r, DevState* st,
                       double adv_dt, hipStream_t s);
// The slots of every cell, in the order the counting met them; slots with a
// negative cell are in none.
hipError_t launch_list(const int* cell, const int* rank, int n, const Work& C, int* list,
                       hipStream_t s);

}  // namespace cells
}  // namespace ld
