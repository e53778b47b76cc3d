// Aggregate statistics the paper extracts in post-processing (section 2.1:
// the number of sub-aggregates and aggregate statistics; section 1: N_surf,
// the number of NPs at the droplet surface; section 3.1: the surface
// fractal dimension, the fractal equation taken at dimension two on the
// sphere).
//
// Sub-aggregates are the connected components of the contact graph, a pair
// in contact when r < contact_factor sigma_ij.  Candidates come from a counted
// cell list (cells of side >= the largest contact distance; the context's slot
// order is left alone, copies of the positions lie in cell order) and are
// united lock-free: a union
// hangs the larger root under the smaller with a compare-and-swap, so parent
// indices only decrease, no cycle can form and every component ends with
// its smallest (cell-sorted) index as root.  The label reported is the
// smallest original index of the component.  Every wait-free retry loop is
// bounded; exceeding the bound raises an error flag instead of spinning.
#include <algorithm>
#include <climits>
#include <cmath>
#include <limits>
#include <vector>

#include "ld_cells.h"
#include "ld_host.h"

namespace ld {

using host::copy_out;
using host::fail;

namespace {

constexpr int kB = 256;
constexpr int kAMaxIter = 1 << 16;      // bound of every retry loop

struct AgTable {
    int T;
    double rc2[kMaxTypes * kMaxTypes];  // (contact_factor sigma_ij)^2
    double half_sigma[kMaxTypes];
};

// Statistics of a call, cleared by its binning: [0] components, [1] aggregates
// of size >= 2, [2] the largest (its size, or packed with its label), [3] error.
using AgRes = unsigned long long;

// Cells of all slots, with SURF of the surface NPs only (| |x| - R | < sigma_t
// / 2; the others' labels are -1 and they are in no list).
template <bool SURF>
__global__ __launch_bounds__(kB) void k_ag_bin(const float4* __restrict__ pos,
                                               const float4* __restrict__ lo,
                                               const int* __restrict__ typ,
                                               const int* __restrict__ oid, int n,
                                               const float* __restrict__ part, double rc, double R,
                                               AgTable tb, cells::Work C, int* cell, int* rank,
                                               int* labels, AgRes* res) {
#pragma clang fp contract(off)
    const float m = cells::absmax_of(part);
    if (blockIdx.x == 0 && threadIdx.x < 4) {
        res[threadIdx.x] = 0ull;
        if (threadIdx.x == 0) C.mx[0] = __float_as_uint(m);
    }
    const int s = blockIdx.x * kB + threadIdx.x;
    bool live = s < n;
    double x[3] = {0.0, 0.0, 0.0};
    if (live) {
        const float4 h = pos[s], l = lo[s];
        x[0] = (double)h.x + (double)l.x;
        x[1] = (double)h.y + (double)l.y;
        x[2] = (double)h.z + (double)l.z;
        if (SURF && !(fabs(sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]) - R) <
                      tb.half_sigma[typ[s]])) {
            live = false;
            cell[s] = -1;
            if (labels) labels[oid[s]] = -1;
        }
    }
    cells::bin<false>(cells::grid_of(m, rc), live, s, x, C, cell, rank);
}

// The listed slots in cell order: positions, type (in lo.w), slot and cell;
// and, unless null, every one its own root.
__global__ __launch_bounds__(kB) void k_ag_place(const float4* __restrict__ pos,
                                                 const float4* __restrict__ lo,
                                                 const int* __restrict__ typ,
                                                 const int* __restrict__ cell,
                                                 const int* __restrict__ list, cells::Work C,
                                                 double rc, int n, float4* shi, float4* slo,
                                                 int* slot, int* scell, int* parent, int* minoid,
                                                 int* size, int* count) {
    const int G = cells::grid_of(__uint_as_float(C.mx[0]), rc).Gc;
    const int m = C.first[G * G * G], k = blockIdx.x * kB + threadIdx.x;
    if (k == 0) *count = m;
    if (k >= m) return;
    const int s = list[k], c = cell[s];
    const float4 h = pos[s];
    float4 l = lo[s];
    l.w = __int_as_float(typ[s]);
    const int d = cells::place(C.first, list, c, s);
    shi[d] = h;
    slo[d] = l;
    slot[d] = s;
    scell[d] = c;
    if (parent) {
        parent[k] = k;
        minoid[k] = INT_MAX;
        size[k] = 0;
    }
}

// Root of a: a bounded walk up the parent links with path halving (a
// non-root's link is moved to its grandparent, still an ancestor with a
// smaller index, so no cycle can form and roots are never written here).
__device__ __forceinline__ int ag_find(int* parent, int a, int* err) {
    for (int it = 0; it < kAMaxIter; ++it) {
        const int p = __hip_atomic_load(&parent[a], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (p == a) return a;
        const int gp = __hip_atomic_load(&parent[p], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (gp != p)
            __hip_atomic_store(&parent[a], gp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        a = gp;
    }
    atomicOr(err, 1);
    return a;
}

__device__ __forceinline__ void ag_unite(int* parent, int a, int b, int* err) {
    for (int it = 0; it < kAMaxIter; ++it) {
        a = ag_find(parent, a, err);
        b = ag_find(parent, b, err);
        if (a == b) return;
        if (a > b) {
            const int x = a;
            a = b;
            b = x;
        }
        if (atomicCAS(&parent[b], b, a) == b) return;   // b was still a root: hung under a
    }
    atomicOr(err, 1);
}

// The particles in cell order, count[0] of them.
struct AgSorted {
    const float4 *hi, *lo;              // lo.w: the type's bits
    const int *slot, *cell, *first, *count;
    const unsigned* mx;
};

// Every contact pair (k, m), m > k in cell order, LANES lanes a particle.
// Bound by the chains of the lock-free unions: 30 011 NPs in patches of 125
// 165 -> 25 us (a lane per particle, FP64 tests of all candidates before),
// 250 000 dispersed ones 83 -> 21.
template <int LANES>
__global__ __launch_bounds__(kB) void k_ag_hook(AgSorted A, AgTable tb, double rc, int* parent,
                                                int* err) {
    // the oracle's operand order, no fused multiply-add: a pair within an ulp
    // of the contact distance lands on the same side in both
#pragma clang fp contract(off)
    constexpr int kList = 16;
    __shared__ int list[kList][kB];
    const int k = blockIdx.x * (kB / LANES) + threadIdx.x / LANES;
    const bool live = k < A.count[0];
    const float m = __uint_as_float(A.mx[0]);
    float4 hi = make_float4(0.f, 0.f, 0.f, 0.f), li = hi;
    int c = 0;
    if (live) {
        hi = A.hi[k];
        li = A.lo[k];
        c = A.cell[k];
    }
    const double xi = (double)hi.x + (double)li.x, yi = (double)hi.y + (double)li.y,
                 zi = (double)hi.z + (double)li.z;
    const int ti = __float_as_int(li.w) * tb.T;
    cells::walk<LANES, true, kB, kList>(
        A.hi, A.first, cells::grid_of(m, rc).Gc, live, k, c, hi, cells::screen2(rc, m), list,
        [&](int j) {
            const float4 hj = A.hi[j], lj = A.lo[j];
            const double ddx = xi - ((double)hj.x + (double)lj.x);
            const double ddy = yi - ((double)hj.y + (double)lj.y);
            const double ddz = zi - ((double)hj.z + (double)lj.z);
            if (ddx * ddx + ddy * ddy + ddz * ddz < tb.rc2[ti + __float_as_int(lj.w)])
                ag_unite(parent, k, j, err);
        });
}

// Roots, and per root the smallest original index (label) and the size.  The
// first few roots of a wavefront are combined over their lanes (a giant
// component costs one atomic per wavefront), the lanes left then go singly.
__global__ __launch_bounds__(kB) void k_ag_roots(int* parent, const int* __restrict__ slot,
                                                 const int* __restrict__ oid,
                                                 const int* __restrict__ count, int* root,
                                                 int* minoid, int* size, int* err) {
    const int k = blockIdx.x * kB + threadIdx.x;
    const bool live = k < *count;
    int r = -1, o = INT_MAX;
    if (live) {
        r = ag_find(parent, k, err);
        root[k] = r;
        o = oid[slot[k]];
    }
    unsigned long long todo = __ballot(live);
    const int lane = threadIdx.x % 64;
    for (int it = 0; it < 4 && todo; ++it) {
        const int leader = __ffsll((long long)todo) - 1;
        const int rl = __shfl(r, leader);
        const unsigned long long same = __ballot(live && r == rl);
        int mo = (same >> lane) & 1ull ? o : INT_MAX;
#pragma unroll
        for (int w = 32; w >= 1; w >>= 1) mo = min(mo, __shfl_xor(mo, w));
        if (lane == leader) {
            atomicMin(&minoid[rl], mo);
            atomicAdd(&size[rl], __popcll(same));
        }
        todo &= ~same;
    }
    if ((todo >> lane) & 1ull) {
        atomicMin(&minoid[r], o);
        atomicAdd(&size[r], 1);
    }
}

// Labels (original order) and the statistics; with SURF the largest is packed
// as size << 32 | (INT_MAX - label), so the maximum is the largest size and,
// among equal sizes, the smallest label.  Few workgroups: each ends with three
// atomics on one line.
template <bool SURF>
__global__ __launch_bounds__(kB) void k_ag_label(const int* __restrict__ root,
                                                 const int* __restrict__ slot,
                                                 const int* __restrict__ oid,
                                                 const int* __restrict__ minoid,
                                                 const int* __restrict__ size,
                                                 const int* __restrict__ count, int* labels,
                                                 AgRes* res) {
    AgRes comp = 0ull, agg = 0ull, big = 0ull;
    const int m = *count;
    for (int k = blockIdx.x * kB + threadIdx.x; k < m; k += gridDim.x * kB) {
        const int r = root[k];
        if (labels) labels[oid[slot[k]]] = minoid[r];
        if (r == k) {
            ++comp;
            agg += size[k] >= 2 ? 1 : 0;
            const AgRes b = SURF ? ((AgRes)size[k] << 32) | (AgRes)(unsigned)(INT_MAX - minoid[k])
                                 : (AgRes)size[k];
            if (b > big) big = b;
        }
    }
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        comp += __shfl_xor(comp, w);
        agg += __shfl_xor(agg, w);
        const AgRes o = __shfl_xor(big, w);
        if (o > big) big = o;
    }
    __shared__ AgRes red[3][kB / 64];
    if (threadIdx.x % 64 == 0) {
        red[0][threadIdx.x / 64] = comp;
        red[1][threadIdx.x / 64] = agg;
        red[2][threadIdx.x / 64] = big;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        AgRes v = 0ull;
        for (int w = 0; w < kB / 64; ++w)
            v = threadIdx.x < 2 ? v + red[threadIdx.x][w]
                                : (red[2][w] > v ? red[2][w] : v);
        if (v && threadIdx.x < 2) atomicAdd(&res[threadIdx.x], v);
        if (v && threadIdx.x == 2) atomicMax(&res[2], v);
    }
}

// N_surf partials per workgroup and type: | |x| - R | < sigma_t / 2.
__global__ __launch_bounds__(kB) void k_ag_surface(const float4* __restrict__ pos,
                                                   const float4* __restrict__ lo,
                                                   const int* __restrict__ typ, int n, double R,
                                                   AgTable tb, long long* part) {
#pragma clang fp contract(off)
    __shared__ int cnt[kMaxTypes];
    if (threadIdx.x < kMaxTypes) cnt[threadIdx.x] = 0;
    __syncthreads();
    const int s = blockIdx.x * kB + threadIdx.x;
    if (s < n) {
        const float4 h = pos[s], l = lo[s];
        const double x = (double)h.x + (double)l.x, y = (double)h.y + (double)l.y,
                     z = (double)h.z + (double)l.z;
        const int t = typ[s];
        if (fabs(sqrt(x * x + y * y + z * z) - R) < tb.half_sigma[t]) atomicAdd(&cnt[t], 1);
    }
    __syncthreads();
    if (threadIdx.x < kMaxTypes) part[(size_t)blockIdx.x * kMaxTypes + threadIdx.x] = cnt[threadIdx.x];
}

// Direction of the surface NP k (FP64 hi + lo) of cell order and whether it
// belongs to the largest component, packed in res[2].
__device__ __forceinline__ bool sf_member(const AgSorted& A, const int* __restrict__ root,
                                          const int* __restrict__ minoid, const AgRes* res, int k,
                                          double u[3], int* type) {
    const int label = INT_MAX - (int)(unsigned)(res[2] & 0xffffffffull);
    if (minoid[root[k]] != label) return false;
    const float4 h = A.hi[k], l = A.lo[k];
    const double x = (double)h.x + (double)l.x, y = (double)h.y + (double)l.y,
                 z = (double)h.z + (double)l.z;
    const double r = sqrt(x * x + y * y + z * z);
    u[0] = x / r;
    u[1] = y / r;
    u[2] = z / r;
    *type = __float_as_int(l.w);
    return true;
}

// Per-workgroup sums over the component's NPs of the unit direction and of
// sigma: dpart[4 * block + {0, 1, 2, 3}].
__global__ __launch_bounds__(kB) void k_sf_sums(AgSorted A, const int* __restrict__ root,
                                                const int* __restrict__ minoid,
                                                const AgRes* __restrict__ res, AgTable tb,
                                                double* dpart) {
    __shared__ double red[4][kB];
    const int k = blockIdx.x * kB + threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (k < A.count[0]) {
        double u[3];
        int ty;
        if (sf_member(A, root, minoid, res, k, u, &ty)) {
            v[0] = u[0];
            v[1] = u[1];
            v[2] = u[2];
            v[3] = 2.0 * tb.half_sigma[ty];
        }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) red[q][threadIdx.x] = v[q];
    __syncthreads();
    for (int w = kB / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) {
#pragma unroll
            for (int q = 0; q < 4; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x < 4) dpart[4 * blockIdx.x + threadIdx.x] = red[threadIdx.x][0];
}

// Per-workgroup sums of the squared angle between each member's direction and
// the mean direction (from the sine and cosine, accurate for small angles).
// Every workgroup adds the k_sf_sums partials itself, in the same order, so
// the host need not come in between.
__global__ __launch_bounds__(kB) void k_sf_theta(AgSorted A, const int* __restrict__ root,
                                                 const int* __restrict__ minoid,
                                                 const AgRes* __restrict__ res,
                                                 const double* __restrict__ dpart,
                                                 double* tpart) {
    __shared__ double red[3][kB];
    double su[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < (int)gridDim.x; b += kB)
        for (int q = 0; q < 3; ++q) su[q] += dpart[4 * (size_t)b + q];
    for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = su[q];
    __syncthreads();
    for (int w = kB / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 3; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
    for (int q = 0; q < 3; ++q) su[q] = red[q][0];
    __syncthreads();
    const double nu = sqrt(su[0] * su[0] + su[1] * su[1] + su[2] * su[2]);
    const double u0x = su[0] / nu, u0y = su[1] / nu, u0z = su[2] / nu;
    const int k = blockIdx.x * kB + threadIdx.x;
    double v = 0.0;
    if (k < A.count[0] && nu > 0.0) {
        double u[3];
        int ty;
        if (sf_member(A, root, minoid, res, k, u, &ty)) {
            const double cx = u[1] * u0z - u[2] * u0y, cy = u[2] * u0x - u[0] * u0z,
                         cz = u[0] * u0y - u[1] * u0x;
            const double th = atan2(sqrt(cx * cx + cy * cy + cz * cz),
                                    u[0] * u0x + u[1] * u0y + u[2] * u0z);
            v = th * th;
        }
    }
    red[0][threadIdx.x] = v;
    __syncthreads();
    for (int w = kB / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) red[0][threadIdx.x] += red[0][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) tpart[blockIdx.x] = red[0][0];
}

constexpr int kRdfMaxBins = 4096;

__global__ __launch_bounds__(kB) void k_ag_zero64(unsigned long long* a, int m) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (k < m) a[k] = 0ull;
}

// Pair-distance histogram of Eq. (6) from the cell-sorted slots (cells of
// side >= r_max): every pair (k, m), m > k in sorted order, over the 27
// cells around k's.  The distance is formed exactly as in the all-pairs
// histogram (FP64 hi + lo, the same operand order, no contraction; the
// squares make it independent of the pair's orientation), so every pair
// falls in the same bin.  250 000 NPs, r_max 10: 70 -> 41 us (60 with two
// lanes a particle).
template <int LANES>
__global__ __launch_bounds__(kB) void k_ag_rdf(AgSorted A, double r_max, int n_bins, double dr,
                                               unsigned long long* counts) {
#pragma clang fp contract(off)
    constexpr int kList = 16;
    __shared__ unsigned int hist[kRdfMaxBins];
    __shared__ int list[kList][kB];
    for (int b = threadIdx.x; b < n_bins; b += kB) hist[b] = 0u;
    __syncthreads();
    const int k = blockIdx.x * (kB / LANES) + threadIdx.x / LANES;
    const bool live = k < A.count[0];
    const float m = __uint_as_float(A.mx[0]);
    float4 hi = make_float4(0.f, 0.f, 0.f, 0.f), li = hi;
    int c = 0;
    if (live) {
        hi = A.hi[k];
        li = A.lo[k];
        c = A.cell[k];
    }
    const double xi = (double)hi.x + (double)li.x, yi = (double)hi.y + (double)li.y,
                 zi = (double)hi.z + (double)li.z;
    cells::walk<LANES, true, kB, kList>(
        A.hi, A.first, cells::grid_of(m, r_max).Gc, live, k, c, hi, cells::screen2(r_max, m),
        list, [&](int j) {
            const float4 hj = A.hi[j], lj = A.lo[j];
            const double ex = xi - ((double)hj.x + (double)lj.x);
            const double ey = yi - ((double)hj.y + (double)lj.y);
            const double ez = zi - ((double)hj.z + (double)lj.z);
            const double r = sqrt(ex * ex + ey * ey + ez * ez);
            if (r < r_max) {
                const int b = (int)floor(r / dr);
                if (b >= 0 && b < n_bins) atomicAdd(&hist[b], 1u);
            }
        });
    __syncthreads();
    for (int b = threadIdx.x; b < n_bins; b += kB)
        if (hist[b]) atomicAdd(&counts[b], (unsigned long long)hist[b]);
}

#define AG_LAUNCH(kernel, grid, block, ...)                                               \
    do {                                                                                  \
        hipLaunchKernelGGL(kernel, grid, block, 0, __VA_ARGS__);                          \
        HIP_TRY(hipGetLastError());                                                       \
    } while (0)

// Scratch of the aggregate calls (allocated on first use, kept by the context).
struct AgBufs {
    int* work;       // the cell lists' workspace
    int* parent;     // [n]
    int* root;       // [n]
    int* minoid;     // [n]
    int* size;       // [n]
    int* labels;     // [n]
    int* slot;       // [n] slots in cell order
    int* count;      // [1] how many
    long long* part; // [blocks * kMaxTypes]
    AgRes* res;      // [4] statistics, with the partial sums right behind
    double* dpart;   // [blocks * 5]
};

constexpr size_t kResDoubles = 32;      // from res to dpart

// Carve the scratch out of one allocation, every piece 256-byte aligned;
// with base == nullptr only the total size is computed.
size_t ag_layout(char* base, size_t n, AgBufs* b) {
    const size_t blocks = (n + kB - 1) / kB;
    size_t off = 0;
    auto take = [&](size_t nbytes) {
        char* q = base ? base + off : nullptr;
        off += (nbytes + 255) / 256 * 256;
        return q;
    };
    b->part = reinterpret_cast<long long*>(take(blocks * kMaxTypes * sizeof(long long)));
    b->res = reinterpret_cast<AgRes*>(take((kResDoubles + blocks * 5) * sizeof(double)));
    b->dpart = base ? reinterpret_cast<double*>(b->res) + kResDoubles : nullptr;
    b->work = reinterpret_cast<int*>(take(cells::kWorkInts * sizeof(int)));
    b->parent = reinterpret_cast<int*>(take(n * sizeof(int)));
    b->root = reinterpret_cast<int*>(take(n * sizeof(int)));
    b->minoid = reinterpret_cast<int*>(take(n * sizeof(int)));
    b->size = reinterpret_cast<int*>(take(n * sizeof(int)));
    b->labels = reinterpret_cast<int*>(take(n * sizeof(int)));
    b->slot = reinterpret_cast<int*>(take(n * sizeof(int)));
    b->count = reinterpret_cast<int*>(take(sizeof(int)));
    return off;
}

ld_status ag_buffers(ld_ctx* c, AgBufs* b) {
    const size_t n = (size_t)c->n;
    if (!c->agg) {
        const size_t bytes = ag_layout(nullptr, n, b);
        if (hipMalloc(&c->agg, bytes) != hipSuccess) {
            c->agg = nullptr;
            return fail(LD_ENOMEM, "cannot allocate the aggregate scratch");
        }
    }
    ag_layout(reinterpret_cast<char*>(c->agg), n, b);
    return LD_OK;
}

// Contact distances (contact_factor sigma_ij)^2 and half diameters; returns
// the largest contact distance.
double ag_table(const ld_ctx* c, double contact_factor, AgTable* tb) {
    tb->T = c->p.n_types;
    double rc = 0.0;
    for (int a = 0; a < tb->T; ++a) {
        for (int q = 0; q < tb->T; ++q) {
            const double d = contact_factor * 0.5 * (c->p.sigma[a] + c->p.sigma[q]);
            tb->rc2[a * tb->T + q] = d * d;
            rc = std::max(rc, d);
        }
        tb->half_sigma[a] = 0.5 * c->p.sigma[a];
    }
    return rc;
}

#define AG_RUN(kernel, grid, ...)                                                         \
    do {                                                                                  \
        hipLaunchKernelGGL(kernel, grid, dim3(kB), 0, s, __VA_ARGS__);                    \
        const hipError_t e_ = hipGetLastError();                                          \
        if (e_ != hipSuccess) return e_;                                                  \
    } while (0)

// Cell lists for cells of side >= rc, and the particles in cell order (in the
// context's FP64 scratch); with surf those within sigma / 2 of R only.  Follows
// launch_absmax.
hipError_t ag_cells(ld_ctx* c, const AgBufs& b, const AgTable& tb, double rc, bool surf, double R,
                    int* labels, bool roots, AgSorted* A) {
    const int n = (int)c->n;
    hipStream_t s = c->stream;
    const dim3 gn((n + kB - 1) / kB);
    const cells::Work C = cells::work_at(b.work);
    int* cell = reinterpret_cast<int*>(c->sb.keys);       // cells and ranks
    int* list = reinterpret_cast<int*>(c->sb.tmp4);       // lists and sorted cells
    float4* hi = reinterpret_cast<float4*>(c->work);
    float4* lo = hi + n;
    hipError_t e;
    if (surf)
        AG_RUN(k_ag_bin<true>, gn, c->pos, c->lo, c->typ, c->oid, n, c->sb.bounds_part, rc, R, tb,
               C, cell, cell + n, labels, b.res);
    else
        AG_RUN(k_ag_bin<false>, gn, c->pos, c->lo, c->typ, c->oid, n, c->sb.bounds_part, rc, R,
               tb, C, cell, cell + n, labels, b.res);
    if ((e = cells::launch_coarse(C, s)) != hipSuccess) return e;
    if ((e = cells::launch_scan(C, 0, 1, rc, c->st, 0.0, s)) != hipSuccess) return e;
    if ((e = cells::launch_list(cell, cell + n, n, C, list, s)) != hipSuccess) return e;
    AG_RUN(k_ag_place, gn, c->pos, c->lo, c->typ, cell, list, C, rc, n, hi, lo, b.slot, list + n,
           roots ? b.parent : nullptr, b.minoid, b.size, b.count);
    *A = AgSorted{hi, lo, b.slot, list + n, C.first, b.count, C.mx};
    return hipSuccess;
}

// Below this size more lanes a particle: a chip that one lane a particle
// leaves idle waits for their chains (the truncated scheme's walk breaks even
// between 50 000 and 100 000).
constexpr int kAgSplitN = 75000;

// Cell lists, lock-free union of the contact pairs (with surf: of surface NPs
// only), roots, per root the size and smallest original index, labels and
// statistics.
hipError_t ag_union(ld_ctx* c, const AgBufs& b, const AgTable& tb, double rc, bool surf, double R,
                    int* labels, AgSorted* A) {
    const int n = (int)c->n;
    hipStream_t s = c->stream;
    const dim3 gn((n + kB - 1) / kB), gl(std::min((n + kB - 1) / kB, 128));
    int* err = reinterpret_cast<int*>(b.res + 3);
    hipError_t e = cells::launch_absmax(c->pos, n, c->sb.bounds_part, cells::work_at(b.work), s);
    if (e == hipSuccess) e = ag_cells(c, b, tb, rc, surf, R, labels, true, A);
    if (e != hipSuccess) return e;
    if (n < kAgSplitN)
        AG_RUN(k_ag_hook<16>, dim3((n + kB / 16 - 1) / (kB / 16)), *A, tb, rc, b.parent, err);
    else
        AG_RUN(k_ag_hook<4>, dim3((n + kB / 4 - 1) / (kB / 4)), *A, tb, rc, b.parent, err);
    AG_RUN(k_ag_roots, gn, b.parent, b.slot, c->oid, b.count, b.root, b.minoid, b.size, err);
    if (surf)
        AG_RUN(k_ag_label<true>, gl, b.root, b.slot, c->oid, b.minoid, b.size, b.count, labels,
               b.res);
    else
        AG_RUN(k_ag_label<false>, gl, b.root, b.slot, c->oid, b.minoid, b.size, b.count, labels,
               b.res);
    return hipSuccess;
}
#undef AG_RUN

// The statistics and, unless null, the labels.
hipError_t ag_read(ld_ctx* c, void* res, const void* dres, size_t bytes, int32_t* labels,
                   const int* dlabels) {
    return copy_out(c->stage,
                    {{res, dres, bytes}, {labels, dlabels, sizeof(int32_t) * (size_t)c->n}},
                    c->stream);
}

}  // namespace

void ag_free(ld_ctx* c) {
    if (c->agg) (void)hipFree(c->agg);
    c->agg = nullptr;
}

// Eq. (6) pair counts into counts[n_bins] (device) through the cell sort,
// when the grid of cells of side >= r_max has at least 3 cells per axis;
// *used = false leaves the counts to the all-pairs histogram.  The slot
// order is not changed.
ld_status ag_rdf_pairs(ld_ctx* c, double r_max, int n_bins, unsigned long long* counts,
                       bool* used) {
    *used = false;
    const int n = (int)c->n;
    hipStream_t s = c->stream;
    // the grid the binning will derive (same partial maxima, same rule)
    AgBufs b{};
    ld_status st = ag_buffers(c, &b);
    if (st != LD_OK) return st;
    const cells::Work C = cells::work_at(b.work);
    HIP_TRY(cells::launch_absmax(c->pos, n, c->sb.bounds_part, C, s));
    float part[64];
    HIP_TRY(copy_out(c->stage, part, c->sb.bounds_part, sizeof part, s));
    float m = 0.f;
    for (float v : part) m = std::max(m, v);
    m = std::max(m, 1e-3f);
    const double L = (double)(m * 1.0009765625f);
    if ((int)std::floor(2.0 * L / r_max) < 3) return LD_OK;
    AgTable tb{};
    AgSorted A{};
    HIP_TRY(ag_cells(c, b, tb, r_max, false, 0.0, nullptr, false, &A));
    AG_LAUNCH(k_ag_zero64, dim3((n_bins + kB - 1) / kB), dim3(kB), s, counts, n_bins);
    if (n < kAgSplitN)
        AG_LAUNCH(k_ag_rdf<4>, dim3((n + kB / 4 - 1) / (kB / 4)), dim3(kB), s, A, r_max, n_bins,
                  r_max / n_bins, counts);
    else
        AG_LAUNCH(k_ag_rdf<1>, dim3((n + kB - 1) / kB), dim3(kB), s, A, r_max, n_bins,
                  r_max / n_bins, counts);
    *used = true;
    return LD_OK;
}

}  // namespace ld

using namespace ld;
using namespace ld::host;

extern "C" {

ld_status ld_aggregates(ld_ctx* c, double contact_factor, int64_t stats[3], int32_t* labels) {
    g_err.clear();
    if (!c || !stats) return fail(LD_EINVAL, "ctx and stats are required");
    if (!(contact_factor > 0.0) || !std::isfinite(contact_factor))
        return fail(LD_EINVAL, "contact_factor must be positive");
    const int n = (int)c->n;
    hipStream_t s = c->stream;
    AgBufs b{};
    ld_status st = ag_buffers(c, &b);
    if (st != LD_OK) return st;
    AgTable tb{};
    const double rc = ag_table(c, contact_factor, &tb);
    AgSorted A{};
    HIP_TRY(ag_union(c, b, tb, rc, false, 0.0, labels ? b.labels : nullptr, &A));
    AgRes res[4];
    HIP_TRY(ag_read(c, res, b.res, sizeof res, labels, b.labels));
    if (res[3]) return fail(LD_EHIP, "contact-graph union did not settle within its bound");
    for (int k = 0; k < 3; ++k) stats[k] = (int64_t)res[k];
    return LD_OK;
}

ld_status ld_surface_fractal(ld_ctx* c, double R, double contact_factor, double k_f, double d,
                             int64_t stats[3], double out[3], int32_t* labels) {
    g_err.clear();
    if (!c || !stats || !out) return fail(LD_EINVAL, "ctx, stats and out are required");
    if (!(contact_factor > 0.0) || !std::isfinite(contact_factor))
        return fail(LD_EINVAL, "contact_factor must be positive");
    if (!(k_f > 0.0) || !std::isfinite(k_f)) return fail(LD_EINVAL, "k_f must be positive");
    if (std::isnan(d)) return fail(LD_EINVAL, "d is NaN");
    const int n = (int)c->n;
    hipStream_t s = c->stream;
    if (!(R >= 0.0)) {      // negative: the droplet's radius at the current time
        DevState ds;
        HIP_TRY(copy_out(c->stage, &ds, c->st, sizeof ds, s));
        R = radius_at(c->R, ds.t);
    }
    AgBufs b{};
    ld_status st = ag_buffers(c, &b);
    if (st != LD_OK) return st;
    AgTable tb{};
    const double rc = ag_table(c, contact_factor, &tb);
    const int blocks = (n + kB - 1) / kB;
    AgSorted A{};
    HIP_TRY(ag_union(c, b, tb, rc, true, R, labels ? b.labels : nullptr, &A));
    // the largest component's mean direction, mean diameter and squared angles
    // (partials summed in workgroup order: nothing depends on timing)
    double* tpart = b.dpart + 4 * (size_t)blocks;
    AG_LAUNCH(k_sf_sums, dim3(blocks), dim3(kB), s, A, b.root, b.minoid, b.res, tb, b.dpart);
    AG_LAUNCH(k_sf_theta, dim3(blocks), dim3(kB), s, A, b.root, b.minoid, b.res, b.dpart, tpart);
    std::vector<double> got(kResDoubles + 5 * (size_t)blocks);
    HIP_TRY(ag_read(c, got.data(), b.res, sizeof(double) * got.size(), labels, b.labels));
    AgRes res[4];
    std::memcpy(res, got.data(), sizeof res);
    const double* dp = got.data() + kResDoubles;
    if (res[3]) return fail(LD_EHIP, "contact-graph union did not settle within its bound");
    const double nan = std::numeric_limits<double>::quiet_NaN();
    out[0] = out[1] = out[2] = nan;
    stats[0] = (int64_t)res[0];
    if (res[0] == 0) {
        stats[1] = 0;
        stats[2] = -1;
        return LD_OK;
    }
    const long long m = (long long)(res[2] >> 32);
    stats[1] = m;
    stats[2] = INT_MAX - (int)(unsigned)(res[2] & 0xffffffffull);
    double su[3] = {0.0, 0.0, 0.0}, ssig = 0.0, s2 = 0.0;
    for (int k = 0; k < blocks; ++k) {
        su[0] += dp[4 * (size_t)k];
        su[1] += dp[4 * (size_t)k + 1];
        su[2] += dp[4 * (size_t)k + 2];
        ssig += dp[4 * (size_t)k + 3];
        s2 += dp[4 * (size_t)blocks + (size_t)k];
    }
    const double nu = std::sqrt(su[0] * su[0] + su[1] * su[1] + su[2] * su[2]);
    if (!(nu > 0.0)) return LD_OK;
    const double dm = d > 0.0 ? d : ssig / (double)m;
    const double Rg = R * std::sqrt(s2 / (double)m);
    out[0] = Rg;
    out[1] = dm;
    if (m >= 2) out[2] = std::log((double)m / k_f) / std::log(2.0 * Rg / dm);
    return LD_OK;
}

ld_status ld_surface_count(ld_ctx* c, double R, int64_t* counts) {
    g_err.clear();
    if (!c || !counts) return fail(LD_EINVAL, "ctx and counts are required");
    const int n = (int)c->n;
    hipStream_t s = c->stream;
    if (!(R >= 0.0)) {      // negative: the droplet's radius at the current time
        DevState ds;
        HIP_TRY(copy_out(c->stage, &ds, c->st, sizeof ds, s));
        R = radius_at(c->R, ds.t);
    }
    AgBufs b{};
    ld_status st = ag_buffers(c, &b);
    if (st != LD_OK) return st;
    AgTable tb{};
    tb.T = c->p.n_types;
    for (int a = 0; a < tb.T; ++a) tb.half_sigma[a] = 0.5 * c->p.sigma[a];
    const int blocks = (n + kB - 1) / kB;
    AG_LAUNCH(k_ag_surface, dim3(blocks), dim3(kB), s, c->pos, c->lo, c->typ, n, R, tb, b.part);
    std::vector<long long> part((size_t)blocks * kMaxTypes);
    HIP_TRY(copy_out(c->stage, part.data(), b.part, sizeof(long long) * part.size(), s));
    for (int t = 0; t < tb.T; ++t) {
        long long v = 0;
        for (int k = 0; k < blocks; ++k) v += part[(size_t)k * kMaxTypes + t];
        counts[t] = v;
    }
    return LD_OK;
}

}  // extern "C"
