// Post-processing on the device (section 3): the pair-distance histogram
// behind the RDF, Eq. (6), the centre-distance histogram behind the radial
// concentration, Eq. (8), moments for the radius of gyration, Eqs. (3)-(4),
// and occupied-box counts for the box-counting dimension.
//
// Distances use the full FP64 positions hi + lo.  Contraction into fma is
// switched off here so each distance rounds exactly as written, which makes
// the integer bin of every pair reproducible.
#include "ld_internal.h"

namespace ld {
namespace {

constexpr int kRdfBlock = 256;
constexpr int kMaxBins = 4096;

__device__ __forceinline__ void full_pos(const float4* pos, const float4* lo, int s,
                                         double x[3]) {
    const float4 h = pos[s], l = lo[s];
    x[0] = (double)h.x + (double)l.x;
    x[1] = (double)h.y + (double)l.y;
    x[2] = (double)h.z + (double)l.z;
}

__global__ __launch_bounds__(kRdfBlock) void k_rdf(const float4* __restrict__ pos,
                                                   const float4* __restrict__ lo, int n,
                                                   double r_max, int n_bins, double dr,
                                                   unsigned long long* counts) {
#pragma clang fp contract(off)
    __shared__ unsigned int hist[kMaxBins];
    __shared__ double sx[kRdfBlock], sy[kRdfBlock], sz[kRdfBlock];
    for (int b = threadIdx.x; b < n_bins; b += kRdfBlock) hist[b] = 0u;
    const int i = blockIdx.x * kRdfBlock + threadIdx.x;
    double xi[3] = {0.0, 0.0, 0.0};
    if (i < n) full_pos(pos, lo, i, xi);
    for (int jt = blockIdx.x * kRdfBlock; jt < n; jt += kRdfBlock) {
        __syncthreads();
        const int j = jt + threadIdx.x;
        if (j < n) {
            double xj[3];
            full_pos(pos, lo, j, xj);
            sx[threadIdx.x] = xj[0];
            sy[threadIdx.x] = xj[1];
            sz[threadIdx.x] = xj[2];
        }
        __syncthreads();
        if (i < n) {
            const int m = min(kRdfBlock, n - jt);
            for (int k = 0; k < m; ++k) {
                if (jt + k <= i) continue;
                const double dx = xi[0] - sx[k];
                const double dy = xi[1] - sy[k];
                const double dz = xi[2] - sz[k];
                const double r = sqrt(dx * dx + dy * dy + dz * dz);
                if (r < r_max) {
                    const int b = (int)floor(r / dr);
                    if (b >= 0 && b < n_bins) atomicAdd(&hist[b], 1u);
                }
            }
        }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < n_bins; b += kRdfBlock)
        if (hist[b]) atomicAdd(&counts[b], (unsigned long long)hist[b]);
}

// Distances from the centre into bins; typ != null keeps type `want` only.
__global__ __launch_bounds__(256) void k_centre_hist(const float4* __restrict__ pos,
                                                     const float4* __restrict__ lo, int n,
                                                     double r_max, int n_bins, double dr,
                                                     const double* __restrict__ centre,
                                                     unsigned long long* counts,
                                                     const int* __restrict__ typ, int want) {
#pragma clang fp contract(off)
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    if (typ && typ[s] != want) return;
    double x[3];
    full_pos(pos, lo, s, x);
    const double dx = x[0] - centre[0], dy = x[1] - centre[1], dz = x[2] - centre[2];
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    if (r < r_max) {
        const int b = (int)floor(r / dr);
        if (b >= 0 && b < n_bins) atomicAdd(&counts[b], 1ull);
    }
}

__global__ __launch_bounds__(256) void k_zero_u64(unsigned long long* p, int m) {
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < m) p[k] = 0ull;
}

// rows: 0..2 positions, 3..5 filled later by k_dev2
__global__ __launch_bounds__(256) void k_pos_rows(const float4* __restrict__ pos,
                                                  const float4* __restrict__ lo, int n,
                                                  double* work) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    double x[3];
    full_pos(pos, lo, s, x);
    work[s] = x[0];
    work[(size_t)n + s] = x[1];
    work[2 * (size_t)n + s] = x[2];
}

__global__ __launch_bounds__(256) void k_dev2(const float4* __restrict__ pos,
                                              const float4* __restrict__ lo, int n,
                                              const double* __restrict__ sums, double* work) {
#pragma clang fp contract(off)
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s >= n) return;
    double x[3];
    full_pos(pos, lo, s, x);
    const double c0 = sums[0] / n, c1 = sums[1] / n, c2 = sums[2] / n;
    const double dx = c0 - x[0], dy = c1 - x[1], dz = c2 - x[2];
    work[s] = dx * dx + dy * dy + dz * dz;
}

__global__ void k_moments_finish(const double* sums, const double* s2, int n, double* out4) {
    out4[0] = sums[0] / n;
    out4[1] = sums[1] / n;
    out4[2] = sums[2] / n;
    out4[3] = sqrt(s2[0] / n);
}

// Sums, extents and type counts of the positions, kFracParts partials of
// kFracWords doubles: sum[3], smallest[3], largest[3], count[kMaxTypes].
__global__ __launch_bounds__(256) void k_frac_stats(const float4* __restrict__ pos,
                                                    const float4* __restrict__ lo,
                                                    const int* __restrict__ typ, int n,
                                                    double* part) {
    __shared__ double red[kFracWords][4];
    const int t = threadIdx.x, lane = t % 64;
    double v[kFracWords];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v[c] = 0.0;
        v[3 + c] = INFINITY;
        v[6 + c] = -INFINITY;
    }
#pragma unroll
    for (int q = 0; q < kMaxTypes; ++q) v[9 + q] = 0.0;
    for (int s = blockIdx.x * 256 + t; s < n; s += kFracParts * 256) {
        double x[3];
        full_pos(pos, lo, s, x);
        const int ty = typ[s];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[c] += x[c];
            v[3 + c] = fmin(v[3 + c], x[c]);
            v[6 + c] = fmax(v[6 + c], x[c]);
        }
#pragma unroll
        for (int q = 0; q < kMaxTypes; ++q) v[9 + q] += ty == q ? 1.0 : 0.0;
    }
#pragma unroll
    for (int k = 0; k < kFracWords; ++k) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const double y = __shfl_xor(v[k], o);
            v[k] = k < 3 || k >= 9 ? v[k] + y : (k < 6 ? fmin(v[k], y) : fmax(v[k], y));
        }
        if (lane == 0) red[k][t / 64] = v[k];
    }
    __syncthreads();
    if (t < kFracWords) {
        double y = red[t][0];
        for (int w = 1; w < 4; ++w)
            y = t < 3 || t >= 9 ? y + red[t][w]
                                : (t < 6 ? fmin(y, red[t][w]) : fmax(y, red[t][w]));
        part[blockIdx.x * kFracWords + t] = y;
    }
}

// Squared distances from the centre of mass (every workgroup adds the partial
// sums itself, in one order), kFracParts partials; empties the first table.
__global__ __launch_bounds__(256) void k_frac_dev2(const float4* __restrict__ pos,
                                                   const float4* __restrict__ lo, int n,
                                                   const double* __restrict__ part, double* dev2,
                                                   unsigned long long* table, size_t entries) {
#pragma clang fp contract(off)
    static_assert(kFracParts == 256, "one partial per thread");
    __shared__ double red[3][256];
    const int t = threadIdx.x;
    for (int c = 0; c < 3; ++c) red[c][t] = part[t * kFracWords + c];
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w)
            for (int c = 0; c < 3; ++c) red[c][t] += red[c][t + w];
        __syncthreads();
    }
    const double c0 = red[0][0] / n, c1 = red[1][0] / n, c2 = red[2][0] / n;
    __syncthreads();
    double v = 0.0;
    for (int s = blockIdx.x * 256 + t; s < n; s += kFracParts * 256) {
        double x[3];
        full_pos(pos, lo, s, x);
        const double dx = c0 - x[0], dy = c1 - x[1], dz = c2 - x[2];
        v += dx * dx + dy * dy + dz * dz;
    }
    for (size_t k = (size_t)blockIdx.x * 256 + t; k < entries; k += kFracParts * 256)
        table[k] = ~0ull;
    red[0][t] = v;
    __syncthreads();
    for (int w = 128; w >= 1; w >>= 1) {
        if (t < w) red[0][t] += red[0][t + w];
        __syncthreads();
    }
    if (t == 0) dev2[blockIdx.x] = red[0][0];
}

// Boxes of side eps that hold a particle: each particle looks its box up in a
// hash table of at least twice n entries (linear probing), and whoever enters
// it is the box's only representative.  Boxes of twice the side hold whole
// boxes of this one (the same FP64 quotient, halved exactly), so only the
// representatives, one flag a slot, look on at the next scale.  Empties the
// table of the next scale.  Bound by one random table access a particle at
// the finest scales: the eight scales of 250 000 NPs 640 us with a sort of box
// keys for each, 160 so.
__global__ __launch_bounds__(256) void k_box_count(const float4* __restrict__ pos,
                                                   const float4* __restrict__ lo, int n, int first,
                                                   double lo0, double lo1, double lo2, double eps,
                                                   unsigned long long ny, unsigned long long nz,
                                                   unsigned long long* table,
                                                   unsigned long long* next, size_t entries,
                                                   unsigned char* rep, int* count) {
    __shared__ int red[4];
    int c = 0;
    const size_t mask = entries - 1;
    for (int s = blockIdx.x * 256 + threadIdx.x; s < n; s += gridDim.x * 256) {
        if (!first && !rep[s]) continue;
        double x[3];
        full_pos(pos, lo, s, x);
        const unsigned long long ix = (unsigned long long)floor((x[0] - lo0) / eps);
        const unsigned long long iy = (unsigned long long)floor((x[1] - lo1) / eps);
        const unsigned long long iz = (unsigned long long)floor((x[2] - lo2) / eps);
        const unsigned long long key = ny ? (ix * ny + iy) * nz + iz : (ix << 42) | (iy << 21) | iz;
        unsigned long long h = key * 0x9E3779B97F4A7C15ull;
        h ^= h >> 32;
        bool mine = false;
        for (size_t probe = 0; probe < entries; ++probe) {
            unsigned long long* e = table + ((h + probe) & mask);
            // (a look first where many may share a box; representatives of half
            // the side are at most eight to a box)
            unsigned long long old = ~0ull;
            if (first) old = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (old == ~0ull) old = atomicCAS(e, ~0ull, key);
            if (old == ~0ull || old == key) {
                mine = old == ~0ull;
                break;
            }
        }
        rep[s] = mine ? 1 : 0;
        c += mine ? 1 : 0;
    }
    for (size_t k = (size_t)blockIdx.x * 256 + threadIdx.x; k < entries; k += gridDim.x * 256)
        next[k] = ~0ull;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) c += __shfl_xor(c, o);
    if (threadIdx.x % 64 == 0) red[threadIdx.x / 64] = c;
    __syncthreads();
    if (threadIdx.x == 0) count[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ __launch_bounds__(256) void k_set_charge(float4* pos, const int* __restrict__ oid,
                                                   const float* __restrict__ qhat, int n) {
    const int s = blockIdx.x * 256 + threadIdx.x;
    if (s < n) pos[s].w = qhat[oid[s]];
}

}  // namespace

hipError_t launch_rdf(const float4* pos, const float4* lo, int n, double r_max, int n_bins,
                      const double* centre, unsigned long long* counts,
                      unsigned long long* ccounts, hipStream_t s) {
    if (n_bins < 1 || n_bins > kMaxBins) return hipErrorInvalidValue;
    const double dr = r_max / n_bins;
    hipLaunchKernelGGL(k_zero_u64, dim3((n_bins + 255) / 256), dim3(256), 0, s, counts, n_bins);
    hipLaunchKernelGGL(k_zero_u64, dim3((n_bins + 255) / 256), dim3(256), 0, s, ccounts, n_bins);
    hipLaunchKernelGGL(k_rdf, dim3((n + kRdfBlock - 1) / kRdfBlock), dim3(kRdfBlock), 0, s, pos,
                       lo, n, r_max, n_bins, dr, counts);
    hipLaunchKernelGGL(k_centre_hist, dim3((n + 255) / 256), dim3(256), 0, s, pos, lo, n, r_max,
                       n_bins, dr, centre, ccounts, nullptr, 0);
    return hipGetLastError();
}

hipError_t launch_centre_hist(const float4* pos, const float4* lo, const int* typ, int want, int n,
                              double r_max, int n_bins, const double* centre,
                              unsigned long long* ccounts, hipStream_t s) {
    if (n_bins < 1 || n_bins > kMaxBins) return hipErrorInvalidValue;
    const double dr = r_max / n_bins;
    hipLaunchKernelGGL(k_zero_u64, dim3((n_bins + 255) / 256), dim3(256), 0, s, ccounts, n_bins);
    hipLaunchKernelGGL(k_centre_hist, dim3((n + 255) / 256), dim3(256), 0, s, pos, lo, n, r_max,
                       n_bins, dr, centre, ccounts, typ, want);
    return hipGetLastError();
}

hipError_t launch_set_charge(float4* pos, const int* oid, const float* qhat, int n,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_set_charge, dim3((n + 255) / 256), dim3(256), 0, s, pos, oid, qhat, n);
    return hipGetLastError();
}

hipError_t launch_moments(const float4* pos, const float4* lo, int n, double* work,
                          double* out4, hipStream_t s) {
    const dim3 g((n + 255) / 256);
    double* sums = work + 3 * (size_t)n;
    double* s2 = sums + 4;
    hipLaunchKernelGGL(k_pos_rows, g, dim3(256), 0, s, pos, lo, n, work);
    hipError_t e = launch_rowsum(work, 3, n, sums, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_dev2, g, dim3(256), 0, s, pos, lo, n, sums, work);
    e = launch_rowsum(work, 1, n, s2, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_moments_finish, dim3(1), dim3(1), 0, s, sums, s2, n, out4);
    return hipGetLastError();
}

hipError_t launch_zero(unsigned long long* p, int m, hipStream_t s) {
    hipLaunchKernelGGL(k_zero_u64, dim3((m + 255) / 256), dim3(256), 0, s, p, m);
    return hipGetLastError();
}

hipError_t launch_frac_stats(const float4* pos, const float4* lo, const int* typ, int n,
                             double* part, unsigned long long* table, size_t entries,
                             hipStream_t s) {
    hipLaunchKernelGGL(k_frac_stats, dim3(kFracParts), dim3(256), 0, s, pos, lo, typ, n, part);
    hipLaunchKernelGGL(k_frac_dev2, dim3(kFracParts), dim3(256), 0, s, pos, lo, n, part,
                       part + kFracParts * kFracWords, table, entries);
    return hipGetLastError();
}

hipError_t launch_box_count(const float4* pos, const float4* lo, int n, bool first,
                            const double lo3[3], double eps, unsigned long long ny,
                            unsigned long long nz, unsigned long long* table,
                            unsigned long long* next, size_t entries, unsigned char* rep,
                            int* count, int parts, hipStream_t s) {
    hipLaunchKernelGGL(k_box_count, dim3(parts), dim3(256), 0, s, pos, lo, n, first ? 1 : 0,
                       lo3[0], lo3[1], lo3[2], eps, ny, nz, table, next, entries, rep, count);
    return hipGetLastError();
}

}  // namespace ld
