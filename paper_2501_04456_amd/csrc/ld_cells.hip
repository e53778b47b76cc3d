// The launches of the counted cell lists.
#include "ld_cells.h"

namespace ld {
namespace cells {

namespace {

constexpr int kB = 256;

__global__ __launch_bounds__(kB) void k_cells_absmax(const float4* __restrict__ pos, int n,
                                                     float* part, Work C) {
    __shared__ float red[kB];
    for (int k = blockIdx.x * kB + threadIdx.x; k < kNC / 4; k += 64 * kB)
        reinterpret_cast<int4*>(C.count)[k] = make_int4(0, 0, 0, 0);
    float m = 0.f;
    for (int s = blockIdx.x * kB + threadIdx.x; s < n; s += 64 * kB) {
        const float4 h = pos[s];
        m = fmaxf(m, fmaxf(fabsf(h.x), fmaxf(fabsf(h.y), fabsf(h.z))));
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = kB / 2; w >= 1; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(kB) void k_cells_coarse(Work C) {
    __shared__ int wsum[kB / 64];
    const int4 v = reinterpret_cast<const int4*>(C.count)[blockIdx.x * kB + threadIdx.x];
    int x = v.x + v.y + v.z + v.w;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) x += __shfl_xor(x, o);
    if (threadIdx.x % 64 == 0) wsum[threadIdx.x / 64] = x;
    __syncthreads();
    if (threadIdx.x == 0) C.coarse[blockIdx.x] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
}

// A workgroup adds the coarse counts before its kCoarse cells, scans those,
// and leaves their counts zero.
__global__ __launch_bounds__(kB) void k_cells_scan(Work C, int grid_mx, int next_mx, double r,
                                                   DevState* st, double adv_dt) {
    static_assert(kCoarse == 4 * kB && kNC / kCoarse == kB, "one int4 and one count per thread");
    __shared__ int wsum[2][4];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        if (adv_dt > 0.0) {
            st->t = st->t + adv_dt;
            st->step = st->step + 1;
        }
        C.mx[next_mx] = 0u;
    }
    const int G = grid_of(__uint_as_float(C.mx[grid_mx]), r).Gc, M = G * G * G;
    const int b = blockIdx.x, t = threadIdx.x, w = t / 64, lane = t % 64;
    if (b * kCoarse >= M) return;
    const int4 v = reinterpret_cast<const int4*>(C.count)[b * kB + t];
    int before = t < b ? C.coarse[t] : 0;
    const int sum = v.x + v.y + v.z + v.w;
    int x = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        before += __shfl_xor(before, o);
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == 63) {
        wsum[0][w] = before;
        wsum[1][w] = x;
    }
    __syncthreads();
    int at = wsum[0][0] + wsum[0][1] + wsum[0][2] + wsum[0][3] + x - sum;
    for (int k = 0; k < w; ++k) at += wsum[1][k];
    const int c = b * kCoarse + 4 * t;               // kNC is a multiple of 4
    C.first[c] = at;
    C.first[c + 1] = at + v.x;
    C.first[c + 2] = at + v.x + v.y;
    C.first[c + 3] = at + v.x + v.y + v.z;
    if (M - 1 >= c && M - 1 < c + 4) C.first[M] = at + sum;   // cells from M on are empty
    reinterpret_cast<int4*>(C.count)[b * kB + t] = make_int4(0, 0, 0, 0);
}

__global__ __launch_bounds__(kB) void k_cells_list(const int* __restrict__ cell,
                                                   const int* __restrict__ rank, int n, Work C,
                                                   int* list) {
    const int s = blockIdx.x * kB + threadIdx.x;
    if (blockIdx.x == 0) C.coarse[threadIdx.x] = 0;
    if (s >= n) return;
    const int c = cell[s];
    if (c >= 0) list[C.first[c] + rank[s]] = s;
}

}  // namespace

hipError_t launch_absmax(const float4* pos, int n, float* part, const Work& C, hipStream_t s) {
    hipLaunchKernelGGL(k_cells_absmax, dim3(64), dim3(kB), 0, s, pos, n, part, C);
    return hipGetLastError();
}

hipError_t launch_coarse(const Work& C, hipStream_t s) {
    hipLaunchKernelGGL(k_cells_coarse, dim3(kNC / kCoarse), dim3(kB), 0, s, C);
    return hipGetLastError();
}

hipError_t launch_scan(const Work& C, int grid_mx, int next_mx, double r, DevState* st,
                       double adv_dt, hipStream_t s) {
    hipLaunchKernelGGL(k_cells_scan, dim3(kNC / kCoarse), dim3(kB), 0, s, C, grid_mx, next_mx, r,
                       st, adv_dt);
    return hipGetLastError();
}

hipError_t launch_list(const int* cell, const int* rank, int n, const Work& C, int* list,
                       hipStream_t s) {
    hipLaunchKernelGGL(k_cells_list, dim3((n + kB - 1) / kB), dim3(kB), 0, s, cell, rank, n, C,
                       list);
    return hipGetLastError();
}

}  // namespace cells
}  // namespace ld
