// The paper's own scheme, section 2.2 steps (i)-(vi) read literally with the
// forces of section 2.1:
//
//   (i)   slots sorted by cells of side >= the largest pair range;
//   (ii)  pair forces of the pairs closer than range_factor (r_i + r_j),
//         r = sigma / 2, LJ and Coulomb both truncated there without shift,
//         summed over the 27 cells around each particle;
//   (iii) R(t + dt);
//   (iv)-(v) surface spring (band-limited with ld_params.wall_band), gravity,
//         centrifugal force;
//   (vi)  Newton's equation with Stokes drag and the random velocity vector:
//         v <- v + dt (F_pair + F_ext - gamma v) / m,  v <- v + kick u,
//         x <- x + dt v,
//         u the normalised Box-Muller triple of the context's noise stream
//         (uniform on the unit sphere).
//
// Pairs in range are few per particle (tens while dispersed, hundreds once
// aggregated), so the pair math is FP64 throughout: the range test agrees
// with FP64 positions and the forces need no compensation.  Velocities are
// FP64, positions stay (hi, lo) FP32 pairs.
#include <algorithm>
#include <cmath>
#include <new>

#include "ld_cells.h"
#include "ld_host.h"
#include "ld_update_core.h"

namespace ld {

using host::fail;

// Pair constants: range^2, sigma^2 and 24 eps per type pair (FP64).
struct PmTable {
    int T;
    double rint2[kMaxTypes * kMaxTypes];
    double sig2[kMaxTypes * kMaxTypes];
    double e24[kMaxTypes * kMaxTypes];
    double inv_m[kMaxTypes];            // 1 / inertial mass
    double gamma[kMaxTypes];
    double rtype[kMaxTypes];            // largest pair range of a type
    double rmax;                        // largest pair range
    double kick;
};

struct PaperMode {
    ld_paper_config cfg{};
    PmTable tab{};
    double* v = nullptr;                // [3][n] velocities, slot order
    double* v2 = nullptr;               // [3][n] second buffer (re-sort)
    double* F = nullptr;                // [3][n] pair forces, slot order
    // Steps since the largest coordinate was taken on its own.  The cells of a
    // step are those of the largest coordinate before the step before it, also
    // across calls (known: the workspace holds it and the present one), so a
    // trajectory does not depend on how its steps are split into calls.
    unsigned turn = 0;
    bool known = false;
    int* cells = nullptr;               // counts, coarse counts, first slots, largest coordinates
};

namespace {

constexpr int kB = 256;
constexpr int kPmSplitN = 60000;        // particles from which a lane takes one by itself

// Cells of all slots at positions no step of the same call has left (the
// steps bin what they move themselves), on the grid of mx[grid_mx]; with
// grid_mx < 0 of the largest coordinate, which becomes mx[0] = mx[1].
__global__ __launch_bounds__(kB) void k_pm_bin(const float4* __restrict__ pos,
                                               const float4* __restrict__ lo, int n,
                                               const float* __restrict__ part, int grid_mx,
                                               double rmax, cells::Work C, int* cell, int* rank) {
    const float m = grid_mx < 0 ? cells::absmax_of(part) : __uint_as_float(C.mx[grid_mx]);
    if (grid_mx < 0 && blockIdx.x == 0 && threadIdx.x == 0)
        C.mx[0] = C.mx[1] = __float_as_uint(m);
    const int s = blockIdx.x * kB + threadIdx.x;
    double x[3] = {0.0, 0.0, 0.0};
    if (s < n) {
        const float4 h = pos[s], l = lo[s];
        x[0] = (double)h.x + (double)l.x;
        x[1] = (double)h.y + (double)l.y;
        x[2] = (double)h.z + (double)l.z;
    }
    cells::bin<false>(cells::grid_of(m, rmax), s < n, s, x, C, cell, rank);
}

// The sort itself.
struct PmPlace {
    const float4 *pos, *lo;
    const int *typ, *oid, *cell, *list, *first;
    const double* v;
    float4 *pos2, *lo2;
    int *typ2, *oid2, *cell2;
    double* v2;
    int n;
};
__global__ __launch_bounds__(kB) void k_pm_place(PmPlace A) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (k >= A.n) return;
    const int s = A.list[k], c = A.cell[s];
    const size_t n = (size_t)A.n;
    const float4 h = A.pos[s], l = A.lo[s];
    const int ty = A.typ[s], id = A.oid[s];
    const double v0 = A.v[s], v1 = A.v[n + s], v2 = A.v[2 * n + s];
    const int d = cells::place(A.first, A.list, c, s);
    A.pos2[d] = h;
    A.lo2[d] = l;
    A.typ2[d] = ty;
    A.oid2[d] = id;
    A.cell2[d] = c;
    A.v2[d] = v0;
    A.v2[n + d] = v1;
    A.v2[2 * n + d] = v2;
}

// Steps (ii)-(vi) of consecutive slots in cell order.
//
// Pairs: LANES lanes share a particle and walk the cells around it; what
// passes the screen (about 5 of 70 candidates at the headline's density) is
// evaluated in FP64.
//
// A step of 250 000: 138 us (a sort of 24-bit keys in three passes, forces a
// lane per particle and an update, 15 launches) -> 65 us in four launches; of
// 5000: 110 -> 23 us.
//
// With STEP the slots are then moved into the second buffers (other
// workgroups still read the first), and with bin counted into the next
// step's cells; without, the forces are stored.
struct PmStep {
    const float4 *pos, *lo;
    const int *typ, *oid, *cell, *first;
    const double* v;
    int n, grid_mx, cur_mx, next_mx;
    double* F;
    float4 *pos2, *lo2;
    double* v2;
    DevState* st;
    double dt;
    unsigned long long seed;
    int bin;
    int *ncell, *nrank;
};

template <int LANES>
constexpr int kPmBlock = LANES == 1 ? 256 : 64 * LANES;   // threads; 64 slots where lanes share

template <bool STEP, int LANES>
__global__ __launch_bounds__(kPmBlock<LANES>) void k_pm_step(PmStep A, PmTable tb, ExtParams P,
                                                             cells::Work C) {
    constexpr int kBlock = kPmBlock<LANES>, kPart = kBlock / LANES;
    constexpr int kList = 16;
    __shared__ double tr[kMaxTypes * kMaxTypes], ts[kMaxTypes * kMaxTypes],
        te[kMaxTypes * kMaxTypes], sF[3][LANES == 1 ? 1 : kPart];
    __shared__ int list[kList][kBlock];
    const int t = threadIdx.x, sub = t % LANES;
    const int i = blockIdx.x * kPart + t / LANES;
    const bool live = i < A.n;
    if (t < tb.T * tb.T) {
        tr[t] = tb.rint2[t];
        ts[t] = tb.sig2[t];
        te[t] = tb.e24[t];
    }
    const float mcur = __uint_as_float(C.mx[A.cur_mx]);
    const int G = cells::grid_of(__uint_as_float(C.mx[A.grid_mx]), tb.rmax).Gc;
    float4 hi = make_float4(0.f, 0.f, 0.f, 0.f), li = hi;
    int ty = 0, c = 0;
    float screen = 0.f;
    if (live) {
        hi = A.pos[i];
        li = A.lo[i];
        ty = A.typ[i];
        c = A.cell[i];
        screen = cells::screen2(tb.rtype[ty], mcur);
    }
    const double xi = (double)hi.x + (double)li.x, yi = (double)hi.y + (double)li.y,
                 zi = (double)hi.z + (double)li.z;
    const double qi = (double)hi.w;                    // q_hat = q sqrt(kT l_B)
    __syncthreads();                                   // the tables

    double fx = 0.0, fy = 0.0, fz = 0.0;
    cells::walk<LANES, false, kBlock, kList>(A.pos, A.first, G, live, i, c, hi, screen, list, [&](int j) {
        const float4 hj = A.pos[j], lj = A.lo[j];
        const double dx = xi - ((double)hj.x + (double)lj.x);
        const double dy = yi - ((double)hj.y + (double)lj.y);
        const double dz = zi - ((double)hj.z + (double)lj.z);
        const double r2 = dx * dx + dy * dy + dz * dz;
        const int p = ty * tb.T + A.typ[j];
        if (!(r2 < tr[p])) return;
        const double ir2 = 1.0 / r2;
        const double s2 = ts[p] * ir2, s6 = s2 * s2 * s2;
        const double glj = te[p] * (2.0 * s6 * s6 - s6) * ir2;
        const double gc = qi * (double)hj.w * ir2 * sqrt(ir2);
        const double gg = glj + gc;
        fx += gg * dx;
        fy += gg * dy;
        fz += gg * dz;
    });
#pragma unroll
    for (int o = 1; o < LANES; o <<= 1) {
        fx += __shfl_xor(fx, o);
        fy += __shfl_xor(fy, o);
        fz += __shfl_xor(fz, o);
    }
    int s = i;
    if (LANES > 1) {
        // one wavefront goes on, a slot a lane
        if (sub == 0) {
            sF[0][t / LANES] = fx;
            sF[1][t / LANES] = fy;
            sF[2][t / LANES] = fz;
        }
        __syncthreads();
        if (t >= kPart) return;
        s = blockIdx.x * kPart + t;
        fx = sF[0][t];
        fy = sF[1][t];
        fz = sF[2][t];
        if (s < A.n) {
            hi = A.pos[s];
            li = A.lo[s];
            ty = A.typ[s];
        }
    }
    const bool on = s < A.n;
    const size_t n = (size_t)A.n;
    if (!STEP) {
        if (on) {
            A.F[s] = fx;
            A.F[n + s] = fy;
            A.F[2 * n + s] = fz;
        }
        return;
    }
    double xn[3] = {0.0, 0.0, 0.0};
    float m = 0.f;
    if (on) {
        const long long step = A.st->step;
        const double R = radius_at(P.R, A.st->t + A.dt);   // the new radius precedes the surface force
        const double x[3] = {(double)hi.x + (double)li.x, (double)hi.y + (double)li.y,
                             (double)hi.z + (double)li.z};
        const double f[3] = {fx, fy, fz};
        double Fe[3];
        upd::ext_force(x, ty, R, P, Fe);
        double u[3] = {0.0, 0.0, 0.0};
        if (tb.kick > 0.0) {
            double xg[3];
            upd::gauss3((uint32_t)A.oid[s], (unsigned long long)step, A.seed, xg);
            const double len = sqrt(xg[0] * xg[0] + xg[1] * xg[1] + xg[2] * xg[2]);
            u[0] = xg[0] / len;
            u[1] = xg[1] / len;
            u[2] = xg[2] / len;
        }
        const double g = tb.gamma[ty], im = tb.inv_m[ty];
        bool ok = true;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            double vc = A.v[c * n + s];
            vc = vc + A.dt * (f[c] + Fe[c] - g * vc) * im;
            vc += tb.kick * u[c];
            const double d = A.dt * vc;
            if (!isfinite(d) || (P.jump_max > 0.0 && fabs(d) > P.jump_max)) ok = false;
            A.v2[c * n + s] = vc;
            xn[c] = x[c] + d;
        }
        if (!ok) atomicMin(&A.st->bad_step, (unsigned long long)step);
        const float4 h = make_float4((float)xn[0], (float)xn[1], (float)xn[2], hi.w);
        const float4 l = make_float4((float)(xn[0] - (double)h.x), (float)(xn[1] - (double)h.y),
                                     (float)(xn[2] - (double)h.z), 0.f);
        A.pos2[s] = h;
        A.lo2[s] = l;
        m = fmaxf(m, fmaxf(fabsf(h.x), fmaxf(fabsf(h.y), fabsf(h.z))));
        xn[0] = (double)h.x + (double)l.x;             // as k_pm_bin would read them
        xn[1] = (double)h.y + (double)l.y;
        xn[2] = (double)h.z + (double)l.z;
    }
    m = upd::wave_max(m);
    if (t % 64 == 0 && m > __uint_as_float(C.mx[A.next_mx]))
        atomicMax(&C.mx[A.next_mx], __float_as_uint(m));
    if (!A.bin) return;
    cells::bin<true>(cells::grid_of(mcur, tb.rmax), on, s, xn, C, A.ncell, A.nrank);
}

// Slot-order [3][n] -> original order [n][3].
__global__ __launch_bounds__(kB) void k_pm_to_orig(const double* __restrict__ src,
                                                   const int* __restrict__ oid, int n,
                                                   double* __restrict__ dst) {
    const int s = blockIdx.x * kB + threadIdx.x;
    if (s >= n) return;
    const size_t o = 3 * (size_t)oid[s];
    dst[o] = src[s];
    dst[o + 1] = src[(size_t)n + s];
    dst[o + 2] = src[2 * (size_t)n + s];
}

// Original order [n][3] -> slot order [3][n].
__global__ __launch_bounds__(kB) void k_pm_from_orig(const double* __restrict__ src,
                                                     const int* __restrict__ oid, int n,
                                                     double* __restrict__ dst) {
    const int s = blockIdx.x * kB + threadIdx.x;
    if (s >= n) return;
    const size_t o = 3 * (size_t)oid[s];
    dst[s] = src[o];
    dst[(size_t)n + s] = src[o + 1];
    dst[2 * (size_t)n + s] = src[o + 2];
}

#define PM_LAUNCH(kernel, grid, block, ...)                                               \
    do {                                                                                  \
        hipLaunchKernelGGL(kernel, grid, block, 0, __VA_ARGS__);                          \
        HIP_TRY(hipGetLastError());                                                       \
    } while (0)

template <class T>
bool pm_alloc(T** p, size_t count) {
    return hipMalloc(p, sizeof(T) * (count > 0 ? count : 1)) == hipSuccess;
}

// Step (i): the slots re-sorted by cell (slot arrays and velocities swapped
// with their second buffers).  binned: the step before counted the cells.
ld_status pm_sort(ld_ctx* c, hipStream_t s, bool binned, double adv_dt) {
    PaperMode* m = c->pm;
    const int n = (int)c->n, blocks = (n + kB - 1) / kB;
    const cells::Work C = cells::work_at(m->cells);
    if (!c->pos2) {
        if (!(pm_alloc(&c->pos2, (size_t)n) && pm_alloc(&c->lo2, (size_t)n) &&
              pm_alloc(&c->typ2, (size_t)n) && pm_alloc(&c->oid2, (size_t)n)))
            return fail(LD_ENOMEM, "cannot allocate the second slot arrays");
    }
    int* cell = reinterpret_cast<int*>(c->sb.keys);       // cells and ranks
    int* list = reinterpret_cast<int*>(c->sb.tmp4);       // lists and sorted cells
    const bool known = m->known;
    m->known = false;                  // until the step or the forces are enqueued
    if (!binned) {
        if (!known) m->turn = 0;
        HIP_TRY(cells::launch_absmax(c->pos, n, c->sb.bounds_part, C, s));   // and no counts
        PM_LAUNCH(k_pm_bin, dim3(blocks), dim3(kB), s, c->pos, c->lo, n, c->sb.bounds_part,
                  known ? (int)(m->turn % 3) : -1, m->tab.rmax, C, cell, cell + n);
        HIP_TRY(cells::launch_coarse(C, s));
    }
    HIP_TRY(cells::launch_scan(C, m->turn % 3, (m->turn + 2) % 3, m->tab.rmax, c->st, adv_dt, s));
    HIP_TRY(cells::launch_list(cell, cell + n, n, C, list, s));
    PmPlace A{};
    A.pos = c->pos;
    A.lo = c->lo;
    A.typ = c->typ;
    A.oid = c->oid;
    A.cell = cell;
    A.list = list;
    A.first = C.first;
    A.v = m->v;
    A.pos2 = c->pos2;
    A.lo2 = c->lo2;
    A.typ2 = c->typ2;
    A.oid2 = c->oid2;
    A.cell2 = list + n;
    A.v2 = m->v2;
    A.n = n;
    PM_LAUNCH(k_pm_place, dim3(blocks), dim3(kB), s, A);
    c->charged_first = c->n_charged == c->n;   // cell order mixes the two kinds
    std::swap(c->pos, c->pos2);
    std::swap(c->lo, c->lo2);
    std::swap(c->typ, c->typ2);
    std::swap(c->oid, c->oid2);
    std::swap(m->v, m->v2);
    c->boxes_stale = true;             // cell order now; a step moves the slots as well
    c->spatial = true;
    c->graph_len = -1;                 // a captured graph holds the old addresses
    c->steps_since_sort = 0;
    return LD_OK;
}

PmStep pm_launch(ld_ctx* c) {
    PaperMode* m = c->pm;
    PmStep A{};
    A.pos = c->pos;
    A.lo = c->lo;
    A.typ = c->typ;
    A.oid = c->oid;
    A.cell = reinterpret_cast<int*>(c->sb.tmp4) + c->n;
    A.first = cells::work_at(m->cells).first;
    A.n = (int)c->n;
    A.grid_mx = m->turn % 3;
    A.cur_mx = (m->turn + 1) % 3;
    A.next_mx = (m->turn + 2) % 3;
    return A;
}

template <bool STEP, int LANES>
void pm_run_as(const PmStep& A, ld_ctx* c, hipStream_t s) {
    constexpr int part = kPmBlock<LANES> / LANES;
    hipLaunchKernelGGL((k_pm_step<STEP, LANES>), dim3((A.n + part - 1) / part),
                       dim3(kPmBlock<LANES>), 0, s, A, c->pm->tab, c->ext,
                       cells::work_at(c->pm->cells));
}

template <bool STEP>
ld_status pm_run(const PmStep& A, ld_ctx* c, hipStream_t s) {
    // eight lanes a particle while a lane each would leave the chip's wavefronts
    // few and their chains long: a step of 5000 23 us (four lanes 25, one 32),
    // of 25 000 28 (28, 36), of 50 000 35 (34, 38), of 100 000 50 (47, 45), of
    // 250 000 97 (77, 65)
    if (A.n < kPmSplitN)
        pm_run_as<STEP, 8>(A, c, s);
    else
        pm_run_as<STEP, 1>(A, c, s);
    HIP_TRY(hipGetLastError());
    return LD_OK;
}

// Steps (i)-(ii) at the current positions into F.
ld_status pm_forces(ld_ctx* c, hipStream_t s) {
    PaperMode* m = c->pm;
    ld_status st = pm_sort(c, s, false, 0.0);
    if (st != LD_OK) return st;
    PmStep A = pm_launch(c);
    A.F = m->F;
    if ((st = pm_run<false>(A, c, s)) == LD_OK) m->known = true;
    return st;
}

}  // namespace

void pm_moved(ld_ctx* c) {
    if (c->pm) c->pm->known = false;
}

void pm_free(ld_ctx* c) {
    if (!c->pm) return;
    PaperMode* m = c->pm;
    void* b[] = {m->v, m->v2, m->F, m->cells};
    for (void* p : b)
        if (p) (void)hipFree(p);
    delete m;
    c->pm = nullptr;
}

ld_status pm_step(ld_ctx* c, double dt, hipStream_t s, bool first, bool last) {
    PaperMode* m = c->pm;
    const double adv = c->pend_dt;
    c->pend_dt = 0.0;
    ld_status st = pm_sort(c, s, !first, adv);
    if (st != LD_OK) return st;
    PmStep A = pm_launch(c);
    A.v = m->v;
    A.pos2 = c->pos2;
    A.lo2 = c->lo2;
    A.v2 = m->v2;
    A.st = c->st;
    A.dt = dt;
    A.seed = (unsigned long long)c->seed;
    A.bin = last ? 0 : 1;
    A.ncell = reinterpret_cast<int*>(c->sb.keys);
    A.nrank = A.ncell + A.n;
    if ((st = pm_run<true>(A, c, s)) != LD_OK) return st;
    std::swap(c->pos, c->pos2);
    std::swap(c->lo, c->lo2);
    std::swap(m->v, m->v2);
    ++m->turn;
    m->known = true;
    c->pend_dt = dt;
    return LD_OK;
}

}  // namespace ld

using namespace ld;
using namespace ld::host;

extern "C" {

ld_status ld_paper_enable(ld_ctx* c, const ld_paper_config* cfg) {
    g_err.clear();
    if (!c || !cfg) return fail(LD_EINVAL, "ctx and cfg are required");
    if (ff_active(c)) return fail(LD_ESTATE, "the learned far field is on (ld_ff_mode 0 first)");
    if (!(cfg->range_factor > 0.0) || !std::isfinite(cfg->range_factor))
        return fail(LD_EINVAL, "range_factor must be positive");
    if (!(cfg->kick >= 0.0) || !std::isfinite(cfg->kick))
        return fail(LD_EINVAL, "kick must be >= 0");
    const int T = c->p.n_types;
    for (int t = 0; t < T; ++t)
        if (!(cfg->inertial_mass[t] > 0.0) || !std::isfinite(cfg->inertial_mass[t]))
            return fail(LD_EINVAL, "inertial_mass[%d] must be positive", t);
    HIP_TRY(hipStreamSynchronize(c->stream));
    pm_free(c);
    PaperMode* m = new (std::nothrow) PaperMode();
    if (!m) return fail(LD_ENOMEM, "host allocation failed");
    m->cfg = *cfg;
    PmTable& tb = m->tab;
    tb.T = T;
    tb.rmax = 0.0;
    for (int a = 0; a < T; ++a)
        for (int b = 0; b < T; ++b) {
            const double sg = 0.5 * (c->p.sigma[a] + c->p.sigma[b]);
            const double e = c->p.use_eps_matrix ? c->p.eps_matrix[a * LD_MAX_TYPES + b]
                                                 : std::sqrt(c->p.eps[a] * c->p.eps[b]);
            const double rint = cfg->range_factor * sg;   // range_factor (r_a + r_b)
            tb.rint2[a * T + b] = rint * rint;
            tb.sig2[a * T + b] = sg * sg;
            tb.e24[a * T + b] = 24.0 * e;
            tb.rtype[a] = b == 0 ? rint : std::max(tb.rtype[a], rint);
            tb.rmax = std::max(tb.rmax, rint);
        }
    for (int t = 0; t < T; ++t) {
        tb.inv_m[t] = 1.0 / cfg->inertial_mass[t];
        tb.gamma[t] = c->p.gamma[t];
    }
    tb.kick = cfg->kick;
    const size_t N = (size_t)c->n;
    bool ok = pm_alloc(&m->v, 3 * N) && pm_alloc(&m->v2, 3 * N) && pm_alloc(&m->F, 3 * N) &&
              pm_alloc(&m->cells, cells::kWorkInts);
    if (ok) {
        std::vector<double> zero(3 * N, 0.0);
        ok = hipMemcpy(m->v, zero.data(), sizeof(double) * 3 * N, hipMemcpyHostToDevice) ==
             hipSuccess;
    }
    c->pm = m;
    if (!ok) {
        pm_free(c);
        return fail(LD_ENOMEM, "cannot allocate the paper scheme's buffers");
    }
    return LD_OK;
}

ld_status ld_paper_disable(ld_ctx* c) {
    g_err.clear();
    if (!c) return fail(LD_EINVAL, "ctx is NULL");
    HIP_TRY(hipStreamSynchronize(c->stream));
    pm_free(c);
    return LD_OK;
}

ld_status ld_paper_forces(ld_ctx* c, double* F) {
    g_err.clear();
    if (!c || !F) return fail(LD_EINVAL, "ctx and F are required");
    if (!c->pm) return fail(LD_ESTATE, "ld_paper_enable first");
    const int n = (int)c->n;
    hipStream_t s = c->stream;
    ld_status st = pm_forces(c, s);
    if (st != LD_OK) return st;
    double* dF = c->work;
    PM_LAUNCH(k_pm_to_orig, dim3((n + kB - 1) / kB), dim3(kB), s, c->pm->F, c->oid, n, dF);
    HIP_TRY(copy_out(c->stage, F, dF, sizeof(double) * 3 * (size_t)n, s));
    return LD_OK;
}

ld_status ld_paper_get_velocities(ld_ctx* c, double* v) {
    g_err.clear();
    if (!c || !v) return fail(LD_EINVAL, "ctx and v are required");
    if (!c->pm) return fail(LD_ESTATE, "ld_paper_enable first");
    const int n = (int)c->n;
    double* d = c->work;
    PM_LAUNCH(k_pm_to_orig, dim3((n + kB - 1) / kB), dim3(kB), c->stream, c->pm->v, c->oid, n, d);
    HIP_TRY(copy_out(c->stage, v, d, sizeof(double) * 3 * (size_t)n, c->stream));
    return LD_OK;
}

ld_status ld_paper_set_velocities(ld_ctx* c, const double* v) {
    g_err.clear();
    if (!c || !v) return fail(LD_EINVAL, "ctx and v are required");
    if (!c->pm) return fail(LD_ESTATE, "ld_paper_enable first");
    const size_t N = (size_t)c->n;
    std::vector<double> h;
    ld_status st = read_host(h, v, 3 * N, c->stream);
    if (st != LD_OK) return st;
    for (double x : h)
        if (!std::isfinite(x)) return fail(LD_EINVAL, "velocities must be finite");
    double* d = c->work;
    HIP_TRY(hipMemcpyAsync(d, h.data(), sizeof(double) * 3 * N, hipMemcpyHostToDevice, c->stream));
    PM_LAUNCH(k_pm_from_orig, dim3(((int)N + kB - 1) / kB), dim3(kB), c->stream, d, c->oid, (int)N,
              c->pm->v);
    HIP_TRY(hipStreamSynchronize(c->stream));
    return LD_OK;
}

}  // extern "C"
