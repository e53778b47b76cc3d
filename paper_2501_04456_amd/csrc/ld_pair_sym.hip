// Forces of a large droplet: the symmetric Coulomb tasks (ld_sym_core.h) and,
// in the same launch, the Lennard-Jones groups, whose latency they hide.
#include "ld_sym_core.h"

namespace ld {
namespace {

struct SymArgs {
    const float4* pos;
    const float4* lo;
    const int* typ;
    const Box* box;
    int n, ngroups;
    double* F;                             // [slots][3][n]
    DevState* st;                          // step clock to advance by adv_dt first (or null)
    double adv_dt;
    int lj_blocks, lj_every;               // workgroups that take Lennard-Jones groups
    PairTable tab;
    SymPlan p;
};

template <int kJB, bool LONG>
__global__ __launch_bounds__(64 * sym::kW, 3) void k_pair_sym(SymArgs A) {
    __shared__ union U {
        sym::Shared<kJB> c;
        pair::LjBlock<sym::kW, 3, LONG> lj;
        __device__ U() {}
    } sh;
    if (A.adv_dt > 0.0 && blockIdx.x == 0 && threadIdx.x == 0) {
        A.st->t = A.st->t + A.adv_dt;
        A.st->step = A.st->step + 1;
    }
    // every lj_every-th workgroup takes a Lennard-Jones group while there are any
    const int turn = (int)blockIdx.x / A.lj_every;
    if ((int)blockIdx.x % A.lj_every == 0 && turn < A.lj_blocks) {
        double sums[3];
        if (!pair::lj_block<false, true, sym::kW, LONG>(A.pos, A.lo, A.typ, A.box, A.n, turn,
                                                        A.tab, sh.lj, sums))
            return;
        const size_t i = (size_t)turn * kGroup + threadIdx.x;
        for (int c = 0; c < 3; ++c) A.F[c * (size_t)A.n + i] = -sums[c];
        return;
    }
    const int t = (int)blockIdx.x - min(A.lj_blocks, turn + 1);
    const int chunk = t / A.p.nA, sa = t % A.p.nA;
    sym::View V;
    V.pos = A.pos;
    V.lo = A.lo;
    V.box = A.box;
    V.n = A.n;
    V.ngroups = A.ngroups;
    V.cull2 = A.tab.rc2max * 1.0001f;
    V.F = A.F;
    V.stride = (size_t)A.n;
    V.nbc = A.p.nbc;
    V.mA = A.p.mA;
    V.nA = A.p.nA;
    V.nds = A.p.nds;
    sym::task<kJB>(V, sa, chunk, A.p.start[chunk], A.p.start[chunk + 1], sh.c);
}

}  // namespace

// Blocks, super-blocks and chunks for n slots of which the first `charged`
// are charged.  Larger super-blocks take fewer partials (each is an FP64
// triple per slot, written once and read once by the update): the smallest
// (from one block of 4 groups, or two of 8) that stays within kSymAimBytes,
// else the largest if it does within kSymMaxBytes.
//   nds: column super-blocks a row super-block can own pairs with (itself
//        first); one column partial each.
//   chunks: runs of those, one row partial each, as long as leaves about twelve
//        rounds of workgroups over the chip's 768 (three per compute unit), the
//        last runs short so that the launch ends evenly.  A run is one
//        super-block at least, so there are fewer workgroups where the
//        super-blocks are few: all charged, 1200 at 12 288 slots, 3280 at
//        81 920, 2046 at 500 000 (super-blocks of 16), 8320 to 11 200 at 32 768,
//        81 919, 250 000 and 1 200 000.
// Blocks of 4 groups below kSymSmallN slots, where blocks of 8 are too few
// workgroups to share out evenly.
bool sym_plan(int64_t n, int64_t charged, SymPlan* p) {
    p->jb = n < kSymSmallN ? 4 : 8;
    const int64_t per = (int64_t)p->jb * kGroup;
    p->nbc = (int)((charged + per - 1) / per);
    p->n_full = (int)(p->nbc * per < n ? p->nbc * per : n);
    const int H = p->nbc / 2;
    for (p->mA = p->jb == 8 ? 2 : 1; p->mA <= 16; p->mA *= 2) {
        const int mA = p->mA;
        p->nA = (p->nbc + mA - 1) / mA;
        const int nds = (mA - 1 + H) / mA + 1 + (p->nbc % mA != 0 ? 1 : 0);
        p->nds = nds < p->nA ? nds : p->nA;
        int len = (int)((int64_t)p->nds * p->nA / 9216);
        if (len < 1) len = 1;
        while ((p->nds + len - 1) / len + 8 > kSymMaxChunks) ++len;
        int k = 0, at = 0;
        while (at < p->nds) {
            p->start[k++] = (short)at;
            const int left = p->nds - at;
            int step = len;
            if (step > 1 && left <= 3 * step) step = left > 3 ? (left + 2) / 3 : 1;
            at += step < left ? step : left;
        }
        p->start[k] = (short)p->nds;
        p->nchunk = p->nA > 0 ? k : 0;
        p->slots = 1 + p->nds + p->nchunk;
        const size_t bytes = sizeof(double) * 3 * (size_t)n * p->slots;
        if (bytes <= kSymAimBytes || p->mA == 16) return bytes <= kSymMaxBytes && p->nds < 32768;
    }
    return false;
}

hipError_t launch_pair_sym(const PairLaunch& L, const PairTable& tab, hipStream_t s,
                           hipEvent_t before_coulomb, hipEvent_t after_coulomb) {
    SymArgs A{};
    A.pos = L.pos;
    A.lo = L.lo;
    A.typ = L.typ;
    A.box = L.box;
    A.n = L.n;
    A.ngroups = (L.n + kGroup - 1) / kGroup;
    A.F = L.Fpart;
    A.st = L.st;
    A.adv_dt = L.adv_dt;
    A.tab = tab;
    A.p = *L.sym;
    const int tasks = A.p.nA * A.p.nchunk;                   // 0: nothing charged
    auto launch = [&](int lj, int coulomb) {
        A.lj_blocks = lj;
        if (lj + coulomb == 0) return;
        A.lj_every = sym::lj_stride(lj, coulomb);
        const bool far = pair::lj_long(tab);
        hipLaunchKernelGGL(A.p.jb == 4 ? (far ? k_pair_sym<4, true> : k_pair_sym<4, false>)
                                       : (far ? k_pair_sym<8, true> : k_pair_sym<8, false>),
                           dim3(lj + coulomb), dim3(64 * sym::kW), 0, s, A);
        A.adv_dt = 0.0;
    };
    if (!after_coulomb) {
        launch(A.ngroups, tasks);
        return hipGetLastError();
    }
    // timed: the Coulomb tasks by themselves
    launch(A.ngroups, 0);
    hipError_t e = hipEventRecord(before_coulomb, s);
    if (e != hipSuccess) return e;
    launch(0, tasks);
    e = hipEventRecord(after_coulomb, s);
    return e != hipSuccess ? e : hipGetLastError();
}

}  // namespace ld
