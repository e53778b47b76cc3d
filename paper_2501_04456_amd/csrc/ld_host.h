// Host-side helpers shared by the C ABI files: error text, pointer kinds,
// parameter checks and the parameter tables handed to kernels.
#pragma once

#include <cstring>
#include <initializer_list>
#include <string>
#include <vector>

#include "ld_internal.h"

namespace ld {
namespace host {

extern thread_local std::string g_err;

// Record an error message and return the status.
ld_status fail(ld_status s, const char* fmt, ...);

#define HIP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return ::ld::host::fail(LD_EHIP, "%s failed: %s", #expr,                    \
                                    hipGetErrorString(e_));                             \
    } while (0)

bool is_device_ptr(const void* p);
hipError_t copy_in(void* dst, const void* src, size_t bytes, hipStream_t s);
hipError_t copy_out(void* dst, const void* src, size_t bytes, hipStream_t s);
constexpr size_t kReadSlot = 512 << 10, kBatchSlot = 1 << 20;

// Plans a stage whose slots together hold about `bytes`, each at most max_slot (read
// back best in pieces of 512 KiB, which the host still finds in its cache: 250
// 000 positions 205 us, with 1 or 2 MiB 245; batches uploaded best in pieces of
// 1 MiB: training passes of 16 MB with 0.5, 1, 2 MiB 760, 640, 780 us, 800 with
// a pageable copy into a buffer allocated for it).  The memory is taken by the
// first copy where a frame is at most kDirectOut, else at once: pinning takes 30
// us of the 250 that a small droplet's context takes to make, and 60 to give
// back; behind work in flight it takes longer for larger contexts (the first
// analysis of 250 000 NPs 1160 us, 1270 with it in there).
void stage_plan(HostStage& h, size_t bytes, size_t max_slot);
void stage_plan_frame(HostStage& h, size_t bytes);
// Whether there are slots; without pinned memory there are none and copies are
// not staged.
bool stage_open(HostStage& h);
void stage_free(HostStage& h);
// The next slot, free for the host to write; stage_mark records that the work
// enqueued on s last uses it.
hipError_t stage_take(HostStage& h, char** slot, int* k);
hipError_t stage_mark(HostStage& h, int k, hipStream_t s);
// copy_out and copy_in through the stage; the first waits for all that the
// stream holds, several pieces (null destinations are left out) share the slots
// and the wait.
struct Piece {
    void* dst;                           // host or device
    const void* src;
    size_t bytes;
};
constexpr int kMaxPieces = 8;
hipError_t copy_out(HostStage& h, std::initializer_list<Piece> pieces, hipStream_t s);
hipError_t copy_out(HostStage& h, void* dst, const void* src, size_t bytes, hipStream_t s);
hipError_t copy_in(HostStage& h, void* dst, const void* src, size_t bytes, hipStream_t s);
ld_status check_params(const ld_params* p);
ld_status check_radius(const ld_radius* R);
void make_tables(const ld_params& p, const ld_radius& R, PairTable& tb, ExtParams& P);

// Read a caller array of `count` elements (host or device) into host memory.
template <class T>
ld_status read_host(std::vector<T>& v, const T* src, size_t count, hipStream_t s) {
    v.resize(count);
    if (is_device_ptr(src)) {
        HIP_TRY(hipMemcpyAsync(v.data(), src, count * sizeof(T), hipMemcpyDeviceToHost, s));
        HIP_TRY(hipStreamSynchronize(s));
    } else {
        std::memcpy(v.data(), src, count * sizeof(T));
    }
    return LD_OK;
}

// Write a host array to a caller pointer (host or device); waits.
inline hipError_t put_out(void* dst, const void* src, size_t bytes, hipStream_t s) {
    if (!dst) return hipSuccess;
    if (is_device_ptr(dst)) {
        hipError_t e = hipMemcpyAsync(dst, src, bytes, hipMemcpyHostToDevice, s);
        return e == hipSuccess ? hipStreamSynchronize(s) : e;
    }
    std::memcpy(dst, src, bytes);
    return hipSuccess;
}

}  // namespace host
}  // namespace ld
