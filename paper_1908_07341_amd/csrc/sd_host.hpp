// Host helpers shared by the C-ABI translation units.
#pragma once

#include <stdint.h>

#include <mutex>

#include "shaken.h"
#include "sd_kernels.hpp"
#include "sd_small.hpp"

namespace sd {

sd_status fail(sd_status s, const char* fmt, ...);
sd_status hip_fail(hipError_t e, const char* what);
bool layout_supported(int32_t L, int32_t layout);
size_t lattice_bytes(int32_t L, int32_t layout);
Geom make_geom(int32_t L, int klay);
int kernel_layout(int32_t L, int32_t layout, const void* p);
int packed_rows_layout(int32_t L);
uint32_t threshold(double h);
void threshold_table(double J, double q, uint32_t T[6]);
// The initial lattice of sd_init: validates kind and p_up and sets whether the
// lattice is random (with the draw parameters dp) or constant, all +1 (up) or
// all -1.
sd_status init_params(const char* name, int32_t kind, double p_up, uint64_t seed, uint32_t stream, DrawParams* dp,
                      bool* random, bool* up);
// The lattice pointer's checks of the entry points (size and layout, null,
// alignment to the word size).
sd_status check_lattice(const void* p, int32_t L, int32_t layout, const char* name);
DrawParams dynamics_params(double J, double q, uint64_t seed, uint32_t stream, uint32_t t, uint32_t flags);

// The stream is being captured into a graph (or cannot be asked).
bool capturing(hipStream_t st);
// The current device's CUs and LDS bytes a workgroup may have.
hipError_t device_limits(uint32_t* n_cu, size_t* max_lds);
// Arguments of the small-lattice kernel for k_steps steps from step0; the
// caller adds the lattices or pairs.
SmallArgs small_args(int32_t L, double J, double q, uint64_t seed, uint32_t stream, uint64_t step0, uint32_t k_steps,
                     uint32_t flags);

// Device scratch of kPartialsWords int64 for per-workgroup partial sums, one
// per (device, stream), allocated on first use and kept for the process.
constexpr size_t kPartialsWords = 65536;
struct Workspace {
    int64_t* p = nullptr;
    void* ahead = nullptr;   // kAheadBytes, made by the first run that draws ahead (AheadScratch)
    std::mutex mu;
    hipEvent_t last_use = nullptr;   // hipStreamPerThread only: behind the last call's work
    bool lost = false;               // ... could not be recorded: later calls have nothing to wait for
};

// A call's use of its stream's workspace, held while it enqueues the launches
// that write and read it, so that calls from several host threads on one
// stream do not interleave.  get() is null while the stream is being captured
// (a graph that held p would share it with the stream's own calls wherever it
// is replayed), or when the workspace cannot be made (the allocation failed);
// callers then use atomics.  hipStreamPerThread is one handle but another queue
// in every host thread: a call on it waits on the device for the last user's
// work and leaves an event behind its own.
class WorkspaceUse {
public:
    WorkspaceUse() = default;
    explicit WorkspaceUse(hipStream_t st);
    ~WorkspaceUse() { release(); }
    WorkspaceUse(const WorkspaceUse&) = delete;
    WorkspaceUse& operator=(WorkspaceUse&& o) {
        release();
        ws_ = o.ws_;
        st_ = o.st_;
        o.ws_ = nullptr;
        return *this;
    }
    Workspace* get() const { return ws_; }

private:
    void release();
    Workspace* ws_ = nullptr;
    hipStream_t st_ = nullptr;
};

// Scratch of the draw-ahead runs (class masks of two rounds), held while a call
// enqueues.  The first kAheadBuffers streams of a device keep a buffer each with
// their workspace (the caller holds it); calls on later ones borrow one of
// kAheadShared, each behind an event that its last borrower left, so that
// speed does not depend on which streams came first, used ones and destroyed
// ones alike, and a device holds 320 MiB at most.  (An event per call costs a
// stream 2.9 us, which the streams with buffers of their own need not pay.)
// get() is null out of memory, and the caller takes the kernels that need none.
constexpr size_t kAheadBytes = 16u << 20;
constexpr uint32_t kAheadBuffers = 16, kAheadShared = 4;
struct AheadShared;
class AheadScratch {
public:
    AheadScratch(Workspace& ws, hipStream_t st);
    ~AheadScratch();
    AheadScratch(const AheadScratch&) = delete;
    void* get() const { return p_; }

private:
    void* p_ = nullptr;
    AheadShared* shared_ = nullptr;   // borrowed from
    hipStream_t st_ = nullptr;
};

}  // namespace sd
