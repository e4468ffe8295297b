// Host memory that a kernel writes its few result words to (entry counts, verdicts), for the entry points that return them.
// A copy of device memory to the host is a launch of its own, and one to unpinned memory waits for it besides: a plan of
// 2,708 nodes 32 us, 24 so, a construction of 5,429 pairs 50, 42; a whole pass over that graph 167, 135.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

constexpr size_t kReportBytes = 2048;

// One piece of kReportBytes of pinned memory, for kernels on one stream; get() is NULL where none is to be had (all
// taken by other threads, or no such memory): the caller then copies from device memory instead.  Pieces come from one
// allocation per process, made on first use and kept; `allocate` false, for an entry point that is documented not to allocate:
// there is a piece only if another call has made that allocation.
// A piece is another call's next, so it goes back only once the stream has been waited for: by wait(), or else by the
// destructor, on the way out of a call that launched kernels and then failed.  Where that fails too, the piece stays out.
class HostReport {
public:
    explicit HostReport(hipStream_t stream, bool allocate = true);
    ~HostReport();
    HostReport(const HostReport&) = delete;
    HostReport& operator=(const HostReport&) = delete;
    void* get() const { return piece_; }
    // after it, what the stream's kernels wrote to the piece is there
    hipError_t wait();

private:
    hipStream_t stream_;
    void* piece_ = nullptr;
    int index_ = -1;
    bool waited_ = false;
};
