// Host memory that a kernel writes its few result words to (entry counts, verdicts), for the entry points that return them.
// A copy of device memory to the host is a launch of its own, and one to unpinned memory waits for it besides: a plan of
// 2,708 nodes 32 us, 24 so, a construction of 5,429 pairs 50, 42; a whole pass over that graph 167, 135.
#pragma once
#include <stddef.h>

constexpr size_t kReportBytes = 2048;

// One piece of kReportBytes of pinned memory, from its construction to its destruction; get() is NULL where none is to be
// had (all taken by other threads, or no such memory): the caller then copies from device memory instead.  Pieces come from one
// allocation per process, made on first use and kept.
class HostReport {
public:
    HostReport();
    ~HostReport();
    HostReport(const HostReport&) = delete;
    HostReport& operator=(const HostReport&) = delete;
    void* get() const { return piece_; }

private:
    void* piece_ = nullptr;
    int index_ = -1;
};
