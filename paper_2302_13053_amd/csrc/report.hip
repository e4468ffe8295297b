#include "report.hpp"

#include <mutex>
#include <stdint.h>

namespace {

constexpr int kPieces = 32;

struct Pool {
    std::mutex lock;
    char* memory = nullptr;
    uint32_t taken = 0;          // bit per piece
};
// never destroyed: a thread may still hold a piece when the process ends
Pool& pool()
{
    static Pool* p = new Pool;
    return *p;
}

}  // namespace

HostReport::HostReport(hipStream_t stream, bool allocate) : stream_(stream)
{
    Pool& p = pool();
    std::lock_guard<std::mutex> guard(p.lock);
    if (!p.memory) {
        if (!allocate) return;
        // (an allocation would end a capture that another thread has begun in the global mode)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        // readable and writable by every device, coherent: what a kernel has written is there once the stream has been waited for
        void* m = nullptr;
        const hipError_t e = hipHostMalloc(&m, kPieces * kReportBytes, hipHostMallocPortable | hipHostMallocMapped);
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return;
        }
        p.memory = (char*)m;
    }
    if (p.taken == 0xffffffffu) return;
    index_ = __builtin_ctz(~p.taken);
    p.taken |= 1u << index_;
    piece_ = p.memory + (size_t)index_ * kReportBytes;
}

hipError_t HostReport::wait()
{
    const hipError_t e = hipStreamSynchronize(stream_);
    waited_ = e == hipSuccess;
    return e;
}

HostReport::~HostReport()
{
    if (index_ < 0 || (!waited_ && wait() != hipSuccess)) return;
    Pool& p = pool();
    std::lock_guard<std::mutex> guard(p.lock);
    p.taken &= ~(1u << index_);
}
