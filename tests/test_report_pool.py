"""The pinned memory of result words (csrc/report.hip) against a HIP runtime of a few lines, on the CPU: when a piece may be
another call's, and what happens where memory or the stream fails."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2302_13053_amd", "csrc")

RUNTIME = r"""
#pragma once
#include <stddef.h>
#include <stdlib.h>
typedef int hipError_t;
typedef struct stream_* hipStream_t;
enum { hipSuccess = 0, hipErrorUnknown = 999 };
enum { hipHostMallocPortable = 1, hipHostMallocMapped = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeGlobal, hipStreamCaptureModeThreadLocal, hipStreamCaptureModeRelaxed };
inline hipStreamCaptureMode capture_mode = hipStreamCaptureModeGlobal;
inline hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m)
{
    const hipStreamCaptureMode t = capture_mode;
    capture_mode = *m;
    *m = t;
    return hipSuccess;
}
inline int waits = 0, allocations = 0, last_error = hipSuccess;
inline bool no_memory = false, stream_broken = false, pending = false;      // pending: a kernel still writes to a piece
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    if (no_memory || capture_mode != hipStreamCaptureModeRelaxed) return last_error = hipErrorUnknown;
    ++allocations;
    *p = malloc(n);
    return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t)
{
    ++waits;
    if (stream_broken) return last_error = hipErrorUnknown;
    pending = false;
    return hipSuccess;
}
inline hipError_t hipGetLastError() { const int e = last_error; last_error = hipSuccess; return e; }
"""

MAIN = r"""
#include <stdio.h>
#include "%s/report.hip"
#define CHECK(x) do { if (!(x)) { printf("line %%d: %%s\n", __LINE__, #x); return 1; } } while (0)
int main()
{
    void* first;
%s
    return 0;
}
"""

CASES = {
    "a call that ends well waits once": """
    { HostReport r(nullptr); first = r.get(); CHECK(first); pending = true; CHECK(r.wait() == hipSuccess); CHECK(!pending); }
    CHECK(waits == 1);
    { HostReport r(nullptr); CHECK(r.get() == first); CHECK(r.wait() == hipSuccess); }
    CHECK(allocations == 1);
""",
    "a call that fails after a launch gives the piece back when the kernel is done": """
    { HostReport r(nullptr); first = r.get(); pending = true; }
    CHECK(!pending);
    { HostReport r(nullptr); CHECK(r.get() == first); }
""",
    "a piece that a kernel may still write to is nobody's": """
    { HostReport r(nullptr); first = r.get(); stream_broken = true; CHECK(r.wait() != hipSuccess); }
    stream_broken = false;
    { HostReport r(nullptr); CHECK(r.get() && r.get() != first); }
""",
    "more calls at once than pieces": """
    { HostReport* all[33];
      for (int i = 0; i < 33; ++i) { all[i] = new HostReport(nullptr); CHECK((all[i]->get() != nullptr) == (i < 32)); }
      for (int i = 0; i < 32; ++i) for (int j = 0; j < i; ++j) {
          const long d = (char*)all[i]->get() - (char*)all[j]->get();
          CHECK(d >= (long)kReportBytes || -d >= (long)kReportBytes);
      }
      for (int i = 0; i < 33; ++i) { CHECK(all[i]->wait() == hipSuccess); delete all[i]; } }
    { HostReport r(nullptr); CHECK(r.get()); }
""",
    "no pinned memory": """
    no_memory = true;
    { HostReport r(nullptr); CHECK(!r.get()); CHECK(r.wait() == hipSuccess); }
    CHECK(hipGetLastError() == hipSuccess);
    no_memory = false;
    { HostReport r(nullptr); CHECK(r.get()); }
    CHECK(capture_mode == hipStreamCaptureModeGlobal);
""",
    "a call that must not allocate": """
    { HostReport r(nullptr, false); CHECK(!r.get()); CHECK(r.wait() == hipSuccess); }
    CHECK(allocations == 0);
    { HostReport r(nullptr); first = r.get(); CHECK(first); }
    { HostReport r(nullptr, false); CHECK(r.get() == first); }
""",
}


@pytest.mark.parametrize("what", list(CASES))
def test_pieces(tmp_path, what):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp_path / "main.cpp").write_text(MAIN % (CSRC, CASES[what]))
    subprocess.run(["g++", "-std=c++17", "-pthread", "-I", str(tmp_path), "-I", CSRC, "-x", "c++", str(tmp_path / "main.cpp"),
                    "-o", str(tmp_path / "main")], check=True)
    r = subprocess.run([str(tmp_path / "main")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
