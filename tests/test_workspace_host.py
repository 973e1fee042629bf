"""The per-stream workspaces (cyc_workspace.hip) on the CPU: its host code compiled against a stand-in for the few HIP calls it
makes, so that allocations can fail, streams can be captured and threads can meet without a GPU."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
SOURCE = os.path.join(HERE, "..", "paper_2511_09987_amd", "csrc", "cyc_workspace.hip")

STAND_IN = r'''
#include <hip/hip_runtime.h>
#define HIP_SYMBOL(x) (&(x))
#define __align__(n) __attribute__((aligned(n)))
#include SOURCE
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <set>
#include <string>
#include <thread>
#include <vector>
#include <chrono>

// ---- the stand-in: memory of `room` bytes, streams 1 .. 9, the calls in the order they came
static std::mutex mu;
static std::map<void *, size_t> live;
static size_t used = 0, room = (size_t)1 << 40;
static hipError_t last = hipSuccess;
static std::set<hipStream_t> capturing, odd;           // odd: asking whether it is captured is an error
static thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;
static std::vector<std::string> calls;
static hipError_t done(hipError_t e) { if (e != hipSuccess) last = e; return e; }
extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { std::lock_guard<std::mutex> g(mu); hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *st)
{
    std::lock_guard<std::mutex> g(mu);
    *st = capturing.count(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return done(odd.count(s) ? hipErrorStreamCaptureImplicit : hipSuccess);
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *m) { std::swap(*m, mode); return hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes)
{
    std::lock_guard<std::mutex> g(mu);
    calls.push_back("malloc");
    if (!capturing.empty() && mode != hipStreamCaptureModeRelaxed) return done(hipErrorStreamCaptureUnsupported);
    if (used + bytes > room) return done(hipErrorOutOfMemory);
    *p = std::malloc(1);
    live[*p] = bytes;
    used += bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> g(mu);
    calls.push_back("free");
    if (!capturing.empty()) return done(hipErrorStreamCaptureUnsupported);
    if (!live.count(p)) { std::puts("freed what is not there"); std::exit(1); }
    used -= live[p];
    live.erase(p);
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *symbol) { *p = (void *)symbol; return hipSuccess; }
}
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); std::exit(1); } } while (0)
static hipStream_t stream(int i) { return (hipStream_t)(uintptr_t)i; }
static void *get(int s, int64_t bytes) { cyc::WorkspaceHold hold; return hold.acquire(stream(s), bytes); }
constexpr int64_t MiB = 1 << 20;

static void no_error_is_left()
{
    room = 4 * MiB;
    CHECK(get(1, 8 * MiB) == nullptr);
    CHECK(last == hipSuccess);
    odd.insert(stream(2));
    CHECK(get(2, MiB) != nullptr);
    CHECK(last == hipSuccess);
    CHECK(!cyc::is_capturing(stream(2)) && last == hipSuccess);
}

static void a_lock_per_buffer()
{
    cyc::WorkspaceHold mine;
    CHECK(mine.acquire(stream(1), MiB) != nullptr);
    // another stream's buffer and the fixed array are there meanwhile
    std::atomic<int> others{0}, same{0};
    std::thread other([&] { CHECK(get(2, MiB) != nullptr); int64_t n; CHECK(cyc::static_workspace(&n) != nullptr); others = 1; });
    for (int i = 0; i < 500 && !others; ++i) std::this_thread::sleep_for(std::chrono::milliseconds(10));
    CHECK(others == 1);
    other.join();
    // this stream's is not, until its holder goes
    std::thread waits([&] { cyc::WorkspaceHold theirs; theirs.acquire(stream(1), 2 * MiB); same = 1; });
    std::this_thread::sleep_for(std::chrono::milliseconds(200));
    CHECK(same == 0);
    mine.~WorkspaceHold();
    new (&mine) cyc::WorkspaceHold();
    waits.join();
    CHECK(same == 1);
}
static size_t frees() { size_t n = 0; for (auto &c : calls) n += c == "free"; return n; }
static void growth()
{
    void *first = get(1, MiB);
    CHECK(get(1, 1) == first && get(1, MiB) == first);
    void *second = get(1, 3 * MiB);
    CHECK(second && live.count(second) && !live.count(first) && used == 3 * MiB);
    CHECK(calls == (std::vector<std::string>{"malloc", "malloc", "free"}));
    room = 5 * MiB;                                      // no room for both: the old one goes first
    CHECK(get(1, 4 * MiB) != nullptr && used == 4 * MiB && last == hipSuccess);
    CHECK(get(1, 6 * MiB) == nullptr && used == 0);      // and none at all: refused, and the next call gets what there is
    CHECK(get(1, MiB) != nullptr && used == MiB);
    // refused for another reason, a capture on another stream: the buffer stays
    capturing.insert(stream(9));
    const size_t before = frees();
    void *kept = get(1, MiB);
    CHECK(get(1, 2 * MiB) == nullptr && last == hipSuccess && get(1, MiB) == kept && frees() == before);
}
static void capture()
{
    // first call of a stream, whatever the capture's mode: it gets its memory, and the thread its mode back
    capturing.insert(stream(1));
    void *graph1 = get(1, MiB);
    CHECK(graph1 && mode == hipStreamCaptureModeGlobal && last == hipSuccess);
    capturing.clear();
    // a larger call leaves the graph its buffer
    void *eager = get(1, 2 * MiB);
    CHECK(eager && live.count(graph1) && frees() == 0);
    // a larger one under a capture leaves the eager buffer, which may be in use, to a later call
    capturing.insert(stream(1));
    void *graph2 = get(1, 3 * MiB);
    CHECK(graph2 && live.count(eager) && frees() == 0);
    CHECK(get(1, 4 * MiB) != nullptr && live.count(graph2));
    capturing.clear();
    CHECK(get(1, 5 * MiB) && !live.count(eager) && live.count(graph1) && live.count(graph2) && frees() == 1);
    // no room under a capture: refused, nothing freed, the buffer still there for what fits
    room = used;
    capturing.insert(stream(1));
    void *before = get(1, MiB);
    CHECK(get(1, 50 * MiB) == nullptr && last == hipSuccess && get(1, MiB) == before && frees() == 1);
}
int main(int argc, char **argv)
{
    const std::string what = argv[1];
    if (what == "no_error_is_left") no_error_is_left();
    else if (what == "a_lock_per_buffer") a_lock_per_buffer();
    else if (what == "growth") growth();
    else if (what == "capture") capture();
    else return 2;
    std::puts("ok");
    return 0;
}
'''


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    at = tmp_path_factory.mktemp("workspace")
    main = at / "main.cpp"
    main.write_text(STAND_IN)
    out = at / "workspace"
    p = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        f'-DSOURCE="{os.path.abspath(SOURCE)}"', str(main), "-o", str(out)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert p.returncode == 0, p.stdout
    return str(out)


SCENARIOS = ["no_error_is_left", "a_lock_per_buffer", "growth", "capture"]


@pytest.mark.parametrize("scenario", SCENARIOS)
def test_workspace(program, scenario):
    p = subprocess.run([program, scenario], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=60)
    assert p.returncode == 0, p.stdout
