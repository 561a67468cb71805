"""Host side of sthosvd_compress with the device replaced by stubs: work that a
call enqueues runs when its stream is synchronised, and the eigensolver's
publication of the scalar block is part of that work.  No call may return
while a publication of its own is still to come: the block belongs to the
thread, whose next call may run on another stream and another device."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#define __align__(n) alignas(n)
#define HIP_SYMBOL(x) (x)
static int __builtin_amdgcn_readfirstlane(int x) { return x; }
#include "api.cpp"

#include <functional>
#include <map>

namespace {
std::map<hipStream_t, std::vector<std::function<void()>>> todo;
int queries_busy, yields;  // the stream is busy for so many queries; a yield lets it run
int eigs, ttms, fail_eig, fail_ttm;  // fail_x: the x-th launch fails after enqueueing its kernel

void drain(hipStream_t st) {
    auto work = std::move(todo[st]);
    todo[st].clear();
    for (auto& w : work) w();
}
}  // namespace

#define EXPORT __attribute__((visibility("default")))
extern "C" {
EXPORT hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return *p = malloc(n), hipSuccess; }
EXPORT hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, hipSuccess; }
EXPORT hipError_t hipGetLastError() { return hipSuccess; }
EXPORT const char* hipGetErrorString(hipError_t) { return "stub"; }
EXPORT hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
EXPORT hipError_t hipGetSymbolAddress(void**, const void*) { return hipErrorUnknown; }
EXPORT hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
EXPORT hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
    todo[st].push_back([=] { memcpy(d, s, n); });
    return hipSuccess;
}
EXPORT hipError_t hipStreamSynchronize(hipStream_t st) { return drain(st), hipSuccess; }
EXPORT hipError_t hipStreamQuery(hipStream_t st) {
    if (queries_busy > 0) return --queries_busy, hipErrorNotReady;
    return drain(st), hipSuccess;
}
EXPORT int sched_yield() {
    ++yields;
    if (queries_busy > 0)
        for (auto& t : todo) drain(t.first);
    return 0;
}
EXPORT hipError_t hipDeviceSynchronize() { return hipSuccess; }  // the other device's
EXPORT hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
EXPORT hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
EXPORT hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return hipSuccess; }
}

namespace tk {
size_t eig_scratch_doubles(int) { return 64; }
int error_metrics_blocks(int64_t) { return 1; }
size_t qr_workspace_doubles(const QrPlan&) { return 0; }
size_t qr_workspace_bound_doubles(int) { return 0; }
QrPlan plan_qr(const ModeView&) { return {}; }
GramPlan plan_gram(const ModeView&, int, int) { return {}; }
int launch_tsqr(const void*, int, const ModeView&, const QrPlan&, double*, double*, double*, hipStream_t) { return TK_OK; }
int launch_jw(const double*, int, double*, hipStream_t) { return TK_OK; }
int launch_jw_extract(const double*, int, int, const int64_t*, double*, hipStream_t) { return TK_OK; }
int launch_error_metrics(const void*, const void*, int, int64_t, double*, int, double*, hipStream_t) { return TK_OK; }
int launch_gram(const void*, int, const ModeView&, int, double*, double*, void*, size_t, hipStream_t, double*, const hipEvent_t*) { return TK_OK; }
int launch_ttm(const void*, int, const ModeView&, const double*, int64_t, int64_t, int, int, void*, hipStream_t) {
    return ++ttms == fail_ttm ? fail(TK_ERR_HIP, "ttm") : TK_OK;
}
int launch_eig_finish(const EigArgs&, int, hipStream_t) { return TK_OK; }
int launch_eig(const EigArgs& a, hipStream_t st) {
    todo[st].push_back([a] {
        *a.rank_out = 2;
        if (!a.host) return;
        memcpy(a.host, a.host_scal, kHostScalars * sizeof(double));
        memcpy(a.host + kHostScalars, &a.host_seq, sizeof a.host_seq);
    });
    return ++eigs == fail_eig ? fail(TK_ERR_HIP, "eig") : TK_OK;
}
}  // namespace tk

static int call(hipStream_t st, bool fixed) {
    static double core[64], u[3][16];
    alignas(256) static char ws[1 << 16];
    tk_shape x{};
    x.ndim = 3;
    x.dtype = TK_F64;
    for (int k = 0; k < 3; ++k) x.dims[k] = 4;
    const int64_t ranks[3] = {2, 2, 2};
    tk_options o{};
    o.eps = 1e-3;
    o.fixed_ranks = fixed ? ranks : nullptr;
    tk_tucker out{};
    out.core_dev = core;
    out.core_capacity = 64;
    for (int k = 0; k < 3; ++k) out.factors_dev[k] = u[k];
    memset(ws, 0, sizeof ws);
    eigs = ttms = 0;
    const int rc = sthosvd_compress(&x, core, &o, &out, ws, sizeof ws, st);
    if (rc == TK_OK)
        for (int k = 0; k < 3; ++k)
            if (out.ranks[k] != 2) return printf("rank %d\n", (int)out.ranks[k]), 1;
    return rc;
}

#define CHECK(c) \
    do { \
        if (!(c)) return printf("line %d: %s\n", __LINE__, #c), 1; \
    } while (0)
"""

MAIN_PENDING = r"""
int main() {
    hipStream_t a = (hipStream_t)1, b = (hipStream_t)2;
    CHECK(call(a, false) == TK_OK && call(b, true) == TK_OK);
    // every launch that can fail with a publication under way
    for (int fixed = 0; fixed < 2; ++fixed)
        for (int n = 1; n <= 3; ++n) {
            fail_eig = n;
            CHECK(call(a, fixed) == TK_ERR_HIP);
            fail_eig = 0;
            if (!(fixed && n == 2)) CHECK(todo[a].empty());  // (mode 2 of 3 publishes nothing there)
            fail_ttm = n;
            CHECK(call(a, fixed) == TK_ERR_HIP);
            fail_ttm = 0;
            if (fixed && n == 3) CHECK(todo[a].empty());
            CHECK(call(b, fixed) == TK_OK);
            drain(a);
        }
    return 0;
}
"""

MAIN_YIELD = r"""
int main() {
    queries_busy = 1000;  // 2 ms apart
    CHECK(call((hipStream_t)1, false) == TK_OK);
    CHECK(yields > 0 && queries_busy == 1000);
    return 0;
}
"""


def _run(tmp_path, main):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs g++")
    src, exe = tmp_path / "host.cpp", tmp_path / "host"
    src.write_text(SOURCE + main)
    subprocess.run([cxx, "-O1", "-w", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_1510_06689_amd", "csrc"),
                    str(src), "-o", str(exe), "-lpthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_no_publication_outlives_its_call(tmp_path):
    _run(tmp_path, MAIN_PENDING)


def test_a_wait_lets_other_threads_run(tmp_path):
    """The wait for a rank spans a whole Gram: on a machine with fewer cores than
    threads it has to give its core away between looks."""
    _run(tmp_path, MAIN_YIELD)
