"""The multi-RHS workspace when an allocation fails, on the CPU: a small program compiles
batch.hip and devmem.cpp for the host alone, with stand-ins for the HIP runtime calls they make
(device memory is host memory, kernels do nothing, the n-th allocation fails)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include "batch.hip"
#include "devmem.cpp"

#include <cstdio>
#include <cstdlib>
#include <set>

namespace {
int calls, fail_at;
hipError_t last = hipSuccess;
std::set<void *> live;
hipError_t give(void **p, size_t bytes) {
    if (++calls == fail_at) return last = hipErrorOutOfMemory;
    live.insert(*p = calloc(1, bytes));
    return hipSuccess;
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void **p, size_t bytes) { return give(p, bytes); }
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned) { return give(p, bytes); }
hipError_t hipFree(void *p) { live.erase(p); free(p); return hipSuccess; }
hipError_t hipHostFree(void *p) { live.erase(p); free(p); return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = last; last = hipSuccess; return e; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *, dim3 *, size_t *, hipStream_t *) { return hipSuccess; }
void **__hipRegisterFatBinary(const void *) { static void *h; return &h; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, void *, void *, dim3 *, dim3 *,
                           int *) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
void dpcg_default_options(dpcg_options *) {}
}

int main(int argc, char **argv) {
    // 4 block rows, two vectors of one entry each, (KZ)^T of one triplet each
    int32_t zt_ptr[] = {0, 1, 2}, zt_idx[] = {0, 3}, kzt_ptr[] = {0, 3, 6}, kzt_idx[] = {0, 1, 2, 3, 4, 5};
    double zt_val[] = {1.0, 1.0};
    dpcg_ctx c;
    c.n = 12;
    c.nb = 4;
    c.k = 2;
    c.bjb_ntiles = 1;
    c.zt_ptr = zt_ptr;
    c.zt_idx = zt_idx;
    c.zt_val = zt_val;
    c.kzt_ptr = kzt_ptr;
    c.kzt_idx = kzt_idx;
    fail_at = atoi(argv[1]);
    const int first = dpcg::ensure_ws(&c);
    const bool made = c.bws != nullptr;
    const size_t held = c.allocations.size();
    const long bytes = (long)c.device_bytes;
    const int left = (int)last;
    fail_at = 0;
    const int second = dpcg::ensure_ws(&c);
    const bool whole = c.bws && c.bws->seg_part && c.bws->seg && c.bws->snap && c.bws->part3;
    printf("%d %d %zu %ld %d %d %d %d\n", first, made, held, bytes, left, second, whole, calls);
    return 0;
}
"""


@pytest.fixture(scope="module")
def workspace(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("workspace")
    src, exe = d / "workspace.cpp", str(d / "workspace")
    src.write_text(PROGRAM)
    subprocess.check_call([HIPCC, "-O0", "-std=c++17", "-x", "hip", "--offload-host-only",
                           "-Wl,--unresolved-symbols=ignore-all", "-I",  # there is no device code to embed
                           os.path.join(ROOT, "paper_2111_09294_amd", "csrc"), str(src), "-o", exe])

    def run(fail_at):
        out = subprocess.run([exe, str(fail_at)], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, (fail_at, out)
        return [int(v) for v in out.stdout.split()]

    return run


def test_a_failed_allocation_leaves_no_half_made_workspace(workspace):
    """Whichever allocation fails: the call says so, nothing of the workspace is kept and no
    error is left behind for the next launch; the next call makes it whole."""
    first, made, held, bytes_, left, second, whole, total = workspace(0)
    assert (first, made, second, whole) == (0, 1, 0, 1)
    for i in range(1, total + 1):
        assert workspace(i)[:7] == [-6, 0, 0, 0, 0, 0, 1], i
