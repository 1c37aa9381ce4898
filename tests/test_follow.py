"""The host loop that keeps a solve's iterations enqueued (follow in dpcg_internal.h), on the
CPU: a small program compiles the loop itself against a stand-in for the stream's query, which
plays the device.  The device runs nothing until the host asks whether the stream is idle, then
everything enqueued at once, and answers "idle": what a host thread sees that loses its core
between reading the posted words and the query's answer.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>

#include "dpcg_internal.h"

using namespace dpcg;

namespace {
constexpr int kMax = 4;
uint64_t words[kMax];
int needed[kMax];      // iterations after which a system has converged
int count, queued, ran, stalls, error_at, posts;

// one iteration: its SpMV posts what it finds, the flag after `ran` iterations
void device_step() {
    for (int i = 0; i < count && posts; ++i)
        words[i] = (uint64_t)(ran >= needed[i] ? kConverged : kRunning) << 32 | (uint32_t)(ran + 1);
    ++ran;
}
}  // namespace

extern "C" hipError_t hipStreamQuery(hipStream_t) {
    if (++stalls == error_at) return hipErrorUnknown;
    while (ran < queued) device_step();
    return hipSuccess;
}

int main(int argc, char **argv) {
    // max_iter check_every error_at fail_at posts needed...
    const int max_iter = atoi(argv[1]), check_every = atoi(argv[2]);
    error_at = atoi(argv[3]);
    const int fail_at = atoi(argv[4]);
    posts = atoi(argv[5]);
    count = argc - 6;
    uint64_t *progress[kMax];
    for (int i = 0; i < count; ++i) {
        needed[i] = atoi(argv[6 + i]);
        progress[i] = &words[i];
    }
    int most = 0;
    const int32_t got = follow(nullptr, progress, count, max_iter, check_every, [&](int32_t i) -> int {
        if (i == fail_at) return DPCG_EINVAL;
        if (i != queued) exit(3);
        ++queued;
        if (queued - ran > most) most = queued - ran;
        return DPCG_OK;
    });
    int running = 0;
    for (int i = 0; i < count; ++i) running += (int32_t)(words[i] >> 32) == kRunning;
    printf("%d %d %d %d\n", (int)got, queued, running, most);
    return 0;
}
"""


@pytest.fixture(scope="module")
def follow(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("follow")
    src, exe = d / "follow.cpp", str(d / "follow")
    src.write_text(PROGRAM)
    subprocess.check_call([HIPCC, "-O1", "-std=c++17", "-x", "hip", "--offload-host-only", "-I",
                           os.path.join(ROOT, "paper_2111_09294_amd", "csrc"), str(src), "-o", exe])

    def run(needed, max_iter=1000, check_every=16, error_at=0, fail_at=-1, posts=1):
        args = [max_iter, check_every, error_at, fail_at, posts] + list(needed)
        out = subprocess.run([exe] + [str(a) for a in args], capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, out
        return [int(v) for v in out.stdout.split()]

    return run


@pytest.mark.parametrize("check_every", [1, 2, 3, 16])
@pytest.mark.parametrize("needed", [[1], [2], [40], [7, 0, 25], [5, 5, 5, 6]])
def test_a_stalled_host_goes_on_until_every_system_is_done(follow, needed, check_every):
    """An idle stream alone does not end the solve: the loop goes on while a system runs, at
    most min(check_every, 3) iterations ahead of the device, and stops within that many of the
    end (the iteration after the last one is what tells)."""
    ahead = min(check_every, 3)
    got, queued, running, most = follow(needed, check_every=check_every)
    assert running == 0 and got == queued and most <= ahead
    assert max(needed) < got <= max(needed) + ahead


@pytest.mark.parametrize("check_every", [1, 3])
def test_the_cap_and_words_that_never_move(follow, check_every):
    assert follow([100], max_iter=8, check_every=check_every)[:3] == [8, 8, 1]
    assert follow([100], max_iter=0, check_every=check_every)[:3] == [0, 0, 1]
    assert follow([2], max_iter=8, check_every=check_every, posts=0)[:3] == [8, 8, 1]


def test_errors_end_the_loop(follow):
    assert follow([100], error_at=2)[0] == -6       # DPCG_EHIP from the stream
    assert follow([100], fail_at=5)[0] == -1        # the enqueue's own status
