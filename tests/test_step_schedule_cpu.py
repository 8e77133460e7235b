"""The host side of tctf_step without a GPU: which iterations are launched eagerly, when the
iteration graph is captured and replayed, and what a failing capture leaves.

A small program includes the library's host source with the HIP calls and kernel launches of
tctf_step replaced by counters, and runs a list of calls; a step "n" is tctf_step(n), "f<k>"
makes the k-th call of a capture fail from then on (1: stream, 2: begin, 3: end, 4: instantiate),
"f0" ends that.
"""
import os
import shutil
import subprocess

import pytest

from paper_2005_09838_amd import _build

CSRC = _build.CSRC

PROGRAM = r'''
#include <hip/hip_runtime.h>
#define hipStreamCreateWithFlags f_stream
#define hipStreamBeginCapture f_begin
#define hipStreamEndCapture f_end
#define hipGraphInstantiate f_inst
#define hipGraphLaunch f_launch
#define hipGetLastError f_last
#define hipStreamDestroy f_sdel
#define hipGraphDestroy f_gdel
static int fail_at = 0, ncap = 0, nrep = 0, neager = 0;
static bool capturing = false;
static hipError_t pending = hipSuccess;   // what hipGetLastError reports
static hipError_t ret(int k) { return fail_at == k ? (pending = hipErrorUnknown) : hipSuccess; }
static hipError_t f_stream(hipStream_t* s, unsigned) { *s = (hipStream_t)8; return ret(1); }
static hipError_t f_begin(hipStream_t, hipStreamCaptureMode) { const hipError_t e = ret(2); capturing = e == hipSuccess; return e; }
static hipError_t f_end(hipStream_t, hipGraph_t* g) { capturing = false; *g = fail_at == 3 ? nullptr : (hipGraph_t)8; return ret(3); }
static hipError_t f_inst(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) { if (fail_at != 4) { *x = (hipGraphExec_t)8; ++ncap; } return ret(4); }
static hipError_t f_launch(hipGraphExec_t, hipStream_t) { ++nrep; return hipSuccess; }
static hipError_t f_last() { const hipError_t e = pending; pending = hipSuccess; return e; }
static hipError_t f_sdel(hipStream_t) { return hipSuccess; }
static hipError_t f_gdel(hipGraph_t) { return hipSuccess; }
#include "api.cpp"
namespace tctf {
void launch_agemm(const Plan&, int, int, int) { if (!capturing) ++neager; }   // one per iteration
void launch_hsolve(const Plan&) {}
void launch_bgemm(const Plan&) {}
void launch_ystep(const Plan&, int) {}
void launch_zgemm(const Plan&, int) {}
void launch_slice(const Plan&, int, float*, float*, int) {}
bool slice_hosts_pinvy(const Plan&) { return true; }
}  // namespace tctf
int main(int argc, char** argv) {
  tctf_ctx c{};
  for (int a = 1; a < argc; ++a) {
    if (argv[a][0] == 'f') {
      fail_at = atoi(argv[a] + 1);
      continue;
    }
    const int s = (int)tctf_step(&c, atoi(argv[a]));
    printf("%d %d %d %d %lld\n", s, ncap, nrep, neager, (long long)c.iters);
  }
}
'''


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    if not shutil.which(_build.hipcc()):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("step")
    (d / "step.cpp").write_text(PROGRAM)
    exe = d / "step"
    subprocess.run([_build.hipcc(), "--offload-host-only", "-O0", "-std=c++17", "-w", "-x", "hip", "-I", CSRC,
                    str(d / "step.cpp"), "-o", str(exe), "-Wl,--unresolved-symbols=ignore-all"], check=True)
    return str(exe)


def _run(program, *calls):
    """Per call (status, graphs captured, replays, eager iterations, iterations counted), totals so far."""
    out = subprocess.run([program, *map(str, calls)], check=True, capture_output=True, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


@pytest.mark.parametrize("calls,want", [
    ([3, 1, 9], [(0, 0, 0, 3, 3), (0, 0, 0, 4, 4), (0, 0, 0, 13, 13)]),   # less than a block: no graph
    ([10], [(0, 0, 0, 10, 10)]),                                          # one block: nothing left to replay
    ([19], [(0, 0, 0, 19, 19)]),
    ([20], [(0, 1, 1, 10, 20)]),
    ([33], [(0, 1, 2, 13, 33)]),
    ([10, 10, 10], [(0, 0, 0, 10, 10), (0, 1, 0, 20, 20), (0, 1, 1, 20, 30)]),   # calls of a block each
    ([5, 20, 20], [(0, 0, 0, 5, 5), (0, 1, 1, 15, 25), (0, 1, 3, 15, 45)]),
])
def test_blocks_and_replays(program, calls, want):
    assert _run(program, *calls) == want


@pytest.mark.parametrize("kind", [1, 2, 3, 4])
def test_a_failed_capture_loses_no_iteration(program, kind):
    """Every iteration of the call runs, eagerly, and is counted; no error is left for the next call."""
    got = _run(program, f"f{kind}", 33, 20, "f0", 20)
    assert got[0] == (0, 0, 0, 33, 33)
    assert got[1] == (0, 0, 0, 53, 53)
    assert got[2] == (0, 0, 0, 73, 73)   # the context does not try again
