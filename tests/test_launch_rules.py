"""The host's launch rules (iod_plan.h), compiled into a small program: the
scratch and the checkpoints of the refinement under any mix of evaluation
lengths and any amount of memory, and the lanes per particle of one problem."""
import os
import shutil
import subprocess

import pytest

from paper_2207_13175_amd import build as B

PROGRAM = r"""
#include "iod_plan.h"
#include <cstdio>
#include <cstdlib>
using namespace iodk;
static int64_t allocations = 0;
void *operator new(size_t n)
{
    ++allocations;
    return malloc(n);
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
int main(int argc, char **argv)
{
    if (argc == 2) {
        // lanes SIMDS: those of one problem by itself, as a batch of it has them,
        // and the allocations of the first
        const int simds = atoi(argv[1]);
        for (int64_t m = 1; m < 40 * 64 * simds; m += 1 + m / 7) {
            const Load one = load_of(m, 500);
            allocations = 0;
            const int lanes = split_lanes(&one, 1, simds);
            const int64_t n = allocations;
            SplitLoad L;
            L.add(m, 500);
            if (L.lanes(simds) != lanes || n) return 1;
            printf("%d ", lanes);
        }
        printf("\n");
        return 0;
    }
    // scratch ROWS ROW_BYTES FREE_BYTES STEPS...: what the refinement takes when
    // FREE_BYTES are to be had, and every size it asked for
    const int64_t rows = atoll(argv[1]), bytes = atoll(argv[2]), have = atoll(argv[3]);
    PipePlan plan;
    for (int i = 4; i < argc; ++i) plan.add(16, atoll(argv[i]));
    plan.decide(1024);
    const bool ok = plan.trial_scratch(rows, bytes, [&](int64_t n) {
        printf("%lld ", (long long)n);
        return n * bytes <= have;
    });
    printf("| %d %d %d\n", (int)ok, (int)plan.ckpt, plan.seg);
    return 0;
}
"""


@pytest.fixture(scope="module")
def scratch(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("rules")
    (d / "main.cpp").write_text(PROGRAM)
    rocm = os.path.dirname(os.path.dirname(os.path.realpath(B.hipcc())))
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", B.CSRC,
                    "-isystem", os.path.join(rocm, "include"), "-o", str(d / "main"), str(d / "main.cpp")],
                   check=True)

    def run(steps, problems=0, have=0):
        """(rows asked for, fitted, checkpoints, segment, rows of the adjoint, bytes of a row)"""
        if not problems:   # lanes, steps SIMDs
            return subprocess.run([str(d / "main"), str(steps)], check=True, capture_output=True,
                                  text=True).stdout.split()
        row = 6 * 8 * 64 * problems
        adj = max((s + 63) // 64 + 64 for s in steps)
        out = subprocess.run([str(d / "main"), str(adj), str(row), str(have), *map(str, steps)],
                             check=True, capture_output=True, text=True).stdout
        asked, got = out.split("|")
        ok, ckpt, seg = map(int, got.split())
        return [int(v) for v in asked.split()], bool(ok), bool(ckpt), seg, adj, row
    return run


@pytest.mark.parametrize("steps", [(1,), (500,), (1377,), (2472,), (2473,), (4033,), (4096,), (4097,),
                                   (2000, 4097), (1377, 5000), (8, 4096), (0, 20000)])
@pytest.mark.parametrize("problems", [1, 384, 2048, 4096, 100000])
def test_refinement_takes_whatever_memory_there_is(scratch, steps, problems):
    ample = 1 << 60
    asked, ok, ckpt, seg, adj, row = scratch(steps, problems, ample)
    assert ok and ckpt == (max(steps) <= 4096) and seg in (8, 16, 32) and len(asked) == 1
    need = -(-max(steps) // seg) + 1
    assert asked[0] == (max(adj, need) if ckpt else adj)
    if ckpt:   # the shortest segments within the limit
        assert seg == 32 or need * row <= 2 << 30
        assert seg == 8 or (-(-max(steps) // (seg // 2)) + 1) * row > 2 << 30
    # with less, longer segments, or none; what the adjoint needs by itself is enough
    tried, ok, ckpt, seg, _, _ = scratch(steps, problems, max(asked[0] - 1, adj) * row)
    assert ok and tried[0] == asked[0] and tried[-1] <= max(asked[0] - 1, adj) and seg in (8, 16, 32)
    tried, ok, ckpt, seg, _, _ = scratch(steps, problems, adj * row)
    assert ok and tried[-1] == adj and seg in (8, 16, 32)
    tried, ok, ckpt, seg, _, _ = scratch(steps, problems, adj * row - 1)
    assert not ok and not ckpt and tried[-1] == adj


@pytest.mark.parametrize("simds", [4, 128, 1024])
def test_lanes_of_one_problem_need_no_memory(scratch, simds):
    """Fitness, propagation, prediction and swarm steps of a handle ask for their
    lanes inside C entries that allocate nothing else, where an exception could
    not be caught: the same answer as a batch's, without an allocation."""
    lanes = scratch(simds)
    assert lanes[0] == "4" and lanes[-1] == "1" and set(lanes) == {"1", "2", "4"}
