"""Plans chosen by the time model: valid over a range of shapes, a pure
function of the product (kept plans do not outlive an override), and grouped
backward plans whose partials fit the workspace."""
import os
import random
import re
import subprocess

import pytest

from paper_2301_06813_amd import sbp

BF, F32 = sbp.SBP_BF16, sbp.SBP_F32
TILES = {(256, 256), (256, 192), (256, 128), (128, 256), (128, 128), (128, 64), (64, 128),
         (64, 64)}


def _extent(rng):
    v = round(2 ** rng.uniform(0, 13))
    return max(1, v // 64 * 64) if rng.random() < 0.5 else v


@pytest.mark.parametrize("seed", range(4))
def test_plans_are_valid_and_repeat(seed):
    rng = random.Random(seed)
    for _ in range(100):
        m, n, k = (_extent(rng) for _ in range(3))
        for op in range(3):
            for din, dout in ((BF, BF), (BF, F32), (F32, F32)):
                tm, tn, splits, kernel = p = sbp.sbp_plan(op, m, n, k, din, dout)
                assert (tm, tn) in TILES and 1 <= splits <= 32
                assert kernel == sbp.KERNEL_F32 if din == F32 else kernel != sbp.KERNEL_F32
                block = 32 if din == F32 else 64
                assert splits == 1 or (splits - 1) * block < k
                ld = -(-n // 4) * 4
                assert splits == 1 or 4 * splits * m * ld <= sbp.SBP_WORKSPACE_BYTES
                assert sbp.sbp_plan(op, m, n, k, din, dout) == p


@pytest.mark.parametrize("seed", range(4))
def test_backward_pair_plans_fit_and_follow_overrides(seed):
    rng = random.Random(100 + seed)
    for _ in range(30):
        M, K, N = (_extent(rng) for _ in range(3))
        fd, fw = rng.choice(((BF, F32), (F32, BF), (F32, F32)))
        args = (M, K, N, fd, K, N, M, fw)
        grouped, tm, tn, sd, sw = p = sbp.sbp_plan_bwd(*args)
        assert (tm, tn) in TILES
        if grouped:
            part = [4 * s * r * (-(-c // 4) * 4) if s > 1 else 0
                    for s, r, c in ((sd, M, K), (sw, K, N))]
            assert sum(part) <= sbp.SBP_WORKSPACE_BYTES
        try:
            sbp.sbp_set_plan_override(64, 64, 1, 1)
            sbp.sbp_set_bwd_override(2, 1)
            q = sbp.sbp_plan_bwd(*args)
            # tight rows of K and N elements: whole 16-byte blocks can be grouped
            assert bool(q[0]) == (K % 8 == 0 and N % 8 == 0)
            assert not q[0] or q[1:] == (64, 64, 1, 1)
        finally:
            sbp.sbp_set_plan_override(0, 0, 1)
        assert sbp.sbp_plan_bwd(*args) == p


def test_attention_tests_cover_the_model_instances():
    # the GPU tests' list is the planner's
    from paper_2301_06813_amd import build
    import test_gpu_attn_group
    src = open(os.path.join(build.CSRC, "plan.cpp")).read()
    rows = src.split("kPipe[] = {")[1].split("};")[0]
    listed = {tuple(map(int, m)) for m in re.findall(r"\{(\d+), (\d+), (\d+), \d+, \{", rows)}
    assert len(listed) == 11 and listed == set(test_gpu_attn_group.INSTANCES)


def test_planning_without_memory_does_not_throw(tmp_path):
    # kept plans are only kept where there is memory: no exception leaves a C entry
    src = tmp_path / "nomem.cpp"
    src.write_text(r"""
#include <dlfcn.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <new>
static bool fail = false;
void *operator new(size_t n) {
    if (fail) throw std::bad_alloc();
    void *p = malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
int main(int, char **argv) {
    void *lib = dlopen(argv[1], RTLD_NOW);
    if (!lib) return 2;
    typedef int (*Plan)(int, int64_t, int64_t, int64_t, int32_t, int32_t, int32_t *, int32_t *,
                        int32_t *, int32_t *);
    typedef int (*Pair)(int64_t, int64_t, int64_t, int32_t, int64_t, int64_t, int64_t, int32_t,
                        int32_t *, int32_t *, int32_t *, int32_t *, int32_t *);
    Plan plan = (Plan)dlsym(lib, "sbp_plan");
    Pair pair = (Pair)dlsym(lib, "sbp_plan_bwd");
    int32_t a[2][4], b[2][5];
    for (int i = 0; i < 2; ++i) {
        fail = i == 0;
        int rc = plan(0, 777, 555, 333, 0, 0, a[i], a[i] + 1, a[i] + 2, a[i] + 3);
        rc |= pair(512, 640, 768, 1, 640, 768, 512, 1, b[i], b[i] + 1, b[i] + 2, b[i] + 3,
                   b[i] + 4);
        fail = false;
        if (rc) return 3;
    }
    for (int i = 0; i < 5; ++i)
        if (b[0][i] != b[1][i] || (i < 4 && a[0][i] != a[1][i])) return 4;
    return 0;
}
""")
    exe = str(tmp_path / "nomem")
    subprocess.run(["g++", "-O1", "-rdynamic", "-o", exe, str(src), "-ldl"], check=True)
    assert subprocess.run([exe, sbp.LIB_PATH]).returncode == 0


def test_forked_child_forgets_the_parents_stream_lookup():
    kept = sbp._raw_stream
    try:
        sbp._raw_stream = (None, None)
        pid = os.fork()
        if pid == 0:
            os._exit(0 if sbp._raw_stream is None else 1)
        assert os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0
        assert sbp._raw_stream == (None, None)
    finally:
        sbp._raw_stream = kept
