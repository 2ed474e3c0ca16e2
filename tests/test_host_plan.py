"""The host-side rules of csrc/lbm_plan.hpp, compiled with the host compiler: the
launch plans of runs (step sums, launch counts, unknown times, least predicted time
and no allocation, since they run inside entry points that must not throw) and
the form of an initialisation."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_01081_amd", "csrc")

SOURCE = r"""
#include "lbm_plan.hpp"
#include <new>
#include <stdlib.h>
static long allocations = 0;
void* operator new(size_t n) { ++allocations; void* p = malloc(n); if (!p) abort(); return p; }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
extern "C" {
long count_allocations() { return allocations; }
int most_steps() { return lbmh::PLAN_MAX_STEPS; }
// the steps of the first `cap` launches; returns the number of launches
int64_t plan(int64_t n, int T, int one, const double* ms, int maxt, int cap, int* out) {
  const lbmh::LaunchPlan p = lbmh::plan_launches(n, T, one != 0, ms, maxt);
  for (int64_t l = 0; l < p.launches() && l < cap; ++l) out[l] = p.steps(l);
  return p.launches();
}
// the buffer after a run from buffer `cur` with a graph built from one plan
int buffer_after(int64_t n, int T, int one, const double* ms, int maxt, int cur) {
  const lbmh::LaunchPlan p = lbmh::plan_launches(n, T, one != 0, ms, maxt);
  const lbmh::RunGraph<int> g{0, p.launches()};
  return g.buffer_after(cur);
}
// the predicted time of a run's launches
double plan_ms(int64_t n, int T, int one, const double* ms, int maxt) {
  return lbmh::plan_ms(lbmh::plan_launches(n, T, one != 0, ms, maxt), ms);
}
int init_form(int nx, size_t bytes) { return lbmh::init_form(nx, bytes); }
int batch_init_nt(size_t pool, size_t full) { return lbmh::batch_init_nt(pool, full); }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, so = str(d / "plan.cpp"), str(d / "plan.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    # (the library's own definition of operator new, not another's)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-Wl,-Bsymbolic", "-I", CSRC, "-o", so, src], check=True)
    return ctypes.CDLL(so)


def _plan(lib, n, T, one, ms, maxt):
    cap = n + 1
    out = (ctypes.c_int * cap)()
    a = (ctypes.c_double * len(ms))(*ms)
    lib.plan.restype = ctypes.c_int64
    k = lib.plan(ctypes.c_int64(n), T, int(one), a, maxt, cap, out)
    return list(out[:k])


def _plain(n, T, one):
    r = n % T
    return [T] * (n // T) + ([] if r == 0 else [r] if one else [1] * r)


def test_six_sevens_and_an_eight(lib):
    # 1000 x 777: 7 steps 31 us, 8 steps 34, a single step 18.6
    ms = [0.0, 18.6, 19.5, 21.0, 23.0, 25.0, 28.0, 31.0, 34.0, 0.0, 0.0]
    # (5 + 8 + 8 + 8 of the last 29 steps take exactly as long as 7 + 7 + 7 + 8)
    got = _plan(lib, 50, 7, True, ms, 10)
    assert len(got) == 7 and sum(got) == 50
    assert sum(ms[t] for t in got) == pytest.approx(6 * 31.0 + 34.0)
    # a saving below 1% of the divided launches is not taken
    assert _plan(lib, 50, 7, True, [0.0, 2.0] + [0.0] * 5 + [31.0, 32.9, 0.0, 0.0], 10) \
        == _plain(50, 7, True)


@pytest.mark.parametrize("T", [2, 3, 4, 5, 7, 8, 10])
def test_unknown_times_leave_the_plain_division(lib, T):
    for n, one in itertools.product(range(0, 45), (True, False)):
        assert _plan(lib, n, T, one, [0.0] * 11, 10) == _plain(n, T, one)
        # the full launch's or the rest's time alone is not enough
        ms = [0.0] * 11
        ms[T] = 5.0
        assert _plan(lib, n, T, one, ms, 10) == _plain(n, T, one)


def test_plans_against_exhaustive_search(lib):
    g = np.random.default_rng(0)
    for _ in range(400):
        T, maxt = int(g.integers(2, 11)), 10
        ms = [0.0] + [float(g.uniform(3, 6) + t * g.uniform(0.5, 3)) for t in range(1, 11)]
        for t in range(1, 11):
            if g.random() < 0.2:
                ms[t] = 0.0
        n, one = int(g.integers(0, 80)), bool(g.random() < 0.7)
        got, plain = _plan(lib, n, T, one, ms, maxt), _plain(n, T, one)
        assert sum(got) == n and len(got) <= len(plain)
        if got == plain:
            chosen = None
        else:
            assert all(ms[t] > 0.0 for t in got)
            chosen = sum(ms[t] for t in got)
        r = n % T
        if r == 0 or ms[T] <= 0.0 or (ms[r] if one else ms[1]) <= 0.0:
            assert chosen is None
            continue
        # least time of K steps in at most `most` launches
        q = min(4, n // T)
        K, most = q * T + r, q + len(plain) - n // T
        best = {0: 0.0}
        least = 1e300
        for _l in range(most):
            nxt = {}
            for k, c in best.items():
                for t in range(1, maxt + 1):
                    if ms[t] > 0.0 and k + t <= K:
                        nxt[k + t] = min(nxt.get(k + t, 1e300), c + ms[t])
            best = nxt
            least = min(least, best.get(K, 1e300))
        head = (n // T - q) * ms[T]
        before = q * ms[T] + (ms[r] if one else r * ms[1])
        if least < 0.99 * before * (1 - 1e-12):
            assert chosen == pytest.approx(head + least, rel=1e-12)
        elif least > 0.99 * before * (1 + 1e-12):
            assert chosen is None


def test_plans_do_not_allocate(lib):
    lib.count_allocations.restype = ctypes.c_long
    before = lib.count_allocations()
    ms = [0.0, 18.6, 19.5, 21.0, 23.0, 25.0, 28.0, 31.0, 34.0, 37.0, 40.0]
    assert lib.most_steps() == 10
    for n in (0, 1, 9, 50, 419, 12345):
        for T in range(2, 11):
            for one in (True, False):
                _plan(lib, n, T, one, ms, 10)
    assert lib.count_allocations() == before


def test_buffer_after_a_cached_graph_is_that_of_its_own_launches(lib):
    # 9 steps with a 4-step variant: 4 + 4 + 1 before launch times are known,
    # 4 + 5 with them.  A graph of either plan decides the buffer it leaves the
    # state in, whatever plan would be made when it is launched again.
    before = [0.0] * 11
    after = [0.0, 18.0, 19.0, 20.0, 21.0, 22.0] + [0.0] * 5
    assert _plan(lib, 9, 4, True, before, 8) == [4, 4, 1]
    assert sorted(_plan(lib, 9, 4, True, after, 8)) == [4, 5]
    for cur in (0, 1):
        for ms, launches in ((before, 3), (after, 2)):
            a = (ctypes.c_double * 11)(*ms)
            assert lib.buffer_after(ctypes.c_int64(9), 4, 1, a, 8, cur) == cur ^ (launches & 1)


def test_batch_step_advances_by_its_graph():
    # the launch count after a graph launch comes from the graph, and a failed
    # autotune leaves selection and launch times (the graphs' own) as they were
    text = open(os.path.join(CSRC, "lbm_batch.hip")).read()
    step = text[text.index("lbm_status lbm_batch_step(lbm_batch* b"):
                text.index("lbm_status lbm_batch_step_eager")]
    assert "launch_plan" not in step and "buffer_after" in step
    tune = text[text.index("lbm_status lbm_batch_autotune(lbm_batch* b"):
                text.index("static lbm_status batch_moments")]
    loop = tune[tune.index("for (int v = -1"):tune.index("hipEventDestroy(e0);\n  hipEventDestroy(e1);\n  if (s ==")]
    assert "b->tb_ms" not in loop and "b->step_ms" not in loop
    assert tune.index("drop_graphs(b)") < tune.index("memcpy(b->tb_ms")


def test_init_form(lib):
    # (tiles with nontemporal stores, tiles with plain ones, consecutive nodes)
    NT, PLAIN, FLAT = 0, 1, 2

    def form(nx, ny):
        state = 20 * 4 * ny * (-(-nx // 64) * 64)  # rows padded to 64 values
        return lib.init_form(nx, ctypes.c_size_t(state))

    # rows shorter than a cache line: no nontemporal stores of parts of lines,
    # and no tiles that leave more than half of their lanes idle
    for nx in range(1, 32):
        for ny in (1, 50, 3000, 60000, 10 ** 6):
            assert form(nx, ny) == FLAT
    # up to 128 MiB of state plain, beyond nontemporal
    assert [form(32, 26214), form(32, 26215)] == [PLAIN, NT]
    assert [form(64, 64), form(1000, 777), form(2048, 1024), form(4096, 4096)] \
        == [PLAIN, PLAIN, NT, NT]


def test_batch_init_stores(lib):
    def nt(pool, full):
        return bool(lib.batch_init_nt(ctypes.c_size_t(pool), ctypes.c_size_t(full)))

    mib = 1 << 20
    assert not nt(128 * mib, 128 * mib) and nt(129 * mib, 129 * mib)
    # narrow instances alone, half of the pool, most of it wide
    assert not nt(640 * mib, 0) and not nt(640 * mib, 320 * mib) and nt(640 * mib, 321 * mib)


def test_predicted_time_is_that_of_the_launches_made(lib):
    lib.plan_ms.restype = ctypes.c_double

    def predicted(n, T, ms):
        return lib.plan_ms(ctypes.c_int64(n), T, 1, (ctypes.c_double * 11)(*ms), 10)

    # 50 steps: 7 x 7 + 1 would be 235.6, the run made is 6 x 7 + 8
    ms = [0.0, 18.6, 19.5, 21.0, 23.0, 25.0, 28.0, 31.0, 34.0, 0.0, 0.0]
    assert predicted(50, 7, ms) == pytest.approx(6 * 31.0 + 34.0)
    # runs that variants of fewer and more steps make alike cost the same: 20 steps
    # of an 8-step variant as 10 + 10
    ms = [0.0, 440.0, 450.0, 460.0, 470.0, 480.0, 490.0, 510.0, 530.0, 650.0, 690.0]
    assert predicted(20, 10, ms) == predicted(20, 8, ms) == 2 * 690.0
    for T in range(2, 11):
        for n in range(1, 60):
            steps = _plan(lib, n, T, True, ms, 10)
            assert predicted(n, T, ms) == pytest.approx(sum(ms[t] for t in steps))
    # a launch that was not timed counts as its single steps
    ms[4] = -1.0
    assert _plan(lib, 20, 8, True, ms, 10) == [8, 8, 4]
    assert predicted(20, 8, ms) == pytest.approx(2 * 530.0 + 4 * 440.0)
