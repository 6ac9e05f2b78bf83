"""The stop rules of the mixed COCG on the host: cocg.h is compiled by g++ and
fed residual sequences (no GPU).

The rules stand twice, with branches for the kernels of each phase
(``step_beta``) and without for the fused and the one-launch step
(``fused_scalars``): both have to decide alike at every iteration. A column that
converges is left alone, one that wanders restarts.
"""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm/include"

HARNESS = r"""
#include <math.h>
#include <algorithm>
#include <hip/hip_runtime.h>
#ifndef __forceinline__
#define __forceinline__ inline
#endif
using std::isfinite;
using std::max;
#include "cocg.h"
using namespace petgem;

// One inner solve over r2[0 .. n - 1] (|r|^2 after each iteration, 1 before the
// first), ended by the rules or the sequence. out per iteration: active,
// restarts, stalled, breakdown, kin, k_best, k_mark; returns the iterations.
extern "C" int run(int form, int n, const double* r2, double inner_rtol, double inner_tol, int k_prev, int* out) {
    ColState S{};
    S.rn2 = S.rn2_best = S.tmark = S.rn2_0 = 1.0;
    S.inner_rtol = inner_rtol;
    S.inner_tol2 = inner_tol * inner_tol;
    S.active = 1;
    S.outer = 1;
    S.k_prev = k_prev;
    S.rho = make_double2(0.3, 0.1);
    const double2 pq = make_double2(1.0, 0.5), some = make_double2(0.2, -0.1);
    auto put = [&](int k) {
        const int v[7] = {S.active, S.restarts, S.stalled, S.breakdown, S.kin, S.k_best, S.k_mark};
        for (int i = 0; i < 7; ++i) out[7 * k + i] = v[i];
    };
    int k = 0;
    if (form == 0) {
        for (; k < n && S.active; ++k) {
            step_beta(S, make_double2(0.3, 0.1), r2[k]);
            put(k);
        }
        return k;
    }
    double2 t[5] = {pq, some, some, make_double2(0.0, 0.0), make_double2(0.0, 0.0)};
    fused_scalars(S, t);   // the first alpha and beta
    for (; k < n && S.active; ++k) {
        t[3] = make_double2(0.3, 0.1);
        t[4] = make_double2(r2[k], 0.0);
        const int kin = S.kin;
        fused_scalars(S, t);
        const int now = S.kin;
        S.kin = kin;       // the state after iteration kin: the next one is counted already
        put(k);
        S.kin = now;
    }
    return k;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    if not os.path.exists(os.path.join(ROCM, "hip", "hip_runtime.h")):
        pytest.skip("no HIP headers")
    d = tmp_path_factory.mktemp("rules")
    src, so = d / "rules.cpp", d / "rules.so"
    src.write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-D__HIP_PLATFORM_AMD__", "-I", ROCM, "-I",
                    os.path.join(ROOT, "paper_1808_00186_amd", "csrc"), str(src), "-o", str(so)], check=True)
    lib = C.CDLL(str(so))

    def run(form, r, inner_tol=3e-5, k_prev=0, inner_rtol=3e-5):
        r2 = np.ascontiguousarray(np.asarray(r, float) ** 2)
        out = np.zeros((len(r2), 7), np.int32)
        k = lib.run(form, len(r2), r2.ctypes.data_as(C.c_void_p), C.c_double(inner_rtol), C.c_double(inner_tol),
                    k_prev, out.ctypes.data_as(C.c_void_p))
        return out[:k]
    return run


def _walk(rng, n):
    """|r| that falls, stays and jumps as COCG's does: a random walk of its
    logarithm with a drift that changes now and then."""
    step = rng.normal(0.0, rng.choice([0.02, 0.2, 0.6]), n)
    k = 0
    while k < n:
        m = int(rng.integers(20, 900))
        step[k:k + m] += rng.choice([-0.05, -0.01, -0.002, 0.0, 0.0005])
        k += m
    level = np.cumsum(step) - rng.choice([0.0, 3.0])
    return np.exp(np.clip(level, -14.0, 5.0))


def test_both_statements_of_the_rules_decide_alike(rules):
    rng = np.random.default_rng(3)
    ended = restarted = 0
    for _ in range(400):
        r = _walk(rng, int(rng.integers(5, 9000)))
        if rng.random() < 0.1:
            r[rng.integers(len(r))] = rng.choice([np.nan, np.inf])
        tol, prev = float(rng.choice([3e-5, 1e-2, 0.5])), int(rng.choice([0, 3, 150, 400, 1500]))
        a, b = rules(0, r, tol, prev), rules(1, r, tol, prev)
        assert a.shape == b.shape and np.array_equal(a[:, :6], b[:, :6])
        on = a[:, 0] == 1     # the mark of a column that has ended is not used again
        assert np.array_equal(a[on, 6], b[on, 6])
        ended += a[-1, 0] == 0
        restarted += a[-1, 1] > 0
    assert ended > 100 and restarted > 20


# (iterations to the quick halvings, level, plateau, iterations of the step before)
# of columns that converged: a mirror of the recurrence on 10,836 to 80,000 unknowns at
# 0.25 and 0.5 Hz, first and later refinement steps
@pytest.mark.parametrize("early,level,plateau,prev", [(3, 0.2, 300, 1383), (48, 0.25, 418, 1551), (2, 0.4, 342, 1596),
                                                      (1, 0.45, 313, 659), (163, 0.05, 230, 0), (450, 0.06, 465, 1637)])
@pytest.mark.parametrize("form", [0, 1])
def test_a_converging_column_is_not_restarted(rules, form, early, level, plateau, prev):
    r = np.concatenate([np.geomspace(0.9, level, early), np.full(plateau, level) * (1.0 + 0.3 * np.sin(np.arange(plateau))),
                        np.geomspace(level, 1e-5, 600)])
    out = rules(form, r, 3e-5, prev)
    assert out[-1, 0] == 0 and out[:, 1].max() == 0


@pytest.mark.parametrize("form", [0, 1])
def test_a_wandering_column_restarts(rules, form):
    """|r| between 0.3 and 3 with a best that creeps down, after a step of 150 iterations."""
    k = np.arange(4000)
    r = 1.0 + 0.6 * np.sin(0.7 * k) - 2e-5 * k
    out = rules(form, r, 3e-5, 150)
    at = np.flatnonzero(np.diff(out[:, 1], prepend=0))
    assert len(at) == 4 and at[0] < 250 and np.all(np.diff(at) >= 199)   # four of them, no more
    # in the first refinement step there is no measure yet
    assert rules(form, r[:3000], 3e-5, 0)[:, 1].max() == 0
