"""The FLOP bounds of the benchmark's solver roofline against an iteration's parts
as they run: n assemblies and n - 1 steps at the least, n + 1 and n at the most, no
trial cost of its own (host only)."""
import importlib.util
import os

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.parametrize("form", [0, 1])
def test_solver_flops_bound_what_an_iteration_runs(form):
    from paper_2301_06399_amd import mpt
    spec = importlib.util.spec_from_file_location("bench_mod", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    tab = mpt.flops_table(form)
    for n in range(1, 6):
        for code in range(0, 4 ** n, 1 + 4 ** n // 40):
            t = {k: int(v[code]) for k, v in tab[n].items()}
            order, codes = np.array([n]), np.array([code])

            def f(it):
                return bench.solver_flops(tab, order, codes, np.array([it]), form)
            assert f(0) == (0, 0)
            assert f(1)[0] == t["assembly"]
            step = f(2)[0] - 2 * t["assembly"]
            # a step is positive, at least the multiplications of the solve, and
            # with an assembly less than the whole iteration by the trial cost
            assert 0 < 2 * n <= step
            assert t["assembly"] + step <= t["lm"] - t["residual"]
            for it in (2, 7, 100):
                lo, up = f(it)
                assert lo == it * t["assembly"] + (it - 1) * step
                assert up - lo == t["assembly"] + step
                assert lo < it * t["lm"]
