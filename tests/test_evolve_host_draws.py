"""The host steps' number reduction, tabu table and lazily ordered top-rank
pass against the oracle, where they change form: lengths around the largest
with a table of reciprocals (64), populations of a power of two, a tabu list
that grows many times, equal and zero fitness throughout.  Exact."""
import numpy as np
import pytest

from test_evolve_host_cpu import _compare, _configs


def _normal(n, m):
    return np.random.default_rng(n + m).standard_normal((n, m)).astype(np.float32)


@pytest.mark.parametrize("a,P,lmin,lmax,sigma,gens", [
    (_normal(70, 90), 40, 61, 70, 2, 4),                 # lengths 61 .. 70
    (_normal(40, 66), 32, 64, 66, 2, 3),                 # length = number of columns
    (_normal(60, 40), 64, 1, 6, 3, 5),
    (_normal(30, 25), 1500, 2, 5, 2, 4),                 # 6000 series listed
    (np.zeros((50, 12), np.float32), 128, 2, 6, 3, 5),   # equal fitness at each length
    (np.full((50, 12), np.nan, np.float32), 50, 3, 6, 0, 3),   # nothing counts
    (_normal(1, 9), 33, 2, 4, 0, 4),                     # one row: zero fitness
])
def test_draws_match(a, P, lmin, lmax, sigma, gens):
    cfg, op = _configs(P, lmin, lmax, (sigma, 0, True), (sigma, 0, True))
    _compare(a, 11, gens, cfg, op)
