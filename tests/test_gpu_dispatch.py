"""Shapes at the edges of the library's dispatch rules, every entry point against the CPU oracle on the same inputs:
each list names the rule whose two sides it stands on.  Needs a real MI355X."""
import pytest

from tests.test_gpu_sweep import run_shape

pytestmark = pytest.mark.gpu

# Parts merged per query: the few-tiles path makes one per 32 pool rows; four parts per thread, 1 to 64 threads per query.
PARTS = [(1, 1), (33, 3), (128, 5), (129, 40), (257, 64), (2048, 3), (2049, 65), (8193, 2)]


@pytest.mark.parametrize("P,Q", PARTS)
def test_merge_parts(oracle, P, Q):
    run_shape(oracle, dict(L=2, P=P, Q=Q, T=16, H=1, mode=0, dtype="f16", planted_frac=0.3, seed=7100 + P), f"parts{P}x{Q}", P)
