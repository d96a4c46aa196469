"""Shapes at the edges of the library's dispatch rules, every entry point against the CPU oracle on the same inputs:
each list names the rule whose two sides it stands on.  Needs a real MI355X."""
import numpy as np
import pytest

from paper_2507_21433_amd import synth
from tests.test_gpu_layer_mean import run_case
from tests.test_gpu_sweep import run_shape

pytestmark = pytest.mark.gpu

# Parts merged per query: the few-tiles path makes one per 32 pool rows; four parts per thread, 1 to 64 threads per query.
PARTS = [(1, 1), (33, 3), (128, 5), (129, 40), (257, 64), (2048, 3), (2049, 65), (8193, 2)]


@pytest.mark.parametrize("P,Q", PARTS)
def test_merge_parts(oracle, P, Q):
    run_shape(oracle, dict(L=2, P=P, Q=Q, T=16, H=1, mode=0, dtype="f16", planted_frac=0.3, seed=7100 + P), f"parts{P}x{Q}", P)


# Tile width (64 columns up to 64 queries, 128 up to 128, 256 beyond) and shares per tile: per-head mode in whole tiles
# (256 tiles: one round) and with one share per head, block mode with a share count that is no power of two.
WIDTHS = [(1, 256, 64, 64, 2), (1, 256, 40, 65, 2), (1, 256, 70, 128, 1), (1, 3, 300, 64, 5), (1, 2, 257, 65, 16),
          (1, 2, 255, 128, 3), (1, 2, 300, 129, 3), (0, 24, 250, 40, 5), (0, 24, 250, 65, 5), (0, 2, 300, 128, 3), (0, 11, 513, 1, 6)]


@pytest.mark.parametrize("mode,L,P,Q,H", WIDTHS)
def test_tile_widths_and_shares(oracle, mode, L, P, Q, H):
    run_shape(oracle, dict(L=L, P=P, Q=Q, T=16, H=H, mode=mode, dtype="bf16" if Q % 2 else "f16", planted_frac=0.3, seed=7300 + P),
              f"width{mode}.{L}.{P}x{Q}", P)


# Shape of whole tiles beyond 128 queries: 256 x 192, 192 x 320 and 256 x 256 with one and more query tiles, pools that end
# on and beside an edge of a tile.
SHAPES = [(0, 260, 8, 129, 1), (0, 260, 193, 192, 1), (0, 260, 257, 193, 1), (0, 260, 192, 257, 1), (0, 260, 193, 320, 1),
          (0, 260, 31, 321, 1), (0, 260, 40, 640, 1), (0, 260, 5, 641, 1), (1, 260, 193, 160, 1), (1, 130, 191, 300, 2), (1, 260, 40, 384, 1),
          (1, 260, 20, 640, 1)]


@pytest.mark.parametrize("mode,L,P,Q,H", SHAPES)
def test_tile_shapes(oracle, mode, L, P, Q, H):
    run_shape(oracle, dict(L=L, P=P, Q=Q, T=16, H=H, mode=mode, dtype="bf16" if Q % 2 else "f16", planted_frac=0.0 if P < 64 else 0.3,
                           seed=7500 + P), f"shape{mode}.{L}.{P}x{Q}", P)


# Layer-mean search at 128 columns (running sums in registers) and at 192 (in memory), layers in groups of 2, 2 and 1: 172
# pool tiles of 5 layers; and at 192 columns with two query tiles.
@pytest.mark.parametrize("L,P,Q", [(5, 44000, 65), (5, 44000, 129), (90, 300, 257)])
def test_layer_mean_widths(oracle, L, P, Q):
    w = synth.scaled(synth.WORKLOADS[2], name=f"lm{L}.{P}x{Q}", L=L, P=P, Q=Q, T=16, H=1, planted_frac=0.3, R=1, E=P + Q, seed=7700)
    run_case(oracle, w, 0.5 * np.sqrt(w.Dh / (w.T * w.H)))


# Shares per pair added by the selection kernels: 8 at a time, then 4, then single ones, K and V layer by layer dealt to four
# threads; pool chunks of 32 rows that end inside a group of four.
@pytest.mark.parametrize("L,P,Q,H", [(1, 1, 1, 16), (1, 37, 66, 3), (1, 250, 9, 5), (3, 35, 129, 7), (9, 259, 2, 3)])
def test_share_selection(oracle, L, P, Q, H):
    for mode in (0, 1):
        run_shape(oracle, dict(L=L, P=P, Q=Q, T=16, H=H, mode=mode, dtype="f16", planted_frac=0.0 if P < 64 else 0.3, seed=7900 + P),
                  f"shares{mode}.{L}.{P}x{Q}", P)
