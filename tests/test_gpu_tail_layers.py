"""Searches in whole tiles that give their last layers to a launch of shares: one to 49 layers of them, two to 32 shares per
pair, every shape of whole tiles in front, against the CPU oracle; and the same calls in a workspace with no room for that."""
import numpy as np
import pytest

from paper_2507_21433_amd import synth
from tests import parity, paths
from tests.test_gpu_parity import run_gpu_match
from tests.test_workspace import guarded, lib, search  # noqa: F401

pytestmark = pytest.mark.gpu


# (mode, layers, heads, pool, queries, whole tiles, columns of a share)
CASES = [(0, 129, 4, 257, 129, (256, 192), 192), (0, 137, 4, 257, 140, (256, 192), 192), (0, 161, 4, 257, 129, (256, 192), 192),
         (0, 129, 4, 257, 193, (192, 320), 256), (1, 129, 4, 257, 129, (256, 192), 192), (1, 129, 5, 257, 193, (256, 256), 256),
         (1, 129, 4, 257, 257, (192, 320), 192)]


@pytest.mark.parametrize("mode,L,H,P,Q,tile,columns", CASES)
def test_last_layers_in_shares(oracle, lib, mode, L, H, P, Q, tile, columns):  # noqa: F811
    print(f"[gpu-case] tail mode {mode} L={L} H={H} P={P} Q={Q}", flush=True)
    w = synth.scaled(synth.WORKLOADS[2], name="tail", L=L, P=P, Q=Q, T=16, H=H, mode=mode, dtype="bf16" if L == 137 else "f16",
                     planted_frac=0.3, R=1, E=P + Q, seed=8600 + L)
    pr = synth.make_problem(w, "cuda:0")
    paths.assert_tiles(lambda: run_gpu_match(pr, w, pr["live"]), (*tile, mode), (256, columns, 3 + mode))
    orc = oracle.match(1 if L == 137 else 0, mode, *(synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")), pr["live"].cpu().numpy(), w.tau,
                       want_scores=True)
    floor, full = paths.needed(lib, mode, L, 16, H, P, Q), paths.size(lib, mode, L, 16, H, P, Q)
    assert floor < full
    got = {}
    for nbytes in (floor, full):
        mem, ws = guarded(nbytes)
        got[nbytes] = search(pr, w, ws)
        assert (mem[nbytes:] == 0xA5).all(), "written past the workspace"
        parity.check_match(got[nbytes], orc, w.tau, parity.score_lookup(orc["scores"], got[nbytes]["best_idx"]))
    if mode == 1:   # scores on a grid, the same on every plan
        for k in got[full]:
            assert np.array_equal(got[floor][k], got[full][k]), k
