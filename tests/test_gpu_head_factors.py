"""Per-head score in tiles of 192 and 320 columns, whose phase ends read a row's factors from another lane: every row of a tile with
norms of its own, heads of norm zero, pools that end inside a row tile, against the CPU oracle; and the same layer in a call of its own
(one share per head), whose scores have the same bits.  Needs a real MI355X."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import synth
from tests import parity, paths
from tests.test_gpu_parity import run_gpu_match

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,T,H,P,Q,tile", [(260, 16, 3, 229, 140, (256, 192)), (130, 16, 2, 275, 300, (192, 320)), (260, 32, 1, 225, 192, (256, 192)),
                                            (130, 16, 5, 191, 257, (192, 320))])
def test_rows_with_norms_of_their_own(oracle, L, T, H, P, Q, tile):
    print(f"[gpu-case] head factors L={L} T={T} H={H} P={P} Q={Q}", flush=True)
    w = synth.scaled(synth.WORKLOADS[2], name="factors", L=L, P=P, Q=Q, T=T, H=H, mode=1, dtype="bf16" if Q % 2 else "f16",
                     planted_frac=0.3, R=1, E=P + Q, seed=9300 + P)
    pr = synth.make_problem(w, "cuda:0")
    scale = torch.linspace(0.25, 4.0, P, device="cuda:0").reshape(1, P, 1, 1, 1)     # a factor that lands on the wrong row shows
    pr["kp"].copy_(pr["kp"] * scale)
    pr["vp"].copy_(pr["vp"] * scale.flip(1))
    pr["kp"][:, 37, :, 0] = 0
    pr["vp"][:, 90, :, H - 1] = 0
    pr["kq"][:, 5, :, 0] = 0
    paths.assert_tiles(lambda: run_gpu_match(pr, w, pr["live"]), (*tile, 1))
    g, _ = run_gpu_match(pr, w, pr["live"])
    some = slice(0, 2)
    orc = oracle.match(1 if w.dtype == "bf16" else 0, 1, *(synth.bits(pr[k][some].contiguous()) for k in ("kq", "vq", "kp", "vp")),
                       pr["live"][some].cpu().numpy(), w.tau, want_scores=True)
    head = {k: v[some] for k, v in g.items()}
    parity.check_match(head, orc, w.tau, parity.score_lookup(orc["scores"], head["best_idx"]))
    for l in (0, L - 1):
        one = {k: pr[k][l:l + 1].contiguous() for k in ("kq", "vq", "kp", "vp", "live")}
        alone, _ = run_gpu_match(one, w, one["live"])
        for k in ("best_idx", "best_score", "match_idx", "second_score"):
            assert np.array_equal(alone[k][0], g[k][l]), (l, k)
