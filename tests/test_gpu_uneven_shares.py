"""Shares of a tile's reduction that are not alike: a tensor's steps cut into 3, 5, 6 or 7 parts of which some are a step longer,
every width of the tiles, block score and layer mean, against the CPU oracle; copies of a pool block in other tiles get the same
score and lose to the lowest index.  Needs a real MI355X."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import binding as rc
from paper_2507_21433_amd import synth
from tests import parity, paths, plans
from tests.test_gpu_layer_mean import gpu_layer_mean, shared_live
from tests.test_gpu_parity import run_gpu_match
from tests.test_workspace import guarded, search

pytestmark = pytest.mark.gpu


def uneven(mean, L, T, H, P, Q):
    """(shares per tile by the plan, columns of the tiles): a number that does not divide the steps, with room in the workspace asked for."""
    columns = 64 if Q <= 64 else 128 if Q <= 128 else 192 if Q <= 192 or 256 < Q <= 384 else 256
    n = plans.shares(mean, L, T, H, P, Q)
    assert T * H * 2 % (n // 2) != 0, "the case is about shares that are not alike"
    size = paths.mean_size(rc.lib(), L, T, H, P, Q) if mean else paths.size(rc.lib(), 0, L, T, H, P, Q)
    assert size >= plans.need(mean, n, columns, L, P, Q)
    return n, columns


@pytest.mark.parametrize("L,T,H,P,Q", [(20, 32, 8, 1226, 13), (1, 32, 5, 4179, 70), (3, 16, 5, 1300, 90), (3, 16, 5, 1300, 140),
                                       (7, 16, 5, 520, 192), (3, 16, 2, 1300, 300), (2, 16, 5, 1300, 513)])
def test_block_score(oracle, L, T, H, P, Q):
    n, columns = uneven(False, L, T, H, P, Q)
    print(f"[gpu-case] uneven shares L={L} T={T} H={H} P={P} Q={Q}: {n}", flush=True)
    w = synth.scaled(synth.WORKLOADS[2], name="uneven", L=L, P=P, Q=Q, T=T, H=H, dtype="bf16" if Q % 2 else "f16", planted_frac=0.3,
                     R=1, E=P + Q, seed=9100 + P)
    pr = synth.make_problem(w, "cuda:0")
    pr["live"][:, 7] = 1
    for kq, kp in ((pr["kq"], pr["kp"]), (pr["vq"], pr["vp"])):
        kp[:, P - 2] = kp[:, 7]              # the last tile
        kp[:, P // 2] = kp[:, 7]
        kq[:, 0] = kp[:, 7]
    pr["live"][:, P - 2] = 1
    g, _ = run_gpu_match(pr, w, pr["live"])
    paths.assert_tiles(lambda: run_gpu_match(pr, w, pr["live"]), (256, columns, 3))
    orc = oracle.match(1 if w.dtype == "bf16" else 0, 0, *(synth.bits(pr[k]) for k in ("kq", "vq", "kp", "vp")),
                       pr["live"].cpu().numpy(), w.tau, want_scores=True)
    parity.check_match(g, orc, w.tau, parity.score_lookup(orc["scores"], g["best_idx"]))
    assert (g["best_idx"][:, 0] == 7).all() and np.array_equal(g["best_score"][:, 0], g["second_score"][:, 0])


@pytest.mark.parametrize("L,T,H,P,Q", [(3, 16, 5, 1300, 140), (2, 16, 5, 1300, 513), (20, 32, 8, 1226, 13)])
def test_in_a_workspace_with_no_room_for_them(oracle, L, T, H, P, Q):
    floor, full = paths.needed(rc.lib(), 0, L, T, H, P, Q), paths.size(rc.lib(), 0, L, T, H, P, Q)
    print(f"[gpu-case] least workspace L={L} T={T} H={H} P={P} Q={Q}: {floor} of {full}", flush=True)
    assert floor < full
    w = synth.scaled(synth.WORKLOADS[2], name="uneven", L=L, P=P, Q=Q, T=T, H=H, planted_frac=0.3, R=1, E=P + Q, seed=9150 + P)
    pr = synth.make_problem(w, "cuda:0")
    orc = oracle.match(0, 0, *(synth.bits(pr[k]) for k in ("kq", "vq", "kp", "vp")), pr["live"].cpu().numpy(), w.tau, want_scores=True)
    for nbytes in (floor, (floor + full) // 32 * 16, full):
        mem, ws = guarded(nbytes)
        got = search(pr, w, ws)
        assert (mem[nbytes:] == 0xA5).all(), "written past the workspace"
        parity.check_match(got, orc, w.tau, parity.score_lookup(orc["scores"], got["best_idx"]))


@pytest.mark.parametrize("L,T,H,P,Q", [(20, 32, 8, 1226, 13), (1, 32, 5, 4179, 70), (7, 16, 5, 1300, 140), (7, 16, 5, 520, 300),
                                       (2, 16, 5, 1300, 513)])
def test_layer_mean(oracle, L, T, H, P, Q):
    n, columns = uneven(True, L, T, H, P, Q)
    print(f"[gpu-case] uneven shares, layer mean L={L} T={T} H={H} P={P} Q={Q}: {n}", flush=True)
    w = synth.scaled(synth.WORKLOADS[2], name="uneven", L=L, P=P, Q=Q, T=T, H=H, dtype="bf16" if Q % 2 else "f16", planted_frac=0.3,
                     R=1, E=P + Q, seed=9200 + P)
    pr = synth.make_problem(w, "cuda:0")
    noisy = pr["kp"][:, 7].float()           # not an exact copy: the root of a sum that rounds to 0 magnifies it (parity.dist_tol)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    pr["kq"][:, 0] = (noisy + 0.1 * torch.randn(noisy.shape, generator=g, device="cuda:0")).to(pr["kq"].dtype)
    pr["vq"][:, 0] = pr["vp"][:, 7] * 0.9
    for kp in (pr["kp"], pr["vp"]):
        kp[:, P - 2] = kp[:, 7]
    live = shared_live(pr)
    live[7] = live[P - 2] = 1
    thr = 0.5 * np.sqrt(128 / (T * H))
    got = gpu_layer_mean(pr, live, thr)
    paths.assert_tiles(lambda: gpu_layer_mean(pr, live, thr), (256, columns, 3))
    orc = oracle.layer_mean(1 if w.dtype == "bf16" else 0, *(synth.bits(pr[k]) for k in ("kq", "vq", "kp", "vp")), live.cpu().numpy(),
                            thr, want_dist=True)
    parity.check_layer_mean(got, orc, thr, parity.dist_lookup(orc["dist"], got["best_idx"]), 0.05 * parity.dist_tol(T, H, 128))
    assert got["best_idx"][0] == 7 and got["best_dist"][0] == got["second_dist"][0]
