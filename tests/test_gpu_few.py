"""Search of a small problem with few queries (64 pool blocks per workgroup, 16, 32 or 64 query rows, shares of the
reduction): edges of its tiles and both sides of the line to the tile kernels, against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import binding as rc
from paper_2507_21433_amd import synth
from tests import parity, paths
from tests.test_gpu_layer_mean import gpu_layer_mean
from tests.test_gpu_parity import run_gpu_match
from tests.test_gpu_sweep import run_shape

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def takes_few(call):
    """Whether call() launches few_shares_kernel or head_shares_kernel, rather than tile kernels; the test is skipped where no kernel
    trace is to be had, and fails where a call launches both."""
    names = paths.kernel_names(call)
    if not names:
        pytest.skip("no kernel trace here")
    few, tiles = (any(k in n for n in names for k in ks) for ks in (("few_shares_kernel", "head_shares_kernel"), ("rc::match_",)))
    assert few != tiles, f"kernels of {'both plans' if few else 'neither plan'}: {sorted(set(names))}"
    return few


# (layers, pool, queries, tokens, heads): one block; ends on and beside a tile of 64; 16 / 17, 32 / 33 and 64 query rows; odd head
# counts (shares that are no power of two, one slice per wave), more pool than one round of the selection (16 x 256 blocks)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("L,P,Q,T,H", [(1, 1, 1, 16, 1), (2, 63, 16, 16, 3), (1, 64, 17, 16, 5), (3, 65, 32, 32, 1), (1, 257, 33, 16, 8),
                                       (2, 129, 64, 16, 7), (1, 4097, 3, 16, 2), (3, 300, 9, 32, 16), (66, 70, 4, 16, 3), (1, 513, 15, 16, 13)])
def test_few_queries(oracle, L, P, Q, T, H, dtype):
    run_shape(oracle, dict(L=L, P=P, Q=Q, T=T, H=H, mode=0, dtype=dtype, planted_frac=0.3 if P > Q else 0.0, seed=8700 + P), f"few{L}.{P}x{Q}", P)
    w = synth.scaled(synth.WORKLOADS[2], name="few", L=L, P=P, Q=Q, T=T, H=H, planted_frac=0.0, R=1, E=P + Q)
    pr = synth.make_problem(w, DEV)
    for call in (lambda: run_gpu_match(pr, w, None), lambda: gpu_layer_mean(pr, None, 0.5)):
        assert takes_few(call)


# 64 queries are few, 65 are not; pools on both sides of 256, 200 and 150 MB of blocks, 768 and 640 rows to select from; layer mean:
# 1000 MB for pools of up to 2048 blocks and 160 tiles of 256, 400 MB for longer ones (600 MB, 1024 and 350 MB from 17 queries on;
# 500 MB, 512 and 200 MB from 33 on)
@pytest.mark.parametrize("mean,L,P,Q,T,H,few", [(False, 1, 300, 64, 16, 2, 1), (False, 1, 300, 65, 16, 2, 0), (False, 2, 1950, 16, 16, 8, 1), (False, 2, 1960, 16, 16, 8, 0),
                                                (False, 3, 1017, 17, 16, 8, 1), (False, 3, 1018, 17, 16, 8, 0), (False, 5, 457, 33, 16, 8, 1), (False, 5, 458, 33, 16, 8, 0),
                                                (False, 48, 70, 16, 16, 1, 1), (False, 49, 70, 16, 16, 1, 0), (False, 24, 70, 32, 16, 1, 1), (False, 25, 70, 32, 16, 1, 0),
                                                (False, 16, 70, 40, 16, 1, 1), (False, 17, 70, 40, 16, 1, 0),
                                                (True, 10, 762, 2, 32, 8, 1), (True, 10, 763, 2, 32, 8, 0), (True, 3, 2034, 2, 16, 8, 1), (True, 2, 2048, 2, 32, 8, 1),
                                                (True, 2, 2049, 2, 32, 8, 0), (True, 160, 60, 2, 32, 3, 1), (True, 161, 60, 2, 32, 3, 0),
                                                (True, 2, 2670, 18, 16, 8, 1), (True, 2, 2671, 18, 16, 8, 0), (True, 6, 1024, 18, 16, 8, 1), (True, 6, 1025, 18, 16, 8, 0),
                                                (True, 9, 1017, 18, 16, 8, 1), (True, 9, 1018, 18, 16, 8, 0),
                                                (True, 2, 1525, 40, 16, 8, 1), (True, 2, 1526, 40, 16, 8, 0), (True, 7, 512, 40, 16, 8, 1), (True, 7, 513, 40, 16, 8, 0)])
def test_lines(mean, L, P, Q, T, H, few):
    w = synth.scaled(synth.WORKLOADS[2], name="line", L=L, P=P, Q=Q, T=T, H=H, planted_frac=0.3, R=1, E=P + Q, seed=8800)
    pr = synth.make_problem(w, DEV)
    assert takes_few((lambda: gpu_layer_mean(pr, None, 0.5)) if mean else (lambda: run_gpu_match(pr, w, None))) == (few == 1)


def test_identical_blocks_tie_everywhere(oracle):
    # copies of one block in every tile, on every side of its edges: equal scores to the bit, the lowest live index wins
    w = synth.scaled(synth.WORKLOADS[2], name="ties", L=2, P=400, Q=20, T=16, H=5, planted_frac=0.0, R=1, E=420, seed=8900)
    pr = synth.make_problem(w, DEV)
    copies = [3, 16, 63, 64, 127, 200, 319, 320, 399]
    for n in ("k", "v"):
        for c in copies:
            pr[n + "p"][:, c] = pr[n + "p"][:, 3]
        pr[n + "q"][:, :] = pr[n + "p"][:, 3:4]
    for dead in range(len(copies) - 1):
        live = torch.ones((w.L, w.P), dtype=torch.uint8, device=DEV)
        live[:, copies[:dead]] = 0
        g, _ = run_gpu_match(pr, w, live)
        assert (g["best_idx"] == copies[dead]).all() and np.array_equal(g["best_score"], g["second_score"])
        m = gpu_layer_mean(pr, live[0].contiguous(), 0.5)
        assert (m["best_idx"] == copies[dead]).all() and np.array_equal(m["best_dist"], m["second_dist"])


@pytest.mark.parametrize("L,P,Q,T,H", [(1, 256, 32, 16, 8), (24, 90, 40, 16, 5), (1, 700, 3, 32, 4)])
def test_small_workspaces(oracle, L, P, Q, T, H):
    # without room for its shares the call takes the plan of the tile kernels; nothing is written past the workspace
    w = synth.scaled(synth.WORKLOADS[2], name="ws", L=L, P=P, Q=Q, T=T, H=H, planted_frac=0.3, R=1, E=P + Q, seed=8950)
    pr = synth.make_problem(w, DEV)
    o = oracle.match(0, 0, *(synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")), pr["live"].cpu().numpy(), w.tau, want_scores=True)
    for nbytes in (paths.needed(rc.lib(), 0, L, T, H, P, Q), paths.size(rc.lib(), 0, L, T, H, P, Q)):
        mem = torch.full((nbytes + (1 << 20),), 0xA5, dtype=torch.uint8, device=DEV)
        g, _ = run_gpu_match(pr, w, pr["live"], workspace=mem[:nbytes])
        assert (mem[nbytes:] == 0xA5).all(), "written past the workspace"
        parity.check_match(g, o, w.tau, parity.score_lookup(o["scores"], g["best_idx"]))


# per head: one block, ends on and beside a tile of 64 and a wave of 32; 1, 8 / 9, 16 / 17 and 32 queries; one head, odd head counts,
# 32 tokens; bits as the tile kernels have them, the lowest index on ties
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("L,P,Q,T,H", [(1, 1, 1, 16, 1), (2, 63, 8, 16, 3), (1, 64, 9, 16, 5), (3, 65, 17, 32, 2), (1, 257, 32, 16, 8), (2, 97, 16, 16, 16),
                                       (5, 300, 5, 32, 10), (1, 4097, 2, 16, 2)])
def test_few_queries_per_head(oracle, L, P, Q, T, H, dtype):
    run_shape(oracle, dict(L=L, P=P, Q=Q, T=T, H=H, mode=1, dtype=dtype, planted_frac=0.3 if P > Q else 0.0, seed=9100 + P), f"heads{L}.{P}x{Q}", P)
    w = synth.scaled(synth.WORKLOADS[5], name="heads", L=L, P=P, Q=Q, T=T, H=H, dtype=dtype, planted_frac=0.3 if P > Q else 0.0, R=1, E=P + Q, seed=9200 + P)
    pr = synth.make_problem(w, DEV)
    if P > 70:
        for n in ("k", "v"):
            pr[n + "p"][:, 70] = pr[n + "p"][:, 2]
            pr[n + "q"][:, 0] = pr[n + "p"][:, 2]
    g, _ = run_gpu_match(pr, w, pr["live"])
    mem = torch.full((paths.size(rc.lib(), 1, L, T, H, P, Q) + (1 << 20),), 0xA5, dtype=torch.uint8, device=DEV)
    again, _ = run_gpu_match(pr, w, pr["live"], workspace=mem[:-(1 << 20)])
    assert (mem[-(1 << 20):] == 0xA5).all(), "written past the workspace"
    # the same layers inside a call with more queries than these kernels take: the tile kernels' bits
    more = dict(pr, **{n: torch.cat([pr[n], pr[n][:, :1].expand(-1, 33, -1, -1, -1)], 1).contiguous() for n in ("kq", "vq")})
    tiles, _ = run_gpu_match(more, synth.scaled(w, Q=Q + 33), pr["live"])
    for k in g:
        assert np.array_equal(g[k], again[k]) and np.array_equal(g[k], tiles[k][:, :Q]), k
    assert takes_few(lambda: run_gpu_match(pr, w, pr["live"]))


# 3, 8, 16 and 32 queries; the lines at 6000, 3000 and 2500 MB are too large for a test; 512 workgroups, 208 and 256 shares of the tile
# kernels, 144 from 17 queries on where a layer has more than 64 blocks; 500 MB of blocks of 32 tokens of two heads
@pytest.mark.parametrize("L,P,Q,T,H,few", [(8, 200, 32, 16, 16, True), (9, 257, 32, 16, 16, False), (9, 257, 16, 16, 16, True), (2, 100, 33, 16, 4, False),
                                           (26, 70, 4, 16, 8, True), (27, 70, 4, 16, 8, False), (32, 70, 4, 16, 8, False), (33, 70, 4, 16, 8, True),
                                           (36, 70, 17, 16, 4, True), (37, 70, 17, 16, 4, False), (37, 64, 17, 16, 4, True), (1, 15258, 2, 32, 2, True),
                                           (1, 15259, 2, 32, 2, False)])
def test_lines_per_head(L, P, Q, T, H, few):
    w = synth.scaled(synth.WORKLOADS[5], name="line", L=L, P=P, Q=Q, T=T, H=H, planted_frac=0.3, R=1, E=P + Q, seed=9300)
    pr = synth.make_problem(w, DEV)
    assert takes_few(lambda: run_gpu_match(pr, w, None)) == few
