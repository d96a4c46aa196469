"""Shapes at the edges of the library's dispatch rules, every entry point against the CPU oracle on the same inputs:
each list names the rule whose two sides it stands on.  Needs a real MI355X."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import binding as rc
from paper_2507_21433_amd import synth
from tests.test_gpu_candidates import compare, compare_distances, gpu_candidates
from tests import paths
from tests.test_gpu_layer_mean import gpu_layer_mean, run_case
from tests.test_gpu_parity import full_check, run_gpu_match
from tests.test_gpu_sweep import run_shape

pytestmark = pytest.mark.gpu

# Parts merged per query: the few-tiles path makes one per 32 pool rows; four parts per thread, 1 to 64 threads per query.
PARTS = [(1, 1), (33, 3), (128, 5), (129, 40), (257, 64), (2048, 3), (2049, 65), (8193, 2)]


@pytest.mark.parametrize("P,Q", PARTS)
def test_merge_parts(oracle, P, Q):
    run_shape(oracle, dict(L=2, P=P, Q=Q, T=16, H=1, mode=0, dtype="f16", planted_frac=0.3, seed=7100 + P), f"parts{P}x{Q}", P)


# Tile width (64 columns up to 64 queries, 128 up to 128, 192 or 256 beyond) and shares per tile: per-head mode in whole tiles
# (256 tiles: one round) and with one share per head, block mode with a share count that is no power of two.
WIDTHS = [(1, 256, 64, 64, 2, (64, 1)), (1, 256, 40, 65, 2, (128, 1)), (1, 256, 70, 128, 1, (128, 1)), (1, 3, 300, 64, 5, (64, 4)),
          (1, 2, 257, 65, 16, (128, 4)), (1, 2, 255, 128, 3, (128, 4)), (1, 2, 300, 129, 3, (192, 4)), (0, 24, 250, 40, 5, (64, 3)),
          (0, 24, 250, 65, 5, (128, 3)), (0, 2, 300, 128, 3, (128, 3)), (0, 11, 513, 1, 6, (64, 3)), (0, 2, 300, 192, 3, (192, 3)),
          (0, 2, 300, 257, 3, (192, 3)), (1, 2, 257, 384, 3, (192, 4)), (1, 2, 40, 385, 5, (256, 4))]


@pytest.mark.parametrize("mode,L,P,Q,H,tile", WIDTHS)
def test_tile_widths_and_shares(oracle, mode, L, P, Q, H, tile):
    run_shape(oracle, dict(L=L, P=P, Q=Q, T=16, H=H, mode=mode, dtype="bf16" if Q % 2 else "f16", planted_frac=0.3, seed=7300 + P),
              f"width{mode}.{L}.{P}x{Q}", P)
    w = synth.scaled(synth.WORKLOADS[2], name="width", L=L, P=P, Q=Q, T=16, H=H, mode=mode, planted_frac=0.0, R=1, E=P + Q)
    pr = synth.make_problem(w, "cuda:0")
    paths.assert_tiles(lambda: run_gpu_match(pr, w, None), (256, *tile))


# Shape of whole tiles beyond 128 queries: 256 x 192, 192 x 320 and 256 x 256 with one and more query tiles, pools that end
# on and beside an edge of a tile (256 x 256 with two query tiles in a workspace without room for tiles of 192 rows).
SHAPES = [(0, 260, 8, 129, 1, (256, 192)), (0, 260, 193, 192, 1, (256, 192)), (0, 260, 257, 193, 1, (192, 320)), (0, 260, 192, 257, 1, (192, 320)),
          (0, 260, 193, 320, 1, (256, 192)), (0, 260, 31, 321, 1, (256, 192)), (0, 260, 40, 640, 1, (192, 320)), (0, 260, 5, 641, 1, (192, 320)),
          (1, 260, 193, 160, 1, (256, 192)), (1, 130, 191, 300, 2, (192, 320)), (1, 260, 40, 384, 1, (256, 192)), (1, 260, 20, 640, 1, (192, 320)),
          (0, 260, 255, 256, 1, (256, 256)), (0, 300, 500, 193, 1, (256, 256)), (1, 260, 129, 250, 1, (256, 256)), (1, 260, 300, 256, 1, (256, 256)),
          (0, 130, 449, 500, 1, (256, 256)), (0, 260, 193, 385, 1, (256, 256)), (1, 260, 193, 512, 1, (256, 256))]


@pytest.mark.parametrize("mode,L,P,Q,H,tile", SHAPES)
def test_tile_shapes(oracle, mode, L, P, Q, H, tile):
    w = synth.scaled(synth.WORKLOADS[2], name=f"shape{mode}.{L}.{P}x{Q}", L=L, P=P, Q=Q, T=16, H=H, mode=mode, dtype="bf16" if Q % 2 else "f16",
                     planted_frac=0.0 if P < 64 else 0.3 * min(1.0, P / Q), R=1, E=P + Q, seed=7500 + P)
    pr = synth.make_problem(w, "cuda:0")
    ws = paths.whole_tiles_workspace(w) if tile == (256, 256) and Q > 256 else None
    paths.assert_tiles(lambda: run_gpu_match(pr, w, pr["live"], workspace=ws), (*tile, mode))
    full_check(oracle, w, pr, pr["live"], ws)


# Layer-mean search at 64 and 128 columns (running sums in registers), 192 and 256 (in memory), layers in groups of 2, 2 and
# 1 (256 pool tiles of 5 layers) and of 2 with a last one of 1 (two query tiles of 192 columns, 21 pool tiles of 27 layers).
@pytest.mark.parametrize("L,P,Q,columns", [(5, 65300, 9, 64), (5, 65300, 65, 128), (5, 65300, 129, 192), (5, 65300, 193, 256), (27, 5200, 257, 192)])
def test_layer_mean_widths(oracle, L, P, Q, columns):
    w = synth.scaled(synth.WORKLOADS[2], name=f"lm{L}.{P}x{Q}", L=L, P=P, Q=Q, T=16, H=1, planted_frac=0.3, R=1, E=P + Q, seed=7700)
    pr, _, _, _ = run_case(oracle, w, 0.5 * np.sqrt(w.Dh / (w.T * w.H)))
    paths.assert_tiles(lambda: gpu_layer_mean(pr, None, 0.5), (256, columns, 2))


# Shares per pair added by the selection kernels: 8 at a time, then 4, then single ones, K and V layer by layer dealt to four
# threads; pool chunks of 32 rows that end inside a group of four.
@pytest.mark.parametrize("L,P,Q,H", [(1, 1, 1, 16), (1, 37, 66, 3), (1, 250, 9, 5), (3, 35, 129, 7), (9, 259, 2, 3)])
def test_share_selection(oracle, L, P, Q, H):
    for mode in (0, 1):
        run_shape(oracle, dict(L=L, P=P, Q=Q, T=16, H=H, mode=mode, dtype="f16", planted_frac=0.0 if P < 64 else 0.3, seed=7900 + P),
                  f"shares{mode}.{L}.{P}x{Q}", P)


# Few samples (one workgroup, up to 16 384) and many; few lists (4 candidates per workgroup) and many, more candidates than lanes.
@pytest.mark.parametrize("n", [0, 1, 1023, 1024, 1025, 16383, 16384, 16385])
def test_percentile_sample_counts(oracle, n):
    rng = np.random.RandomState(n)
    x = rng.choice(np.float32([0.15, -0.15, 1.4, np.inf, np.nan, -np.inf, 0.0, 1e-40]), size=n) * (1 + rng.randint(0, 3, size=n).astype(np.float32) * 2**-20)
    x = torch.as_tensor(x.astype(np.float32), device="cuda:0")
    for p in (0.0, 37.5, 100.0):
        got = rc.rc_pat_threshold(x, p)
        want, n_finite = oracle.pat_threshold(x.cpu().numpy(), p)
        assert got["threshold"].cpu().numpy()[0] == want and int(got["n_finite"][0]) == n_finite


@pytest.mark.parametrize("L,Q,C", [(1, 1, 5), (3, 109, 17), (1, 256, 17), (2, 112, 16), (2, 113, 16), (2, 130, 70)])
def test_candidates_per_workgroup(oracle, L, Q, C):
    w = synth.scaled(synth.WORKLOADS[2], name=f"lists{L}.{Q}x{C}", L=L, P=90, Q=Q, T=16, H=3, planted_frac=0.0, R=1, E=90 + Q, seed=8100)
    pr = synth.make_problem(w, "cuda:0")
    bits = [synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")]
    cand = np.random.RandomState(C).randint(-1, 90, size=(L, Q, C)).astype(np.int32)
    for mode in (0, 1):
        g = gpu_candidates(synth.scaled(w, mode=mode), pr, cand, pr["live"])
        compare(g, oracle.candidates(0, mode, *bits, cand, pr["live"].cpu().numpy(), w.tau), cand, w.tau, tol=2e-5)   # as in the sweep
    live = pr["live"][0].contiguous()
    unit = np.sqrt(w.Dh / (w.T * w.H))
    thr = float(np.sqrt(2.0)) * unit          # fresh blocks lie on both sides of it
    g = rc.rc_candidate_distances(pr["kq"], pr["vq"], pr["kp"], pr["vp"], live, torch.as_tensor(cand[0], device="cuda:0"), thr)
    o = oracle.candidate_distances(0, *bits, cand[0], live.cpu().numpy(), thr)
    compare_distances({k: v.cpu().numpy() for k, v in g.items()}, o, cand[0], thr, 1e-5 * unit)   # fp32 sums of exact differences


# Equal distances go to the lowest pool index, wherever the copies stand in the list: in one lane's trips (64 apart), in
# different lanes, before and behind lane 63, the higher index first or last.
@pytest.mark.parametrize("first,second", [(0, 1), (0, 64), (1, 65), (5, 69), (3, 130), (63, 64), (40, 127), (62, 63), (10, 100), (0, 149)])
def test_tied_candidates_go_to_the_lowest_index(first, second):
    w = synth.scaled(synth.WORKLOADS[2], name="ties", L=3, P=200, Q=6, T=16, H=3, planted_frac=0.0, R=1, E=206, seed=8200)
    pr = synth.make_problem(w, "cuda:0")
    C, copies = 150, (150, 20, 77, 190, 33, 120)
    cand = np.random.RandomState(first).permutation(np.setdiff1d(np.arange(200), (*copies, 7)))[None, :C].repeat(w.Q, 0).astype(np.int32)
    for n in ("k", "v"):
        for p in copies:
            pr[n + "p"][:, p] = pr[n + "p"][:, 7]
        pr[n + "q"][:, :] = pr[n + "p"][:, 7:8]      # every copy at distance 0 and score 1
    for q, (a, b) in enumerate([(150, 20), (20, 150), (190, 77), (77, 190), (120, 33), (33, 120)]):
        cand[q, first], cand[q, second] = a, b
    want = np.minimum(cand[:, first], cand[:, second])
    g = rc.rc_candidate_distances(pr["kq"], pr["vq"], pr["kp"], pr["vp"], None, torch.as_tensor(cand, device="cuda:0"), 0.5)
    assert np.array_equal(g["best_idx"].cpu().numpy(), want) and np.array_equal(g["match_idx"].cpu().numpy(), want)
    assert (g["best_dist"] == 0).all()
    for mode in (0, 1):
        s = gpu_candidates(synth.scaled(w, mode=mode, tau=0.9), pr, cand[None].repeat(w.L, 0), None)
        assert np.array_equal(s["best_idx"], want[None].repeat(w.L, 0)) and np.array_equal(s["match_idx"], s["best_idx"])


# Candidates per workgroup, both sides of the lines of cand_per_wg for blocks of 32, 64 and 128 KB: counts of lists at which
# workgroups of 4 fill one, one and a half and two rounds of the compute units, and of 16 a round and a little more.
LINES = [(16, 8, 176, 5), (16, 8, 177, 5), (16, 8, 224, 8), (16, 8, 225, 8), (16, 8, 170, 12), (16, 8, 171, 12), (16, 8, 257, 7), (16, 8, 342, 10),
         (16, 8, 320, 13), (16, 8, 321, 13), (32, 8, 128, 6), (32, 8, 129, 6), (32, 8, 213, 24), (32, 16, 64, 16), (32, 16, 149, 9), (32, 16, 257, 4)]


@pytest.mark.parametrize("T,H,Q,C", LINES)
def test_candidates_at_the_lines(oracle, T, H, Q, C):
    w = synth.scaled(synth.WORKLOADS[2], name=f"lines{T}.{H}.{Q}x{C}", L=1, P=60, Q=Q, T=T, H=H, planted_frac=0.0, R=1, E=60 + Q, seed=8300)
    pr = synth.make_problem(w, "cuda:0")
    bits = [synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")]
    cand = np.random.RandomState(C).randint(-1, 60, size=(1, Q, C)).astype(np.int32)
    live = pr["live"].cpu().numpy()
    for mode in (0, 1):
        compare(gpu_candidates(synth.scaled(w, mode=mode), pr, cand, pr["live"]), oracle.candidates(0, mode, *bits, cand, live, w.tau), cand, w.tau, tol=2e-5)
    unit = np.sqrt(w.Dh / (T * H))
    g = rc.rc_candidate_distances(pr["kq"], pr["vq"], pr["kp"], pr["vp"], pr["live"][0].contiguous(), torch.as_tensor(cand[0], device="cuda:0"), 0.5 * unit)
    compare_distances({k: v.cpu().numpy() for k, v in g.items()}, oracle.candidate_distances(0, *bits, cand[0], live[0], 0.5 * unit), cand[0],
                      0.5 * unit, 1e-5 * unit)
