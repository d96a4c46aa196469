"""Listed candidates with a wave per list (many lists that share blocks, and lists a little longer than 16): edges of its
slots and of the rule that takes calls there, against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import binding as rc
from paper_2507_21433_amd import synth
from tests.test_gpu_candidates import compare, compare_distances, gpu_candidates

pytestmark = pytest.mark.gpu


# (layers, pool, queries, tokens, heads, candidates): 2, 4, 6 and 8 slots, one and two (three) waves per list, a last wave with
# a candidate less; lists dealt out by XCD (448 waves of a layer) and one after the other; on and below 3000 and 4000 slots;
# half as many pairs as blocks and one fewer (1000 x 2 against 4000 and 4002)
SHAPES = [(3, 90, 500, 16, 1, 1), (2, 70, 380, 16, 3, 4), (2, 70, 380, 32, 1, 5), (1, 200, 448, 16, 2, 8), (1, 200, 449, 16, 2, 9),
          (2, 64, 250, 16, 1, 12), (2, 33, 190, 16, 5, 13), (5, 40, 75, 16, 1, 16), (1, 60, 375, 16, 1, 13), (1, 60, 374, 16, 1, 13),
          (2, 300, 167, 16, 1, 17), (2, 5000, 167, 16, 1, 17), (2, 5000, 166, 16, 1, 17), (1, 77, 224, 16, 16, 24), (1, 77, 170, 16, 2, 33),
          (2, 4000, 1000, 16, 1, 2), (2, 4002, 1000, 16, 1, 2)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("L,P,Q,T,H,C", SHAPES)
def test_wide_lists(oracle, L, P, Q, T, H, C, dtype):
    w = synth.scaled(synth.WORKLOADS[2], name=f"wide{L}.{P}x{Q}x{C}", L=L, P=P, Q=Q, T=T, H=H, dtype=dtype, planted_frac=0.0, R=1,
                     E=P + Q, seed=8400)
    print(f"[gpu-case] {w.name} T={T} H={H} {dtype}", flush=True)
    pr = synth.make_problem(w, "cuda:0")
    d = 0 if dtype == "f16" else 1
    bits = [synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")]
    rng = np.random.RandomState(C)
    cand = rng.randint(-1, P + 1, size=(L, Q, C)).astype(np.int32)      # empty and out-of-range entries, repeats
    cand[:, ::9] = -1                                                   # empty lists
    pr["live"][:, rng.permutation(P)[:P // 10]] = 0
    live = pr["live"].cpu().numpy()
    compare(gpu_candidates(w, pr, cand, pr["live"]), oracle.candidates(d, 0, *bits, cand, live, w.tau), cand, w.tau, tol=2e-5)   # as in the sweep
    unit = np.sqrt(w.Dh / (T * H))
    thr = float(np.sqrt(2.0)) * unit          # fresh blocks lie on both sides of it
    one = pr["live"][0].contiguous()
    g = rc.rc_candidate_distances(pr["kq"], pr["vq"], pr["kp"], pr["vp"], one, torch.as_tensor(cand[0], device="cuda:0"), thr)
    o = oracle.candidate_distances(d, *bits, cand[0], live[0], thr)
    compare_distances({k: v.cpu().numpy() for k, v in g.items()}, o, cand[0], thr, 1e-5 * unit)   # fp32 sums of exact differences


def test_wide_ties_go_to_the_lowest_index():
    w = synth.scaled(synth.WORKLOADS[2], name="wide_ties", L=1, P=60, Q=400, T=16, H=3, planted_frac=0.0, R=1, E=460, seed=8500)
    pr = synth.make_problem(w, "cuda:0")
    copies = [11, 20, 33, 47]
    for n in ("k", "v"):
        for c in copies:
            pr[n + "p"][:, c] = pr[n + "p"][:, 11]
        pr[n + "q"][:, :] = pr[n + "p"][:, 11:12]
    rng = np.random.RandomState(3)
    others = np.setdiff1d(np.arange(60), copies)
    cand = np.stack([rng.permutation(np.concatenate([rng.permutation(others)[:14], rng.permutation(copies)[:2]])) for _ in range(w.Q)]).astype(np.int32)
    want = np.array([min(c for c in row if c in copies) for row in cand])
    s = gpu_candidates(synth.scaled(w, tau=0.9), pr, cand[None], None)
    assert np.array_equal(s["best_idx"][0], want) and np.array_equal(s["match_idx"][0], want)
    g = rc.rc_candidate_distances(pr["kq"], pr["vq"], pr["kp"], pr["vp"], None, torch.as_tensor(cand, device="cuda:0"), 0.5)
    assert np.array_equal(g["best_idx"].cpu().numpy(), want) and (g["best_dist"] == 0).all()


# Eight waves to a workgroup: waves of a layer in whole workgroups and with six idle ones in the last; one layer and two in a
# group of the distances, a last group of one layer; by XCD and dealt out; 1800 waves and four fewer, 1700 of a layer and 20 more
EIGHTS = [(16, 64, 256, 16, 1, 3), (30, 64, 250, 16, 1, 4), (11, 50, 680, 16, 1, 3), (4, 40, 449, 16, 2, 5), (4, 40, 450, 16, 2, 5),
          (2, 60, 850, 16, 1, 17), (2, 60, 860, 16, 1, 17), (8, 700, 500, 16, 1, 2)]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("L,P,Q,T,H,C", EIGHTS)
def test_wide_lists_in_workgroups(oracle, L, P, Q, T, H, C, dtype):
    test_wide_lists(oracle, L, P, Q, T, H, C, dtype)


# lists that are partly or wholly empty: every number of valid candidates in 2, 4, 6 and 8 slots (a wave walks 2, 4 or all of
# them), a wave to a workgroup and eight, whole workgroups of empty lists and of nearly empty ones; a pair reports the bits that
# it has in a full list
@pytest.mark.parametrize("L,P,Q,T,H,C", [(1, 200, 448, 16, 2, 8), (1, 60, 375, 16, 1, 13), (1, 200, 449, 32, 1, 12), (30, 64, 250, 16, 1, 4),
                                         (30, 64, 250, 16, 1, 8), (30, 64, 250, 16, 1, 12), (30, 64, 250, 16, 1, 16), (5, 64, 850, 16, 1, 17)])
def test_wide_lists_partly_filled(oracle, L, P, Q, T, H, C):
    w = synth.scaled(synth.WORKLOADS[2], name=f"fill{L}.{P}x{Q}x{C}", L=L, P=P, Q=Q, T=T, H=H, planted_frac=0.0, R=1, E=P + Q, seed=8600)
    print(f"[gpu-case] {w.name} T={T} H={H}", flush=True)
    pr = synth.make_problem(w, "cuda:0")
    bits = [synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")]
    rng = np.random.RandomState(C)
    full = rng.randint(0, P, size=(L, Q, C)).astype(np.int32)
    n = rng.randint(0, C + 1, size=(L, Q, 1))
    n[:, 40:80], n[:, 120:200] = 0, rng.randint(0, C // 4 + 1, size=(L, 80, 1))
    keep = rng.random_sample(full.shape).argsort(-1) < n
    cand = np.where(keep, full, rng.choice([-1, P], size=full.shape)).astype(np.int32)
    live = np.ones((L, P), np.uint8)
    live[:, rng.permutation(P)[:P // 10]] = 0
    on_gpu = torch.as_tensor(live, device="cuda:0")
    g, f = gpu_candidates(w, pr, cand, on_gpu), gpu_candidates(w, pr, full, None)
    compare(g, oracle.candidates(0, 0, *bits, cand, live, w.tau), cand, w.tau, tol=2e-5)   # as in the sweep
    valid = keep & (np.take_along_axis(live, full.reshape(L, -1), 1).reshape(full.shape) != 0)
    assert np.array_equal(g["scores"][valid], f["scores"][valid]) and (g["scores"][~valid] == -np.inf).all()
    unit = np.sqrt(w.Dh / (T * H))
    thr = float(np.sqrt(2.0)) * unit
    d = [rc.rc_candidate_distances(pr["kq"], pr["vq"], pr["kp"], pr["vp"], lv, torch.as_tensor(c[0], device="cuda:0"), thr)
         for c, lv in ((cand, on_gpu[0].contiguous()), (full, None))]
    g, f = ({k: v.cpu().numpy() for k, v in x.items()} for x in d)
    compare_distances(g, oracle.candidate_distances(0, *bits, cand[0], live[0], thr), cand[0], thr, 1e-5 * unit)
    assert np.array_equal(g["dist"][valid[0]], f["dist"][valid[0]]) and (g["dist"][~valid[0]] == np.inf).all()
