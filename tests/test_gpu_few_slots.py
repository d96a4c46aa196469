"""The percentile in its two workspaces, and the pool's upkeep at the edges of what one workgroup holds in registers."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import binding as rc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV)


# below and above what one workgroup does, one and several samples per thread, one and several trips; both clusters, ties,
# infinities and NaN; the state of 24 KB and, in 4112 bytes, the one of 4 KB
@pytest.mark.parametrize("n", [8192, 8193, 11264, 11265, 16384, 16385, 262145, 1048577])
@pytest.mark.parametrize("nbytes", [4112, None])
def test_percentile_workspaces(oracle, n, nbytes):
    rng = np.random.RandomState(n % 1000)
    x = np.where(rng.rand(n) < 0.3, 0.15 + 0.02 * rng.randn(n), np.sqrt(2.0) + 0.01 * rng.randn(n)).astype(np.float32)
    x[rng.rand(n) < 0.02] = np.inf
    x[rng.rand(n) < 0.01] = np.nan
    x[rng.rand(n) < 0.05] = np.float32(-0.25)
    ws = torch.full(((nbytes or rc.lib().rc_pat_workspace_size()) + 256,), 0xA5, dtype=torch.uint8, device=DEV)
    for p in (0.0, 33.3, 80.0, 100.0):
        g = rc.rc_pat_threshold(t(x), p, workspace=ws[:-256])
        want, n_finite = oracle.pat_threshold(x, p)
        assert g["threshold"].cpu().numpy()[0] == want and int(g["n_finite"][0]) == n_finite
    assert (ws[-256:] == 0xA5).all(), "written past the workspace"
    x[rng.rand(n) < 0.98] = -np.inf                              # hardly a list had a candidate
    g = rc.rc_pat_threshold(t(x), 33.3, workspace=ws[:-256])
    want, n_finite = oracle.pat_threshold(x, 33.3)
    assert g["threshold"].cpu().numpy()[0] == want and int(g["n_finite"][0]) == n_finite
    g = rc.rc_pat_threshold(t(np.full(n, np.nan, np.float32)), 50.0, workspace=ws[:-256])
    assert g["threshold"].cpu().numpy()[0] == -np.inf and int(g["n_finite"][0]) == 0


# 2048 and 16 384 slots: two and sixteen per thread
@pytest.mark.parametrize("P", [1, 63, 1024, 1025, 2047, 2048, 2049, 16383, 16384, 16385])
@pytest.mark.parametrize("stamps", [1, 3, 1 << 30])
def test_evict_slots(oracle, P, stamps):
    rng = np.random.RandomState(P)
    for refs in (True, False):
        live = (rng.rand(P) < 0.9).astype(np.uint8)
        refc = rng.randint(0, 2, P).astype(np.int32) if refs else None
        used = rng.randint(-stamps, stamps, P).astype(np.int32)
        for unmatched in (0, 1, P // 3, P):
            match = np.full(unmatched + 2, 5, np.int32)
            match[:unmatched] = -1
            lv, want = t(live.copy()), live.copy()
            out = rc.rc_pool_evict(lv, t(refc) if refs else None, t(used), t(match), 1)
            n = oracle.pool_evict(want, refc, used, match, 1)
            assert np.array_equal(lv.cpu().numpy(), want) and (int(out["n_free"][0]), int(out["n_evicted"][0])) == tuple(n)


# 16 384 slots and 4096 queries go through one workgroup; flags that do not start on 16 bytes
@pytest.mark.parametrize("P,Q", [(1, 1), (15, 3), (17, 40), (1000, 1023), (1000, 1025), (16384, 4096), (16385, 10), (300, 4097)])
@pytest.mark.parametrize("shift", [0, 3])
def test_admit_slots(oracle, P, Q, shift):
    rng = np.random.RandomState(P + Q)
    L, T, H = 1, 16, 1
    kv = lambda n: torch.as_tensor(rng.randint(0, 999, (L, n, T, H, 128)).astype(np.float16), device=DEV)
    norm = lambda n: torch.as_tensor(rng.rand(L, n).astype(np.float32), device=DEV)
    kq, vq, kp, vp, qk, qv, pk, pv = kv(Q), kv(Q), kv(P), kv(P), norm(Q), norm(Q), norm(P), norm(P)
    live = (rng.rand(P) < 0.6).astype(np.uint8)
    match = np.where(rng.rand(Q) < 0.3, 0, -1).astype(np.int32)
    mem = torch.zeros(P + 16, dtype=torch.uint8, device=DEV)
    flags = mem[shift:shift + P]
    flags.copy_(t(live))
    before = [x.clone() for x in (kp, vp, pk, pv)]
    g = rc.rc_pool_admit(kq, vq, qk, qv, kp, vp, pk, pv, flags, t(match))
    free, open_q = np.flatnonzero(live == 0), np.flatnonzero(match < 0)
    n = min(free.size, open_q.size)
    slots = np.full(Q, -1, np.int32)
    slots[open_q[:n]] = free[:n]
    live[free[:n]] = 1
    assert int(g["n_admitted"][0]) == n and np.array_equal(g["slot_of_query"].cpu().numpy(), slots)
    assert np.array_equal(flags.cpu().numpy(), live) and not mem[:shift].any() and not mem[shift + P:].any()
    for got, was, src in zip((kp, vp, pk, pv), before, (kq, vq, qk, qv)):
        was[:, free[:n]] = src[:, open_q[:n]]
        assert torch.equal(got, was)
