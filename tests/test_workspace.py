"""The bytes of workspace a search call insists on.  They do not follow the tile shapes and shares that are fastest: a
smaller workspace than rc_match_workspace_size() gives a slower plan, down to a floor that is stated in include/rc.h."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import binding as rc
from paper_2507_21433_amd import synth
from tests import parity
from tests.paths import mean_needed, mean_size, needed, size, whole_tiles

DEV = "cuda:0"


@pytest.fixture(scope="module")
def lib():
    import os
    if not os.path.exists(rc.LIB_PATH):
        from paper_2507_21433_amd import build
        build.build()
    return rc.lib()


# more than 256 tiles of 256 x 256, or (block score, at most 128 queries) more than 128: never more than the partials
@pytest.mark.parametrize("mode,L,T,H,P,Q", [(0, 48, 32, 10, 1289, 102), (1, 32, 32, 8, 2531, 24), (0, 24, 16, 10, 1635, 4),
                                            (0, 7, 16, 10, 6272, 1), (1, 46, 16, 8, 1515, 1), (0, 40, 16, 10, 6201, 300),
                                            (1, 16, 32, 8, 4100, 300), (0, 64, 16, 8, 4096, 256), (0, 260, 16, 1, 193, 640)])
def test_search_takes_the_partials_of_whole_tiles(lib, mode, L, T, H, P, Q):
    assert needed(lib, mode, L, T, H, P, Q) == whole_tiles(L, P, Q) <= size(lib, mode, L, T, H, P, Q)


# fewer tiles: 256 KB per share and tile, and the partials of the pool chunks
@pytest.mark.parametrize("mode,L,T,H,P,Q,nbytes", [(0, 1, 16, 8, 4096, 16, 67141632), (0, 2, 16, 8, 64, 4, 33554688),
                                                   (1, 2, 16, 8, 257, 4, 8389760), (0, 2, 16, 8, 4096, 300, 68337664),
                                                   (1, 3, 16, 4, 11147, 133, 140640048)])
def test_search_takes_256_column_shares(lib, mode, L, T, H, P, Q, nbytes):
    assert needed(lib, mode, L, T, H, P, Q) == nbytes <= size(lib, mode, L, T, H, P, Q)


def test_one_workspace_for_the_largest_call(lib):
    # an engine that sizes once for its largest step: every smaller step of more than one round of tiles is taken
    for mode, L, T, H, P in [(0, 64, 16, 8, 4096), (1, 32, 32, 8, 2531), (0, 48, 16, 10, 3100), (1, 64, 16, 4, 1289)]:
        largest = size(lib, mode, L, T, H, P, 256)
        for Q in (1, 24, 40, 64, 65, 102, 128, 129, 192, 200, 255):
            assert needed(lib, mode, L, T, H, P, Q) <= largest, (mode, L, P, Q)


# the sums of 256 x 256 tiles (256 KB) of each group of layers, as few groups as make 1024 tiles, and 16-byte partials: a
# call never needs more, however many shares it is fastest with
@pytest.mark.parametrize("L,T,H,P,Q", [(43, 16, 10, 704, 27), (64, 16, 8, 1280, 16), (64, 16, 8, 2048, 128), (61, 16, 16, 1100, 8),
                                       (25, 16, 8, 13134, 3), (13, 16, 8, 11504, 36), (32, 32, 8, 2900, 64), (12, 16, 8, 6144, 169)])
def test_layer_mean_takes_the_sums_of_whole_tiles(lib, L, T, H, P, Q):
    tiles = -(-P // 256) * -(-Q // 256)
    groups = min(L, -(-1024 // tiles))
    chunks = -(-P // 32)
    assert mean_needed(lib, L, T, H, P, Q) <= groups * tiles * 262144 + chunks * Q * 16
    assert mean_needed(lib, L, T, H, P, Q) <= mean_size(lib, L, T, H, P, Q)


@pytest.mark.parametrize("L,T,H,P,Q,nbytes", [(1, 16, 8, 459, 8, 33556352), (12, 16, 8, 1537, 169, 177750720)])
def test_layer_mean_takes_256_column_shares(lib, L, T, H, P, Q, nbytes):
    assert mean_needed(lib, L, T, H, P, Q) == nbytes <= mean_size(lib, L, T, H, P, Q)


# at most 2048 shares of at most 256 tiles, and a share is as large as its tile: 64 KB up to 64 queries, 128 KB up to 128
@pytest.mark.parametrize("mode,L,T,H,P,Q", [(0, 24, 16, 10, 1635, 4), (0, 7, 16, 10, 6272, 1), (1, 46, 16, 8, 915, 1), (0, 45, 16, 8, 700, 65)])
def test_narrow_shares_take_no_more_than_they_store(lib, mode, L, T, H, P, Q):
    partials = L * -(-P // 32) * Q * 16
    assert size(lib, mode, L, T, H, P, Q) <= 2048 * 256 * (64 if Q <= 64 else 128) * 4 + partials


# ---- the slower plans give the oracle's results, and no plan writes past its workspace

GUARD = 1 << 20


def guarded(nbytes):
    t = torch.full((nbytes + GUARD,), 0xA5, dtype=torch.uint8, device=DEV)
    return t, t[:nbytes]


def search(pr, w, ws):
    qk, qv = rc.rc_block_norms(pr["kq"], pr["vq"], w.mode)
    pk, pv = rc.rc_block_norms(pr["kp"], pr["vp"], w.mode)
    out = rc.rc_match_blocks(pr["kq"], pr["vq"], qk, qv, pr["kp"], pr["vp"], pk, pv, pr["live"], w.tau, w.mode, workspace=ws)
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items()}


# a small workspace takes 64- and 128-column shares to whole tiles (both modes) and 192 x 320 tiles to 256 x 256; 192 and 64
# columns that fit either way
@pytest.mark.gpu
@pytest.mark.parametrize("mode,L,T,H,P,Q", [(0, 24, 16, 3, 1635, 4), (0, 100, 16, 3, 513, 65), (1, 90, 16, 8, 513, 40), (1, 90, 16, 4, 513, 97),
                                            (0, 90, 16, 1, 577, 300), (1, 90, 16, 2, 577, 300), (0, 2, 16, 3, 300, 180), (0, 3, 16, 8, 257, 5)])
def test_search_in_a_small_workspace(oracle, lib, mode, L, T, H, P, Q):
    print(f"[gpu-case] small workspace mode {mode} L={L} T={T} H={H} P={P} Q={Q}", flush=True)
    w = synth.scaled(synth.WORKLOADS[2], name="small_ws", L=L, P=P, Q=Q, T=T, H=H, mode=mode, planted_frac=0.3 if P > Q else 0.0,
                     R=1, E=P + Q, seed=61)
    pr = synth.make_problem(w, DEV)
    orc = oracle.match(0, mode, *(synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")), pr["live"].cpu().numpy(), w.tau, want_scores=True)
    floor, full = needed(lib, mode, L, T, H, P, Q), size(lib, mode, L, T, H, P, Q)
    got = {}
    for nbytes in {floor, full}:
        mem, ws = guarded(nbytes)
        got[nbytes] = search(pr, w, ws)
        assert (mem[nbytes:] == 0xA5).all(), "written past the workspace"
        parity.check_match(got[nbytes], orc, w.tau, parity.score_lookup(orc["scores"], got[nbytes]["best_idx"]))
    if mode == 1:   # scores on a grid, the same on every plan
        for k in got[full]:
            assert np.array_equal(got[floor][k], got[full][k]), k
    with pytest.raises(rc.RcError) as e:
        search(pr, w, guarded(floor - 1)[1])
    assert e.value.code == 3


# whole tiles of 64 and 128 columns where shares are faster, shares and whole tiles that fit either way
@pytest.mark.gpu
@pytest.mark.parametrize("L,T,H,P,Q", [(40, 16, 3, 1900, 9), (50, 16, 4, 1300, 100), (2, 16, 3, 300, 180), (30, 16, 1, 9000, 65)])
def test_layer_mean_in_a_small_workspace(oracle, lib, L, T, H, P, Q):
    print(f"[gpu-case] layer mean, small workspace L={L} T={T} H={H} P={P} Q={Q}", flush=True)
    w = synth.scaled(synth.WORKLOADS[2], name="small_ws_lm", L=L, P=P, Q=Q, T=T, H=H, planted_frac=0.3, R=1, E=P + Q, seed=62)
    pr = synth.make_problem(w, DEV)
    live = pr["live"].min(dim=0).values.contiguous()
    thr = 0.5 * np.sqrt(w.Dh / (T * H))
    orc = oracle.layer_mean(0, *(synth.bits(pr[n]) for n in ("kq", "vq", "kp", "vp")), live.cpu().numpy(), thr, want_dist=True)
    norms = [*rc.rc_block_norms(pr["kq"], pr["vq"], 0), *rc.rc_block_norms(pr["kp"], pr["vp"], 0)]

    def call(ws):
        out = rc.rc_match_blocks_layer_mean(pr["kq"], pr["vq"], *norms[:2], pr["kp"], pr["vp"], *norms[2:], live, thr, workspace=ws)
        torch.cuda.synchronize()
        return {k: v.cpu().numpy() for k, v in out.items()}

    floor, full = mean_needed(lib, L, T, H, P, Q), mean_size(lib, L, T, H, P, Q)
    for nbytes in {floor, full}:
        mem, ws = guarded(nbytes)
        got = call(ws)
        assert (mem[nbytes:] == 0xA5).all(), "written past the workspace"
        parity.check_layer_mean(got, orc, thr, parity.dist_lookup(orc["dist"], got["best_idx"]), 0.05 * parity.dist_tol(T, H, w.Dh))
    with pytest.raises(rc.RcError) as e:
        call(guarded(floor - 1)[1])
    assert e.value.code == 3


@pytest.mark.gpu
@pytest.mark.parametrize("mode,L,T,H,P,Q", [(0, 2, 16, 3, 300, 180), (1, 2, 16, 5, 257, 180), (0, 1, 16, 3, 300, 300), (0, 1, 16, 3, 300, 256)])
def test_shares_stay_within_their_tiles(lib, mode, L, T, H, P, Q):
    # few tiles: a share is stored as 256 x 192 or 256 floats, behind the shares follow the partials of the pool chunks
    # (32 rows here), and what a workspace holds beyond is never touched (narrower shares fill theirs: the guards above)
    print(f"[gpu-case] extent of the shares mode {mode} L={L} T={T} H={H} P={P} Q={Q}", flush=True)
    w = synth.scaled(synth.WORKLOADS[2], name="extent", L=L, P=P, Q=Q, T=T, H=H, mode=mode, planted_frac=0.0, R=1, E=P + Q, seed=63)
    pr = synth.make_problem(w, DEV)
    columns = 192 if Q <= 192 or 256 < Q <= 384 else 256
    npt, partials = -(-P // 256), L * -(-P // 32) * Q * 16
    shares, rest = divmod(needed(lib, mode, L, T, H, P, Q) - partials, L * npt * -(-Q // 256) * 262144)
    assert rest == 0 and shares > 1
    end = L * npt * -(-Q // columns) * shares * 256 * columns * 4 + partials
    mem, ws = guarded(size(lib, mode, L, T, H, P, Q))
    search(pr, w, ws)
    assert (mem[end:] == 0xA5).all() and not (mem[end - partials:end] == 0xA5).all()
