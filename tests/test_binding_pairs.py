"""A V tensor is read with the descriptor and the block count of its K tensor: one of another type, of another block shape, or with fewer
blocks or layers than K is refused before the library is called.  CPU only: the library's place is taken by a recorder."""
import pytest
import torch

from paper_2507_21433_amd import binding as rc

L, Q, P, T, H, C = 3, 3, 5, 16, 2, 4
HALF = torch.float16


class Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            if name.endswith("_size"):
                return 16
            self.calls.append(name)
            return rc.RC_OK
        return call


@pytest.fixture
def library(monkeypatch):
    rec = Recorder()
    monkeypatch.setattr(rc, "lib", lambda: rec)
    monkeypatch.setattr(rc, "_dev", lambda *ts: None)
    monkeypatch.setattr(rc, "_stream", lambda: 0)
    return rec


def blocks(n, layers=L, t=T, h=H, dtype=HALF, room=8):
    """[layers][n][t][h][128], the layers `room` blocks apart whatever n is."""
    return torch.zeros((layers, room, t, h, 128), dtype=dtype)[:, :n]


def norms(n):
    return torch.zeros((L, n))


def calls(kq, vq, kp, vp):
    """Every entry point that takes queries and a pool as pairs of K and V."""
    norm = (norms(Q), norms(Q), kp, vp, norms(P), norms(P))
    live, ids = torch.ones((L, P), dtype=torch.uint8), torch.zeros((L, Q, C), dtype=torch.int32)
    return {
        "rc_match_blocks": lambda: rc.rc_match_blocks(kq, vq, *norm, live, 0.9),
        "rc_match_blocks_layer_mean": lambda: rc.rc_match_blocks_layer_mean(kq, vq, *norm, live[0], 0.9),
        "rc_pool_admit": lambda: rc.rc_pool_admit(kq, vq, *norm, live[0], ids[0, :, 0].contiguous()),
        "rc_score_candidates": lambda: rc.rc_score_candidates(kq, vq, *norm, live, ids, 0.9),
        "rc_candidate_distances": lambda: rc.rc_candidate_distances(kq, vq, kp, vp, live[0], ids[0], 0.9),
    }


ENTRIES = sorted(calls(*[blocks(Q)] * 2, *[blocks(P)] * 2))
WRONG = {
    "another type": lambda n: blocks(n, dtype=torch.bfloat16),
    "fewer blocks": lambda n: blocks(n - 1),
    "fewer layers": lambda n: blocks(n, layers=L + 1)[:L - 1],
    "half the heads": lambda n: blocks(n, t=2 * T, h=H // 2),
}


@pytest.mark.parametrize("what", sorted(WRONG))
@pytest.mark.parametrize("entry", ENTRIES)
def test_a_value_tensor_that_its_key_tensor_does_not_describe_is_refused(library, entry, what):
    kq, kp = blocks(Q), blocks(P)
    for vq, vp in ((WRONG[what](Q), blocks(P)), (blocks(Q), WRONG[what](P))):
        with pytest.raises(AssertionError):
            calls(kq, vq, kp, vp)[entry]()
    assert library.calls == []


def test_listed_candidates_of_a_value_tensor_with_another_layer_stride_are_refused(library):
    kq, kp = blocks(Q), blocks(P)
    for vq, vp in ((blocks(Q, room=9), blocks(P)), (blocks(Q), blocks(P, room=9))):
        for entry in ("rc_score_candidates", "rc_candidate_distances"):
            with pytest.raises(AssertionError):
                calls(kq, vq, kp, vp)[entry]()
    assert library.calls == []


@pytest.mark.parametrize("entry", ENTRIES)
def test_what_the_descriptor_covers_is_taken(library, entry):
    kq, kp = blocks(Q), blocks(P)
    calls(kq, blocks(Q), kp, blocks(P))[entry]()                   # just like K
    calls(kq, blocks(Q + 1), kp, blocks(P + 2))[entry]()           # more blocks at the same strides
    calls(kq, blocks(Q, layers=L + 1), kp, blocks(P))[entry]()     # more layers
    assert library.calls == [entry] * 3
