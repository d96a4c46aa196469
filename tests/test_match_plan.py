"""Shares of a search's tiles against timed calls (CPU only: the plan is plain C++): the estimate may take another number of shares
than the older rules only where that number was not slower.  L, T, H, P, Q, us per call of every number of shares (1 = whole tiles)."""
import pytest

from tests import plans

# the layer mean, near a full round of whole tiles, which are a kernel of their own, 256 rows high at every query count
MEAN_WHOLE = [
    (51, 16, 4, 899, 3, {1: 297, 2: 422, 4: 439, 6: 410, 8: 421, 10: 425}),
    (63, 16, 8, 870, 16, {1: 562, 2: 673, 4: 695, 6: 709, 8: 698}),
    (6, 16, 8, 9904, 1, {1: 640, 2: 672, 4: 683, 6: 706, 8: 703}),
    (40, 16, 8, 1071, 66, {1: 593, 2: 686, 4: 686, 6: 683, 8: 707, 10: 696}),
    (27, 16, 8, 1946, 73, {1: 631, 2: 707, 4: 720, 6: 772, 8: 767}),
    (54, 16, 10, 922, 124, {1: 906, 2: 993, 4: 1094, 6: 1122, 8: 1126, 10: 1147}),
    (44, 16, 4, 1243, 111, {1: 373, 2: 454, 4: 484, 6: 495, 8: 497, 10: 579}),
    (2, 32, 8, 15486, 458, {1: 1770, 2: 1858, 4: 1902, 6: 2018, 8: 1986}),
    (7, 16, 16, 2094, 534, {1: 1184, 4: 1379}),      # three query tiles share the pool slices
    (2, 16, 10, 4751, 905, {1: 984, 2: 952, 4: 828, 6: 820, 8: 833, 10: 963, 12: 1022}),
]
# the layer mean with few layers, whose shares cost less to add than with many
MEAN_FEW_LAYERS = [
    (2, 16, 8, 5750, 16, {1: 438, 2: 237, 4: 182, 6: 194, 8: 164, 10: 163, 12: 170, 14: 165, 16: 153, 20: 167}),
    (6, 16, 8, 1894, 24, {1: 422, 2: 235, 4: 176, 6: 212, 8: 177, 10: 162, 12: 177, 14: 171, 16: 161, 20: 182}),
    (1, 16, 8, 11475, 20, {1: 447, 2: 236, 4: 170, 6: 212, 8: 181, 10: 158, 12: 174, 14: 167, 16: 156, 20: 177}),
    (4, 16, 4, 5958, 8, {1: 241, 2: 161, 4: 180, 6: 168, 8: 149, 10: 164, 12: 167, 14: 170, 16: 162}),
    (1, 16, 8, 899, 67, {1: 392, 16: 57, 20: 53, 24: 50, 32: 49, 36: 49, 48: 47, 64: 47}),
]
# 64 columns: layer mean or not; the estimate was too low for long shares
LONG_SHARES = [
    (False, 2, 16, 8, 8278, 42, {1: 452, 2: 294, 4: 285, 6: 246, 8: 251, 10: 235, 12: 244, 14: 238, 16: 236, 20: 268}),
    (False, 5, 32, 4, 3305, 16, {1: 453, 2: 295, 4: 276, 6: 237, 8: 234, 10: 228, 12: 229, 14: 221, 16: 230, 20: 238}),
    (False, 2, 16, 8, 9541, 20, {1: 448, 2: 294, 4: 302, 6: 250, 8: 271, 10: 241, 12: 259, 14: 272, 16: 257, 20: 276}),
    (True, 2, 16, 8, 8278, 42, {1: 451, 2: 302, 4: 290, 6: 254, 8: 240, 10: 249, 12: 251, 14: 247, 16: 244, 20: 275}),
    (True, 5, 32, 4, 3187, 39, {1: 458, 2: 298, 4: 241, 6: 250, 8: 234, 10: 231, 12: 241, 14: 237, 16: 242, 20: 263}),
]
# 256 columns, few tiles: a round that leaves most compute units idle is not that much shorter
FEW_TILES = [
    (True, 1, 16, 8, 427, 208, {1: 540, 32: 53, 34: 53, 64: 48}),
]


def check(mean, L, T, H, P, Q, us):
    new, old = plans.shares(mean, L, T, H, P, Q), plans.alike(L, T, H, P, Q)
    assert us[new] <= 1.03 * min(us[old], us[1]), f"{new} shares take {us[new]} us, {old} took {us[old]}"


@pytest.mark.parametrize("L,T,H,P,Q,us", MEAN_WHOLE)
def test_layer_mean_in_whole_tiles(L, T, H, P, Q, us):
    check(True, L, T, H, P, Q, us)


@pytest.mark.parametrize("L,T,H,P,Q,us", MEAN_FEW_LAYERS)
def test_layer_mean_of_few_layers(L, T, H, P, Q, us):
    check(True, L, T, H, P, Q, us)


@pytest.mark.parametrize("mean,L,T,H,P,Q,us", LONG_SHARES)
def test_few_long_shares(mean, L, T, H, P, Q, us):
    check(mean, L, T, H, P, Q, us)


@pytest.mark.parametrize("mean,L,T,H,P,Q,us", FEW_TILES)
def test_few_tiles(mean, L, T, H, P, Q, us):
    check(mean, L, T, H, P, Q, us)


# A workspace without room for the chosen number of shares: the older rules' plan where that fits, and only then the least one.
@pytest.mark.parametrize("mean", [False, True])
def test_middling_workspace_takes_the_former_number(mean):
    L, T, H, P, Q = 7, 16, 10, 6134, 13
    new, old = plans.shares(mean, L, T, H, P, Q), plans.alike(L, T, H, P, Q)
    full, former = plans.need(mean, new, 64, L, P, Q), plans.need(mean, old, 64, L, P, Q)
    assert 1 < old < new and plans.least(mean, L, T, H, P, Q) < former < full
    for avail, want in ((full, new), (full - 16, old), (former, old), (former - 16, 1), (plans.least(mean, L, T, H, P, Q), 1)):
        assert plans.shares_in(avail, mean, L, T, H, P, Q)[0] == want


def test_least_workspace_keeps_the_columns_of_whole_tiles():
    L, T, H, P, Q = 128, 16, 10, 312, 129
    assert plans.shares(False, L, T, H, P, Q) > 1 == plans.alike(L, T, H, P, Q)
    least = plans.least(False, L, T, H, P, Q)
    assert least == plans.need(False, 1, 256, L, P, Q)
    assert plans.shares_in(least, False, L, T, H, P, Q) == (1, 192)      # not the 256 that pad 129 queries to twice their work
