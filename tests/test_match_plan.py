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
    (2, 16, 10, 4751, 905, {1: 984, 2: 952, 4: 828, 6: 820, 8: 833, 10: 963, 12: 1022}),
]


def check(mean, L, T, H, P, Q, us):
    new, old = plans.shares(mean, L, T, H, P, Q), plans.alike(L, T, H, P, Q)
    assert us[new] <= 1.03 * us[old], f"{new} shares take {us[new]} us, {old} took {us[old]}"


@pytest.mark.parametrize("L,T,H,P,Q,us", MEAN_WHOLE)
def test_layer_mean_in_whole_tiles(L, T, H, P, Q, us):
    check(True, L, T, H, P, Q, us)
