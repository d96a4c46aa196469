"""Block-table remap where several workgroups read a layer's table, at the edges of what one workgroup holds in LDS."""
import numpy as np
import pytest
import torch

from paper_2507_21433_amd import binding as rc

pytestmark = pytest.mark.gpu


# (layers, entries, blocks, query blocks, pool ids given, id range wider than the LDS table)
@pytest.mark.parametrize("L,RE,NB,Q,with_pids,wide", [
    (1, 1, 2, 1, False, False),
    (3, 4099, 301, 63, True, False),            # no vector access: odd entries, odd counts
    (2, 16384, 31744, 1024, False, False),      # one batch of entries; two full shares of the counts
    (2, 16388, 31748, 1025, True, False),       # one group more of each: the counts no longer fit
    (9, 49664, 50176, 4096, False, False),      # as many query blocks as there are targets in LDS; nine layers on eight XCDs
    (2, 30000, 33000, 4097, False, False),      # one query block more
    (1, 131072, 60000, 500, True, True),        # ids some 59 000 apart, a table too long for every workgroup to look them up
    (1, 131076, 60000, 500, False, True),
    (1, 49151, 20000, 20, False, False),        # entries one by one: the longest table that every workgroup reads, and the next
    (1, 49153, 20000, 20, False, False),
    (1, 32769, 20000, 15, True, False),         # few query blocks
    (2, 81919, 20000, 256, True, False),
    (2, 81921, 20000, 256, True, False),
    (1, 81920, 20000, 31, False, False),        # few query blocks, 16 bytes at a time
    (1, 81924, 20000, 31, False, False),
    (130, 700, 15872, 40, True, False),         # a workgroup per layer, a full share of the counts
    (130, 701, 15873, 40, False, False),
])
@pytest.mark.parametrize("in_place", [False, True])
def test_remap_layers(oracle, L, RE, NB, Q, with_pids, wide, in_place):
    rng = np.random.RandomState(L * 1000 + RE % 997 + Q)
    if with_pids:                                                 # targets anywhere, never a query block
        ids = rng.permutation(NB).astype(np.int32)
        qids, pids = ids[:Q], ids[Q:]
        P = pids.size
    else:
        P = 50 if wide else NB - Q
        qids, pids = np.sort(rng.permutation(np.arange(P, NB, dtype=np.int32))[:Q]), None
    match = rng.randint(-2, P + 2, (L, Q)).astype(np.int32)
    match[:, ::7] = match[:, :1]                                  # many query blocks onto one target
    tables = rng.randint(-1, NB + 1, (L, 1, RE)).astype(np.int32)
    some = rng.random_sample(tables.shape) < 0.4
    tables[some] = rng.choice(qids, int(some.sum()))
    refcount = rng.randint(0, 4, (L, NB)).astype(np.int32)
    t = lambda a: None if a is None else torch.as_tensor(a, device="cuda:0").contiguous()
    print(f"remap layers L={L} RE={RE} NB={NB} Q={Q} in_place={in_place}", flush=True)
    g = rc.rc_remap_block_table(t(tables), t(qids), t(pids), t(match), P, NB, t(refcount), in_place=in_place)
    torch.cuda.synchronize()
    o = oracle.remap(tables, qids, pids, match, P, NB, refcount)
    for k in ("tables", "refcount", "freed", "n_remapped"):
        np.testing.assert_array_equal(g[k].cpu().numpy(), o[k], err_msg=k)


# long tables over few blocks: with the counts dealt out in fours, the last workgroups of a layer own none (the share of one
# starts exactly at the end: 17 x 4 blocks, 16 workgroups and more); most entries are padding
@pytest.mark.parametrize("L,RE,NB,Q", [(1, 131072, 3460, 500), (8, 131072, 1025, 200), (1, 100000, 2113, 63), (16, 65536, 897, 100),
                                       (1, 49152, 433, 16), (64, 49664, 33, 16), (2, 16384, 33, 8), (1, 131072, 68, 30), (1, 131072, 3843, 700)])
@pytest.mark.parametrize("with_pids", [False, True])
def test_remap_few_blocks(oracle, L, RE, NB, Q, with_pids):
    rng = np.random.RandomState(NB + Q)
    ids = rng.permutation(NB).astype(np.int32)
    if with_pids:
        qids, pids, P = ids[:Q], ids[Q:], NB - Q
    else:
        qids, pids, P = np.arange(NB - Q, NB, dtype=np.int32), None, NB - Q
    match = rng.randint(-1, P, (L, Q)).astype(np.int32)
    tables = np.where(rng.random_sample((L, 1, RE)) < 0.1, rng.randint(0, NB, (L, 1, RE)), -1).astype(np.int32)
    refcount = np.stack([np.bincount(t[t >= 0], minlength=NB) for t in tables.reshape(L, RE)]).astype(np.int32)
    refcount += rng.randint(0, 2, refcount.shape).astype(np.int32)        # references left, and gone
    t = lambda a: None if a is None else torch.as_tensor(a, device="cuda:0").contiguous()
    print(f"remap few blocks L={L} RE={RE} NB={NB} Q={Q} pids={with_pids}", flush=True)
    g = rc.rc_remap_block_table(t(tables), t(qids), t(pids), t(match), P, NB, t(refcount))
    torch.cuda.synchronize()
    o = oracle.remap(tables, qids, pids, match, P, NB, refcount)
    assert 0 < o["freed"].sum() < (match >= 0).sum()
    for k in ("tables", "refcount", "freed", "n_remapped"):
        np.testing.assert_array_equal(g[k].cpu().numpy(), o[k], err_msg=k)


# query blocks further apart than the 16-bit table of slots reaches: as many as the hash table takes; odd sizes; ids that all
# fall on the last places of the hash table, so that searches are long and wrap around
@pytest.mark.parametrize("L,RE,NB,Q,collide", [(1, 98304, 60000, 4096, False), (1, 98308, 60000, 500, False), (8, 49152, 50176, 1024, False),
                                               (3, 30001, 45001, 63, False), (64, 12288, 33000, 2, False), (1, 98304, 380000, 4096, True)])
def test_remap_scattered_ids(oracle, L, RE, NB, Q, collide):
    rng = np.random.RandomState(NB + Q)
    ids = np.arange(1, NB - 1, dtype=np.int64)
    if collide:
        place = (ids * 0x9E3779 % (1 << 32)) >> (32 - 14)
        ids = ids[np.argsort(-place, kind="stable")]
        assert place.max() == 16383 and np.unique((np.sort(-place))[:Q]).size < 200
    else:
        ids = rng.permutation(ids)
    qids, pids = ids[:Q].astype(np.int32), ids[Q:].astype(np.int32)
    qids[:2] = 0, NB - 1
    P = pids.size
    match = rng.randint(-1, P, (L, Q)).astype(np.int32)
    match[:, :2] = [0, 3]                                         # both ends of the range are matched
    tables = rng.randint(-1, NB + 1, (L, 1, RE)).astype(np.int32)
    some = rng.random_sample(tables.shape) < 0.4
    tables[some] = rng.choice(qids, int(some.sum()))
    refcount = rng.randint(0, 4, (L, NB)).astype(np.int32)
    t = lambda a: torch.as_tensor(a, device="cuda:0").contiguous()
    print(f"remap scattered ids L={L} RE={RE} NB={NB} Q={Q}", flush=True)
    g = rc.rc_remap_block_table(t(tables), t(qids), t(pids), t(match), P, NB, t(refcount))
    torch.cuda.synchronize()
    o = oracle.remap(tables, qids, pids, match, P, NB, refcount)
    for k in ("tables", "refcount", "freed", "n_remapped"):
        np.testing.assert_array_equal(g[k].cpu().numpy(), o[k], err_msg=k)
