"""What this library is timed on: the calls that a serving engine makes to it, at the sizes it makes them with.

A case is a dict of plain values; `prepare` makes what the engine holds before the call (KV blocks, cached norms of the
pool, tables, workspaces, output buffers), `run` is one pass through the public entry points of
`paper_2507_21433_amd.binding`, and `work` and `tolerance` say what the pass cannot do without and how far apart two
correct results may be.

Five kinds of pass:
  step        one decoding or prefill step of the per-layer search: norms of the new blocks, exhaustive search over
              the resident pool, block tables rewritten (block score or per-head score)
  capacity    one step of the steady-state loop on a full pool with the paper's own layer-mean measure: norms, search,
              decision, tables, stamps, released references, eviction, admission
  candidates  one step in which only listed candidates are scored, layer by layer
  listed      the step that closes the warm-up: layer-mean distances of listed candidates, the percentile of the
              distances collected so far, the decision against it, a layer-shared table rewritten
  tables      the block tables of all layers rewritten for decisions that are already there
"""
import math

import numpy as np
import torch

from paper_2507_21433_amd import binding as rc
from paper_2507_21433_amd import synth

DEV = "cuda:0"
HEAD_DIM = 128
BLOCKS_PER_REQUEST = 775        # 12.4k tokens in blocks of 16


def _case(name, kind, L, P, Q, T=16, H=8, dtype="f16", mode=0, clustered=False, C=0, samples=0):
    c = dict(kind=kind, L=L, P=P, Q=Q, T=T, H=H, dtype=dtype, mode=mode, clustered=clustered, C=C, samples=samples)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one layer, one short request: the smallest call there is, three launches' worth of latency
        _case("tiny_step", "step", 1, 256, 32),
        # an engine that hooks into every layer calls for one layer at a time; a request's sealed blocks of one step
        _case("layer_call", "step", 1, 4096, 16),
        # decoding: five requests' caches, a handful of them seal blocks in this step; nothing is a round number
        _case("decode_step", "step", 64, 5 * BLOCKS_PER_REQUEST + 2, 40),
        # the benchmark's decoding step of a 64-layer model
        _case("qwq_step", "step", 64, 4096, 256),
        # ten KV heads, bf16, sizes that fit no tile
        _case("ragged_step", "step", 40, 8 * BLOCKS_PER_REQUEST + 1, 300, H=10, dtype="bf16"),
        # high concurrency, clustered near-duplicates: the largest search (half the layers of the benchmark's workload)
        _case("clustered_step", "step", 32, 16384, 1024, dtype="bf16", clustered=True),
        # per-head decisions, blocks of 32 tokens: the benchmark's small model
        _case("head_step", "step", 32, 8192, 512, T=32, mode=1),
        # per-head decisions while decoding
        _case("head_decode", "step", 32, 2531, 24, T=32, dtype="bf16", mode=1),
        # the steady-state loop at capacity
        _case("capacity_step", "capacity", 64, 2048, 128),
        # the paper's shape of Stage 2: a few candidates per new block, per layer ...
        _case("candidates", "candidates", 64, 4096, 256, C=16),
        # ... and with one list for all layers, at the end of the warm-up
        _case("listed_warmup", "listed", 48, 3100, 96, H=10, dtype="bf16", C=12, samples=1 << 20),
        # tables of 64 requests of 776 entries, 64 layers
        _case("tables", "tables", 64, 49152, 1024),
    ]


def _log_uniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the listed ranges: 1 to 64 layers, 64 to 16384 resident blocks, 1 to 1024 new ones, 4 to 16 KV
    heads, blocks of 16 or 32 tokens, fp16 or bf16; never more KV or more matrix work than the largest listed case."""
    kind = rng.choice(["step", "step", "step", "heads", "heads", "capacity", "candidates", "listed", "tables"])
    while True:
        L, P, Q = _log_uniform(rng, 1, 64), _log_uniform(rng, 64, 16384), _log_uniform(rng, 1, 1024)
        T, H = rng.choice([16, 16, 32]), rng.choice([4, 8, 8, 10, 16])
        dtype = rng.choice(["f16", "bf16"])
        if Q > P // 2:
            continue
        if kind == "tables":
            return _case(None, "tables", L, _log_uniform(rng, max(1024, 2 * Q), 49152), Q)
        block = 4 * T * H * HEAD_DIM
        if L * (P + Q) * block > (10e9 if kind == "capacity" else 72e9) or 2.0 * block // 2 * L * P * Q * 2 > 3.4e13:
            continue
        if kind == "heads":
            return _case(None, "step", L, P, Q, T, H, dtype, mode=1)
        if kind == "candidates" or kind == "listed":
            C = rng.randint(1, 24)
            if L * Q * C * block > 60e9:
                continue
            return _case(None, kind, L, P, Q, T, H, dtype, C=C, samples=_log_uniform(rng, 1000, 1 << 22) if kind == "listed" else 0)
        return _case(None, kind, L, P, Q, T, H, dtype, clustered=kind == "step" and P >= 1024 and rng.random() < 0.25)


# ---------------------------------------------------------------------------------------------------------------------

def _tables_shape(P, Q):
    """Requests and entries per request of the block tables: each request lists its share of the pool and its new blocks."""
    R = max(1, min(64, Q // 8))
    return R, P // R + Q // R


def _workload(c, seed):
    R, E = _tables_shape(c["P"], c["Q"])
    return synth.Workload("case", L=c["L"], P=c["P"], Q=c["Q"], T=c["T"], H=c["H"], dtype=c["dtype"], mode=c["mode"],
                          tau=0.9 if c["clustered"] else 0.95, seed=int(seed) % (1 << 31),
                          recipe="clustered" if c["clustered"] else "planted", n_centroids=128 if c["clustered"] else 0,
                          planted_frac=0.3, sigma=0.1 if c["mode"] else 0.15, head_subset_noise=bool(c["mode"]), R=R, E=E)


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEV)


def _scratch(nbytes):
    return _empty(max(16, int(nbytes)), torch.uint8)


def _remap_buffers(tables, refcount, Q):
    L, R, E = tables.shape
    NB = refcount.shape[1]
    return dict(ws=_scratch(rc.rc_remap_workspace_size(L, R, E, Q, NB)),
                out=dict(tables=torch.empty_like(tables), refcount=torch.empty_like(refcount),
                         freed=_empty((L, Q), torch.uint8), n_remapped=_empty((L,), torch.int32)))


def _norm_buffers(c):
    shape = (c["L"], c["Q"]) if c["mode"] == 0 else (c["L"], c["Q"], c["H"])
    return _empty(shape, torch.float32), _empty(shape, torch.float32)


def prepare(case, seed):
    return dict(dict(step=_prepare_step, capacity=_prepare_capacity, candidates=_prepare_candidates, listed=_prepare_listed,
                     tables=_prepare_tables)[case["kind"]](case, seed), case=case)


def run(state):
    return dict(step=_run_step, capacity=_run_capacity, candidates=_run_candidates, listed=_run_listed,
                tables=_run_tables)[state["case"]["kind"]](state)


# ---- step

def _prepare_step(c, seed):
    L, P, Q = c["L"], c["P"], c["Q"]
    w = _workload(c, seed)
    pr = synth.make_problem(w, DEV)
    # one resident block in a hundred is sealed but no longer referenced
    rng = np.random.RandomState(int(seed) % (1 << 31))
    pr["live"][:, torch.as_tensor(rng.choice(P, P // 100, replace=False), device=DEV)] = 0
    pk, pv = rc.rc_block_norms(pr["kp"], pr["vp"], w.mode)
    qk, qv = _norm_buffers(c)
    return dict(pr=pr, tau=w.tau, mode=w.mode, pk=pk, pv=pv, qk=qk, qv=qv, ws=_scratch(rc.rc_match_workspace_size(pr["kq"], w.mode, Q, P)),
                out=dict(best_idx=_empty((L, Q), torch.int32), best_score=_empty((L, Q), torch.float32),
                         match_idx=_empty((L, Q), torch.int32), second_score=_empty((L, Q), torch.float32)),
                remap=_remap_buffers(pr["tables"], pr["refcount"], Q))


def _run_step(s):
    c, pr = s["case"], s["pr"]
    qk, qv = rc.rc_block_norms(pr["kq"], pr["vq"], s["mode"], s["qk"], s["qv"])
    m = rc.rc_match_blocks(pr["kq"], pr["vq"], qk, qv, pr["kp"], pr["vp"], s["pk"], s["pv"], pr["live"], s["tau"], s["mode"],
                           workspace=s["ws"], out=s["out"])
    r = rc.rc_remap_block_table(pr["tables"], pr["query_ids"], None, m["match_idx"], c["P"], c["P"] + c["Q"], pr["refcount"],
                                workspace=s["remap"]["ws"], out=s["remap"]["out"])
    return dict(k_sqnorm=qk, v_sqnorm=qv, match=m, remap=r)


# ---- steady-state loop on a full pool

def _prepare_capacity(c, seed):
    """A pool without a free slot and two batches of new blocks, three in ten of them near-copies of resident blocks.

    The passes take the batches in turn.  The request whose blocks were admitted by one pass has ended when the next
    begins: its references are released, its blocks are the ones that make room, and the pool is as full as before."""
    L, P, Q, T, H = (c[n] for n in ("L", "P", "Q", "T", "H"))
    dt = torch.float16 if c["dtype"] == "f16" else torch.bfloat16
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1_000_003 + 29)
    copies = int(round(0.3 * Q))

    def blocks(n):
        t = _empty((L, n, T, H, HEAD_DIM), dt)
        for l in range(L):
            t[l].copy_(torch.randn((n, T, H, HEAD_DIM), generator=g, device=DEV))
        return t

    kp, vp = blocks(P), blocks(P)
    batches = []
    for _ in range(2):
        kq, vq = blocks(Q), blocks(Q)
        # the copied blocks belong to requests that are still running: not the last Q slots, which change hands
        src = torch.randperm(P - Q, generator=g, device=DEV)[:copies]
        dst = torch.randperm(Q, generator=g, device=DEV)[:copies]
        for q, p in ((kq, kp), (vq, vp)):
            for l in range(L):
                noise = torch.randn((copies, T, H, HEAD_DIM), generator=g, device=DEV)
                q[l, dst] = (p[l, src].float() + 0.15 * noise).to(dt)
        batches.append((kq, vq))
    pk, pv = rc.rc_block_norms(kp, vp)
    qk, qv = _norm_buffers(c)
    ids = torch.arange(P, P + Q, dtype=torch.int32, device=DEV)
    table, refcount = ids.reshape(1, 1, Q).contiguous(), torch.ones((1, P + Q), dtype=torch.int32, device=DEV)
    ended = torch.full((Q,), -1, dtype=torch.int32, device=DEV)
    ended[:Q - copies] = torch.arange(P - (Q - copies), P, dtype=torch.int32, device=DEV)
    slots = [_empty((Q,), torch.int32), ended]
    decisions = [_empty((Q,), torch.int32), torch.full((Q,), -1, dtype=torch.int32, device=DEV)]
    return dict(
        batches=batches, kp=kp, vp=vp, pk=pk, pv=pv, qk=qk, qv=qv, step=0, ids=ids, table=table, refcount=refcount,
        live=torch.ones(P, dtype=torch.uint8, device=DEV), stamp=torch.zeros(P, dtype=torch.int32, device=DEV),
        # between the distance of a near-copy (noise 0.15) and that of an unrelated block (sqrt 2), in the measure's unit
        threshold=torch.full((1,), 0.6 * math.sqrt(HEAD_DIM / (T * H)), dtype=torch.float32, device=DEV),
        slots=slots, decisions=decisions, ws_search=_scratch(rc.rc_layer_mean_workspace_size(batches[0][0], Q, P)),
        ws_admit=_scratch(rc.lib().rc_pool_admit_workspace_size(Q, P)), remap=_remap_buffers(table, refcount, Q),
        search=dict(best_idx=_empty((Q,), torch.int32), best_dist=_empty((Q,), torch.float32),
                    match_idx=_empty((Q,), torch.int32), second_dist=_empty((Q,), torch.float32)),
        evicted=dict(n_free=_empty((1,), torch.int32), n_evicted=_empty((1,), torch.int32)), n_admitted=_empty((1,), torch.int32))


def _run_capacity(s):
    P, Q = s["case"]["P"], s["case"]["Q"]
    now, before = s["step"] % 2, (s["step"] + 1) % 2
    s["step"] += 1
    kq, vq = s["batches"][now]
    decision, slots = s["decisions"][now], s["slots"][now]
    qk, qv = rc.rc_block_norms(kq, vq, k_sqnorm=s["qk"], v_sqnorm=s["qv"])
    m = rc.rc_match_blocks_layer_mean(kq, vq, qk, qv, s["kp"], s["vp"], s["pk"], s["pv"], s["live"], math.inf,
                                      workspace=s["ws_search"], out=s["search"])
    rc.rc_apply_threshold(m["best_idx"], m["best_dist"], s["threshold"], decision)
    r = rc.rc_remap_block_table(s["table"], s["ids"], None, decision.reshape(1, Q), P, P + Q, s["refcount"],
                                workspace=s["remap"]["ws"], out=s["remap"]["out"])
    held = r["refcount"][0, :P]
    rc.rc_pool_touch(decision, s["step"], s["stamp"])
    rc.rc_refcount_release(s["slots"][before], held)
    rc.rc_refcount_release(s["decisions"][before], held)
    e = rc.rc_pool_evict(s["live"], held, s["stamp"], decision, out=s["evicted"])
    a = rc.rc_pool_admit(kq, vq, qk, qv, s["kp"], s["vp"], s["pk"], s["pv"], s["live"], decision, workspace=s["ws_admit"],
                         out=dict(slot_of_query=slots, n_admitted=s["n_admitted"]))
    rc.rc_pool_touch(slots, s["step"], s["stamp"])
    rc.rc_pool_touch(slots, 1, held)
    s["refcount"][0, :P].copy_(held)
    return dict(k_sqnorm=qk, v_sqnorm=qv, match=m, decision=decision, remap=r, evicted=e, admitted=a, kp=s["kp"], vp=s["vp"],
                pk=s["pk"], pv=s["pv"], live=s["live"], stamp=s["stamp"], refcount=s["refcount"])


# ---- listed candidates

def _prepare_candidates(c, seed):
    L, P, Q, C = c["L"], c["P"], c["Q"], c["C"]
    w = _workload(c, seed)
    pr = synth.make_problem(w, DEV)
    pk, pv = rc.rc_block_norms(pr["kp"], pr["vp"])
    qk, qv = _norm_buffers(c)
    return dict(pr=pr, tau=w.tau, pk=pk, pv=pv, qk=qk, qv=qv, cand=_lists(pr, (L, Q, C), P, seed),
                out=dict(scores=_empty((L, Q, C), torch.float32), best_idx=_empty((L, Q), torch.int32),
                         best_score=_empty((L, Q), torch.float32), match_idx=_empty((L, Q), torch.int32)))


def _lists(pr, shape, P, seed):
    """Candidate lists: random blocks, the true partner where there is one, one slot in twenty empty."""
    rng = np.random.RandomState((int(seed) + 7) % (1 << 31))
    cand = rng.randint(0, P, size=shape).astype(np.int32)
    cand[rng.random_sample(shape) < 0.05] = -1
    plan = pr["plan"]
    cand[..., plan.planted_slots, rng.randint(0, shape[-1], size=plan.planted_slots.size)] = plan.planted_targets
    return torch.as_tensor(cand, device=DEV)


def _run_candidates(s):
    pr = s["pr"]
    qk, qv = rc.rc_block_norms(pr["kq"], pr["vq"], k_sqnorm=s["qk"], v_sqnorm=s["qv"])
    m = rc.rc_score_candidates(pr["kq"], pr["vq"], qk, qv, pr["kp"], pr["vp"], s["pk"], s["pv"], pr["live"], s["cand"], s["tau"],
                               out=s["out"])
    return dict(k_sqnorm=qk, v_sqnorm=qv, match=m)


def _prepare_listed(c, seed):
    L, P, Q, C, n = c["L"], c["P"], c["Q"], c["C"], c["samples"]
    pr = synth.make_problem(_workload(c, seed), DEV)
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 3)
    # distances collected so far: near-duplicates and unrelated blocks form two clusters, one list in fifty had no candidate
    unit = math.sqrt(HEAD_DIM / (c["T"] * c["H"]))
    u = torch.rand(n, generator=g, device=DEV)
    near = 0.15 + 0.02 * torch.randn(n, generator=g, device=DEV)
    far = math.sqrt(2.0) + 0.01 * torch.randn(n, generator=g, device=DEV)
    samples = torch.where(u < 0.3, near, far) * unit
    samples[u > 0.98] = math.inf
    tables, refcount = pr["tables"][:1].contiguous(), pr["refcount"][:1].contiguous()
    return dict(pr=pr, samples=samples, cand=_lists(pr, (Q, C), P, seed), live=pr["live"][0].contiguous(), tables=tables,
                refcount=refcount, remap=_remap_buffers(tables, refcount, Q),
                ws=_scratch(rc.lib().rc_candidate_distances_workspace_size(rc.kv_desc(pr["kq"]), Q, C)),
                ws_pat=_scratch(rc.lib().rc_pat_workspace_size()),
                pat=dict(threshold=_empty((1,), torch.float32), n_finite=_empty((1,), torch.int64)),
                out=dict(dist=_empty((Q, C), torch.float32), best_idx=_empty((Q,), torch.int32),
                         best_dist=_empty((Q,), torch.float32), match_idx=_empty((Q,), torch.int32)),
                decision=_empty((Q,), torch.int32))


def _run_listed(s):
    c, pr = s["case"], s["pr"]
    P, Q = c["P"], c["Q"]
    m = rc.rc_candidate_distances(pr["kq"], pr["vq"], pr["kp"], pr["vp"], s["live"], s["cand"], -math.inf, workspace=s["ws"],
                                  out=s["out"])
    seen = min(Q, c["samples"])
    s["samples"][:seen].copy_(m["best_dist"][:seen])
    t = rc.rc_pat_threshold(s["samples"], 80.0, workspace=s["ws_pat"], out=s["pat"])
    rc.rc_apply_threshold(m["best_idx"], m["best_dist"], t["threshold"], s["decision"])
    r = rc.rc_remap_block_table(s["tables"], pr["query_ids"], None, s["decision"].reshape(1, Q), P, P + Q, s["refcount"],
                                workspace=s["remap"]["ws"], out=s["remap"]["out"])
    return dict(match=m, threshold=t, decision=s["decision"], remap=r)


# ---- tables

def _prepare_tables(c, seed):
    L, P, Q = c["L"], c["P"], c["Q"]
    R, E = _tables_shape(P, Q)
    plan = synth.make_plan(synth.Workload("case", L=L, P=P, Q=Q, seed=int(seed) % (1 << 31), R=R, E=E))
    rng = np.random.RandomState((int(seed) + 5) % (1 << 31))
    match = np.where(rng.random_sample((L, Q)) < 0.4, rng.randint(0, P, size=(L, Q)), -1).astype(np.int32)
    tables = torch.as_tensor(plan.tables, device=DEV)[None].repeat(L, 1, 1).contiguous()
    refcount = torch.as_tensor(plan.refcount, device=DEV)[None].repeat(L, 1).contiguous()
    return dict(tables=tables, refcount=refcount, query_ids=torch.as_tensor(plan.query_ids, device=DEV),
                match=torch.as_tensor(match, device=DEV), remap=_remap_buffers(tables, refcount, Q))


def _run_tables(s):
    c = s["case"]
    return rc.rc_remap_block_table(s["tables"], s["query_ids"], None, s["match"], c["P"], c["P"] + c["Q"], s["refcount"],
                                   workspace=s["remap"]["ws"], out=s["remap"]["out"])


# ---------------------------------------------------------------------------------------------------------------------

def work(case):
    """Bytes: every input read once, every output written once.  Operations: two dot products per scored pair and layer."""
    L, P, Q, C, n = (case[k] for k in ("L", "P", "Q", "C", "samples"))
    D = case["T"] * case["H"] * HEAD_DIM
    block = 4 * D                                    # a K and a V tensor of 16-bit values
    heads = case["H"] if case["mode"] else 1
    R, E = _tables_shape(P, Q)

    def remap(layers):
        return layers * (8 * R * E + 8 * (P + Q) + 5 * Q + 4) + 4 * Q

    norms = 8 * L * Q * heads                        # written once (and read by the search)
    if case["kind"] == "tables":
        return dict(bytes=remap(L), flops=0)
    if case["kind"] == "step":
        return dict(bytes=L * (P + Q) * block + norms + L * P * (8 * heads + 1) + 16 * L * Q + remap(L), flops=4.0 * D * L * P * Q)
    if case["kind"] == "capacity":
        admitted = Q - int(round(0.3 * Q))
        return dict(bytes=L * (P + Q + admitted) * block + norms + 8 * L * (P + admitted) + 16 * Q + 17 * P + 8 * (P + Q) + 24 * Q,
                    flops=4.0 * D * L * P * Q)
    pairs = 0.95 * L * Q * C
    pool = L * P * -math.expm1(0.95 * Q * C * math.log1p(-1.0 / P))   # a block that several lists name is read once
    if case["kind"] == "candidates":
        return dict(bytes=(pool + L * Q) * block + norms + 8 * pool + 8 * L * Q * C + 12 * L * Q, flops=4.0 * D * pairs)
    return dict(bytes=(pool + L * Q) * block + 8 * Q * C + 20 * Q + 4 * n + remap(1), flops=6.0 * D * pairs)


def tolerance(case):
    """About four times what the path differs by from itself in 64 bits: fp32 sums over 16-bit products are within 2e-7
    (fp16) to 9e-7 (bf16) of it, single values within 3.5e-6 of the root mean square.  The index of the best block may
    differ where two blocks are that close (clustered blocks: one in a thousand)."""
    if case["kind"] == "tables":
        return "exact"
    if case["mode"] == 1:
        # scores are on a grid of 1/32767: one that lies between two points of it goes to either, 3e-5 of a score of 0.01
        return {"rel": 1e-3, "max": 1e-2, "differ": 4e-3}
    if case["kind"] == "capacity":
        # |x|^2 + |y|^2 - 2 x.y of a near-copy (noise 0.15) is 1/45 of its terms
        return {"rel": 1e-5, "max": 1e-4, "differ": 2e-3}
    return {"rel": 4e-6, "max": 3e-5, "differ": 4e-3 if case["clustered"] else 2e-3}
