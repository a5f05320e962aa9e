"""Accumulator residency under a device-memory budget (hubs, eviction to
pinned host memory, reload) and host-resident chunks and outputs, on the GPU
(needs an MI355X)."""
import dataclasses
import sys

import numpy as np
import pytest

import fixtures as F
from fixtures import workloads as WL
from tests import harness as H

pytestmark = pytest.mark.gpu

PIECE = 512          # the library's hub-piece length (work units per long segment)


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _note(msg):
    print(f"[case] {msg}", flush=True)
    sys.stdout.flush()


def _max_chunk_destinations(src, dst, n, chunk):
    """Upper bound of the destinations one chunk touches: its work units
    (segments, long ones counted per piece) plus its own vertices."""
    key = (src.astype(np.int64) // chunk) * n + dst
    seg, lens = np.unique(key, return_counts=True)
    units = np.where(lens > 8, (lens + PIECE - 1) // PIECE, 1)
    per_chunk = np.bincount(seg // n, weights=units, minlength=(n + chunk - 1) // chunk)
    rows = np.minimum(chunk, n - np.arange(per_chunk.size) * chunk)
    return int((per_chunk + rows).max())


def _run(torch, w, row_off, col_dst, X, budget=0, hub_fraction=0.0):
    import paper_2607_17374_amd as T
    from paper_2607_17374_amd.api import torch_dtype
    outs, stats = [], []
    h = X
    for li, spec in enumerate(H.layer_specs(w), start=1):
        out = torch.empty((w.n, spec["d_out"]), dtype=torch_dtype(spec["out_dtype"]), device="cuda")
        b = budget[li - 1] if isinstance(budget, list) else budget
        L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, hbm_budget=b, hub_fraction=hub_fraction, **spec)
        L.push_all(h)
        stats.append(L.finalize())
        L.destroy()
        outs.append(out)
        h = out
    return outs, stats


def test_budget_eviction_matches_incore_c4_shape(torch_cuda):
    """C4's model (GraphSAGE-mean 512 -> 256 -> 128, fp32, U[-1,1) features,
    RMAT(.57,.19,.19), vertex IDs shuffled) at 1/2000 of the vertices, with 1% hub vertices and a
    budget that holds well under half of the accumulator rows: outputs equal
    the in-core run bit for bit, rows were evicted and reloaded, and sampled
    destinations match the oracle."""
    import oracle as O
    torch = torch_cuda
    # random vertex IDs: with natural RMAT IDs the first chunks alone touch
    # most vertices at this scale, leaving nothing to evict
    w = dataclasses.replace(WL.SAGE_OOC_RMAT_269M, random_ids=True).scaled(n=1 << 17, e=1 << 21, chunk=1024)
    _note(f"{w.name}: in core")
    src, dst = WL.graph(w)
    row_off, col_dst = H.gpu_graph(w, src, dst)
    X = torch.from_numpy(WL.input_features(w)).cuda()
    ref, ref_stats = _run(torch, w, row_off, col_dst, X)
    need = _max_chunk_destinations(src, dst, w.n, w.chunk)
    hubs = int(np.ceil(0.01 * w.n))
    slots = hubs + need + (w.n - hubs - need) // 4
    assert slots < w.n * 0.6, (need, slots)
    budgets = [H.pool_budget(s, w.n, spec["d_out"], spec["d_in"], w.chunk, slots)
               for s, spec in zip(ref_stats, H.layer_specs(w))]
    _note(f"  budgets {budgets} (slots {slots}, chunk destinations {need})")
    outs, stats = _run(torch, w, row_off, col_dst, X, budget=budgets, hub_fraction=0.01)
    for li, (a, b, st) in enumerate(zip(outs, ref, stats), start=1):
        assert torch.equal(a, b), li
        assert st["evictions"] > 0 and st["reloads"] > 0, st
        assert 0.0 < st["hub_message_share"] < 1.0
        assert st["d2h_bytes"] == st["evictions"] * w.dims[li] * 4
        assert st["device_bytes"] <= budgets[li - 1] + (1 << 20)
    # sampled destinations against the oracle, each layer fed the oracle's own previous layer
    g = O.Graph(w.n, src, dst)
    rng = np.random.default_rng(9)
    d_in = np.diff(g.in_off)
    ids = np.unique(np.concatenate([rng.choice(w.n, 1024, replace=False), np.argsort(-d_in, kind="stable")[:32],
                                    np.flatnonzero(d_in == 0)[:32]]))
    zs = H.oracle_sampled_layers(w, g, WL.input_features(w), [ids] * w.layers)
    for li, z in enumerate(zs, start=1):
        r = H.compare(outs[li - 1].cpu().numpy()[ids], z, H.RTOL[F.F32])
        assert r["n_bad"] == 0, (li, r)


@pytest.mark.parametrize("policy", ["pending", "random", "fifo", "lru"])
def test_eviction_policies_match_oracle_simulation(torch_cuda, policy):
    """Every eviction policy on the C4-shaped graph at 1/2000 with 1% hubs and
    a pool of about 35% of the rows: the output equals the in-core run bit for
    bit, and the evictions, reloads and per-vertex reload histogram equal the
    oracle's slot-level simulation of the same pool (integers, exactly)."""
    import oracle as O
    import paper_2607_17374_amd as T
    torch = torch_cuda
    w = dataclasses.replace(WL.SAGE_OOC_RMAT_269M, random_ids=True).scaled(n=1 << 17, e=1 << 21, chunk=1024)
    src, dst = WL.graph(w)
    _note(f"eviction {policy}: {w.name}")
    row_off, col_dst = H.gpu_graph(w, src, dst)
    X = torch.from_numpy(WL.input_features(w)).cuda()
    spec = H.layer_specs(w)[0]
    ref = torch.empty((w.n, spec["d_out"]), dtype=torch.float32, device="cuda")
    L = T.Layer(w.n, row_off, col_dst, out=ref, chunk=w.chunk, **spec)
    L.push_all(X)
    st0 = L.finalize()
    L.destroy()
    budget = H.pool_budget(st0, w.n, spec["d_out"], spec["d_in"], w.chunk, int(0.35 * w.n))
    out = torch.empty_like(ref)
    L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, hbm_budget=budget, hub_fraction=0.01,
                eviction=policy, **spec)
    L.push_all(X)
    st = L.finalize()
    hist = L.reload_histogram(64)
    L.destroy()
    assert torch.equal(out, ref)
    _note(f"  pool {st['pool_rows']} rows ({st['hub_rows']} hubs): {st['evictions']} evictions, "
          f"{st['reloads']} reloads")
    g = O.Graph(w.n, src, dst)
    ev, rl, per = O.residency_sim(g, w.chunk, st["pool_rows"], st["hub_rows"], policy, seed=w.seed)
    assert (st["evictions"], st["reloads"]) == (ev, rl) and ev > 0
    assert np.array_equal(hist, np.bincount(np.minimum(per, 63), minlength=64))


@pytest.mark.parametrize("share", [0.3, 0.4, 0.9])
def test_free_rows_reported_by_the_device(torch_cuda, share):
    """Pushes that wait for each chunk, so that the host has seen the device's
    count of free rows and takes the short path between evictions: the same
    output, evictions, reloads and histogram as the simulation, and as pushes
    queued at once."""
    import oracle as O
    import paper_2607_17374_amd as T
    torch = torch_cuda
    w = dataclasses.replace(WL.SAGE_OOC_RMAT_269M, random_ids=True).scaled(n=1 << 16, e=1 << 20, chunk=512)
    src, dst = WL.graph(w)
    _note(f"free rows reported: pool {share}")
    row_off, col_dst = H.gpu_graph(w, src, dst)
    X = torch.from_numpy(WL.input_features(w)).cuda()
    spec = H.layer_specs(w)[0]
    ref = torch.empty((w.n, spec["d_out"]), dtype=torch.float32, device="cuda")
    L = T.Layer(w.n, row_off, col_dst, out=ref, chunk=w.chunk, **spec)
    L.push_all(X)
    st0 = L.finalize()
    L.destroy()
    budget = H.pool_budget(st0, w.n, spec["d_out"], spec["d_in"], w.chunk, int(share * w.n))
    g = O.Graph(w.n, src, dst)
    for wait in (True, False):
        out = torch.empty_like(ref)
        L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, hbm_budget=budget, hub_fraction=0.01, **spec)
        for b in range(0, w.n, w.chunk):
            L.push_chunk(b, min(w.n, b + w.chunk), X[b:b + w.chunk])
            if wait:
                torch.cuda.synchronize()
        st = L.finalize()
        hist = L.reload_histogram(64)
        L.destroy()
        assert torch.equal(out, ref)
        _note(f"  pool {st['pool_rows']} rows: {st['evictions']} evictions, {st['reloads']} reloads")
        ev, rl, per = O.residency_sim(g, w.chunk, st["pool_rows"], st["hub_rows"], "pending")
        assert (st["evictions"], st["reloads"]) == (ev, rl)
        assert np.array_equal(hist, np.bincount(np.minimum(per, 63), minlength=64))


def test_completion_lists_do_not_count_in_a_budget(torch_cuda):
    """A GIN perceptron layer leaves its completion lists in the plan's chunk
    index: a budgeted layer over the same plan has the pool it had before."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    w = WL.SAGE_OOC_RMAT_269M.scaled(n=1 << 16, e=1 << 19, chunk=512)
    row_off, col_dst = H.gpu_graph(w)
    X = torch.from_numpy(WL.input_features(w)).cuda()
    spec = H.layer_specs(w)[0]
    out = torch.empty((w.n, spec["d_out"]), device="cuda")
    plan = T.Plan(w.n, row_off, col_dst, w.chunk)

    def run(**kw):
        L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, plan=plan, **{**spec, **kw})
        L.push_all(X)
        st = L.finalize()
        L.destroy()
        return st

    budget = H.pool_budget(run(), w.n, spec["d_out"], spec["d_in"], w.chunk, int(0.4 * w.n))
    pool = run(hbm_budget=budget, hub_fraction=0.01)["pool_rows"]
    rng = np.random.default_rng(1)
    d = spec["d_out"]
    run(agg=4, d_hidden=d, weight_cat=rng.uniform(-0.1, 0.1, (spec["d_in"], d)).astype(np.float32),
        weight2=rng.uniform(-0.1, 0.1, (d, d)).astype(np.float32))
    assert run(hbm_budget=budget, hub_fraction=0.01)["pool_rows"] == pool > 0
    plan.destroy()


def big_pending_graph(groups=4, per=4, chunks_per_group=48, chunk=512, seed=3):
    """16 destinations with 13,500-24,600 in-edges each: chunk k's sources
    send to the 4 destinations of group k mod 4, destination j keeping each
    such edge with probability 1 - 0.03 j.  A pool of a few rows beyond one
    chunk's 516 destinations must evict destinations of the other groups,
    most of them with 16,383 or more pending messages early on."""
    rng = np.random.default_rng(seed)
    nch = groups * chunks_per_group
    n = nch * chunk
    nb = groups * per
    big = (np.arange(nb) * (n // nb) + 7).astype(np.int64)
    srcs, dsts = [], []
    for k in range(nch):
        gi = k % groups
        u = np.arange(k * chunk, (k + 1) * chunk)
        for j in range(per):
            b = big[gi * per + j]
            keep = rng.random(chunk) < 1.0 - 0.03 * (gi * per + j)
            uu = u[keep]
            uu = uu[uu != b]
            srcs.append(uu)
            dsts.append(np.full(uu.size, b))
    return n, chunk, np.concatenate(srcs).astype(np.int32), np.concatenate(dsts).astype(np.int32)


def test_fewest_pending_exact_above_histogram_range(torch_cuda):
    """Fewest-pending eviction ranks candidates by their exact pending count
    (Sec. 3.5.3) also where the counts pass the kernel's 14-bit histogram:
    the per-vertex reload histogram and totals equal the oracle's
    simulation, whose victims differ from those of capped counts on this
    graph at pools of 518-524 rows."""
    import oracle as O
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk, src, dst = big_pending_graph()
    _note(f"eviction above the histogram range: n={n} e={src.size}")
    s_d = torch.from_numpy(src).cuda()
    d_d = torch.from_numpy(dst).cuda()
    row_off, col_dst = T.build_csr(n, s_d, d_d)
    rng = np.random.default_rng(11)
    # wide rows, so that a pool of a few hundred rows is far below the dense
    # accumulators and the layer runs under its budget
    d_in, d = 16, 256
    X = torch.from_numpy(rng.uniform(-1, 1, (n, d_in)).astype(np.float32)).cuda()
    spec = dict(agg=O.SAGE_MEAN, d_in=d_in, d_out=d,
                weight_cat=rng.uniform(-0.3, 0.3, (d_in, 2 * d)).astype(np.float32),
                bias=np.zeros(d, np.float32), relu=False)
    ref = torch.empty((n, d), dtype=torch.float32, device="cuda")
    L = T.Layer(n, row_off, col_dst, out=ref, chunk=chunk, **spec)
    L.push_all(X)
    st0 = L.finalize()
    L.destroy()
    g = O.Graph(n, src, dst)
    checked = 0
    budget = H.pool_budget(st0, n, d, d_in, chunk, 520)
    for attempt in range(4):
        out = torch.empty_like(ref)
        L = T.Layer(n, row_off, col_dst, out=out, chunk=chunk, hbm_budget=budget, hub_fraction=0.0,
                    eviction="pending", **spec)
        L.push_all(X)
        st = L.finalize()
        hist = L.reload_histogram(64)
        L.destroy()
        S = st["pool_rows"]
        _note(f"  budget {budget}: pool {S} rows, {st['evictions']} evictions, {st['reloads']} reloads")
        assert S > 0, "the layer did not run under its budget"
        assert torch.equal(out, ref)
        ev, rl, per = O.residency_sim(g, chunk, S, 0, "pending")
        assert (st["evictions"], st["reloads"]) == (ev, rl)
        assert np.array_equal(hist, np.bincount(np.minimum(per, 63), minlength=64))
        if 518 <= S <= 524 and ev > 0:
            checked += 1
            break
        # move the pool toward 520 rows (each row costs d_out * 4 + 4 bytes, planned with 1/8 room)
        budget += (520 - S) * (d * 4 + 4) * 9 // 8
    assert checked > 0


def test_host_chunks_and_host_outputs(torch_cuda):
    """Chunks in pinned host memory (staged on the layer's copy stream) and
    outputs written straight into pinned host memory give the device run's
    values bit for bit."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    w = WL.SAGE_RMAT_4K
    _note("host chunks / host outputs")
    row_off, col_dst = H.gpu_graph(w)
    xh = torch.from_numpy(WL.input_features(w))
    X = xh.cuda()
    Xp = xh.pin_memory()
    spec = H.layer_specs(w)[0]
    ref = torch.empty((w.n, spec["d_out"]), dtype=torch.float32, device="cuda")
    L = T.Layer(w.n, row_off, col_dst, out=ref, chunk=w.chunk, **spec)
    L.push_all(X)
    L.finalize()
    L.destroy()
    out_h = torch.empty((w.n, spec["d_out"]), dtype=torch.float32).pin_memory()
    L = T.Layer(w.n, row_off, col_dst, out=out_h, chunk=w.chunk, **spec)
    L.push_all(Xp)
    st = L.finalize()
    L.destroy()
    assert torch.equal(out_h, ref.cpu())
    assert st["h2d_bytes"] == w.n * spec["d_in"] * 4
    assert st["d2h_bytes"] == w.n * spec["d_out"] * 4
    # pageable host memory is refused
    with pytest.raises(ValueError):
        T.Layer(w.n, row_off, col_dst, out=torch.empty((w.n, spec["d_out"])), chunk=w.chunk, **spec)


def test_budget_errors(torch_cuda):
    import paper_2607_17374_amd as T
    torch = torch_cuda
    w = WL.SAGE_RMAT_4K
    _note("budget errors")
    row_off, col_dst = H.gpu_graph(w)
    spec = H.layer_specs(w)[0]
    out = torch.empty((w.n, spec["d_out"]), dtype=torch.float32, device="cuda")
    L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, **spec)
    L.push_all(torch.from_numpy(WL.input_features(w)).cuda())
    incore = L.finalize()["device_bytes"]
    L.destroy()
    half = incore - w.n * spec["d_out"] * 4 // 2      # the pool, not the dense rows: half the rows at most
    for bad in (dict(hbm_budget=1 << 20), dict(hbm_budget=half, hub_fraction=0.9)):
        with pytest.raises(T.TaurusError) as ex:
            T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, **dict(spec, **bad))
        assert ex.value.status == -6, bad
    for bad in (dict(hub_fraction=1.5), dict(eviction=7), dict(eviction=-1)):
        with pytest.raises(T.TaurusError) as ex:
            T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, **dict(spec, **bad))
        assert ex.value.status == -1, bad
    # an in-core layer reports no reloads
    L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, **spec)
    assert L.reload_histogram(4).tolist() == [w.n, 0, 0, 0]
    L.destroy()


def test_release_cached_memory(torch_cuda):
    """A destroyed layer's buffers stay cached for the next layer; releasing
    hands them back to the runtime (partly: at least the bytes asked for,
    smallest blocks first), and a second full release finds nothing."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    w = WL.SAGE_RMAT_4K
    _note("release cached memory")
    row_off, col_dst = H.gpu_graph(w)
    spec = H.layer_specs(w)[0]
    out = torch.empty((w.n, spec["d_out"]), dtype=torch.float32, device="cuda")
    L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, **spec)
    L.push_all(torch.from_numpy(WL.input_features(w)).cuda())
    L.finalize()
    L.destroy()
    part = T.release_cached_memory(4096)
    assert part >= 4096
    rest = T.release_cached_memory(0)
    assert rest > 0 and T.release_cached_memory(0) == 0
    # the next layer allocates afresh and still works
    L = T.Layer(w.n, row_off, col_dst, out=out, chunk=w.chunk, **spec)
    L.push_all(torch.from_numpy(WL.input_features(w)).cuda())
    L.finalize()
    L.destroy()
