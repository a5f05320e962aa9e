"""Sampled layers kept in core (aggregated by destination) against
a 64-bit evaluation of the edges the layer says it keeps: widths at the edges
of the k-blocks and column groups, every family and type, lists of 0 to k
in-edges, partial pushes, host-fed chunks, values that are not finite.

Tolerance: fp32 outputs 2e-5 of the output's RMS per element -- a sum of at
most k = 64 messages and 256 products in fp32 errs by at most
(64 + 3 * 256) * 2^-24 = 5e-5 of the sum of magnitudes, and a tenth of that
with rounding of either sign; 16-bit outputs one rounding, 2^-8 of the value.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SAGE, GCN, GIN = 0, 1, 2
F32, BF16, F16 = 0, 1, 2


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _graph(torch, n, e, seed):
    """Distinct pairs, no loops; vertex 0 has many in-edges, the last none."""
    import paper_2607_17374_amd as T
    rng = np.random.default_rng(seed)
    u = np.concatenate([rng.integers(0, n, e), np.arange(1, n)])
    v = np.concatenate([rng.integers(0, n - 1, e), np.zeros(n - 1, np.int64)])
    key = np.unique((u * n + v)[u != v])
    src, dst = (key // n).astype(np.int32), (key % n).astype(np.int32)
    row_off, col_dst = T.build_csr(n, torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda())
    return src, dst, row_off, col_dst


def _reference(agg, n, src, dst, words, x, W, b, relu, d_out):
    keep = np.unpackbits(words.view(np.uint8), bitorder="little")[:len(src)].astype(bool)
    order = np.lexsort((dst, src))              # CSR order
    u, v = src[order][keep], dst[order][keep]
    d_in = np.bincount(v, minlength=n)
    s = np.zeros((n, x.shape[1]))
    if agg == SAGE:
        np.add.at(s, v, x[u])
        z = (s / np.maximum(d_in, 1)[:, None]) @ W[:, :d_out] + x @ W[:, d_out:]
    elif agg == GCN:
        no = 1 / np.sqrt(np.bincount(u, minlength=n) + 1.0)
        np.add.at(s, v, x[u] * no[u][:, None])
        z = ((s + x * no[:, None]) / np.sqrt(d_in + 1.0)[:, None]) @ W
    else:
        np.add.at(s, v, x[u])
        z = (s + x) @ W
    z = z + b
    return np.maximum(z, 0) if relu else z


def _layer(torch, n, row_off, col_dst, agg, d_in, d_out, dtype, out_dtype, k, seed=3, chunk=192, relu=True, **more):
    import paper_2607_17374_amd as T
    rng = np.random.default_rng(seed)
    td = [torch.float32, torch.bfloat16, torch.float16]
    W = (rng.standard_normal((d_in, d_out * (2 if agg == SAGE else 1))) / np.sqrt(d_in)).astype(np.float32)
    b = rng.uniform(-0.1, 0.1, d_out).astype(np.float32)
    x = torch.from_numpy(rng.standard_normal((n, d_in)).astype(np.float32)).to(td[dtype])
    Wx = torch.from_numpy(W).to(td[dtype]).double().numpy() if dtype else W.astype(np.float64)
    out = torch.full((n, d_out), -7.0, dtype=td[out_dtype], device="cuda")
    L = T.Layer(n, row_off, col_dst, agg=agg, d_in=d_in, d_out=d_out, weight_cat=W, bias=b, out=out, in_dtype=dtype,
                out_dtype=out_dtype, relu=relu, fanout=k, layer=1, seed=seed, chunk=chunk, **more)
    return L, x, Wx, b, out


def _check(out, z, out_dtype):
    y = out.double().cpu().numpy()
    rms = np.sqrt(np.mean(z * z))
    tol = 2e-5 * (np.abs(z) + rms) + (2.0 ** -8 * np.abs(z) if out_dtype else 0)
    assert np.all(np.abs(y - z) <= tol), float(np.max(np.abs(y - z) / (np.abs(z) + rms)))


CASES = [(agg, d_in, d_out, dt, od, k)
         for agg, d_in, d_out, dt, od, k in [
             (SAGE, 128, 256, BF16, BF16, 15), (SAGE, 256, 172, BF16, F32, 5), (SAGE, 8, 4, BF16, F32, 1),
             (SAGE, 104, 128, BF16, F16, 10), (SAGE, 64, 16, F32, F32, 7), (SAGE, 4, 12, F32, BF16, 3),
             (SAGE, 256, 200, F32, F32, 64), (SAGE, 132, 260, F32, F32, 10), (SAGE, 72, 1024, BF16, BF16, 4),
             (GCN, 128, 64, BF16, F32, 10), (GCN, 68, 44, F32, F32, 15), (GCN, 200, 132, BF16, BF16, 25),
             (GIN, 64, 64, BF16, F32, 5), (GIN, 100, 300, F32, F16, 10), (GIN, 248, 68, BF16, F32, 64),
             (SAGE, 264, 256, BF16, F32, 5), (SAGE, 128, 64, F16, F32, 5), (GCN, 256, 16, F32, F32, 5)]]


@pytest.mark.parametrize("agg,d_in,d_out,dt,od,k", CASES)
@pytest.mark.parametrize("n", [1000, 1025])
def test_sampled_layer(torch_cuda, n, agg, d_in, d_out, dt, od, k):
    torch = torch_cuda
    print(f"gather n={n} agg={agg} {d_in}->{d_out} dt={dt}/{od} k={k}", flush=True)
    src, dst, row_off, col_dst = _graph(torch, n, 6 * n, 1)
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, agg, d_in, d_out, dt, od, k)
    L.push_all(x.cuda())
    st = L.finalize()
    words, kept = L.sampled_edges()
    L.destroy()
    assert st["completed"] == n and st["messages"] == kept
    _check(out, _reference(agg, n, src, dst, words, x.double().numpy(), W, b, True, d_out), od)


def test_partial_pushes_write_complete_rows_only(torch_cuda):
    """finalize with chunks missing: INCOMPLETE, the rows whose messages have
    all arrived written, the others untouched; then the rest, in any order."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk = 1000, 192
    src, dst, row_off, col_dst = _graph(torch, n, 3000, 2)
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, SAGE, 32, 16, F32, F32, 3, chunk=chunk, relu=False)
    xd = x.cuda()
    with pytest.raises(T.TaurusError) as ex:
        L.finalize()
    assert ex.value.status == -5 and bool((out == -7.0).all())
    for k in (4, 0, 2):
        L.push_chunk(k * chunk, min(n, k * chunk + chunk), xd[k * chunk:k * chunk + chunk])
    with pytest.raises(T.TaurusError) as ex:
        L.finalize()
    assert ex.value.status == -5
    words, _ = L.sampled_edges()
    z = _reference(SAGE, n, src, dst, words, x.double().numpy(), W, b, False, 16)
    keep = np.unpackbits(words.view(np.uint8), bitorder="little")[:len(src)].astype(bool)
    order = np.lexsort((dst, src))
    u, v = src[order][keep], dst[order][keep]
    done = np.isin(np.arange(n) // chunk, (0, 2, 4))
    done[v[~np.isin(u // chunk, (0, 2, 4))]] = False
    assert 0 < done.sum() < n
    y = out.cpu().numpy()
    assert np.all(y[~done] == -7.0)
    _check(out[torch.from_numpy(done).cuda()], z[done], F32)
    for k in (3, 1, 5):
        L.push_chunk(k * chunk, min(n, k * chunk + chunk), xd[k * chunk:min(n, k * chunk + chunk)])
    st = L.finalize()
    assert st["completed"] == n and st["pending_left"] == 0
    first = out.clone()
    assert L.finalize()["completed"] == n and torch.equal(out, first)   # a second finalize changes nothing
    L.destroy()
    _check(out, z, F32)


@pytest.mark.parametrize("agg", [SAGE, GCN])
@pytest.mark.parametrize("first_on_host", [True, False])
def test_host_fed_chunks(torch_cuda, agg, first_on_host):
    """A layer fed from pinned memory is broadcast chunk by chunk; one whose
    first chunk was on the device keeps gathering.  Statistics that describe
    the sample are the same."""
    torch = torch_cuda
    n, chunk = 1025, 192
    src, dst, row_off, col_dst = _graph(torch, n, 6000, 3)
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, agg, 64, 48, BF16, F32, 6, chunk=chunk)
    xh, xd = x.pin_memory(), x.cuda()
    for i, c in enumerate(range(0, n, chunk)):
        on_host = first_on_host or i % 2 == 1
        L.push_chunk(c, min(n, c + chunk), (xh if on_host else xd)[c:min(n, c + chunk)])
    st = L.finalize()
    words, kept = L.sampled_edges()
    L.destroy()
    _check(out, _reference(agg, n, src, dst, words, x.double().numpy(), W, b, True, 48), F32)
    L, _, _, _, out2 = _layer(torch, n, row_off, col_dst, agg, 64, 48, BF16, F32, 6, chunk=chunk)
    L.push_all(xd)
    st2 = L.finalize()
    L.destroy()
    for key in ("messages", "pairs", "short_units", "wave_units", "split_segments", "completed", "pending_left",
                "chunks_pushed", "self_in_transform"):
        assert st[key] == st2[key], key


def test_statistics_match_the_broadcast(torch_cuda):
    """Counts of a gathered layer equal those of the same layer's chunk index
    (a profiled layer builds it); k = 512 gives a segment of several pieces."""
    torch = torch_cuda
    n = 1025
    src, dst, row_off, col_dst = _graph(torch, n, 6000, 4)
    for k, chunk in ((6, 192), (512, 1025)):
        got = []
        for profile in (0, 1):
            L, x, _, _, _ = _layer(torch, n, row_off, col_dst, SAGE, 64, 48, BF16, F32, k, chunk=chunk,
                                   profile=profile)
            L.push_all(x.cuda())
            got.append(L.finalize())
            L.destroy()
        for key in ("messages", "pairs", "short_units", "wave_units", "split_segments", "completed",
                    "self_in_transform"):
            assert got[0][key] == got[1][key], (k, key)
        assert k < 512 or got[0]["split_segments"] == 1


def test_values_that_are_not_finite(torch_cuda):
    """An infinite input reaches exactly the rows it is sent to, as infinity
    of the product's sign, and large finite means do not overflow the parts."""
    torch = torch_cuda
    n = 1000
    src, dst, row_off, col_dst = _graph(torch, n, 4000, 5)
    for bad in (np.inf, 3.0e38):
        L, x, W, b, out = _layer(torch, n, row_off, col_dst, SAGE, 64, 16, BF16, F32, 4, relu=False)
        W[:] = np.abs(W)
        import paper_2607_17374_amd as T
        L.destroy()
        Wp = np.abs((np.random.default_rng(3).standard_normal((64, 32)) / 8).astype(np.float32)) / 64
        x = x.clone()
        x[7, 3] = bad
        L = T.Layer(n, row_off, col_dst, agg=SAGE, d_in=64, d_out=16, weight_cat=Wp, bias=b, out=out, in_dtype=BF16,
                    out_dtype=F32, fanout=4, layer=1, seed=3, chunk=192)
        L.push_all(x.cuda())
        L.finalize()
        words, _ = L.sampled_edges()
        L.destroy()
        z = _reference(SAGE, n, src, dst, words, x.double().numpy(),
                       torch.from_numpy(Wp).bfloat16().double().numpy(), b, False, 16)
        y = out.double().cpu().numpy()
        assert np.array_equal(np.isinf(y), np.isinf(z)) and np.isfinite(y).sum() == np.isfinite(z).sum()
        fin = np.isfinite(z)
        rms = np.sqrt(np.mean(z[fin & (np.abs(z) < 1e30)] ** 2))
        assert np.all(np.abs(y[fin] - z[fin]) <= 2e-5 * (np.abs(z[fin]) + rms))


@pytest.mark.parametrize("agg,d_in,d_out,dt,od,k", [
    (SAGE, 104, 44, BF16, F32, 10),      # both halves' weights resident
    (SAGE, 256, 172, BF16, F32, 5),      # halves apart, partial products added
    (SAGE, 128, 256, F32, BF16, 6),      # fp32 weights: halves apart
    (GCN, 64, 100, F32, F32, 7), (GIN, 128, 260, BF16, BF16, 3)])
def test_large_layers(torch_cuda, agg, d_in, d_out, dt, od, k):
    """Enough destinations for the persistent kernels and the order by list
    length (from 262,144 on), against float64 on the GPU."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n = 300_001
    print(f"gather large agg={agg} {d_in}->{d_out} dt={dt}/{od} k={k}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(9)
    u = torch.randint(0, n, (1_500_000,), generator=g, device="cuda")
    v = (torch.rand(1_500_000, generator=g, device="cuda") ** 3 * (n - 1)).long()   # many lists empty, some long
    key = torch.unique((u * n + v)[u != v])
    row_off, col_dst = T.build_csr(n, (key // n).int(), (key % n).int())
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, agg, d_in, d_out, dt, od, k, chunk=65536)
    xd = x.cuda()
    L.push_all(xd)
    st = L.finalize()
    words, kept = L.sampled_edges()
    L.destroy()
    assert st["completed"] == n and st["messages"] == kept < key.numel()
    keep = torch.from_numpy(np.unpackbits(words.view(np.uint8), bitorder="little")[:key.numel()].astype(bool)).cuda()
    u, v = key[keep] // n, key[keep] % n
    xd, W, b = xd.double(), torch.from_numpy(np.ascontiguousarray(W)).cuda().double(), torch.from_numpy(b).cuda().double()
    d = torch.bincount(v, minlength=n).double()
    if agg == SAGE:
        s = torch.zeros_like(xd).index_add_(0, v, xd[u])
        z = (s / d.clamp(min=1)[:, None]) @ W[:, :d_out] + xd @ W[:, d_out:]
    elif agg == GCN:
        no = (torch.bincount(u, minlength=n) + 1).double().rsqrt()
        s = torch.zeros_like(xd).index_add_(0, v, xd[u] * no[u][:, None])
        z = ((s + xd * no[:, None]) * (d + 1).rsqrt()[:, None]) @ W
    else:
        z = (torch.zeros_like(xd).index_add_(0, v, xd[u]) + xd) @ W
    _check(out, torch.relu(z + b).cpu().numpy(), od)


def _fail_alloc(what):
    """The next device allocation of that name on this thread fails."""
    import paper_2607_17374_amd as T
    import ctypes
    f = T.lib().taurus_test_fail_alloc
    f.restype, f.argtypes = None, [ctypes.c_char_p]
    f(what.encode() if what else None)


def test_oversize_chunk_is_refused_at_init(torch_cuda):
    """A chunk whose transform would exceed 2 GiB is an argument error of
    init, also for a layer that would be gathered: the first host chunk would
    broadcast it."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n = 1_100_000
    src = torch.arange(0, 999, dtype=torch.int32, device="cuda")
    row_off, col_dst = T.build_csr(n, src, torch.full_like(src, 999))
    with pytest.raises(T.TaurusError) as ex:
        _layer(torch, n, row_off, col_dst, SAGE, 8, 256, BF16, BF16, 2, chunk=1 << 21)
    assert ex.value.status == -1 and "2 GiB" in str(ex.value)


def test_memory_that_is_not_pinned_changes_nothing(torch_cuda):
    """x_on_host with ordinary memory is refused before the layer's form
    changes: the layer still gathers device chunks."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk = 1025, 192
    src, dst, row_off, col_dst = _graph(torch, n, 6000, 3)
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, SAGE, 64, 48, F32, F32, 6, chunk=chunk)
    assert T.lib().taurus_push_chunk(L._h, 0, chunk, x.data_ptr(), 1) == -1
    _fail_alloc("work lists")                       # only the broadcast allocates these
    L.push_all(x.cuda())
    st = L.finalize()
    _fail_alloc(None)
    words, _ = L.sampled_edges()
    L.destroy()
    assert st["completed"] == n
    _check(out, _reference(SAGE, n, src, dst, words, x.double().numpy(), W, b, True, 48), F32)


@pytest.mark.parametrize("what", ["index keys", "work lists", "chunk transform", "accumulators"])
def test_failed_switch_to_the_broadcast_poisons(torch_cuda, what):
    """A first host chunk whose broadcast cannot be set up: every later push
    and finalize is refused, nothing is launched, the sample can still be read."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk = 1025, 192
    src, dst, row_off, col_dst = _graph(torch, n, 6000, 3)
    L, x, _, _, out = _layer(torch, n, row_off, col_dst, GCN, 64, 48, F32, F32, 6, chunk=chunk)
    xh, xd = x.pin_memory(), x.cuda()
    _fail_alloc(what)
    status = []
    for _ in range(2):
        with pytest.raises(T.TaurusError) as ex:
            L.push_chunk(0, chunk, xh[:chunk])
        status.append(ex.value.status)
    _fail_alloc(None)
    with pytest.raises(T.TaurusError) as ex:
        L.push_chunk(0, chunk, xd[:chunk])
    status.append(ex.value.status)
    with pytest.raises(T.TaurusError) as ex:
        L.finalize()
    status.append(ex.value.status)
    # (the index's temporaries live in the accumulators: "index keys" is carved there)
    assert status == [-2, -4, -4, -4], status
    _, kept = L.sampled_edges()
    assert 0 < kept < len(src)
    L.destroy()
    torch.cuda.synchronize()
    assert bool((out == -7.0).all())


def test_host_fed_layer_sets_up_the_broadcast_alone(torch_cuda):
    """Order, norms, weights and table of the gather wait for a first device
    chunk; a host-fed layer takes none of them, with a set-up stream or not,
    and both give the same bits."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk = 300_001, 65536
    g = torch.Generator(device="cuda").manual_seed(4)
    u, v = (torch.randint(0, n, (900_000,), generator=g, device="cuda") for _ in range(2))
    key = torch.unique((u * n + v)[u != v])
    row_off, col_dst = T.build_csr(n, (key // n).int(), (key % n).int())
    outs = []
    for setup in (None, torch.cuda.Stream()):
        for what in ("destination order", "input rows", "source norms"):
            _fail_alloc(what)
            L, x, _, _, out = _layer(torch, n, row_off, col_dst, SAGE, 256, 172, BF16, F32, 3, chunk=chunk,
                                     setup_stream=setup)
            xh = x.pin_memory()
            L.push_all(xh)
            st = L.finalize()
            _fail_alloc(None)
            L.destroy()
            assert st["completed"] == n
        outs.append(out)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("what", ["input rows", "destination order", "source norms", "packed weights and bias",
                                  "aggregate products"])
@pytest.mark.parametrize("setup", [False, True])
def test_gather_that_does_not_fit_is_broadcast(torch_cuda, what, setup):
    """Each allocation of the gather refused in turn: the layer is broadcast,
    with the broadcast's bits (a profiled layer's)."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk = 300_001, 65536
    g = torch.Generator(device="cuda").manual_seed(4)
    u, v = (torch.randint(0, n, (900_000,), generator=g, device="cuda") for _ in range(2))
    key = torch.unique((u * n + v)[u != v])
    row_off, col_dst = T.build_csr(n, (key // n).int(), (key % n).int())
    agg, d_in, d_out = (GCN, 64, 32) if what == "source norms" else (SAGE, 256, 172)
    outs = []
    for profile in (1, 0):
        L, x, _, _, out = _layer(torch, n, row_off, col_dst, agg, d_in, d_out, BF16, F32, 3, chunk=chunk,
                                 profile=profile, setup_stream=torch.cuda.Stream() if setup else None)
        if not profile:
            _fail_alloc(what)
        L.push_all(x.cuda())
        st = L.finalize()
        _fail_alloc(None)
        L.destroy()
        assert st["completed"] == n
        outs.append(out)
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("n", [1025, 300_001])
def test_rows_are_written_by_the_last_push(torch_cuda, n):
    """Every row is there, in stream order, after the last push: the next
    layer reads them before this one is finalized."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    g = torch.Generator(device="cuda").manual_seed(6)
    u, v = (torch.randint(0, n, (5 * n,), generator=g, device="cuda") for _ in range(2))
    key = torch.unique((u * n + v)[u != v])
    row_off, col_dst = T.build_csr(n, (key // n).int(), (key % n).int())
    got = []
    for early in (False, True):
        A, x, _, _, h = _layer(torch, n, row_off, col_dst, SAGE, 32, 64, BF16, BF16, 3, chunk=65536)
        B, _, _, _, out = _layer(torch, n, row_off, col_dst, GCN, 64, 16, BF16, F32, 4, chunk=65536)
        A.push_all(x.cuda())
        if not early:
            A.finalize()
        B.push_all(h)
        torch.cuda.synchronize()
        got.append((h.clone(), out.clone()))
        for L in (A, B):
            assert L.finalize()["completed"] == n
            L.destroy()
        assert torch.equal(h, got[-1][0]) and torch.equal(out, got[-1][1])
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert not bool((got[1][1] == -7.0).any())


@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("agg", [SAGE, GCN, GIN])
def test_weights_that_are_not_finite(torch_cuda, agg, dt):
    """An infinite weight (in bf16 also a finite fp32 one past its range), and
    a NaN, give what the broadcast gives, bit for bit: the layer is broadcast."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n = 1000
    src, dst, row_off, col_dst = _graph(torch, n, 4000, 5)
    rng = np.random.default_rng(1)
    x = torch.from_numpy(rng.standard_normal((n, 64)).astype(np.float32)).cuda()
    x = x.bfloat16() if dt else x
    x[11] = 0
    for bad in (np.inf, np.nan, 3.4e38):
        W = (rng.standard_normal((64, 64 if agg == SAGE else 32)) / 8).astype(np.float32)
        W[5, 3] = bad
        got = []
        for profile in (1, 0):
            out = torch.full((n, 32), -7.0, device="cuda")
            L = T.Layer(n, row_off, col_dst, agg=agg, d_in=64, d_out=32, weight_cat=W, bias=None, out=out,
                        in_dtype=dt, fanout=4, layer=1, seed=3, chunk=192, profile=profile)
            L.push_all(x)
            L.finalize()
            L.destroy()
            got.append(out)
        if bad == 3.4e38 and dt == F32:          # finite there: the same up to rounding where it does not overflow
            a, b = got[0].double(), got[1].double()
            ok = torch.isfinite(a) & torch.isfinite(b)
            assert ok.float().mean() > 0.5 and torch.allclose(a[ok], b[ok], rtol=1e-4, atol=1e-5)
        else:
            assert torch.equal(got[0].isnan(), got[1].isnan())
            assert torch.equal(got[0].nan_to_num(7.0), got[1].nan_to_num(7.0))
            assert bool(got[0].isinf().any() | got[0].isnan().any())


@pytest.mark.parametrize("n", [1000, 270_001])
@pytest.mark.parametrize("dt", [F32, BF16])
@pytest.mark.parametrize("agg", [SAGE, GCN, GIN])
def test_sums_past_the_type_before_the_linear_map(torch_cuda, agg, dt, n):
    """Inputs whose sum over a list exceeds fp32 while the outputs do not."""
    torch = torch_cuda
    src, dst, row_off, col_dst = _graph(torch, n, 6 * n, 5)
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, agg, 256, 128, dt, F32, 6, chunk=65536)
    xd = x.cuda()
    xd[:, 9] = 1e38
    _fail_alloc("work lists")                       # the layer is gathered
    L.push_all(xd)
    L.finalize()
    _fail_alloc(None)
    words, _ = L.sampled_edges()
    L.destroy()
    z = _reference(agg, n, src, dst, words, xd.double().cpu().numpy(), W, b, True, 128)
    assert np.abs(z).max() > 1e36
    _check(out, z, F32)


@pytest.mark.parametrize("n,hubs", [(1000, 1), (5000, 3), (4097, 4097)])
def test_gcn_norms_of_hub_sources(torch_cuda, n, hubs):
    """Sampled GCN where some sources are in every list, or every source is
    in few: the norms count each kept out-edge once (tiles of 4,096 entries,
    a source's two table slots taken or not)."""
    torch = torch_cuda
    import paper_2607_17374_amd as T
    rng = np.random.default_rng(n)
    u = np.concatenate([rng.integers(0, n, 8 * n)] + [np.full(n, h) for h in range(hubs if hubs < 10 else 0)])
    v = np.concatenate([rng.integers(0, n, 8 * n)] + [np.arange(n)] * (hubs if hubs < 10 else 0))
    key = np.unique((u * n + v)[u != v])
    src, dst = (key // n).astype(np.int32), (key % n).astype(np.int32)
    row_off, col_dst = T.build_csr(n, torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda())
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, GCN, 64, 32, F32, F32, 7, chunk=1024, relu=False)
    L.push_all(x.cuda())
    L.finalize()
    words, _ = L.sampled_edges()
    L.destroy()
    _check(out, _reference(GCN, n, src, dst, words, x.double().numpy(), W, b, False, 32), F32)


def test_long_lists_of_few_chunks_are_broadcast(torch_cuda):
    """Lists that read more as input rows than as transformed rows added up
    per chunk: broadcast, from the sample's offsets (no lists are drawn), with
    the bits and statistics of a profiled layer."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n = 30_000
    g = torch.Generator(device="cuda").manual_seed(8)
    u, v = (torch.randint(0, n, (6_000_000,), generator=g, device="cuda") for _ in range(2))
    key = torch.unique((u * n + v)[u != v])
    row_off, col_dst = T.build_csr(n, (key // n).int(), (key % n).int())
    got = []
    for profile in (1, 0):
        if not profile:
            _fail_alloc("kept sources")
        L, x, _, _, out = _layer(torch, n, row_off, col_dst, GIN, 256, 128, F32, F32, 190, chunk=65536,
                                 profile=profile)
        _fail_alloc(None)
        L.push_all(x.cuda())
        got.append((L.finalize(), out))
        L.destroy()
    assert torch.equal(got[0][1], got[1][1])
    assert 0 < got[0][0]["messages"] < key.numel()
    for k in ("messages", "pairs", "short_units", "wave_units", "split_segments", "completed"):
        assert got[0][0][k] == got[1][0][k], k


def _large_graph(torch, n, e, seed):
    import paper_2607_17374_amd as T
    g = torch.Generator(device="cuda").manual_seed(seed)
    u = torch.randint(0, n, (e,), generator=g, device="cuda")
    v = (torch.rand(e, generator=g, device="cuda") ** 3 * (n - 1)).long()   # many lists empty, some long
    key = torch.unique((u * n + v)[u != v])
    return key, *T.build_csr(n, (key // n).int(), (key % n).int())


def _large_reference(torch, agg, n, key, words, xd, W, b, d_out):
    """float64 on the GPU, before the activation; also the kept edges."""
    keep = torch.from_numpy(np.unpackbits(words.view(np.uint8), bitorder="little")[:key.numel()].astype(bool)).cuda()
    u, v = key[keep] // n, key[keep] % n
    xd, W = xd.double(), torch.from_numpy(np.ascontiguousarray(W)).cuda().double()
    d = torch.bincount(v, minlength=n).double()
    s = torch.zeros_like(xd)
    if agg == SAGE:
        s.index_add_(0, v, xd[u])
        z = (s / d.clamp(min=1)[:, None]) @ W[:, :d_out] + xd @ W[:, d_out:]
    elif agg == GCN:
        no = (torch.bincount(u, minlength=n) + 1).double().rsqrt()
        s.index_add_(0, v, xd[u] * no[u][:, None])
        z = ((s + xd * no[:, None]) * (d + 1).rsqrt()[:, None]) @ W
    else:
        z = (s.index_add_(0, v, xd[u]) + xd) @ W
    return z + torch.from_numpy(b).cuda().double(), u, v


@pytest.mark.parametrize("agg,d_in,d_out,dt,od,k", [
    (SAGE, 104, 44, BF16, F32, 10),      # both halves' weights resident
    (SAGE, 256, 172, BF16, F32, 5),      # halves apart, partial products added
    (SAGE, 128, 256, F32, BF16, 6),      # fp32 weights: halves apart
    (GCN, 64, 100, F32, F32, 7), (GIN, 128, 260, BF16, BF16, 3)])
def test_early_finalize_of_large_layers(torch_cuda, agg, d_in, d_out, dt, od, k):
    """The persistent kernels with chunks missing: complete rows written, the
    others untouched, also where partial products of a skipped row were never
    written; then the rest, in another order."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk = 300_001, 65536
    print(f"gather early finalize agg={agg} {d_in}->{d_out} dt={dt}/{od} k={k}", flush=True)
    key, row_off, col_dst = _large_graph(torch, n, 900_000, 9)
    L, x, W, b, out = _layer(torch, n, row_off, col_dst, agg, d_in, d_out, dt, od, k, chunk=chunk)
    _fail_alloc("work lists")
    xd = x.cuda()
    first = (4, 0, 2)
    for c in first:
        L.push_chunk(c * chunk, min(n, c * chunk + chunk), xd[c * chunk:c * chunk + chunk])
    with pytest.raises(T.TaurusError) as ex:
        L.finalize()
    _fail_alloc(None)
    assert ex.value.status == -5
    words, _ = L.sampled_edges()
    z, u, v = _large_reference(torch, agg, n, key, words, xd, W, b, d_out)
    z = torch.relu(z)
    here = torch.isin(torch.arange(n, device="cuda") // chunk, torch.tensor(first, device="cuda"))
    done = here.clone()
    done[v[~here[u]]] = False
    assert 0 < int(done.sum()) < n
    assert bool((out[~done] == -7.0).all())
    _check(out[done], z[done].cpu().numpy(), od)
    for c in (3, 1):
        L.push_chunk(c * chunk, c * chunk + chunk, xd[c * chunk:c * chunk + chunk])
    st = L.finalize()
    L.destroy()
    assert st["completed"] == n and st["pending_left"] == 0
    _check(out, z.cpu().numpy(), od)


@pytest.mark.parametrize("agg,d_in,d_out,dt,od,k", [
    (SAGE, 256, 200, F32, F32, 25), (GIN, 256, 136, F32, BF16, 30), (GCN, 132, 68, F32, F32, 40),
    (SAGE, 64, 20, BF16, F32, 100)])
@pytest.mark.parametrize("n", [1025, 270_001])
def test_long_lists_that_are_gathered(torch_cuda, n, agg, d_in, d_out, dt, od, k):
    """The widest rows and the longest lists that the gather takes (refusing
    the broadcast's work lists shows that it does), and their statistics."""
    torch = torch_cuda
    print(f"gather long lists n={n} agg={agg} {d_in}->{d_out} dt={dt}/{od} k={k}", flush=True)
    key, row_off, col_dst = _large_graph(torch, n, 60 * n if n < 5000 else 8 * n, 3)
    got = []
    for profile in (1, 0):
        if not profile:
            _fail_alloc("work lists")
        L, x, W, b, out = _layer(torch, n, row_off, col_dst, agg, d_in, d_out, dt, od, k, chunk=4096 if n > 5000 else 192,
                                 profile=profile)
        L.push_all(x.cuda())
        got.append(L.finalize())
        _fail_alloc(None)
        words, _ = L.sampled_edges()
        L.destroy()
    z, u, v = _large_reference(torch, agg, n, key, words, x.cuda(), W, b, d_out)
    assert int(torch.bincount(v).max()) == k
    _check(out, torch.relu(z).cpu().numpy(), od)
    for name in ("messages", "pairs", "short_units", "wave_units", "split_segments", "completed", "self_in_transform"):
        assert got[0][name] == got[1][name], name


def test_no_exception_leaves_an_entry(torch_cuda):
    """An exception of the C++ library inside finalize or sampled_edges
    becomes a status; a handle whose finalize threw is refused from then on."""
    import paper_2607_17374_amd as T
    torch = torch_cuda
    n, chunk = 1025, 192
    _, _, row_off, col_dst = _graph(torch, n, 6000, 3)
    L, x, _, _, _ = _layer(torch, n, row_off, col_dst, SAGE, 64, 48, F32, F32, 6, chunk=chunk)
    for call, what in ((L.sampled_edges, "!fanout mask"), (lambda: L.push_all(x.cuda()), "!input rows")):
        _fail_alloc(what)
        with pytest.raises(T.TaurusError) as ex:
            call()
        assert ex.value.status == -3, what
    L.destroy()
    L, x, _, _, _ = _layer(torch, n, row_off, col_dst, SAGE, 64, 48, F32, F32, 6, chunk=chunk)
    L.push_all(x.cuda())
    status = []
    for what in ("!list counts", None):
        _fail_alloc(what)
        with pytest.raises(T.TaurusError) as ex:
            L.finalize()
        status.append(ex.value.status)
    L.destroy()
    assert status == [-3, -4]
