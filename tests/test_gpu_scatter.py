"""GPU parity of the gather, its transpose (float scatter-accumulate) and the
integer histogram against the oracle. Integer results must be bit-exact; float
results within 1e-5 relative L2 (FP32)."""
import numpy as np
import pytest
import torch

import workloads
from oracle import scatter as osc

pytestmark = pytest.mark.gpu


def rel(a, b):
    a = np.asarray(a, np.float64).ravel()
    b = np.asarray(b, np.float64).ravel()
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300))


def gather_vjp(T, idx, w, g, dev, want_dw=True, config=0):
    from paper_2104_05372_amd import dex
    V, R = T.shape
    n = idx.shape[0]
    d = dex.gather_desc(V, R, n)
    tT = torch.tensor(T, device=dev)
    ti = torch.tensor(idx, device=dev)
    tw = torch.tensor(w, device=dev)
    tg = torch.tensor(g, device=dev)
    out = torch.empty(n, R, device=dev)
    print(f"  gather V={V} R={R} n={n}", flush=True)
    dex.dex_fwd(d, [tT, ti, tw], [out], [])
    dT = torch.empty_like(tT)
    dw = torch.empty_like(tw) if want_dw else None
    d.config = config
    ws = dex.workspace(dex.dex_workspace_bytes(d, dex.DEX_WS_VJP), dev)
    dex.dex_vjp(d, [tT, ti, tw], [], [tg], [dT, dw], 0 if want_dw else dex.DEX_NO_DW, ws)
    torch.cuda.synchronize()
    return out.cpu().numpy(), dT.cpu().numpy(), (dw.cpu().numpy() if want_dw else None)


@pytest.mark.parametrize("config", [1, 2])
@pytest.mark.parametrize("V,R,n,seed", [(50, 8, 1000, 0), (1000, 128, 50_000, 1), (7, 3, 5000, 2),
                                        (300, 100, 4097, 3), (20_000, 130, 2049, 4), (1, 64, 3000, 5),
                                        (70_000, 16, 9000, 6)])
def test_gather_and_transpose(dev, V, R, n, seed, config):
    si = workloads.scatter_inputs(V, R, n, 1.1, seed)
    out, dT, dw = gather_vjp(si.table, si.idx, si.w, si.g, dev, config=config)
    assert rel(out, osc.gather(si.table, si.idx, si.w)) <= 1e-6
    want = osc.scatter(V, si.idx, si.w, si.g)
    assert rel(dT, want) <= 1e-5
    untouched = np.setdiff1d(np.arange(V), si.idx)
    assert np.all(dT[untouched] == 0)
    assert rel(dw, osc.scatter_dw(si.table, si.idx, si.g)) <= 1e-5


# The two cotangents from one read: row lengths of every vector width (and more than
# one pass over the columns), entry counts on either side of a segment (64 and 512
# entries, from 2^19 on) and of a sort tile (2048 and 8192 keys, from 2^20 on),
# indices outside the table, buffers that are only 4-byte aligned, accumulation.
@pytest.mark.parametrize("V,R,n,offset", [(40, 1, 63, 0), (40, 2, 65, 0), (9, 3, 2048, 0), (500, 4, 2049, 1),
                                          (300, 50, 1000, 0), (33, 260, 700, 0), (33, 300, 129, 3),
                                          (64, 513, 200, 0), (3000, 2, (1 << 19) + 5, 0),
                                          (70_000, 1, (1 << 20) + 3, 0)])
def test_both_cotangents(dev, V, R, n, offset):
    from paper_2104_05372_amd import dex
    rng = np.random.default_rng(V + R + n)
    idx = rng.integers(-2, V + 2, n).astype(np.int32)
    idx[rng.random(n) < 0.3] = V // 2  # one hot row: its run spans segments
    T, g = (rng.standard_normal(s).astype(np.float32) for s in ((V, R), (n, R)))
    w = rng.uniform(-1, 1, n).astype(np.float32)
    ok = (idx >= 0) & (idx < V)
    safe = np.where(ok, idx, 0)
    want_T = osc.scatter(V, safe, np.where(ok, w, 0), g)
    want_w = np.where(ok, osc.scatter_dw(T, safe, g), 0)
    want_out = np.where(ok[:, None], osc.gather(T, safe, w), 0)

    def put(a):  # contiguous, `offset` floats into its storage
        t = torch.empty(a.size + offset, device=dev, dtype=torch.from_numpy(a).dtype)[offset:]
        return t.copy_(torch.from_numpy(a).reshape(-1)).view(a.shape)

    ins = [put(T), torch.tensor(idx, device=dev), put(w)]
    d = dex.gather_desc(V, R, n)
    out = put(np.full((n, R), 7, np.float32))
    dex.dex_fwd(d, ins, [out], [])
    assert rel(out.cpu().numpy(), want_out) <= 1e-6
    ws = dex.workspace(dex.dex_workspace_bytes(d, dex.DEX_WS_VJP), dev)
    for flags, base in ((0, 0.0), (dex.DEX_ACCUMULATE, 0.5)):
        dT, dw = put(np.full((V, R), 0.5, np.float32)), put(np.full(n, 0.5, np.float32))
        dex.dex_vjp(d, ins, [], [put(g)], [dT, dw], flags, ws)
        assert rel(dT.cpu().numpy(), want_T + base) <= 1e-5
        assert rel(dw.cpu().numpy(), want_w + base) <= 1e-5


def test_dense_one_hot_invariant(dev):
    si = workloads.scatter_inputs(50, 8, 1000, 1.1, 0)
    _, dT, _ = gather_vjp(si.table, si.idx, si.w, si.g, dev)
    S = np.zeros((1000, 50))
    S[np.arange(1000), si.idx] = 1
    assert rel(dT, S.T @ (si.w[:, None].astype(np.float64) * si.g)) <= 1e-5


@pytest.mark.parametrize("config", [1, 2])
@pytest.mark.parametrize("order", ["equal", "sorted", "reverse", "distinct"])
def test_contention_patterns(dev, order, config):
    rng = np.random.default_rng(7)
    n, V, R = 200_000, 5000, 32
    if order == "equal":
        idx = np.full(n, 17, np.int32)
    elif order == "sorted":
        idx = np.sort(rng.integers(0, V, n)).astype(np.int32)
    elif order == "reverse":
        idx = np.sort(rng.integers(0, V, n))[::-1].astype(np.int32).copy()
    else:
        n = V
        idx = rng.permutation(V).astype(np.int32)
    w = rng.uniform(-1, 1, n).astype(np.float32)
    g = rng.standard_normal((n, R)).astype(np.float32)
    T = rng.standard_normal((V, R)).astype(np.float32)
    _, dT, _ = gather_vjp(T, idx, w, g, dev, want_dw=False, config=config)
    if order == "equal":
        want = np.zeros((V, R))
        want[17] = (w[:, None].astype(np.float64) * g).sum(0)
    else:
        want = osc.scatter(V, idx, w, g)
    assert rel(dT, want) <= 1e-5


def test_deterministic_scatter_is_bit_reproducible(dev):
    """The sorted form fixes every row's summation order: repeated runs agree
    bit for bit (and with the oracle to FP32 accuracy), including hot rows."""
    from paper_2104_05372_amd import dex
    si = workloads.scatter_inputs(20_000, 64, 300_000, 1.1, 8)
    res = []
    for _ in range(3):
        acc = torch.zeros(20_000, 64, device=dev)
        dex.dex_accum_scatter(acc, torch.tensor(si.idx, device=dev), torch.tensor(si.g, device=dev),
                              torch.tensor(si.w, device=dev), flags=dex.DEX_DETERMINISTIC)
        res.append(acc.cpu().numpy())
    assert np.array_equal(res[0], res[1]) and np.array_equal(res[0], res[2])
    assert rel(res[0], osc.scatter(20_000, si.idx, si.w, si.g)) <= 1e-5


def test_deterministic_scatter_bounds_and_accumulate(dev):
    from paper_2104_05372_amd import dex
    rng = np.random.default_rng(9)
    idx = rng.integers(-3, 1003, 7000).astype(np.int32)
    vals = rng.standard_normal((7000, 9)).astype(np.float32)
    acc = torch.full((1000, 9), -1.5, device=dev)
    oob = torch.zeros(1, dtype=torch.int64, device=dev)
    dex.dex_accum_scatter(acc, torch.tensor(idx, device=dev), torch.tensor(vals, device=dev), None,
                          dex.DEX_DETERMINISTIC | dex.DEX_CHECK_BOUNDS, oob)
    want, nbad = osc.scatter(1000, idx, None, vals, check_bounds=True)
    assert oob.item() == nbad
    assert rel(acc.cpu().numpy() + 1.5, want) <= 1e-5


def test_accum_scatter_entry_point_and_bounds(dev):
    from paper_2104_05372_amd import autograd, dex
    rng = np.random.default_rng(3)
    idx = rng.integers(-5, 105, 3000).astype(np.int32)
    vals = rng.standard_normal((3000, 5)).astype(np.float32)
    scale = rng.uniform(-1, 1, 3000).astype(np.float32)
    acc = torch.full((100, 5), 2.0, device=dev)
    bad = autograd.accum_scatter(acc, torch.tensor(idx, device=dev), torch.tensor(vals, device=dev),
                                 torch.tensor(scale, device=dev), check_bounds=True)
    want, nbad = osc.scatter(100, idx, scale, vals, check_bounds=True)
    assert bad == nbad
    assert rel(acc.cpu().numpy() - 2.0, want) <= 1e-5
    # DEX_SYNC_CHECK turns found indices into an error status
    oob = torch.zeros(1, dtype=torch.int64, device=dev)
    with pytest.raises(dex.DexError) as ei:
        dex.dex_accum_scatter(acc, torch.tensor(idx, device=dev), torch.tensor(vals, device=dev), None,
                              dex.DEX_CHECK_BOUNDS | dex.DEX_SYNC_CHECK, oob)
    assert ei.value.status == dex.DEX_ERR_OUT_OF_RANGE
    # empty input is a no-op
    dex.dex_accum_scatter(acc, torch.zeros(0, dtype=torch.int32, device=dev))


def test_integer_rows_exact(dev):
    from paper_2104_05372_amd import dex
    rng = np.random.default_rng(5)
    for R in (3, 70):
        idx = rng.integers(0, 40, 20_000).astype(np.int32)
        vals = rng.integers(-1000, 1000, (20_000, R)).astype(np.int32)
        acc = torch.zeros(40, R, dtype=torch.int32, device=dev)
        dex.dex_accum_scatter(acc, torch.tensor(idx, device=dev), torch.tensor(vals, device=dev))
        want = np.zeros((40, R), np.int64)
        np.add.at(want, idx, vals)
        assert np.array_equal(acc.cpu().numpy(), want)


# Segments of 256 entries (from 320 K of them): a hot row over many segments, one column a
# lane, two and four.
@pytest.mark.parametrize("V,R,n", [(700, 3, 320 * 1024), (50, 66, 320 * 1024 + 257),
                                   (9, 260, 320 * 1024 + 1)])
def test_transpose_middle_segments(dev, V, R, n):
    si = workloads.scatter_inputs(V, R, n, 1.1, 14)
    idx = np.where(np.random.default_rng(n).random(n) < 0.4, V - 1, si.idx).astype(np.int32)
    _, dT, dw = gather_vjp(si.table, idx, si.w, si.g, dev, config=1)
    assert rel(dT, osc.scatter(V, idx, si.w, si.g)) <= 1e-5
    assert rel(dw, osc.scatter_dw(si.table, idx, si.g)) <= 1e-5


@pytest.mark.parametrize("config", [1, 2])
def test_table_updated_in_place(dev, config):
    """dT over T itself with DEX_ACCUMULATE (a step of w = -rate, in place): the table
    takes the transposed gather, and dw is formed with the table it has become."""
    from paper_2104_05372_amd import dex
    si = workloads.scatter_inputs(300, 50, 5000, 1.1, 15)
    T, idx, w, g = (torch.tensor(a, device=dev) for a in (si.table, si.idx, si.w, si.g))
    d = dex.gather_desc(300, 50, 5000)
    d.config = config
    dw = torch.zeros_like(w)
    dex.dex_vjp(d, [T, idx, w], [], [g], [T, dw], dex.DEX_ACCUMULATE,
                dex.workspace(dex.dex_workspace_bytes(d, dex.DEX_WS_VJP), dev))
    want = si.table + osc.scatter(300, si.idx, si.w, si.g)
    assert rel(T.cpu().numpy(), want) <= 1e-5
    assert rel(dw.cpu().numpy(), osc.scatter_dw(want, si.idx, si.g)) <= 1e-5


@pytest.mark.parametrize("n,bins,seed", [(1 << 20, 65536, 0), (100_003, 17, 1), (5, 65536, 2),
                                         (300_000, 1, 3), (1 << 18, 1000, 4)])
def test_histogram_bit_exact(dev, n, bins, seed):
    from paper_2104_05372_amd import autograd
    keys = workloads.histogram_keys(n, bins, 1.1, seed)
    tk = torch.tensor(keys.view(np.int32), device=dev)
    print(f"  histogram n={n} bins={bins}", flush=True)
    h1 = autograd.histogram(tk, bins).cpu().numpy()
    h2 = autograd.histogram(tk, bins).cpu().numpy()
    want = osc.histogram(keys, bins)
    assert np.array_equal(h1, want) and np.array_equal(h2, want)


@pytest.mark.parametrize("n,bins", [(1, 65536), (16_384, 10), (16_385, 10), (65_536, 65536),
                                    (65_537, 65536), (3 * 65_535 + 3, 65535)])
def test_histogram_few_blocks(dev, n, bins):
    """Both sides of where a second (third, fourth) block takes part."""
    from paper_2104_05372_amd import autograd
    keys = np.random.default_rng(n).integers(0, bins, n).astype(np.int32)
    h = autograd.histogram(torch.tensor(keys, device=dev), bins).cpu().numpy()
    assert np.array_equal(h, np.bincount(keys, minlength=bins))


def test_histogram_single_hot_bin_drains(dev):
    """All keys equal: the LDS counter crosses the drain threshold many times."""
    from paper_2104_05372_amd import autograd
    keys = np.full(3_000_000, 40_001, np.uint32)
    keys[::7] = 3
    h = autograd.histogram(torch.tensor(keys.view(np.int32), device=dev), 65536).cpu().numpy()
    assert h[40_001] == np.count_nonzero(keys == 40_001) and h[3] == np.count_nonzero(keys == 3)
    assert h.sum() == keys.size


@pytest.mark.parametrize("bins", [1, 2, 3, 1001, 65535, 65536])
def test_histogram_full_rounds(dev, bins):
    """Enough keys for whole rounds in every block, most of them on the two bins of one
    counter word (both are emptied several times a block) and on its neighbours, and a
    few out of range."""
    from paper_2104_05372_amd import dex
    rng = np.random.default_rng(bins)
    n, half = (1 << 23) + 5, (bins + 1) // 2
    hot = np.array([0, half, 1, bins - 1])[rng.integers(0, 4, n)] % bins
    keys = np.where(rng.random(n) < 0.8, hot, rng.integers(0, bins, n)).astype(np.int32)
    keys[::100_003] = bins
    keys[1::100_003] = -1
    h = torch.zeros(bins, dtype=torch.int32, device=dev)
    oob = torch.zeros(1, dtype=torch.int64, device=dev)
    dex.dex_accum_scatter(h, torch.tensor(keys, device=dev), flags=dex.DEX_CHECK_BOUNDS, oob=oob)
    ok = (keys >= 0) & (keys < bins)
    assert oob.item() == np.count_nonzero(~ok)
    assert np.array_equal(h.cpu().numpy(), np.bincount(keys[ok], minlength=bins))


# Waves whose lanes share a key (some, most, all), with keys outside the table among
# them: full rounds, the keys left over, both halves of a word.
@pytest.mark.parametrize("hot", [0.2, 0.6, 0.97, 1.0])
@pytest.mark.parametrize("n,bins", [(1000, 3), (16_384 * 3 + 77, 65_535), ((1 << 22) + 3, 1)])
def test_histogram_crowded_waves(dev, n, bins, hot):
    from paper_2104_05372_amd import dex
    rng = np.random.default_rng(n + int(100 * hot))
    for key in (0, bins - 1, bins, -1):
        keys = np.where(rng.random(n) < hot, key, rng.integers(-3, bins + 3, n)).astype(np.int32)
        h = torch.zeros(bins, dtype=torch.int32, device=dev)
        oob = torch.zeros(1, dtype=torch.int64, device=dev)
        dex.dex_accum_scatter(h, torch.tensor(keys, device=dev), flags=dex.DEX_CHECK_BOUNDS, oob=oob)
        ok = (keys >= 0) & (keys < bins)
        assert oob.item() == np.count_nonzero(~ok)
        assert np.array_equal(h.cpu().numpy(), np.bincount(keys[ok], minlength=bins))


def test_histogram_out_of_range_keys(dev):
    from paper_2104_05372_amd import dex
    keys = np.array([1, 2, 70_000, 2, 65_535, 65_536], np.uint32)
    h = torch.zeros(65536, dtype=torch.int32, device=dev)
    oob = torch.zeros(1, dtype=torch.int64, device=dev)
    dex.dex_accum_scatter(h, torch.tensor(keys.view(np.int32), device=dev), flags=dex.DEX_CHECK_BOUNDS,
                          oob=oob, idx_dtype=dex.DEX_U32)
    hh = h.cpu().numpy()
    assert oob.item() == 2 and hh[2] == 2 and hh[1] == 1 and hh[65535] == 1 and hh.sum() == 4


@pytest.fixture(scope="module")
def full_scatter():
    """The benchmarked problem (1e6 x 128 table, 2^22 Zipf(1.1) indices) and the
    oracle's whole transposed gather, computed once for the tests below."""
    c = workloads.SCATTER
    si = workloads.scatter_inputs(c["rows"], c["row_len"], c["n"], c["s"], c["seed"])
    return si, osc.scatter(c["rows"], si.idx, si.w, si.g)


def _check_table(dT, want, idx):
    touched = np.unique(idx)
    assert rel(dT, want) <= 1e-5
    # row by row over every touched row (an error confined to a few rows would
    # hide in the table-wide norm)
    num = np.linalg.norm(dT[touched].astype(np.float64) - want[touched], axis=1)
    den = np.linalg.norm(want[touched], axis=1)
    worst = int(np.argmax(num / np.maximum(den, 1e-300)))
    assert np.all(num <= 1e-5 * den), (int(touched[worst]), float(num[worst] / den[worst]))
    untouched = np.ones(dT.shape[0], bool)
    untouched[touched] = False
    assert not np.any(dT[untouched])


@pytest.mark.timeout(300)
@pytest.mark.parametrize("config", [1, 2])
def test_full_size_scatter(dev, full_scatter, config):
    """The whole 1e6 x 128 cotangent table against the oracle, both scatter
    forms, in the launch configuration the benchmark times."""
    si, want = full_scatter
    print(f"  full-size scatter, config {config}", flush=True)
    out, dT, dw = gather_vjp(si.table, si.idx, si.w, si.g, dev, want_dw=False, config=config)
    del out
    _check_table(dT, want, si.idx)


@pytest.mark.timeout(300)
def test_full_size_gather_and_dw(dev, full_scatter):
    """Every gathered row and every dw_j at full size."""
    si, _ = full_scatter
    out, _, dw = gather_vjp(si.table, si.idx, si.w, si.g, dev, config=1)
    assert rel(out, osc.gather(si.table, si.idx, si.w)) <= 1e-6
    del out
    assert rel(dw, osc.scatter_dw(si.table, si.idx, si.g)) <= 1e-5


def test_full_size_histogram(dev):
    from paper_2104_05372_amd import autograd
    c = workloads.HISTOGRAM
    keys = workloads.histogram_keys(c["n"], c["bins"], c["s"], c["seed"])
    h = autograd.histogram(torch.tensor(keys.view(np.int32), device=dev), c["bins"]).cpu().numpy()
    assert np.array_equal(h, osc.histogram(keys, c["bins"]))


def gather_jvp_gpu(T, idx, w, tT, tw, dev):
    from paper_2104_05372_amd import dex
    V, R = T.shape
    n = idx.shape[0]
    d = dex.gather_desc(V, R, n)
    out = torch.empty(n, R, device=dev)
    print(f"  gather jvp V={V} R={R} n={n}", flush=True)
    ws = dex.workspace(dex.dex_workspace_bytes(d, dex.DEX_WS_JVP), dev)
    dex.dex_jvp(d, [torch.tensor(T, device=dev), torch.tensor(idx, device=dev),
                    torch.tensor(w, device=dev)],
                [torch.tensor(tT, device=dev), torch.tensor(tw, device=dev)], [out], ws)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("V,R,n,seed", [(50, 8, 1000, 0), (300, 100, 4097, 3), (7, 3, 5000, 2),
                                        (20_000, 130, 2049, 4), (1, 64, 3000, 5), (10, 4, 0, 6)])
def test_gather_forward_mode(dev, V, R, n, seed):
    """dex_jvp of the gather against the oracle (several tiles, ragged row
    lengths, n = 0), and the dot-product identity <J t, g> = <t, J^T g> against
    dex_vjp on the same inputs."""
    si = workloads.scatter_inputs(V, R, n, 1.1, seed)
    rng = np.random.default_rng(seed + 100)
    tT = rng.standard_normal((V, R)).astype(np.float32)
    tw = rng.standard_normal(n).astype(np.float32)
    got = gather_jvp_gpu(si.table, si.idx, si.w, tT, tw, dev)
    if n == 0:
        assert got.size == 0
        return
    assert rel(got, osc.gather_jvp(si.table, si.idx, si.w, tT, tw)) <= 1e-6
    _, dT, dw = gather_vjp(si.table, si.idx, si.w, si.g, dev, config=1)
    lhs = np.sum(got.astype(np.float64) * si.g)
    rhs = np.sum(tT.astype(np.float64) * dT) + np.dot(tw.astype(np.float64), dw)
    assert abs(lhs - rhs) <= 1e-5 * (np.linalg.norm(got) * np.linalg.norm(si.g))


def test_gather_forward_mode_out_of_range_rows(dev):
    T = np.arange(24, dtype=np.float32).reshape(6, 4)
    idx = np.array([-1, 6, 2, 5, 1 << 30], dtype=np.int32)
    w = np.array([1, 2, 3, 4, 5], dtype=np.float32)
    tT = np.ones_like(T)
    tw = np.full(5, 0.5, dtype=np.float32)
    got = gather_jvp_gpu(T, idx, w, tT, tw, dev)
    assert np.array_equal(got, osc.gather_jvp(T, idx, w, tT, tw).astype(np.float32))


@pytest.mark.parametrize("R", [1, 3, 4, 6, 50, 128])
def test_out_of_range_rows_are_zero_whatever_their_weight(dev, R):
    """A row of zeros for an index outside the table, also where its weight is an
    infinity or NaN (every width of the gather's vectors)."""
    from paper_2104_05372_amd import dex
    rng = np.random.default_rng(R)
    T = rng.standard_normal((9, R)).astype(np.float32)
    idx = np.array([-1, 3, 9, 8, 1 << 30, 0, -5], dtype=np.int32)
    w = np.array([np.inf, 2, np.nan, -1, -np.inf, 0.5, 1], dtype=np.float32)
    out = torch.full((7, R), 7.0, device=dev)
    dex.dex_fwd(dex.gather_desc(9, R, 7),
                [torch.tensor(a, device=dev) for a in (T, idx, w)], [out], [])
    ok = (idx >= 0) & (idx < 9)
    want = np.zeros((7, R), np.float32)
    want[ok] = osc.gather(T, idx[ok], w[ok])
    assert np.array_equal(out.cpu().numpy(), want)


def test_full_size_gather_forward_mode_sampled(dev):
    """The benchmarked 1e6 x 128 table with 2^22 Zipf(1.1) indices; sampled rows."""
    c = workloads.SCATTER
    si = workloads.scatter_inputs(c["rows"], c["row_len"], c["n"], c["s"], c["seed"])
    rng = np.random.default_rng(1)
    tT = rng.standard_normal(si.table.shape, dtype=np.float32)
    tw = rng.standard_normal(si.w.shape[0], dtype=np.float32)
    got = gather_jvp_gpu(si.table, si.idx, si.w, tT, tw, dev)
    js = np.concatenate([[0, c["n"] - 1], rng.integers(0, c["n"], 64)])
    assert rel(got[js], osc.gather_jvp(si.table, si.idx, si.w, tT, tw, js)) <= 1e-6


@pytest.mark.parametrize("config", [1, 2])
def test_nan_cotangent_row_stays_in_its_row(dev, config):
    """A NaN in one upstream row makes exactly the cotangent row it is added
    into NaN (both scatter forms); every other row matches the oracle."""
    si = workloads.scatter_inputs(2000, 40, 30_000, 1.1, 12)
    g = si.g.copy()
    j = 777
    g[j, 5] = np.nan
    _, dT, dw = gather_vjp(si.table, si.idx, si.w, g, dev, config=config)
    want = osc.scatter(2000, si.idx, si.w, g)
    bad = int(si.idx[j])
    assert np.isnan(dT[bad, 5]) and np.isnan(want[bad, 5])
    assert np.array_equal(np.isnan(dT), np.isnan(want))
    keep = np.ones(2000, bool)
    keep[bad] = False
    assert rel(dT[keep], want[keep]) <= 1e-5
    assert np.isnan(dw[j]) and np.all(np.isfinite(np.delete(dw, j)))
