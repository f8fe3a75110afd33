"""The edges of the bf16 / d = 128 compression: chunk lengths around the 128 rows of a window (and twice that), windows
of more chunks than a wavefront has lanes, sequences that end just before and after the 1024 rows of a planning segment,
long chunks with more clusters than their key means are kept for (16), head counts that do and do not tie a head to one
XCD (a multiple of 8), non-finite and very large values, and workgroups that stop waiting.  Indices, sizes and lengths must equal the oracle's
bit for bit; fp32 means within 2e-5: a sum of m terms of size x is off by some sqrt(m) * 2^-24 * its own size, sqrt(m) x, so a mean by
2^-24 x, and the largest of its 128 entries is x / sqrt(m) or more: sqrt(4000) * 6e-8 = 4e-6."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_14303_amd import binding as sc
from paper_2603_14303_amd import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_common as g

D = 128
GAPS = {
    "window": [126, 127, 128, 129, 130],            # chunk lengths that just fit and just do not fit
    "two windows": [255, 256, 257, 128, 384, 385],
    "every row": [1],                               # 128 chunks in one window
    "pairs": [1, 2, 2, 1, 3],                       # more than 64 chunks in a window
    "long": [700, 3, 150, 40, 1025, 129, 1],        # several long chunks, across planning segments
    "none": [],                                     # one chunk
}


def _case(seed, gaps, lens, heads, centres):
    rng = np.random.default_rng(seed)
    B, N = len(lens), max(lens)
    mask = np.zeros((B, N), np.uint8)
    K = np.zeros((B, heads, N, D), np.float32)
    V = np.zeros_like(K)
    for b, n in enumerate(lens):
        if gaps:
            p = np.cumsum(np.roll(np.resize(gaps, n), b)) - 1
            mask[b, p[p < n]] = 1
        for h in range(heads):
            c = rng.standard_normal((centres, D))
            K[b, h, :n] = c[rng.integers(0, centres, n)] + 0.1 * rng.standard_normal((n, D))
            V[b, h, :n] = rng.standard_normal((n, D))
    return mask, wl.round_to_bf16(K), wl.round_to_bf16(V)


def _merge(mask, K, V, lens, tau, out_dtype=torch.float32):
    off, nch, sl = g.check_segment(mask, np.array(lens, np.int32))
    out = sc.sc_gsc_merge(g.to_device(K, True), g.to_device(V, True), off, nch, tau, seq_lens=sl, out_dtype=out_dtype,
                          want_cluster_id=True)
    torch.cuda.synchronize()
    return out


def _check_head(out, b, h, r, n):
    Kc, Vc, counts, clens, cid = out
    rows = r["n_rows"]
    assert int(clens[b, h]) == rows, (b, h, int(clens[b, h]), rows)
    assert np.array_equal(cid[b, h, :n].cpu().numpy(), r["cid"]), (b, h)
    assert np.array_equal(counts[b, h, :rows].cpu().numpy(), r["counts"][:rows]), (b, h)
    for got, ref in ((Kc, r["Kc"]), (Vc, r["Vc"])):
        got, ref = got[b, h, :rows].float().cpu().numpy(), ref[:rows]
        finite = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got), finite) and np.array_equal(np.isnan(got), np.isnan(ref)), (b, h)
        assert np.array_equal(np.isposinf(got), np.isposinf(ref)), (b, h)
        assert g.rowwise_err(np.where(finite, got, 0), np.where(finite, ref, 0)) <= 2e-5, (b, h)


@pytest.mark.parametrize("per_window", [0, 1])
@pytest.mark.parametrize("layout", list(GAPS))
@pytest.mark.parametrize("lens,heads", [((1023, 1025), 3), ((2047, 2050, 1, 0), 2), ((3000,), 8)])
def test_edges(layout, lens, heads, per_window):
    mask, K, V = _case(7 + len(layout), GAPS[layout], lens, heads, 40)
    tau = 0.6
    old = sc.tune_get("gsc_chunks_per_task")
    sc.tune_set("gsc_chunks_per_task", per_window)
    try:
        out = _merge(mask, K, V, lens, tau)
        half = _merge(mask, K, V, lens, tau, torch.bfloat16)
    finally:
        sc.tune_set("gsc_chunks_per_task", old)
    compared = 0
    for b, n in enumerate(lens):
        if n == 0:
            assert (out[3][b] == 0).all() and (half[3][b] == 0).all()
            continue
        o = oracle.segment(mask[b], n)
        for h in range(heads):
            r = oracle.compress_head(K[b, h, :n], V[b, h, :n], o, tau)
            if r["chunk_margin"].min() <= 1e-9:
                continue                                            # a coin toss in fp64 itself
            compared += n > 128
            _check_head(out, b, h, r, n)
            rows = r["n_rows"]
            for i in (0, 1):                                        # bf16 rows are the RNE rounding of the fp32 ones
                assert torch.equal(half[i][b, h, :rows], out[i][b, h, :rows].to(torch.bfloat16)), (b, h)
    assert compared >= heads


@pytest.mark.parametrize("centres", [6, 40])                       # up to sixteen clusters in a long chunk, and more
@pytest.mark.parametrize("keys", [False, True])
@pytest.mark.parametrize("layout", ["window", "pairs", "long"])
@pytest.mark.parametrize("fast", [1, 0])
def test_values_that_are_not_finite_stay_in_their_cluster(fast, layout, keys, centres):
    """A key that is not finite resembles nothing: its row is a cluster of its own, and its neighbours' sums are theirs alone; on the generic path, too."""
    lens, heads, tau = (1500,), 2, 0.6
    mask, K, V = _case(50 if centres == 6 else 51, GAPS[layout], lens, heads, centres)
    for i, x in enumerate((np.inf, np.nan, -np.inf)):
        V[0, 0, 40 + 400 * i, 5 * i] = x
        V[0, 1, 1499 - i, 127] = x
        if keys:
            K[0, 0, 60 + 400 * i, 3 * i] = x
            K[0, 1, 1490 - i, 100] = x
    old = sc.tune_get("gsc_fast_path")
    sc.tune_set("gsc_fast_path", fast)
    try:
        out = _merge(mask, K, V, lens, tau)
    finally:
        sc.tune_set("gsc_fast_path", old)
    o = oracle.segment(mask[0], lens[0])
    for h in range(heads):
        r = oracle.compress_head(K[0, h], V[0, h], o, tau)
        assert r["chunk_margin"].min() > 1e-9 and not np.isfinite(r["Vc"][:r["n_rows"]]).all()
        assert keys != np.isfinite(r["Kc"][:r["n_rows"]]).all()
        _check_head(out, 0, h, r, lens[0])


@pytest.mark.parametrize("centres", [6, 40])                       # up to sixteen clusters in a long chunk, and more
@pytest.mark.parametrize("layout", ["window", "pairs", "long"])
def test_values_near_the_largest_finite_one(layout, centres):
    """Every third cluster or delimiter is scaled until its sums lie up to 2^128, and some rows of size 1 hold the largest bf16
    value itself: means must stay finite and as exact as others (keys and values, the cosines are not changed by the scale)."""
    n, heads, tau = 1500, 2, 0.6
    mask, K, V = _case(70 + centres, GAPS[layout], (n,), heads, centres)
    K, V = np.clip(K, -3.875, 3.875), np.clip(V, -3.875, 3.875)
    top = float(torch.finfo(torch.bfloat16).max)
    o = oracle.segment(mask[0], n)
    expected = []
    for h in range(heads):
        r = oracle.compress_head(K[0, h], V[0, h], o, tau)
        assert r["chunk_margin"].min() > 1e-9
        chunk = np.searchsorted(o, np.arange(n), side="right") - 1
        group = np.unique(chunk * (n + 1) + np.where(r["cid"] < 0, n, r["cid"]), return_inverse=True)[1]
        scale = np.exp2(126 - np.ceil(np.log2(np.bincount(group))))[group]
        scaled = group % 3 == 0
        assert scaled.any() and not scaled.all()
        for x in (K, V):
            x[0, h, scaled] *= scale[scaled, None].astype(np.float32)
            assert np.abs(x[0, h]).max() >= 2.0 ** 127
        single = np.flatnonzero((np.bincount(group)[group] == 1) & ~scaled)
        V[0, h, single[::2], 3] = top
        V[0, h, single[1::2], 64] = -top
        expected.append(oracle.compress_head(K[0, h], V[0, h], o, tau))
        assert np.isfinite(expected[h]["Kc"]).all() and np.isfinite(expected[h]["Vc"]).all()
    out = _merge(mask, K, V, (n,), tau)
    half = _merge(mask, K, V, (n,), tau, torch.bfloat16)
    for h in range(heads):
        r = expected[h]
        _check_head(out, 0, h, r, n)
        alone = np.flatnonzero(r["counts"][:r["n_rows"]] == 1)
        for i, name in ((0, "Kc"), (1, "Vc")):
            assert np.array_equal(out[i][0, h].cpu().numpy()[alone].astype(np.float64), r[name][alone]), (h, name)
            assert torch.equal(half[i][0, h, :r["n_rows"]], out[i][0, h, :r["n_rows"]].to(torch.bfloat16)), (h, name)


def test_a_wait_that_is_given_up_is_reported():
    """No waiting at all: every head is either complete and right or reported by a length of -1, and every call ends."""
    lens, heads, tau = (3000, 2500), 4, 0.6
    mask, K, V = _case(60, GAPS["long"] + [9, 17, 40] * 40, lens, heads, 10)
    old = sc.tune_get("gsc_polls")
    sc.tune_set("gsc_polls", -1)
    try:
        out = _merge(mask, K, V, lens, tau)
    finally:
        sc.tune_set("gsc_polls", old)
    again = _merge(mask, K, V, lens, tau)
    assert (again[3] > 0).all()
    for b, n in enumerate(lens):
        o = oracle.segment(mask[b], n)
        for h in range(heads):
            r = oracle.compress_head(K[b, h, :n], V[b, h, :n], o, tau)
            assert r["chunk_margin"].min() > 1e-9
            _check_head(again, b, h, r, n)
            if int(out[3][b, h]) != -1:
                _check_head(out, b, h, r, n)


@pytest.fixture
def polls():
    old = sc.tune_get("gsc_polls")
    yield lambda n: sc.tune_set("gsc_polls", n)
    sc.tune_set("gsc_polls", old)


def _same(a, b, lens):
    """Every output of two calls, rows and tokens that exist, bit for bit."""
    assert torch.equal(a[3], b[3])
    for i, n in enumerate(lens):
        assert torch.equal(a[4][i, :, :n], b[4][i, :, :n])
        for h in range(a[3].shape[1]):
            rows = int(a[3][i, h])
            assert all(torch.equal(a[j][i, h, :rows], b[j][i, h, :rows]) for j in range(3)), (i, h)


@pytest.mark.parametrize("looks", [-2, -1, 0, 5])                    # -2: every window and long chunk is left to others
@pytest.mark.parametrize("layout", ["window", "every row", "long", "none", "mixed"])
@pytest.mark.parametrize("lens,heads,centres", [((3000, 2500), 4, 10), ((1100, 1, 0), 3, 40), ((4500,), 8, 25)])
def test_windows_that_stop_waiting_are_finished(polls, layout, lens, heads, centres, looks):
    """The same cache, whoever writes it: with few looks, or none, windows are finished by the workgroups that complete their segments."""
    gaps = {**GAPS, "mixed": GAPS["long"] + [9, 17, 40] * 40}[layout]
    mask, K, V = _case(60 + centres, gaps, lens, heads, centres)
    tau = 0.6
    want = _merge(mask, K, V, lens, tau)
    half = _merge(mask, K, V, lens, tau, torch.bfloat16)
    polls(looks)
    for _ in range(2):
        _same(_merge(mask, K, V, lens, tau), want, lens)
        _same(_merge(mask, K, V, lens, tau, torch.bfloat16), half, lens)
    compared = 0
    for b, n in enumerate(lens):
        if n < 128:
            continue
        o = oracle.segment(mask[b], n)
        for h in range(heads):
            r = oracle.compress_head(K[b, h, :n], V[b, h, :n], o, tau)
            if r["chunk_margin"].min() > 1e-9:
                compared += 1
                _check_head(want, b, h, r, n)
    assert compared >= heads


@pytest.mark.parametrize("looks", [-2, 100])
def test_a_long_chunk_takes_longer_than_anybody_waits(polls, looks):
    """Two thousand rows that hardly merge in one chunk, and windows behind it that stop waiting long before it is decided."""
    n, heads, tau = 4200, 2, 0.9
    mask, K, V = _case(90, [2100, 30, 12, 60, 700, 5], (n,), heads, n)
    polls(looks)
    out = _merge(mask, K, V, (n,), tau)
    o = oracle.segment(mask[0], n)
    for h in range(heads):
        r = oracle.compress_head(K[0, h], V[0, h], o, tau)
        assert r["chunk_margin"].min() > 1e-9 and r["n_rows"] > 0.8 * n
        _check_head(out, 0, h, r, n)


@pytest.mark.parametrize("looks", [1 << 16, 100])
def test_one_chunk_of_forty_thousand_rows(polls, looks):
    """Beyond the 32768 tokens that sc_gsc_merge_global's own kernels take."""
    n, heads, tau = 40000, 2, 0.6
    _, K, V = _case(92, [], (n,), heads, 40)
    polls(looks)
    out = sc.sc_gsc_merge_global(g.to_device(K, True), g.to_device(V, True), tau, out_dtype=torch.float32, want_cluster_id=True)
    torch.cuda.synchronize()
    for h in range(heads):
        r = oracle.compress_head(K[0, h], V[0, h], oracle.segment(np.zeros(n, np.uint8), n), tau)
        assert r["chunk_margin"].min() > 1e-9
        _check_head(out, 0, h, r, n)


def test_windows_left_behind_a_cache_that_is_too_small_or_appended_to(polls):
    """Capacity and append, every window left: lengths and rows as with waiting; rows beyond the capacity stay untouched."""
    n, heads, tau = 2600, 3, 0.6
    mask, K, V = _case(95, GAPS["long"] + [9, 17, 40] * 20, (n,), heads, 10)
    off, nch, _ = g.check_segment(mask, np.array([n], np.int32))
    Kd, Vd = g.to_device(K, True), g.to_device(V, True)
    full = int(_merge(mask, K, V, (n,), tau)[3].max())
    results = []
    for looks in (1 << 20, -2):
        polls(looks)
        for cap, base in ((full // 2, None), (2 * full, [[0, full // 3, full]]), (full, [[1, 0, -1]])):
            Kc = torch.full((1, heads, cap, D), -7.0, device="cuda")
            Vc, counts = Kc.clone(), torch.full((1, heads, cap), -7, dtype=torch.int32, device="cuda")
            clens = torch.full((1, heads), -7, dtype=torch.int32, device="cuda")
            lens = None if base is None else torch.tensor(base, dtype=torch.int32, device="cuda")
            sc.sc_gsc_merge(Kd, Vd, off, nch, tau, cap=cap, out_dtype=torch.float32, Kc=Kc, Vc=Vc, counts=counts, comp_lens=clens, base_lens=lens)
            torch.cuda.synchronize()
            results.append((Kc, Vc, counts, clens))
    for a, b in zip(results[:3], results[3:]):
        assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_two_calls_at_once(polls):
    """Two streams, heads that no XCD has to itself: windows of either call can hold up those of the other until they stop waiting."""
    n, heads, tau = 20000, 3, 0.6
    calls = []
    for seed in (97, 98):
        mask, K, V = _case(seed, [9, 17, 40, 24, 200], (n,), heads, 10)
        off, nch, _ = g.check_segment(mask, np.array([n], np.int32))
        args = (g.to_device(K, True), g.to_device(V, True), off, nch, tau)
        calls.append((args, sc.sc_gsc_merge(*args, want_cluster_id=True), torch.cuda.Stream(),
                      sc.gsc_merge_workspace(1, heads, n, D, "cuda")))
    torch.cuda.synchronize()
    for looks in (1 << 10, 4):
        polls(looks)
        got = []
        for _ in range(5):
            for args, _, stream, ws in calls:
                with torch.cuda.stream(stream):
                    got.append(sc.sc_gsc_merge(*args, want_cluster_id=True, workspace=ws))
        torch.cuda.synchronize()
        for i, out in enumerate(got):
            _same(out, calls[i % 2][1], (n,))


def test_more_windows_than_one_launch_can_have():
    """Six million heads of two tokens: a workgroup for each window there is room for would be more than 2^32 threads."""
    B, heads, tau = 65535, 90, 0.6
    gen = torch.Generator(device="cuda").manual_seed(99)
    K = torch.randn((B, heads, 2, D), generator=gen, device="cuda", dtype=torch.bfloat16)
    K[:, ::2, 1] = K[:, ::2, 0]                                     # every other head has two tokens alike, the others two that have nothing in common
    off, nch = sc.sc_segment(torch.zeros((B, 2), dtype=torch.uint8, device="cuda"))
    Kc, Vc, counts, clens, _ = sc.sc_gsc_merge(K, K, off, nch, tau)
    torch.cuda.synchronize()
    assert (clens[:, ::2] == 1).all() and (clens[:, 1::2] == 2).all()
    assert (counts[:, ::2, 0] == 2).all() and (counts[:, 1::2] == 1).all()
    for x in (Kc, Vc):
        assert torch.equal(x[:, ::2, 0], K[:, ::2, 0]) and torch.equal(x[:, 1::2], K[:, 1::2])
