"""GPU parity for sc_gsc_merge_budget: the bisection on the device must probe the thresholds the oracle's
bisection probes (every probe's row count is an integer the two sides agree on exactly), end on the
same fp32 threshold, and leave the merged cache of that threshold in the outputs."""
import threading

import numpy as np
import pytest
import torch

import oracle
from paper_2603_14303_amd import binding as sc
from paper_2603_14303_amd import workloads as wl
from helpers import build_case

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_common as g


def _oracle_rows(case, heads):
    cache = {}

    def rows_at(tau):
        if tau not in cache:
            tot = 0
            for b in range(case["K"].shape[0]):
                n = int(case["seq_lens"][b])
                for h in range(heads):
                    tot += oracle.compress_head(case["K"][b, h, :n], case["V"][b, h, :n], case["offsets"][b], tau)["n_rows"]
            cache[tau] = tot
        return cache[tau]
    return rows_at


@pytest.mark.parametrize("name,n,heads,fracs,iters", [
    ("tiny", None, 2, (0.2, 0.5, 0.95), 12),                 # fp32, d = 64: generic kernels
    ("layer32k", 4096 + 37, 2, (0.2, 0.35), 10),             # bf16 fast path; budgets of the paper
    ("batch_gqa7", 1536, 2, (0.35,), 8),                     # ragged batch
])
def test_budget_search_matches_oracle(name, n, heads, fracs, iters):
    w = wl.get_workload(name)
    batch = 3 if name == "batch_gqa7" else None
    case = build_case(w, 0.7, n_max=n, heads=heads, batch=batch, exclude_near=False)
    bf16 = w.dtype == "bf16"
    K, V = g.to_device(case["K"], bf16), g.to_device(case["V"], bf16)
    off, nch, sl = g.run_segment(case["mask"], case["seq_lens"])
    rows_at = _oracle_rows(case, heads)
    total = int(case["seq_lens"].sum()) * heads
    for frac in fracs:
        budget = int(round(frac * total))
        want_tau, probed = oracle.tau_for_budget(rows_at, budget, -1.01, 1.0, iters)
        Kc, Vc, counts, lens, cid, tau, rows = sc.sc_gsc_merge_budget(K, V, off, nch, budget, -1.01, 1.0, iters, seq_lens=sl,
                                                                      out_dtype=torch.float32, want_cluster_id=True)
        torch.cuda.synchronize()
        got_tau = tau.cpu().numpy()[0]
        assert got_tau == want_tau, (frac, got_tau, want_tau, probed)
        assert int(rows.item()) == rows_at(float(want_tau)) == int(lens.sum().item())
        if rows_at(-1.01) <= budget:
            assert int(rows.item()) <= budget
        # the outputs are those of a plain call at that threshold
        Kc2, Vc2, counts2, lens2, cid2 = sc.sc_gsc_merge(K, V, off, nch, float(got_tau), seq_lens=sl,
                                                         out_dtype=torch.float32, want_cluster_id=True)
        torch.cuda.synchronize()
        assert torch.equal(lens, lens2) and torch.equal(cid, cid2)
        for b in range(K.shape[0]):
            for h in range(heads):
                r = int(lens[b, h])
                assert torch.equal(counts[b, h, :r], counts2[b, h, :r])
                assert torch.equal(Kc[b, h, :r], Kc2[b, h, :r]) and torch.equal(Vc[b, h, :r], Vc2[b, h, :r])
        print(name, "budget %.2f -> tau %.6f rows %d of %d (%.1f %%)" % (frac, got_tau, int(rows.item()), total,
                                                                      100.0 * int(rows.item()) / total))
    # no iterations: the call is sc_gsc_merge at tau_lo
    _, _, _, lens0, _, tau0, rows0 = sc.sc_gsc_merge_budget(K, V, off, nch, total, 0.7, 0.9, 0, seq_lens=sl)
    torch.cuda.synchronize()
    assert tau0.item() == np.float32(0.7) and int(rows0.item()) == rows_at(0.7) == int(lens0.sum().item())
    # a capacity that the probes overflow counts as "over budget" and the search still ends below it
    small_cap = max(8, int(lens0.max().item()) + 4)
    out = sc.sc_gsc_merge_budget(K, V, off, nch, total, -1.01, 1.0, iters, seq_lens=sl, cap=small_cap)
    torch.cuda.synchronize()
    assert (out[3] >= 0).all() and (out[3] <= small_cap).all()


def test_budget_search_replays_from_a_graph():
    # the whole search is a fixed sequence of launches: capture it once, replay it with other work and
    # synchronisations in between, and get the eager result every time
    w = wl.get_workload("layer32k")
    case = build_case(w, 0.7, n_max=2048 + 5, heads=2, exclude_near=False)
    K, V = g.to_device(case["K"], True), g.to_device(case["V"], True)
    off, nch, sl = g.run_segment(case["mask"], case["seq_lens"])
    budget = int(0.3 * 2 * int(case["seq_lens"][0]))
    eager = sc.sc_gsc_merge_budget(K, V, off, nch, budget, -1.01, 1.0, 9, seq_lens=sl)
    torch.cuda.synchronize()
    ws = sc.Workspace(sc.load_library().sc_gsc_merge_budget_workspace_bytes(1, 2, K.shape[2], 128), g.DEV)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        warm = sc.sc_gsc_merge_budget(K, V, off, nch, budget, -1.01, 1.0, 9, seq_lens=sl, workspace=ws)
        side.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            out = sc.sc_gsc_merge_budget(K, V, off, nch, budget, -1.01, 1.0, 9, seq_lens=sl, workspace=ws)
    torch.cuda.synchronize()
    for replay in range(3):
        out[5].zero_(); out[3].zero_(); out[0].zero_()
        scratch = torch.randn(1 << 20, device=g.DEV).sum()          # unrelated eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert out[5].item() == eager[5].item() and out[6].item() == eager[6].item(), replay
        assert torch.equal(out[3], eager[3])
        for h in range(2):
            r = int(eager[3][0, h])
            assert torch.equal(out[0][0, h, :r], eager[0][0, h, :r]) and torch.equal(out[2][0, h, :r], eager[2][0, h, :r])
        del scratch


def test_knobs_that_change_during_the_search():
    """A search is many launches that share one layout of the workspace: all go by the knobs of the moment the call was made."""
    w = wl.get_workload("layer32k")
    case = build_case(w, 0.7, n_max=3000, heads=2, exclude_near=False)
    K, V = g.to_device(case["K"], True), g.to_device(case["V"], True)
    off, nch, sl = g.run_segment(case["mask"], case["seq_lens"])
    budget = int(0.3 * 2 * int(case["seq_lens"][0]))

    def search():
        return sc.sc_gsc_merge_budget(K, V, off, nch, budget, -1.01, 1.0, 12, seq_lens=sl, out_dtype=torch.float32, want_cluster_id=True)

    want = search()
    torch.cuda.synchronize()
    old = {k: sc.tune_get(k) for k in ("gsc_chunks_per_task", "gsc_polls", "gsc_fast_path")}
    stop = threading.Event()

    def turn():
        i = 0
        while not stop.is_set():
            sc.tune_set("gsc_chunks_per_task", i % 4)
            sc.tune_set("gsc_polls", 1 << (i % 20))
            sc.tune_set("gsc_fast_path", int(i % 5 != 0))
            i += 1

    t = threading.Thread(target=turn)
    t.start()
    try:
        got = [search() for _ in range(40)]
    finally:
        stop.set()
        t.join()
        for k, v in old.items():
            sc.tune_set(k, v)
    torch.cuda.synchronize()
    for out in got:
        assert out[5].item() == want[5].item() and out[6].item() == want[6].item()
        assert torch.equal(out[3], want[3]) and torch.equal(out[4], want[4])
        for h in range(2):
            rows = int(want[3][0, h])
            assert torch.equal(out[2][0, h, :rows], want[2][0, h, :rows])
            for i in (0, 1):        # fp32 means of bf16 rows, summed in another order where another path was taken
                assert torch.allclose(out[i][0, h, :rows], want[i][0, h, :rows], rtol=1e-5, atol=1e-5)


PROBE_GAPS = {
    "short": [24, 3, 61, 40, 1, 17, 90],
    "window": [126, 127, 128, 129, 130],            # chunk lengths that just fit a window and just do not fit
    "every row": [1],
    "long": [700, 3, 150, 40, 1025, 129, 1],
    "two blocks": [130, 257, 200, 258, 144],        # many long chunks
    "none": [],
}


def _bundles(rng, n, tau):
    """Keys at angles of their own around thirty centres, so that thresholds of every size split clusters."""
    c = rng.standard_normal((30, 128))
    return c[rng.integers(0, 30, n)] + rng.choice([0.05, 0.15, 0.5, 1.0], size=(n, 1)) * rng.standard_normal((n, 128))


def _inside_the_band(rng, n, tau):
    """Rows whose cosine with one of four directions is one of the thresholds, to within what rounding to bf16 leaves (some 1e-4, the
    width of the band that fp64 decides), and a few of the directions themselves in front."""
    e = np.linalg.qr(rng.standard_normal((128, 128)))[0]
    t = rng.choice(np.asarray(tau), size=(n, 1))
    rest = rng.standard_normal((n, 128))
    rest -= (rest @ e[:, :4]) @ e[:, :4].T
    rest /= np.linalg.norm(rest, axis=1, keepdims=True)
    k = t * e[:, rng.integers(0, 4, n)].T + np.sqrt(1 - t * t) * rest
    some = rng.random(n) < 0.05
    k[some] = e[:, rng.integers(0, 4, int(some.sum()))].T
    return 3.0 * k


@pytest.mark.parametrize("layout,lens,heads,keys", [
    *[(layout, lens, heads, _bundles) for layout in PROBE_GAPS for lens, heads in (((1023, 1025), 3), ((2600, 1, 0), 8), ((100,), 1))],
    # long chunks at a threshold for every workgroup, and (enough of them for the workgroups) at all thresholds by one
    *[(layout, lens, heads, _inside_the_band) for layout in ("short", "two blocks", "long") for lens, heads in (((2600, 1025), 2), ((2600, 2500), 32))],
    ("two blocks", (2600, 2500), 32, _bundles), ("long", (2600, 2500), 32, _bundles), ("two blocks", (5200,), 256, _bundles),
])
def test_every_threshold_of_a_probe_counts_exactly(layout, lens, heads, keys):
    """A probe counts at seven thresholds and the search goes down their tree: with the budget set to the rows at a threshold, and to one
    row less, a count that is off by one anywhere on the way turns the search.  A zero row and a key that is not finite are among the
    keys (a norm that is not usable)."""
    rng = np.random.default_rng(sum(lens) + 10 * heads + len(layout))
    B, N = len(lens), max(lens)
    thresholds, todo = [], [(np.float32(-1.01), np.float32(1.0))]
    for _ in range(7):      # what a search from this bracket may ask for in its first three steps
        x, y = todo.pop(0)
        m = np.float32(0.5) * (x + y)
        thresholds.append(float(m))
        todo += [(x, m), (m, y)]
    mask = np.zeros((B, N), np.uint8)
    K = np.zeros((B, heads, N, 128), np.float32)
    for b, n in enumerate(lens):
        if PROBE_GAPS[layout]:
            p = np.cumsum(np.roll(np.resize(PROBE_GAPS[layout], n), b)) - 1
            mask[b, p[p < n]] = 1
        for h in range(heads):
            K[b, h, :n] = keys(rng, n, thresholds) if h < 4 else np.roll(K[b, h % 4, :n], h, axis=0)
    K[0, 0, lens[0] // 2] = 0.0
    K[0, heads - 1, lens[0] // 3, 5] = np.inf
    K = wl.round_to_bf16(K)
    Kd = g.to_device(K, True)
    off, nch, sl = g.run_segment(mask, np.array(lens, np.int32))
    known = {}

    def rows_at(tau):
        if tau not in known:
            known[tau] = int(sc.sc_gsc_merge(Kd, Kd, off, nch, float(tau), seq_lens=sl)[3].sum().item())
        return known[tau]

    lo, hi = -1.01, 1.0
    mids = [(a + b) / 2 for a, b in ((lo, hi), (0.0, 1.0), (0.5, 1.0), (0.25, 0.5), (-0.5, 0.5), (0.75, 1.0), (0.9, 1.0))]
    for iters in (1, 2, 3, 4, 6, 8):
        for at in mids:
            # the rows at the midpoint that the search comes nearest to `at` with
            a, b = np.float32(lo), np.float32(hi)
            for _ in range(iters):
                mid = np.float32(0.5) * (a + b)
                a, b = (mid, b) if mid <= at else (a, mid)
            for budget in (rows_at(mid), rows_at(mid) - 1):
                want, _ = oracle.tau_for_budget(rows_at, budget, lo, hi, iters)
                out = sc.sc_gsc_merge_budget(Kd, Kd, off, nch, max(0, budget), lo, hi, iters, seq_lens=sl)
                assert out[5].item() == want and int(out[6].item()) == rows_at(want), (iters, at, budget)


def test_probes_have_more_workgroups_than_a_merge():
    """A window per token for 13 heads of 1.29 million tokens: with the workgroups that take long chunks in a merge these are fewer than 2^32 threads, with a
    probe's they are more, so neither has windows of that kind."""
    H, N = 13, 1259 * 1024
    gen = torch.Generator(device=g.DEV).manual_seed(12)
    K = torch.randn((1, H, N, 128), generator=gen, device=g.DEV, dtype=torch.bfloat16)
    K[:, :, 1::2] = K[:, :, ::2]                                    # tokens in pairs
    mask = torch.zeros((1, N), dtype=torch.uint8, device=g.DEV)
    mask[0, 49::50] = 1
    off, nch = sc.sc_segment(mask)
    budget = H * N * 6 // 10
    out = []
    for knob in (0, 1):
        sc.tune_set("gsc_chunks_per_task", knob)
        try:
            out.append(sc.sc_gsc_merge_budget(K, K, off, nch, budget, -1.01, 1.0, 3, cap=N * 6 // 10, out_dtype=torch.bfloat16)[2:])
            torch.cuda.synchronize()
        finally:
            sc.tune_set("gsc_chunks_per_task", 0)
    # a chunk of 49 tokens is 25 rows (its last token's twin is the delimiter), and its delimiter one: at every threshold from 0.5 on
    rows = H * (N // 50) * 26 + H * ((N % 50 + 1) // 2)
    for counts, lens, _, tau, total in out:
        assert int(total) == rows == int(lens.sum()) and float(tau) > 0.4 and torch.equal(lens, out[0][1])
    assert torch.equal(out[0][0][:, :, :rows // H], out[1][0][:, :, :rows // H])
