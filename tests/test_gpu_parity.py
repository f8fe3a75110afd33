"""GPU parity: the HIP path (through the C ABI binding) against the CPU oracle, element by element."""
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


# ------------------------------------------------------------------ sc_segment
def test_segment_edge_cases():
    N = 40
    rows = [
        np.zeros(N, np.uint8),                                   # no delimiter: one chunk
        np.ones(N, np.uint8),                                    # all delimiters: N+1 empty chunks
        np.array([1] + [0] * (N - 2) + [1], np.uint8),           # leading and trailing delimiter
        np.array(([1, 1, 0, 0, 0] * 8), np.uint8),               # adjacent delimiters
    ]
    mask = np.stack(rows)
    g.check_segment(mask, None)
    g.check_segment(mask, np.array([0, 1, 17, 39], np.int32))    # ragged, including an empty sequence


@pytest.mark.parametrize("name", ["tiny", "layer32k", "long128k"])
def test_segment_workloads(name):
    w = wl.get_workload(name)
    mask = np.stack([wl.delimiter_mask(w, b) for b in range(w.batch)])
    g.check_segment(mask, None)


def test_segment_ragged_batch_and_unaligned_rows():
    w = wl.get_workload("batch_gqa7")
    lens = wl.seq_lens(w)[:6]
    mask = np.zeros((6, w.n_max + 3), np.uint8)
    for b in range(6):
        mask[b, : w.n_max] = wl.delimiter_mask(w, b)
    g.check_segment(mask, lens)                                   # row stride 16387: rows are not 16-byte aligned
    rng = np.random.default_rng(0)
    dense = (rng.random((3, 70001)) < 0.5).astype(np.uint8)      # several tiles, ragged tail, half delimiters
    g.check_segment(dense, np.array([70001, 33333, 16384], np.int32))


def test_segment_capacity_overflow_is_flagged():
    mask = torch.ones((2, 64), dtype=torch.uint8, device=g.DEV)
    mask[1, 5:] = 0
    off = torch.full((2, 10), -5, dtype=torch.int32, device=g.DEV)
    _, nch = sc.sc_segment(mask, None, offsets=off)
    torch.cuda.synchronize()
    assert nch.tolist() == [-1, 6]
    assert off[1, :7].tolist() == [0, 1, 2, 3, 4, 5, 65]
    # several tiles of mask per sequence, each filed by a workgroup of its own: none writes beyond the capacity
    mask = torch.ones((2, 70000), dtype=torch.uint8, device=g.DEV)
    mask[1, 40:69990] = 0
    wide = torch.full((2, 200), -5, dtype=torch.int32, device=g.DEV)
    _, nch = sc.sc_segment(mask, None, offsets=wide[:, :100])
    torch.cuda.synchronize()
    assert nch.tolist() == [-1, 51]
    assert wide[0, :100].tolist() == list(range(100)) and (wide[:, 100:] == -5).all()
    assert wide[1, :52].tolist() == list(range(41)) + list(range(69991, 70001)) + [70001]


# ------------------------------------------------------------------ sc_gsc_merge + sc_decode_attn
@pytest.mark.parametrize("tau", [0.7, 1.0, -1.01, 0.9745])
def test_tiny_full(tau):
    w = wl.get_workload("tiny")
    case = build_case(w, tau)
    out = g.check_compress(case)
    errs = g.check_decode(case, out, range(w.decode_steps))
    print("tiny tau=%g redraws=%d merge_err=%.2e decode_err=%s" % (tau, case["redraws"], out["worst_merge_err"], errs))


@pytest.mark.parametrize("name,n,tau", [("layer32k", 4096 + 37, 0.7), ("layer32k", 3000, 0.9745),
                                        ("long128k", 8192 + 5, 0.7), ("long128k", 6000, 0.03)])
def test_truncated_workloads(name, n, tau):
    # a few thousand tokens: several work items per head, chunks longer than one 64-row block, ragged tail
    w = wl.get_workload(name)
    case = build_case(w, tau, n_max=n, heads=3)
    out = g.check_compress(case)
    errs = g.check_decode(case, out, range(3), q_heads=3 * w.group)
    print(name, n, tau, "redraws", case["redraws"], "merge_err %.2e" % out["worst_merge_err"], "decode", errs)


@pytest.mark.parametrize("base,dtype,d", [("layer32k", "bf16", 64), ("tiny", "f32", 128), ("tiny", "bf16", 128)])
def test_other_dtype_and_head_dim_combinations(base, dtype, d):
    # the combinations the header promises beyond the two the workloads use (bf16 / 128 and fp32 / 64):
    # bf16 with d = 64 and fp32 with d = 128 through sc_gsc_merge (generic kernels) and sc_decode_attn
    import dataclasses
    w = dataclasses.replace(wl.get_workload(base), dtype=dtype, head_dim=d, kv_heads=2, q_heads=8)
    case = build_case(w, 0.7, n_max=1500 + 3)
    out = g.check_compress(case)
    errs = g.check_decode(case, out, range(3))
    print(base, dtype, d, "redraws", case["redraws"], "merge_err %.2e" % out["worst_merge_err"], "decode", errs)


def test_layer32k_full_size():
    w = wl.get_workload("layer32k")
    case = build_case(w, 0.7)
    out = g.check_compress(case)
    errs = g.check_decode(case, out, [0, 1, 31, 63])
    print("layer32k full: redraws", case["redraws"], "pairs/token %.2f" % (case["n_pairs"] / (8 * 32768)),
          "rows", out["comp_lens"].tolist(), "merge_err %.2e" % out["worst_merge_err"], "decode", errs)


def test_batch_ragged_gqa7():
    w = wl.get_workload("batch_gqa7")
    case = build_case(w, 0.975, n_max=2048, batch=5)
    assert len(set(case["seq_lens"].tolist())) > 1
    out = g.check_compress(case)
    lens = out["comp_lens"].cpu().numpy()
    assert len(set(lens.ravel().tolist())) > 4                     # per-sequence, per-head lengths differ
    errs = g.check_decode(case, out, range(2))
    print("gqa7 ragged: lens", lens.tolist(), "decode", errs)


def test_capacity_overflow_and_empty_sequences():
    w = wl.get_workload("tiny")
    case = build_case(w, 0.7)
    full = g.run_compress(case, torch.float32)
    rows = full["comp_lens"].cpu().numpy()
    cap = int(rows.min()) - 3
    small = g.run_compress(case, torch.float32, cap=cap)
    assert small["comp_lens"].tolist() == [[-1, -1]]
    assert sc.check_lengths(small["comp_lens"]) == 0 and sc.check_lengths(full["comp_lens"]) == -1
    assert torch.equal(small["Kc"][:, :, :cap], full["Kc"][:, :, :cap])
    assert torch.equal(small["counts"][:, :, :cap], full["counts"][:, :, :cap])
    # a sequence of length 0 gives an empty merged cache, and decode over it returns zeros
    case0 = build_case(w, 0.7)
    case0["seq_lens"] = np.array([0], np.int32)
    out0 = g.run_compress(case0, torch.float32)
    assert out0["comp_lens"].tolist() == [[0, 0]]
    Q = g.to_device(wl.queries(w, 0, 0), False)
    O, lse = sc.sc_decode_attn(Q, out0["Kc"], out0["Vc"], out0["counts"], out0["comp_lens"], want_lse=True)
    torch.cuda.synchronize()
    assert (O == 0).all() and torch.isinf(lse).all() and (lse < 0).all()


def test_zero_norm_and_duplicate_keys():
    # degenerate keys: zero rows never merge, exact duplicates merge at any tau < 1
    d = 64
    rng = np.random.default_rng(7)
    n = 200
    K = rng.standard_normal((n, d)).astype(np.float32)
    K[10] = 0; K[11] = 0; K[50] = K[40]; K[51] = K[40] * 3.0
    V = rng.standard_normal((n, d)).astype(np.float32)
    mask = np.zeros((1, n), np.uint8)
    mask[0, [30, 90, 91, 150]] = 1
    off = oracle.segment(mask[0], n)
    ref = oracle.compress_head(K, V, off, 0.999)
    Kd = torch.from_numpy(K).to(g.DEV).view(1, 1, n, d)
    Vd = torch.from_numpy(V).to(g.DEV).view(1, 1, n, d)
    offs, nch, _ = g.run_segment(mask, None)
    Kc, Vc, counts, lens, cid = sc.sc_gsc_merge(Kd, Vd, offs, nch, 0.999, want_cluster_id=True)
    torch.cuda.synchronize()
    assert lens.item() == ref["n_rows"]
    assert np.array_equal(cid[0, 0].cpu().numpy(), ref["cid"])
    assert np.array_equal(counts[0, 0, : ref["n_rows"]].cpu().numpy(), ref["counts"][: ref["n_rows"]])


def test_strided_kv_views():
    # K/V handed over as strided views of a [B, N, H, d] allocation (a common cache layout)
    w = wl.get_workload("tiny")
    case = build_case(w, 0.7)
    base = g.run_compress(case, torch.float32)
    K = torch.from_numpy(case["K"]).to(g.DEV).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    V = torch.from_numpy(case["V"]).to(g.DEV).permute(0, 2, 1, 3).contiguous().permute(0, 2, 1, 3)
    assert not K.is_contiguous()
    Kc, Vc, counts, lens, _ = sc.sc_gsc_merge(K, V, base["offsets"], base["num_chunks"], 0.7)
    torch.cuda.synchronize()
    assert torch.equal(lens, base["comp_lens"])
    for h in range(2):
        r = int(lens[0, h])
        assert torch.equal(Kc[0, h, :r], base["Kc"][0, h, :r]) and torch.equal(Vc[0, h, :r], base["Vc"][0, h, :r])
        assert torch.equal(counts[0, h, :r], base["counts"][0, h, :r])


def test_repeatable_bit_for_bit():
    w = wl.get_workload("layer32k")
    case = build_case(w, 0.7, n_max=5000, heads=2, exclude_near=False)
    a = g.run_compress(case, torch.bfloat16)
    ws = sc.decode_attn_workspace(1, 8, 2, 5000, 128, g.DEV)
    Q = g.to_device(wl.queries(w, 0, 0)[:, :8], True)
    O0, _ = sc.sc_decode_attn(Q, a["Kc"], a["Vc"], a["counts"], a["comp_lens"], workspace=ws)
    O0 = O0.clone()
    for _ in range(5):
        b = g.run_compress(case, torch.bfloat16)
        assert torch.equal(a["comp_lens"], b["comp_lens"]) and torch.equal(a["cid"], b["cid"])
        for h in range(2):
            r = int(a["comp_lens"][0, h])
            assert torch.equal(a["Kc"][0, h, :r], b["Kc"][0, h, :r]) and torch.equal(a["Vc"][0, h, :r], b["Vc"][0, h, :r])
            assert torch.equal(a["counts"][0, h, :r], b["counts"][0, h, :r])
        O1, _ = sc.sc_decode_attn(Q, a["Kc"], a["Vc"], a["counts"], a["comp_lens"], workspace=ws)
        torch.cuda.synchronize()
        # split partials are combined in a fixed order, so the result does not depend on arrival order
        assert torch.equal(O0, O1)


@pytest.mark.parametrize("knobs", [
    dict(gsc_chunks_per_task=1), dict(gsc_chunks_per_task=3), dict(gsc_chunks_per_task=5),
    dict(gsc_chunks_per_task=32), dict(gsc_fast_path=0), dict(gsc_fast_path=0, gsc_grid_x=7),
    dict(gsc_fast_path=0, gsc_chunks_per_item=3, gsc_grid_x=5),
    dict(decode_mfma_min_group=1), dict(decode_mfma_min_group=9), dict(decode_max_splits=3, decode_min_rows=64),
])
def test_launch_shape_knobs_do_not_change_results(knobs):
    # fewer chunks to a window, the generic kernels on the fast path's inputs, also with grids narrower than the
    # item count (workgroups then walk several items), and single-row decode on either attention kernel:
    # same integers, merged rows and attention outputs within the same bounds
    w = wl.get_workload("long128k")
    case = build_case(w, 0.7, n_max=5000 + 11, heads=2)
    old = {k: sc.tune_get(k) for k in knobs}
    try:
        for k, v in knobs.items():
            sc.tune_set(k, v)
        out = g.check_compress(case)
        errs = g.check_decode(case, out, range(2), q_heads=2 * w.group)
    finally:
        for k, v in old.items():
            sc.tune_set(k, v)
    print(knobs, "merge_err %.2e" % out["worst_merge_err"], "decode", errs)


def test_decode_capacity_beyond_32bit_row_offsets():
    # the fast decode kernel addresses the rows of a (sequence, head) with 32-bit byte offsets; a cache
    # whose capacity does not fit is served by the generic kernel: same result within the decode tolerance
    rows, d, G = 3000 + 7, 128, 4
    rng = np.random.default_rng(11)
    Ks = torch.from_numpy(rng.standard_normal((1, 1, rows, d)).astype(np.float32)).to(g.DEV).to(torch.bfloat16)
    Vs = torch.from_numpy(rng.standard_normal((1, 1, rows, d)).astype(np.float32)).to(g.DEV).to(torch.bfloat16)
    cs = torch.from_numpy(rng.integers(1, 9, (1, 1, rows)).astype(np.int32)).to(g.DEV)
    lens = torch.tensor([[rows]], dtype=torch.int32, device=g.DEV)
    Q = torch.from_numpy(rng.standard_normal((1, G, d)).astype(np.float32)).to(g.DEV).to(torch.bfloat16)
    O_small, lse_small = sc.sc_decode_attn(Q, Ks, Vs, cs, lens, want_lse=True)
    cap = (1 << 31) // (d * 2) + 5
    Kb = torch.empty((1, 1, cap, d), dtype=torch.bfloat16, device=g.DEV)
    Vb = torch.empty_like(Kb)
    cb = torch.empty((1, 1, cap), dtype=torch.int32, device=g.DEV)
    Kb[:, :, :rows], Vb[:, :, :rows], cb[:, :, :rows] = Ks, Vs, cs
    O_big, lse_big = sc.sc_decode_attn(Q, Kb, Vb, cb, lens, want_lse=True)
    torch.cuda.synchronize()
    want_O, want_l = oracle.decode_attn(Q.float().cpu().numpy().astype(np.float64), Ks.float().cpu().numpy().astype(np.float64),
                                        Vs.float().cpu().numpy().astype(np.float64), cs.cpu().numpy(), lens.cpu().numpy())
    for O, lse in ((O_small, lse_small), (O_big, lse_big)):
        assert np.abs(O.float().cpu().numpy() - want_O).max() <= 4e-3 * max(1.0, np.abs(want_O).max())
        assert np.abs(lse.cpu().numpy() - want_l).max() <= 1e-3


@pytest.mark.parametrize("n,knobs", [(2600, {}), (33000, {}), (2600, dict(gsc_grid_x=1)), (33000, dict(gsc_grid_x=3, gsc_chunks_per_item=32))])
def test_generic_merge_long_items(n, knobs):
    # fp32 / d = 64: a chunk longer than the cluster indices held in LDS, next to short ones and runs of delimiters, with
    # the row bases added up inside the merge kernel (up to 32768 tokens) and by the scan kernel (beyond); narrow grids
    # make a workgroup carry its prefix from item to item
    rng = np.random.default_rng(n)
    mask = np.zeros((1, n), dtype=np.uint8)
    mask[0, np.cumsum(rng.integers(1, 40, size=n // 10))[: n // 40]] = 1
    mask[0, 100:2401] = 0
    mask[0, 2402:2470] = 1
    off = oracle.segment(mask[0], n)
    centers = rng.standard_normal((7, 64))
    k = (centers[rng.integers(0, 7, size=n)] + 0.1 * rng.standard_normal((n, 64))).astype(np.float32)
    v = rng.standard_normal((n, 64)).astype(np.float32)
    ref = oracle.compress_head(k, v, off, 0.7)
    K, V = (torch.from_numpy(x[None, None]).to(g.DEV) for x in (k, v))
    old = {key: sc.tune_get(key) for key in knobs}
    try:
        for key, val in knobs.items():
            sc.tune_set(key, val)
        offsets, num_chunks, _ = g.run_segment(mask, None)
        Kc, Vc, counts, lens, cid = sc.sc_gsc_merge(K, V, offsets, num_chunks, 0.7, want_cluster_id=True)
        torch.cuda.synchronize()
    finally:
        for key, val in old.items():
            sc.tune_set(key, val)
    rows = ref["n_rows"]
    assert int(lens[0, 0]) == rows
    assert np.array_equal(cid[0, 0].cpu().numpy(), ref["cid"])
    assert np.array_equal(counts[0, 0, :rows].cpu().numpy(), ref["counts"][:rows])
    # fp32 sums of up to l members in member order: (l + 1) half-ulps of the largest partial sum, relative to the mean
    tol = 2.0 ** -24 * (int(ref["counts"][:rows].max()) + 2)
    for got, want in ((Kc, ref["Kc"]), (Vc, ref["Vc"])):
        err = np.abs(got[0, 0, :rows].cpu().numpy() - want[:rows])
        assert err.max() <= tol * max(np.abs(k).max(), np.abs(v).max())


@pytest.mark.parametrize("H,n,gap", [
    (17, 2000, 1), (17, 2000, 2.6), (17, 2000, 9.9), (17, 2000, 10.1),    # more than 64k rows: items of 32, 16, 16 and eight chunks
    (9, 3600, 1), (9, 3600, 2.4), (9, 3600, 2.6), (9, 3600, 4.4), (9, 3600, 4.6),     # fewer: of 32, 16, eight, eight, four
    (1, 700, 2),                                                            # fewer chunks than workgroups
    (1, 34000, 2), (1, 34000, 3),                                          # with the scan kernel
])
def test_generic_merge_short_chunks(H, n, gap):
    # fp32 / d = 64, two sequences, one of them with chunks long enough for the items of other calls, appended to three rows: the
    # same bits as with a fixed item size, and the oracle's rows
    rng = np.random.default_rng(int(10 * gap) + n)
    mask = np.zeros((2, n), dtype=np.uint8)
    at = np.floor(np.arange(1, int((n - 1) / gap) + 1) * gap).astype(np.int64) - 1
    mask[0, at] = 1
    mask[1, 30::31] = 1
    K = rng.standard_normal((2, H, n, 64)).astype(np.float32)
    K[:, :, 1::2] = K[:, :, :n - n % 2:2] + 0.1 * K[:, :, 1::2]
    V = rng.standard_normal((2, H, n, 64)).astype(np.float32)
    dK, dV = torch.from_numpy(K).to(g.DEV), torch.from_numpy(V).to(g.DEV)
    offsets, num_chunks, _ = g.run_segment(mask, None)
    base = torch.full((2, H), 3, dtype=torch.int32, device=g.DEV)

    def call():
        Kc, Vc = (torch.zeros((2, H, n + 3, 64), dtype=torch.float32, device=g.DEV) for _ in range(2))
        counts = torch.zeros((2, H, n + 3), dtype=torch.int32, device=g.DEV)
        out = sc.sc_gsc_merge(dK, dV, offsets, num_chunks, 0.7, cap=n + 3, Kc=Kc, Vc=Vc, counts=counts, base_lens=base,
                              comp_lens=torch.zeros_like(base), want_cluster_id=True)
        torch.cuda.synchronize()
        return out
    got = call()
    sc.tune_set("gsc_chunks_per_item", 3)
    try:
        fixed = call()
    finally:
        sc.tune_set("gsc_chunks_per_item", 0)
    for a, b in zip(got, fixed):
        assert torch.equal(a, b)
    for b in range(2):
        ref = oracle.compress_head(K[b, H - 1], V[b, H - 1], oracle.segment(mask[b], n), 0.7)
        assert int(got[3][b, H - 1]) == 3 + ref["n_rows"]
        assert np.array_equal(got[4][b, H - 1].cpu().numpy(), ref["cid"])
        assert np.array_equal(got[2][b, H - 1, 3:3 + ref["n_rows"]].cpu().numpy(), ref["counts"][:ref["n_rows"]])


@pytest.mark.parametrize("H,n,gaps", [
    (1, 3000, [11, 13]), (1, 3000, [11, 12]),                       # chunks of twelve tokens on average, and of fewer
    (2, 1500, [8, 24, 9, 8, 24]), (2, 1500, [8, 8, 8, 8, 30]),      # room on the chip: split from 9 tokens on; some items are, others not
    (8, 6000, [32, 33, 2, 3, 5]), (8, 6000, [32, 31, 2, 3, 5]),     # none: from 33 tokens on; more items than second workgroups
    (5, 4000, [40, 2, 2, 2]),                                       # long chunks among short ones, eleven tokens on average
    (3, 5000, [2600, 7, 900]), (600, 80, [30, 40]),                 # one beyond the cluster indices held in LDS; more heads than second workgroups
])
def test_generic_merge_split_items(H, n, gaps):
    # keys and values of an item by a workgroup each, or both by one: the same bits as in a call of so many rows that no item is split, and
    # the oracle's rows.  Two sequences, one a token shorter.
    rng = np.random.default_rng(n + H)
    lens = np.array([n, n - 1], np.int32)
    wide = min(32768, 49152 // (2 * H) + n)
    mask = np.zeros((2, wide), dtype=np.uint8)
    for b in range(2):
        at = np.cumsum(np.roll(np.resize(gaps, n), b)) - 1
        mask[b, at[at < lens[b]]] = 1
    K, V = (rng.standard_normal((2, H, wide, 64)).astype(np.float32) for _ in range(2))
    K[:, :, 3:n] = K[:, :, np.arange(3, n) % 3] + 0.1 * K[:, :, 3:n]
    out = []
    for N in (n, wide):
        offsets, num_chunks, sl = g.run_segment(np.ascontiguousarray(mask[:, :N]), lens)
        dK, dV = (torch.from_numpy(np.ascontiguousarray(x[:, :, :N])).to(g.DEV) for x in (K, V))
        Kc, Vc = (torch.zeros((2, H, n, 64), dtype=torch.float32, device=g.DEV) for _ in range(2))
        counts = torch.zeros((2, H, n), dtype=torch.int32, device=g.DEV)
        out.append(sc.sc_gsc_merge(dK, dV, offsets, num_chunks, 0.7, seq_lens=sl, cap=n, Kc=Kc, Vc=Vc, counts=counts)[:4])
    torch.cuda.synchronize()
    for a, b in zip(*out):
        assert torch.equal(a, b)
    for b, h in ((0, 0), (1, H - 1)):
        m = int(lens[b])
        ref = oracle.compress_head(K[b, h, :m], V[b, h, :m], oracle.segment(mask[b], m), 0.7)
        rows = ref["n_rows"]
        assert int(out[0][3][b, h]) == rows and np.array_equal(out[0][2][b, h, :rows].cpu().numpy(), ref["counts"][:rows])
        # fp32 sums of up to l members in member order: (l + 1) half-ulps of the largest partial sum, relative to the mean
        tol = 2.0 ** -24 * (int(ref["counts"][:rows].max()) + 2)
        for got, want, x in ((out[0][0], ref["Kc"], K), (out[0][1], ref["Vc"], V)):
            assert np.abs(got[b, h, :rows].cpu().numpy() - want[:rows]).max() <= tol * np.abs(x[b, h, :m]).max()


@pytest.mark.parametrize("d,bf16,G,tail", [(128, True, 4, 0), (128, True, 7, 40), (64, True, 2, 0), (64, False, 1, 25), (128, False, 3, 0)])
def test_heads_of_one_split(d, bf16, G, tail):
    # heads that one workgroup takes alone store their outputs directly, beside heads of several splits in the same launch: no rows at
    # all, one row, remainders of a step, the last count of one split and the first of two, of a step for every split and of two
    rng = np.random.default_rng(d + G)
    step, alone = (96, 3) if bf16 and d == 128 else (8192 // d, 2)
    rows = np.array([[0, 1], [17, step], [alone * step, alone * step + 1], [24 * step, 24 * step + 1]], np.int32)
    rows = np.maximum(rows - np.where(rows > step, tail, 0), 0).astype(np.int32)
    B, H, cap = 4, 2, 24 * step + 3
    Kc, Vc = (g.to_device(rng.standard_normal((B, H, cap, d)).astype(np.float32), bf16) for _ in range(2))
    Q = g.to_device(rng.standard_normal((B, H * G, d)).astype(np.float32), bf16)
    counts = torch.from_numpy(rng.integers(1, 30, size=(B, H, cap)).astype(np.int32)).to(g.DEV)
    lens = torch.from_numpy(rows).to(g.DEV)
    ws = sc.decode_attn_workspace(B, H * G, H, cap, d, g.DEV)
    host = [x.float().cpu().numpy() for x in (Q, Kc, Vc)]
    if tail:
        Kt, Vt = (g.to_device(rng.standard_normal((B, H, tail, d)).astype(np.float32), bf16) for _ in range(2))
        tl = torch.full((B,), tail, dtype=torch.int32, device=g.DEV)
        O, lse = sc.sc_decode_attn(Q, Kc, Vc, counts, lens, want_lse=True, workspace=ws, Kt=Kt, Vt=Vt, tail_lens=tl)
        want, want_lse = oracle.decode_attn_tail(*host, counts.cpu().numpy(), rows, Kt.float().cpu().numpy(), Vt.float().cpu().numpy(), tl.cpu().numpy())
    else:
        O, lse = sc.sc_decode_attn(Q, Kc, Vc, counts, lens, want_lse=True, workspace=ws)
        want, want_lse = oracle.decode_attn(*host, counts.cpu().numpy(), rows)
    torch.cuda.synchronize()
    got, got_lse = O.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    seen = np.isfinite(want_lse)
    assert np.array_equal(np.isneginf(got_lse), np.isneginf(want_lse)) and (got[~seen] == 0).all()
    # bf16: half an ulp of the stored result (2^-8 of it) is the larger part, fp32: sums of up to 400 terms
    assert np.abs(got - want).max() <= (4e-3 if bf16 else 2e-5) * max(1.0, np.abs(want).max())
    assert np.abs(got_lse[seen] - want_lse[seen]).max() <= 1e-3


@pytest.mark.parametrize("d,bf16,H,rows", [(128, True, 1, 12287), (128, True, 2, 20000), (64, False, 1, 12289), (128, False, 4, 6200)])
def test_a_few_heads_with_many_rows_take_up_to_64_splits(d, bf16, H, rows):
    rng = np.random.default_rng(rows)
    G, cap = 3, rows + 5
    Kc, Vc = (g.to_device(rng.standard_normal((1, H, cap, d)).astype(np.float32), bf16) for _ in range(2))
    Q = g.to_device(rng.standard_normal((1, H * G, d)).astype(np.float32), bf16)
    counts = rng.integers(1, 30, size=(1, H, cap)).astype(np.int32)
    lens = np.full((1, H), rows, np.int32)
    O, lse = sc.sc_decode_attn(Q, Kc, Vc, torch.from_numpy(counts).to(g.DEV), torch.from_numpy(lens).to(g.DEV), want_lse=True)
    torch.cuda.synchronize()
    want, want_lse = oracle.decode_attn(*[x.float().cpu().numpy() for x in (Q, Kc, Vc)], counts, lens)
    # bf16: half an ulp of the stored result is the larger part; fp32: sums of 20000 terms
    assert np.abs(O.float().cpu().numpy() - want).max() <= (4e-3 if bf16 else 2e-5) * max(1.0, np.abs(want).max())
    assert np.abs(lse.cpu().numpy() - want_lse).max() <= 1e-3


def test_calls_that_the_native_marshalling_leaves_to_the_wrappers():
    # what _native does not take (-1) ends as it did before: in the general path or in its error; what it takes gives the same
    rng = np.random.default_rng(9)
    B, H, G, cap, d = 2, 2, 2, 70, 128
    Kc, Vc = (g.to_device(rng.standard_normal((B, H, cap, d)).astype(np.float32), True) for _ in range(2))
    Q = g.to_device(rng.standard_normal((B, H * G, d)).astype(np.float32), True)
    counts = torch.ones((B, H, cap), dtype=torch.int32, device=g.DEV)
    lens = torch.full((B, H), cap - 3, dtype=torch.int32, device=g.DEV)
    ws = sc.decode_attn_workspace(B, H * G, H, cap, d, g.DEV)
    want, _ = sc.sc_decode_attn(Q, Kc, Vc, counts, lens, workspace=ws)                      # allocates: the general path
    O = torch.empty_like(Q)
    stream = sc._stream()

    def native(q=Q, o=O, kc=Kc, n=lens):
        return sc._native.decode(q, kc, Vc, counts, n, 0.0, o, None, None, None, None, ws.ptr, ws.nbytes, stream)
    assert native() == 0 and torch.equal(O, want)
    sub = type("Sub", (torch.Tensor,), {})
    for other in (Q.cpu(), Q.double(), Q[0], Q.transpose(0, 1), Q.as_subclass(sub), None, 3):
        assert native(q=other) == -1
    assert native(kc=Kc.transpose(2, 3)) == -1 and native(o=O.double()) == -1 and native(n=lens.cpu()) == -1
    with pytest.raises(sc.SemantiCacheError, match="contiguous"):
        sc.sc_decode_attn(Q, Kc.transpose(2, 3).contiguous().transpose(2, 3), Vc, counts, lens, O=O, workspace=ws)
    with pytest.raises(sc.SemantiCacheError, match="dtype"):
        sc.sc_decode_attn(Q, Kc, Vc, counts, lens, O=O.double(), workspace=ws)
    small = sc.Workspace(256, g.DEV)
    with pytest.raises(sc.SemantiCacheError, match="sc_decode_attn failed"):                # the library's own refusal
        sc.sc_decode_attn(Q, Kc, Vc, counts, lens, O=O, workspace=small)
    got, _ = sc.sc_decode_attn(Q.as_subclass(sub), Kc, Vc, counts, lens, O=O.zero_(), workspace=ws)
    assert torch.equal(got, want)
    got, _ = sc.sc_decode_attn(torch.nn.Parameter(Q), Kc, Vc, counts, lens, O=O.zero_(), workspace=ws)
    assert torch.equal(got, want)


def test_native_marshalling_and_the_wrappers_agree(monkeypatch):
    # every call that _native takes, with it and without it: the same outputs bit for bit, and the same refusals
    rng = np.random.default_rng(10)
    B, H, G, n, d, nq, tcap = 2, 2, 3, 200, 128, 5, 9
    K, V = (g.to_device(rng.standard_normal((B, H, n, d)).astype(np.float32), True) for _ in range(2))
    K[:, :, 1::2] = K[:, :, ::2]
    mask = torch.zeros((B, n), dtype=torch.uint8, device=g.DEV)
    mask[:, 9::10] = 1
    seq = torch.tensor([n, n - 33], dtype=torch.int32, device=g.DEV)
    Q, Qn = (g.to_device(rng.standard_normal(s).astype(np.float32), True) for s in ((B, H * G, d), (nq, B, H * G, d)))
    Kt, Vt = (g.to_device(rng.standard_normal((B, H, tcap, d)).astype(np.float32), True) for _ in range(2))
    tail = torch.tensor([tcap, 6], dtype=torch.int32, device=g.DEV)
    ws = sc.gsc_merge_workspace(B, H, n, d, g.DEV, torch.bfloat16)
    ws_d = sc.decode_attn_workspace(B, H * G, H, 2 * n, d, g.DEV)
    ws_m = sc.Workspace(sc.load_library().sc_multi_attn_workspace_bytes(B, H * G, H, nq, 2 * n + tcap, d), g.DEV)
    z = lambda *s, t=torch.bfloat16: torch.zeros(s, dtype=t, device=g.DEV)
    i32 = torch.int32

    def segment(**kw):
        a = dict(dict(mask=mask, seq_lens=seq, offsets=z(B, n + 2, t=i32), num_chunks=z(B, t=i32)), **kw)
        return sc.sc_segment(**a)
    off, nch = segment()

    def merge(**kw):
        a = dict(dict(K=K, V=V, offsets=off, num_chunks=nch, tau=0.7, seq_lens=seq, cap=2 * n, Kc=z(B, H, 2 * n, d), Vc=z(B, H, 2 * n, d), counts=z(B, H, 2 * n, t=i32),
                      comp_lens=z(B, H, t=i32), cluster_id=z(B, H, n, t=i32), workspace=ws), **kw)
        return sc.sc_gsc_merge(**a)
    Kc, Vc, counts, lens, _ = merge()
    cache = dict(Kc=Kc, Vc=Vc, counts=counts, comp_lens=lens)

    def decode(**kw):
        a = dict(dict(cache, Q=Q, O=z(B, H * G, d), lse=z(B, H * G, t=torch.float32), workspace=ws_d), **kw)
        return sc.sc_decode_attn(**a)

    def multi(**kw):
        a = dict(dict(cache, Q=Qn, O=z(nq, B, H * G, d), lse=z(nq, B, H * G, t=torch.float32), workspace=ws_m), **kw)
        return sc.sc_multi_attn(**a)
    with_tail = dict(Kt=Kt, Vt=Vt, tail_lens=tail)
    across = K.transpose(2, 3).contiguous().transpose(2, 3)
    fine = [(segment, {}), (segment, dict(seq_lens=None)), (segment, dict(mask=torch.cat([mask, mask], 1)[:, :n])), (merge, {}), (merge, dict(seq_lens=None, cluster_id=None)),
            (merge, dict(base_lens=torch.full((B, H), 7, dtype=i32, device=g.DEV))), (merge, dict(Kc=z(B, H, 2 * n, d, t=torch.float32), Vc=z(B, H, 2 * n, d, t=torch.float32),
            workspace=sc.gsc_merge_workspace(B, H, n, d, g.DEV))), (merge, dict(K=K[:, :, ::2], V=V[:, :, ::2], offsets=off[:, ::1], seq_lens=seq // 2)),
            (merge, dict(cap=np.int64(2 * n), tau=np.float32(0.7))), (decode, {}), (decode, with_tail), (decode, dict(scale=0.5, lse=None)), (multi, {}), (multi, with_tail),
            (multi, dict(with_tail, causal=True, tail_lens=torch.full((B,), tcap, dtype=i32, device=g.DEV))), (multi, dict(O=z(nq, B, H * G, d, t=torch.float32), scale=0.5))]
    refused = [(segment, dict(mask=mask.to(torch.int8))), (segment, dict(mask=mask.t())), (segment, dict(offsets=z(B, 1, t=i32))), (segment, dict(num_chunks=nch.cpu())),
               (merge, dict(K=across)), (merge, dict(V=V.float())), (merge, dict(K=K.double(), V=V.double())), (merge, dict(V=V.cpu())), (merge, dict(Kc=z(B, H, d, 2 * n).transpose(2, 3))),
               (merge, dict(cap=0)), (merge, dict(workspace=sc.Workspace(256, g.DEV))), (merge, dict(tau=float("nan"))),
               (merge, dict(base_lens=torch.full((B, H), 7, dtype=i32, device=g.DEV), cap=n)), (decode, dict(with_tail, Vt=Vt[:, :, :5])), (decode, dict(with_tail, Kt=Kt.float())),
               (decode, dict(scale=float("nan"))), (multi, dict(Kc=Kc.transpose(2, 3).contiguous().transpose(2, 3))), (multi, dict(O=z(nq, B, H * G, d, t=torch.float64))),
               (multi, dict(Q=Qn.cpu())), (multi, dict(with_tail, Kt=Kt[:, :1])), (multi, dict(with_tail, tail_lens=tail.cpu())), (multi, dict(workspace=sc.Workspace(256, g.DEV)))]
    native = sc._native
    taken = []
    for name in ("segment", "merge", "decode", "multi"):
        monkeypatch.setattr(sc._native, name, (lambda f: lambda *a: (taken.append(f(*a)), taken[-1])[1])(getattr(native, name)))
    for call, kw in fine:
        got = call(**{k: (v.clone() if k in ("Kc", "Vc", "workspace") and torch.is_tensor(v) else v) for k, v in kw.items()})
        assert taken and taken.pop() == 0 and not taken, (call.__name__, sorted(kw))
        got = [x.clone() for x in got if x is not None]
        with monkeypatch.context() as m:
            m.setattr(sc, "_native", None)
            want = [x for x in call(**kw) if x is not None]
        assert len(got) == len(want) and all(torch.equal(a, b) for a, b in zip(got, want)), (call.__name__, sorted(kw))
    for call, kw in refused:
        with pytest.raises(sc.SemantiCacheError) as first:
            call(**kw)
        with monkeypatch.context() as m:
            m.setattr(sc, "_native", None)
            with pytest.raises(sc.SemantiCacheError) as second:
                call(**kw)
        assert str(first.value) == str(second.value), (call.__name__, sorted(kw))
    torch.cuda.synchronize()
