"""GPU parity of sc_gsc_merge_global (Alg. 1 over the whole sequence as one chunk: the "no chunking"
variant of the paper's ablation, Sec. 3.4) against the oracle run on one-chunk offsets: cluster ids,
sizes and lengths bit for bit, merged rows and decode within the bounds of gpu_common."""
import dataclasses

import numpy as np
import pytest
import torch

import gpu_common as g
from helpers import build_case
from paper_2603_14303_amd import binding as sc
from paper_2603_14303_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _global_case(w, tau, **kw):
    case = build_case(w, tau, chunking="global", **kw)
    assert case["num_chunks"].tolist() == [1] * len(case["num_chunks"]) and not case["mask"].any()
    case["global_call"] = True
    return case


@pytest.mark.parametrize("n,heads,tau", [(63, 2, 0.7), (64, 1, 0.7), (1000, 2, 0.7), (8192 + 11, 2, 0.7),
                                         (3000, 2, 0.9745), (2000, 1, 1.0), (2000, 1, -1.01),
                                         (2048, 2, 0.9745), (2047, 1, 1.0), (2048, 1, 1.0), (2049, 1, 1.0), (2048, 1, -1.01)])
def test_dedicated_path(n, heads, tau):
    # blocks of 64 rows: less than one, exactly one, many with a ragged tail; a threshold inside the band of
    # the similarities (pairs decided in fp64, many clusters); no merging at all; everything in one cluster; the
    # longest sequences that one workgroup numbers, and one row more
    w = wl.get_workload("layer32k")
    case = _global_case(w, tau, n_max=n, heads=heads, exclude_near=(tau == 0.7))
    out = g.check_compress(case)
    errs = g.check_decode(case, out, range(2), q_heads=heads * w.group)
    print("global n=%d tau=%g: rows %s merge_err %.2e decode %s" % (n, tau, out["comp_lens"].tolist(), out["worst_merge_err"], errs))


def test_full_length_one_head_checked():
    # 32768 tokens, all 8 heads computed, the oracle recomputes one of them (thousands of clusters in one chunk)
    w = wl.get_workload("layer32k")
    case = _global_case(w, 0.7, sample=[(0, 3)])
    out = g.check_compress(case)
    errs = g.check_decode_sampled(case, out, [0])
    print("global full: rows", out["comp_lens"].tolist(), "merge_err %.2e" % out["worst_merge_err"], "decode", errs)


def test_ragged_batch_and_capacity():
    w = dataclasses.replace(wl.get_workload("batch_gqa7"), batch=3, kv_heads=2, q_heads=14)
    case = _global_case(w, 0.7, n_max=1500, batch=3)
    assert len(set(case["seq_lens"].tolist())) > 1
    out = g.check_compress(case)
    rows = out["comp_lens"].cpu().numpy()
    cap = int(rows.max()) - 1
    small = g.run_compress(case, torch.float32, cap=cap)
    got = small["comp_lens"].cpu().numpy()
    assert ((got == -1) == (rows > cap)).all() and (got[rows <= cap] == rows[rows <= cap]).all()
    for b in range(rows.shape[0]):
        for h in range(rows.shape[1]):
            r = min(int(rows[b, h]), cap)      # a head that does not fit still gets its first cap rows
            assert torch.equal(small["counts"][b, h, :r], out["counts"][b, h, :r])
            assert torch.equal(small["Kc"][b, h, :r], out["Kc"][b, h, :r]) and torch.equal(small["Vc"][b, h, :r], out["Vc"][b, h, :r])


@pytest.mark.parametrize("base,knob", [("tiny", None), ("layer32k", "gsc_fast_path")])
def test_other_shapes_go_through_the_ordinary_kernels(base, knob):
    # fp32 / d = 64, and bf16 / d = 128 with the dedicated path switched off: same call, same comparisons
    w = wl.get_workload(base)
    old = sc.tune_get(knob) if knob else None
    try:
        if knob:
            sc.tune_set(knob, 0)
        case = _global_case(w, 0.7, n_max=700, heads=2)
        out = g.check_compress(case)
    finally:
        if knob:
            sc.tune_set(knob, old)
    print(base, "rows", out["comp_lens"].tolist(), "merge_err %.2e" % out["worst_merge_err"])


def _run_rows(K, V, tau):
    """K, V [n, 128] float arrays (bf16-exact) as one (sequence, head): GPU call and oracle on one-chunk offsets."""
    import oracle
    n = K.shape[0]
    Kd = torch.from_numpy(K).to(g.DEV).to(torch.bfloat16).view(1, 1, n, 128)
    Vd = torch.from_numpy(V).to(g.DEV).to(torch.bfloat16).view(1, 1, n, 128)
    Kc, Vc, counts, lens, cid = sc.sc_gsc_merge_global(Kd, Vd, tau, out_dtype=torch.float32, want_cluster_id=True)
    torch.cuda.synchronize()
    ref = oracle.compress_head(K.astype(np.float64), V.astype(np.float64), np.array([0, n + 1], np.int32), tau)
    assert lens.item() == ref["n_rows"]
    assert np.array_equal(cid[0, 0].cpu().numpy(), ref["cid"])
    r = ref["n_rows"]
    assert np.array_equal(counts[0, 0, :r].cpu().numpy(), ref["counts"][:r])
    assert g.rowwise_err(Kc[0, 0, :r].cpu().numpy(), ref["Kc"][:r]) <= 1e-3
    assert g.rowwise_err(Vc[0, 0, :r].cpu().numpy(), ref["Vc"][:r]) <= 1e-3
    return ref


def _bf16_exact(x):
    return torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16).float().numpy()


def test_more_candidates_than_a_list_holds_and_none_is_a_seed():
    # Row j resembles 40 rows b_k of an earlier block, all of which were absorbed by a seed that j does not
    # resemble; the seed that does take j comes after them.  j's candidate list (32 entries) then holds no
    # seed although j has one: the kernel must go back to the bit arrays.  Unit vectors in a plane:
    # a at 0, b_k at 18, j at 36, s at 50 degrees, tau = 0.9 (cos 18 = 0.951, cos 36 = 0.809, cos 14 = 0.970, cos 32 = 0.848).
    rng = np.random.default_rng(3)
    n, d = 200, 128
    e0, e1 = np.zeros(d), np.zeros(d)
    e0[5], e1[77] = 1.0, 1.0

    def at(deg, scale=1.0):
        return scale * (np.cos(np.radians(deg)) * e0 + np.sin(np.radians(deg)) * e1)
    K = np.zeros((n, d))
    filler = rng.standard_normal((n, d))
    filler[:, 5] = 0
    filler[:, 77] = 0                      # orthogonal to the plane: resembles nothing in it
    K[:] = filler
    K[0] = at(0)
    for k in range(40):
        K[3 + k] = at(18, 1.0 + 0.1 * k)    # block 0: absorbed by row 0
    K[70] = at(50)                          # block 1: a seed (resembles neither a nor the b_k)
    K[150] = at(36)                         # block 2: candidates = 40 b_k (no seeds) and then row 70
    K[151] = at(36.5, 3.0)
    K = _bf16_exact(K)
    V = _bf16_exact(rng.standard_normal((n, d)))
    ref = _run_rows(K, V, 0.9)
    assert ref["cid"][150] == ref["cid"][70] and ref["cid"][3] == ref["cid"][0] and ref["cid"][150] != ref["cid"][0]


@pytest.mark.parametrize("n,tau,polls", [(1000, 0.25, 4096), (1000, 0.25, 0), (3000, 0.9745, 0), (64 * 64 + 65, 0.3, 4096), (700, 0.7, 0)])
def test_blocks_that_wait_for_others(n, tau, polls):
    # thresholds that random rows exceed: nearly every block has candidates in many earlier ones (batches of words, words
    # of flags beyond the first); without patience the ordered pass finishes the blocks, with the same outcome
    w = wl.get_workload("layer32k")
    old = sc.tune_get("global_polls")
    try:
        sc.tune_set("global_polls", polls)
        case = _global_case(w, tau, n_max=n, heads=2)
        out = g.check_compress(case)
    finally:
        sc.tune_set("global_polls", old)
    print("n=%d tau=%g polls=%d rows %s" % (n, tau, polls, out["comp_lens"].tolist()))


@pytest.mark.parametrize("n,step,tau,polls", [(700, 0.2, 0.9, 4096), (700, 0.4, 0.8, 0), (900, 0.1, 0.8, 4096), (700, 0.05, 0.99875, 4096)])
def test_rows_that_drift(n, step, tau, polls):
    # every row resembles its neighbours: chains through a block, taken in order, from block to block; clusters of a few
    # rows, of dozens, and (last) neighbours whose cosines lie in the band that fp64 settles
    rng = np.random.default_rng(n)
    K = rng.standard_normal((n, 128))
    for i in range(1, n):
        K[i] = np.sqrt(1 - step * step) * K[i - 1] + step * K[i]
    K[200:203] = 0.0
    old = sc.tune_get("global_polls")
    try:
        sc.tune_set("global_polls", polls)
        ref = _run_rows(_bf16_exact(K), _bf16_exact(rng.standard_normal((n, 128))), tau)
    finally:
        sc.tune_set("global_polls", old)
    assert 4 < ref["n_rows"] < 0.8 * n


def test_zero_rows_duplicates_and_scaled_rows():
    # zero rows resemble nothing (also inside a block and across blocks), exact duplicates and scaled copies merge
    rng = np.random.default_rng(5)
    n, d = 300, 128
    K = rng.standard_normal((n, d))
    K[10] = 0; K[11] = 0; K[200] = 0
    K[50] = K[40]; K[130] = K[40] * 3.0; K[270] = K[40] * 0.01; K[271] = K[41]
    K = _bf16_exact(K)
    K[130] = _bf16_exact(K[40] * 4.0)       # exact in bf16: a power of two
    K[270] = _bf16_exact(K[40] * 0.0078125)
    V = _bf16_exact(rng.standard_normal((n, d)))
    ref = _run_rows(K, V, 0.999)
    for j in (50, 130, 270):
        assert ref["cid"][j] == ref["cid"][40]
    assert ref["cid"][271] == ref["cid"][41] and len({ref["cid"][10], ref["cid"][11], ref["cid"][200]}) == 3


@pytest.mark.parametrize("seed", range(8))
def test_random_structures_as_one_chunk(seed):
    # the key mixtures of test_gpu_random.py (centres drawn per stretch, duplicates, zero rows, rows scaled by 0.01
    # and 30, thresholds inside the similarity bands) clustered as ONE chunk per sequence: ragged batch of three
    import oracle
    from test_gpu_random import _random_mask, _random_keys
    rng = np.random.default_rng(1000 + seed)
    B, H, d = 3, 2, 128
    N = int(rng.integers(100, 1200))
    lens = rng.integers(1, N + 1, size=B).astype(np.int32)
    lens[0] = N
    K = np.zeros((B, H, N, d), np.float32)
    V = np.zeros_like(K)
    for b in range(B):
        n = int(lens[b])
        shape_mask = _random_mask(rng, n)          # shapes the keys only; the clustering sees no boundary
        for h in range(H):
            K[b, h, :n], V[b, h, :n] = _random_keys(rng, shape_mask, n, d, True)
    tau = float(rng.choice([0.3, 0.7, 0.9, 0.97, 0.985, 0.995, 0.9999, -0.5]))
    dK, dV = g.to_device(K, True), g.to_device(V, True)
    sl = torch.from_numpy(lens).to(g.DEV)
    Kc, Vc, counts, clens, cid = sc.sc_gsc_merge_global(dK, dV, tau, seq_lens=sl, out_dtype=torch.float32, want_cluster_id=True)
    torch.cuda.synchronize()
    compared = 0
    for b in range(B):
        n = int(lens[b])
        for h in range(H):
            r = oracle.compress_head(K[b, h, :n], V[b, h, :n], np.array([0, n + 1], np.int32), tau)
            if r["chunk_margin"].min() <= 1e-9:
                continue                                             # a coin toss in fp64 itself: not a parity case
            compared += 1
            rows = r["n_rows"]
            assert int(clens[b, h]) == rows, (seed, b, h, int(clens[b, h]), rows)
            assert np.array_equal(cid[b, h, :n].cpu().numpy(), r["cid"]), (seed, b, h)
            assert np.array_equal(counts[b, h, :rows].cpu().numpy(), r["counts"][:rows]), (seed, b, h)
            assert g.rowwise_err(Kc[b, h, :rows].cpu().numpy(), r["Kc"][:rows]) <= 1e-3
            assert g.rowwise_err(Vc[b, h, :rows].cpu().numpy(), r["Vc"][:rows]) <= 1e-3
    assert compared >= (B * H + 1) // 2, (seed, compared)
    print("seed", seed, "compared", compared, "N", N, "tau", tau, "rows", clens.cpu().numpy().tolist())


@pytest.mark.parametrize("tau,polls,drift,B,H,N", [
    # 12365 rows, two stages of 8192 and the rest
    (0.7, 1 << 20, 0.0, 2, 8, 12365), (0.9745, 1 << 20, 0.0, 2, 8, 12365), (0.9745, 0, 0.0, 2, 8, 12365), (0.8, 1 << 20, 0.4, 2, 8, 12365),
    (0.99875, 0, 0.05, 2, 8, 12365),
    # three stages of 4096, the last one with 77 rows more
    (0.9745, 1 << 20, 0.0, 4, 8, 12365), (0.9745, 0, 0.0, 4, 8, 12365), (0.8, 1 << 20, 0.4, 4, 8, 12365),
    # five of 4096, the last one with fewer rows; two of 4096 and 65 rows more; eight, with items of 32 column blocks
    (0.9745, 1 << 20, 0.0, 4, 8, 20000), (0.9745, 0, 0.0, 4, 8, 20000), (0.9745, 0, 0.0, 2, 32, 8257), (0.9745, 1 << 20, 0.0, 4, 8, 32768),
])
def test_sequences_long_enough_for_stages(tau, polls, drift, B, H, N):
    # Rows of the second stage are compared with the seeds of the first, listed without gaps (pairs decided in fp64 among them); one
    # sequence ends inside another stage's first blocks, one inside the first stage where rows drift.
    # Rows that drift: chains that a stage ends in the middle of; without patience every stage is finished by its last wavefront.
    import oracle
    rng = np.random.default_rng(int(1000 * tau) + polls % 7)
    tau = float(np.float32(tau))      # the call takes a float: the oracle compares with the same number (3e-8 from 0.99875, and a pair lies between)
    d, kinds = 128, 4      # heads of their own keys, the others have the same
    lens = np.full((B,), N, np.int32)
    lens[:2] = [N, 5003] if drift else [8192 + 65, N]
    look = [(0, 1), (1, 2)]
    if drift:
        base = rng.standard_normal((kinds, N, d)).astype(np.float32)
        for i in range(1, N):
            base[:, i] = np.sqrt(1 - drift * drift) * base[:, i - 1] + drift * base[:, i]
        base[:, 8190:8195] = 0.0
        base[:, 4094:4098] = 0.0
    else:
        centers = rng.standard_normal((kinds, N // 24, d)).astype(np.float32)
        near = np.clip(np.arange(N) // 24 + rng.integers(-6, 7, size=N), 0, N // 24 - 1)
        near[::97] = rng.integers(0, N // 24, size=len(near[::97]))      # some resemble rows of other stages
        base = centers[:, near] + 0.15 * rng.standard_normal((kinds, N, d)).astype(np.float32)
    base = _bf16_exact(base)
    values = _bf16_exact(rng.standard_normal((kinds, N, d)))
    which = (np.arange(B * H) % kinds).reshape(B, H)
    at = torch.from_numpy(which).to(g.DEV)
    Kd, Vd = g.to_device(base, True)[at], g.to_device(values, True)[at]
    K = {bh: base[which[bh]] for bh in look}
    V = {bh: values[which[bh]] for bh in look}
    old = sc.tune_get("global_polls")
    try:
        sc.tune_set("global_polls", polls)
        Kc, Vc, counts, clens, cid = sc.sc_gsc_merge_global(Kd, Vd, tau, seq_lens=torch.from_numpy(lens).to(g.DEV), out_dtype=torch.float32,
                                                            want_cluster_id=True)
        torch.cuda.synchronize()
    finally:
        sc.tune_set("global_polls", old)
    for b, h in look:
        n = int(lens[b])
        r = oracle.compress_head(K[b, h][:n], V[b, h][:n], np.array([0, n + 1], np.int32), tau)
        assert r["chunk_margin"].min() > 1e-9
        rows = r["n_rows"]
        assert int(clens[b, h]) == rows
        assert np.array_equal(cid[b, h, :n].cpu().numpy(), r["cid"])
        assert np.array_equal(counts[b, h, :rows].cpu().numpy(), r["counts"][:rows])
        assert g.rowwise_err(Kc[b, h, :rows].cpu().numpy(), r["Kc"][:rows]) <= 1e-3
        assert g.rowwise_err(Vc[b, h, :rows].cpu().numpy(), r["Vc"][:rows]) <= 1e-3
        print("b %d h %d: rows %d of %d" % (b, h, rows, n))


def test_stages_in_a_captured_graph():
    # the launches of a staged call, replayed on new keys with eager work in between, give what an eager call gives
    gen = torch.Generator(g.DEV).manual_seed(4)
    H, N, d = 16, 12365, 128
    K = torch.empty((1, H, N, d), dtype=torch.bfloat16, device=g.DEV)
    V = torch.empty_like(K)

    def fill():
        centers = torch.randn((H, 700, d), generator=gen, device=g.DEV)
        pick = torch.randint(0, 700, (H, N), generator=gen, device=g.DEV)
        K[0] = (torch.gather(centers, 1, pick[:, :, None].expand(-1, -1, d)) + 0.1 * torch.randn((H, N, d), generator=gen, device=g.DEV)).to(torch.bfloat16)
        V.normal_(generator=gen)
    fill()
    lib = sc.load_library()
    ws = sc.Workspace(lib.sc_gsc_merge_global_workspace_bytes(1, H, N, d), g.DEV)
    Kc, Vc = torch.zeros((1, H, N, d), device=g.DEV), torch.zeros((1, H, N, d), device=g.DEV)
    counts, lens = torch.zeros((1, H, N), dtype=torch.int32, device=g.DEV), torch.zeros((1, H), dtype=torch.int32, device=g.DEV)

    def call():
        st = lib.sc_gsc_merge_global(K.data_ptr(), V.data_ptr(), sc.SC_BF16, K.stride(0), K.stride(1), K.stride(2), None, 1, H, N, d, 0.9, Kc.data_ptr(),
                                     Vc.data_ptr(), sc.SC_F32, N, counts.data_ptr(), lens.data_ptr(), None, ws.ptr, ws.nbytes, sc._stream())
        assert st == sc.SC_OK
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for _ in range(3):
        fill()
        want = sc.sc_gsc_merge_global(K, V, 0.9, out_dtype=torch.float32)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(lens, want[3]) and (lens > 500).all()
        for h in range(H):
            r = int(lens[0, h])
            assert torch.equal(counts[0, h, :r], want[2][0, h, :r])
            assert torch.equal(Kc[0, h, :r], want[0][0, h, :r]) and torch.equal(Vc[0, h, :r], want[1][0, h, :r])
