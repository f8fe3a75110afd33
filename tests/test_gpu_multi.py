"""GPU parity for sc_multi_attn (Eq. 4 with a matrix of query rows, Sec. 2.4) against the CPU oracle.

Same bounds as for single-row decode on the same cache: <= 4e-3 * max(1, |O|) with bf16 output (half an ulp of the
output; on the matrix-core path the probabilities enter as two bf16 parts, 2^-18 at most per term), 2e-5 with
fp32 output through the row-by-row path; lse <= 1e-3."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_14303_amd import binding as sc
from paper_2603_14303_amd import workloads as wl

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_common as g


def _round_like(x, bf16):
    return wl.round_to_bf16(x.astype(np.float32)) if bf16 else x.astype(np.float32)


@pytest.mark.parametrize("bf16,d,Hkv,G,B,cap,nq", [
    (True, 128, 8, 4, 1, 6000, 16),      # two row blocks per KV head, many splits
    (True, 128, 4, 7, 3, 1500, 5),       # 35 rows: a full block and a ragged one, G does not divide 32
    (True, 128, 2, 1, 2, 300, 1),        # a single query row (one lane of a tile in use)
    (True, 128, 2, 8, 1, 40, 9),         # cache shorter than one step
    (False, 64, 2, 2, 2, 300, 3),        # row by row through the decode kernels, fp32
])
def test_multi_attn_against_oracle(bf16, d, Hkv, G, B, cap, nq):
    rng = np.random.default_rng(500 + cap + nq)
    Hq = Hkv * G
    Q = _round_like(rng.standard_normal((nq, B, Hq, d)), bf16)
    Kc, Vc = _round_like(rng.standard_normal((B, Hkv, cap, d)), bf16), _round_like(rng.standard_normal((B, Hkv, cap, d)), bf16)
    counts = rng.integers(1, 40, (B, Hkv, cap)).astype(np.int32)
    lens = rng.integers(cap // 2, cap + 1, (B, Hkv)).astype(np.int32)
    lens[0, 0] = cap
    lens[-1, -1] = 0
    dQ, dKc, dVc = g.to_device(Q, bf16), g.to_device(Kc, bf16), g.to_device(Vc, bf16)
    dcounts, dlens = torch.from_numpy(counts).to(g.DEV), torch.from_numpy(lens).to(g.DEV)
    want_O, want_L = oracle.multi_attn(Q, Kc, Vc, counts, lens)
    tol = 4e-3 if bf16 else 2e-5
    for trial in range(2):       # twice on one workspace: it carries no state
        if trial == 0:
            ws = sc.Workspace(sc.load_library().sc_multi_attn_workspace_bytes(B, Hq, Hkv, nq, cap, d), g.DEV)
        O, lse = sc.sc_multi_attn(dQ, dKc, dVc, dcounts, dlens, want_lse=True, workspace=ws)
        torch.cuda.synchronize()
        got = O.float().cpu().numpy().astype(np.float64)
        err = np.abs(got - want_O) / np.maximum(1.0, np.abs(want_O))
        assert err.max() <= tol, (trial, err.max(), np.unravel_index(err.argmax(), err.shape))
        got_l = lse.cpu().numpy().astype(np.float64)
        finite = np.isfinite(want_L)
        assert np.array_equal(np.isneginf(got_l), np.isneginf(want_L))
        assert np.abs(got_l[finite] - want_L[finite]).max() <= 1e-3
    # one query row of the call is what sc_decode_attn gives for that row (same cache, same tolerance)
    Od, _ = sc.sc_decode_attn(dQ[nq - 1].contiguous(), dKc, dVc, dcounts, dlens)
    torch.cuda.synchronize()
    diff = (Od.float() - O[nq - 1].float()).abs().max().item()
    assert diff <= 2 * tol * max(1.0, float(np.abs(want_O).max())), diff


def test_multi_attn_on_a_compressed_layer():
    # the real pipeline: compress a truncated layer, then 8 query rows over it; fp32 output to see the
    # kernel's own error against the oracle on the same cache
    from helpers import build_case
    w = wl.get_workload("layer32k")
    case = build_case(w, 0.7, n_max=4096 + 37, heads=3)
    out = g.run_compress(case, torch.bfloat16)
    nq, Hq = 8, 3 * w.group
    Q = np.stack([wl.queries(w, 0, s)[:1, :Hq] for s in range(nq)])
    dQ = g.to_device(Q, True)
    O32 = torch.empty((nq, 1, Hq, w.head_dim), dtype=torch.float32, device=g.DEV)
    O, lse = sc.sc_multi_attn(dQ, out["Kc"], out["Vc"], out["counts"], out["comp_lens"], O=O32, want_lse=True)
    torch.cuda.synchronize()
    gK, gV = out["Kc"].float().cpu().numpy(), out["Vc"].float().cpu().numpy()
    want_O, want_L = oracle.multi_attn(Q, gK, gV, out["counts"].cpu().numpy(), out["comp_lens"].cpu().numpy())
    err = np.abs(O.cpu().numpy() - want_O).max()
    assert err <= 4e-3 * max(1.0, np.abs(want_O).max()), err
    assert np.abs(lse.cpu().numpy() - want_L).max() <= 1e-3
    print("multi_attn on compressed layer: err %.2e" % err)


@pytest.mark.parametrize("Hkv,G,B,cap,tcap,nq,causal", [
    (8, 4, 1, 6000, 300, 16, True),      # two row blocks, tail spread over the last splits
    (4, 7, 3, 1500, 64, 5, True),        # ragged row blocks, per-sequence tails, one shorter than the query block
    (2, 2, 2, 300, 40, 3, False),        # no mask
    (2, 8, 1, 40, 100, 9, True),         # tail longer than the merged cache
])
def test_multi_attn_tail_against_oracle(Hkv, G, B, cap, tcap, nq, causal):
    rng = np.random.default_rng(900 + cap + nq)
    Hq, d = Hkv * G, 128
    Q = _round_like(rng.standard_normal((nq, B, Hq, d)), True)
    Kc, Vc = _round_like(rng.standard_normal((B, Hkv, cap, d)), True), _round_like(rng.standard_normal((B, Hkv, cap, d)), True)
    Kt, Vt = _round_like(rng.standard_normal((B, Hkv, tcap, d)), True), _round_like(rng.standard_normal((B, Hkv, tcap, d)), True)
    counts = rng.integers(1, 40, (B, Hkv, cap)).astype(np.int32)
    lens = rng.integers(cap // 2, cap + 1, (B, Hkv)).astype(np.int32)
    lens[-1, -1] = 0
    tails = rng.integers(nq, tcap + 1, (B,)).astype(np.int32)
    if B > 1:
        tails[1] = max(1, nq - 2)                                   # fewer tail rows than query rows
    dQ, dKc, dVc = g.to_device(Q, True), g.to_device(Kc, True), g.to_device(Vc, True)
    dKt, dVt = g.to_device(Kt, True), g.to_device(Vt, True)
    dcounts, dlens = torch.from_numpy(counts).to(g.DEV), torch.from_numpy(lens).to(g.DEV)
    dtails = torch.from_numpy(tails).to(g.DEV)
    O, lse = sc.sc_multi_attn(dQ, dKc, dVc, dcounts, dlens, want_lse=True, Kt=dKt, Vt=dVt, tail_lens=dtails, causal=causal)
    torch.cuda.synchronize()
    want_O, want_L = oracle.multi_attn_tail(Q, Kc, Vc, counts, lens, Kt, Vt, tails, causal)
    got = O.float().cpu().numpy().astype(np.float64)
    err = np.abs(got - want_O) / np.maximum(1.0, np.abs(want_O))
    assert err.max() <= 4e-3, (err.max(), np.unravel_index(err.argmax(), err.shape))
    got_l = lse.cpu().numpy().astype(np.float64)
    finite = np.isfinite(want_L)
    assert np.array_equal(np.isneginf(got_l), np.isneginf(want_L))
    assert np.abs(got_l[finite] - want_L[finite]).max() <= 1e-3
    # one query row, no mask: what sc_decode_attn with the same tail gives (either kernel, same tolerance)
    O1, _ = sc.sc_multi_attn(dQ[:1].contiguous(), dKc, dVc, dcounts, dlens, Kt=dKt, Vt=dVt, tail_lens=dtails)
    Od, _ = sc.sc_decode_attn(dQ[0].contiguous(), dKc, dVc, dcounts, dlens, Kt=dKt, Vt=dVt, tail_lens=dtails)
    torch.cuda.synchronize()
    assert (O1[0].float() - Od.float()).abs().max().item() <= 8e-3 * max(1.0, float(np.abs(want_O).max()))


def test_multi_attn_tail_mask_needs_the_matrix_core_path():
    B, Hkv, G, cap, tcap, nq, d = 1, 2, 1, 64, 16, 2, 64
    z = lambda *s: torch.zeros(s, dtype=torch.float32, device=g.DEV)
    with pytest.raises(sc.SemantiCacheError, match="UNSUPPORTED"):
        sc.sc_multi_attn(z(nq, B, Hkv * G, d), z(B, Hkv, cap, d), z(B, Hkv, cap, d),
                         torch.ones((B, Hkv, cap), dtype=torch.int32, device=g.DEV),
                         torch.full((B, Hkv), cap, dtype=torch.int32, device=g.DEV), Kt=z(B, Hkv, tcap, d),
                         Vt=z(B, Hkv, tcap, d), tail_lens=torch.full((B,), tcap, dtype=torch.int32, device=g.DEV), causal=True)
    # without the mask the same shapes go row by row through the decode kernels
    O, _ = sc.sc_multi_attn(z(nq, B, Hkv * G, d), z(B, Hkv, cap, d), z(B, Hkv, cap, d) + 2.0,
                            torch.ones((B, Hkv, cap), dtype=torch.int32, device=g.DEV),
                            torch.full((B, Hkv), cap, dtype=torch.int32, device=g.DEV), Kt=z(B, Hkv, tcap, d),
                            Vt=z(B, Hkv, tcap, d) + 2.0, tail_lens=torch.full((B,), tcap, dtype=torch.int32, device=g.DEV))
    torch.cuda.synchronize()
    assert torch.allclose(O, torch.full_like(O, 2.0), atol=1e-5)


@pytest.mark.parametrize("nq,tcap", [(7, 0), (7, 30), (33, 0), (33, 70)])      # 28 and 132 query rows per KV head
@pytest.mark.parametrize("knobs", [
    dict(multi_block_rows=32, multi_target_wgs=64), dict(multi_block_rows=128, multi_target_wgs=1024),
    dict(multi_block_rows=32, multi_target_wgs=1024), dict(multi_block_rows=128, multi_target_wgs=8),
])
def test_multi_attn_launch_shapes(knobs, nq, tcap):
    # either kernel with rows for a part of its workgroup and for several of them, few and many splits, without a tail and with
    # a masked one: the workspace query and the launch follow the same knobs, the result stays within the bound of the default
    # shape, and a decode workspace made before serves sc_decode_attn as before
    rng = np.random.default_rng(641)
    B, Hkv, G, cap, d = 2, 4, 4, 3000, 128
    Hq = Hkv * G
    Q = _round_like(rng.standard_normal((nq, B, Hq, d)), True)
    Kc, Vc = _round_like(rng.standard_normal((B, Hkv, cap, d)), True), _round_like(rng.standard_normal((B, Hkv, cap, d)), True)
    counts = rng.integers(1, 40, (B, Hkv, cap)).astype(np.int32)
    lens = rng.integers(cap // 2, cap + 1, (B, Hkv)).astype(np.int32)
    lens[0, 0] = cap
    tail = {}
    if tcap:
        Kt, Vt = _round_like(rng.standard_normal((B, Hkv, tcap, d)), True), _round_like(rng.standard_normal((B, Hkv, tcap, d)), True)
        tails = np.array([tcap, nq + 1], np.int32)
        want_O, want_L = oracle.multi_attn_tail(Q, Kc, Vc, counts, lens, Kt, Vt, tails, True)
        tail = dict(Kt=g.to_device(Kt, True), Vt=g.to_device(Vt, True), tail_lens=torch.from_numpy(tails).to(g.DEV), causal=True)
    else:
        want_O, want_L = oracle.multi_attn(Q, Kc, Vc, counts, lens)
    dQ, dKc, dVc = g.to_device(Q, True), g.to_device(Kc, True), g.to_device(Vc, True)
    dcounts, dlens = torch.from_numpy(counts).to(g.DEV), torch.from_numpy(lens).to(g.DEV)
    ws = sc.decode_attn_workspace(B, Hq, Hkv, cap, d, g.DEV)
    want_D, _ = sc.sc_decode_attn(dQ[0].contiguous(), dKc, dVc, dcounts, dlens, workspace=ws)
    old = {k: sc.tune_get(k) for k in knobs}
    try:
        for k, v in knobs.items():
            sc.tune_set(k, v)
        O, lse = sc.sc_multi_attn(dQ, dKc, dVc, dcounts, dlens, want_lse=True, **tail)
        if knobs["multi_target_wgs"] <= 256:      # (a larger target may ask for a larger workspace)
            got_D, _ = sc.sc_decode_attn(dQ[0].contiguous(), dKc, dVc, dcounts, dlens, workspace=ws)
            assert torch.equal(got_D, want_D)
        torch.cuda.synchronize()
    finally:
        for k, v in old.items():
            sc.tune_set(k, v)
    err = np.abs(O.float().cpu().numpy().astype(np.float64) - want_O) / np.maximum(1.0, np.abs(want_O))
    assert err.max() <= 4e-3, (knobs, err.max())
    assert np.abs(lse.cpu().numpy().astype(np.float64) - want_L).max() <= 1e-3


@pytest.mark.parametrize("Hkv,G,B,cap,tcap,nq,causal,o_f32,scale", [
    (2, 4, 1, 700, 0, 16, False, False, 0.0),       # 64 rows: half a workgroup of the block kernel idle
    (1, 1, 2, 1500, 0, 129, False, True, -0.05),    # one row beyond a block of 128; a negative scale; several splits
    (3, 7, 1, 63, 70, 37, True, False, 0.0),        # 259 rows, cache shorter than a tile, tiles that hold merged and tail rows
    (1, 8, 2, 900, 300, 60, True, True, 0.2),       # 480 rows; a sequence with fewer tail rows than query rows
    (8, 8, 10, 40, 0, 100, False, False, 0.0),      # as many blocks as fill the chip: one split, no second kernel
])
def test_multi_attn_blocks_against_oracle(Hkv, G, B, cap, tcap, nq, causal, o_f32, scale):
    rng = np.random.default_rng(77 + cap + nq)
    Hq, d = Hkv * G, 128
    Q = _round_like(rng.standard_normal((nq, B, Hq, d)), True)
    Kc, Vc = _round_like(rng.standard_normal((B, Hkv, cap, d)), True), _round_like(rng.standard_normal((B, Hkv, cap, d)), True)
    counts = rng.integers(1, 40, (B, Hkv, cap)).astype(np.int32)
    lens = rng.integers(cap // 2, cap + 1, (B, Hkv)).astype(np.int32)
    lens[0, 0] = cap
    if B > 1:
        lens[-1, -1] = 0
    dQ, dKc, dVc = g.to_device(Q, True), g.to_device(Kc, True), g.to_device(Vc, True)
    dcounts, dlens = torch.from_numpy(counts).to(g.DEV), torch.from_numpy(lens).to(g.DEV)
    O = torch.full((nq, B, Hq, d), 7.0, dtype=torch.float32 if o_f32 else torch.bfloat16, device=g.DEV)
    tail = {}
    if tcap:
        Kt, Vt = _round_like(rng.standard_normal((B, Hkv, tcap, d)), True), _round_like(rng.standard_normal((B, Hkv, tcap, d)), True)
        tails = np.full((B,), tcap - 3, np.int32)
        tails[-1] = nq // 2 if B > 1 else tcap
        tail = dict(Kt=g.to_device(Kt, True), Vt=g.to_device(Vt, True), tail_lens=torch.from_numpy(tails).to(g.DEV), causal=causal)
        want_O, want_L = oracle.multi_attn_tail(Q, Kc, Vc, counts, lens, Kt, Vt, tails, causal, scale or None)
    else:
        want_O, want_L = oracle.multi_attn(Q, Kc, Vc, counts, lens, scale or None)
    for knob in (0, 128):       # the kernel chosen from the shape, and the block kernel
        sc.tune_set("multi_block_rows", knob)
        try:
            O.fill_(7.0)
            _, lse = sc.sc_multi_attn(dQ, dKc, dVc, dcounts, dlens, scale=scale, O=O, want_lse=True, **tail)
            torch.cuda.synchronize()
        finally:
            sc.tune_set("multi_block_rows", 0)
        got = O.float().cpu().numpy().astype(np.float64)
        if o_f32:
            # probabilities enter with 16 bits (2^-18 each at most): 2.4e-6 of the outputs' rms on average, and the largest of a
            # hundred thousand outputs at a few times that where a handful of rows carry the sum
            assert np.abs(got - want_O).max() <= 4e-5 * np.sqrt(np.mean(want_O ** 2))
        else:       # half an ulp of the output
            err = np.abs(got - want_O) / np.maximum(1.0, np.abs(want_O))
            assert err.max() <= 4e-3, (knob, err.max(), np.unravel_index(err.argmax(), err.shape))
        got_l = lse.cpu().numpy().astype(np.float64)
        finite = np.isfinite(want_L)
        assert np.array_equal(np.isneginf(got_l), np.isneginf(want_L))
        assert np.abs(got_l[finite] - want_L[finite]).max() <= 1e-3


@pytest.mark.parametrize("o_f32", [True, False])
@pytest.mark.parametrize("kv_bf16,d,cap,nq", [
    (True, 128, 2000, 3),       # few rows, partials folded by the second kernel
    (True, 128, 100, 3),        # few rows, one split
    (True, 128, 2000, 40),      # blocks of 128 rows
    (True, 128, 100, 40),       # ... one split
    (False, 64, 700, 3),        # row by row through the decode kernels
])
def test_multi_attn_output_at_a_multiple_of_four_bytes(kv_bf16, d, cap, nq, o_f32):
    rng = np.random.default_rng(cap + nq)
    B, Hkv, G = 1, 2, 4
    Q = g.to_device(_round_like(rng.standard_normal((nq, B, Hkv * G, d)), kv_bf16), kv_bf16)
    Kc, Vc = (g.to_device(_round_like(rng.standard_normal((B, Hkv, cap, d)), kv_bf16), kv_bf16) for _ in range(2))
    counts = torch.from_numpy(rng.integers(1, 40, (B, Hkv, cap)).astype(np.int32)).to(g.DEV)
    lens = torch.full((B, Hkv), cap, dtype=torch.int32, device=g.DEV)
    dt = torch.float32 if o_f32 else torch.bfloat16
    step = 4 // dt.itemsize
    want = torch.zeros(Q.shape, dtype=dt, device=g.DEV)
    sc.sc_multi_attn(Q, Kc, Vc, counts, lens, O=want)
    for at in (1, 2, 3):        # 4, 8 and 12 bytes behind a 16-byte boundary
        buf = torch.full((want.numel() + 8 * step,), 7.0, dtype=dt, device=g.DEV)
        sc.sc_multi_attn(Q, Kc, Vc, counts, lens, O=buf[at * step:at * step + want.numel()].view(want.shape))
        torch.cuda.synchronize()
        assert torch.equal(buf[at * step:at * step + want.numel()].view(want.shape), want), at
        assert (buf[:at * step] == 7.0).all() and (buf[at * step + want.numel():] == 7.0).all(), at


# rms error of fp32 outputs over the rms of the outputs, in 1e-7, at the scales 1/sqrt(128), 0.3 and 1.  A weight enters the
# second product in two bf16 parts: rounded at 2^-18 at most, 2.3e-6 (rms) over many weights; less where a few rows
# carry the sum, as long as the largest weight is 1 and not rounded.  The bounds are 1.1 times what 16 x 16 x 32 products with
# 32 query rows per workgroup and the true maximum as reference gave (15.4 / 5.6 / 7.4 and 20.6 / 8.3 / 9.0); a reference
# that lags behind the maximum by up to 2^8 gives 19.3 / 6.5 / 8.4 and 24.6 / 19.4 / 12.9.
@pytest.mark.parametrize("nq,rows,tcap,causal,bounds", [
    (8, 5500, 0, False, (16.9, 6.2, 8.1)),        # 32 query rows per head
    (512, 5400, 512, True, (22.6, 9.2, 9.9)),      # sixteen blocks of 128
])
def test_multi_attn_error_of_fp32_outputs(nq, rows, tcap, causal, bounds):
    B, Hkv, G, d = 1, 8, 4, 128
    gen = torch.Generator().manual_seed(nq)
    bf16 = lambda *s: torch.randn(s, generator=gen).to(torch.bfloat16).to(g.DEV)
    Q, Kc, Vc = bf16(nq, B, Hkv * G, d), bf16(B, Hkv, rows, d), bf16(B, Hkv, rows, d)
    counts = (1 + torch.empty((B, Hkv, rows)).exponential_(1 / 6.0, generator=gen).int()).to(g.DEV)
    lens = torch.full((B, Hkv), rows, dtype=torch.int32, device=g.DEV)
    tail = dict(Kt=bf16(B, Hkv, tcap, d), Vt=bf16(B, Hkv, tcap, d), causal=causal,
                tail_lens=torch.full((B,), tcap, dtype=torch.int32, device=g.DEV)) if tcap else {}
    O = torch.empty((nq, B, Hkv * G, d), dtype=torch.float32, device=g.DEV)
    for scale, bound in zip((1 / np.sqrt(d), 0.3, 1.0), bounds):
        sc.sc_multi_attn(Q, Kc, Vc, counts, lens, scale=float(scale), O=O, **tail)
        err, total = 0.0, 0.0
        for h in (0, Hkv - 1):
            k, v, bias = Kc[0, h].double(), Vc[0, h].double(), counts[0, h].double().log()
            if tcap:
                k, v = torch.cat([k, tail["Kt"][0, h].double()]), torch.cat([v, tail["Vt"][0, h].double()])
                bias = torch.cat([bias, torch.zeros(tcap, dtype=torch.float64, device=g.DEV)])
            z = Q[:, 0, h * G:(h + 1) * G].double().reshape(nq * G, d) @ k.t().contiguous() * float(scale) + bias
            if causal:
                seen = rows + tcap - nq + 1 + torch.arange(nq, device=g.DEV).repeat_interleave(G)
                z.masked_fill_(torch.arange(rows + tcap, device=g.DEV)[None, :] >= seen[:, None], -np.inf)
            want = (torch.softmax(z, 1) @ v).reshape(nq, G, d)
            err += float((O[:, 0, h * G:(h + 1) * G].double() - want).square().sum())
            total += float(want.square().sum())
        rel = np.sqrt(err / total)
        print("nq %d scale %.3f: rms error %.3e" % (nq, scale, rel))
        assert rel <= bound * 1e-7, (scale, rel)
