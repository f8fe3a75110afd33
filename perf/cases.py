"""Performance cases of the compress-then-attend path: the calls a program that serves a model with a
compressed KV cache makes, over the range of shapes it makes them with.

Kinds
  prefill   sc_segment + sc_gsc_merge of one layer: a prompt (or a batch of prompts of different lengths) is
            compressed once.  Rows that are not written stay zero, so whole buffers can be compared.
  passes    the same on a small layer, followed by a few decode steps on the cache just made: the three calls in
            the order a short request makes them.
  decode    one decode step: sc_decode_attn for every layer of the model, each on its own merged cache, with the
            uncompressed tail of the tokens generated so far where the case has one.
  append    the tokens generated since the last delimiter leave the tail: sc_segment + the appending sc_gsc_merge,
            for every layer.
  multi     sc_multi_attn for every layer: several query rows at once over cache and tail (draft tokens to verify,
            or a chunk of a further prompt behind a compressed one).
  budget    sc_segment + sc_gsc_merge_budget: the threshold is searched for a target cache size.
  global    sc_gsc_merge_global: the whole sequence is one chunk.

Shapes are those of the workloads in paper_2603_14303_amd/workloads.py and of the tests; keys and values follow the
recipe of that module (a few centres per delimiter-bounded chunk plus noise), drawn on the GPU.
"""
import math

import numpy as np
import torch

from paper_2603_14303_amd import binding as sc

MAX_CENTERS = 6
NOISE_STD = 0.15
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
# merged rows per token at the thresholds used here (chunks of 24 tokens on average / of the power law), for sizes only:
# 0.7 lies on the plateau where every centre becomes one row, the others inside the band of the similarities
ROW_SHARE = {("geom", 0.7): 0.165, ("geom", 0.9745): 0.256, ("geom", 0.979): 0.497,
             ("zipf", 0.7): 0.117, ("zipf", 0.9745): 0.24, ("zipf", 0.979): 0.50}
EMPTY = {"B": 1, "Hkv": 8, "G": 4, "N": 32768, "d": 128, "dtype": "bf16", "out": "bf16", "tau": 0.7, "gaps": "geom",
         "ragged": False}


def listed():
    return [
        # a short request on a small fp32 model: every call is latency
        {"name": "passes_1k_f32", **EMPTY, "kind": "passes", "Hkv": 2, "G": 1, "N": 1024, "d": 64, "dtype": "f32", "out": "f32",
         "steps": 8},
        # a 32k-token prompt, one layer of a model with eight KV heads: the benchmark's own shape
        {"name": "prefill_32k", **EMPTY, "kind": "prefill"},
        # a 128k-token prompt with chunks of one to 256 tokens
        {"name": "prefill_128k", **EMPTY, "kind": "prefill", "N": 131072, "gaps": "zipf"},
        # 32 prompts of 8k to 16k tokens, at a threshold that lies inside the band of the similarities
        {"name": "prefill_batch32", **EMPTY, "kind": "prefill", "B": 32, "Hkv": 4, "G": 7, "N": 16384, "tau": 0.975, "ragged": True},
        # one generated token of one sequence through 32 layers, 100 tokens since the last delimiter
        {"name": "decode_32layers", **EMPTY, "kind": "decode", "layers": 32, "rows": 5385, "tail": 100, "lse": False},
        # one generated token of each of 32 sequences through 28 layers with seven query heads per KV head
        {"name": "decode_batch32", **EMPTY, "kind": "decode", "B": 32, "Hkv": 4, "G": 7, "layers": 28, "rows": 2035, "ragged": True,
         "tail": 0, "lse": False},
        # a stretch of 256 generated tokens joins the cache of eight layers
        {"name": "append_256", **EMPTY, "kind": "append", "N": 256, "layers": 8, "rows": 5385},
        # eight draft tokens are verified in 32 layers
        {"name": "verify_8", **EMPTY, "kind": "multi", "layers": 32, "rows": 5385, "tail": 108, "nq": 8, "causal": True},
        # a further 512 tokens of prompt behind a compressed one, eight layers
        {"name": "chunk_512", **EMPTY, "kind": "multi", "layers": 8, "rows": 5385, "tail": 512, "nq": 512, "causal": True},
        # a 32k-token prompt squeezed to 20 % of its entries
        {"name": "budget_32k", **EMPTY, "kind": "budget", "share": 0.2, "iterations": 12},
        # the same prompt as one chunk
        {"name": "global_32k", **EMPTY, "kind": "global"},
        # four 32k-token prompts of one layer that keep half of their entries
        {"name": "prefill_stack4", **EMPTY, "kind": "prefill", "B": 4, "tau": 0.979},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "passes", "decode", "decode", "append", "multi", "multi", "budget", "global"])
    c = dict(EMPTY, kind=kind)
    c["Hkv"] = rng.choice([1, 2, 4, 8])
    c["G"] = rng.choice([1, 2, 4, 7, 8])
    if kind in ("prefill", "budget"):
        # tokens times heads from a few thousand to the batch of 32 prompts (less where probes repeat the work)
        most = 1 << 18 if kind == "budget" else 1 << 20
        c["dtype"], c["d"] = rng.choice([("bf16", 128)] * 7 + [("bf16", 64), ("f32", 128), ("f32", 64)])
        if (c["dtype"], c["d"]) != ("bf16", 128):
            most >>= 2
        c["N"] = _log_int(rng, 700, min(131072, most // c["Hkv"]))
        c["B"] = _log_int(rng, 1, max(1, min(32, most // (c["Hkv"] * c["N"]))))
        c["ragged"] = c["B"] > 1
        c["gaps"] = rng.choice(["geom", "geom", "zipf"])
        c["out"] = rng.choice([c["dtype"], c["dtype"], c["dtype"], "f32"])
        c["tau"] = rng.choice([0.7, 0.7, 0.9745, 0.979])
        if kind == "budget":
            c["share"] = round(rng.uniform(0.2, 0.5), 3)
            c["iterations"] = rng.choice([8, 12])
    elif kind == "passes":
        c["dtype"], c["d"] = rng.choice([("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
        c["out"] = c["dtype"]
        c["Hkv"] = rng.choice([1, 2, 4])
        c["N"] = _log_int(rng, 300, 4000)
        c["steps"] = rng.randint(4, 12)
    elif kind == "decode":
        c["B"] = _log_int(rng, 1, 32)
        c["ragged"] = c["B"] > 1
        c["rows"] = _log_int(rng, 150, min(34000, (1 << 18) // (c["B"] * c["Hkv"])))
        c["tail"] = rng.choice([0, rng.randint(1, 256)])
        c["lse"] = rng.random() < 0.3
        c["layers"] = rng.randint(4, 16)
    elif kind == "append":
        c["B"] = _log_int(rng, 1, 16)
        c["ragged"] = c["B"] > 1
        c["N"] = _log_int(rng, 24, 1500)
        c["rows"] = _log_int(rng, 200, 8000)
        c["layers"] = rng.randint(2, 8)
    elif kind == "multi":
        c["B"] = _log_int(rng, 1, 8)
        c["ragged"] = c["B"] > 1
        c["nq"] = _log_int(rng, 2, max(2, 1024 // c["B"]))
        c["rows"] = _log_int(rng, 150, (1 << 16) // (c["B"] * c["Hkv"]))
        c["causal"] = rng.random() < 0.6
        c["tail"] = c["nq"] + rng.randint(0, 200) if c["causal"] else 0
        c["layers"] = rng.randint(2, 8)
    else:
        c["Hkv"] = rng.choice([1, 2, 4, 8])
        c["N"] = _log_int(rng, 1000, 32768)
        c["tau"] = rng.choice([0.7, 0.7, 0.9745])
    return c


# ------------------------------------------------------------------------------------------------ inputs
def _host_rng(seed, *tag):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([seed & 0xFFFFFFFFFFFF, *tag])))


def _gap_mean(c):
    if c["gaps"] == "geom":
        return 24.0 * (1.0 - (23.0 / 24.0) ** 128)
    g = np.arange(1, 257, dtype=np.float64)
    p = g ** -1.2
    return float((g * p).sum() / p.sum())


def _lengths(c, rng):
    n = np.full((c["B"],), c["N"], dtype=np.int32)
    return rng.integers(c["N"] // 2, c["N"] + 1, size=c["B"]).astype(np.int32) if c["ragged"] else n


def _masks(c, rng, lens, close=False):
    """u8 [B, N]: nonzero = delimiter; with `close` the last token of every sequence is one."""
    mask = np.zeros((c["B"], c["N"]), dtype=np.uint8)
    for b, n in enumerate(lens):
        pos = -1
        while pos < n:
            if c["gaps"] == "geom":
                g = np.minimum(rng.geometric(1.0 / 24.0, size=max(64, n // 8)), 128)
            else:
                p = np.arange(1, 257, dtype=np.float64) ** -1.2
                g = rng.choice(np.arange(1, 257), size=max(64, n // 8), p=p / p.sum())
            at = pos + np.cumsum(g)
            mask[b, at[at < n]] = 1
            pos = int(at[-1])
        if close:
            mask[b, n - 1] = 1
    return mask


def _mixture(c, gen, mask_b):
    """[Hkv, N, d]: per chunk up to six centres, every token one of them plus noise; delimiters rows of their own."""
    H, N, d = c["Hkv"], c["N"], c["d"]
    is_delim = mask_b != 0
    chunk = torch.cumsum(is_delim, 0) - is_delim.to(torch.int64)
    n_chunks = N + 1 if N < 4096 else int(is_delim.sum()) + 1
    many = torch.randint(1, MAX_CENTERS + 1, (H, n_chunks), generator=gen, device="cuda")
    centers = torch.randn((H, n_chunks * MAX_CENTERS, d), generator=gen, device="cuda")
    pick = (torch.rand((H, N), generator=gen, device="cuda") * many[:, chunk]).to(torch.int64).clamp_(max=MAX_CENTERS - 1)
    rows = torch.randn((H, N, d), generator=gen, device="cuda")
    spread = torch.where(is_delim, 1.0, NOISE_STD)[None, :, None]
    at = (chunk[None, :] * MAX_CENTERS + pick)[:, :, None].expand(-1, -1, d)
    rows.mul_(spread).add_(torch.gather(centers, 1, at).mul_((~is_delim)[None, :, None]))
    return rows.to(DTYPES[c["dtype"]])


def _keys_values(c, gen, mask):
    K = torch.empty((c["B"], c["Hkv"], c["N"], c["d"]), dtype=DTYPES[c["dtype"]], device="cuda")
    V = torch.empty_like(K)
    for b in range(c["B"]):
        K[b], V[b] = _mixture(c, gen, mask[b]), _mixture(c, gen, mask[b])
    return K, V


def _capacity(c):
    """Rows a program sets aside for the merged cache: a good margin over what the threshold keeps."""
    if c["N"] < 4096 or c["kind"] == "global":
        return c["N"]
    if c["kind"] == "budget":
        return min(c["N"], int(1.5 * c["share"] * c["N"]))
    return min(c["N"], int(1.5 * _share(c) * c["N"]))


def _share(c):
    tau = min((t for g, t in ROW_SHARE if g == c["gaps"]), key=lambda t: abs(t - c["tau"]))
    return ROW_SHARE[c["gaps"], tau]


def _cache(c, gen, rng, cap):
    """A merged cache as the compression leaves it: mean keys and values, a third of the rows clusters of one."""
    B, H, d = c["B"], c["Hkv"], c["d"]
    dt = DTYPES[c["dtype"]]
    rows = rng.integers(int(0.97 * c["rows"]), int(1.03 * c["rows"]) + 1, size=(B, H))
    if c["ragged"]:
        rows = np.maximum(1, (rows * rng.uniform(0.67, 1.33, size=(B, 1))).astype(np.int64))
    lens = torch.from_numpy(np.minimum(rows, c["rows"] * 3 // 2 + 16).astype(np.int32)).cuda()
    Kc = torch.empty((B, H, cap, d), dtype=dt, device="cuda").normal_(generator=gen)
    Vc = torch.empty((B, H, cap, d), dtype=dt, device="cuda").normal_(generator=gen)
    size = torch.rand((B, H, cap), generator=gen, device="cuda")
    counts = torch.where(size < 0.36, 1, 2 + (-8.0 * torch.log1p(-(size - 0.36) / 0.6401)).to(torch.int32)).to(torch.int32)
    return {"Kc": Kc, "Vc": Vc, "counts": counts, "lens": lens}


def _outputs(c, cap, dt):
    B, H, d = c["B"], c["Hkv"], c["d"]
    return {"Kc": torch.zeros((B, H, cap, d), dtype=dt, device="cuda"), "Vc": torch.zeros((B, H, cap, d), dtype=dt, device="cuda"),
            "counts": torch.zeros((B, H, cap), dtype=torch.int32, device="cuda"),
            "lens": torch.zeros((B, H), dtype=torch.int32, device="cuda")}


def prepare(case, seed):
    c = dict(case)
    rng = _host_rng(seed, 1)
    gen = torch.Generator("cuda").manual_seed(seed)
    B, H, N, d, Hq = c["B"], c["Hkv"], c["N"], c["d"], c["Hkv"] * c["G"]
    dt, kind = DTYPES[c["dtype"]], c["kind"]
    s = {"c": c}
    if kind in ("prefill", "passes", "budget", "global", "append"):
        lens = _lengths(c, rng)
        mask = torch.from_numpy(_masks(c, rng, lens, close=kind == "append")).cuda()
        s.update(mask=mask, seq_lens=torch.from_numpy(lens).cuda(), cap=_capacity(c))
        s["offsets"] = torch.zeros((B, N + 2), dtype=torch.int32, device="cuda")
        s["num_chunks"] = torch.zeros((B,), dtype=torch.int32, device="cuda")
    if kind in ("prefill", "passes", "budget", "global"):
        s["K"], s["V"] = _keys_values(c, gen, mask)
        s["out"] = _outputs(c, s["cap"], DTYPES[c["out"]])
    lib = sc.load_library()
    if kind in ("prefill", "passes"):
        s["ws"] = sc.gsc_merge_workspace(B, H, N, d, "cuda", DTYPES[c["out"]])
    if kind == "passes":
        s["Q"] = torch.empty((c["steps"], B, Hq, d), dtype=dt, device="cuda").normal_(generator=gen)
        s["O"] = torch.zeros_like(s["Q"])
        s["ws_d"] = sc.decode_attn_workspace(B, Hq, H, s["cap"], d, "cuda")
    if kind == "budget":
        s["ws"] = sc.Workspace(lib.sc_gsc_merge_budget_workspace_bytes(B, H, N, d), "cuda")
        s["rows_wanted"] = int(c["share"] * H * int(lens.sum()))
        s["tau"], s["rows"] = torch.zeros((1,), device="cuda"), torch.zeros((1,), dtype=torch.int64, device="cuda")
    if kind == "global":
        s["ws"] = sc.Workspace(lib.sc_gsc_merge_global_workspace_bytes(B, H, N, d), "cuda")
    if kind in ("decode", "multi"):
        cap = c["rows"] * 3 // 2 + 16
        s["layers"] = [_cache(c, gen, rng, cap) for _ in range(c["layers"])]
        many = (c["nq"],) if kind == "multi" else ()
        s["Q"] = torch.empty((c["layers"], *many, B, Hq, d), dtype=dt, device="cuda").normal_(generator=gen)
        s["O"] = torch.zeros_like(s["Q"])
        s["lse"] = torch.zeros(s["Q"].shape[:-1], dtype=torch.float32, device="cuda") if c.get("lse") else None
        if c["tail"]:
            for x in s["layers"]:
                x["Kt"] = torch.empty((B, H, c["tail"], d), dtype=dt, device="cuda").normal_(generator=gen)
                x["Vt"] = torch.empty((B, H, c["tail"], d), dtype=dt, device="cuda").normal_(generator=gen)
            s["tail_lens"] = torch.full((B,), c["tail"], dtype=torch.int32, device="cuda")
        if kind == "decode":
            s["ws"] = sc.decode_attn_workspace(B, Hq, H, cap, d, "cuda")
        else:
            s["ws"] = sc.Workspace(lib.sc_multi_attn_workspace_bytes(B, Hq, H, c["nq"], cap + c["tail"], d), "cuda")
    if kind == "append":
        cap = c["rows"] * 3 // 2 + 16 + N
        s["layers"] = []
        for _ in range(c["layers"]):
            x = _cache(c, gen, rng, cap)
            x["Kt"], x["Vt"] = _keys_values(c, gen, mask)
            x["new_lens"] = torch.zeros_like(x["lens"])
            s["layers"].append(x)
        s["cap"] = cap
        s["ws"] = sc.gsc_merge_workspace(B, H, N, d, "cuda", dt)
    return s


def run(s):
    c = s["c"]
    kind, o = c["kind"], s.get("out")
    if kind in ("prefill", "passes"):
        sc.sc_segment(s["mask"], s["seq_lens"], offsets=s["offsets"], num_chunks=s["num_chunks"])
        sc.sc_gsc_merge(s["K"], s["V"], s["offsets"], s["num_chunks"], c["tau"], seq_lens=s["seq_lens"], cap=s["cap"],
                        Kc=o["Kc"], Vc=o["Vc"], counts=o["counts"], comp_lens=o["lens"], workspace=s["ws"])
        if kind == "prefill":
            return [s["num_chunks"], s["offsets"], o]
        for i in range(c["steps"]):
            sc.sc_decode_attn(s["Q"][i], o["Kc"], o["Vc"], o["counts"], o["lens"], O=s["O"][i], workspace=s["ws_d"])
        return [s["num_chunks"], s["offsets"], o, s["O"]]
    if kind == "decode":
        for i, x in enumerate(s["layers"]):
            tail = dict(Kt=x["Kt"], Vt=x["Vt"], tail_lens=s["tail_lens"]) if c["tail"] else {}
            sc.sc_decode_attn(s["Q"][i], x["Kc"], x["Vc"], x["counts"], x["lens"], O=s["O"][i],
                              lse=s["lse"][i] if c["lse"] else None, workspace=s["ws"], **tail)
        return [s["O"], s["lse"]]
    if kind == "multi":
        for i, x in enumerate(s["layers"]):
            tail = dict(Kt=x["Kt"], Vt=x["Vt"], tail_lens=s["tail_lens"], causal=c["causal"]) if c["tail"] else {}
            sc.sc_multi_attn(s["Q"][i], x["Kc"], x["Vc"], x["counts"], x["lens"], O=s["O"][i], workspace=s["ws"], **tail)
        return s["O"]
    if kind == "append":
        sc.sc_segment(s["mask"], s["seq_lens"], offsets=s["offsets"], num_chunks=s["num_chunks"])
        for x in s["layers"]:
            sc.sc_gsc_merge(x["Kt"], x["Vt"], s["offsets"], s["num_chunks"], c["tau"], seq_lens=s["seq_lens"], cap=s["cap"],
                            Kc=x["Kc"], Vc=x["Vc"], counts=x["counts"], comp_lens=x["new_lens"], base_lens=x["lens"],
                            workspace=s["ws"])
        return [s["num_chunks"], [[x["Kc"], x["Vc"], x["counts"], x["new_lens"]] for x in s["layers"]]]
    # the two calls below through the C boundary: their outputs go to buffers that the program keeps
    lib, K, V = sc.load_library(), s["K"], s["V"]
    B, H, N, d = K.shape
    code = {torch.float32: sc.SC_F32, torch.bfloat16: sc.SC_BF16}
    at = dict(stream=torch.cuda.current_stream().cuda_stream)
    head = (K.data_ptr(), V.data_ptr(), code[K.dtype], K.stride(0), K.stride(1), K.stride(2), s["seq_lens"].data_ptr())
    outs = (o["Kc"].data_ptr(), o["Vc"].data_ptr(), code[o["Kc"].dtype], s["cap"], o["counts"].data_ptr(), o["lens"].data_ptr(), None)
    if kind == "budget":
        sc.sc_segment(s["mask"], s["seq_lens"], offsets=s["offsets"], num_chunks=s["num_chunks"])
        status = lib.sc_gsc_merge_budget(*head, s["offsets"].data_ptr(), s["offsets"].stride(0), s["num_chunks"].data_ptr(),
                                         B, H, N, d, s["rows_wanted"], -1.01, 1.0, c["iterations"], *outs,
                                         s["tau"].data_ptr(), s["rows"].data_ptr(), s["ws"].ptr, s["ws"].nbytes, at["stream"])
    else:
        status = lib.sc_gsc_merge_global(*head, B, H, N, d, c["tau"], *outs, s["ws"].ptr, s["ws"].nbytes, at["stream"])
    if status != sc.SC_OK:
        raise RuntimeError(lib.sc_status_string(status).decode())
    return [o, s["tau"], s["rows"]] if kind == "budget" else o


# ------------------------------------------------------------------------------------------------ what a pass cannot do without
def work(case):
    c = case
    B, H, N, d, G = c["B"], c["Hkv"], c["N"], c["d"], c["G"]
    e, eo = (2 if c["dtype"] == "bf16" else 4), (2 if c["out"] == "bf16" else 4)
    n = B * N * (0.75 if c["ragged"] else 1.0)          # tokens
    chunks = n / _gap_mean(c)
    share = c["share"] if c["kind"] == "budget" else _share(c)
    merge_bytes = 2 * n * H * d * e + share * n * H * (2 * d * eo + 4) + n + 4 * (chunks + B)
    # Alg. 1 compares a token with the seeds of its chunk up to the one it joins: about two on average; then the means
    merge_flops = n * H * (2 * 2 * d + 2 * d)
    if c["kind"] == "prefill":
        return {"bytes": merge_bytes, "flops": merge_flops}
    if c["kind"] == "budget":
        return {"bytes": merge_bytes, "flops": merge_flops * (c["iterations"] + 1)}
    if c["kind"] == "global":
        # every token against the seeds before it
        return {"bytes": 2 * n * H * d * e + share * n * H * (2 * d * eo + 4), "flops": H * B * N * share * N / 2 * 2 * d}
    if c["kind"] == "append":
        return {"bytes": n + c["layers"] * (merge_bytes - n), "flops": c["layers"] * merge_flops}
    if c["kind"] == "passes":
        rows = share * n * H
        step = rows * (2 * d * e + 4) + 2 * B * H * G * d * e
        return {"bytes": merge_bytes + c["steps"] * step, "flops": merge_flops + c["steps"] * 4 * d * rows * G}
    nq = c.get("nq", 1)
    rows = B * H * c["rows"]
    seen = rows + B * H * (c["tail"] - (nq / 2 if c.get("causal") and c["tail"] else 0))
    return {"bytes": c["layers"] * (rows * (2 * d * e + 4) + B * H * c["tail"] * 2 * d * e + 2 * nq * B * H * G * d * e),
            "flops": c["layers"] * 4 * d * seen * G * nq}


def tolerance(case):
    """Whole numbers (offsets, cluster sizes, lengths) are exact: every decision equals its evaluation in fp64.  Floating
    outputs: about four times what the path differs from the same sums in fp64 by (bf16: half an ulp of the result)."""
    if case["dtype"] == "bf16" and (case["out"] == "bf16" or case["kind"] in ("decode", "multi", "append", "passes")):
        return {"rel": 7e-3, "max": 0.02, "differ": 0.0}
    return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
