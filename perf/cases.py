"""The work a serving program has this library do, as cases that can be timed and compared.

Each case is one call of a public entry point (`paper_2505_02922_amd.binding`) on one
transformer layer:

  decode   one decode step of tripartite attention over an index built beforehand
  budget   the same with a budget for the estimation zone
  full     brute-force attention over the whole context (what the index is compared with)
  build    the index construction at prefill
  append   the index update during decoding, written into room kept in the index's arrays

Inputs come from `paper_2505_02922_amd.synth` (Gaussian-mixture keys, rotary encoding, queries aimed
at mixture components), with the case's seed as the recipe's base seed.  Buffers that a serving
program keeps from step to step (outputs, workspaces, the index's arrays) are made by `prepare`.
"""
import math

import torch

from paper_2505_02922_amd import binding as wb
from paper_2505_02922_amd import synth

# One transformer layer of the workloads the benchmark names; a case replaces what differs.
_LLAMA = dict(dtype="bf16", B=1, Hq=32, Hkv=8, d=128, N=32768, n_sink=4, n_local=1024, L=8192, k=512,
              iters=10, r_frac=0.018, components=2048, sigma=0.25, rope=500000.0, heavy=0, outliers=0.0)
_QWEN = dict(_LLAMA, B=64, Hq=28, Hkv=4, N=65536, iters=20, r_frac=0.02, rope=1000000.0, heavy=4)
_TINY = dict(_LLAMA, dtype="f32", Hq=1, Hkv=1, d=64, N=4096, n_local=64, L=2048, k=128, r_frac=16 / 256,
             components=128, sigma=0.3, rope=0.0, outliers=0.02)


def listed():
    return [
        # One short sequence with one head in fp32: the smallest step, nothing but launches and latency.
        dict(_TINY, name="decode_f32_4k_b1", op="decode"),
        # A single chat at 32K tokens: the interactive step, one layer of an 8-KV-head model.
        dict(_LLAMA, name="decode_bf16_32k_b1", op="decode"),
        # The headline workload: 16 sequences of 120K tokens.
        dict(_LLAMA, name="decode_bf16_120k_b16", op="decode", B=16, N=122880),
        # One sequence of a million tokens: few heads, very many clusters.
        dict(_LLAMA, name="decode_bf16_1m_b1", op="decode", N=1048576, r_frac=0.01, components=65536),
        # A large batch on a seven-queries-per-KV-head model whose keys have a few heavy-tailed
        # channels (very uneven clusters).
        dict(_QWEN, name="decode_bf16_64k_b64", op="decode"),
        # The evaluation's zone budgets (1.8 % retrieved, 23.2 % estimated) on a few sequences of
        # ragged length: neither the context nor its last segment is a round number.
        dict(_LLAMA, name="budget_bf16_50k_b6", op="budget", B=6, N=50021, e_frac=0.232),
        # Exact attention on a batch of ragged contexts: the quality check beside the index.
        dict(_LLAMA, name="full_bf16_65k_b8", op="full", B=8, N=65521),
        # Prefill of the smallest sequence, fp32.
        dict(_TINY, name="build_f32_4k_b1", op="build"),
        # Prefill of a single 32K chat: the time to first token.
        dict(_LLAMA, name="build_bf16_32k_b1", op="build"),
        # Prefill of the headline batch.
        dict(_LLAMA, name="build_bf16_120k_b16", op="build", B=16, N=122880),
        # Prefill of the large batch with heavy-tailed channels, twenty rounds.
        dict(_QWEN, name="build_bf16_64k_b64", op="build"),
        # After every 1024 generated tokens the headline batch's indexes take an update segment in.
        dict(_LLAMA, name="append_bf16_120k_b16", op="append", B=16, N=122880, n_new=1024, U=1024, ku=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: any operation, 4K .. 1M tokens, 1 .. 64 sequences, up to
    8 query heads per KV head, segments of 1K .. 8K tokens, fp32 and bf16."""
    op = rng.choice(["decode", "decode", "decode", "build", "build", "budget", "full", "append"])
    f32 = rng.random() < 0.2
    d = rng.choice([64, 128]) if f32 else rng.choice([64, 128, 128, 128])
    Hkv = rng.choice([1, 2, 4, 8])
    # tokens over all units of a case: what the largest listed case of its kind holds; fp32 prefill
    # (no matrix instructions) is kept to what costs about as much
    most = 16.7e6
    if f32:
        most = 0.5e6 if op in ("build", "append") else 4e6
    N = _log(rng, 4096, 1048576 if not f32 else 131072)
    N = max(4096, min(N, int(most / Hkv)))
    B = _log(rng, 1, max(1, min(64, int(most / (Hkv * N)))))
    L = rng.choice([1024, 2048, 4096, 8192])
    heavy = 4 if rng.random() < 0.25 else 0
    c = dict(dtype="f32" if f32 else "bf16", B=B, Hq=Hkv * rng.choice([1, 2, 4, 4, 7, 8]), Hkv=Hkv, d=d, N=N,
             n_sink=rng.choice([0, 4, 16]), n_local=rng.choice([64, 256, 1000, 1024]), L=L, k=L // 16,
             iters=rng.choice([5, 10, 10, 20]), r_frac=rng.uniform(0.01, 0.05), components=2048,
             sigma=rng.choice([0.25, 0.3]), rope=rng.choice([0.0, 500000.0, 1000000.0]), heavy=heavy,
             outliers=rng.choice([0.0, 0.02]), op=op)
    if op == "budget":
        c["e_frac"] = rng.uniform(0.05, 0.4)
    if op == "append":
        c["U"] = rng.choice([512, 1024, 2048])
        c["ku"] = c["U"] // 16
        c["n_new"] = rng.choice([1, _log(rng, 1, 4096), c["U"]])
    return c


def _workload(case, seed):
    return synth.Workload(
        name="case", dtype=case["dtype"], B=case["B"], Hq=case["Hq"], Hkv=case["Hkv"], d=case["d"], N=case["N"],
        n_sink=case["n_sink"], n_local=case["n_local"], segment_len=case["L"], clusters_per_segment=case["k"],
        iters=case["iters"], retrieve_frac=case["r_frac"], retrieve_abs=None, n_components=case["components"],
        sigma=case["sigma"], rope_base=case["rope"] or None, outlier_token_frac=case["outliers"],
        outlier_token_scale=4.0, heavy_channels=case["heavy"], base_seed=int(seed) % 1000003)


def _build_args(wl):
    return (wl.n_sink, wl.n_local, wl.segment_len, wl.clusters_per_segment, wl.iters, 0)


def _empty_index(wl, rows=0, clusters=0, steady=0):
    return wb.alloc_index(wl.torch_dtype(), wl.B, wl.Hkv, wl.d, wl.N, wl.n_sink, wl.n_local, wl.segment_len,
                          wl.clusters_per_segment, "cuda", row_capacity=rows, cluster_capacity=clusters,
                          steady_capacity=steady)


def prepare(case, seed):
    wl = _workload(case, seed)
    st = {"op": case["op"], "wl": wl}
    K, V = synth.make_kv(wl, device="cuda")
    if case["op"] == "build":
        st["K"], st["V"] = K, V
        st["ix"] = _empty_index(wl)
        st["ws"] = wb.workspace(st["ix"].build_ws_bytes)
        return st
    if case["op"] == "append":
        # an index with room for this update, and the generated tokens' keys and values (made by
        # the same recipe, from the end of a context of its own)
        U, ku, n_new = case["U"], case["ku"], case["n_new"]
        plain = wb.wave_index_plan(wl.torch_dtype(), wl.B, wl.Hkv, wl.d, wl.N, wl.n_sink, wl.n_local,
                                   wl.segment_len, wl.clusters_per_segment)[0]
        segs = n_new // U
        ix = _empty_index(wl, rows=plain.N_idx + segs * U, clusters=plain.m + segs * ku, steady=plain.p + n_new)
        for t in ix.t.values():
            t.zero_()
        wb.wave_index_build(K, V, *_build_args(wl), index=ix)
        torch.cuda.synchronize()
        ix._keepalive = None
        del K, V
        nk, nv = synth.make_kv(synth.scaled(wl, N=n_new, base_seed=wl.base_seed + 1), device="cuda")
        st.update(ix=ix, K_new=nk, V_new=nv, U=U, ku=ku)
        return st
    q = synth.make_queries(wl, 0, device="cuda")
    st["q"] = q
    st["out"] = torch.empty(wl.B, wl.Hq, wl.d, dtype=torch.float32, device="cuda")
    st["lse"] = torch.empty(wl.B, wl.Hq, dtype=torch.float32, device="cuda")
    if case["op"] == "full":
        st["K"], st["V"] = K, V
        st["ws"] = wb.workspace(wb.wave_full_attention_workspace(wl.B, wl.Hq, wl.N, wl.d))
        return st
    ix = wb.wave_index_build(K, V, *_build_args(wl))
    torch.cuda.synchronize()
    ix._keepalive = None
    r = max(1, wl.retrieve_count(ix.m))
    st.update(ix=ix, r=r)
    st["sel"] = torch.empty(wl.B, wl.Hq, r, dtype=torch.int32, device="cuda")
    if case["op"] == "budget":
        st["e"] = int(case["e_frac"] * ix.m + 0.5)
        st["ws"] = wb.workspace(wb.wave_attention_decode_budget_workspace(ix, wl.Hq, r, st["e"]))
    else:
        st["ws"] = wb.workspace(wb.decode_workspace_bytes(ix, wl.Hq, r))
    return st


def run(st):
    op, wl = st["op"], st["wl"]
    if op == "decode":
        return wb.wave_attention_decode(st["q"], st["ix"], st["r"], out=st["out"], lse=st["lse"],
                                        selected=st["sel"], ws=st["ws"])
    if op == "budget":
        return wb.wave_attention_decode_budget(st["q"], st["ix"], st["r"], st["e"], out=st["out"], lse=st["lse"],
                                               selected=st["sel"], ws=st["ws"])
    if op == "full":
        return wb.wave_full_attention_decode(st["q"], st["K"], st["V"], out=st["out"], lse=st["lse"], ws=st["ws"])
    if op == "build":
        ix = wb.wave_index_build(st["K"], st["V"], *_build_args(wl), ws=st["ws"], index=st["ix"])
    else:
        ix = wb.wave_index_append(st["ix"], st["K_new"], st["V_new"], wl.n_local, st["U"], st["ku"], wl.iters, 0)
    return {name: ix.t[name] for name in wb.BUFFER_NAMES}


def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    units, d, N = case["B"] * case["Hkv"], case["d"], case["N"]
    heads, row = case["B"] * case["Hq"], d * es
    steady = min(N, case["n_sink"] + case["n_local"])
    n_idx = N - steady
    full, tail = divmod(n_idx, case["L"])
    m = full * case["k"] + min(case["k"], tail)
    io = heads * d * (es + 4) + heads * 4
    if case["op"] == "full":
        return {"bytes": 2 * units * N * row + io, "flops": 4.0 * heads * N * d}
    if case["op"] == "build":
        # keys and values in and out, the meta index out; every point is compared with every
        # centroid of its segment at least once (how much of that the later rounds repeat depends
        # on the data)
        sims = units * (full * case["L"] * case["k"] + tail * min(case["k"], tail))
        return {"bytes": 4 * units * N * row + 2 * units * m * row + 4 * units * (n_idx + 2 * m),
                "flops": 2.0 * sims * d}
    if case["op"] == "append":
        # the window that moves (read and written once), the new tokens, the new clusters
        n_new, flush = case["n_new"], case["n_new"] // case["U"] * case["U"]
        moved = (case["n_local"] if flush else 0) + n_new
        return {"bytes": units * (4 * moved * row + flush // case["U"] * case["ku"] * (2 * row + 8) + 4 * flush),
                "flops": 2.0 * units * flush * min(case["ku"], case["U"]) * d}
    # decode: centroids (and value sums) once per KV head, the steady rows once per KV head, and per
    # query head the rows of its retrieved clusters at the mean cluster size
    r = max(1, int(math.floor(case["r_frac"] * m + 0.5)))
    tokens = min(n_idx, r * n_idx // max(m, 1))
    est = m if case["op"] == "decode" else min(m, int(case["e_frac"] * m + 0.5) * case["Hq"] // case["Hkv"])
    return {"bytes": units * (m + est) * row + 4 * units * m + 2 * units * steady * row + 2 * heads * tokens * row
            + io + 4 * heads * r,
            "flops": heads * d * (2.0 * m + 2.0 * min(est, m) + 4.0 * (tokens + steady))}


def tolerance(case):
    if case["op"] in ("build", "append"):
        # the partition is the 64-bit argmax and the sums are 64-bit, rounded once to the storage
        # type: another order of a sum can flip a rounding, one in about 2^30
        return {"rel": 1e-5, "max": 2e-2, "differ": 0.0}
    # fp32 accumulation and fp32 exponentials: against a 64-bit evaluation of the same zones the
    # decode cases are off by rel 1e-7 .. 8e-7, at most 3e-6 per value in a dozen sampled heads; the
    # selected ids are the 64-bit ranking's
    return {"rel": 4e-6, "max": 5e-5, "differ": 1e-5}
