"""GPU parity of the k-means rounds at the sizes where their launch shapes and tiles change: the
index arrays of whole builds against the oracle's, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import wave_oracle as wo
from paper_2505_02922_amd import binding as wb
from paper_2505_02922_amd import synth
from tests import parity_util as pu

pytestmark = pytest.mark.gpu


def _keys(kind, B, N, d, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(B, 1, N, d, generator=g)
    if kind == "mixture":    # well separated: few points change cluster after the first rounds
        centre = torch.randn(64, d, generator=g)
        x = centre[torch.randint(0, 64, (B, 1, N), generator=g)] + 0.3 * x
    elif kind == "ties":     # few distinct keys: equal similarities and clusters that stay empty
        few = torch.randn(23, d, generator=g)
        x = few[torch.randint(0, 23, (B, 1, N), generator=g)]
    elif kind == "wide":     # a zero-mean channel with values so far apart that their fp64 sums round
        i = torch.arange(N) - 2                      # (two sink tokens; +1, -1, tiny, tiny, ...)
        tiny = torch.randn(N, generator=g) * 2.0 ** -42
        x[..., 0] = torch.where(i % 4 < 2, 1.0 - 2.0 * (i % 2), tiny)
    return x                 # "plain": no clusters, most points near a boundary


# (N - 5 tokens are indexed.  4097 points: the last of two or three workgroups' shares has one
# fragment with one point; k = 33: a tile with one row; k = 1000 at d = 64: 32 tiles, as many as
# stay resident; plain keys: hundreds of points per workgroup need the full comparison, and of 20000
# points in 33 clusters more move in a round than the update lists at once)
@pytest.mark.parametrize("kind,d,N,L,k,iters", [
    ("mixture", 128, 4102, 4097, 33, 7), ("plain", 128, 9000, 8192, 512, 8), ("mixture", 64, 4205, 4200, 1000, 5),
    ("ties", 128, 3000, 2100, 65, 5), ("plain", 64, 8197, 8192, 40, 6), ("plain", 128, 2205, 2200, 1, 4),
    ("plain", 128, 20005, 20000, 33, 4), ("wide", 128, 4605, 2300, 200, 5), ("wide", 64, 4405, 4400, 1000, 4)])
def test_rounds_match_oracle(kind, d, N, L, k, iters):
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="rounds", B=2, Hq=1, Hkv=1, N=N, d=d, n_sink=2, n_local=3,
                      segment_len=L, clusters_per_segment=k, iters=iters)
    K = _keys(kind, 2, N, d, N + k).to(torch.bfloat16)
    V = torch.randn(2, 1, N, d, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), wl.n_sink, wl.n_local, L, k, iters, 0, row_capacity=N + 9)
    torch.cuda.synchronize()
    for name in wb.BUFFER_NAMES:
        got = ix.t[name].cpu()
        got = got[:, :, :N - 5] if name in ("perm", "k_perm", "v_perm") else got
        assert torch.equal(got.double(), ref[name].reshape(got.shape).double()), name


# A cluster that loses its last members in a round keeps the centroid it had, also when so many points
# move that the update takes them in ranges of 2048 and the members leave in different ones.
@pytest.mark.parametrize("d,scale,seed", [(64, 400.0, 3), (128, 2000.0, 2)])
def test_cluster_emptied_across_ranges_keeps_its_centroid(d, scale, seed):
    L, k, iters = 8192, 100, 6
    x = torch.randn(L, d, generator=torch.Generator().manual_seed(seed))
    x[:, 5] *= scale
    x = x.to(torch.bfloat16)
    trace = []
    wo.kmeans_segment(x.double().numpy(), wo.init_indices(0, 0, 0, 0, L, k), iters, "bf16", trace)
    split = 0
    for (_, _, before), (_, _, after) in zip(trace[:-2], trace[1:-1]):   # (the last round has no update)
        if (before != after).sum() > 2048:
            for c in np.setdiff1d(before, after):
                split += len(set(np.nonzero(before == c)[0] // 2048)) > 1
    assert split > 0
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="emptied", B=1, Hq=1, Hkv=1, N=L, d=d, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=iters)
    K, V = x.view(1, 1, L, d), torch.randn(1, 1, L, d, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 0, 0, L, k, iters, 0)
    torch.cuda.synchronize()
    for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
        got = ix.t[name].cpu()
        assert torch.equal(got.double(), ref[name].reshape(got.shape).double()), name


# The points that moved in a round: as many as the update lists at once, and one more.
@pytest.mark.parametrize("d,L,k,seed,moved", [(64, 10750, 130, 192, 2048), (64, 10750, 130, 88, 2049),
                                              (128, 10650, 70, 67, 2048), (128, 10650, 70, 63, 2049)])
def test_most_points_that_an_update_lists(d, L, k, seed, moved):
    iters = 4
    x = torch.randn(L, d, generator=torch.Generator().manual_seed(seed)).to(torch.bfloat16)
    trace = []
    wo.kmeans_segment(x.double().numpy(), wo.init_indices(0, 0, 0, 0, L, k), iters, "bf16", trace)
    assert (trace[0][2] != trace[1][2]).sum() == moved
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="moved", B=1, Hq=1, Hkv=1, N=L, d=d, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=iters)
    K, V = x.view(1, 1, L, d), torch.randn(1, 1, L, d, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 0, 0, L, k, iters, 0)
    torch.cuda.synchronize()
    for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
        got = ix.t[name].cpu()
        assert torch.equal(got.double(), ref[name].reshape(got.shape).double()), name


# (33 points: a fragment with one; k = 33, 129, 289: a tile with one centroid; equal centroids: the lowest wins)
@pytest.mark.parametrize("d,L,k", [(128, 33, 33), (64, 4097, 129), (128, 1000, 289), (64, 1, 1), (64, 70, 31)])
def test_assign_step_f32_tile_edges(d, L, k):
    g = np.random.default_rng(1000 * L + k)
    xhat, chat = (x / np.linalg.norm(x, axis=1, keepdims=True)
                  for x in (g.standard_normal((L, d)), g.standard_normal((k, d))))
    xhat, chat = wo.quant(xhat, "f32"), wo.quant(chat, "f32")
    chat[k // 2:] = np.where(np.arange(k // 2, k)[:, None] % 5 == 0, chat[0], chat[k // 2:])
    a = wb.wave_kmeans_assign_step(torch.from_numpy(xhat).float().cuda(), torch.from_numpy(chat).float().cuda())
    torch.cuda.synchronize()
    assert pu.check_assign(a.cpu().numpy(), xhat, chat, f"d={d} L={L} k={k}") == 0


# Which rounds run.  Short segments whose one-workgroup kernel is switched off go the way of the long ones:
# incremental rounds, or (fewer than four points per cluster, a ragged last segment counted as a whole one)
# a full pass every round.
@pytest.mark.parametrize("N,d,L,k,no_small,assign", [
    (2125, 128, 1024, 64, "1", "assign_delta"), (700, 64, 300, 128, "1", "refine"), (2048, 128, 1024, 256, "", "assign_delta"),
    (2125, 128, 1024, 256, "", "refine"), (2125, 128, 1024, 64, "", "kmeans_small")])
def test_short_segments_and_few_points_per_cluster(N, d, L, k, no_small, assign, monkeypatch):
    iters = 4
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="short", B=1, Hq=2, Hkv=2, N=N, d=d, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=iters, n_components=64)
    K, V = synth.make_kv(wl)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    monkeypatch.setenv("WAVE_NO_SMALL_KMEANS", no_small)
    wb.wave_profile_enable(True)
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 0, 0, L, k, iters, 0)
    launches = {name: n for name, (_, n) in wb.wave_profile_read().items()}
    wb.wave_profile_enable(False)
    for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
        got = ix.t[name].cpu()
        assert torch.equal(got.double(), ref[name].reshape(got.shape).double()), name
    assert {"assign_delta", "refine", "kmeans_small"} & set(launches) == {assign}, launches


# Keys that are no numbers: every similarity of their segment is NaN, and no comparison decides.  The
# partition is still one of all tokens, and the units beside them are what they are without.
@pytest.mark.parametrize("dtype,L,k", [("bf16", 256, 16), ("bf16", 2100, 64), ("bf16", 300, 250), ("f32", 300, 40)])
@pytest.mark.parametrize("bad", [float("nan"), -float("nan"), float("inf")])
def test_keys_that_are_no_numbers(dtype, L, k, bad):
    N = 4300
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="nan", dtype=dtype, B=1, Hq=2, Hkv=2, N=N, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=4, n_components=64)
    K, V = synth.make_kv(wl)
    K[0, 0, 10, 3] = K[0, 0, N - 1] = bad
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 0, 0, L, k, wl.iters, 0)
    torch.cuda.synchronize()
    sizes, offsets, perm = (ix.t[name][0].cpu() for name in ("sizes", "offsets", "perm"))
    assert (perm.sort(-1).values == torch.arange(N)).all() and (sizes >= 0).all()
    assert (offsets[:, 0] == 0).all() and torch.equal(offsets.diff(dim=-1), sizes) and (offsets[:, -1] == N).all()
    ref = pu.oracle_build(wl, K, V, units=[(0, 1)])[(0, 1)]
    for name in ("centroids", "vsum", "sizes", "perm"):
        assert np.array_equal(ix.t[name][0, 1].double().cpu().numpy(), getattr(ref, name)), name


# Segments around the rows that the normalise step takes at once (64 of bf16 at d = 128, 32 of f32) and that a
# workgroup takes (128): whole batches, rows one by one behind them, none of either.  (The segment mean takes batches of
# eight and four rows of a lane group: 96 and 200 rows have fours and single rows behind them.)
@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("L", [1, 15, 16, 33, 64, 96, 127, 129, 191, 200, 257])
def test_segments_around_the_normalise_batches(dtype, d, L):
    N, k = 5 * L + 3, 4
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="rows", dtype=dtype, B=1, Hq=2, Hkv=2, N=N, d=d, n_sink=1, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=3, n_components=8)
    K, V = synth.make_kv(wl)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 1, 0, L, k, wl.iters, 0)
    torch.cuda.synchronize()
    for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
        got = ix.t[name].cpu()
        assert torch.equal(got.double(), ref[name].reshape(got.shape).double()), name


# Around the most segments that the normalise step takes in pieces of 64 rows: a piece for each row of workgroups that
# 128 rows leave without one, the second short; with the exponent range, a workgroup a CU (four segments of 4096).
@pytest.mark.parametrize("dtype,d,B,S,L,k", [
    ("bf16", 128, 51, 5, 100, 4), ("bf16", 64, 64, 4, 127, 4), ("f32", 64, 51, 5, 65, 4), ("f32", 128, 64, 4, 65, 4),
    ("bf16", 128, 4, 1, 4096, 20), ("bf16", 128, 5, 1, 4096, 20), ("bf16", 64, 1, 1, 4097, 20)])
def test_segments_around_the_normalise_pieces(dtype, d, B, S, L, k):
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="pieces", dtype=dtype, B=B, Hq=1, Hkv=1, N=S * L, d=d, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=3, n_components=16)
    K, V = synth.make_kv(wl)
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 0, 0, L, k, wl.iters, 0)
    for (b, h), ref in pu.oracle_build(wl, K, V, units=[(b, 0) for b in sorted({0, B - 1})]).items():
        for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
            assert np.array_equal(ix.t[name][b, h].double().cpu().numpy(), getattr(ref, name)), (b, name)


# Clusters of few members: eight or two of them in flight (all workgroups resident, the first that are not, four members a
# cluster and fewer), clusters of no member, of one and of more than eight; a ragged last segment.
@pytest.mark.parametrize("kind,dtype,d,B,L,k,N", [
    ("plain", "bf16", 128, 24, 1024, 512, 1024), ("plain", "bf16", 128, 25, 1024, 512, 1024), ("ties", "bf16", 64, 49, 600, 512, 600),
    ("mixture", "f32", 128, 13, 1100, 500, 1100), ("plain", "bf16", 64, 30, 512, 500, 960), ("plain", "bf16", 128, 50, 1024, 256, 1024),
    ("plain", "bf16", 128, 50, 1023, 256, 1023)])
def test_clusters_of_few_members_match_oracle(kind, dtype, d, B, L, k, N):
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="few", dtype=dtype, B=B, Hq=1, Hkv=1, N=N, d=d, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=2)
    K = _keys(kind, B, N, d, N + k).to(tdt)
    V = torch.randn(B, 1, N, d, generator=torch.Generator().manual_seed(1)).to(tdt)
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 0, 0, L, k, wl.iters, 0)
    for (b, h), ref in pu.oracle_build(wl, K, V, units=[(0, 0), (B - 1, 0)]).items():
        for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
            assert np.array_equal(ix.t[name][b, h].double().cpu().numpy(), getattr(ref, name)), (b, name)


# Full passes with the centroids in LDS and one list of near-ties for all segments: 2048 segments of 1537 points
# (a fragment with one point) with 31 * 13 clusters; three units against the oracle.  (refine, not
# assign_listed, takes the near-ties.)
def test_full_passes_of_many_segments_keep_their_centroids_in_lds():
    B, Hkv, L, k, iters, N = 64, 8, 1537, 403, 3, 4 * 1537
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="many", B=B, Hq=Hkv, Hkv=Hkv, N=N, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=iters)
    g = torch.Generator(device="cuda").manual_seed(3)
    K, V = (torch.randn(B, Hkv, N, 128, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    wb.wave_profile_enable(True)
    ix = wb.wave_index_build(K, V, 0, 0, L, k, iters, 0)
    launches = {name: n for name, (_, n) in wb.wave_profile_read().items()}
    wb.wave_profile_enable(False)
    assert launches["refine"] == launches["assign_mfma"] == iters and "assign_listed" not in launches
    units = [(0, 0), (31, 5), (B - 1, Hkv - 1)]
    for (b, h), ref in pu.oracle_build(wl, K, V, units=units).items():
        for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
            assert np.array_equal(ix.t[name][b, h].double().cpu().numpy(), getattr(ref, name)), (b, h, name)


# Segments that one workgroup clusters: points in registers up to 1024 (d = 128) or 2048 (d = 64), member
# sums in LDS up to 64 or 128 clusters, their edges and remainders; segments whose sums round (wide), clusters
# that run empty (ties), and rounds enough that the points stop moving before the last.
@pytest.mark.parametrize("kind,d,L,k,iters", [
    ("mixture", 128, 1024, 64, 9), ("plain", 128, 1024, 65, 6), ("plain", 128, 1025, 64, 6), ("mixture", 128, 2048, 128, 8),
    ("mixture", 64, 2048, 128, 9), ("plain", 64, 2047, 127, 5), ("ties", 128, 1000, 64, 7), ("ties", 64, 33, 32, 6),
    ("wide", 128, 700, 40, 5), ("wide", 64, 2040, 128, 4), ("wide", 128, 2048, 33, 4), ("plain", 128, 31, 1, 30),
    ("mixture", 128, 513, 33, 1), ("mixture", 64, 257, 64, 2)])
def test_segments_of_one_workgroup_match_oracle(kind, d, L, k, iters):
    N = 5 + 2 * L + L // 3 + 1
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="short", B=2, Hq=1, Hkv=1, N=N, d=d, n_sink=2, n_local=3,
                      segment_len=L, clusters_per_segment=k, iters=iters)
    K = _keys(kind, 2, N, d, N + k).to(torch.bfloat16)
    V = torch.randn(2, 1, N, d, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), wl.n_sink, wl.n_local, L, k, iters, 0)
    torch.cuda.synchronize()
    for name in wb.BUFFER_NAMES:
        assert torch.equal(ix.t[name].cpu().double(), ref[name].reshape(ix.t[name].shape).double()), name


# f32 rounds: the tiles shared by the waves of a workgroup, or (1024 fragments of points or more: the last two)
# a wave per fragment; workgroups of 16 .. 64 clusters with a remainder; clusters of more than 128 members
# whose sums are exact in any order and ("wide") are not; clusters that stay empty.
@pytest.mark.parametrize("kind,B,d,N,L,k,iters", [
    ("mixture", 2, 64, 4101, 2048, 128, 6), ("plain", 2, 128, 1005, 1000, 33, 5), ("ties", 2, 64, 700, 333, 65, 5),
    ("plain", 1, 128, 805, 800, 1, 3), ("wide", 2, 64, 2405, 1200, 7, 4), ("plain", 1, 64, 2405, 2400, 200, 4),
    ("mixture", 2, 64, 17005, 8500, 17, 4), ("plain", 2, 128, 17005, 17000, 40, 3)])
def test_f32_rounds_match_oracle(kind, B, d, N, L, k, iters):
    wl = synth.scaled(synth.WORKLOADS["tiny_f32"], name="f32", dtype="f32", B=B, Hq=1, Hkv=1, N=N, d=d, n_sink=2,
                      n_local=3, segment_len=L, clusters_per_segment=k, iters=iters)
    K = _keys(kind, B, N, d, N + k)
    V = torch.randn(B, 1, N, d, generator=torch.Generator().manual_seed(1))
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), wl.n_sink, wl.n_local, L, k, iters, 0)
    torch.cuda.synchronize()
    for name in wb.BUFFER_NAMES:
        assert torch.equal(ix.t[name].cpu().double(), ref[name].reshape(ix.t[name].shape).double()), name


# The front of a build: segment means from pieces of 256 rows or more (the last one short), key scales at which the
# fp32 quotient of the normalise step has to give way to the fp64 one (subnormal and huge keys, a row equal to
# the mean, quotients in the middle between two bf16 values), seeds of nearly all points of a segment.
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,L,k,scale", [(2053, 2048, 64, 1.0), (1505, 1100, 20, 2.0 ** -118), (1505, 1500, 33, 2.0 ** 60),
                                         (4105, 513, 8, 2.0 ** -30), (305, 300, 299, 1.0), (8197, 8192, 2000, 0.0)])
def test_front_of_the_build_matches_oracle(dtype, N, L, k, scale):
    d = 64
    g = torch.Generator().manual_seed(N + k)
    # halves, quarters, ...: sums and quotients land on and next to the middle between two bf16 values
    x = torch.randint(-8, 9, (1, 1, N, d), generator=g).float() / 8
    x[0, 0, 2:N - 3:2] *= 1 + torch.randint(0, 3, (1,), generator=g).float()
    if scale == 0.0:
        x = torch.randn(1, 1, N, d, generator=g)
        scale = 1.0
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="front", dtype=dtype, B=1, Hq=1, Hkv=1, N=N, d=d, n_sink=2,
                      n_local=3, segment_len=L, clusters_per_segment=k, iters=2)
    K = (x * scale).to(tdt)
    V = torch.randn(1, 1, N, d, generator=g).to(tdt)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), wl.n_sink, wl.n_local, L, k, 2, 0)
    torch.cuda.synchronize()
    for name in ("sizes", "perm", "centroids"):
        assert torch.equal(ix.t[name].cpu().double(), ref[name].reshape(ix.t[name].shape).double()), name


# Around the most segments whose workgroups decide their near-ties and listed points themselves (128 segments of
# two workgroups) and whose first and last rounds sort and sum in one launch (127); more changed centroids than half of
# a CU's LDS holds, the most that are resident, and more listed points than one batch; a ragged last segment.
@pytest.mark.parametrize("kind,B,d,L,k,listed,sort", [
    ("plain", 42, 128, 2100, 300, 0, 0), ("mixture", 43, 128, 2100, 512, 1, 1), ("plain", 43, 64, 2050, 500, 1, 1),
    ("ties", 43, 128, 2049, 65, 1, 1), ("plain", 32, 64, 2080, 200, 0, 1), ("wide", 42, 128, 2100, 100, 0, 0)])
def test_rounds_around_the_most_segments_decided_at_once(kind, B, d, L, k, listed, sort):
    S = 4 if B == 32 else 3
    iters, N = 5, S * L - 70
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="at_once", B=B, Hq=1, Hkv=1, N=N, d=d, n_sink=0, n_local=0,
                      segment_len=L, clusters_per_segment=k, iters=iters)
    K = _keys(kind, B, N, d, N + k).to(torch.bfloat16)
    V = torch.randn(B, 1, N, d, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16)
    wb.wave_profile_enable(True)
    ix = wb.wave_index_build(K.cuda(), V.cuda(), 0, 0, L, k, iters, 0)
    launches = {name: n for name, (_, n) in wb.wave_profile_read().items()}
    wb.wave_profile_enable(False)
    assert launches.get("assign_listed", 0) == listed * iters and launches.get("sort", 0) == 2 * sort, launches
    for (b, h), ref in pu.oracle_build(wl, K, V, units=[(0, 0), (B - 1, 0)]).items():
        for name in ("centroids", "vsum", "sizes", "offsets", "perm", "k_perm", "v_perm"):
            assert np.array_equal(ix.t[name][b, h].double().cpu().numpy(), getattr(ref, name)), (b, name)


# f32: the points of a workgroup whose two best are closer than fp32 tells apart, decided from fp64 similarities by
# a wave each and, what is left of four, by the workgroup: 0 .. 32 of a fragment's points (a workgroup has one
# fragment, from 1024 fragments on four), the centroids of a lane at their edges.
@pytest.mark.parametrize("d,L,k", [(64, 229, 2), (128, 229, 64), (64, 1000, 65), (128, 500, 129), (64, 300, 300), (64, 32900, 40)])
def test_f32_near_ties_of_a_workgroup(d, L, k):
    g = np.random.default_rng(L + k)
    chat = g.standard_normal((k, d))
    chat /= np.linalg.norm(chat, axis=1, keepdims=True)
    chat = chat.astype(np.float32)
    pairs = min(4, k // 2)
    first, second = np.arange(pairs), k - 1 - np.arange(pairs)
    chat[second] = chat[first]
    chat[second[1::2], 3] = np.nextafter(chat[first[1::2], 3], np.float32(2.0))   # (every other pair: one step apart)
    counts = [0, 1, 3, 4, 5, 7, 31, 32]                                            # near-ties of a fragment of 32 points
    others = np.arange(pairs, k - pairs) if k > 2 * pairs else np.zeros(0, dtype=int)
    target = np.empty(L, dtype=int)
    for f in range((L + 31) // 32):
        n = min(32, L - 32 * f)
        near = np.arange(n) < counts[f % len(counts)] if others.size else np.ones(n, dtype=bool)
        near = g.permutation(near)
        target[32 * f:32 * f + n] = np.where(near, g.choice(np.concatenate([first, second]), n),
                                             g.choice(others, n) if others.size else 0)
    x = (chat[target] + 0.02 * g.standard_normal((L, d))).astype(np.float32)
    # (equal rows get equal sums: one order for every centroid, which a matrix product does not promise)
    x64 = x.astype(np.float64)
    sims = np.stack([(x64 * c).sum(1) for c in chat.astype(np.float64)], axis=1)
    a = wb.wave_kmeans_assign_step(torch.from_numpy(x).cuda(), torch.from_numpy(chat).cuda())
    torch.cuda.synchronize()
    # (a pair one step apart: the two fp64 sums, in whatever order, differ by 1e-9 where their rounding is 1e-16)
    assert np.array_equal(a.cpu().numpy(), np.argmax(sims, axis=1))


# Channels that are constant in a segment (head dimensions padded with zeros, of either sign): their normalised keys are
# zero beside quotients that fp32 decides and others that it does not, rows that are zero as a whole, tiny and huge keys.
@pytest.mark.parametrize("d,scale", [(64, 1.0), (128, 1.0), (128, 2.0 ** -60), (64, 2.0 ** 110)])
def test_constant_channels_match_oracle(d, scale):
    N, L, k = 705, 350, 20
    g = torch.Generator().manual_seed(d)
    x = torch.randn(1, 1, N, d, generator=g)
    x[..., d // 2:] = 0.0
    x[:, :, ::3, d // 2:] = -0.0
    x[..., 1] = 3.0
    x[:, :, 9:12] = x[:, :, 9:10]
    x[:, :, 2:352, 2] = torch.randint(0, 2, (350,), generator=g) * 2.0 ** -40    # (zero on average or next to it)
    wl = synth.scaled(synth.WORKLOADS["llama8b_32k"], name="padded", B=1, Hq=1, Hkv=1, N=N, d=d, n_sink=2, n_local=3,
                      segment_len=L, clusters_per_segment=k, iters=3)
    K = (x * scale).to(torch.bfloat16)
    V = torch.randn(1, 1, N, d, generator=g).to(torch.bfloat16)
    ref = pu.oracle_index_arrays(wl, pu.oracle_build(wl, K, V))
    ix = wb.wave_index_build(K.cuda(), V.cuda(), wl.n_sink, wl.n_local, L, k, 3, 0)
    torch.cuda.synchronize()
    for name in ("sizes", "perm", "centroids"):
        assert torch.equal(ix.t[name].cpu().double(), ref[name].reshape(ix.t[name].shape).double()), name
