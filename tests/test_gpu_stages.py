"""Stage-isolated GPU parity: each libasl kernel is fed the oracle-side input of its stage
(cast to the kernel's input dtype) and compared with the oracle's output for that stage.
Integer outputs (ranks, statistic integers, top-k indices, gathered bytes) must be bit-exact."""
import ctypes as C

import numpy as np
import pytest

from oracle import asl_oracle as orc
from paper_2601_07667_amd import asl, synth
import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_device):
    c = asl.Asl(262144, 8, 32 * 64)
    yield c
    assert c.asl_device_fault() == 0, "a workgroup gave up waiting for its peers during this module"
    c.close()


def _torch():
    import torch
    return torch


# ----------------------------------------------------------------------------- pool
@pytest.mark.parametrize("rows,T,S", [(1, 1, 1), (2, 5, 7), (8, 496, 7), (3, 1000, 1), (8, 32736, 7),
                                      (2, 777, 129), (8, 131040, 7)])
def test_pool(ctx, gpu_device, rows, T, S):
    torch = _torch()
    rng = np.random.default_rng(rows * 7 + T)
    u = rng.random((rows, T), dtype=np.float32)
    ud = torch.from_numpy(u).to(gpu_device)
    p = torch.empty_like(ud)
    s = torch.empty(T, dtype=torch.float32, device=gpu_device)
    ctx.asl_pool(ud, rows, T, S, p, s)
    ref = orc.avg_pool1d(u.astype(np.float64), S)
    np.testing.assert_allclose(p.cpu().numpy(), ref, rtol=2e-6, atol=1e-7)
    np.testing.assert_allclose(s.cpu().numpy(), ref.sum(axis=0), rtol=4e-6, atol=1e-7)


# ----------------------------------------------------------------------------- rank
def _rank_case(ctx, dev, s: np.ndarray):
    torch = _torch()
    T = s.shape[0]
    sd = torch.from_numpy(s).to(dev)
    out = torch.full((T,), -1, dtype=torch.int32, device=dev)
    ctx.asl_rank(sd, T, out)
    np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), orc.rank_desc(s.astype(np.float64)))


@pytest.mark.parametrize("T", [1, 2, 63, 64, 65, 2047, 2048, 2049, 5000, 32736, 131040, 262080])
def test_rank_random_with_ties(ctx, gpu_device, T):
    rng = np.random.default_rng(T)
    s = rng.standard_normal(T).astype(np.float32)
    if T > 10:
        s[rng.integers(0, T, T // 4)] = s[rng.integers(0, T, T // 4)]     # exact ties
        s[rng.integers(0, T, T // 8)] = 0.0
        s[rng.integers(0, T, T // 8)] = -0.0                               # -0 ties with +0
    _rank_case(ctx, gpu_device, s)


@pytest.mark.parametrize("T", [1, 33, 500, 12288, 12289])
def test_rank_over_its_own_scores(ctx, gpu_device, T):
    """Ranks written over the scores they are made from, over part of them, and right behind them."""
    torch = _torch()
    s = np.round(np.random.default_rng(T).standard_normal(T), 2).astype(np.float32)
    ref = orc.rank_desc(s.astype(np.float64))
    for shift in (0, T // 2, T):
        for rank in (ctx.asl_rank, asl.asl_rank_static):
            buf = torch.zeros(2 * T, dtype=torch.float32, device=gpu_device)
            buf[:T] = torch.from_numpy(s).to(gpu_device)
            out = buf.view(torch.int32)[shift:shift + T]
            rank(buf[:T], T, out)
            np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), ref)


@pytest.mark.parametrize("T", [524288, 524289, 700001])
def test_rank_beyond_the_small_tile_limit(gpu_device, T):
    """Sizes with half as many tiles of 4096 tokens as one ranking takes, one more with a single token in it, and a ragged one, with
    heavy ties.  (The tiles change at 131072 and 1048576 tokens: test_rank_buckets, test_rank_where_the_bucket_count_changes.)"""
    torch = _torch()
    c = asl.Asl(T, 1, 32)
    rng = np.random.default_rng(T)
    s = np.round(rng.standard_normal(T), 2).astype(np.float32)        # heavy ties
    sd = torch.from_numpy(s).to(gpu_device)
    out = torch.full((T,), -1, dtype=torch.int32, device=gpu_device)
    c.asl_rank(sd, T, out)
    np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), orc.rank_desc(s.astype(np.float64)))
    assert c.asl_device_fault() == 0
    c.close()


def _rank_sample_positions(T):
    """Where a ranking of T > 12288 scores takes its sample from."""
    most = min(4096 if T <= 262144 else 8192, max(1024, T // 32))
    stride = -(-T // most)
    j = np.arange(T // stride, dtype=np.uint64)
    return (j * stride + (((j * 2654435761 % 2 ** 32) >> 16) * stride >> 16)).astype(np.int64)


@pytest.mark.parametrize("T", [12289, 131072, 262145])
@pytest.mark.parametrize("kind", ["lognormal", "two-signs", "equal", "third-zero", "few", "sorted", "outliers",
                                  "unsampled-equal", "unsampled-close"])
def test_rank_buckets(gpu_device, T, kind):
    """Scores that fill the ranking's buckets evenly, that its sample's bins do not tell apart, and
    that the sample misses (a bucket of more pairs than LDS holds): integers, exact.  Sizes: the smallest that
    takes buckets, the 2048-token tiles' and the first of the 4096-token tiles, with one token in the last."""
    rng = np.random.default_rng(T)
    s = np.exp(2 * rng.standard_normal(T)).astype(np.float32)
    if kind == "two-signs":
        s = rng.standard_normal(T).astype(np.float32)
    elif kind == "equal":
        s[:] = 0.25
    elif kind == "third-zero":
        s[rng.random(T) < 1 / 3] = 0.0
    elif kind == "few":
        s = np.round(3 * rng.standard_normal(T)).astype(np.float32)
    elif kind == "sorted":
        s = np.sort(s)
    elif kind == "outliers":
        s = (1e-3 * (1 + 0.02 * rng.standard_normal(T))).astype(np.float32)
        s[::T // 40] = 50.0
    elif kind.startswith("unsampled"):
        rest = np.ones(T, dtype=bool)
        rest[_rank_sample_positions(T)] = False
        s[rest] = 0.5 if kind == "unsampled-equal" else 0.5 + 1e-6 * np.round(rng.random(int(rest.sum())) * 10)
    c = asl.Asl(T, 1, 32)
    _rank_case(c, gpu_device, s)
    c.close()


def _graph_us(f, n=20):
    """Duration of one call of f in a replayed graph of n, in us: the median of five replays."""
    import torch
    f()
    torch.cuda.synchronize()
    g, times = torch.cuda.CUDAGraph(), []
    with torch.cuda.graph(g):
        for _ in range(n):
            f()
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) / n * 1e3)
    return sorted(times[1:])[2]


@pytest.mark.parametrize("T", [16000, 131040, 262080, 1048544])
def test_rank_time_hardly_depends_on_the_scores(gpu_device, T):
    """Scores that repeat, have a period or lie close together beside outliers: a ranking takes at most twice as long as that of
    distinct, spread ones (a radix sort, whatever the scores, takes twice as long), and is exact."""
    import torch
    rng = np.random.default_rng(T)
    spread = np.exp(2 * rng.standard_normal(T)).astype(np.float32)
    near, far = (1 + 0.02 * rng.standard_normal(T)).astype(np.float32), (1 + 1e-5 * rng.random(T)).astype(np.float32)
    near[rng.integers(0, T, T // 300)] += 300 * rng.random(T // 300).astype(np.float32) + 50
    far[5] = -3e38
    kinds = {"third-zero": np.where(rng.random(T) < 1 / 3, np.float32(0), spread), "equal": np.full(T, 0.25, np.float32),
             "few": np.round(3 * rng.standard_normal(T)).astype(np.float32), "two": np.where(rng.random(T) < 0.5, 0.25, 0.5).astype(np.float32),
             "period": np.tile(spread[:32], T // 32 + 1)[:T], "sorted": np.sort(spread), "cluster": near, "one far": far}
    c = asl.Asl(T, 1, 32)
    out = torch.empty((T,), dtype=torch.int32, device=gpu_device)
    d = torch.from_numpy(spread).to(gpu_device)
    limit = 2 * _graph_us(lambda: c.asl_rank(d, T, out))
    for kind, s in kinds.items():
        _rank_case(c, gpu_device, s)
        d = torch.from_numpy(s).to(gpu_device)
        us = _graph_us(lambda: c.asl_rank(d, T, out))
        assert us <= limit, f"{kind}: {us:.1f} us, limit {limit:.1f}"
    c.close()


@pytest.mark.parametrize("T", [40000, 131040, 262080, 1048544])
def test_rank_time_of_scores_few_ulps_apart(gpu_device, T):
    """Half of the scores, or a third, so close together that neither the sample's bins nor the sub-bins of the full ones tell them
    apart, beside spread ones: the sample is sorted, and a ranking takes at most five times as long as that of spread ones (before:
    in one bucket of a single workgroup, up to 140 times), and is exact."""
    import torch
    rng = np.random.default_rng(T)
    spread = np.exp(2 * rng.standard_normal(T)).astype(np.float32)
    part, one = rng.random(T), np.float32(1).view(np.int32)
    wide = np.exp(4 * rng.standard_normal(T))
    kinds = {f"within {n} ulps": np.where(part < 0.5, (one + rng.integers(0, n, T)).astype(np.int32).view(np.float32), spread) for n in (3, 100)}
    kinds["two clusters"] = np.select([part < 1 / 3, part < 2 / 3], [1 + 1e-6 * rng.standard_normal(T), 1 + 1e-3 * rng.standard_normal(T)],
                                      wide).astype(np.float32)
    kinds["mostly"] = np.where(part < 0.97, (one + rng.integers(0, 20, T)).astype(np.int32).view(np.float32), wide).astype(np.float32)
    c = asl.Asl(T, 1, 32)
    out = torch.empty((T,), dtype=torch.int32, device=gpu_device)
    d = torch.from_numpy(spread).to(gpu_device)
    limit = 5 * _graph_us(lambda: c.asl_rank(d, T, out))
    for kind, s in kinds.items():
        _rank_case(c, gpu_device, s)
        d = torch.from_numpy(s).to(gpu_device)
        us = _graph_us(lambda: c.asl_rank(d, T, out))
        assert us <= limit, f"{kind}: {us:.1f} us, limit {limit:.1f}"
    c.close()


def _score_kinds(T):
    """Spread scores, scores that repeat, and scores that lie close together beside an outlier."""
    rng = np.random.default_rng(T)
    spread = np.exp(2 * rng.standard_normal(T)).astype(np.float32)
    near = (1 + 0.02 * rng.standard_normal(T)).astype(np.float32)
    near[T // 2] = 1e3
    return {"spread": spread, "third-zero": np.where(rng.random(T) < 1 / 3, np.float32(0), spread),
            "two": np.where(rng.random(T) < 0.5, 0.25, 0.5).astype(np.float32), "near": near}


@pytest.mark.parametrize("T,limit", [(8000, 1.5), (12000, 2.6)])
def test_short_ranking_times(gpu_device, T, limit):
    """Rankings in one launch: counting does not depend on the scores (8000 tokens), and long bins are cut in turn (before: 2.4 to
    2.8 and 2.6 to 3.4 times the spread scores' time, everything once more by counting)."""
    import torch
    c = asl.Asl(T, 1, 32)
    out, us = torch.empty((T,), dtype=torch.int32, device=gpu_device), {}
    for kind, s in _score_kinds(T).items():
        d = torch.from_numpy(s).to(gpu_device)
        us[kind] = _graph_us(lambda: c.asl_rank(d, T, out))
    c.close()
    assert max(us.values()) <= limit * us["spread"], us


@pytest.mark.parametrize("rows,T", [(8, 8000), (8, 12000), (8, 16000), (64, 30000)])
def test_short_top_k_times(gpu_device, rows, T):
    """Top-k by one workgroup per row: the bin that holds the threshold is cut in turn (before: up to 2.6 times the spread scores'
    time, the whole row again by digits)."""
    import torch
    c, k, us = asl.Asl(T + 32, rows, 32), 2048, {}
    idx = torch.empty((rows, k + 32), dtype=torch.int32, device=gpu_device)
    p = asl.make_params(1, 1, 64, T + 32, 32, 7, k + 32)
    for kind, s in _score_kinds(T).items():
        d = torch.from_numpy(s).to(gpu_device)[None].repeat(rows, 1).contiguous()
        us[kind] = _graph_us(lambda: c.asl_select_topk(p, d, rows, idx))
    c.close()
    assert max(us.values()) <= 2 * us["spread"], us


def test_top_k_time_of_scores_with_a_period(gpu_device):
    """Rows that repeat every 32 scores, where one run of four is sampled per 128: no more than a few times as long as rows without a
    period (with the runs at one phase, eight times: the bound let too many or too few pass)."""
    import torch
    T, rows, us = 131040, 8, []
    rng = np.random.default_rng(1)
    spread = np.exp(2 * rng.standard_normal(T)).astype(np.float32)
    c = asl.Asl(T + 32, rows, 32)
    idx = torch.empty((rows, 2048 + 32), dtype=torch.int32, device=gpu_device)
    p = asl.make_params(1, 1, 64, T + 32, 32, 7, 2048 + 32)
    for s in (spread, np.tile(spread[:32], T // 32)):
        d = torch.from_numpy(s).to(gpu_device)[None].repeat(rows, 1).contiguous()
        us.append(_graph_us(lambda: c.asl_select_topk(p, d, rows, idx)))
    c.close()
    assert us[1] <= 4 * us[0], us


def test_rank_special(ctx, gpu_device):
    T = 5000
    _rank_case(ctx, gpu_device, np.ones(T, dtype=np.float32))                               # all equal
    _rank_case(ctx, gpu_device, np.arange(T, dtype=np.float32))                             # increasing
    _rank_case(ctx, gpu_device, -np.arange(T, dtype=np.float32))                            # decreasing
    _rank_case(ctx, gpu_device, np.exp(np.random.default_rng(1).normal(0, 3, T)).astype(np.float32))
    tiny = (np.random.default_rng(2).random(T) * 1e-40).astype(np.float32)                  # denormals
    _rank_case(ctx, gpu_device, tiny)


def test_rank_is_deterministic(ctx, gpu_device):
    torch = _torch()
    T = 131040
    s = torch.from_numpy(np.random.default_rng(3).random(T, dtype=np.float32)).to(gpu_device)
    a = torch.empty(T, dtype=torch.int32, device=gpu_device)
    b = torch.empty(T, dtype=torch.int32, device=gpu_device)
    ctx.asl_rank(s, T, a)
    ctx.asl_rank(s, T, b)
    assert torch.equal(a, b)


@pytest.mark.parametrize("T", [2048 * 3 - 1, 2048 * 3, 2048 * 3 + 1, 4095, 4096, 4097, 64 * 33 + 7, 2048 * 17 - 1, 2048 * 17,
                               2048 * 17 + 1, 4096 * 9 - 1, 4096 * 9, 4096 * 9 + 1, 64 * 533 + 7])
def test_rank_and_select_at_tile_boundaries(ctx, gpu_device, T):
    """Sizes one below, at and one above multiples of the sort tile (2048) and the select tile (4096), above 12288
    scores, from where the tiles are in use; and the same below, where one launch takes the whole row."""
    rng = np.random.default_rng(T)
    s = np.round(rng.standard_normal(T), 2).astype(np.float32)            # heavy ties
    _rank_case(ctx, gpu_device, s)
    for budget in (9, T // 3 + 8, T + 8):                                   # k = 1, ~T/3, T
        _select_case(ctx, gpu_device, np.stack([s, -s]), budget, 8)


# Up to 12288 scores are ranked in one launch (up to 8192 of them 32 tokens per workgroup, then 64 places) and selected
# from by one workgroup per row; above, the partition (tiles of 2048) and the bound / filter / finish launches (tiles of 4096) take over.
@pytest.mark.parametrize("T", [31, 32, 33, 95, 1023, 1025, 8192, 12256, 12257, 12287, 12288, 12289, 14335, 14336, 14337,
                               16383, 16384, 16385])
def test_short_vectors_and_their_limit(ctx, gpu_device, T):
    rng = np.random.default_rng(T)
    s = np.round(rng.standard_normal(T), 2).astype(np.float32)            # heavy ties
    wild = rng.standard_normal(T).astype(np.float32) * np.float32(1e-39)  # denormals, both zeros, infinities
    wild[rng.integers(0, T, T // 3 + 1)] = 0.0
    wild[rng.integers(0, T, T // 4 + 1)] = -0.0
    wild[rng.integers(0, T, 2)] = np.inf
    wild[rng.integers(0, T, 2)] = -np.inf
    for v in (s, wild, np.ones(T, dtype=np.float32), np.arange(T, dtype=np.float32)):
        _rank_case(ctx, gpu_device, v)
    for budget in (9, T // 3 + 8, T + 8):                                   # k = 1, ~T/3, T
        _select_case(ctx, gpu_device, np.stack([s, -s, wild]), budget, 8)


@pytest.mark.parametrize("T", [1, 2, 127, 128, 129, 255, 257, 1024, 5120, 5121, 8192, 8193, 9994, 12287, 12288, 12289, 16385, 32736, 32767,
                               32768, 32769])
@pytest.mark.parametrize("kind", ["lognormal", "pairs", "third-zero", "few", "two", "outlier"])
def test_short_vectors_by_bins(ctx, gpu_device, T, kind):
    """Vectors up to and just beyond what one workgroup takes, whose scores their bins tell apart (with equal neighbours, so
    that bins of a few keys straddle the workgroups' places) and whose do not: repeated scores, in one, some or all bins,
    and one outlier that pushes different scores into one bin.  Integers, exact."""
    rng = np.random.default_rng(T)
    s = np.exp(2 * rng.standard_normal(T)).astype(np.float32)
    if kind == "pairs":
        s = s[rng.permutation(T) // 3]
    elif kind == "third-zero":
        s[rng.random(T) < 1 / 3] = 0.0
    elif kind == "few":
        s = np.round(3 * rng.standard_normal(T)).astype(np.float32)
    elif kind == "two":
        s = np.where(rng.random(T) < 0.5, 0.25, 0.5).astype(np.float32)
    elif kind == "outlier":
        s = (1 + 1e-5 * rng.random(T)).astype(np.float32)
        s[T // 2] = -3e38
    _rank_case(ctx, gpu_device, s)
    for budget in sorted({9, T // 3 + 9, T + 8}):                           # k = 1, ~T/3, T
        _select_case(ctx, gpu_device, np.stack([s, -s]), budget, 8)


@pytest.mark.parametrize("T", [12289, 40000, 131072, 300000])
@pytest.mark.parametrize("share", [1e-3, 3e-3, 0.02, 0.3])
@pytest.mark.parametrize("side", ["above", "below", "both"])
def test_rank_of_a_cluster_and_outliers(gpu_device, T, share, side):
    """Scores close to each other and a share of outliers far above, below or on both sides: fewer than the ranking's end
    buckets are made for, about as many, and more.  Integers, exact."""
    rng = np.random.default_rng(T)
    s = (1 + 0.02 * rng.standard_normal(T)).astype(np.float32)
    out = rng.random(T) < share
    far = np.exp(4 + 2 * rng.random(T)).astype(np.float32)
    if side == "below":
        far = 1 / far
    elif side == "both":
        far = np.where(rng.random(T) < 0.5, far, 1 / far)
    s[out] = far[out]
    c = asl.Asl(T, 1, 32)
    _rank_case(c, gpu_device, s)
    c.close()


@pytest.mark.parametrize("rows,T", [(63, 16385), (64, 16385), (64, 32768), (64, 32769)])
def test_select_rows_one_workgroup_takes(gpu_device, rows, T):
    """The fewest rows and longest that one workgroup per row selects from, and one beyond each: integers, exact."""
    rng = np.random.default_rng(rows + T)
    s = np.exp(2 * rng.standard_normal((rows, T))).astype(np.float32)
    s[::3, ::4] = 0.0
    c = asl.Asl(T + 8, rows, rows * 8)
    for budget in (9, T // 20, T + 8):
        _select_case(c, gpu_device, s, budget, 8)
    c.close()


@pytest.mark.parametrize("T", [264000, 264001, 1048576, 1048577])
def test_rank_where_the_bucket_count_changes(gpu_device, T):
    """The last size of 240 buckets, the first and last of 512 and the first beyond, scores mostly distinct: exact."""
    c = asl.Asl(T, 1, 32)
    _rank_case(c, gpu_device, np.exp(2 * np.random.default_rng(T).standard_normal(T)).astype(np.float32))
    c.close()


@pytest.mark.parametrize("kind", ["distinct", "third-zero"])
def test_longest_ranking(gpu_device, kind):
    """The longest vector one call takes (2^21 tokens: 256 tiles of 8192, 1024 buckets): exact.  One more token is refused."""
    import torch
    T = 1 << 21
    c = asl.Asl(T + 1, 1, 32)
    rng = np.random.default_rng(T)
    s = np.exp(2 * rng.standard_normal(T)).astype(np.float32)
    if kind == "third-zero":
        s[rng.random(T) < 1 / 3] = 0.0
    _rank_case(c, gpu_device, s)
    with pytest.raises(asl.AslError) as e:
        c.asl_rank(torch.zeros(T + 1, device=gpu_device), T + 1, torch.zeros(T + 1, dtype=torch.int32, device=gpu_device))
    assert e.value.status == asl.ASL_EUNSUPPORTED
    c.close()


# ----------------------------------------------------------------------------- statistic
def _stat_case(ctx, dev, R: np.ndarray, l_obs: int, k: int, tau: float, layer_idx: int,
               init_var=None):
    """Place the rows of R (oldest first) in the ring as the library expects and run asl_rankvar."""
    torch = _torch()
    n, T = R.shape
    ring = np.full((l_obs, T), 10**9, dtype=np.int32)                 # poison unused rows
    for j in range(n):
        layer = layer_idx - (n - 1) + j
        ring[layer % l_obs] = R[j]
    ringd = torch.from_numpy(ring).to(dev)
    state = asl.new_state(dev)
    asl.write_state(state, init_var=init_var or 0.0, init_set=int(init_var is not None),
                    n_valid_rows=n, last_layer=layer_idx)
    out = asl.new_stat(dev)
    ctx.asl_rankvar(ringd, l_obs, T, layer_idx, 0, k, tau, state, out)
    return asl.read_struct(out, asl.AslStat), asl.read_struct(state, asl.AslState)


@pytest.mark.parametrize("n,l_obs,T,k", [(2, 8, 100, 10), (8, 8, 5000, 300), (5, 8, 32736, 992),
                                         (8, 8, 131040, 2016), (3, 3, 1000, 1000), (8, 8, 262080, 4032),
                                         # more rows than one load batch holds; rings that wrap part-way
                                         (12, 12, 3001, 200), (9, 16, 70001, 500), (17, 24, 131073, 640),
                                         (64, 64, 2500, 100)])
def test_rankvar_exact(ctx, gpu_device, n, l_obs, T, k):
    rng = np.random.default_rng(n + T)
    base = rng.standard_normal(T)
    R = np.stack([orc.rank_desc(base + 0.5 * rng.standard_normal(T)) for _ in range(n)])
    ref = orc.rank_variance(R, k)
    st, state = _stat_case(ctx, gpu_device, R, l_obs, k, tau=0.3, layer_idx=37)
    assert st.evaluated == 1 and st.n_rows == n
    assert st.numerator == ref.numerator and st.union_size == ref.union_size
    assert st.var_top == ref.var_top                                   # same integer, same single division
    assert st.rel_var == 1.0 and st.selected == 0                      # first evaluation: relative variance 1
    assert state.init_set == 1 and state.init_var == ref.var_top and state.n_valid_rows == n
    # second evaluation against a given init_var: decision and release of the ring
    st2, state2 = _stat_case(ctx, gpu_device, R, l_obs, k, tau=0.3, layer_idx=37, init_var=ref.var_top * 4)
    assert st2.rel_var == ref.var_top / (ref.var_top * 4) and st2.selected == 1
    assert state2.n_valid_rows == 0 and state2.init_var == ref.var_top * 4


def test_rankvar_guards_and_degenerate(ctx, gpu_device):
    torch = _torch()
    T = 300
    R = np.stack([np.arange(T), np.arange(T)])
    st, state = _stat_case(ctx, gpu_device, R[:1], 8, 10, 0.3, layer_idx=12)          # one row only
    assert st.evaluated == 0 and st.selected == 0 and state.init_set == 0
    st, state = _stat_case(ctx, gpu_device, R, 8, 10, 0.3, layer_idx=12)              # identical rows
    assert st.evaluated == 1 and st.var_top == 0.0 and np.isnan(st.rel_var) and st.selected == 0
    assert state.init_set == 1 and state.init_var == 0.0
    st, _ = _stat_case(ctx, gpu_device, np.stack([np.arange(T), np.arange(T)[::-1]]), 8, 10, 0.3,
                       layer_idx=13, init_var=0.0)
    assert np.isinf(st.rel_var) and st.selected == 0
    # layer below L_min: nothing evaluated, state untouched
    ring = torch.zeros((8, T), dtype=torch.int32, device=gpu_device)
    state = asl.new_state(gpu_device)
    asl.write_state(state, n_valid_rows=5, last_layer=4)
    out = asl.new_stat(gpu_device)
    ctx.asl_rankvar(ring, 8, T, 4, 10, 10, 0.3, state, out)
    assert asl.read_struct(out, asl.AslStat).evaluated == 0
    assert asl.read_struct(state, asl.AslState).n_valid_rows == 5


# ----------------------------------------------------------------------------- select
def _select_case(ctx, dev, scores: np.ndarray, budget: int, W: int):
    torch = _torch()
    rows, T = scores.shape
    N = T + W
    p = asl.make_params(rows, rows, 64, N, W, 7, budget)
    k = min(budget, N) - W
    sd = torch.from_numpy(scores).to(dev)
    out = torch.full((rows, k + W), -7, dtype=torch.int32, device=dev)
    ctx.asl_select_topk(p, sd, rows, out)
    ref = orc.select_indices(scores.astype(np.float64), k, W)
    np.testing.assert_array_equal(out.cpu().numpy().astype(np.int64), ref)


@pytest.mark.parametrize("rows,T,budget,W", [(1, 10, 6, 2), (2, 496, 128, 16), (8, 32736, 2048, 32),
                                             (8, 131040, 2048, 32), (1, 131040, 2048, 32),
                                             (8, 262080, 4096, 64), (3, 4097, 5000, 8), (2, 9000, 33, 32)])
def test_select_random_with_ties(ctx, gpu_device, rows, T, budget, W):
    rng = np.random.default_rng(T + rows)
    s = rng.random((rows, T), dtype=np.float32)
    if T > 100:
        s = np.round(s, 3).astype(np.float32)           # many exact ties around the threshold
    _select_case(ctx, gpu_device, s, budget, W)


def test_rank_select_pool_random_shapes(ctx, gpu_device):
    """Fifty-six seeded random cases: sizes, budgets, window widths, tie densities and value ranges drawn at
    random (positive-only scores, mixed signs, a few distinct values, tiny magnitudes); forty with rows that are
    ranked and selected from in one launch, sixteen with longer ones."""
    rng = np.random.default_rng(20260127)
    for case in range(56):
        T = int(rng.integers(1, 9000)) if case < 40 else int(rng.integers(12289, 60000))
        rows = int(rng.integers(1, 4))
        W = int(rng.integers(1, 40))
        budget = W + int(rng.integers(1, T + 20))
        kind = case % 4
        if kind == 0:
            s = rng.random((rows, T)).astype(np.float32)                          # positive, few ties
        elif kind == 1:
            s = np.round(rng.standard_normal((rows, T)), 1).astype(np.float32)     # mixed signs, heavy ties
        elif kind == 2:
            s = rng.integers(0, 3, (rows, T)).astype(np.float32)                   # three distinct values
        else:
            s = (rng.random((rows, T)) * 1e-30).astype(np.float32)                 # tiny magnitudes / denormals
        print(f"case {case}: T={T} rows={rows} W={W} budget={budget} kind={kind}", flush=True)
        _rank_case(ctx, gpu_device, s[0])
        _select_case(ctx, gpu_device, s, budget, W)


@pytest.mark.parametrize("rows,T,budget", [(96, 100000, 1056), (96, 100001, 1056), (300, 9000, 532),
                                           (128, 131040, 2080), (130, 100001, 1056), (256, 20000, 8192),
                                           (129, 70000, 35000), (128, 5, 4), (140, 4096, 33)])
def test_select_many_rows(gpu_device, rows, T, budget):
    """96 rows x 25 tiles, with rows on 16-byte boundaries and, T = 100001, off them.  300 rows: more than the candidate buffers hold at once,
    so the three launches run twice.  Further: 128 full-size rows, a budget of 8192 on many rows, a
    budget of half the row (the candidates overflow: selection from the whole row), rows of five
    tokens, rows of exactly one tile."""
    W = 32 if T > 100 else 2
    rng = np.random.default_rng(rows + T)
    s = np.round(rng.random((rows, T), dtype=np.float32), 4).astype(np.float32)
    c = asl.Asl(T + W, rows, rows * W)
    try:
        _select_case(c, gpu_device, s, budget, W)
        assert c.asl_device_fault() == 0
    finally:
        c.close()


def test_select_many_hard_rows(gpu_device):
    """Many rows at once whose sampled bound is useless or whose candidates overflow (top tokens
    clustered at either end or inside one tile, a few distinct values, all equal, sorted either way,
    negative scores), several of each kind in one call, beside ordinary rows."""
    rng = np.random.default_rng(77)
    rows, T, W, budget = 144, 70000, 32, 2048
    s = rng.random((rows, T), dtype=np.float32)
    for r in range(rows):
        kind = r % 9
        if kind == 1:
            s[r, :3000] += 10.0
        elif kind == 2:
            s[r, -3000:] += 10.0
        elif kind == 3:
            s[r] = rng.integers(0, 4, T).astype(np.float32)
        elif kind == 4:
            s[r] = 0.25
        elif kind == 5:
            s[r] = np.sort(s[r])[::-1]
        elif kind == 6:
            s[r] = np.sort(s[r])
        elif kind == 7:
            s[r, 16384:20480] = 5.0 + rng.random(4096, dtype=np.float32)
        elif kind == 8:
            s[r] = -s[r] - 1.0
    c = asl.Asl(T + W, rows, rows * W)
    try:
        _select_case(c, gpu_device, np.ascontiguousarray(s), budget, W)
        _select_case(c, gpu_device, np.ascontiguousarray(s), W + 1, W)             # k = 1
        _select_case(c, gpu_device, np.ascontiguousarray(s[:, :3000]), 4000, W)    # budget >= N: keep all
        assert c.asl_device_fault() == 0
    finally:
        c.close()


@pytest.mark.parametrize("rows", [3, 130])
def test_select_around_zero(gpu_device, rows):
    """Scores drawn from a few values on both sides of zero (+0, -0, denormals of either sign, small
    and large magnitudes), so that for one budget or another the threshold falls on each of them:
    -0 and +0 tie (lower index first), denormals do not count as zero, negative scores order by
    magnitude downwards (the filter decides on the scores' bits: every sign and zero case matters)."""
    rng = np.random.default_rng(rows)
    T, W = 20000, 16
    vals = np.array([0.0, -0.0, 1e-40, -1e-40, 1e-45, -1e-45, 1.0, -1.0, 3e38, -3e38, 1e-20, -1e-20], dtype=np.float32)
    s = vals[rng.integers(0, len(vals), (rows, T))]
    assert np.signbit(s).any() and (s == 0).any()
    c = asl.Asl(T + W, rows, rows * W)
    try:
        for k in (1, 900, 1700, 2500, 3400, 5000, 8400, 10000, 12000, 15000, 19999):
            _select_case(c, gpu_device, s, k + W, W)
        assert c.asl_device_fault() == 0
    finally:
        c.close()


# as many tiles as take one and two a workgroup, and one more of each; the last workgroup's second tile missing, one token long, full
@pytest.mark.parametrize("rows,T", [(8, 32 * 4096), (8, 32 * 4096 + 1), (8, 64 * 4096), (8, 64 * 4096 + 1), (1, 16385), (64, 4 * 4096 + 1),
                                    (64, 8 * 4096 + 1), (256, 32769), (51, 9 * 4096 + 1)])
def test_select_rows_whose_filter_takes_the_bound(gpu_device, rows, T):
    rng = np.random.default_rng(rows + T)
    s = np.exp(2 * rng.standard_normal((rows, T), dtype=np.float32))
    s[::4, ::3] = s[0, 5]                                 # a third of the row ties
    s[1::4] = np.sort(s[1::4])
    c = asl.Asl(T + 8, rows, rows * 8)
    for budget in (9, 2048, T // 3):
        _select_case(c, gpu_device, s, budget, 8)
    c.close()


# candidates beyond what the finishing workgroup holds: a bound tightened by bins, by bins that hold a run of equal scores (too long
# for any bound, then the whole row), rows beside which others fit, a tile's last candidates off a round of 256
@pytest.mark.parametrize("rows,T,k", [(16, 131040, 8160), (9, 200001, 8160), (5, 262080, 8128), (3, 300007, 12000), (2, 90001, 16384)])
def test_select_more_candidates_than_fit(gpu_device, rows, T, k):
    W = 16
    rng = np.random.default_rng(T + k)
    s = np.exp(2 * rng.standard_normal((rows, T + 6)))
    s = np.stack([np.convolve(r, np.full(7, 1 / 7), "valid") for r in s]).astype(np.float32)
    s[1] = np.round(s[1], 1)                              # ties around the threshold
    s[-1, ::3] = s[-1].max()                              # a third of the row
    if rows > 3:
        s[2, T // 2:] = np.sort(s[2, T // 2:])
        s[3, ::40] = np.quantile(s[3], 1 - k / T).astype(np.float32)   # a run of the threshold's own value
    c = asl.Asl(T + W, rows, rows * W)
    _select_case(c, gpu_device, s, k + W, W)
    c.close()


def test_select_special(ctx, gpu_device):
    T, W = 6000, 16
    _select_case(ctx, gpu_device, np.ones((2, T), dtype=np.float32), 100, W)               # all equal: first k
    _select_case(ctx, gpu_device, np.zeros((1, T), dtype=np.float32), 100, W)
    s = np.random.default_rng(5).standard_normal((2, T)).astype(np.float32)                 # negatives
    _select_case(ctx, gpu_device, s, 1000, W)
    _select_case(ctx, gpu_device, s, T + W + 50, W)                                         # budget >= N: keep all


@pytest.mark.parametrize("kind", ["clustered-front", "clustered-back", "few-values", "half-kept", "all-equal-large",
                                  "sorted-desc", "sorted-asc", "one-outlier-tile"])
def test_select_when_the_sampled_bound_does_not_help(ctx, gpu_device, kind):
    """Inputs on which the top-k's sampled bound is useless or its candidate buffers overflow, so the
    finishing kernel selects from the whole row: every top token inside one 4096-token tile (the tile's
    2048-slot segment overflows), a handful of distinct values (tens of thousands of keys tie with the
    bound), half the row kept (the candidates exceed what one workgroup holds), monotone rows."""
    rng = np.random.default_rng(len(kind) * 31 + ord(kind[0]))
    T, W = 70000, 32
    budget = 2048
    s = rng.random((3, T), dtype=np.float32)
    if kind == "clustered-front":
        s[:, :3000] += 10.0
    elif kind == "clustered-back":
        s[:, -3000:] += 10.0
    elif kind == "few-values":
        s = rng.integers(0, 4, (3, T)).astype(np.float32)
    elif kind == "half-kept":
        budget = T // 2
    elif kind == "all-equal-large":
        s[:] = 0.25
    elif kind == "sorted-desc":
        s = np.sort(s, axis=1)[:, ::-1].copy()
    elif kind == "sorted-asc":
        s = np.sort(s, axis=1)
    elif kind == "one-outlier-tile":
        s[1, 8192:12288] = 5.0 + rng.random(4096, dtype=np.float32)      # exactly one tile holds the whole top-k
    _select_case(ctx, gpu_device, np.ascontiguousarray(s), budget, W)


# ----------------------------------------------------------------------------- gather
@pytest.mark.parametrize("cfg", [1, 2])
def test_gather_bit_exact(ctx, gpu_device, cfg):
    torch = _torch()
    L = synth.config_layer(cfg)
    sh = L.shape
    p = gu.params_of(sh)
    kd, vd = gu.to_dev(L.k, sh.dtype, gpu_device), gu.to_dev(L.v, sh.dtype, gpu_device)
    rng = np.random.default_rng(cfg)
    n_idx = sh.k + sh.W
    idx = np.stack([np.sort(rng.choice(sh.N, n_idx, replace=False)) for _ in range(sh.Hk)]).astype(np.int32)
    for idx_rows, I in ((sh.Hk, idx), (1, idx[:1])):
        Id = torch.from_numpy(I).to(gpu_device)
        ko = torch.zeros((sh.Hk, n_idx, sh.d), dtype=kd.dtype, device=gpu_device)
        vo = torch.zeros_like(ko)
        ctx.asl_gather_kv(p, kd, vd, Id, idx_rows, n_idx, ko, vo)
        kr, vr = orc.gather_kv(L.k, L.v, I if idx_rows > 1 else I[0])
        assert np.array_equal(ko.float().cpu().numpy(), kr)            # bf16/f32 values are exact in fp32
        assert np.array_equal(vo.float().cpu().numpy(), vr)
    # identity index = plain copy; strided K (token stride 2d) reads the right rows
    Id = torch.arange(sh.N, dtype=torch.int32, device=gpu_device)
    ko = torch.zeros_like(kd)
    ctx.asl_gather_kv(p, kd, None, Id, 1, sh.N, ko, None)
    assert torch.equal(ko, kd)
    wide = torch.zeros((sh.Hk, sh.N, 2 * sh.d), dtype=kd.dtype, device=gpu_device)
    wide[:, :, :sh.d] = kd
    p2 = asl.make_params(sh.Hq, sh.Hk, sh.d, sh.N, sh.W, sh.S, sh.budget, dtype=p.dtype,
                         k_strides=(sh.N * 2 * sh.d, 2 * sh.d))
    ko.zero_()
    ctx.asl_gather_kv(p2, wide, None, Id, 1, sh.N, ko, None)
    assert torch.equal(ko, kd)


def test_gather_empty_and_f32(ctx, gpu_device):
    torch = _torch()
    sh = synth.shape_of(1)                                   # fp32 storage, d = 64
    L = synth.config_layer(1)
    p = gu.params_of(sh)
    kd, vd = gu.to_dev(L.k, "f32", gpu_device), gu.to_dev(L.v, "f32", gpu_device)
    ko = torch.full((sh.Hk, 4, sh.d), 7.0, device=gpu_device)
    vo = torch.full_like(ko, 7.0)
    I = torch.tensor([[3, 0, 511, 3]], dtype=torch.int32, device=gpu_device)     # repeats allowed
    ctx.asl_gather_kv(p, kd, vd, I, 1, 0, ko, vo)                                  # n_idx = 0: nothing written
    assert torch.all(ko == 7.0) and torch.all(vo == 7.0)
    ctx.asl_gather_kv(p, kd, vd, I, 1, 4, ko, vo)
    assert np.array_equal(ko.cpu().numpy(), L.k[:, [3, 0, 511, 3], :])
    assert np.array_equal(vo.cpu().numpy(), L.v[:, [3, 0, 511, 3], :])


@pytest.mark.parametrize("row_bytes,n_idx", [(8192, 6400), (8192, 6399), (192, 273067), (16, 3276801)])
def test_gather_of_more_than_the_caches_hold(gpu_device, row_bytes, n_idx):
    """100 MiB read and written is where the copies become non-temporal: at it, one row below, and past it with
    rows that are no power of two of pieces and of a single piece."""
    torch = _torch()
    c = asl.Asl(64, 1, 1)
    n_src = 5000
    src = torch.randint(-2**31, 2**31 - 1, (n_src, row_bytes // 4), dtype=torch.int32, device=gpu_device)
    idx = torch.randint(0, n_src, (n_idx,), dtype=torch.int32, device=gpu_device)
    out = torch.zeros((n_idx, row_bytes // 4), dtype=torch.int32, device=gpu_device)
    c.asl_gather_rows(src, row_bytes, row_bytes, idx, n_idx, out)
    assert torch.equal(out, src[idx.long()])
    c.close()


# ----------------------------------------------------------------------------- errors
def test_argument_errors(ctx, gpu_device):
    torch = _torch()
    sh = synth.shape_of(1)
    good = gu.params_of(sh)
    t = torch.zeros(16, device=gpu_device)

    def expect(status, fn):
        with pytest.raises(asl.AslError) as e:
            fn()
        assert e.value.status == status, str(e.value)

    def with_(**kw):
        p = gu.params_of(sh)
        for a, b in kw.items():
            setattr(p, a, b)
        return p

    sc = lambda p: ctx.asl_score_layer(p, t, t, t, t)
    expect(asl.ASL_EINVAL, lambda: sc(with_(n_q_heads=3)))               # Hq % Hk
    expect(asl.ASL_EINVAL, lambda: sc(with_(window=0)))
    expect(asl.ASL_EINVAL, lambda: sc(with_(window=sh.N)))               # W < N
    expect(asl.ASL_EINVAL, lambda: sc(with_(pool_kernel=4)))             # even S
    expect(asl.ASL_EINVAL, lambda: sc(with_(budget=sh.W)))               # k <= 0
    expect(asl.ASL_EUNSUPPORTED, lambda: sc(with_(dtype=5)))
    expect(asl.ASL_EINVAL, lambda: sc(with_(flags=64)))                  # unknown flag bit
    expect(asl.ASL_ENOMEM, lambda: sc(with_(seq_len=1 << 20)))           # beyond the context limits
    expect(asl.ASL_EINVAL, lambda: ctx.asl_score_layer(good, None, t, t, t))
    expect(asl.ASL_EINVAL, lambda: ctx.asl_rank(t, 0, t))
    expect(asl.ASL_EINVAL, lambda: ctx.asl_pool(t, 1, 16, 2, t))
    expect(asl.ASL_EINVAL, lambda: ctx.asl_gather_kv(good, t, None, t, 3, 4, t, None))   # idx_rows not 1/Hk
    expect(asl.ASL_EINVAL, lambda: ctx.asl_rankvar(t, 1, 16, 0, 0, 4, 0.3, t, t))        # L_obs < 2
    expect(asl.ASL_EUNSUPPORTED, lambda: ctx.asl_rankvar(t, 64, 2_000_000, 0, 0, 4, 0.3, t, t))
    # a shape beside the main ones (d = 96) beyond the size those are taken up to
    big = asl.Asl(1 << 20, 1, 64 * 128)
    pb = asl.make_params(64, 1, 96, 1 << 20, 128, 7, 4096)
    expect(asl.ASL_EUNSUPPORTED, lambda: big.asl_score_layer(pb, t, t, t, t))
    expect(asl.ASL_EUNSUPPORTED, lambda: big.asl_window_lse(pb, t, t, t))
    big.close()
    # ranking more tokens than one launch can hold
    expect(asl.ASL_ENOMEM, lambda: ctx.asl_rank(t, 1 << 22, t))
    h = C.c_void_p()
    assert ctx.lib.asl_create(C.byref(h), 0, 1, 8, 8) == asl.ASL_EINVAL
    assert ctx.lib.asl_create(C.byref(h), 99, 1024, 8, 8) == asl.ASL_EHIP


def test_stat_written_straight_to_pinned_host_memory(ctx, gpu_device):
    """The decision record may live in page-locked host memory: the statistic kernel writes it there
    and the host reads it after a stream synchronisation, with no copy of its own."""
    import torch
    T, l_obs, k = 5000, 4, 300
    rng = np.random.default_rng(5)
    ring = torch.zeros((l_obs, T), dtype=torch.int32, device=gpu_device)
    state = asl.new_state(gpu_device)
    stat_dev = asl.new_stat(gpu_device)
    stat_host = torch.zeros(stat_dev.numel(), dtype=torch.uint8).pin_memory()
    p = asl.make_params(4, 2, 64, T + 8, 8, 7, k + 8)
    for layer in range(l_obs + 2):
        s = torch.from_numpy(rng.standard_normal(T).astype(np.float32)).to(gpu_device)
        st2 = state.clone()
        ctx.asl_rank_stat(p, s, layer, 0, l_obs, 0.0, ring.clone(), st2, stat_dev)
        ctx.asl_rank_stat(p, s, layer, 0, l_obs, 0.0, ring, state, stat_host)
        torch.cuda.synchronize()
        assert bytes(stat_host.numpy().tobytes()) == bytes(stat_dev.cpu().numpy().tobytes())
    assert asl.AslStat.from_buffer_copy(bytes(stat_host.numpy().tobytes())).evaluated == 1
