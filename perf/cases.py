"""The work a program has libasl do during prefill, as cases that can be timed and compared.

A case is one public call as a prefill loop makes it: a whole layer (asl_layer_step), or one of its
parts where a program uses that part on its own (scoring, ranking + statistic, top-k over many rows,
compaction of many layers' caches, propagation of hidden states).  Inputs are drawn on the GPU:

* queries and keys whose window logits follow a per-token latent importance of standard deviation 2
  (attention scores of real prompts span several nats) plus noise, with a few dominant first tokens;
* earlier rank rows that are the orders of correlated latents, as neighbouring layers' are;
* score rows that are pooled lognormals.

Whole numbers (ranks, indices) are compared as such.  Where the scores themselves are computed by the
call, two tokens whose scores are within rounding of each other may swap ranks.
"""
import math

import torch
import torch.nn.functional as F

from paper_2601_07667_amd import asl

LATENT_STD = 2.0
NOISE = 0.5
N_SINKS = 4              # first tokens of a prompt that draw attention whatever the query
HIDDEN = 4096            # hidden size of the 8B shape (token propagation)


def _step(name, Hq, Hk, d, N, W, S, budget, dtype="bf16", L_obs=8, lse=False, evaluated=True):
    return {"name": name, "kind": "step", "Hq": Hq, "Hk": Hk, "d": d, "N": N, "W": W, "S": S, "budget": budget,
            "dtype": dtype, "L_obs": L_obs, "lse": lse, "evaluated": evaluated}


def _score(name, Hq, Hk, d, N, W, S, dtype="bf16", lse=False):
    return {"name": name, "kind": "score", "Hq": Hq, "Hk": Hk, "d": d, "N": N, "W": W, "S": S, "dtype": dtype, "lse": lse}


def listed():
    return [
        # the smallest problem of the repository (tiny fp32 configuration): launches and latency
        _step("step_tiny_f32", 4, 2, 64, 512, 16, 7, 128, dtype="f32", L_obs=3),
        # odd sizes everywhere, d = 64, a layer below L_min (a third of a model's layers are)
        _step("step_ragged_10k", 6, 2, 64, 10007, 13, 5, 777, evaluated=False),
        # ordinary layer: 8B shape, 32K context
        _step("step_8b_32k", 32, 8, 128, 32768, 32, 7, 2048),
        # the headline: 8B shape, 128K context
        _step("step_8b_128k", 32, 8, 128, 131072, 32, 7, 2048),
        # the same when the layer's attention kernel hands over the window rows' log-sum-exp
        _step("step_8b_128k_lse", 32, 8, 128, 131072, 32, 7, 2048, lse=True),
        # second model geometry (seven query heads per KV head) at the large budget
        _step("step_28h_128k_b8192", 28, 4, 128, 131072, 32, 7, 8192),
        # the longest context: 256K, window 64
        _step("step_8b_256k_w64", 32, 8, 128, 262144, 64, 7, 4096),
        # a head size beside 64 and 128, an ordinary prompt
        _score("score_d256_8k", 8, 4, 256, 8192, 32, 7),
        # ranking + statistic of a million-token context's scores
        {"name": "rank_stat_1m", "kind": "rank_stat", "T": 1048544, "k": 2016, "L_obs": 8},
        # top-k of the per-head scores of 32 layers at once
        {"name": "select_256x128k", "kind": "select", "rows": 256, "T": 131040, "W": 32, "budget": 2048},
        # compaction of every layer's cache in one call, 32 layers
        {"name": "gather_32layers_32k", "kind": "gather", "layers": 32, "Hk": 8, "d": 128, "N": 32768, "n_idx": 2048},
        # token propagation: hidden states of the selected tokens
        {"name": "propagate_128k", "kind": "rows", "N": 131072, "n_idx": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["step", "score", "rank_stat", "select", "gather", "rows"], [8, 4, 2, 3, 1, 1])[0]
    if kind == "step":
        if rng.random() < 0.1:
            Hq, Hk = rng.choice([(4, 2), (4, 4), (3, 1)])
            c = _step("", Hq, Hk, 64, _log_int(rng, 300, 4096), rng.choice([8, 13, 16]), 7, _log_int(rng, 64, 512),
                      dtype="f32", L_obs=3, evaluated=rng.random() < 0.7)
        else:
            Hq, Hk, d = rng.choice([(32, 8, 128), (32, 8, 128), (28, 4, 128), (6, 2, 64), (4, 2, 64), (8, 1, 128),
                                    (3, 3, 128), (14, 2, 128)])
            W = rng.choice([8, 13, 16, 32, 32, 48, 64])
            c = _step("", Hq, Hk, d, _log_int(rng, 512, 262144), W, rng.choice([1, 3, 5, 7, 7, 7, 15, 31]),
                      W + _log_int(rng, 32, 8192), lse=rng.random() < 0.25, evaluated=rng.random() < 0.7)
    elif kind == "score":
        if rng.random() < 0.5:              # shapes beside bf16 with d in {64, 128} and G*W <= 512
            Hq, Hk, d, dtype = rng.choice([(8, 4, 256, "bf16"), (4, 2, 96, "bf16"), (8, 2, 80, "f32"), (4, 2, 64, "f32"),
                                           (8, 8, 128, "f32"), (16, 1, 128, "bf16")])
            W = 48 if Hk == 1 else rng.choice([8, 13, 16, 32])
            N = _log_int(rng, 256, min(16384, 8 * 32 * 256 * 8192 // (Hq * W * d)))
        else:
            Hq, Hk, d, dtype = rng.choice([(32, 8, 128, "bf16"), (28, 4, 128, "bf16"), (4, 2, 64, "bf16"), (7, 1, 128, "bf16")])
            W = rng.choice([5, 16, 32, 33, 64])
            N = _log_int(rng, 512, 262144)
        c = _score("", Hq, Hk, d, N, W, rng.choice([1, 7, 7, 31]), dtype=dtype, lse=rng.random() < 0.3)
    elif kind == "rank_stat":
        T = _log_int(rng, 500, 1048544)
        c = {"kind": kind, "T": T, "k": max(1, min(T // 2, _log_int(rng, 64, 8192))), "L_obs": rng.choice([3, 5, 8, 8])}
    elif kind == "select":
        rows = rng.choice([1, 4, 8, 9, 32, 64, 130, 256])
        W = rng.choice([13, 32, 64])
        c = {"kind": kind, "rows": rows, "T": _log_int(rng, 2000, min(262080, 256 * 131040 // rows)), "W": W,
             "budget": W + _log_int(rng, 64, 8192)}
    elif kind == "gather":
        layers = rng.choice([1, 5, 16, 32])
        c = {"kind": kind, "layers": layers, "Hk": rng.choice([4, 8]), "d": rng.choice([64, 96, 128]),
             "N": _log_int(rng, 4096, 32768), "n_idx": _log_int(rng, 128, 2048)}
    else:
        N = _log_int(rng, 2000, 131072)
        c = {"kind": kind, "N": N, "n_idx": min(N, _log_int(rng, 128, 8192))}
    c.pop("name", None)
    return c


# ------------------------------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _randn(g, *shape, dtype=torch.float32):
    return torch.randn(*shape, generator=g, device="cuda", dtype=dtype)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _window_inputs(case, g):
    """q_obs [Hq, W, d], k [Hk, N, d] and the latent importance [T] behind them."""
    Hq, Hk, d, N, W = (case[x] for x in ("Hq", "Hk", "d", "N", "W"))
    T, a = N - W, d ** 0.25
    z = LATENT_STD * _randn(g, T)
    z[:N_SINKS] = 3 * LATENT_STD
    zf = torch.zeros(N, device="cuda")
    zf[:T] = z
    u = F.normalize(_randn(g, Hk, d), dim=1)
    q = (NOISE * _randn(g, Hq, W, d) + a * u.repeat_interleave(Hq // Hk, 0)[:, None, :]).to(_dtype(case))
    k = torch.empty(Hk, N, d, dtype=_dtype(case), device="cuda")
    for h in range(Hk):
        k[h] = NOISE * _randn(g, N, d) + a * zf[:, None] * u[h]
    return q.contiguous(), k, z


def _ranks(s):
    """RankDesc: the place of every token in the order (score descending, index ascending)."""
    order = torch.sort(s, descending=True, stable=True).indices
    r = torch.empty_like(order)
    r[order] = torch.arange(s.numel(), device=s.device)
    return r


def _ring(g, z, L_obs, layer):
    """A ring that holds the ranks of the L_obs - 1 layers before `layer`, as correlated orders."""
    ring = torch.zeros(L_obs, z.numel(), dtype=torch.int32, device="cuda")
    for l in range(layer - L_obs + 1, layer):
        ring[l % L_obs] = _ranks(0.8 * z + 0.6 * LATENT_STD * _randn(g, z.numel())).to(torch.int32)
    return ring


def _new_state(T, L_obs, layer):
    st = asl.new_state("cuda:0")
    asl.write_state(st, init_var=_init_var(T), init_set=1, n_valid_rows=L_obs - 1, last_layer=layer - 1)
    return st


def _init_var(T):
    return float(T) * float(T) / 16.0


def _first_layer(L_obs):
    return 2 * L_obs - 1


def _log_sum_exp(case, q, k):
    """[Hq, W] natural log-sum-exp of the window rows' masked, scaled logits, in 64 bits."""
    return torch.cat([torch.logsumexp(l, -1) for l in _logits(case, q, k)]).reshape(case["Hq"], case["W"])


def _logits(case, q, k):
    """Per KV head [G * W, N]: scaled logits with the causal mask on the last W x W block, in 64 bits."""
    Hq, Hk, d, N, W = (case[x] for x in ("Hq", "Hk", "d", "N", "W"))
    G, T = Hq // Hk, N - W
    hidden = torch.ones(W, W, dtype=torch.bool, device="cuda").triu(1).repeat(G, 1)
    for h in range(Hk):
        l = q[h * G:(h + 1) * G].reshape(G * W, d).double() @ k[h].double().T
        l /= math.sqrt(d)
        l[:, T:].masked_fill_(hidden, -math.inf)
        yield l


def _score_rows(g, rows, T):
    """Pooled lognormal scores, a row at a time."""
    out = torch.empty(rows, T, device="cuda")
    for r in range(rows):
        x = torch.exp(LATENT_STD * _randn(g, T)) / T
        out[r] = F.avg_pool1d(x[None, None], 7, 1, 3)[0, 0]
    return out


def _pick(g, n, N):
    return torch.sort(torch.randperm(N, generator=g, device="cuda")[:n]).values.to(torch.int32)


def _params(case, budget):
    return asl.make_params(case["Hq"], case["Hk"], case["d"], case["N"], case["W"], case["S"], budget,
                           dtype=asl.ASL_BF16 if case["dtype"] == "bf16" else asl.ASL_F32)


def prepare(case, seed):
    g = _gen(seed)
    f32, i32 = torch.float32, torch.int32
    kind = case["kind"]
    st = {"kind": kind}
    if kind in ("step", "score"):
        Hq, Hk, d, N, W = (case[x] for x in ("Hq", "Hk", "d", "N", "W"))
        T = N - W
        st["q"], st["k"], z = _window_inputs(case, g)
        st["lse"] = _log_sum_exp(case, st["q"], st["k"]).float() if case["lse"] else None
        if kind == "score":
            st["ctx"] = asl.Asl(N, Hk, Hq * W)
            st["p"] = _params(case, W + 1)
            st["P"] = torch.empty(Hk, T, dtype=f32, device="cuda")
            st["s"] = torch.empty(T, dtype=f32, device="cuda")
            return st
        n = min(case["budget"], N)
        st["ctx"] = asl.Asl(N, Hk + 1, Hq * W)
        st["p"] = _params(case, case["budget"])
        st["v"] = _randn(g, Hk, N, d, dtype=_dtype(case))
        st["L_obs"], st["layer"] = case["L_obs"], _first_layer(case["L_obs"])
        st["l_min"] = 0 if case["evaluated"] else 1 << 30
        st["ring"] = _ring(g, z, case["L_obs"], st["layer"])
        st["state"], st["stat"] = _new_state(T, case["L_obs"], st["layer"]), asl.new_stat("cuda:0")
        st["scores"] = torch.empty(Hk + 1, T, dtype=f32, device="cuda")
        st["idx"] = torch.empty(Hk + 1, n, dtype=i32, device="cuda")
        st["k_out"] = torch.empty(Hk, n, d, dtype=_dtype(case), device="cuda")
        st["v_out"] = torch.empty(Hk, n, d, dtype=_dtype(case), device="cuda")
    elif kind == "rank_stat":
        T, L_obs, W = case["T"], case["L_obs"], 32
        st["ctx"] = asl.Asl(T + W, 1, W)
        st["p"] = asl.make_params(1, 1, 64, T + W, W, 7, W + case["k"])
        z = LATENT_STD * _randn(g, T)
        st["s"] = F.avg_pool1d(torch.exp(z)[None, None], 7, 1, 3)[0, 0].contiguous() / T
        st["L_obs"], st["layer"], st["l_min"] = L_obs, _first_layer(L_obs), 0
        st["ring"] = _ring(g, torch.log(st["s"]), L_obs, st["layer"])
        st["state"], st["stat"] = _new_state(T, L_obs, st["layer"]), asl.new_stat("cuda:0")
    elif kind == "select":
        T, W, rows = case["T"], case["W"], case["rows"]
        st["ctx"], st["rows"] = asl.Asl(T + W, rows, W), rows
        st["p"] = asl.make_params(1, 1, 64, T + W, W, 7, case["budget"])
        st["scores"] = _score_rows(g, rows, T)
        st["idx"] = torch.empty(rows, min(case["budget"], T + W), dtype=i32, device="cuda")
    elif kind == "gather":
        Hk, d, N, n, layers = (case[x] for x in ("Hk", "d", "N", "n_idx", "layers"))
        st["ctx"], st["n_idx"], st["layers"], st["Hk"] = asl.Asl(N, Hk, Hk), n, layers, Hk
        st["p"] = asl.make_params(Hk, Hk, d, N, 1, 7, 2)
        st["ks"] = [_randn(g, Hk, N, d, dtype=torch.bfloat16) for _ in range(layers)]    # each its own cache
        st["vs"] = [_randn(g, Hk, N, d, dtype=torch.bfloat16) for _ in range(layers)]
        st["idx"] = torch.stack([_pick(g, n, N) for _ in range(layers * Hk)]).reshape(layers, Hk, n).contiguous()
        st["k_out"] = torch.empty(layers, Hk, n, d, dtype=torch.bfloat16, device="cuda")
        st["v_out"] = torch.empty_like(st["k_out"])
        st["ptrs"] = [torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device="cuda")
                      for ts in (st["ks"], st["vs"], list(st["k_out"]), list(st["v_out"]))]
    else:
        N, n = case["N"], case["n_idx"]
        st["ctx"], st["n_idx"] = asl.Asl(N, 1, 1), n
        st["hidden"] = _randn(g, N, HIDDEN, dtype=torch.bfloat16)
        st["idx"] = _pick(g, n, N)
        st["out"] = torch.empty(n, HIDDEN, dtype=torch.bfloat16, device="cuda")
    return st


# -------------------------------------------------------------------------------------------- the call
def run(st):
    kind, ctx = st["kind"], st["ctx"]
    if kind == "step":
        # tau = 0 never selects, so the ring stays full however often the layer loop goes on
        ctx.asl_layer_step(st["p"], st["q"], st["k"], st["v"], st["layer"], st["l_min"], st["L_obs"], 0.0, st["scores"],
                           st["ring"], st["state"], st["stat"], st["idx"], st["k_out"], st["v_out"], lse=st["lse"])
        st["layer"] += 1
        # the statistic's integer numerator is var_top * n_rows^2 * union_size: it follows var_top's rounding
        return {"scores": st["scores"], "ring": st["ring"], "idx": st["idx"], "k": st["k_out"], "v": st["v_out"],
                "var": st["stat"][:16].view(torch.float64), "counts": st["stat"][24:].view(torch.int32),
                "state": st["state"][8:].view(torch.int32)}
    if kind == "score":
        ctx.asl_score_layer(st["p"], st["q"], st["k"], st["P"], st["s"], lse=st["lse"])
        return {"P": st["P"], "s": st["s"]}
    if kind == "rank_stat":
        ctx.asl_rank_stat(st["p"], st["s"], st["layer"], st["l_min"], st["L_obs"], 0.0, st["ring"], st["state"], st["stat"])
        st["layer"] += 1
        return {"ring": st["ring"], "var": st["stat"][:16].view(torch.float64), "numerator": st["stat"][16:24].view(torch.int64),
                "counts": st["stat"][24:].view(torch.int32), "state": st["state"][8:].view(torch.int32)}
    if kind == "select":
        ctx.asl_select_topk(st["p"], st["scores"], st["rows"], st["idx"])
        return {"idx": st["idx"]}
    if kind == "gather":
        kp, vp, ko, vo = st["ptrs"]
        ctx.asl_gather_kv_layers(st["p"], kp, vp, st["idx"], st["Hk"], st["n_idx"], st["layers"], ko, vo)
        return {"k": st["k_out"], "v": st["v_out"]}
    ctx.asl_gather_rows(st["hidden"], HIDDEN * 2, HIDDEN * 2, st["idx"], st["n_idx"], st["out"])
    return {"out": st["out"]}


# -------------------------------------------------------------------------------------------- its measure
def work(case):
    kind = case["kind"]
    flops = 0
    if kind in ("step", "score"):
        Hq, Hk, d, N, W = (case[x] for x in ("Hq", "Hk", "d", "N", "W"))
        T, eb = N - W, 2 if case["dtype"] == "bf16" else 4
        flops = 2 * Hq * W * N * d
        b = (Hq * W + Hk * N) * d * eb + (Hq * W * 4 if case["lse"] else 0) + (Hk + 1) * T * 4
        if kind == "step":
            n = min(case["budget"], N)
            b += T * 4 + ((case["L_obs"] - 1) * T * 4 if case["evaluated"] else 0)     # the new rank row, the others
            b += (Hk + 1) * n * 4 + 2 * 2 * Hk * n * d * eb
    elif kind == "rank_stat":
        b = case["T"] * 4 * (1 + case["L_obs"])
    elif kind == "select":
        b = case["rows"] * (case["T"] + min(case["budget"], case["T"] + case["W"])) * 4
    elif kind == "gather":
        b = case["layers"] * case["Hk"] * case["n_idx"] * (4 + 2 * 2 * case["d"] * 2)
    else:
        b = case["n_idx"] * (4 + 2 * HIDDEN * 2)
    return {"bytes": b, "flops": flops}


def tolerance(case):
    if case["kind"] == "step":
        # fp32 sums and exponentials: the scores are 1e-7 to 3.2e-7 off their 64-bit values; tokens that
        # close swap ranks (a few per thousand at 256K tokens)
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.01}
    if case["kind"] == "score":
        return {"rel": 2e-6, "max": 2e-5}
    return "exact"


def _exact_scores(case, q, k):
    Hk, N, W, S = (case[x] for x in ("Hk", "N", "W", "S"))
    u = torch.stack([torch.softmax(l, -1)[:, :N - W].sum(0) for l in _logits(case, q, k)])
    P = F.avg_pool1d(u[:, None], S, 1, S // 2)[:, 0]
    return P, P.sum(0)


def _exact_var(ring, layer, L_obs, k, T):
    r = ring.long()
    kept = r.amin(0) < k
    r = r[:, kept]
    num = (L_obs * (r * r).sum(0) - r.sum(0) ** 2).sum()
    var = num.double() / (L_obs * L_obs * int(kept.sum()))
    return torch.stack([var, var / _init_var(T)])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "score"):
        g = _gen(seed)
        q, k, z = _window_inputs(case, g)
        P, s = _exact_scores(case, q, k)
        if kind == "score":
            return {"P": P, "s": s}
        N, W, Hk, L_obs = (case[x] for x in ("N", "W", "Hk", "L_obs"))
        T, n = N - W, min(case["budget"], N)
        v = _randn(g, Hk, N, case["d"], dtype=_dtype(case))
        layer = _first_layer(L_obs)
        ring = _ring(g, z, L_obs, layer)
        ring[layer % L_obs] = _ranks(s).to(torch.int32)
        window = torch.arange(T, N, device="cuda")
        idx = [torch.cat([torch.sort(torch.sort(P[h], descending=True, stable=True).indices[:n - W]).values, window])
               for h in range(Hk)]
        return {"scores": torch.cat([P, s[None]]), "ring": None, "idx": None,
                "k": torch.stack([k[h][idx[h]] for h in range(Hk)]), "v": torch.stack([v[h][idx[h]] for h in range(Hk)]),
                "var": _exact_var(ring, layer, L_obs, n - W, T) if case["evaluated"] else None, "counts": None, "state": None}
    if kind == "rank_stat":
        st = prepare(case, seed)
        ring, layer = st["ring"], st["layer"]
        ring[layer % case["L_obs"]] = _ranks(st["s"]).to(torch.int32)
        return {"ring": None, "var": _exact_var(ring, layer, case["L_obs"], case["k"], case["T"]), "numerator": None,
                "counts": None, "state": None}
    if kind == "gather":
        st = prepare(case, seed)
        take = lambda ts: torch.stack([torch.stack([t[h][st["idx"][l, h].long()] for h in range(case["Hk"])])
                                       for l, t in enumerate(ts)])
        return {"k": take(st["ks"]), "v": take(st["vs"])}
    if kind == "rows":
        st = prepare(case, seed)
        return {"out": st["hidden"][st["idx"].long()]}
    return None              # whole numbers only
