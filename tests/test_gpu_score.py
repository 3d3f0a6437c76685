"""GPU parity of asl_score_layer (Alg. 1 steps 5-8) against the float64 oracle on the same seeded
inputs: |gpu - oracle| <= 1e-5 + 2e-3 |oracle| element by element (bf16 in, fp32 accumulate)."""
import numpy as np
import pytest

import gpu_util as gu
from oracle import asl_oracle as orc
from paper_2601_07667_amd import asl, synth

pytestmark = pytest.mark.gpu


def _run_score(dev, L, flags=0, lse=None, scale=0.0):
    import torch
    sh = L.shape
    ctx = gu.ctx_for(sh)
    p = gu.params_of(sh, flags=flags, scale=scale)
    qd, kd = gu.to_dev(L.q_obs, sh.dtype, dev), gu.to_dev(L.k, sh.dtype, dev)
    P = torch.full((sh.Hk, sh.T), float("nan"), dtype=torch.float32, device=dev)
    s = torch.full((sh.T,), float("nan"), dtype=torch.float32, device=dev)
    lsed = None if lse is None else torch.from_numpy(lse.astype(np.float32)).to(dev)
    ctx.asl_score_layer(p, qd, kd, P, s, lse=lsed)
    out = P.cpu().numpy(), s.cpu().numpy()
    ctx.close()
    return out


def _small(Hq, Hk, d, N, W, S=7, dtype="bf16", seed=0):
    sh = synth.Shape(Hq=Hq, Hk=Hk, d=d, N=N, W=W, S=S, budget=W + 8, dtype=dtype)
    return synth.iid_layer(sh, seed, name=f"small-{Hq}-{Hk}-{d}-{N}-{W}-{dtype}")


def _compare(dev, L, flags=0, use_lse=False, scale=0.0):
    sh = L.shape
    sc = scale if scale > 0 else None
    P_ref, s_ref = orc.score_layer(L.q_obs, L.k, sh.W, sh.S, sc)
    lse = orc.row_lse(L.q_obs, L.k, sh.W, sc) if use_lse else None
    P, s = _run_score(dev, L, flags=flags, lse=lse, scale=scale)
    gu.assert_scores_close(P, P_ref, f"{L.name} P")
    gu.assert_scores_close(s, s_ref, f"{L.name} s")
    return P, s


def test_config1_f32_and_bf16(gpu_device):
    L = synth.config_layer(1)                                   # fp32 storage: fp32 MFMA kernels
    P, s = _compare(gpu_device, L)
    Pg, sg = _compare(gpu_device, L, flags=asl.ASL_FLAG_GENERIC_SCORE)      # on-GPU cross-check: plain-FMA kernels
    np.testing.assert_allclose(P, Pg, rtol=1e-4, atol=1e-7)
    sh = synth.shape_of(1)
    sh.dtype = "bf16"                                           # bf16-rounded copy: MFMA kernels, d = 64
    Lb = synth.iid_layer(sh, synth.BASE_SEED + 1, name="C1-bf16")
    P, s = _compare(gpu_device, Lb)
    Pg, sg = _compare(gpu_device, Lb, flags=asl.ASL_FLAG_GENERIC_SCORE)     # on-GPU cross-check
    np.testing.assert_allclose(P, Pg, rtol=1e-4, atol=1e-7)


# several tiles and a ragged tail; row counts that do not fill a 32-row block; d = 64 and 128;
# M = 224 (seven heads per group) and M = 256 (W = 64)
@pytest.mark.parametrize("Hq,Hk,d,N,W", [
    (4, 2, 128, 1000, 16), (3, 1, 64, 333, 5), (8, 2, 128, 4096 + 77, 32), (7, 1, 128, 2500, 32),
    (4, 1, 128, 3000, 64), (2, 2, 64, 130, 1), (4, 4, 128, 129, 128), (8, 8, 128, 40, 33)])
def test_small_shapes(gpu_device, Hq, Hk, d, N, W):
    L = _small(Hq, Hk, d, N, W, seed=N)
    _compare(gpu_device, L)


@pytest.mark.parametrize("N", [64 * 5 + 16, 64 * 5 + 15, 64 * 5 + 17, 64 * 6 + 32, 64 * 40 + 1])
def test_key_counts_around_tile_edges(gpu_device, N):
    """N - W one below / at / one above a multiple of the 64-key tile; several chunks per head."""
    _compare(gpu_device, _small(4, 2, 128, N, 16, seed=N))
    _compare(gpu_device, _small(4, 2, 128, N, 16, seed=N + 1), use_lse=True)


@pytest.mark.parametrize("d,dtype", [(96, "bf16"), (256, "bf16"), (80, "f32")])
def test_other_head_dims(gpu_device, d, dtype):
    """Head dimensions outside {64, 128}: the MFMA kernels for padded and other row lengths, and the plain-FMA kernels."""
    L = _small(4, 2, d, 700, 8, dtype=dtype, seed=d)
    for use_lse in (False, True):
        P, s = _compare(gpu_device, L, use_lse=use_lse)
        Pg, sg = _compare(gpu_device, L, flags=asl.ASL_FLAG_GENERIC_SCORE, use_lse=use_lse)
        np.testing.assert_allclose(P, Pg, rtol=1e-4, atol=1e-7)


def _close_to_64_bits(P, s, L):
    """Tighter than the score tolerance: a logit's error is a few 2^-24 of the sum of its |products| (below
    20 in base 2 for these inputs), so a probability is within 2e-5 of itself however the sums are ordered."""
    P_ref, s_ref = orc.score_layer(L.q_obs, L.k, L.shape.W, L.shape.S)
    np.testing.assert_allclose(P, P_ref, rtol=2e-5, atol=1e-12)
    np.testing.assert_allclose(s, s_ref, rtol=2e-5, atol=1e-12)


# Row lengths around the built ones (128, 256, 384, 512, 768 and 1024 bytes): shorter by one 16-byte
# piece, full, longer by one; row lengths with no whole pieces (bf16 d = 20, fp32 d = 30) and beyond 256
# elements stay with the plain kernels.  Key counts at and around the 32- and 64-key tiles.
@pytest.mark.parametrize("dtype,d", [("bf16", d) for d in (8, 56, 72, 80, 96, 120, 136, 192, 200, 248, 256, 264, 20)] +
                         [("f32", d) for d in (4, 28, 32, 36, 64, 68, 96, 100, 128, 132, 192, 196, 256, 260, 30)])
def test_row_lengths(gpu_device, dtype, d):
    for i, (Hq, Hk, W, N) in enumerate([(4, 2, 16, 512), (3, 1, 13, 97 + d), (5, 1, 64, 32 * 9 + 64), (2, 2, 1, 2)]):
        L = _small(Hq, Hk, d, N, W, dtype=dtype, seed=d + i)
        print(f"{dtype} d={d} {L.name}", flush=True)
        P, s = _run_score(gpu_device, L)
        _close_to_64_bits(P, s, L)
        _compare(gpu_device, L, use_lse=True)


def test_heads_that_share_their_keys(gpu_device):
    """A head stride of 0: 8 KV heads read one set of keys (84 MB if it were eight)."""
    import torch
    L = _small(8, 8, 128, 43000, 16, seed=43)
    L.k[:] = L.k[:1]
    sh = L.shape
    lse = orc.row_lse(L.q_obs, L.k, sh.W)
    p = asl.make_params(sh.Hq, sh.Hk, sh.d, sh.N, sh.W, sh.S, sh.budget, k_strides=(0, sh.d))
    q, k = gu.to_dev(L.q_obs, "bf16", gpu_device), gu.to_dev(L.k[:1], "bf16", gpu_device)
    for given in (None, torch.from_numpy(lse.astype(np.float32)).to(gpu_device)):
        ctx = gu.ctx_for(sh)
        P = torch.full((sh.Hk, sh.T), float("nan"), device=gpu_device)
        s = torch.full((sh.T,), float("nan"), device=gpu_device)
        ctx.asl_score_layer(p, q, k, P, s, lse=given)
        _close_to_64_bits(P.cpu().numpy(), s.cpu().numpy(), L)
        ctx.close()


@pytest.mark.parametrize("Hq,Hk,d,W,dtype", [(16, 1, 128, 48, "bf16"), (33, 1, 64, 16, "bf16"), (9, 1, 256, 64, "bf16"),
                                             (10, 2, 128, 64, "f32")])
def test_row_groups(gpu_device, Hq, Hk, d, W, dtype):
    """More query rows per KV head than one launch takes (512 for bf16 with d in {64, 128}, else 128): 768,
    528, 576 and 320 rows, the last group partly filled."""
    L = _small(Hq, Hk, d, 1500 + Hq, W, dtype=dtype, seed=Hq)
    P, s = _run_score(gpu_device, L)
    _close_to_64_bits(P, s, L)
    _compare(gpu_device, L, use_lse=True)


# Rows that end inside the built row lengths and rows that fill them; 16 and 224 query rows, so that blocks of 32
# are partly and wholly filled up; a row group that is (528 rows: 512 + 16).
@pytest.mark.parametrize("Hq,Hk,d,W,dtype", [(4, 2, 80, 8, "f32"), (4, 2, 4, 8, "f32"), (4, 2, 64, 8, "f32"), (4, 2, 132, 8, "f32"),
                                             (4, 2, 96, 8, "bf16"), (4, 2, 248, 8, "bf16"), (4, 2, 256, 8, "bf16"),
                                             (4, 2, 128, 8, "bf16"), (7, 1, 64, 32, "bf16"), (33, 1, 64, 16, "bf16")])
def test_infinite_keys(gpu_device, Hq, Hk, d, W, dtype):
    """A key whose logits are all -Inf has probability 0 and leaves the other keys' scores alone (keys of the first
    and of later tiles, the last past one, and a window key; the infinite element is the row's last)."""
    L = _small(Hq, Hk, d, 700, W, dtype=dtype, seed=d)
    past = [5, 333, 700 - W - 1]
    L.q_obs[:, :, -1] = 1.5
    L.k[:, past + [699], -1] = -np.inf
    L.shape.S = 1
    for use_lse in (False, True):
        P, s = _compare(gpu_device, L, use_lse=use_lse)
        assert np.isfinite(P).all() and np.isfinite(s).all()
        assert (P[:, past] == 0).all() and (s[past] == 0).all()
        Pg, _ = _compare(gpu_device, L, flags=asl.ASL_FLAG_GENERIC_SCORE, use_lse=use_lse)
        # both kernels within 2e-5 of the 64-bit value (see _close_to_64_bits)
        np.testing.assert_allclose(P, Pg, rtol=4e-5, atol=1e-12)


@pytest.mark.parametrize("Hq,Hk,W,N", [(2, 1, 32, 64 * 96), (2, 1, 32, 64 * 96 + 1), (2, 1, 32, 64 * 192 + 1), (3, 1, 64, 64 * 128 + 1),
                                       (3, 1, 64, 64 * 64), (8, 8, 16, 64 * 65 + 3), (4, 4, 40, 64 * 257),
                                       (8, 8, 16, 64 * 256 + 1), (24, 8, 64, 64 * 119 + 1)])
def test_chunk_counts(gpu_device, Hq, Hk, W, N):
    """Key chunks of one tile and more, several tile counts around multiples of the chunk counts, one and more
    workgroups per compute unit, with weighted and equal shares."""
    L = _small(Hq, Hk, 64, N, W, S=1, seed=N)
    P, s = _run_score(gpu_device, L)
    _close_to_64_bits(P, s, L)


@pytest.mark.parametrize("Hq,Hk,d,W,N,dtype", [(8, 1, 128, 16, 20001, "bf16"), (4, 2, 64, 16, 65600, "bf16"), (7, 1, 128, 64, 20000, "bf16"),
                                                (3, 3, 128, 32, 65537, "bf16"), (14, 2, 128, 32, 65536, "bf16"),
                                                (16, 1, 96, 48, 20000, "bf16"), (4, 2, 64, 32, 20000, "f32")])
def test_partials_combined_by_a_launch_of_their_own(gpu_device, Hq, Hk, d, W, N, dtype):
    """More than 64 chunks per KV head: full, padded and fp32 rows, one and several launches of query rows, chunk counts off
    a multiple of 16."""
    L = _small(Hq, Hk, d, N, W, dtype=dtype, seed=Hq + N)
    P, s = _run_score(gpu_device, L)
    _close_to_64_bits(P, s, L)


# (tiles, chunks per head) on 256 compute units: partials folded in batches of each size and combined by a launch of their
# own, tile counts that leave ragged shares, and the last tile ragged too
@pytest.mark.parametrize("Hq,Hk,d,W,N", [
    (1, 1, 64, 16, 64 * 14), (1, 1, 64, 16, 64 * 48), (6, 2, 64, 32, 64 * 95 + 1),       # 14, 48; 96 tiles in 64
    (8, 8, 64, 32, 64 * 2000 + 1),                                                        # 2001 in 96
    (1, 1, 64, 32, 64 * 600 + 5), (4, 4, 64, 64, 64 * 1100 + 3), (1, 1, 64, 32, 64 * 4096),   # 601 in 256; 1101 in 192; 4096 in 256
    (6, 1, 64, 32, 64 * 300), (6, 1, 64, 32, 64 * 2048 + 1), (48, 8, 64, 32, 64 * 65 + 9)])   # 192 rows: 300 in 64; 2049 in 256; 66 in 32
def test_chunk_counts_of_two_passes(gpu_device, Hq, Hk, d, W, N):
    L = _small(Hq, Hk, d, N, W, S=1, seed=N)
    P, s = _run_score(gpu_device, L)
    _close_to_64_bits(P, s, L)


# the same with the log-sum-exp supplied: one to four workgroups per compute unit, a single tile each and more
@pytest.mark.parametrize("Hq,Hk,d,W,N", [
    (8, 8, 64, 32, 64 * 128), (8, 8, 64, 32, 64 * 512 + 3), (8, 8, 64, 16, 64 * 300), (32, 8, 64, 32, 64 * 128 + 1),
    (8, 8, 128, 16, 64 * 65), (8, 8, 128, 16, 64 * 400 + 1), (32, 8, 128, 32, 64 * 97), (32, 8, 128, 32, 64 * 400),
    (48, 8, 64, 32, 64 * 70), (48, 8, 64, 32, 64 * 333)])
def test_chunk_counts_of_one_pass(gpu_device, Hq, Hk, d, W, N):
    """A supplied log-sum-exp is rounded to fp32: half an ulp of a number below 16 moves a probability by 1e-6."""
    L = _small(Hq, Hk, d, N, W, S=1, seed=N)
    lse = orc.row_lse(L.q_obs, L.k, W)
    assert np.abs(lse).max() < 16
    P, s = _run_score(gpu_device, L, lse=lse)
    _close_to_64_bits(P, s, L)


# keys of 80 MB and, read by both passes, 112 MB are where the loads change their cache policy: a key or two to either side; every
# kind of kernel that has both, and sizes below
@pytest.mark.parametrize("N,use_lse,dtype,d", [(N, l, dtype, d) for N, l in ((49151, False), (49154, False), (32767, True), (32770, True))
                                               for dtype, d in (("bf16", 128), ("f32", 64))] +
                         [(57343, False, "bf16", 128), (57346, False, "bf16", 128), (40959, True, "bf16", 128),
                          (40962, True, "bf16", 128), (57346, False, "f32", 64), (28674, False, "bf16", 256),
                          (54615, True, "bf16", 96), (81922, True, "bf16", 64)])
def test_keys_loaded_past_the_last_level_cache(gpu_device, N, use_lse, dtype, d):
    L = _small(8, 8, d, N, 16, dtype=dtype, seed=N)
    lse = orc.row_lse(L.q_obs, L.k, 16) if use_lse else None
    P, s = _run_score(gpu_device, L, lse=lse)
    _close_to_64_bits(P, s, L)


def test_misaligned_rows_stay_with_the_plain_kernels(gpu_device):
    """fp32 K one element off a 16-byte boundary, and with a token stride of d + 1."""
    import torch
    L = _small(4, 2, 64, 300, 16, dtype="f32", seed=9)
    sh = L.shape
    ctx = gu.ctx_for(sh)
    P = torch.empty((sh.Hk, sh.T), dtype=torch.float32, device=gpu_device)
    s = torch.empty((sh.T,), dtype=torch.float32, device=gpu_device)
    q, k = gu.to_dev(L.q_obs, "f32", gpu_device), gu.to_dev(L.k, "f32", gpu_device)
    for off, st in ((1, sh.d), (0, sh.d + 1), (3, sh.d + 4)):
        buf = torch.zeros(off + sh.Hk * sh.N * st, device=gpu_device)
        kv = buf[off:].view(sh.Hk, sh.N, st)[:, :, :sh.d]
        kv.copy_(k)
        p = asl.make_params(sh.Hq, sh.Hk, sh.d, sh.N, sh.W, sh.S, sh.budget, dtype=asl.ASL_F32, k_strides=(sh.N * st, st))
        ctx.asl_score_layer(p, q, kv, P, s)
        _close_to_64_bits(P.cpu().numpy(), s.cpu().numpy(), L)
    ctx.close()


def test_random_shapes(gpu_device):
    """Sixteen seeded random shapes: group sizes 1-8, windows 1-64 (M = G*W up to 256, so both the
    one-block and the two-block wavefront layouts and every wavefront count occur), d in {64, 128},
    sequence lengths that are not multiples of anything, pooling kernels 1-15."""
    rng = np.random.default_rng(20260128)
    done = 0
    while done < 16:
        G = int(rng.integers(1, 9))
        W = int(rng.integers(1, 65))
        if G * W > 256:
            continue
        Hk = int(rng.integers(1, 4))
        d = int(rng.choice([64, 128]))
        N = W + int(rng.integers(1, 3000))
        S = int(rng.choice([1, 3, 7, 15]))
        print(f"case {done}: Hq={G * Hk} Hk={Hk} d={d} N={N} W={W} S={S} (M={G * W})", flush=True)
        _compare(gpu_device, _small(G * Hk, Hk, d, N, W, S=S, seed=1000 + done), use_lse=bool(done % 2))
        done += 1


def test_lse_supplied_mode_and_scale(gpu_device):
    L = _small(8, 2, 128, 5000, 32, seed=3)
    P1, s1 = _compare(gpu_device, L)
    P2, s2 = _compare(gpu_device, L, use_lse=True)              # single pass over K
    np.testing.assert_allclose(P1, P2, rtol=1e-4, atol=1e-7)
    _compare(gpu_device, L, scale=0.05)
    Lf = _small(4, 2, 64, 700, 16, dtype="f32", seed=4)
    _compare(gpu_device, Lf, use_lse=True)


def test_pool_kernel_one_and_large(gpu_device):
    _compare(gpu_device, _small(4, 2, 128, 900, 16, S=1, seed=5))
    _compare(gpu_device, _small(4, 2, 128, 900, 16, S=31, seed=6))


def test_strided_k(gpu_device):
    """K as a slice of a fused [Hk, N, 2d] buffer (token stride 2d)."""
    import torch
    L = _small(8, 2, 128, 3000, 32, seed=7)
    sh = L.shape
    ctx = gu.ctx_for(sh)
    kd = gu.to_dev(L.k, "bf16", gpu_device)
    wide = torch.zeros((sh.Hk, sh.N, 2 * sh.d), dtype=torch.bfloat16, device=gpu_device)
    wide[:, :, sh.d:] = kd
    p = asl.make_params(sh.Hq, sh.Hk, sh.d, sh.N, sh.W, sh.S, sh.budget,
                        k_strides=(sh.N * 2 * sh.d, 2 * sh.d))
    P = torch.empty((sh.Hk, sh.T), dtype=torch.float32, device=gpu_device)
    s = torch.empty((sh.T,), dtype=torch.float32, device=gpu_device)
    ctx.asl_score_layer(p, gu.to_dev(L.q_obs, "bf16", gpu_device), wide[:, :, sh.d:], P, s)
    P_ref, s_ref = orc.score_layer(L.q_obs, L.k, sh.W, sh.S)
    gu.assert_scores_close(P.cpu().numpy(), P_ref, "strided P")
    gu.assert_scores_close(s.cpu().numpy(), s_ref, "strided s")
    ctx.close()


def test_heavy_tailed_keys(gpu_device):
    """Per-token lognormal key scale: logits of a few hundred, exercises the running maximum."""
    sh = synth.Shape(Hq=8, Hk=2, d=128, N=6000, W=64, S=7, budget=512)
    L = synth.needle_layer(sh, 11, 16, synth.needle_gain_strong(sh), heavy_tail=True, name="heavy")
    _compare(gpu_device, L)


# what each sub-tile of 32 keys adds to its logits, times a constant: small steps up and down, one above the bound that makes the
# reference of the row sums move, one that overflows without it, a first sub-tile far above all others, two waves of them
@pytest.mark.parametrize("Hq,Hk,d,W,dtype", [(8, 2, 128, 16, "bf16"), (6, 1, 128, 32, "bf16"), (4, 2, 64, 16, "f32"), (4, 2, 256, 8, "bf16")])
@pytest.mark.parametrize("levels", [(0, 1, 2, 1), (0, 4, 8, 12, 16), (0, 100, 30), (60, 0), (0, 200, 0, 201, 90), (-90, -60, -90)])
def test_logits_on_several_levels(gpu_device, Hq, Hk, d, W, dtype, levels):
    """A tile or two a workgroup of pass 1: first references far apart, and the combination of what the workgroups found (many tiles
    a workgroup: the test below).  The logits are up to 200 here, where their own rounding to fp32 (and of the product with log2 e) moves a probability by up to 200 * 2^-23 * 2: 5e-5."""
    L = _small(Hq, Hk, d, 64 * 40 + 7, W, S=1, dtype=dtype, seed=d + len(levels))
    L.q_obs[:, :, 0] = 1.0
    for i, lo in enumerate(range(0, L.shape.N, 32)):
        L.k[:, lo:lo + 32, 0] = levels[i * len(levels) // ((L.shape.N + 31) // 32)] * np.sqrt(d)
    L.k = synth.round_bf16(L.k) if dtype == "bf16" else L.k.astype(np.float32)
    P_ref, s_ref = orc.score_layer(L.q_obs, L.k, W, 1)
    P, s = _run_score(gpu_device, L)
    np.testing.assert_allclose(P, P_ref, rtol=5e-5, atol=1e-30)
    np.testing.assert_allclose(s, s_ref, rtol=5e-5, atol=1e-30)


# 64 KV heads leave each workgroup of pass 1 a dozen or fewer per head, 24 or more of the 289 tiles each, one after the other through the
# range of keys: levels that stay within what a reference holds; that leave it behind now and then, once by more than fp32 holds without it;
# that rise with every tile, where a wavefront soon keeps a running maximum; that fall.  Three and four wavefronts of 32 rows, three of 64;
# the rows of each query head, which are a wavefront's or half of one's, meet another share of the levels, so that wavefronts of a
# workgroup part.
@pytest.mark.parametrize("G,d", [(3, 128), (4, 128), (3, 64), (4, 64), (5, 128), (5, 64)])
@pytest.mark.parametrize("levels", [(0, 2, 1, 3, 0), (0, 12, 5, 24, 24, 40), (0, 150, 20, 190), tuple(range(0, 168, 6)),
                                    tuple(range(168, 0, -6))], ids=["stay", "move", "overflow", "rise", "fall"])
def test_reference_of_the_sums_over_many_tiles(gpu_device, G, d, levels):
    """The bound is that of test_logits_on_several_levels: logits of up to 200, rounded to fp32."""
    import torch
    Hk, own, W, N = 64, 4, 32, 64 * 288 + 7                    # four KV heads' queries, each 16 times
    rng = np.random.default_rng(G * d + len(levels))
    q = rng.standard_normal((own * G, W, d))
    k = rng.standard_normal((N, d))
    q[:, :, 0] = np.tile(np.resize([1.0, 0.0, 0.5, -0.25, 1.0], G), own)[:, None]
    k[:, 0] = np.asarray(levels)[np.arange(N) * len(levels) // N] * np.sqrt(d)
    q, k = synth.round_bf16(q), synth.round_bf16(k)
    sh = synth.Shape(Hq=Hk * G, Hk=Hk, d=d, N=N, W=W, S=1, budget=W + 8)
    P_ref, _ = orc.score_layer(q, np.broadcast_to(k.astype(np.float64), (own, N, d)), W, 1)
    q, P_ref = np.tile(q, (Hk // own, 1, 1)), np.tile(P_ref, (Hk // own, 1))
    ctx = gu.ctx_for(sh)
    p = asl.make_params(sh.Hq, Hk, d, N, W, 1, sh.budget, k_strides=(0, d))                     # one set of keys for all heads
    P = torch.full((Hk, sh.T), float("nan"), device=gpu_device)
    s = torch.full((sh.T,), float("nan"), device=gpu_device)
    ctx.asl_score_layer(p, gu.to_dev(q, "bf16", gpu_device), gu.to_dev(k, "bf16", gpu_device), P, s)
    np.testing.assert_allclose(P.cpu().numpy(), P_ref, rtol=5e-5, atol=1e-30)
    np.testing.assert_allclose(s.cpu().numpy(), P_ref.sum(axis=0), rtol=5e-5, atol=1e-30)
    ctx.close()


def test_config2_full(gpu_device):
    L = synth.config_layer(2)
    P, s = _compare(gpu_device, L)
    P2, s2 = _run_score(gpu_device, L)                          # determinism: bit-identical rerun
    assert np.array_equal(P, P2) and np.array_equal(s, s2)


def test_config3_full_128k(gpu_device):
    L = synth.config_layer(3)
    _compare(gpu_device, L)
    gu.report_margins(L.name)


def test_config3_lse_supplied_128k(gpu_device):
    """The one-pass mode at the size the benchmark times it: the rows' log-sum-exp comes from the
    oracle (float64, rounded to fp32), K is streamed once."""
    L = synth.config_layer(3)
    L.name += "-lse"
    _compare(gpu_device, L, use_lse=True)
    gu.report_margins(L.name)


def _window_lse(dev, L, flags=0):
    import torch
    sh = L.shape
    ctx = gu.ctx_for(sh)
    p = gu.params_of(sh, flags=flags)
    qd, kd = gu.to_dev(L.q_obs, sh.dtype, dev), gu.to_dev(L.k, sh.dtype, dev)
    lse = torch.full((sh.Hq, sh.W), float("nan"), dtype=torch.float32, device=dev)
    ctx.asl_window_lse(p, qd, kd, lse)
    P0 = torch.empty((sh.Hk, sh.T), dtype=torch.float32, device=dev)
    s0 = torch.empty((sh.T,), dtype=torch.float32, device=dev)
    P1, s1 = torch.empty_like(P0), torch.empty_like(s0)
    ctx.asl_score_layer(p, qd, kd, P0, s0)                       # self-contained: both passes
    ctx.asl_score_layer(p, qd, kd, P1, s1, lse=lse)              # with the library's own log-sum-exp
    torch.cuda.synchronize()
    ctx.close()
    return lse.cpu().numpy().astype(np.float64), (P0, s0), (P1, s1)


# plain-*: the plain-FMA kernels, by the flag and by rows that are no whole 16-byte pieces or longer than 256 elements
@pytest.mark.parametrize("case", ["small-d64", "ragged-rows", "w64", "f32", "heavy-tail", "c2", "plain-f32", "plain-d96",
                                  "plain-rows-d20", "plain-rows-f32-d30", "plain-rows-d264"])
def test_window_lse_matches_oracle_and_hands_back_exactly(gpu_device, case):
    """asl_window_lse against the oracle's log-sum-exp of the masked, scaled logits (fp32 accumulation
    of a sum of N positive terms: 1e-5 absolute + 2e-6 relative on a logarithm), and the hand-off:
    scoring with these values supplied equals the self-contained call up to the rounding of the
    natural-log <-> base-2 conversion of the normaliser (one ulp of a number near 20 in the exponent:
    a few 1e-6 relative on every score)."""
    import torch
    if case == "small-d64":
        L = _small(4, 2, 64, 700, 16, seed=21)
    elif case == "ragged-rows":
        L = _small(7, 1, 128, 2500, 32, seed=22)                 # 224 query rows per KV head
    elif case == "w64":
        L = _small(8, 2, 128, 4096 + 77, 64, seed=23)
    elif case in ("f32", "plain-f32"):
        L = _small(4, 2, 64, 700, 16, dtype="f32", seed=24)
    elif case == "plain-d96":
        L = _small(4, 2, 96, 700, 16, seed=25)
    elif case.startswith("plain-rows"):
        L = _small(4, 2, int(case.split("-d")[1]), 700, 16, dtype="f32" if "f32" in case else "bf16", seed=26)
    elif case == "heavy-tail":
        sh = synth.Shape(Hq=8, Hk=2, d=128, N=6000, W=64, S=7, budget=512)
        L = synth.needle_layer(sh, 11, 16, synth.needle_gain_strong(sh), heavy_tail=True, name="heavy")
    else:
        L = synth.config_layer(2)
    sh = L.shape
    by_flag = case in ("plain-f32", "plain-d96")
    lse, (P0, s0), (P1, s1) = _window_lse(gpu_device, L, flags=asl.ASL_FLAG_GENERIC_SCORE if by_flag else 0)
    ref = orc.row_lse(L.q_obs, L.k, sh.W)
    err = np.abs(lse - ref)
    assert np.all(err <= 1e-5 + 2e-6 * np.abs(ref)), f"{case}: worst lse error {err.max()}"
    for a, b in ((P0, P1), (s0, s1)):
        a, b = a.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(a - b) <= 1e-5 * np.abs(a) + 1e-12), f"{case}: hand-back differs by {np.abs(a / b - 1).max()}"


def test_config5_full_256k(gpu_device):
    L = synth.config_layer(5)
    _compare(gpu_device, L)
    gu.report_margins(L.name)


# The 28-layer model's head geometry (App. B.3: 4 KV heads, 7 query heads per group) at the paper's
# long contexts: 224 query rows per KV head at window 32, 448 at window 64.
@pytest.mark.parametrize("N,W,budget", [(131072, 32, 8192), (262144, 64, 8192)])
def test_second_model_geometry_full_size(gpu_device, N, W, budget):
    sh = synth.Shape(Hq=28, Hk=4, d=128, N=N, W=W, S=7, budget=budget, L_min=9)
    L = synth.needle_layer(sh, 91 + W, 64, synth.needle_gain_strong(sh), name=f"qwen-like-N{N}-W{W}")
    print(f"score {L.name}", flush=True)
    _compare(gpu_device, L)
    gu.report_margins(L.name)


@pytest.mark.parametrize("Hq,Hk,W", [(5, 1, 64), (6, 1, 64), (16, 2, 64), (12, 1, 32), (7, 1, 48)])
def test_row_counts_up_to_512(gpu_device, Hq, Hk, W):
    """G*W = 320, 384, 512, 384, 336 query rows per KV head: five to eight wavefronts of two 32-row
    blocks, with and without padded rows."""
    _compare(gpu_device, _small(Hq, Hk, 128, 3000 + 13 * Hq, W, seed=30 + Hq))
    _compare(gpu_device, _small(Hq, Hk, 64, 1500 + 7 * Hq, W, seed=40 + Hq))


@pytest.mark.parametrize("Hq,Hk,W,N,reps", [(32, 8, 32, 131072, 300), (16, 4, 64, 65536, 200), (8, 4, 32, 40000, 200),
                                            (14, 2, 32, 50000, 200)])
def test_scoring_is_reproducible(gpu_device, Hq, Hk, W, N, reps):
    """The same call on the same inputs gives the same bits every time (all reductions have a fixed
    order), with another key tensor scored in between.  Regression test: a missing wait for the LDS
    writes of pass 2's column partials once made one 32-key sub-tile differ in a few runs per hundred."""
    import torch
    dev = gpu_device
    torch.manual_seed(Hq * 1000 + W)
    ctx = asl.Asl(N, Hk, Hq * W)
    p = asl.make_params(Hq, Hk, 128, N, W, 7, 2048)
    q = torch.randn(Hq, W, 128, device=dev).to(torch.bfloat16)
    k = torch.randn(Hk, N, 128, device=dev).to(torch.bfloat16)
    other = torch.randn(Hk, N, 128, device=dev).to(torch.bfloat16)
    P = torch.empty(Hk, N - W, dtype=torch.float32, device=dev)
    s = torch.empty(N - W, dtype=torch.float32, device=dev)
    ctx.asl_score_layer(p, q, k, P, s)
    P0, s0 = P.clone(), s.clone()
    for i in range(reps):
        if i % 3 == 0:
            ctx.asl_score_layer(p, q, other, P, s)
        P.fill_(-1.0)
        s.fill_(-1.0)
        ctx.asl_score_layer(p, q, k, P, s)
        if not (torch.equal(P, P0) and torch.equal(s, s0)):
            d = torch.nonzero(P != P0)
            raise AssertionError(f"run {i} differs from run 0 at {d.shape[0]} places of P, KV heads "
                                 f"{sorted(set(d[:, 0].tolist()))}, keys {int(d[:, 1].min())}..{int(d[:, 1].max())}")
    ctx.close()
