"""Kernel-level GPU parity: the bf16 MFMA GEMM in its three operand layouts and the flash
attention kernels, each against the fp64 oracle on the same bf16-rounded inputs, at sizes
that span several tiles and end in ragged tails."""
import numpy as np
import pytest
import torch

import synth
from oracle import revffn_oracle as O

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import paper_2512_20920_amd as R
    from paper_2512_20920_amd import harness as Hn
    from helpers import relerr


def _bf(rng, shape, scale=1.0):
    return synth.round_bf16(scale * rng.standard_normal(shape).astype(np.float32))


@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
@pytest.mark.parametrize("M,N,K", [(128, 128, 64), (200, 328, 136), (1, 64, 520), (300, 8, 72), (257, 129 * 8, 24),
                                   # 64 tiles or more: the XCD-aware tile placement, with ragged last tiles and
                                   # rectangles that do not divide the tile grid evenly
                                   (1100, 1304, 72), (2056, 520, 40), (392, 4104, 24),
                                   # 64x64 tiles with fewer k-tiles than stages and more
                                   (600, 1000, 136), (900, 968, 520)])
def test_mfma_gemm_layouts(layout, M, N, K):
    if layout == "tn":
        M = (M + 7) // 8 * 8
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    A, Bm = _bf(rng, (M, K)), _bf(rng, (K, N))
    ref = A @ Bm
    a_trans, b_trans = layout == "tn", layout in ("nn", "tn")
    a_host = A.T.copy() if a_trans else A
    b_host = Bm if b_trans else Bm.T.copy()
    ad, bd = Hn.upload(a_host, "bf16"), Hn.upload(b_host, "bf16")
    for out_f32 in (False, True):
        cd = torch.full((M, N), float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
        R.revffn_op_gemm(1, 2, ad, bd, cd, M, N, K, a_host.shape[1], b_host.shape[1], N, a_trans, b_trans, out_f32)
        torch.cuda.synchronize()
        assert relerr(Hn.download(cd), ref) < (1e-5 if out_f32 else 6e-3), (layout, out_f32)
    # the generic kernel computes the same thing
    cd = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")
    R.revffn_op_gemm(1, 1, ad, bd, cd, M, N, K, a_host.shape[1], b_host.shape[1], N, a_trans, b_trans, False)
    torch.cuda.synchronize()
    assert relerr(Hn.download(cd), ref) < 6e-3


@pytest.mark.parametrize("tile", [1, 2, 3, 4])
@pytest.mark.parametrize("layout", ["nt", "nn", "tn"])
def test_mfma_gemm_every_tile_shape(layout, tile):
    """Every tile shape of the MFMA kernel (forced per launch) on shapes with ragged last tiles in m, n and k,
    including problems smaller than one tile."""
    for (M, N, K) in [(264, 328, 136), (520, 264, 200), (40, 72, 24)]:
        rng = np.random.default_rng(M + 3 * N + 5 * K + tile)
        A, Bm = _bf(rng, (M, K)), _bf(rng, (K, N))
        ref = A @ Bm
        a_trans, b_trans = layout == "tn", layout in ("nn", "tn")
        a_host = A.T.copy() if a_trans else A
        b_host = Bm if b_trans else Bm.T.copy()
        ad, bd = Hn.upload(a_host, "bf16"), Hn.upload(b_host, "bf16")
        for out_f32 in (False, True):
            cd = torch.full((M, N), float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
            R.revffn_op_gemm(1, 2 + 256 * tile, ad, bd, cd, M, N, K, a_host.shape[1], b_host.shape[1], N, a_trans,
                             b_trans, out_f32)
            torch.cuda.synchronize()
            assert relerr(Hn.download(cd), ref) < (1e-5 if out_f32 else 6e-3), (layout, tile, M, N, K, out_f32)


@pytest.mark.parametrize("layout", ["nt", "nn"])
# one row, tails in every dimension around 32 rows and columns and the 64-wide pieces of k, fewer pieces than waves, one
# more than a round of them, and the most tiles the rule sends there
@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (31, 40, 72), (33, 64, 504), (64, 1000, 520), (97, 264, 1096), (384, 1024, 64),
                                   # the most tiles the rule sends there; as many workgroups with several pieces of k per wave
                                   (512, 1024, 256), (200, 1304, 1032)])
def test_few_rows_gemm(layout, M, N, K):
    rng = np.random.default_rng(M + 3 * N + 5 * K)
    A, Bm = _bf(rng, (M, K)), _bf(rng, (K, N))
    b_trans = layout == "nn"
    ad, bd = Hn.upload(A, "bf16"), Hn.upload(Bm if b_trans else Bm.T.copy(), "bf16")
    for out_f32 in (False, True):
        cd = torch.full((M + 1, N), float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device="cuda")
        R.revffn_op_gemm(1, 2, ad, bd, cd, M, N, K, K, bd.shape[1], N, 0, b_trans, out_f32)
        torch.cuda.synchronize()
        # 24-bit sums of at most 1096 products; 2 ** -9 for a result rounded to bfloat16
        assert relerr(Hn.download(cd[:M]), A @ Bm) < (1e-5 if out_f32 else 6e-3)
        assert torch.isnan(cd[M]).all()                       # nothing past the last row


def _attention_case(B, S, H, dh, causal, mode, dtype, offset=0, rise=0.0):
    rng = np.random.default_rng(S * 31 + H + (7 if causal else 0))
    rnd = (lambda s, sc=1.0: _bf(rng, s, sc)) if dtype == 1 else \
          (lambda s, sc=1.0: (sc * rng.standard_normal(s)).astype(np.float32).astype(np.float64))
    d = H * dh
    q, k, v, do = rnd((B * S, d), 1.5), rnd((B * S, d), 1.5), rnd((B * S, d)), rnd((B * S, d))
    if rise:              # scores that rise by `rise` powers of two from one tile of 64 keys to the next, half way, then fall
        u = rng.choice((-1.0, 1.0), d)
        ramp = rise / 64 * np.log(2.0) / np.sqrt(dh) * np.minimum(np.arange(S), S - np.arange(S))
        q, k = (synth.round_bf16(a.astype(np.float32)) for a in (q + u, k + np.tile(ramp, B)[:, None] * u))
    r4 = lambda a: a.reshape(B, S, H, dh)
    if S > 2048:          # long sequences: one S x S matrix in flight instead of a stored probability tensor
        o_ref, _ = O.attention_core(r4(q), r4(k), r4(v), causal, keep_probs=False)
        dq_ref, dk_ref, dv_ref = O.attention_core_backward_streaming(r4(do), r4(q), r4(k), r4(v), causal)
    else:
        o_ref, P = O.attention_core(r4(q), r4(k), r4(v), causal)
        dq_ref, dk_ref, dv_ref = O.attention_core_backward(r4(do), r4(q), r4(k), r4(v), P)
    sname = "bf16" if dtype == 1 else "f32"
    def put(a):                  # a tensor that starts `offset` elements into its allocation
        t = Hn.upload(a, sname)
        return torch.cat([t.new_zeros(offset), t.flatten()])[offset:].view(t.shape)
    qd, kd, vd, dod = (put(a) for a in (q, k, v, do))
    od = torch.full_like(qd, float("nan"))
    lse = torch.full((B, H, S), float("nan"), dtype=torch.float32, device="cuda")
    R.revffn_op_attention_fwd(dtype, mode, qd, kd, vd, od, lse, B, S, H, dh, causal)
    torch.cuda.synchronize()
    tol = 2e-2 if dtype == 1 else 1e-4
    assert relerr(Hn.download(od), o_ref.reshape(B * S, d)) < tol
    sc = np.einsum("bshd,bthd->bhst", r4(q), r4(k)) / np.sqrt(dh)
    if causal:
        sc = np.where(np.tril(np.ones((S, S), dtype=bool)), sc, -np.inf)
    lse_ref = np.log(np.exp(sc - sc.max(-1, keepdims=True)).sum(-1)) + sc.max(-1)
    assert np.abs(Hn.download(lse) - lse_ref).max() < (2e-2 if dtype == 1 else 1e-4)
    dvec = torch.empty((B, H, S), dtype=torch.float32, device="cuda")
    dqd, dkd, dvd = (torch.full_like(qd, float("nan")) for _ in range(3))
    R.revffn_op_attention_bwd(dtype, mode, qd, kd, vd, od, dod, lse, dvec, dqd, dkd, dvd, B, S, H, dh, causal)
    torch.cuda.synchronize()
    assert relerr(Hn.download(dvd), dv_ref.reshape(B * S, d)) < tol
    assert relerr(Hn.download(dqd), dq_ref.reshape(B * S, d)) < tol
    assert relerr(Hn.download(dkd), dk_ref.reshape(B * S, d)) < tol


@pytest.mark.parametrize("causal", [True, False])
# (one query, one past a tile of 32, fewer tiles of keys than the four waves that share them and more, several batches; the last:
# 128 queries per workgroup)
@pytest.mark.parametrize("B,S,H", [(1, 128, 1), (2, 200, 3), (1, 64, 2), (1, 1, 1), (1, 451, 2), (3, 33, 5), (1, 161, 17), (5, 97, 2), (6, 400, 17),
                                   # 128 queries per workgroup for sequences that end inside their first tile: one row, one past
                                   # a tile of 32, one past a tile of 64 keys, a whole one, one short of 128
                                   (1100, 1, 16), (64, 33, 16), (40, 65, 17), (35, 64, 8), (17, 127, 8),
                                   # both sides of the line for many heads
                                   (1, 128, 168), (1, 128, 176), (1, 64, 192), (1, 64, 200)])
def test_flash_attention(B, S, H, causal):
    _attention_case(B, S, H, 128, causal, 2, 1)


@pytest.mark.parametrize("causal", [True, False])
def test_flash_attention_long_sequence(causal):
    """One head at the long-context sequence length (S = 8192): forward, dQ, dK and dV element by element."""
    _attention_case(1, 8192, 1, 128, causal, 2, 1)


def test_flash_attention_ragged_long_sequence():
    _attention_case(1, 2500, 2, 128, True, 2, 1)


# 128 queries per workgroup: one and two groups of waves (eight and more tiles), an odd and an even number of key tiles, the last of
# 1, 63 and 64 keys; scores that rise slowly and fast, so that the running maximum goes up in every tile, then in none.  (1 x 1216, 17
# heads, takes 32 queries per workgroup; three such sequences, below, 128.)
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,H,rise", [(1, 2049, 2, 3.0), (1, 2111, 1, 11.0), (1, 1216, 17, 0.0), (3, 705, 16, 3.0), (3, 448, 16, 11.0)])
def test_flash_attention_key_tiles(B, S, H, rise, causal):
    _attention_case(B, S, H, 128, causal, 2, 1, rise=rise)


# Two groups of waves, group 1 on the odd tiles: 33 key tiles (it ends first) of which the last has 64 keys, 34 with a last one of 1 and
# of 64 keys; maxima that differ between the groups where their results meet.  And one group, 19 tiles, the last full.
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,H,rise", [(1, 2112, 2, 3.0), (1, 2113, 2, 11.0), (1, 2176, 2, 3.0), (3, 1216, 17, 0.0)])
def test_flash_attention_two_groups_key_tiles(B, S, H, rise, causal):
    _attention_case(B, S, H, 128, causal, 2, 1, rise=rise)


# 128 queries per workgroup and no more key tiles than are on their way before the loop: one, two of which the second has 1, 36 and
# 64 keys, and three
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S", [64, 65, 100, 128, 129])
def test_flash_attention_first_key_tiles(S, causal):
    _attention_case(17, S, 16, 128, causal, 2, 1, rise=3.0)


@pytest.mark.parametrize("dtype,dh", [(0, 16), (1, 32), (0, 80)])
def test_generic_attention(dtype, dh):
    _attention_case(2, 70, 3, dh, True, 1, dtype)
    _attention_case(1, 33, 2, dh, False, 1, dtype)


# what neither matrix-core form takes: other head widths, up to several columns per thread, and rows that are not aligned to
# four elements
@pytest.mark.parametrize("dtype,dh,offset", [(1, 80, 0), (0, 6, 0), (1, 300, 0)] + [(t, w, 1) for t in (0, 1) for w in (16, 32, 64, 128)])
def test_vector_attention(dtype, dh, offset):
    _attention_case(2, 70, 3, dh, True, 1, dtype, offset)
    _attention_case(1, 261, 1, dh, False, 1, dtype, offset)


# 128 queries per workgroup, more workgroups than CUs and no more than two for each: the second part of the grid runs in
# reverse (16 and 24 heads: a whole and a broken row of heads where it starts; 100 heads: three tiles each); 48 heads of 2 x 451
# tokens: 32 queries per workgroup both ways; 16 and 24 heads: two groups of waves forward
@pytest.mark.parametrize("B,S,H", [(2, 451, 48), (1, 300, 100), (1, 2200, 16), (1, 2100, 24)])
def test_flash_attention_paired_tiles(B, S, H):
    _attention_case(B, S, H, 128, True, 2, 1)


# more heads than 256 workgroups take, against the same heads a quarter at a time.  The first three take 32 queries per workgroup
# both ways; in the others (128 per workgroup) dK/dV works on 32 queries at a time for all heads and on 64 for a quarter of them (one
# workgroup per CU), in the same order
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,S,H", [(2, 451, 48), (1, 129, 160), (8, 33, 40), (1, 2100, 20), (9, 127, 48), (5, 300, 40)])
def test_flash_attention_gradients_do_not_depend_on_the_grid(B, S, H, causal):
    rng = np.random.default_rng(S + H)
    q, k, v, do = (Hn.upload(_bf(rng, (B * S, H * 128)), "bf16") for _ in range(4))

    def run(h0, h1):
        cut = lambda a: a[:, h0 * 128:h1 * 128].contiguous()
        qh, kh, vh, doh = cut(q), cut(k), cut(v), cut(do)
        o, dq, dk, dv = (torch.full_like(qh, float("nan")) for _ in range(4))
        lse, dvec = (torch.empty((B, h1 - h0, S), dtype=torch.float32, device="cuda") for _ in range(2))
        R.revffn_op_attention_fwd(1, 2, qh, kh, vh, o, lse, B, S, h1 - h0, 128, causal)
        R.revffn_op_attention_bwd(1, 2, qh, kh, vh, o, doh, lse, dvec, dq, dk, dv, B, S, h1 - h0, 128, causal)
        torch.cuda.synchronize()
        return o, dq, dk, dv

    whole, n = run(0, H), H // 4
    for i in range(4):
        for a, b in zip(whole, run(i * n, i * n + n)):
            assert torch.isfinite(b).all() and torch.equal(a[:, i * n * 128:(i + 1) * n * 128], b)


# The same where fewer heads than 16 decide for 32 queries per workgroup: what a quarter of the heads takes all of them take too
@pytest.mark.parametrize("B,S,H", [(1, 1400, 12), (1, 1600, 12), (2, 1024, 8)])
def test_flash_attention_some_heads_have_the_bits_of_all(B, S, H):
    test_flash_attention_gradients_do_not_depend_on_the_grid(B, S, H, True)


# 32 queries per workgroup for heads between 8 and 16, and for few heads of many sequences
@pytest.mark.parametrize("B,S,H", [(1, 1400, 9), (1, 1800, 11), (2, 1100, 7), (5, 1024, 3)])
def test_flash_attention_few_heads(B, S, H):
    _attention_case(B, S, H, 128, True, 2, 1)


@pytest.mark.parametrize("dtype", [0, 1])
# every head width; one row, a tail of one past a tile of 32, more tiles than the four waves of a workgroup
@pytest.mark.parametrize("dh,B,S,H", [(16, 2, 33, 2), (32, 1, 1, 1), (64, 3, 131, 2), (64, 1, 300, 1), (128, 2, 97, 1)])
def test_float32_matrix_attention(dtype, dh, B, S, H):
    _attention_case(B, S, H, dh, True, 1, dtype)
    _attention_case(B, S, H, dh, False, 1, dtype)


# more sequences than half of what a grid's third dimension takes (65536): the batch alone is what counts along it
@pytest.mark.parametrize("dtype", [0, 1])
def test_float32_matrix_attention_of_many_sequences(dtype):
    _attention_case(33000, 1, 1, 16, True, 1, dtype)


# (dtype, head width, mode, granularity): the float32 matrix kernels and the vector kernel keep a token that is not finite from
# every token that does not see it; the bf16 kernels, which multiply whole tiles by zero probabilities, only from those outside
# its block of 64
@pytest.mark.parametrize("dtype,dh,mode,block", [(0, 16, 1, 1), (0, 32, 1, 1), (0, 64, 1, 1), (0, 128, 1, 1), (1, 16, 1, 1), (1, 32, 1, 1),
                                                 (1, 64, 1, 1), (1, 128, 1, 1), (0, 80, 1, 1), (1, 80, 1, 1), (1, 128, 2, 64)])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
# the middle of a tile, the last row of a ragged one, and the first row of one
@pytest.mark.parametrize("t", [77, 130, 96])
def test_attention_keeps_non_finite_tokens_apart(dtype, dh, mode, block, bad, t):
    B, S, H = 1, 131, 2
    rng = np.random.default_rng(dh + t)
    up = lambda a: Hn.upload(a, "bf16" if dtype == 1 else "f32")
    base = {n: _bf(rng, (B * S, H * dh), sc) for n, sc in (("q", 0.5), ("k", 0.5), ("v", 1.0), ("do", 1.0))}

    def run(causal, **poison):
        x = {n: a.copy() for n, a in base.items()}
        for n, cells in poison.items():
            for row, value in cells:
                x[n][row, 3] = value
        q, k, v, do = (up(x[n]) for n in ("q", "k", "v", "do"))
        o, dq, dk, dv = (torch.zeros_like(q) for _ in range(4))
        lse, dvec = (torch.zeros((B, H, S), dtype=torch.float32, device="cuda") for _ in range(2))
        R.revffn_op_attention_fwd(dtype, mode, q, k, v, o, lse, B, S, H, dh, causal)
        R.revffn_op_attention_bwd(dtype, mode, q, k, v, o, do, lse, dvec, dq, dk, dv, B, S, H, dh, causal)
        torch.cuda.synchronize()
        return [a.float().cpu().numpy() for a in (o, dq, dk, dv)]

    o0, dq0, dk0, dv0 = run(True)
    lo, hi = t // block * block, t // block * block + block
    for n in ("k", "v"):                                   # a key (value): queries before it do not see it
        o, dq, _, _ = run(True, **{n: [(t, bad)]})
        assert np.array_equal(o[:lo], o0[:lo]) and np.array_equal(dq[:lo], dq0[:lo]), n
    for n in ("q", "do"):                                  # a query: nothing but the keys up to it
        o, dq, dk, dv = run(True, **{n: [(t, bad)]})
        rest = np.arange(S) != t
        assert np.array_equal(o[rest], o0[rest]) and np.array_equal(dq[rest], dq0[rest]), n
        assert np.array_equal(dk[hi:], dk0[hi:]) and np.array_equal(dv[hi:], dv0[hi:]), n
    # the values: a probability is positive, so a column of V with one infinity sums to it, with two opposite ones to no
    # number, and the other columns keep their bits
    cols = np.arange(H * dh) != 3
    same = lambda a, b: np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(a[~np.isnan(a)], b[~np.isnan(b)])
    o, _, _, _ = run(True, v=[(t, bad)])
    assert np.array_equal(o[:, cols], o0[:, cols]) and same(o[t:, 3], np.full(S - t, bad, np.float32))
    o, _, _, _ = run(True, v=[(40, bad), (t, -bad)])
    first = 40 // block * block
    assert np.array_equal(o[:first], o0[:first]) and np.isnan(o[t:, 3]).all()
    if block == 1:
        assert same(o[40:t, 3], np.full(t - 40, bad, np.float32))
    _, _, _, dv = run(True, do=[(t, bad)])
    assert np.array_equal(dv[:, cols], dv0[:, cols]) and same(dv[:t + 1, 3], np.full(t + 1, bad, np.float32))
    o1, _, _, _ = run(False)
    o, _, _, dv = run(False, v=[(t, bad)], do=[(t, bad)])   # (every query sees every key, and the last row is read for the tail)
    assert np.array_equal(o[:, cols], o1[:, cols]) and same(o[:, 3], np.full(S, bad, np.float32))
    assert same(dv[:, 3], np.full(S, bad, np.float32))
