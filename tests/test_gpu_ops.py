"""Parity of the dense contractions (linear layers, attention) with the oracle's
plain definitions, through the C ABI (speca_linear, speca_attention).

Tolerance: inputs are bf16-representable on both sides, products are exact in fp32,
sums differ by fp32 rounding (<= K * 2^-24 relative to the sum of magnitudes), and the
bf16 result is rounded once: the device value must lie within one bf16 step of the
oracle's value rounded to bf16, plus that fp32 noise."""
import numpy as np
import pytest

import branch_tiles
import speca_inputs as si
from oracle import dit as odit, speca_core as core

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _bd():
    from paper_2509_11628_amd import binding as bd
    return bd


def _dev(a, dtype):
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda().to(td).contiguous()


def _check(got, exp, dtype, K):
    got = got.float().cpu().numpy().astype(np.float64)
    scale = np.max(np.abs(exp))
    if dtype == "f32":
        assert np.max(np.abs(got - exp)) <= 1e-5 * scale
    else:
        expb = core.bf16_round(exp)
        tol = np.abs(expb) * 2.0 ** -7 + K * 2.0 ** -22 * scale + 1e-30
        bad = np.abs(got - expb) > tol
        assert not bad.any(), (int(bad.sum()), float(np.max(np.abs(got - expb))))


SHAPES = [  # M, N, K
    (128, 128, 64), (256, 64, 128), (200, 192, 72), (1, 64, 64), (130, 1152, 1152), (515, 256, 4608), (16, 2304, 1152),
    (300, 16, 64),
    # middle and large bf16 tiles with ragged M and N (every tile by name: test_linear_bf16_tiles)
    (1000, 3304, 128), (4000, 1160, 256), (4000, 1160, 320), (4000, 3400, 2048),
    # one and two K-steps on middle tiles and on 256x256, and many
    (4096, 3456, 64), (4000, 1160, 64), (4096, 3456, 128), (4608, 3072, 2048),
    # the MLP GEMMs of configuration 3 at full size
    (4096, 4608, 1152), (4096, 1152, 4608),
]


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("act", [0, 1, 2])
def test_linear(M, N, K, dtype, act):
    # activations: two shapes on small tiles (one with a tail of K), three on middle and large ones, and the fc1 shape of
    # configuration 3 (one round of 256x256 tiles plus a remainder launch)
    if act and (M, N, K) not in ((200, 192, 72), (130, 1152, 1152), (4000, 1160, 256), (4000, 3400, 2048), (4096, 3456, 128),
                                 (4096, 4608, 1152)):
        return
    bd = _bd()
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    a = si._store(rng.standard_normal((M, K)).astype(np.float32), dtype)
    w = si._store((rng.standard_normal((N, K)) * 0.05).astype(np.float32), dtype)
    b = si._store(rng.standard_normal(N).astype(np.float32) * 0.1, dtype)
    out = bd.linear(_dev(a, dtype), _dev(w, dtype), _dev(b, dtype), act)
    exp = odit.linear(a.astype(np.float64), w.astype(np.float64), b.astype(np.float64))
    if act == 1:
        exp = odit.gelu_tanh(exp)
    if act == 2:
        exp = odit.silu(exp)
    _check(out, exp, dtype, K)


def test_linear_row_result_independent_of_m():
    bd = _bd()
    rng = np.random.default_rng(0)
    a = _dev(rng.standard_normal((700, 1152)), "bf16"); w = _dev(rng.standard_normal((1152, 1152)) * 0.03, "bf16")
    full = bd.linear(a, w)
    part = bd.linear(a[300:333].contiguous(), w)
    assert torch.equal(full[300:333], part)         # bitwise: fixed K order, no split-K
    # the same across main loops and tile shapes: 4096 rows take middle or large tiles, 33 rows the small ones
    a = _dev(rng.standard_normal((4096, 1152)), "bf16")
    full = bd.linear(a, w)
    assert torch.equal(full[1000:1033], bd.linear(a[1000:1033].contiguous(), w))
    a = _dev(rng.standard_normal((4096, 2048)), "bf16"); w = _dev(rng.standard_normal((3072, 2048)) * 0.03, "bf16")
    full = bd.linear(a, w)
    assert torch.equal(full[4000:4096], bd.linear(a[4000:4096].contiguous(), w))


@pytest.mark.parametrize("M,N,K", [(1, 4, 4), (15, 20, 12), (17, 516, 260), (33, 1028, 20), (129, 1100, 16), (300, 2052, 100), (2100, 132, 72), (40, 64, 7),
                                   # through LDS: 64x48 (two), 32x64, 32x32, 32x64 (two) and 64x64 (two) tiles, one to nine stages, ragged rows and columns
                                   (4100, 516, 64), (513, 1148, 384), (2047, 1156, 128), (515, 388, 192), (130, 2300, 576), (33, 4612, 320),
                                   (5001, 516, 128), (4999, 516, 192)])
def test_linear_f32_tiles(M, N, K):
    """fp32 layers at the edges of every tile of the fp32 matrix kernel (16 to 64 rows and columns, K in four interleaved
    parts of 16, tails of 4) and a K that only the plain kernel takes; a row's bits do not depend on M or on the tile."""
    bd = _bd()
    rng = np.random.default_rng(M + N + K)
    a, w, b = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32), rng.standard_normal(N).astype(np.float32)
    da, dw, db = _dev(a, "f32"), _dev(w, "f32"), _dev(b, "f32")
    out = bd.linear(da, dw, db)
    _check(out, odit.linear(a.astype(np.float64), w.astype(np.float64), b.astype(np.float64)), "f32", K)
    r = M // 2
    assert torch.equal(bd.linear(da[r:r + 1].contiguous(), dw, db)[0], out[r])


@pytest.mark.parametrize("M,N,K", branch_tiles.STORES)
def test_linear_bf16_tiles(M, N, K):
    """bf16 layers at the edges of the tiles of 32x64 to 256x256 (ragged rows and columns, K tails of 8): sampled rows against
    the oracle, and the same bits for a row computed alone (the smallest tile)."""
    bd = _bd()
    rng = np.random.default_rng(M + N + K)
    a, w, b = si._store(rng.standard_normal((M, K)).astype(np.float32), "bf16"), si._store(rng.standard_normal((N, K)).astype(np.float32), "bf16"), \
        si._store(rng.standard_normal(N).astype(np.float32), "bf16")
    da, dw, db = _dev(a, "bf16"), _dev(w, "bf16"), _dev(b, "bf16")
    out = bd.linear(da, dw, db)
    rows = sorted({0, M // 3, M // 2, M - 1} | {r for t in (32, 64, 96, 128, 192, 256) for r in (t - 1, t, M // t * t - 1, M // t * t) if 0 <= r < M})
    exp = odit.linear(a[rows].astype(np.float64), w.astype(np.float64), b.astype(np.float64))
    _check(out[rows], exp, "bf16", K)
    for r in (0, M - 1):
        assert torch.equal(bd.linear(da[r:r + 1].contiguous(), dw, db)[0], out[r])


@pytest.mark.parametrize("M,N,K,act", branch_tiles.LARGEST)
def test_linear_bf16_largest_tile(M, N, K, act):
    """One round of 256x256 tiles: one to five K-steps (the loop ends with two or three of them), rows and columns that end inside
    a tile, widths that put every other row at 8-byte alignment (N % 8 == 4), every activation; the bits of a row alone (the smallest tile)."""
    bd = _bd()
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    b = (torch.randn((N,), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    pool = torch.full((M * N + 64,), 7.0, dtype=torch.bfloat16, device="cuda")
    out = bd.linear(a, w, b, act, out=pool[:M * N].view(M, N))
    exp = odit.linear(a.float().cpu().numpy().astype(np.float64), w.float().cpu().numpy().astype(np.float64), b.float().cpu().numpy().astype(np.float64))
    _check(out, odit.gelu_tanh(exp) if act == 1 else odit.silu(exp) if act == 2 else exp, "bf16", K)
    for r in (0, 127, 128, 255, M - 1):
        assert torch.equal(bd.linear(a[r:r + 1].contiguous(), w, b, act)[0], out[r]), r
    assert bool((pool[M * N:] == 7.0).all())                   # nothing written past the end


@pytest.mark.parametrize("rows,T,H,hd", [(2, 16, 4, 16), (1, 100, 2, 72), (2, 256, 3, 72), (1, 77, 2, 64), (1, 300, 2, 128), (1, 64, 1, 32),
                                          (1, 256, 2, 128), (3, 200, 2, 64), (1, 257, 2, 72), (1, 33, 1, 128),
                                          (1, 2000, 2, 128), (1, 1111, 1, 72),       # many key tiles, ragged tail
                                          (2, 641, 3, 128), (1, 320, 1, 128)])       # several rows and heads; whole tiles only
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention(rows, T, H, hd, dtype):
    bd = _bd()
    rng = np.random.default_rng(T + hd)
    qkv = si._store(rng.standard_normal((rows, T, 3, H, hd)).astype(np.float32), dtype)
    out = bd.attention(_dev(qkv.reshape(rows, T, 3 * H * hd), dtype), H)
    q, k, v = (qkv[:, :, i].transpose(0, 2, 1, 3).astype(np.float64) for i in range(3))
    exp = odit.attention(q, k, v).transpose(0, 2, 1, 3).reshape(rows, T, H * hd)
    got = out.float().cpu().numpy().astype(np.float64)
    scale = np.max(np.abs(exp))
    # bf16: probabilities and the output are rounded to bf16 on the device (2^-9 relative each)
    assert np.max(np.abs(got - exp)) <= (2e-5 if dtype == "f32" else 1.2e-2) * scale


@pytest.mark.parametrize("T", [257, 288, 320, 384, 449, 1025])      # 1, 32, 0 queries in the last block of 128; keys 1, 32, 0 past a tile of 64
@pytest.mark.parametrize("hd", [64, 72])
def test_attention_tiles_of_narrow_heads(T, hd):
    """bf16 heads of 64 and 72: rows that share no multiple of 128 bytes, waves without queries, the column step past the head."""
    bd = _bd()
    rows, H = 2, 3
    rng = np.random.default_rng(T * hd)
    qkv = si._store(rng.standard_normal((rows, T, 3, H, hd)).astype(np.float32), "bf16")
    dq = _dev(qkv.reshape(rows, T, 3 * H * hd), "bf16")
    got = bd.attention(dq, H)
    q, k, v = (qkv[:, :, i].transpose(0, 2, 1, 3).astype(np.float64) for i in range(3))
    exp = odit.attention(q, k, v).transpose(0, 2, 1, 3).reshape(rows, T, H * hd)
    # probabilities and the output are rounded to bf16 on the device (2^-9 relative each)
    assert np.max(np.abs(got.float().cpu().numpy().astype(np.float64) - exp)) <= 1.2e-2 * np.max(np.abs(exp))
    assert torch.equal(bd.attention(dq[1:].contiguous(), H)[0], got[1])


@pytest.mark.parametrize("T,hd", [(257, 64), (300, 72), (1025, 128), (200, 72)])
def test_attention_is_exact_at_the_largest_weight(T, hd):
    """Two keys share the weight, the second, in a later tile, d = 0 .. 8 doublings above the first, and all values are alike: the result is
    that value, bit for bit.  The largest probability is 1 without rounding; the other one, w0 <= 1/2 of the sum, is rounded by
    2^-9 (just under 1) to 2^-8 (just over 1/2, w0 = 1/3) of itself, so the sums differ by less than 2^-9, half a step of the result at
    the least.  A probability above 1 at the maximum would be off by up to 2^-8 of the whole."""
    bd = _bd()
    rng = np.random.default_rng(T + hd)
    qkv = np.zeros((1, T, 3, 2, hd), np.float32)
    d = np.linspace(0.0, 7.9, T)
    rng.shuffle(d)
    qkv[0, :, 0, :, 0] = (d * np.sqrt(hd) / np.log2(np.e))[:, None]
    qkv[0, :, 0, :, 1] = 64.0
    qkv[0, :, 1, :, 1] = -64.0                                 # weight 2^-500 and less for all keys but two
    qkv[0, [3, T - 30], 1, :, 1] = 0.0
    qkv[0, T - 30, 1, :, 0] = 1.0
    value = si._store(rng.uniform(1.0, 2.0, (2, hd)).astype(np.float32), "bf16")
    qkv[0, :, 2] = value
    got = bd.attention(_dev(qkv.reshape(1, T, -1), "bf16"), 2).float().cpu().numpy().reshape(T, 2, hd)
    assert np.array_equal(got, np.broadcast_to(value, got.shape)), int((got != value).any(axis=(1, 2)).sum())


@pytest.mark.parametrize("T,hd,dtype", [(257, 64, "bf16"), (300, 72, "bf16"), (1025, 72, "bf16"), (300, 128, "bf16"), (200, 72, "bf16"), (33, 16, "bf16"),
                                        (17, 32, "f32"), (33, 64, "f32"), (300, 72, "f32"), (77, 128, "f32")])
def test_attention_infinite_value_in_the_last_row(T, hd, dtype):
    """A ragged last key tile holds keys past T with probability 0; they must not be copies of the last value row, where an
    infinity would turn into NaN (0 x inf).  The infinite dimension is infinite for every query, all others keep their bits."""
    bd = _bd()
    H = 2
    rng = np.random.default_rng(T + hd)
    qkv = rng.standard_normal((1, T, 3, H, hd)).astype(np.float32)
    qkv[0, T - 1, 2, 1, 3] = 0.0
    base = bd.attention(_dev(qkv.reshape(1, T, -1), dtype), H)
    qkv[0, T - 1, 2, 1, 3] = np.inf
    got = bd.attention(_dev(qkv.reshape(1, T, -1), dtype), H)
    assert bool((got[0, :, hd + 3] == float("inf")).all())
    keep = torch.ones(H * hd, dtype=torch.bool, device="cuda")
    keep[hd + 3] = False
    assert torch.equal(got[..., keep], base[..., keep])


@pytest.mark.parametrize("T,hd,dtype,first,last", [(17, 64, "f32", 16, 17), (40, 16, "f32", 32, 40), (17, 16, "bf16", 16, 17), (300, 72, "f32", 288, 300),
                                                   (70, 128, "f32", 16, 32), (70, 32, "bf16", 48, 70), (257, 64, "bf16", 0, 16)])
def test_attention_keys_of_minus_infinity(T, hd, dtype, first, last):
    """Scores of -inf over whole 16-key tiles, so that a wave of the fp32 kernel, or one that shares the last query with others and
    takes 16 keys of every tile, sees no finite score: those keys have weight 0 and the result is the attention over the others (fp32 rounding; bf16 rounds the result once)."""
    bd = _bd()
    rng = np.random.default_rng(T + hd)
    qkv = si._store(rng.standard_normal((1, T, 3, 1, hd)).astype(np.float32), dtype)
    qkv[:, :, :2] = np.abs(qkv[:, :, :2])                      # positive queries: every score against a key of -inf is -inf
    rest = np.r_[0:first, last:T]
    q, k, v = (qkv[:, :, i].transpose(0, 2, 1, 3).astype(np.float64) for i in range(3))
    exp = odit.attention(q, k[:, :, rest], v[:, :, rest]).transpose(0, 2, 1, 3).reshape(1, T, hd)
    qkv[0, first:last, 1] = -np.inf
    got = bd.attention(_dev(qkv.reshape(1, T, -1), dtype), 1).float().cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - exp)) <= (1e-5 if dtype == "f32" else 2.0 ** -8) * np.max(np.abs(exp))
    qkv[0, :, 1] = -np.inf                                     # no finite score at all: no softmax
    assert np.isnan(bd.attention(_dev(qkv.reshape(1, T, -1), dtype), 1).float().cpu().numpy()).all()


@pytest.mark.parametrize("T,hd,first,last", [(257, 64, 0, 64), (300, 72, 0, 128), (1025, 128, 0, 64), (300, 128, 64, 256)])
def test_attention_key_tiles_of_minus_infinity(T, hd, first, last):
    """The same over whole tiles of 64 keys, the first ones among them: an online softmax has no finite maximum to start from.  Every
    probability and the result are rounded by at most 2^-8 of themselves, sums are fp32."""
    bd = _bd()
    rng = np.random.default_rng(T + hd)
    qkv = si._store(rng.standard_normal((1, T, 3, 1, hd)).astype(np.float32), "bf16")
    qkv[:, :, :2] = np.abs(qkv[:, :, :2])                      # positive queries: every score against a key of -inf is -inf
    rest = np.r_[0:first, last:T]
    q, k, v = (qkv[:, :, i].transpose(0, 2, 1, 3).astype(np.float64) for i in range(3))
    exp, size = (odit.attention(q, k[:, :, rest], x[:, :, rest]).transpose(0, 2, 1, 3).reshape(1, T, hd) for x in (v, np.abs(v)))
    qkv[0, first:last, 1] = -np.inf
    got = bd.attention(_dev(qkv.reshape(1, T, -1), "bf16"), 1).float().cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - exp) <= 2.0 ** -8 * (np.abs(exp) + size) + 1e-5)
    qkv[0, :, 1] = -np.inf                                     # no finite score at all: no softmax
    assert np.isnan(bd.attention(_dev(qkv.reshape(1, T, -1), "bf16"), 1).float().cpu().numpy()).all()


@pytest.mark.parametrize("rows,H,dtype", [(65541, 1, "f32"), (65541, 1, "bf16"), (1, 65541, "f32")])
def test_attention_of_more_rows_or_heads_than_a_grid_dimension(rows, H, dtype):
    bd = _bd()
    T, hd = 3, 16
    rng = np.random.default_rng(5)
    qkv = si._store(rng.standard_normal((rows, T, 3, H, hd)).astype(np.float32), dtype)
    got = bd.attention(_dev(qkv.reshape(rows, T, -1), dtype), H).float().cpu().numpy().astype(np.float64)
    q, k, v = (qkv[:, :, i].transpose(0, 2, 1, 3).astype(np.float64) for i in range(3))
    exp = odit.attention(q, k, v).transpose(0, 2, 1, 3).reshape(rows, T, H * hd)
    assert np.max(np.abs(got - exp)) <= (1e-5 if dtype == "f32" else 2.0 ** -8) * np.max(np.abs(exp))


def test_linear_f32_of_more_row_tiles_than_a_grid_dimension():
    bd = _bd()
    M, N, K = 64 * 65536 + 70, 4, 4                            # tiles of 64 rows
    rng = np.random.default_rng(6)
    a, w = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    _check(bd.linear(_dev(a, "f32"), _dev(w, "f32")), odit.linear(a.astype(np.float64), w.astype(np.float64), None), "f32", K)


@pytest.mark.parametrize("K", [2 ** 23 + 64, 2 ** 23 + 8])
def test_linear_bf16_of_very_long_rows_keeps_the_matrix_kernels(K):
    """Row strides past 2^23: offsets inside a small tile still fit into 32 bits.  The plain kernel, an order of magnitude slower
    per column, is told apart by its time against a sixteenth of the columns."""
    bd = _bd()
    M, N = 3, 8
    g = torch.Generator(device="cuda").manual_seed(1)
    a = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randn((N, K), generator=g, device="cuda").to(torch.bfloat16)
    exp = (a.double() @ w.double().T).cpu().numpy()
    # fp32 sums of K products in order: rounding errors of random sign, 2^-24 sqrt(K) of the magnitude; then one bf16 rounding
    err = np.abs(bd.linear(a, w).double().cpu().numpy() - exp)
    assert np.all(err <= 2.0 ** -8 * np.abs(exp) + 2.0 ** -24 * np.sqrt(K) * 8 * np.max(np.abs(exp)))

    def ms(x, y):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        bd.linear(x, y)
        start.record()
        for _ in range(3):
            bd.linear(x, y)
        end.record()
        end.synchronize()
        return start.elapsed_time(end)

    k = K // 128 * 8
    assert ms(a, w) < 16 * 4 * ms(a[:, :k].contiguous(), w[:, :k].contiguous())


@pytest.mark.parametrize("T,hd", [(256, 72), (200, 72), (96, 64)])
def test_attention_short_sequence_into_an_output_at_8_byte_alignment(T, hd):
    """The whole-sequence kernel (T <= 256) stores 16-byte chunks; an output that is only 8-byte aligned takes the tiled
    kernel instead.  Same values either way."""
    bd = _bd()
    rows, H = 3, 4
    rng = np.random.default_rng(7 * T + hd)
    qkv = si._store(rng.standard_normal((rows, T, 3, H, hd)).astype(np.float32), "bf16")
    dq = _dev(qkv.reshape(rows, T, 3 * H * hd), "bf16")
    aligned = bd.attention(dq, H)
    pool = torch.zeros(rows * T * H * hd + 4, dtype=torch.bfloat16, device="cuda")
    shifted = pool[4:].view(rows, T, H * hd)                   # data pointer 8 bytes past a 16-byte boundary
    assert shifted.data_ptr() % 16 == 8
    bd.attention(dq, H, out=shifted)
    q, k, v = (qkv[:, :, i].transpose(0, 2, 1, 3).astype(np.float64) for i in range(3))
    exp = odit.attention(q, k, v).transpose(0, 2, 1, 3).reshape(rows, T, H * hd)
    scale = np.max(np.abs(exp))
    for got in (aligned, shifted):
        assert np.max(np.abs(got.float().cpu().numpy().astype(np.float64) - exp)) <= 1.2e-2 * scale
    assert float(pool[:4].abs().max()) == 0.0                  # nothing written in front of the output


@pytest.mark.parametrize("M,N,K,act", [(27286, 3072, 3072, 0), (27286, 12288, 3072, 1), (4608, 3072, 12288, 0), (4608, 15360 // 5 * 3, 3072, 0)])
def test_linear_at_mmdit_sizes_sampled_rows(M, N, K, act):
    """The linear layers at the row counts of configurations 4 and 5 (4608 / 27286 tokens, hidden 3072, MLP 12288):
    the device computes the whole product, the oracle a sample of its rows (first and last tile, ragged tail
    included) by the plain definition."""
    bd = _bd()
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn((N, K), generator=g, device="cuda") * 0.03).to(torch.bfloat16)
    b = (torch.randn((N,), generator=g, device="cuda") * 0.1).to(torch.bfloat16)
    out = bd.linear(a, w, b, act)
    rng = np.random.default_rng(M)
    rows = np.unique(np.concatenate([np.arange(0, 8), np.arange(M - 40, M), rng.integers(0, M, 80)]))
    ridx = torch.from_numpy(rows).cuda()
    exp = odit.linear(a[ridx].float().cpu().numpy().astype(np.float64), w.float().cpu().numpy().astype(np.float64),
                      b.float().cpu().numpy().astype(np.float64))
    if act == 1:
        exp = odit.gelu_tanh(exp)
    _check(out[ridx], exp, "bf16", K)


@pytest.mark.parametrize("T,H", [(4608, 2), (27286, 1)])
def test_attention_at_mmdit_lengths_sampled_queries(T, H):
    """Attention at the sequence lengths of configurations 4 (4096 + 512 tokens) and 5 (27030 + 256), head_dim 128:
    the device computes every query; the oracle's plain softmax over ALL keys is evaluated for a few hundred sampled
    query rows (first tile, ragged last tile, random ones).  Keys are given a per-key offset along one direction so
    that the scores are far from uniform and the running maximum really moves along the hundreds of key tiles."""
    bd = _bd()
    hd = 128
    g = torch.Generator(device="cuda").manual_seed(T)
    qkv = torch.randn((1, T, 3, H, hd), generator=g, device="cuda")
    qkv[:, :, 1, :, 0] += torch.linspace(-3.0, 3.0, T, device="cuda")[None, :, None]        # keys drift along dim 0
    qkv[:, :, 0, :, 0] += 2.0                                                                 # every query looks along it
    qkv[:, :, 0] *= 2.5                                                                       # peaked softmax (score std 2.5)
    qkv[:, :, 2, :, 1] += torch.linspace(-2.0, 2.0, T, device="cuda")[None, :, None]        # values say which keys were attended
    qkv = qkv.to(torch.bfloat16)
    out = bd.attention(qkv.reshape(1, T, 3 * H * hd).contiguous(), H)
    rng = np.random.default_rng(T)
    qs = np.unique(np.concatenate([np.arange(0, 70), np.arange(T - 150, T), rng.integers(0, T, 160)]))
    host = qkv.float().cpu().numpy().astype(np.float64)
    q = host[:, qs, 0].transpose(0, 2, 1, 3)                       # [1, H, nq, hd]
    k = host[:, :, 1].transpose(0, 2, 1, 3)                        # [1, H, T, hd]
    v = host[:, :, 2].transpose(0, 2, 1, 3)
    exp = odit.attention(q, k, v).transpose(0, 2, 1, 3).reshape(len(qs), H * hd)
    got = out[0, torch.from_numpy(qs).cuda()].float().cpu().numpy().astype(np.float64)
    scale = np.max(np.abs(exp))
    assert np.max(np.abs(got - exp)) <= 1.2e-2 * scale, float(np.max(np.abs(got - exp)) / scale)


def test_linear_rejects_bad_arguments():
    bd = _bd()
    a = torch.zeros((4, 8), device="cuda"); w = torch.zeros((6, 8), device="cuda")
    with pytest.raises(bd.SpecaError) as e:
        bd.linear(a, w)                              # N not a multiple of 4
    assert e.value.code == bd.EINVAL
