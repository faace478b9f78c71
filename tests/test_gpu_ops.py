"""GPU parity of the single operators (called through the C ABI) against the
CPU reference, with adversarial inputs that the end-to-end configurations
cannot see: non-zero biases, ragged shapes, peaked softmax, segment leaks."""
import numpy as np
import pytest
import torch

from oracle import encoder as oe
from paper_2603_26498_amd import binding as B
from util import assert_tokens_close, bf16_grid

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    return t.to(dtype) if dtype is not None else t


def sync():
    torch.cuda.synchronize()


# ---------------------------------------------------------------- LayerNorm
@pytest.mark.parametrize("rows,d", [(1, 256), (7, 160), (197, 256), (1030, 1280), (513, 1024), (33, 2048), (5, 64)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_layernorm(rows, d, dtype):
    rng = np.random.default_rng(rows * 7 + d)
    x = (rng.normal(0, 3, (rows, d)) + rng.normal(0, 2, (rows, 1))).astype(np.float32)
    g = (1 + rng.normal(0, 0.3, d)).astype(np.float32)
    b = rng.normal(0, 0.2, d).astype(np.float32)
    ref = oe.layernorm(x.astype(np.float64), g.astype(np.float64), b.astype(np.float64), 1e-6)
    y = torch.empty((rows, d), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV)
    B.tcmv_op_layernorm(B.TCMV_BF16 if dtype == "bf16" else B.TCMV_F32, dev(x), dev(g), dev(b), y, rows, d, 1e-6)
    sync()
    got = y.float().cpu().numpy()
    if dtype == "f32":
        assert np.abs(got - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())
    else:
        assert np.abs(got - ref).max() <= 2 ** -8 * np.abs(ref).max() + 1e-6
        assert_tokens_close(got, ref, 1e-2, 0.9999, "layernorm")


def test_layernorm_in_place_f32():
    rng = np.random.default_rng(3)
    x = rng.normal(0, 1, (37, 256)).astype(np.float32)
    ref = oe.layernorm(x.astype(np.float64), np.ones(256), np.zeros(256), 1e-6)
    t = dev(x)
    B.tcmv_op_layernorm(B.TCMV_F32, t, dev(np.ones(256, np.float32)), dev(np.zeros(256, np.float32)), t, 37, 256, 1e-6)
    sync()
    assert np.abs(t.cpu().numpy() - ref).max() <= 2e-5


# ---------------------------------------------------------------- GEMM
def _gemm_ref(a, w, bias, epi, c0):
    y = a.astype(np.float64) @ w.astype(np.float64).T + (bias.astype(np.float64) if bias is not None else 0)
    if epi == B.EPI_GELU:
        y = oe.gelu(y)
    if epi == B.EPI_RESID:
        y = c0.astype(np.float64) + y
    return y


@pytest.mark.parametrize("m,n,k", [(1, 64, 64), (127, 128, 64), (128, 128, 128), (300, 320, 640), (1000, 1280, 1216),
                                   (257, 136, 192), (129, 3840, 1280), (2050, 1280, 5120),
                                   (2050, 1928, 320), (1500, 2560, 128), (3333, 1280, 192)])
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_GELU, B.EPI_RESID])
def test_gemm_bf16(m, n, k, epi):
    rng = np.random.default_rng(m + 3 * n + 7 * k + epi)
    a = bf16_grid(rng.normal(0, 1, (m, k)))
    w = bf16_grid(rng.normal(0, 0.05, (n, k)))
    bias = rng.normal(0, 0.5, n).astype(np.float32)
    c0 = rng.normal(0, 1, (m, n)).astype(np.float32)
    ref = _gemm_ref(a, w, bias, epi, c0)
    if epi == B.EPI_RESID:
        c = dev(c0)
    else:
        c = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, epi, dev(a, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), c, m, n, k)
    sync()
    got = c.float().cpu().numpy()
    if epi == B.EPI_RESID:      # fp32 output: only accumulation-order error
        assert np.abs(got - ref).max() <= 1e-4 * max(1.0, np.abs(ref).max())
    else:
        assert np.abs(got - ref).max() <= 2 ** -8 * np.abs(ref).max() + 1e-5
        assert_tokens_close(got, ref, 1e-2, 0.9999, "gemm")


@pytest.mark.parametrize("m,n,k", [(40000 + 37, 2560, 128), (100000, 1024, 64)])
def test_residual_epilogue_on_an_output_larger_than_the_cache(m, n, k):
    """fp32 outputs above 400 MB take the form of the residual epilogue that requests the old values one group of
    columns ahead (both large tile families, ragged rows); every row is checked."""
    rng = np.random.default_rng(m + n)
    a = bf16_grid(rng.normal(0, 1, (m, k)))
    w = bf16_grid(rng.normal(0, 0.05, (n, k)))
    bias = rng.normal(0, 0.5, n).astype(np.float32)
    c0 = rng.normal(0, 1, (m, n)).astype(np.float32)
    assert m * n * 4 > 400e6
    c = dev(c0)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_RESID, dev(a, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), c, m, n, k)
    sync()
    got = c.cpu().numpy()
    for lo in range(0, m, 8192):                      # reference in slabs: float64 of the whole output would be 0.5 GB
        hi = min(m, lo + 8192)
        ref = _gemm_ref(a[lo:hi], w, bias, B.EPI_RESID, c0[lo:hi])
        assert np.abs(got[lo:hi] - ref).max() <= 1e-4 * max(1.0, np.abs(ref).max()), (lo, hi)


def test_gemm_bf16_no_bias_and_exact_small_integers():
    """Small integer inputs make every product and sum exact: bit-exact result expected."""
    rng = np.random.default_rng(0)
    m, n, k = 200, 192, 128
    a = rng.integers(-3, 4, (m, k)).astype(np.float32)
    w = rng.integers(-3, 4, (n, k)).astype(np.float32)
    c = dev(np.zeros((m, n), np.float32))
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_RESID, dev(a, torch.bfloat16), dev(w, torch.bfloat16), None, c, m, n, k)
    sync()
    assert np.array_equal(c.cpu().numpy(), a @ w.T)


@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (197, 256, 768), (70, 100, 50), (197, 1024, 256), (65, 64, 147)])
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_GELU, B.EPI_RESID])
def test_gemm_f32(m, n, k, epi):
    rng = np.random.default_rng(m + n + k + epi)
    a = rng.normal(0, 1, (m, k)).astype(np.float32)
    w = rng.normal(0, 0.1, (n, k)).astype(np.float32)
    bias = rng.normal(0, 0.5, n).astype(np.float32)
    c0 = rng.normal(0, 1, (m, n)).astype(np.float32)
    ref = _gemm_ref(a, w, bias, epi, c0)
    c = dev(c0) if epi == B.EPI_RESID else torch.full((m, n), float("nan"), device=DEV)
    B.tcmv_op_gemm(B.TCMV_F32, epi, dev(a), dev(w), dev(bias), c, m, n, k)
    sync()
    assert np.abs(c.cpu().numpy() - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())


# ---------------------------------------------------------------- attention
def _attn(dtype, qkv, cu, d, heads):
    T = qkv.shape[0]
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    cd = B.TCMV_BF16 if dtype == "bf16" else B.TCMV_F32
    ws_bytes = B.tcmv_op_attention_workspace(cd, cu, d, heads)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device=DEV)
    ws.fill_(0xFF)                                   # poison: padding must never be used
    index = torch.frombuffer(bytearray(B.tcmv_op_attention_index(cd, cu, d, heads)), dtype=torch.uint8).to(DEV)
    out = torch.full((T, d), float("nan"), dtype=tdt, device=DEV)
    B.tcmv_op_attention(cd, dev(qkv, tdt), cu, d, heads, index, out, ws, ws.numel())
    sync()
    return out.float().cpu().numpy()


def _qkv(rng, T, d, q_scale, dtype):
    q = rng.normal(0, q_scale, (T, d)); k = rng.normal(0, 1, (T, d)); v = rng.normal(0, 1, (T, d))
    x = np.concatenate([q, k, v], 1).astype(np.float32)
    return bf16_grid(x) if dtype == "bf16" else x


ATTN_CASES = [
    # (segment lengths, d, heads, std of q): scores have std ~ q_scale
    ([64], 64, 1, 1.0),
    ([1], 128, 2, 1.0),                                 # single key: output = V
    ([130, 0, 5, 257], 160, 2, 1.0),                    # ragged, empty segment, head size 80
    ([576, 576], 128, 2, 0.3),                          # near-uniform softmax
    ([300, 77, 1, 640], 160, 2, 6.0),                   # peaked softmax
    ([1000], 320, 4, 8.0),                              # peaked, several query tiles and heads
    ([63, 65, 127, 129], 64, 2, 4.0),
    ([200], 96, 1, 2.0),
    ([333], 32, 1, 2.0),
]


@pytest.mark.parametrize("lens,d,heads,qs", ATTN_CASES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention(lens, d, heads, qs, dtype):
    rng = np.random.default_rng(sum(lens) + d + heads)
    cu = [0] + list(np.cumsum(lens))
    T = cu[-1]
    qkv = _qkv(rng, T, d, qs, dtype)
    x = qkv.astype(np.float64)
    ref = oe.attention(x[:, :d], x[:, d:2 * d], x[:, 2 * d:], cu, heads)
    got = _attn(dtype, qkv, [int(c) for c in cu], d, heads)
    if dtype == "f32":
        assert np.abs(got - ref).max() <= 2e-5 * max(1.0, np.abs(ref).max())
    else:
        # probabilities and outputs are rounded to bf16 (2^-9 relative each)
        assert np.abs(got - ref).max() <= 1.2e-2 * np.abs(ref).max()
        assert_tokens_close(got, ref, 2e-2, 0.9995, "attention")
        assert np.sqrt(((got - ref) ** 2).mean()) <= 4e-3 * np.sqrt((ref ** 2).mean())


@pytest.mark.parametrize("lens,qs,big_head,rows", [
    ([1000, 333, 1, 0, 640, 257, 129, 2048], 6.0, None, 256), # ragged: 256-row work items (4 waves x 2 query tiles), peaked
    ([2048, 2048, 1024], 6.0, None, 512),                     # multiples of 512: 512-row work items (8 waves), peaked
    ([4096, 3072], 1.0, 3, 512),                              # long segments: key-norm bound holds except for one head
    ([4096], 1.0, 3, 256),                                    # the same with as many 256-row items as CUs
    ([1000, 333, 2085, 640, 1500, 64], 1.0, None, 256),       # small scores, ragged: the reference-free loop with masked last tiles
    ([4096, 2560, 1536], 0.5, None, 512),                     # small scores, full tiles, 512-row items: the reference-free loop without masks
])
def test_attention_large_work_items(lens, qs, big_head, rows):
    """Enough work items for the kernels with two query tiles per wave to be chosen (a single small problem
    gets 128-row items): 16 heads of 80, ragged and aligned segments, peaked scores (rescaling path), and long
    segments on which the reference-free copy handles all heads but one."""
    rng = np.random.default_rng(sum(lens))
    d, heads, dh = 1280, 16, 80
    cu = [0] + list(np.cumsum(lens))
    T = cu[-1]
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, [int(c) for c in cu], d, heads) == rows
    q = rng.normal(0, qs, (T, d)); k = rng.normal(0, 1, (T, d)); v = rng.normal(0, 1, (T, d))
    if big_head is not None:
        q[:, big_head * dh:(big_head + 1) * dh] *= 8.0
    qkv = bf16_grid(np.concatenate([q, k, v], 1).astype(np.float32))
    x = qkv.astype(np.float64)
    ref = oe.attention(x[:, :d], x[:, d:2 * d], x[:, 2 * d:], cu, heads)
    got = _attn("bf16", qkv, [int(c) for c in cu], d, heads)
    assert np.abs(got - ref).max() <= 1.2e-2 * np.abs(ref).max()
    assert_tokens_close(got, ref, 2e-2, 0.9995, "attention, large work items")
    assert np.sqrt(((got - ref) ** 2).mean()) <= 4e-3 * np.sqrt((ref ** 2).mean())


@pytest.mark.parametrize("lens,heads,dh,rows", [([64, 37, 64], 64, 64, 128), ([100], 120, 32, 128), ([300], 60, 64, 128), ([700, 60], 60, 64, 128), ([1250], 60, 64, 256)])
def test_attention_wider_than_the_pass_over_the_keys(lens, heads, dh, rows):
    """More heads than the separate pass over the keys holds: the operator goes without key norms, as the encoder does, with
    128-row items, over one and two groups of keys, and with 256-row items."""
    d, cu = heads * dh, [0] + [int(c) for c in np.cumsum(lens)]
    qkv = _qkv(np.random.default_rng(heads + rows), cu[-1], d, 3.0, "bf16")
    x = qkv.astype(np.float64)
    ref = oe.attention(x[:, :d], x[:, d:2 * d], x[:, 2 * d:], cu, heads)
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, cu, d, heads) == rows
    got = _attn("bf16", qkv, cu, d, heads)
    assert np.abs(got - ref).max() <= 1.2e-2 * np.abs(ref).max()
    assert_tokens_close(got, ref, 2e-2, 0.9995, "wide attention")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_attention_segments_do_not_leak(dtype):
    """Encode {A, B} together == A and B alone; huge values in B must not move A."""
    rng = np.random.default_rng(42)
    d, heads = 160, 2
    la, lb = 150, 90
    qkv = _qkv(rng, la + lb, d, 2.0, dtype)
    both = _attn(dtype, qkv, [0, la, la + lb], d, heads)
    a_alone = _attn(dtype, qkv[:la], [0, la], d, heads)
    b_alone = _attn(dtype, qkv[la:], [0, lb], d, heads)
    assert np.array_equal(both[:la], a_alone) and np.array_equal(both[la:], b_alone)
    poisoned = qkv.copy()
    poisoned[la:, 2 * d:] = 3e4            # V of segment B
    poisoned[la:, d:2 * d] *= 50           # K of segment B
    got = _attn(dtype, poisoned, [0, la, la + lb], d, heads)
    assert np.array_equal(got[:la], both[:la])


def test_attention_zero_queries_give_mean_of_values():
    rng = np.random.default_rng(9)
    d, heads, T = 160, 2, 200
    qkv = _qkv(rng, T, d, 1.0, "bf16")
    qkv[:, :d] = 0
    got = _attn("bf16", qkv, [0, T], d, heads)
    ref = qkv[:, 2 * d:].astype(np.float64).mean(0, keepdims=True)
    assert np.abs(got - ref).max() <= 1e-2 * np.abs(qkv[:, 2 * d:]).max()


def test_empty_inputs_are_no_ops():
    B.tcmv_op_layernorm(B.TCMV_BF16, None, None, None, None, 0, 256, 1e-6)
    B.tcmv_op_gemm(B.TCMV_BF16, 0, None, None, None, None, 0, 128, 64)
    B.tcmv_op_attention(B.TCMV_BF16, None, [0, 0, 0], 128, 2, None, None, None, 0)
    sync()


def _bf16_round(v):
    """fp64 -> nearest bf16 value (ties to even), as fp64; the fp32 step in between is harmless here because the
    values tested are never within 2^-24 relative of a bf16 tie."""
    u = np.asarray(v, np.float32).view(np.uint32).astype(np.uint64)
    u = ((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16
    return u.astype(np.uint32).view(np.float32).astype(np.float64)


@pytest.mark.parametrize("m,n,k", [(192, 64, 64), (16384 + 37, 2560, 128)])
@pytest.mark.parametrize("with_bias", [False, True])
def test_gelu_epilogue_on_an_exact_grid(m, n, k, with_bias):
    """The activation of the fc1 epilogue on known arguments.  Rows of A are one-hot, so the accumulator is exactly
    one weight (plus an fp32 bias chosen so that the sum is exact): the weights run over every bf16 value with
    2^-12 <= |x| <= 10, i.e. an exact grid that is dense near 0.  The bf16 output must be within one bf16 unit in
    the last place of the rounded exact erf-form GELU (or 2^-22 where that is larger) for every argument; a tanh-form
    or a sigmoid-form activation misses this by several units.  Both tile families are driven (small shape: 64-row
    tiles; large shape: persistent 256-row tiles)."""
    e, mant = np.meshgrid(np.arange(-12, 4), np.arange(128), indexing="ij")
    mag = (np.ldexp(1.0 + mant / 128.0, e)).reshape(-1)
    mag = mag[mag <= 10.0]
    grid = np.concatenate([mag, -mag, [0.0]]).astype(np.float32)
    assert np.array_equal(bf16_grid(grid), grid)
    rng = np.random.default_rng(11)
    w = grid[rng.integers(0, grid.size, (n, k))]
    w.reshape(-1)[:grid.size] = grid                                  # every grid value occurs at least once
    a = np.zeros((m, k), np.float32)
    a[np.arange(m), np.arange(m) % k] = 1.0
    # bias: multiples of 2^-13 below 2; |x| < 16 with a last place of 2^-19 fits the 24 bits of an fp32
    bias = (rng.integers(-16000, 16000, n) * 2.0 ** -13).astype(np.float32) if with_bias else np.zeros(n, np.float32)
    x = w.astype(np.float64).T[np.arange(m) % k] + bias.astype(np.float64)            # [m, n], exact
    assert np.array_equal(x.astype(np.float32).astype(np.float64), x)
    want = _bf16_round(oe.gelu(x))
    c = torch.full((m, n), float("nan"), dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_GELU, dev(a, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), c, m, n, k)
    sync()
    got = c.float().cpu().numpy().astype(np.float64)
    ulp = np.ldexp(1.0, np.floor(np.log2(np.maximum(np.abs(want), 1e-300))).astype(np.int64) - 7)
    tol = np.maximum(ulp, 2.0 ** -22)
    bad = np.abs(got - want) > tol
    assert not bad.any(), (x[bad][:5], got[bad][:5], want[bad][:5])
    # the pin has teeth: the tanh form of the activation, rounded the same way, breaks the bound
    tanh_form = _bf16_round(0.5 * x * (1 + np.tanh(np.sqrt(2 / np.pi) * (x + 0.044715 * x ** 3))))
    assert (np.abs(tanh_form - want) > tol).any()


def test_gemm_bf16_large_tile_path_with_ragged_rows():
    """Enough 256x256 tiles to select the large-tile kernel, with a ragged last row tile."""
    rng = np.random.default_rng(77)
    m, n, k = 16384 + 37, 2560, 128
    a = bf16_grid(rng.normal(0, 1, (m, k)))
    w = bf16_grid(rng.normal(0, 0.05, (n, k)))
    bias = rng.normal(0, 0.5, n).astype(np.float32)
    for epi in (B.EPI_STORE, B.EPI_GELU, B.EPI_RESID):
        c0 = rng.normal(0, 1, (m, n)).astype(np.float32)
        ref = _gemm_ref(a, w, bias, epi, c0)
        c = dev(c0) if epi == B.EPI_RESID else torch.full((m, n), float("nan"), dtype=torch.bfloat16, device=DEV)
        B.tcmv_op_gemm(B.TCMV_BF16, epi, dev(a, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), c, m, n, k)
        sync()
        got = c.float().cpu().numpy()
        tol = 1e-4 * max(1.0, np.abs(ref).max()) if epi == B.EPI_RESID else 2 ** -8 * np.abs(ref).max() + 1e-5
        assert np.abs(got - ref).max() <= tol, epi


def test_gemm_bf16_wide_tile_path_with_ragged_rows_and_columns():
    """A shape for which tiles 320 columns wide need fewer rounds over the CUs than 256x256 ones (640 -> 512
    tiles on 256 CUs): the wave tiles are 160 columns wide and leave the kernel in column groups of 64, 64
    and 32.  Last row tile and last column tile ragged; the gated epilogue goes the same way."""
    rng = np.random.default_rng(78)
    m, n, k = 8100, 5112, 128
    a = bf16_grid(rng.normal(0, 1, (m, k)))
    w = bf16_grid(rng.normal(0, 0.05, (n, k)))
    bias = rng.normal(0, 0.5, n).astype(np.float32)
    for epi in (B.EPI_STORE, B.EPI_GELU, B.EPI_RESID):
        c0 = rng.normal(0, 1, (m, n)).astype(np.float32)
        ref = _gemm_ref(a, w, bias, epi, c0)
        c = dev(c0) if epi == B.EPI_RESID else torch.full((m, n), float("nan"), dtype=torch.bfloat16, device=DEV)
        B.tcmv_op_gemm(B.TCMV_BF16, epi, dev(a, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), c, m, n, k)
        sync()
        got = c.float().cpu().numpy()
        tol = 1e-4 * max(1.0, np.abs(ref).max()) if epi == B.EPI_RESID else 2 ** -8 * np.abs(ref).max() + 1e-5
        assert np.abs(got - ref).max() <= tol, epi
    u = a.astype(np.float64) @ w.astype(np.float64).T + bias
    ref = oe.silu(u[:, 0::2]) * u[:, 1::2]
    c = torch.full((m, n // 2), 7.0, dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_GATED, dev(a, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), c, m, n, k)
    sync()
    assert np.abs(c.float().cpu().numpy() - ref).max() <= 2 ** -7 * np.abs(ref).max()


# ---------------------------------------------------------------- encoder-family variants
@pytest.mark.parametrize("rows,d", [(3, 320), (1030, 1280), (77, 64)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rmsnorm(rows, d, dtype):
    rng = np.random.default_rng(rows + d)
    x = (rng.normal(0.5, 3, (rows, d))).astype(np.float32)
    g = (1 + rng.normal(0, 0.3, d)).astype(np.float32)
    ref = oe.rmsnorm(x.astype(np.float64), g.astype(np.float64), 1e-6)
    y = torch.empty((rows, d), dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device=DEV)
    B.tcmv_op_layernorm(B.TCMV_BF16 if dtype == "bf16" else B.TCMV_F32, dev(x), dev(g), None, y, rows, d, 1e-6)
    sync()
    got = y.float().cpu().numpy()
    tol = 2e-5 if dtype == "f32" else 2 ** -8
    assert np.abs(got - ref).max() <= tol * max(1.0, np.abs(ref).max())


@pytest.mark.parametrize("rows,d", [(64, 1280), (33, 1024), (5, 320)])
def test_rmsnorm_adds_in_one_written_out_order(rows, d):
    """Results do not change with the compiler's choices: the squares of four neighbours are added as
    fma(x, x, y*y) + fma(z, z, w*w), a lane adds its groups (64 lanes apart) in order, the lanes are added pairwise."""
    rng = np.random.default_rng(d)
    x = rng.normal(0.5, 3, (rows, d)).astype(np.float32)
    g = (1 + rng.normal(0, 0.3, d)).astype(np.float32)
    y = torch.empty((rows, d), dtype=torch.float32, device=DEV)
    B.tcmv_op_layernorm(B.TCMV_F32, dev(x), dev(g), None, y, rows, d, 1e-6)
    sync()
    v = x.reshape(rows, d // 4, 4)
    sq = lambda a, b: (a.astype(np.float64) ** 2 + (b * b).astype(np.float64)).astype(np.float32)   # fma: one rounding
    q4 = sq(v[..., 0], v[..., 1]) + sq(v[..., 2], v[..., 3])
    q4 = np.concatenate([q4, np.zeros((rows, -(d // 4) % 64), np.float32)], 1).reshape(rows, -1, 64)
    q = np.zeros((rows, 64), np.float32)
    for j in range(q4.shape[1]):
        q = q + q4[:, j]
    while q.shape[1] > 1:
        q = q[:, :q.shape[1] // 2] + q[:, q.shape[1] // 2:]
    rstd = np.float32(1) / np.sqrt(q / np.float32(d) + np.float32(1e-6))
    assert np.array_equal(y.cpu().numpy(), x * rstd * g)


@pytest.mark.parametrize("m,n2,k", [(300, 256, 128), (1029, 1280, 320), (4100, 6912, 1280)])
def test_gated_epilogue(m, n2, k):
    """Columns arrive as (gate, up) pairs; the kernel writes silu(gate) * up."""
    rng = np.random.default_rng(m)
    a = bf16_grid(rng.normal(0, 1, (m, k)).astype(np.float32))
    w = bf16_grid(rng.normal(0, 0.08, (n2, k)).astype(np.float32))
    bias = rng.normal(0, 0.3, n2).astype(np.float32)
    u = a.astype(np.float64) @ w.astype(np.float64).T + bias
    ref = oe.silu(u[:, 0::2]) * u[:, 1::2]
    c = torch.full((m, n2 // 2), 7.0, dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_GATED, dev(a, torch.bfloat16), dev(w, torch.bfloat16), dev(bias), c, m, n2, k)
    sync()
    got = c.float().cpu().numpy()
    assert np.abs(got - ref).max() <= 2 ** -7 * np.abs(ref).max()
    assert_tokens_close(got, ref, 1e-2, 0.9999, "gated epilogue")


def test_gated_epilogue_extreme_gates():
    """exp(-gate) overflows below -88.7: the output is then 0 (the value itself is below 1e-36), above it is gate * up."""
    m, n2, k = 64, 512, 64
    gate = np.tile(np.array([-3e38, -1e4, -100.0, -88.0, -87.0, -30.0, -1.0, 0.0, 1e-30, 1.0, 30.0, 87.0, 100.0, 1e4, 3e30, 1e38], np.float32), n2 // 32)
    w = np.zeros((n2, k), np.float32)
    bias = np.empty(n2, np.float32)
    bias[0::2], bias[1::2] = gate, 0.5
    c = torch.full((m, n2 // 2), 7.0, dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_GATED, torch.zeros((m, k), dtype=torch.bfloat16, device=DEV), dev(w, torch.bfloat16), dev(bias), c, m, n2, k)
    sync()
    g = gate.astype(np.float64)
    ref = 0.5 * g / (1.0 + np.exp(np.minimum(-g, 700.0)))
    got = c.float().cpu().numpy().astype(np.float64)
    # bf16 keeps 8 significant bits: rounding moves a value by up to 2^-8 of itself; the exponent's rounding (89 * 2^-24) is
    # in the 2^-7.99; 2e-36: exp(-gate) has overflowed
    assert np.all(np.abs(got - ref) <= 2.0 ** -7.99 * np.abs(ref) + 2e-36)


def _gates_next_to_bf16_ties():
    """Gates 6 .. 17 whose quotient gate / (1 + exp(-gate)), rounded to fp32, is half way between two bf16 values or one fp32
    step beside, where one step more or less changes the bf16.  The denominator is known for certain: 1 + exp(-gate) is
    a whole number of steps of 2^-23 above 1, and gates whose exp(-gate) comes within a tenth of a step of where that
    number changes are left out (exp is off by less than 1e-6 of itself, 0.02 steps at 6)."""
    # bf16 values are 1/32 apart between 4 and 8, 1/16 up to 16, then 1/8
    ties = np.concatenate([np.arange(6 * 64 + 1, 8 * 64, 2) / 64, np.arange(8 * 32 + 1, 16 * 32, 2) / 32, np.arange(16 * 16 + 1, 17 * 16, 2) / 16])
    gates = []
    for t in ties.astype(np.float32):
        for q in (np.nextafter(t, np.float32(0)), t, np.nextafter(t, np.float32(99))):
            x = float(q)
            for _ in range(8):
                x = float(q) * (1.0 + np.exp(-x))
            x = np.float32(x)
            for x in (np.nextafter(x, np.float32(0)), x, np.nextafter(x, np.float32(99))):
                steps = np.exp(-float(x)) * 2.0 ** 23
                if x / np.float32(1.0 + np.rint(steps) * 2.0 ** -23) == q and abs(steps % 1.0 - 0.5) > 0.1:
                    gates.append(x)
                    break
    return np.array(gates, np.float32)


def _gated_of(gate, up):
    """silu(gate) * up through the operator: one output column for each pair, the product itself is zero."""
    n = len(gate)
    bias = np.stack([gate, np.broadcast_to(np.float32(up), gate.shape)], 1).reshape(-1).astype(np.float32)
    c = torch.full((64, n), 7.0, dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_GATED, torch.zeros((64, 64), dtype=torch.bfloat16, device=DEV),
                   torch.zeros((2 * n, 64), dtype=torch.bfloat16, device=DEV), dev(bias), c, 64, 2 * n, 64)
    sync()
    got = c.float().cpu().numpy()
    assert (got == got[0]).all()
    return got[0]


def test_gated_epilogue_quotient_is_correctly_rounded():
    """The quotient of the gate has the fp32 rounding of a division: one step off and the bf16 beside is stored."""
    gate = _gates_next_to_bf16_ties()
    gate = gate[: len(gate) // 4 * 4]
    assert len(gate) > 400
    d = (1.0 + np.rint(np.exp(-gate.astype(np.float64)) * 2.0 ** 23) * 2.0 ** -23).astype(np.float32)
    got = _gated_of(gate, 1.0)
    wrong = np.nonzero(got != _bf16_round(gate / d))[0]
    assert len(wrong) == 0, (len(wrong), len(gate), gate[wrong[:8]], got[wrong[:8]])


def test_gated_epilogue_denominators_whose_reciprocal_is_subnormal():
    """Gates of -87.4 to -88.7: 1 + exp(-gate) is above 2^126, the quotient (2.7e-37 and more) is an ordinary number and
    a large factor brings it back.  exp of such an argument is off by 2^-17 of itself at most, the bf16 by 2^-9."""
    gate = np.linspace(-88.7, -87.0, 256).astype(np.float32)
    got = _gated_of(gate, 2.0 ** 110).astype(np.float64)
    ref = gate.astype(np.float64) / (1.0 + np.exp(-gate.astype(np.float64))) * 2.0 ** 110
    assert np.all(np.abs(got - ref) <= (2.0 ** -8 + 2.0 ** -15) * np.abs(ref))


def test_gelu_epilogue_far_from_zero():
    """Beyond the range of the fit the lower tail has to go on falling: 0 for negative values, the value itself for others."""
    m, n, k = 64, 512, 64
    x = np.tile(np.array([-3e38, -1e30, -1e10, -1e4, -300.0, -50.0, -20.0, -9.0, 6.0, 9.0, 20.0, 300.0, 1e4, 1e10, 1e30, 3e38], np.float32), n // 16)
    c = torch.full((m, n), 7.0, dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_GELU, torch.zeros((m, k), dtype=torch.bfloat16, device=DEV),
                   dev(np.zeros((n, k), np.float32), torch.bfloat16), dev(x), c, m, n, k)
    sync()
    got = c.float().cpu().numpy()
    assert np.array_equal(got[:, x > 0], np.broadcast_to(_bf16_round(x[x > 0]), (m, n // 2)))
    assert np.abs(got[:, x < 0]).max() <= 1e-17          # 9 * Phi(-9) = 1e-18


def test_gelu_epilogue_keeps_overflow_visible():
    """Infinite sums and NaN leave GELU as NaN on the bf16 path (inf * 0; the erf form of the fp32 path agrees but for +inf,
    which it keeps): an overflow does not turn into an ordinary number.  Their neighbours are untouched."""
    m, n, k = 64, 512, 64
    x = np.tile(np.array([np.inf, 1.0, -np.inf, -1.0, np.nan, 3.0, 0.0, -3.0], np.float32), n // 8)
    c = torch.full((m, n), 7.0, dtype=torch.bfloat16, device=DEV)
    B.tcmv_op_gemm(B.TCMV_BF16, B.EPI_GELU, torch.zeros((m, k), dtype=torch.bfloat16, device=DEV), torch.zeros((n, k), dtype=torch.bfloat16, device=DEV),
                   dev(x), c, m, n, k)
    sync()
    got, ok = c.float().cpu().numpy(), np.isfinite(x)
    assert np.isnan(got[:, ~ok]).all()
    assert np.abs(got[:, ok] - oe.gelu(x[ok].astype(np.float64))).max() <= 2.0 ** -8 * 3


def test_attention_mixed_norm_bounds_in_one_launch():
    """Some (segment, head, query tile) combinations have provably small scores and are exponentiated without
    a softmax reference, others in the same launch are not: head 0 has large queries, one block of query rows
    of head 1 is large, one segment has large keys.  Every row must come out right whichever copy handled it."""
    rng = np.random.default_rng(123)
    d, heads, dh = 240, 3, 80
    lens = [700, 1300, 520]
    cu = [0] + list(np.cumsum(lens))
    T = cu[-1]
    q = rng.normal(0, 1.0, (T, d)); k = rng.normal(0, 1.0, (T, d)); v = rng.normal(0, 1.0, (T, d))
    q[:, :dh] *= 7.0                       # head 0: bound far above the limit everywhere
    q[300:556, dh:2 * dh] *= 7.0           # head 1: one tile of queries in segment 0
    k[cu[2]:, 2 * dh:] *= 6.0              # head 2: large keys in the last segment only
    qkv = bf16_grid(np.concatenate([q, k, v], 1).astype(np.float32))
    x = qkv.astype(np.float64)
    ref = oe.attention(x[:, :d], x[:, d:2 * d], x[:, 2 * d:], cu, heads)
    got = _attn("bf16", qkv, [int(c) for c in cu], d, heads)
    assert np.isfinite(got).all()
    assert np.abs(got - ref).max() <= 1.2e-2 * np.abs(ref).max()
    assert_tokens_close(got, ref, 2e-2, 0.9995, "attention, mixed bounds")
    # the same rows, recomputed with uniformly small inputs elsewhere, do not change (no interaction between copies)
    small = qkv.copy()
    small[:, :dh] = qkv[:, :dh] / 7.0
    got2 = _attn("bf16", bf16_grid(small), [int(c) for c in cu], d, heads)
    assert np.array_equal(got[:, dh:], got2[:, dh:])


# ---------------------------------------------------------------- bandwidth reference
def test_stream_reference_reads_and_writes_what_it_says():
    """Words written are the XOR of the words each thread read (threads stride over the input), so no read can be
    dropped; a size of zero on either side is allowed, misaligned sizes are refused."""
    nt = 2048 * 256
    n_in, n_out = nt + nt // 2 + 5, nt + 77
    rng = np.random.default_rng(0)
    src = rng.integers(0, 2 ** 32, (n_in, 4), dtype=np.uint64).astype(np.uint32)
    acc = np.zeros((nt, 4), np.uint32)
    for k in range(0, n_in, nt):
        blk = src[k:k + nt]
        acc[:len(blk)] ^= blk
    want = acc[np.arange(n_out) % nt]
    d_in = torch.from_numpy(src.view(np.int32)).to(DEV)
    d_out = torch.zeros((n_out, 4), dtype=torch.int32, device=DEV)
    B.tcmv_op_stream(d_in, n_in * 16, d_out, n_out * 16)
    sync()
    assert np.array_equal(d_out.cpu().numpy().view(np.uint32), want)
    B.tcmv_op_stream(None, 0, d_out, 16 * 10)             # nothing read: zeros written
    B.tcmv_op_stream(d_in, 16 * 10, None, 0)
    B.tcmv_op_stream(None, 0, None, 0)
    sync()
    assert not d_out[:10].any() and np.array_equal(d_out[10:].cpu().numpy().view(np.uint32), want[10:])
    with pytest.raises(B.TcmvError):
        B.tcmv_op_stream(d_in, 24, d_out, 16)


# (m, n, k): 16x16 tiles (k a multiple of 16, few tiles) at their edges, 64x64 tiles with vector loads and a ragged last
# slice, and with many tiles
@pytest.mark.parametrize("m,n,k", [(1, 1, 16), (17, 33, 4096), (16, 16, 80), (65, 64, 148), (1100, 1024, 32), (1025, 1001, 64)])
@pytest.mark.parametrize("epi", [B.EPI_STORE, B.EPI_RESID])
def test_gemm_f32_tile_edges(m, n, k, epi):
    test_gemm_f32(m, n, k, epi)


@pytest.mark.parametrize("dh", [16, 48, 112, 128])
def test_attention_f32_head_sizes(dh):
    """Segments around the 16-query and 16-key tiles and the four waves that share the keys; every remaining head size."""
    test_attention([15, 16, 17, 1, 63, 64, 65, 80], 2 * dh, 2, 3.0 / dh ** 0.5 * 4, "f32")


@pytest.mark.parametrize("dh", [16, 64])
def test_attention_f32_infinities_stay_where_they_belong(dh):
    """An infinite value in the last row of V reaches its own column only, although the last tile of keys is padded
    with that row; keys that score -inf weigh nothing, also where they fill the first tile of 16 keys that a wave sees
    (keys 16..31 of 80, 0..15 of 40).  A row whose keys all score -inf has no softmax."""
    rng = np.random.default_rng(dh)
    lens, heads = [17, 80, 40, 20], 2
    d = heads * dh
    cu = [0] + [int(c) for c in np.cumsum(lens)]
    qkv = _qkv(rng, cu[-1], d, 1.0, "f32")
    qkv[:, 0] = 1.0 + np.abs(qkv[:, 0])                    # first element of the first head's queries: positive
    qkv[16, 2 * d + 3] = np.inf                             # segment of 17: V of the last row
    qkv[cu[1] + 16:cu[1] + 32, d] = -np.inf                 # segment of 80: scores of the first head
    qkv[cu[2]:cu[2] + 16, d] = -np.inf                      # segment of 40
    qkv[cu[3]:cu[4], d] = -np.inf                           # segment of 20: every key
    x = qkv.astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = oe.attention(x[:, :d], x[:, d:2 * d], x[:, 2 * d:], cu, heads)
    got = _attn("f32", qkv, cu, d, heads)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref[cu[3]:, :dh]).all() and np.isnan(ref).sum() == 20 * dh
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.isinf(ref).sum() == 17
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= 2e-5 * max(1.0, np.abs(ref[ok]).max())


@pytest.mark.parametrize("dh", [32, 64, 80, 96])
@pytest.mark.parametrize("lens,rows", [([256, 130, 64, 100, 33, 200, 77], 64), ([600, 300, 129, 100, 33, 200, 77], 128)])
def test_attention_bf16_infinities_stay_where_they_belong(lens, rows, dh):
    """Keys that score -inf weigh nothing: a run of them, whole tiles, those of whole groups of waves (64-row items: also the
    first keys of a segment); a segment whose keys all score -inf, or one of whose keys scores +inf or is not a number, has
    no softmax in that head.  Nothing reaches another head or segment."""
    rng = np.random.default_rng(dh + rows)
    heads = 2
    d = heads * dh
    cu = [0] + [int(c) for c in np.cumsum(lens)]
    assert B.tcmv_op_attention_rows(B.TCMV_BF16, cu, d, heads) == rows
    qkv = _qkv(rng, cu[-1], d, 1.0, "bf16")
    qkv[:, 0] = 1.0 + np.abs(qkv[:, 0])                    # first element of the first head's queries: positive
    qkv = bf16_grid(qkv)
    first = 0 if rows == 64 else 40                        # an undivided loop sets its reference from the first 32 keys
    qkv[first:128, d] = -np.inf                            # runs of keys of the first head
    qkv[cu[1] + 64:cu[2], d] = -np.inf
    qkv[cu[2] + 32:cu[2] + 64, d] = -np.inf
    qkv[cu[3]:cu[4], d] = -np.inf                          # every key
    qkv[cu[4] + 7, d] = np.inf
    qkv[cu[5] + 150, d] = np.nan
    x = qkv.astype(np.float64)
    with np.errstate(invalid="ignore"):
        ref = oe.attention(x[:, :d], x[:, d:2 * d], x[:, 2 * d:], cu, heads)
    got = _attn("bf16", qkv, cu, d, heads)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.isnan(ref).sum() == (cu[6] - cu[3]) * dh
    ok = np.isfinite(ref)
    assert np.isfinite(got[ok]).all() and np.abs(got[ok] - ref[ok]).max() <= 1.2e-2 * np.abs(ref[ok]).max()


# one product for every tile kernel and epilogue, ragged in both directions, with short contractions (fewer k-tiles than
# stages where the kernel is taken for them)
TILE_KERNEL_CASES = [
    (B.EPI_STORE, 37, 136, 64, "64x64"), (B.EPI_STORE, 12747, 200, 64, "128x128"), (B.EPI_STORE, 10881, 136, 512, "128x128 k/2"),
    (B.EPI_STORE, 11047, 280, 1536, "128x160"), (B.EPI_STORE, 1349, 6832, 2048, "192x256"), (B.EPI_STORE, 13927, 272, 256, "256x128"),
    (B.EPI_STORE, 13379, 568, 256, "256x160"), (B.EPI_STORE, 13091, 520, 192, "256x256 persistent"), (B.EPI_STORE, 2827, 5656, 256, "256x320 persistent"),
    (B.EPI_GELU, 9803, 272, 64, "128x128"), (B.EPI_GELU, 12331, 136, 448, "128x128 k/2"), (B.EPI_GELU, 11037, 280, 1536, "128x160"),
    (B.EPI_GELU, 10977, 840, 2048, "192x256"), (B.EPI_GELU, 9347, 392, 256, "256x128"), (B.EPI_GELU, 1153, 6584, 256, "256x160"),
    (B.EPI_RESID, 33, 144, 64, "64x64"), (B.EPI_RESID, 10475, 264, 64, "128x128"), (B.EPI_RESID, 10969, 152, 1536, "128x128 k/2"),
    (B.EPI_RESID, 13393, 264, 1280, "128x160"), (B.EPI_RESID, 1685, 7064, 1536, "192x256"), (B.EPI_RESID, 12287, 336, 1536, "256x128"),
    (B.EPI_RESID, 7455, 1032, 1024, "256x160"), (B.EPI_RESID, 6181, 3944, 128, "256x256 persistent"), (B.EPI_RESID, 14463, 2144, 128, "256x320 persistent"),
    (B.EPI_GATED, 33, 144, 64, "64x64"), (B.EPI_GATED, 12667, 208, 64, "128x128"), (B.EPI_GATED, 11251, 144, 448, "128x128 k/2"),
    (B.EPI_GATED, 11051, 272, 1536, "128x160"), (B.EPI_GATED, 13325, 656, 2048, "192x256"), (B.EPI_GATED, 13813, 272, 256, "256x128"),
    (B.EPI_GATED, 13279, 528, 256, "256x160"), (B.EPI_GATED, 9441, 800, 192, "256x256 persistent"), (B.EPI_GATED, 12563, 1552, 192, "256x320 persistent")]


@pytest.mark.parametrize("epi,m,n,k,kernel", TILE_KERNEL_CASES)
def test_gemm_bf16_tile_kernels(epi, m, n, k, kernel):
    assert B.tcmv_op_gemm_kernel(epi, m, n, k) == kernel
    (test_gated_epilogue if epi == B.EPI_GATED else test_gemm_bf16)(*((m, n, k) if epi == B.EPI_GATED else (m, n, k, epi)))


@pytest.mark.parametrize("epi,m,n,k,kernel", [
    (B.EPI_STORE, 14851, 1288, 1024, "256x256 persistent + 256x128"), (B.EPI_GELU, 7688, 2568, 1152, "256x320 persistent + 64x64"),
    (B.EPI_RESID, 16897, 1288, 1024, "256x320 persistent + 128x128"), (B.EPI_RESID, 20226, 1032, 1024, "256x256 persistent + 256x160"),
    (B.EPI_GATED, 10246, 1928, 1152, "256x256 persistent + 128x160")])
def test_gemm_bf16_whole_rounds_and_the_rest(epi, m, n, k, kernel):
    """Whole rounds of large tiles for the first rows, another kernel for the ragged rest."""
    test_gemm_bf16_tile_kernels(epi, m, n, k, kernel)


@pytest.mark.parametrize("lens,qs,big_head", [([4096, 2048, 2048], 6.0, None), ([4096, 4096], 1.0, 3)])
def test_attention_work_items_of_512_rows(lens, qs, big_head):
    """16 items of 512 rows for 16 heads, one for every CU: peaked scores, and the reference-free copy for all heads but one."""
    test_attention_large_work_items(lens, qs, big_head, 512)
