"""Decode attention at the edges of its arithmetic against the float64 oracle:
block exponents up to the largest, a negative score scale,
heads that fill one or both halves of the score tile, chunks that end in
either half."""
import numpy as np
import pytest
import torch

from oracle import attn as oattn
from paper_2607_17733_amd import mxq
from paper_2607_17733_amd import workloads as W
from parity_util import say, to_dev_bf16

pytestmark = pytest.mark.gpu


def _bits(x):
    return W.to_bf16_bits(np.ascontiguousarray(x, dtype=np.float32))


@pytest.mark.parametrize("widths,G,T,kexp,vexp,scale", [
    ([4, 4, 4, 4], 8, 77, 122, 121, 0.02), ([3, 4, 4, 8], 5, 40, 124, 0, 0.02),
    ([4, 4, 6, 8], 9, 49, 0, 121, 0.05), ([4, 4, 4, 4], 16, 33, 0, 0, -0.1),
    ([6, 6, 8, 8], 3, 16, 0, 0, -0.1), ([4, 6, 6, 6], 8, 15, 0, -125, 0.1),
    ([3, 3, 3, 3], 1, 97, -100, 0, 0.1), ([8, 8, 8, 8], 8, 130, 60, -60, 0.1)])
def test_attention_edges(widths, G, T, kexp, vexp, scale):
    say("attn-edges", widths, G, T, kexp, vexp, scale)
    B, Hkv, D = 2, 2, 128
    g = np.random.Generator(np.random.PCG64(T))
    qb = _bits(np.ldexp(g.normal(size=(B, G * Hkv, D)), -kexp))
    kb = _bits(np.ldexp(np.clip(g.normal(size=(B * T * Hkv, D)), -3, 3), kexp))
    vb = _bits(np.ldexp(np.clip(g.normal(size=(B * T * Hkv, D)), -3, 3), vexp))
    fmt = mxq.Format(D, widths)
    o = mxq.attn_decode(to_dev_bf16(qb.reshape(-1, D)).reshape(B, G * Hkv, D),
                        mxq.quantize_rows(to_dev_bf16(kb), fmt),
                        mxq.quantize_rows(to_dev_bf16(vb), fmt), fmt, B, G * Hkv, Hkv, T, scale)
    o = o.cpu().numpy().astype(np.float64)
    qf = W.bf16_bits_to_f32(qb).astype(np.float64)
    rows = T * Hkv
    for b in range(B):
        kd = oattn.dequantize_cache(kb[b * rows:(b + 1) * rows], widths)
        vd = oattn.dequantize_cache(vb[b * rows:(b + 1) * rows], widths)
        ref = oattn.attention(qf[b:b + 1], kd, vd, 1, G * Hkv, Hkv, T, scale)[0]
        vmax = np.abs(vd.reshape(T, Hkv, D)).max(axis=(0, 2))
        err = np.abs(o[b] - ref).max(axis=1) / vmax[np.arange(G * Hkv) // G]
        # scores of a few units in float32 (2^-22 relative) and float32 sums of T terms
        assert err.max() <= 1e-5, err.max()


def _top_rows(g, rows, m, E, where):
    """Cache rows whose block 2, in the rows of `where`, has exponent E: values of
    every size down to zero below a largest one (E = 255: it holds an infinity);
    the other blocks N(0, 1)."""
    x = g.normal(size=(rows, 128)).astype(np.float32)
    q = g.integers(-(2 ** (m - 1)) + 1, 2 ** (m - 1), size=(rows, 32)).astype(np.float64)
    q[:, 5], q[:, 6], q[:, 9] = 2 ** (m - 1) - 1, 0, -(2 ** (m - 2))
    lsb = np.ldexp(1.0, min(E, 254) - 127 - (m - 2))
    top = (q * lsb).astype(np.float32)
    if E == 255:
        top[:, 9] = np.inf
    x[where, 64:96] = top[where]
    return _bits(x)


@pytest.mark.parametrize("widths", [[6] * 4, [8] * 4, [4] * 4, [3, 4, 6, 8], [4, 6, 8, 8]])
@pytest.mark.parametrize("E", [248, 253, 254, 255])
@pytest.mark.parametrize("T", [1, 45])
def test_attention_largest_exponents(widths, E, T):
    """Blocks at the top of the exponent range, as K and as V: finite values at
    E = 253 and 254, zeros where the quantizer met an infinity (E = 255)."""
    say("attn-largest-exponents", widths, E, T)
    B, G, Hkv, D = 1, 3, 2, 128
    g = np.random.Generator(np.random.PCG64(E + T))
    fmt = mxq.Format(D, widths)
    top = np.zeros(T * Hkv, bool)
    top[(T // 2) * Hkv:(T // 2 + 1) * Hkv] = True          # one token's rows: the sums stay finite

    def check(q, kb, vb, scale):
        qb = _bits(q)
        o = mxq.attn_decode(to_dev_bf16(qb.reshape(-1, D)).reshape(B, G * Hkv, D),
                            mxq.quantize_rows(to_dev_bf16(kb), fmt),
                            mxq.quantize_rows(to_dev_bf16(vb), fmt), fmt, B, G * Hkv, Hkv, T, scale)
        o = o.cpu().numpy().astype(np.float64)
        kd, vd = oattn.dequantize_cache(kb, widths), oattn.dequantize_cache(vb, widths)
        for d in (kd, vd):
            np.nan_to_num(d, copy=False, nan=0.0)          # (the oracle's value of an E = 255 block)
        ref = oattn.attention(W.bf16_bits_to_f32(qb).astype(np.float64), kd, vd, B, G * Hkv, Hkv,
                              T, scale)
        assert np.isfinite(o).all()
        if T == 1:                                         # the token's own values
            assert np.abs(o - ref).max() <= 1e-6 * np.abs(ref).max()
            big = np.abs(ref) > 0
            assert (np.abs(o - ref)[big] <= 1e-6 * np.abs(ref)[big]).all() and not o[~big].any()
        for b in range(4):                                 # float32 sums of T terms, per block
            s = slice(32 * b, 32 * b + 32)
            lim = 1e-5 * np.abs(vd[:, s]).max()
            assert np.abs(o[..., s] - ref[..., s]).max() <= lim

    plain = _bits(g.normal(size=(T * Hkv, D)).astype(np.float32))
    qn = g.normal(size=(B, G * Hkv, D))
    # as V: scores of a few units
    check(qn, plain, _top_rows(g, T * Hkv, widths[2], E, top), 0.05)
    # as K: the queries bring the large block's scores down to a few units, the
    # other blocks' to nothing
    qs = qn.copy()
    qs[..., 64:96] = np.ldexp(qs[..., 64:96], -120)
    check(qs, _top_rows(g, T * Hkv, widths[2], E, top), plain, 1e-3)


def _run(fmt, q, k, v, B, Hq, Hkv, T, scale):
    D = 128
    qb, kb, vb = _bits(q), _bits(k), _bits(v)
    o = mxq.attn_decode(to_dev_bf16(qb.reshape(-1, D)).reshape(B, Hq, D),
                        mxq.quantize_rows(to_dev_bf16(kb.reshape(-1, D)), fmt),
                        mxq.quantize_rows(to_dev_bf16(vb.reshape(-1, D)), fmt), fmt, B, Hq, Hkv, T,
                        scale)
    kd = oattn.dequantize_cache(kb.reshape(-1, D), fmt.widths)
    vd = oattn.dequantize_cache(vb.reshape(-1, D), fmt.widths)
    ref = oattn.attention(W.bf16_bits_to_f32(qb).astype(np.float64), kd, vd, B, Hq, Hkv, T, scale)
    return o.cpu().numpy().astype(np.float64), ref, vd


@pytest.mark.parametrize("widths", [[4] * 4, [3] * 4, [4, 4, 6, 8]])
@pytest.mark.parametrize("G", [1, 9])
def test_attention_large_values(widths, G):
    """A head whose scores rise by 3.9 in a wave's second chunk, with values near
    2^120: sums of probabilities up to 1 stay finite."""
    say("attn-large-values", widths, G)
    B, Hkv, T, D = 64, 8, 200, 128                         # one split: 4 waves of one or two chunks
    g = np.random.Generator(np.random.PCG64(G))
    q = np.zeros((B, G * Hkv, D))
    q[..., 0] = 1.0
    k = np.zeros((B, T, Hkv, D))
    k[:, 128:160, :, 0] = 4.0                              # exact in every width
    v = np.ldexp(g.uniform(1, 1.9, size=(B, T, Hkv, D)), 120)
    o, ref, vd = _run(mxq.Format(D, widths), q, k, v, B, G * Hkv, Hkv, T, 3.9 / 4)
    assert np.abs(o - ref).max() <= 1e-5 * np.abs(vd).max()


@pytest.mark.parametrize("low", [range(16), range(0, 100), range(64, 160), range(16, 200)])
def test_attention_scores_of_minus_infinity(low):
    """Tokens whose scores overflow to -inf weigh nothing, also where they fill a
    half chunk, a wave's first chunk or a split; a query with a NaN gives NaN."""
    say("attn-minus-infinity", low)
    g = np.random.Generator(np.random.PCG64(low.stop))
    for B, G, Hkv, T in ((64, 2, 8, 200), (1, 9, 1, 200)):  # one split; splits of 64 tokens
        D, widths = 128, [4, 4, 6, 8]
        q = g.normal(size=(B, G * Hkv, D))
        q[..., 0] = np.ldexp(1.0, 100)
        k = g.normal(size=(B, T, Hkv, D))
        k[..., 0] = 0.0
        k[:, low, :, 0] = -np.ldexp(1.0, 40)               # 2^140 in float32
        v = g.normal(size=(B, T, Hkv, D))
        q[0, 1, 5] = np.nan
        o, ref, vd = _run(mxq.Format(D, widths), q, k, v, B, G * Hkv, Hkv, T, 0.05)
        assert np.isnan(o[0, 1]).all()
        o[0, 1] = ref[0, 1] = 0.0
        assert np.abs(o - ref).max() <= 1e-5 * np.abs(vd).max()


@pytest.mark.parametrize("T", [1024, 1025, 4096, 4097, 16385, 32700])
def test_attention_merge_of_splits(T):
    """Splits of 64 tokens on both sides of the merge's sizes (16, 64, 256 splits)."""
    say("attn-splits", T)
    g = np.random.Generator(np.random.PCG64(T))
    B, G, Hkv, D = 1, 2, 1, 128
    q, k, v = (g.normal(size=(B, n, Hkv * h, D)) for n, h in ((1, G), (T, 1), (T, 1)))
    o, ref, vd = _run(mxq.Format(D, [4, 4, 6, 8]), q[:, 0], k, v, B, G * Hkv, Hkv, T, 0.2)
    assert np.abs(o - ref).max() <= 1e-5 * np.abs(vd).max()


def test_attention_more_threads_than_one_grid_dimension():
    """68 million heads of one token: a wave each, more than 2^32 threads.  Every
    head returns its own V row, 2^(E - 129) throughout."""
    B, Hkv, T, D = 65535, 1040, 1, 128
    rows = B * Hkv
    assert rows * 64 > 1 << 32
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 100 GB of device memory")
    say("attn-grid", rows)
    fmt = mxq.Format(D, [4] * 4)
    dev = torch.device("cuda")
    q = torch.zeros((B, Hkv, D), dtype=torch.bfloat16, device=dev)
    mant = torch.full((rows, fmt.act_packed_bytes()), 0x11, dtype=torch.uint8, device=dev)
    E = (torch.arange(rows, dtype=torch.int32, device=dev) % 50 + 100).to(torch.uint8)
    exps = E[:, None].expand(rows, fmt.exp_row_bytes()).contiguous()
    o = mxq.attn_decode(q, (mant, exps), (mant, exps), fmt, B, Hkv, Hkv, T, 0.1).view(rows, D)
    for r in range(0, rows, 1 << 22):
        want = torch.exp2(E[r:r + (1 << 22)].float() - 129)
        assert bool((o[r:r + (1 << 22)] == want[:, None]).all()), r
    del o, q, mant, exps
    torch.cuda.empty_cache()
