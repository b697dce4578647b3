"""Decode attention at the edges of its arithmetic against the float64 oracle:
block exponents past the scaled conversion's range, a negative score scale,
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
