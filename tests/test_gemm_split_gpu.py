"""The GEMM that splits K over a workgroup's waves, against the oracle: each
variant (32-row tiles in four shares, with cached and non-temporal weight
loads; 64-row tiles in four and in two shares) with ragged rows and columns,
shares without a step, shares that cut segments, both clamps, and the shapes on
both sides of its limits."""
import numpy as np
import pytest

import oracle
from paper_2607_17733_amd import workloads as W
from parity_util import check_gemm, fmt_for, gpu_run, oracle_quant, say

pytestmark = pytest.mark.gpu

SHAPES = [
    # M, K, N, (3-, 4-, 6-, 8-bit blocks), clamp or rounding (256 CUs)
    (65, 32, 130, (0, 1, 0, 0), "sym"),        # four shares of 32 rows: one step
    (97, 512, 1000, (0, 8, 4, 4), "sym"),
    (200, 1056, 390, (9, 14, 5, 5), "sym"),    # 3-bit blocks, short groups
    (77, 800, 260, (6, 9, 5, 5), "full"),
    (33, 256, 16, (0, 0, 8, 0), "rna"),
    (64, 320, 300, (0, 0, 0, 10), "full"),
    (20, 256, 8321, (0, 4, 2, 2), "sym"),      # at most 32 rows, 66 column tiles
    (16, 256, 24449, (0, 4, 2, 2), "sym"),     # at most 16 rows over short K: streamed
    (257, 256, 3700, (0, 4, 2, 2), "sym"),     # four shares of 64 rows
    (300, 640, 3500, (5, 7, 5, 3), "full"),
    (600, 256, 4500, (0, 4, 2, 2), "sym"),     # two shares of 64 rows
    (449, 352, 8190, (3, 4, 2, 2), "full"),
    (449, 256, 8250, (0, 4, 2, 2), "sym"),     # beyond: the tiled kernel
]


@pytest.mark.parametrize("M,K,N,counts,mode", SHAPES)
def test_split_gemm(M, K, N, counts, mode):
    say("gemm-split", M, K, N, counts, mode)
    n3, n4, n6, n8 = counts
    case = W.random_case(M * 17 + N, M, K, N, (n3 + n4, n6, n8), perm="scales")
    case.widths[:n3] = [3] * n3 if isinstance(case.widths, list) else 3
    clamp, round_ = ("full" if mode == "full" else "sym"), ("rna" if mode == "rna" else "rne")
    out = gpu_run(case, fmt_for(case, round_, clamp))
    qa, ea, qw, ew = oracle_quant(case, round_, clamp)
    Y = out["y"].cpu().numpy()
    check_gemm(Y, oracle.gemm(qa, ea, qw, ew, case.widths), qa, ea, qw, ew, case.widths, case.name)


def test_split_gemm_reads_large_weights_once():
    """One row tile over more than 64 MB of weights."""
    M, K, N = 7, 4800, 24600              # 0.59 bytes per weight: 70 MB
    say("gemm-split-once", M, K, N)
    case = W.random_case(11, M, K, N, (120, 15, 15), perm="random")
    out = gpu_run(case, fmt_for(case))
    assert out["w_mant"].numel() > 64 << 20
    qa, ea, qw, ew = oracle_quant(case)
    cols = np.r_[0:300, 12000:12300, N - 300:N]
    Yref = oracle.gemm(qa, ea, np.ascontiguousarray(qw[cols]), np.ascontiguousarray(ew[cols]),
                       case.widths)
    check_gemm(out["y"].cpu().numpy()[:, cols], Yref, qa, ea, qw[cols], ew[cols], case.widths,
               case.name)


@pytest.mark.parametrize("M,K,N,counts,clamp", [
    # at most 16 rows: 43 and 44 steps of 8-bit blocks over 225 column tiles; 3-bit
    # blocks up to 224 column tiles; a mixed full-clamp map of 35 and 36 steps
    (16, 2752, 28673, (0, 0, 0, 86), "sym"),
    (9, 2816, 28673, (0, 0, 0, 88), "sym"),
    (5, 5216, 28672, (152, 0, 6, 5), "sym"),
    (16, 2240, 24577, (0, 0, 36, 34), "full"),
    (3, 2304, 24577, (0, 0, 36, 36), "full"),
    # two column tiles per four CUs; more column tiles than CUs, 9 and 10 steps
    (24, 256, 16384, (0, 4, 2, 2), "sym"),
    (40, 576, 32800, (0, 0, 10, 8), "sym"),
    (40, 640, 32800, (0, 0, 10, 10), "sym"),
    # 33 to 64 rows: up to 16 column tiles, and the lines of one and two segments
    (48, 6272, 1000, (0, 0, 0, 196), "sym"),
    (33, 6336, 1000, (0, 0, 0, 198), "sym"),
    (40, 3840, 2100, (0, 120, 0, 0), "sym"),
    (40, 3968, 2100, (0, 124, 0, 0), "sym"),
    (64, 5024, 2100, (0, 0, 79, 78), "sym"),
    (50, 5120, 2100, (0, 0, 80, 80), "sym"),
    # and under the full clamp: mixed maps with and without 3-bit blocks
    (40, 1824, 2100, (0, 0, 29, 28), "full"),
    (40, 1888, 2100, (0, 0, 30, 29), "full"),
    (64, 4480, 2100, (70, 0, 35, 35), "full"),
])
def test_up_to_64_rows_on_both_sides(M, K, N, counts, clamp):
    """Shapes of up to 64 rows on both sides of the lines between the streaming
    kernel and split (256 CUs), over a part of the columns where there are many."""
    say("gemm-split-small", M, K, N, counts, clamp)
    n3, n4, n6, n8 = counts
    assert K == 32 * sum(counts)
    case = W.random_case(M * 13 + N, M, K, N, (n3 + n4, n6, n8), perm="scales")
    case.widths[:n3] = [3] * n3 if isinstance(case.widths, list) else 3
    out = gpu_run(case, fmt_for(case, "rne", clamp))
    qa, ea, qw, ew = oracle_quant(case, "rne", clamp)
    cols = np.r_[0:150, N // 2:N // 2 + 150, N - 150:N]
    qc, ec = np.ascontiguousarray(qw[cols]), np.ascontiguousarray(ew[cols])
    check_gemm(out["y"].cpu().numpy()[:, cols], oracle.gemm(qa, ea, qc, ec, case.widths), qa, ea,
               qc, ec, case.widths, case.name)
