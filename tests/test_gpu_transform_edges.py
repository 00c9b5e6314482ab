"""GPU parity of btc_transform's matrix-core kernel where it changes over: rows of the n1 x n2 view that start inside words
(odd n2), that end inside a step of 16 and inside a pair, blocks of 32 rows and columns that are full, ragged and single,
factors whose operands do not all fit LDS, more items than waves, both activation types and every output type; rows of
zeros and of infinities next to others."""
import numpy as np
import pytest

import btc_synth as S
from test_gpu_transform import G, _check, _run  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    (41, 64, 70, "bf16", "bf16"), (61, 64, 65, "f16", "f16"), (64, 73, 60, "bf16", "bf16"), (33, 81, 41, "f16", "f32"),
    (72, 34, 90, "bf16", "f32"), (32, 106, 50, "bf16", "f16"), (31, 22, 300, "f16", "bf16"), (97, 17, 140, "f16", "f16"),
    (128, 224, 13, "f16", "f16"), (128, 255, 10, "bf16", "bf16"), (128, 256, 9, "f16", "f32"), (1, 7, 500, "f16", "f32"),
    (5, 15, 300, "bf16", "bf16"), (65, 40, 1000, "bf16", "bf16"), (4, 2, 700, "f16", "f16"), (108, 128, 270, "f16", "f16"),
]


@pytest.mark.parametrize("n1,n2,M,kind,yd", CASES)
def test_transform(G, oracle, n1, n2, M, kind, yd):
    B = G.B
    print(f"transform edges n1={n1} n2={n2} M={M} {kind}->{yd}", flush=True)
    y_dtype = {"f32": B.BTC_F32, "f16": B.BTC_F16, "bf16": B.BTC_BF16}[yd]
    bits, P1, P2 = S.draw_transform(9 + n1 + n2, n1, n2)
    xb = S.draw_x(np.random.default_rng(n1 + n2 + M), M, n1 * n2, kind)
    xb[1] = 0
    y = _run(G, xb, kind, bits, P1, P2, y_dtype)
    rows = np.unique(np.concatenate([np.arange(min(M, 8)), np.arange(3, M, 61), [M - 2, M - 1]]))
    ref = oracle.transform(xb[rows], bits, P1, P2, kind)
    _check(y[rows], ref, y_dtype, B, (n1, n2, M, kind, yd))
    # the accuracy of fp32 sums, whatever the output's rounding: of fp32 outputs itself
    if yd == "f32":
        assert np.linalg.norm(y[rows] - ref) < 2e-6 * np.linalg.norm(ref)
    assert not np.any(y[1])
    inf = {"f16": 0x7C00, "bf16": 0x7F80}[kind]
    xb[3, n1 * n2 // 2] = inf
    y2 = _run(G, xb, kind, bits, P1, P2, y_dtype)
    others = np.arange(M) != 3
    assert np.array_equal(y2[others], y[others])


# one or a few rows: rows of n1 past four and n2 past eight, single rows and columns, rows that start inside a word, the
# largest factors, and workgroups of two half-waves up to thirty-two
FEW = [
    (1, 1, 1, "f16", "f32"), (1, 256, 3, "bf16", "f32"), (4, 9, 2, "f16", "f16"), (3, 250, 3, "bf16", "bf16"), (5, 8, 1, "f16", "f32"),
    (128, 1, 2, "f16", "f32"), (7, 255, 3, "f16", "f32"), (33, 63, 3, "bf16", "f16"), (65, 131, 4, "bf16", "f32"),
    (72, 104, 1, "f16", "f16"), (97, 145, 5, "f16", "bf16"), (127, 255, 2, "bf16", "f32"), (128, 256, 8, "f16", "f32"),
]


@pytest.mark.parametrize("n1,n2,M,kind,yd", FEW)
def test_few_rows(G, oracle, n1, n2, M, kind, yd):
    B = G.B
    print(f"transform few rows n1={n1} n2={n2} M={M} {kind}->{yd}", flush=True)
    y_dtype = {"f32": B.BTC_F32, "f16": B.BTC_F16, "bf16": B.BTC_BF16}[yd]
    bits, P1, P2 = S.draw_transform(5 + n1 + n2, n1, n2)
    xb = S.draw_x(np.random.default_rng(n1 + n2 + M), M, n1 * n2, kind)
    y = _run(G, xb, kind, bits, P1, P2, y_dtype)
    ref = oracle.transform(xb, bits, P1, P2, kind)
    _check(y, ref, y_dtype, B, (n1, n2, M, kind, yd))
    if yd == "f32":
        assert np.linalg.norm(y - ref) < 2e-6 * np.linalg.norm(ref)
    if M > 1:      # a row of infinities stays among itself
        xb[1] = {"f16": 0x7C00, "bf16": 0x7F80}[kind]
        y2 = _run(G, xb, kind, bits, P1, P2, y_dtype)
        others = np.arange(M) != 1
        assert np.array_equal(y2[others], y[others])
