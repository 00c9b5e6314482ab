"""GPU parity of the one-kernel engine for few activation rows (btc_gemv_few.hip) where it changes over: rows of odd length
(activations that start inside a word), the numbers of rows around its four widths, rows around a super-group and around
one and several pieces of activations in LDS, outputs around a workgroup's share; fp16 through btc_gemv, bf16 through
btc_gemm, 8-bit codes (rows that start on any byte) through btc_gemm_aq."""
import numpy as np
import pytest

import btc_synth as S
from test_gpu_engines import G, _run_engine  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [(1, 1, 10, 256, 2), (17, 639, 10, 512, 2), (64, 640, 10, 128, 3), (65, 641, 10, 1000, 4), (300, 2561, 10, 256, 5),
         (33, 575, 9, 1024, 7), (129, 577, 9, 512, 8), (40, 4093, 9, 1024, 9), (257, 2559, 10, 256, 16), (31, 2563, 10, 512, 16),
         (96, 20483, 10, 256, 2), (700, 10241, 10, 512, 3), (5000, 1923, 9, 1024, 15), (4097, 5121, 10, 200, 6), (16, 7, 9, 512, 13)]


@pytest.mark.parametrize("out,n_in,v,K,batch", CASES)
def test_gemv(G, oracle, out, n_in, v, K, batch):
    print(f"few out={out} in={n_in} v={v} K={K} batch={batch}", flush=True)
    layer, x = S.make_case(5, out, n_in, v, K, batch, dist="uniform", outlier_frac=0.01)
    dl = G.DeviceLayer(layer, oracle)
    y = _run_engine(G, dl, x, 3)
    assert y is not None
    G.assert_close(y, G.oracle_all_rows(oracle, dl, x), "one kernel, few rows")


@pytest.mark.parametrize("out,n_in,v,K,M,y", [(65, 1283, 10, 512, 3, "bf16"), (200, 1152, 9, 1024, 11, "f32"), (48, 643, 10, 256, 16, "f16")])
def test_gemm_bf16(G, oracle, out, n_in, v, K, M, y):
    import torch
    B = G.B
    print(f"few, bf16 out={out} in={n_in} v={v} K={K} M={M} y={y}", flush=True)
    layer, x = S.make_case(6, out, n_in, v, K, M, dist="uniform")
    dl = G.DeviceLayer(layer, oracle)
    xb = torch.from_numpy(x.view(np.float16).astype(np.float32)).to(torch.bfloat16)
    dt = {"bf16": torch.bfloat16, "f32": torch.float32, "f16": torch.float16}[y]
    Y = G.GuardedOutput(M, out, dt)
    ws = torch.empty(B.btc_workspace_bytes(dl.shape, M, True), dtype=torch.uint8, device="cuda")
    B.btc_gemm(dl.shape, dl.packed, dl.codebook, dl.alpha, dl.mu, xb.cuda(), B.BTC_BF16, M, Y.payload,
               {"bf16": B.BTC_BF16, "f32": B.BTC_F32, "f16": B.BTC_F16}[y], ws)
    Y.check_guards()
    W = torch.from_numpy(np.asarray(layer_dense(layer))).double()
    ref = xb.double() @ W.T
    err = (Y.payload.double().cpu().reshape(M, out) - ref).norm() / ref.norm()
    assert err < {"bf16": 4e-3, "f32": 1e-5, "f16": 1e-3}[y]


@pytest.mark.parametrize("out,n_in,v,K,M", [(1, 3, 10, 256, 1), (65, 641, 10, 512, 2), (130, 1283, 10, 128, 3), (33, 577, 9, 1024, 4),
                                           (200, 5762, 10, 256, 7), (70, 2303, 9, 512, 16), (47, 2561, 10, 600, 15)])
def test_codes(G, oracle, out, n_in, v, K, M):
    import torch
    B = G.B
    print(f"few, codes out={out} in={n_in} v={v} K={K} M={M}", flush=True)
    layer, _ = S.make_case(7, out, n_in, v, K, M, dist="uniform")
    dl = G.DeviceLayer(layer, oracle)
    rng = np.random.default_rng(M)
    Q = rng.integers(0, 256, size=(M, n_in), dtype=np.uint8)
    lo, step, wsum = (rng.standard_normal(n).astype(np.float32) for n in (M, M, out))
    Y = G.GuardedOutput(M, out, torch.float32)
    ws = torch.empty(B.btc_aq_workspace_bytes(dl.shape, M), dtype=torch.uint8, device="cuda")
    B.btc_gemm_aq(dl.shape, dl.packed, dl.codebook, dl.alpha, dl.mu, G.dev(wsum), G.dev(Q), G.dev(lo), G.dev(step), M, Y.payload,
                  B.BTC_F32, ws)
    Y.check_guards()
    ref = step[:, None].astype(np.float64) * (Q.astype(np.float64) @ layer_dense(layer).T) + lo[:, None].astype(np.float64) * wsum
    got = Y.payload.double().cpu().numpy().reshape(M, out)
    assert np.linalg.norm(got - ref) < 1e-5 * np.linalg.norm(ref)


def layer_dense(layer):
    bits = (layer.codebook[layer.idx][..., None] >> np.arange(layer.v, dtype=np.uint32)) & 1
    signs = (2.0 * bits - 1.0).reshape(layer.out, -1)[:, : layer.n_in]
    return layer.alpha[:, None].astype(np.float64) * signs + layer.mu[:, None].astype(np.float64)
