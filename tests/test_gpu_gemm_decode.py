"""GPU parity of the prefill kernel that decodes the weights inside the contraction (btc_gemm, btc_gemm_aq on chunk
lengths 9 and 10) at the sizes where its tiling can go wrong: one column tile and less, a last tile partly past the
rows, weight rows and activation rows that leave tiles ragged, every index width and both chunk lengths (a chunk that
starts in the tile before), out % 4 != 0, calls split along k and calls that are not.  Every output against the oracle."""
import numpy as np
import pytest

import btc_synth as S

pytestmark = pytest.mark.gpu

CASES = [
    # out, in, v, K, M, activations
    (33, 16, 10, 128, 65, "bf16"), (160, 80, 9, 512, 129, "f16"), (161, 96, 10, 700, 257, "bf16"),
    (96, 2544, 9, 128, 128, "bf16"), (65, 4096, 9, 1024, 203, "f16"), (257, 1296, 10, 1024, 300, "f16"),
    (2049, 720, 9, 300, 511, "bf16"), (4100, 1600, 10, 256, 640, "f16"), (642, 8208, 9, 1024, 90, "bf16"),
    (5120, 528, 9, 1024, 1025, "bf16"),
]


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("out,n_in,v,K,M,xd", CASES)
def test_gemm_edges(G, oracle, out, n_in, v, K, M, xd):
    B = G.B
    print(f"gemm decode out={out} in={n_in} v={v} K={K} M={M} {xd}", flush=True)
    layer, x = S.make_case(7, out, n_in, v, K, M, x_dtype=xd)
    dl = G.DeviceLayer(layer, oracle)
    ref = G.oracle_all_rows(oracle, dl, x, xd)
    y = G.gemm(dl, x, B.BTC_BF16 if xd == "bf16" else B.BTC_F16, B.BTC_F32)
    rel, _ = G.assert_close(y, ref, "fp32 out")
    assert rel < 1e-5          # exact products, fp32 sums
    G.assert_close_bf16_out(G.gemm(dl, x, B.BTC_BF16 if xd == "bf16" else B.BTC_F16, B.BTC_BF16), ref, "bf16 out")


@pytest.mark.parametrize("out,n_in,v,K,M,bits", [(33, 16, 10, 128, 65, 8), (161, 144, 9, 1024, 130, 4), (97, 2544, 9, 128, 17, 8),
                                                 (2049, 1296, 10, 700, 300, 8), (4100, 528, 9, 512, 1025, 4)])
def test_codes_edges(G, oracle, out, n_in, v, K, M, bits):
    import torch
    B = G.B
    print(f"gemm_aq decode out={out} in={n_in} v={v} K={K} M={M} bits={bits}", flush=True)
    layer, x = S.make_case(8, out, n_in, v, K, M, x_dtype="f16")
    dl = G.DeviceLayer(layer, oracle)
    q, lo, step = oracle.quantize_rows(x, "f16", bits)
    ref = oracle.linear_aq(dl.packed_host, dl.codebook_host, layer.alpha, layer.mu, q, lo, step, n_in, v, K)
    wsum = torch.empty(out, dtype=torch.float32, device="cuda")
    ws = torch.full((max(B.btc_aq_workspace_bytes(dl.shape, M), B.btc_aq_workspace_bytes(dl.shape, 1)),), 0xFF,
                    dtype=torch.uint8, device="cuda")
    B.btc_weight_rowsums(dl.shape, dl.packed, dl.codebook, dl.alpha, dl.mu, wsum, ws)
    Y = G.GuardedOutput(M, out, torch.float32)
    B.btc_gemm_aq(dl.shape, dl.packed, dl.codebook, dl.alpha, dl.mu, wsum, G.dev(q.astype(np.uint8)),
                  G.dev(np.asarray(lo, np.float32)), G.dev(np.asarray(step, np.float32)), M, Y.payload, B.BTC_F32, ws)
    Y.check_guards()
    rel, _ = G.assert_close(Y.numpy(), ref, "codes")
    assert rel < 1e-5          # exact integer sums
