"""GPU parity of btc_gemv_groups on the settings that run by pairs of weights (chunk lengths 9 and 10), at the sizes
where its slots, row pairs and tables can go wrong: one chunk, one chunk more or less than a slot of 64, odd row
lengths, an odd number of rows on either side of two rows per wave, scales of very different sizes."""
import numpy as np
import pytest

import btc_synth as S
from test_groups_pins import pack_groups

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    import gpu_util
    return gpu_util


@pytest.mark.parametrize("out,n_in,v,K,ng,size", [
    (3, 7, 10, 128, 2, 1.0), (65, 640, 10, 256, 3, 1.0), (33, 641, 10, 1024, 4, 1e-6), (31, 576, 9, 512, 3, 1.0),
    (4097, 575, 9, 1024, 2, 1e4), (4999, 1281, 9, 128, 4, 1.0), (4100, 2570, 10, 100, 1, 1.0), (14001, 330, 10, 256, 3, 1.0)])
def test_pairs(G, oracle, out, n_in, v, K, ng, size):
    import torch
    B = G.B
    print(f"groups pairs out={out} in={n_in} v={v} K={K} G={ng} size={size}", flush=True)
    layer, x = S.make_case(43, out, n_in, v, K, 1)
    rng = np.random.default_rng(out + ng)
    g = rng.integers(0, ng, size=(out, n_in))
    alpha = (np.abs(rng.normal(0, 0.02, size=(out, ng))) * size).astype(np.float32)
    mu = (rng.normal(0, 0.002, size=(out, ng)) * size).astype(np.float32)
    alpha[1 % out] = mu[1 % out] = 0.0
    gm = pack_groups(g)
    dl = G.DeviceLayer(layer, oracle)
    ref = oracle.linear_groups(dl.packed_host, dl.codebook_host, alpha, mu, gm, x, n_in, v, K)
    Y = G.GuardedOutput(1, out, torch.float32)
    B.btc_gemv_groups(dl.shape, dl.packed, dl.codebook, G.dev(alpha), G.dev(mu), G.dev(gm), ng, G.dev(x), Y.payload, B.BTC_F32)
    Y.check_guards()
    rel, _ = G.assert_close(Y.numpy(), ref, "pairs")
    assert rel < 1e-5
