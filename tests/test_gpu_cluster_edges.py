"""GPU parity (bit-exact) of btc_assign, btc_update and btc_pack where their kernels change over: codebooks around one
segment of the all-pairs kernel and around whole blocks of 32 codewords, vector lengths whose halves are partly or wholly
empty, the longest vectors of the table of patterns; assignments that agree with the patterns, nearly agree, and do
not; rows of indices around 64 words."""
import numpy as np
import pytest

from test_gpu_assign import G, _run, _update, _vectors  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,v,K", [(1000, 16, 8096), (1000, 16, 8097), (515, 15, 16193), (129, 31, 33), (700, 17, 31),
                                   (4001, 24, 65), (524288, 13, 40), (524287, 13, 40), (63, 3, 9)])
def test_assign(G, oracle, N, v, K):
    print(f"assign edges N={N} v={v} K={K}", flush=True)
    rng = np.random.default_rng(N + v)
    cb = rng.integers(0, 1 << v, size=K, dtype=np.uint64).astype(np.uint32)
    vec = _vectors(rng, N, v, cb)
    z, d2 = _run(G, vec, v, cb)
    z_ref, d_ref = oracle.assign(vec, v, cb)
    assert np.array_equal(z, z_ref) and np.array_equal(d2, d_ref)


@pytest.mark.parametrize("N,v,K,odd", [(300001, 10, 256, 0.0), (300001, 10, 256, 0.01), (300000, 10, 1400, 0.5),
                                       (70003, 4, 3, 1.0), (1048579, 12, 3000, 0.1), (16, 1, 4, 0.0)])
def test_update(G, oracle, N, v, K, odd):
    print(f"update edges N={N} v={v} K={K} odd={odd}", flush=True)
    rng = np.random.default_rng(N + K)
    cb = rng.integers(0, 1 << v, size=K, dtype=np.uint64).astype(np.uint32)
    vec = _vectors(rng, N, v, cb)
    home = rng.integers(0, K, size=1 << v)
    z = np.where(rng.random(N) < odd, rng.integers(0, K, size=N), home[vec & ((1 << v) - 1)]).astype(np.int32)
    new, _ = _update(G, vec, z, v, cb)
    assert np.array_equal(new, oracle.update(vec, z, v, cb))


@pytest.mark.parametrize("out,n_in,v,K", [(5, 640, 10, 256), (3, 2560, 10, 256), (3, 2570, 10, 200), (7, 2050, 1, 2),
                                          (4, 4099, 2, 4), (9, 18450, 9, 1024), (2, 33, 32, 65536), (1, 1, 5, 3)])
def test_pack(G, oracle, out, n_in, v, K):
    import torch
    B = G.B
    print(f"pack edges out={out} in={n_in} v={v} K={K}", flush=True)
    s = B.btc_shape_init(out, n_in, v, K)
    idx = np.random.default_rng(out + n_in).integers(0, K, size=(out, s.nchunks), dtype=np.int32)
    packed = G.GuardedOutput(out, s.words_per_row, torch.int32)
    ws = torch.zeros(16, dtype=torch.uint8, device="cuda")
    B.btc_pack(s, G.dev(idx), packed.payload, ws)
    packed.check_guards()
    ref = oracle.pack(idx, K)
    assert np.array_equal(packed.payload.cpu().numpy().view(np.uint32).reshape(ref.shape), ref)
    idx[out - 1, s.nchunks - 1] = K
    with pytest.raises(B.BtcError):
        B.btc_pack(s, G.dev(idx), packed.payload, ws)
    idx[out - 1, s.nchunks - 1] = 0
    B.btc_pack(s, G.dev(idx), packed.payload, ws)
