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


@pytest.mark.parametrize("N,K,kinds", [(65536, 4096, 0), (65535, 4096, 0), (134217, 2000, 0), (1100003, 4096, 0), (300007, 1500, 3),
                                       (262149, 1024, 1), (70001, 4096, 1)])
def test_assign_16(G, oracle, N, K, kinds):
    """The table of 16-bit keys; with few different codewords most patterns are further away than a key can say."""
    print(f"assign edges N={N} v=16 K={K} kinds={kinds}", flush=True)
    rng = np.random.default_rng(N + K)
    cb = rng.integers(0, 1 << 16, size=K, dtype=np.uint64).astype(np.uint32)
    if kinds:
        cb = np.full(K, 0x1234, dtype=np.uint32)
        cb[K // 2:] = (0x1234, 0x1235, 0x9234)[kinds - 1]
    vec = _vectors(rng, N, 16, cb)
    vec[::5000] = cb[0] ^ 0xFFFF
    z, d2 = _run(G, vec, 16, cb)
    z_ref, d_ref = oracle.assign(vec, 16, cb)
    assert np.array_equal(z, z_ref) and np.array_equal(d2, d_ref)


@pytest.mark.parametrize("N,v,K,odd", [(400003, 16, 4096, 0.1), (99999, 16, 4096, 1.0), (70000, 24, 6000, 0.5), (50001, 32, 3, 0.0),
                                       (300001, 13, 65536, 0.2), (130001, 20, 1, 1.0), (300001, 10, 256, 0.0), (300001, 10, 256, 0.01), (300000, 10, 1400, 0.5),
                                       (70003, 4, 3, 1.0), (1048579, 12, 3000, 0.1), (16, 1, 4, 0.0)])
def test_update(G, oracle, N, v, K, odd):
    print(f"update edges N={N} v={v} K={K} odd={odd}", flush=True)
    rng = np.random.default_rng(N + K)
    cb = rng.integers(0, 1 << v, size=K, dtype=np.uint64).astype(np.uint32)
    vec = _vectors(rng, N, v, cb)
    home = rng.integers(0, K, size=1 << min(v, 20))
    z = np.where(rng.random(N) < odd, rng.integers(0, K, size=N), home[vec & ((1 << min(v, 20)) - 1)]).astype(np.int32)
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
