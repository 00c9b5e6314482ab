"""GPU parity of the long-vector engine (btc_gemv_code.hip) where it changes over: rows of one step and of full and partly
empty shares, codebooks in LDS as 16, 20 and 32 bits and gathered from memory, the last index of a matrix, odd rows of
activations, more rows per workgroup than waves, fewer rows than a workgroup has."""
import numpy as np
import pytest

import btc_synth as S
from test_gpu_engines import G, _run_engine  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [(1, 12, 12, 3000), (5, 1023, 16, 65536), (8192, 1025, 16, 65536), (4100, 4096, 16, 65536), (4099, 5137, 20, 65536),
         (9000, 1281, 18, 65536), (2100, 16384, 20, 65536), (700, 16383, 12, 4096), (1030, 16384, 16, 4096), (3000, 2049, 14, 9000),
         (260, 12287, 16, 32768), (28000, 515, 20, 40000), (6000, 3001, 20, 20000)]


@pytest.mark.parametrize("out,n_in,v,K", CASES)
def test_code_engine(G, oracle, out, n_in, v, K):
    print(f"code edges out={out} in={n_in} v={v} K={K}", flush=True)
    layer, x = S.make_case(3, out, n_in, v, K, 1, dist="uniform", outlier_frac=0.01)
    dl = G.DeviceLayer(layer, oracle)
    y = _run_engine(G, dl, x, 8)
    assert y is not None
    G.assert_close(y, G.oracle_all_rows(oracle, dl, x), "long vectors")
