"""Performance cases of the binary-codebook linear layer: what programs that hold a compressed decoder model have the
library do, from one product on one activation row to whole layers on thousands of them.

Six kinds of case:
  gemv     one decode product, called by itself (btc_gemv): any matrix, 1..16 activation rows
  decode   one token through the linear layers of a decoder (q, k, v in one launch, o, gate and up in one launch,
           down), with or without the online activation transform in front of every one of them, called one by one or
           replayed from a captured graph
  groups   one decode product of the storage variant with several (alpha, mu) pairs per weight row (btc_gemv_groups)
  gemm     many activation rows through the seven projections of a decoder layer (btc_gemm): a batch of sequences at
           decode, short and long prompts; with or without the transform (btc_transform)
  act      the same on 8- or 4-bit activation codes (btc_quantize_rows, btc_gemm_aq)
  cluster  one round of the codebook clustering and the storing of its result (btc_assign, btc_update, btc_pack)

Bit settings are (v, K): vector length and codebook entries, log2(K)/v bits per weight.  Index distributions:
"uniform", and "zipf" (exponent 1.1), where few codewords dominate as they do after clustering."""
import math

import numpy as np
import torch

import paper_2506_12040_amd as B

SETTINGS = [(10, 256), (10, 512), (10, 128), (9, 1024)]      # 0.8, 0.9, 0.7, 1.11 bit
LONG_SETTINGS = [(16, 65536), (20, 65536), (16, 4096)]       # long vectors, large codebooks
TORCH = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
BTC = {"f16": B.BTC_F16, "bf16": B.BTC_BF16, "f32": B.BTC_F32}
SIZE = {"f16": 2, "bf16": 2, "f32": 4}


def listed():
    return [
        # the smallest product in use: one attention projection of a 7B-shaped layer, one token, called by itself
        dict(name="gemv-4096", kind="gemv", out=4096, **{"in": 4096}, v=10, K=512, batch=1, y="f16", dist="uniform",
             outliers=False),
        # sixteen sequences decoded together through an up projection, with outlier channels as activations have them
        dict(name="gemv-batch16", kind="gemv", out=11008, **{"in": 4096}, v=10, K=512, batch=16, y="f16",
             dist="uniform", outliers=True),
        # vectors of 16 weights with a codebook of 65536 entries (1 bit), one token
        dict(name="gemv-long-vectors", kind="gemv", out=8192, **{"in": 8192}, v=16, K=65536, batch=1, y="f16",
             dist="uniform", outliers=False),
        # one token through all 40 layers of a 13B-shaped model at 0.8 bit, as a serving loop replays it
        dict(name="decode-13b", kind="decode", d=5120, kv=5120, ff=13824, v=10, K=256, layers=40, dist="zipf",
             transform=False, graph=True),
        # one token through layers of the 70B shape (grouped-query attention) at 0.9 bit, called layer by layer
        dict(name="decode-70b", kind="decode", d=8192, kv=1024, ff=28672, v=10, K=512, layers=8, dist="uniform",
             transform=False, graph=False),
        # one token through 13B-shaped layers with the four activation transforms that each of them needs
        dict(name="decode-13b-transform", kind="decode", d=5120, kv=5120, ff=13824, v=10, K=256, layers=16, dist="zipf",
             transform=True, graph=True),
        # two split points (three groups per weight row) on an up projection, one token, called by itself
        dict(name="groups-3", kind="groups", out=13824, **{"in": 5120}, v=10, K=256, ngroups=3, y="f16", dist="zipf"),
        # 32 sequences decoded together through a 13B-shaped layer
        dict(name="gemm-rows32", kind="gemm", d=5120, kv=5120, ff=13824, v=10, K=256, rows=32, x="bf16", y="bf16",
             dist="zipf", transform=False),
        # a short prompt of odd length through a 7B-shaped layer at 1.11 bit, fp32 outputs
        dict(name="gemm-rows203", kind="gemm", d=4096, kv=4096, ff=11008, v=9, K=1024, rows=203, x="f16", y="f32",
             dist="uniform", transform=False),
        # a prompt of 2048 tokens through a 13B-shaped layer with its transforms
        dict(name="gemm-rows2048", kind="gemm", d=5120, kv=5120, ff=13824, v=10, K=256, rows=2048, x="bf16", y="bf16",
             dist="zipf", transform=True),
        # a prompt of 1024 tokens on 8-bit activation codes
        dict(name="act8-rows1024", kind="act", d=5120, kv=5120, ff=13824, v=10, K=256, rows=1024, bits=8, x="bf16",
             y="bf16", dist="zipf"),
        # one clustering round over the sign vectors of an up projection, and its indices packed
        dict(name="cluster-13824", kind="cluster", out=13824, **{"in": 5120}, v=10, K=256),
    ]


# ---- drawn cases ------------------------------------------------------------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _step(value, step):
    return max(step, (value + step // 2) // step * step)


def _layer_sizes(rng, d_max, ff_max, transform):
    """Widths of a decoder layer: multiples of 64 (of 16 for the keys and values), that factor where a transform
    needs it."""
    while True:
        d = _step(_log(rng, 1024, d_max), 64)
        ff = _step(int(d * rng.uniform(2.0, 3.5)), 64)
        kv = _step(d // rng.choice([1, 1, 4, 8]), 16)
        if ff <= ff_max and (not transform or (factors(d) and factors(ff))):
            return dict(d=d, kv=kv, ff=ff)


def draw(rng):
    kind = rng.choice(["gemv", "decode", "groups", "gemm", "act", "cluster"])
    v, K = rng.choice(SETTINGS)
    dist = rng.choice(["uniform", "zipf"])
    if kind == "gemv":
        batch = _log(rng, 1, 16)
        if rng.random() < 0.2:
            (v, K), batch = rng.choice(LONG_SETTINGS), 1
        n_in = _log(rng, 512, 16384 if v > 10 else 28672)
        out = _log(rng, 256, min(28672, 28672 * 8192 // n_in))
        return dict(kind=kind, out=out, **{"in": n_in}, v=v, K=K, batch=batch, y=rng.choice(["f16", "f16", "f32"]), dist=dist,
                    outliers=rng.random() < 0.5)
    if kind == "decode":
        transform = rng.random() < 0.5
        size = _layer_sizes(rng, 8192, 28672, transform)
        return dict(kind=kind, **size, v=v, K=K, layers=rng.randint(1, 8), dist=dist, transform=transform,
                    graph=rng.random() < 0.5)
    if kind == "groups":
        return dict(kind=kind, out=_log(rng, 512, 13824), **{"in": _log(rng, 1024, 13824)}, v=v, K=K,
                    ngroups=rng.choice([2, 3, 3, 4]), y=rng.choice(["f16", "f32"]), dist=dist)
    if kind == "gemm":
        transform = rng.random() < 0.5
        x = rng.choice(["bf16", "bf16", "f16"])
        return dict(kind=kind, **_layer_sizes(rng, 5120, 13824, transform), v=v, K=K, rows=_log(rng, 17, 2048), x=x,
                    y=rng.choice([x, "f32"]), dist=dist, transform=transform)
    if kind == "act":
        x = rng.choice(["bf16", "f16"])
        return dict(kind=kind, **_layer_sizes(rng, 5120, 13824, False), v=v, K=K, rows=_log(rng, 1, 2048),
                    bits=rng.choice([8, 4]), x=x, y=rng.choice([x, "f32"]), dist=dist)
    v, K = rng.choice(SETTINGS + [(12, 512), (16, 4096)])
    return dict(kind=kind, out=_log(rng, 512, 13824), **{"in": _log(rng, 1024, 13824)}, v=v, K=K)


# ---- what a program has in hand ----------------------------------------------------------------------------------
def factors(n):
    """The pair n1 <= n2 nearest to a square with n1 * n2 = n that btc_transform takes, or None."""
    n1 = next(i for i in range(min(128, math.isqrt(n)), 0, -1) if n % i == 0)
    return (n1, n // n1) if n // n1 <= 256 else None


def _bits(K):
    return (K - 1).bit_length()


def _chunks(n_in, v):
    return -(-n_in // v)


def _codebook(g, v, K):
    """K distinct sign patterns of v bits; every pattern equally often where K > 2^v."""
    n = 1 << v
    cb = torch.randperm(n, generator=g, device="cuda")[:K]
    if K > n:
        cb = cb.repeat(-(-K // n))[:K][torch.randperm(K, generator=g, device="cuda")]
    return cb.to(torch.int32)


def _indices(g, out, n_in, v, K, dist):
    shape = (out, _chunks(n_in, v))
    if dist == "uniform":
        return torch.randint(0, K, shape, generator=g, device="cuda", dtype=torch.int32)
    w = torch.arange(1, K + 1, device="cuda", dtype=torch.float64).pow(-1.1)
    cdf = (torch.cumsum(w, 0) / w.sum()).float()
    u = torch.rand(shape, generator=g, device="cuda")
    return torch.searchsorted(cdf, u, out_int32=True).clamp_(max=K - 1)


class Matrix:
    """One compressed weight matrix."""

    def __init__(self, g, out, n_in, v, K, dist, codebook=None):
        self.s = B.btc_shape_init(out, n_in, v, K)
        self.packed = torch.empty(B.btc_packed_bytes(self.s) // 4, dtype=torch.int32, device="cuda")
        B.btc_pack(self.s, _indices(g, out, n_in, v, K, dist), self.packed, torch.zeros(16, dtype=torch.uint8, device="cuda"))
        self.codebook = _codebook(g, v, K) if codebook is None else codebook
        self.alpha = (torch.randn(out, generator=g, device="cuda") * 0.02).abs_()
        self.mu = torch.randn(out, generator=g, device="cuda") * 0.002


def _activations(g, rows, n, dtype, outliers=False):
    x = torch.randn((rows, n), generator=g, device="cuda")
    if outliers:      # one channel in a hundred twenty times as large, the same ones in every row
        x[:, torch.randperm(n, generator=g, device="cuda")[: n // 100]] *= 20.0
    return x.to(TORCH[dtype])


class Transform:
    """The activation transform of rows of n channels: signs and two well-conditioned Kronecker factors."""

    def __init__(self, g, n):
        self.n1, self.n2 = factors(n)
        rng = np.random.default_rng(int(torch.randint(0, 1 << 30, (1,), generator=g, device="cuda")))
        self.signs = torch.randint(-2 ** 31, 2 ** 31, (-(-n // 32),), generator=g, device="cuda").to(torch.int32)
        self.P1, self.P2 = (torch.from_numpy((np.linalg.qr(rng.standard_normal((m, m)))[0] +
                                              0.02 * rng.standard_normal((m, m))).astype(np.float32)).cuda()
                            for m in (self.n1, self.n2))
        nbytes = B.btc_transform_prepared_bytes(self.n1, self.n2)
        self.prepared = torch.empty(nbytes, dtype=torch.uint8, device="cuda") if nbytes else None
        if nbytes:
            B.btc_transform_prepare(self.n1, self.n2, self.P1, self.P2, self.prepared)


def _projections(case):
    """(rows, columns) of q, k, v, o, gate, up, down."""
    d, kv, ff = case["d"], case["kv"], case["ff"]
    return [(d, d), (kv, d), (kv, d), (d, d), (ff, d), (ff, d), (d, ff)]


INPUT_OF = [0, 0, 0, 1, 2, 2, 3]      # which of the layer's four inputs each projection reads


def _inputs(case):
    return [case["d"], case["d"], case["d"], case["ff"]]


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return globals()["_prepare_" + case["kind"]](case, g)


def run(state):
    return globals()["_run_" + state["kind"]](state)


def _prepare_gemv(c, g):
    m = Matrix(g, c["out"], c["in"], c["v"], c["K"], c["dist"])
    return dict(kind="gemv", m=m, x=_activations(g, c["batch"], c["in"], "f16", c["outliers"]), batch=c["batch"],
                y=torch.empty((c["batch"], c["out"]), dtype=TORCH[c["y"]], device="cuda"), y_dtype=BTC[c["y"]],
                ws=torch.zeros(B.btc_workspace_bytes(m.s, c["batch"], False), dtype=torch.uint8, device="cuda"))


def _run_gemv(st):
    m = st["m"]
    B.btc_gemv(m.s, m.packed, m.codebook, m.alpha, m.mu, st["x"], st["batch"], st["y"], st["y_dtype"], st["ws"])
    return st["y"]


def _prepare_decode(c, g):
    codebook = _codebook(g, c["v"], c["K"])
    proj = _projections(c)
    starts = np.cumsum([0] + [-(-out // 8) * 8 for out, _ in proj]).tolist()      # every output starts on 16 bytes
    y = torch.zeros((c["layers"], starts[-1]), dtype=torch.float16, device="cuda")
    layers, need = [], 16
    for i in range(c["layers"]):
        ms = [Matrix(g, out, n_in, c["v"], c["K"], c["dist"], codebook) for out, n_in in proj]
        ys = [y[i, a:a + out] for a, (out, _) in zip(starts, proj)]
        xs = [_activations(g, 1, n, "f16") for n in _inputs(c)]
        ts = [Transform(g, n) for n in _inputs(c)] if c["transform"] else None
        groups = []
        for a, b in ((0, 3), (3, 4), (4, 6), (6, 7)):
            part = ms[a:b]
            groups.append(dict(shapes=[m.s for m in part], packed=[m.packed for m in part], codebook=[m.codebook for m in part],
                               alpha=[m.alpha for m in part], mu=[m.mu for m in part], y=ys[a:b]))
        layers.append(dict(groups=groups, xs=xs, ts=ts))
        for m in ms:
            need = max(need, B.btc_workspace_bytes(m.s, 1, False), B.btc_gemv_transformed_workspace_bytes(m.s))
    st = dict(kind="decode", layers=layers, y=y, graph=None,
              xt=torch.empty(c["ff"], dtype=torch.float16, device="cuda"),
              ws=torch.zeros(need, dtype=torch.uint8, device="cuda"))
    if c["graph"]:
        _decode(st)      # once by itself, then recorded
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _decode(st)
        st["graph"] = graph
    return st


def _decode(st):
    for layer in st["layers"]:
        for i, p in enumerate(layer["groups"]):
            x, t = layer["xs"][i], layer["ts"][i] if layer["ts"] else None
            n = len(p["y"])
            if t is None and n == 1:
                B.btc_gemv(p["shapes"][0], p["packed"][0], p["codebook"][0], p["alpha"][0], p["mu"][0], x, 1, p["y"][0],
                           B.BTC_F16, st["ws"])
            elif t is None:
                B.btc_gemv_multi_shapes(p["shapes"], p["packed"], p["codebook"], p["alpha"], p["mu"], x, p["y"],
                                        B.BTC_F16, st["ws"])
            elif all(s.out == p["shapes"][0].out for s in p["shapes"]):
                B.btc_gemv_transformed_multi(p["shapes"][0], p["packed"], p["codebook"], p["alpha"], p["mu"], x, t.n1, t.n2,
                                             t.signs, t.P1, t.P2, t.prepared, p["y"], B.BTC_F16, st["ws"])
            else:      # keys and values with fewer rows: they read the transformed row that the queries' call hands out
                B.btc_gemv_transformed(p["shapes"][0], p["packed"][0], p["codebook"][0], p["alpha"][0], p["mu"][0], x, t.n1,
                                       t.n2, t.signs, t.P1, t.P2, t.prepared, p["y"][0], B.BTC_F16, st["ws"], xt_out=st["xt"])
                B.btc_gemv_multi_shapes(p["shapes"][1:], p["packed"][1:], p["codebook"][1:], p["alpha"][1:], p["mu"][1:],
                                        st["xt"], p["y"][1:], B.BTC_F16, st["ws"])


def _run_decode(st):
    if st["graph"] is not None:
        st["graph"].replay()
    else:
        _decode(st)
    return st["y"]


def _prepare_groups(c, g):
    out, n_in, G = c["out"], c["in"], c["ngroups"]
    m = Matrix(g, out, n_in, c["v"], c["K"], c["dist"])
    words = -(-2 * n_in // 32)
    u = torch.rand((out, words, 16), generator=g, device="cuda")
    of = (u * u * G).to(torch.int32).clamp_(max=G - 1)      # the groups of large weights have fewer members
    of <<= torch.arange(0, 32, 2, device="cuda", dtype=torch.int32)
    return dict(kind="groups", m=m, G=G, map=of.sum(2, dtype=torch.int32),
                alpha=(torch.randn((out, G), generator=g, device="cuda") * 0.02).abs_(),
                mu=torch.randn((out, G), generator=g, device="cuda") * 0.002, x=_activations(g, 1, n_in, "f16"),
                y=torch.empty(out, dtype=TORCH[c["y"]], device="cuda"), y_dtype=BTC[c["y"]])


def _run_groups(st):
    m = st["m"]
    B.btc_gemv_groups(m.s, m.packed, m.codebook, st["alpha"], st["mu"], st["map"], st["G"], st["x"], st["y"], st["y_dtype"])
    return st["y"]


def _prepare_gemm(c, g):
    M, codebook = c["rows"], _codebook(g, c["v"], c["K"])
    ms = [Matrix(g, out, n_in, c["v"], c["K"], c["dist"], codebook) for out, n_in in _projections(c)]
    need = max(B.btc_workspace_bytes(m.s, M, True) for m in ms)
    return dict(kind="gemm", ms=ms, M=M, x_dtype=BTC[c["x"]], y_dtype=BTC[c["y"]],
                xs=[_activations(g, M, n, c["x"]) for n in _inputs(c)],
                ts=[Transform(g, n) for n in _inputs(c)] if c["transform"] else None,
                xt=torch.empty(M * max(_inputs(c)), dtype=TORCH[c["x"]], device="cuda"),
                ys=[torch.empty((M, m.s.out), dtype=TORCH[c["y"]], device="cuda") for m in ms],
                ws=torch.empty(need, dtype=torch.uint8, device="cuda"))


def _run_gemm(st):
    M, last = st["M"], -1
    for m, i, y in zip(st["ms"], INPUT_OF, st["ys"]):
        x = st["xs"][i]
        if st["ts"] is not None:
            if i != last:      # one transform for all the projections that read this input
                t, last = st["ts"][i], i
                B.btc_transform(x, st["x_dtype"], M, t.n1, t.n2, t.signs, t.P1, t.P2, st["xt"], st["x_dtype"])
            x = st["xt"]
        B.btc_gemm(m.s, m.packed, m.codebook, m.alpha, m.mu, x, st["x_dtype"], M, y, st["y_dtype"], st["ws"])
    return st["ys"]


def _prepare_act(c, g):
    M, codebook = c["rows"], _codebook(g, c["v"], c["K"])
    ms = [Matrix(g, out, n_in, c["v"], c["K"], c["dist"], codebook) for out, n_in in _projections(c)]
    ws = torch.empty(max(B.btc_aq_workspace_bytes(m.s, M) for m in ms), dtype=torch.uint8, device="cuda")
    wsums = [torch.empty(m.s.out, device="cuda") for m in ms]      # a constant of each matrix
    for m, w in zip(ms, wsums):
        B.btc_weight_rowsums(m.s, m.packed, m.codebook, m.alpha, m.mu, w, ws)
    return dict(kind="act", ms=ms, wsums=wsums, M=M, bits=c["bits"], x_dtype=BTC[c["x"]], y_dtype=BTC[c["y"]], ws=ws,
                xs=[_activations(g, M, n, c["x"]) for n in _inputs(c)],
                qs=[torch.empty((M, n), dtype=torch.uint8, device="cuda") for n in _inputs(c)],
                los=[torch.empty(M, device="cuda") for _ in range(4)], steps=[torch.empty(M, device="cuda") for _ in range(4)],
                ys=[torch.empty((M, m.s.out), dtype=TORCH[c["y"]], device="cuda") for m in ms])


def _run_act(st):
    M, last = st["M"], -1
    for m, w, i, y in zip(st["ms"], st["wsums"], INPUT_OF, st["ys"]):
        q, lo, step = st["qs"][i], st["los"][i], st["steps"][i]
        if i != last:      # one quantisation for all the projections that read this input
            last = i
            B.btc_quantize_rows(st["xs"][i], st["x_dtype"], M, m.s.in_, st["bits"], q, lo, step)
        B.btc_gemm_aq(m.s, m.packed, m.codebook, m.alpha, m.mu, w, q, lo, step, M, y, st["y_dtype"], st["ws"])
    return dict(y=st["ys"], q=st["qs"], lo=st["los"], step=st["steps"])


def _prepare_cluster(c, g):
    v, K = c["v"], c["K"]
    s = B.btc_shape_init(c["out"], c["in"], v, K)
    N = s.out * s.nchunks
    codebook = _codebook(g, v, K)
    # sign vectors around the centroids, three elements flipped with probability 0.4 each; one vector in five any pattern
    vectors = codebook[torch.randint(0, K, (N,), generator=g, device="cuda")]
    for _ in range(3):
        flip = torch.ones(N, dtype=torch.int32, device="cuda") << torch.randint(0, v, (N,), generator=g, device="cuda").to(torch.int32)
        vectors = torch.where(torch.rand(N, generator=g, device="cuda") < 0.4, vectors ^ flip, vectors)
    anything = torch.randint(0, 1 << v, (N,), generator=g, device="cuda", dtype=torch.int32)
    vectors = torch.where(torch.rand(N, generator=g, device="cuda") < 0.2, anything, vectors)
    return dict(kind="cluster", s=s, N=N, v=v, K=K, vectors=vectors, codebook=codebook, new=torch.empty_like(codebook),
                z=torch.empty(N, dtype=torch.int32, device="cuda"), dist2=torch.empty(N, dtype=torch.int32, device="cuda"),
                packed=torch.empty(B.btc_packed_bytes(s) // 4, dtype=torch.int32, device="cuda"),
                ws=torch.zeros(max(16, B.btc_update_workspace_bytes(v, K)), dtype=torch.uint8, device="cuda"),
                ws_pack=torch.zeros(16, dtype=torch.uint8, device="cuda"))


def _run_cluster(st):
    st["new"].copy_(st["codebook"])      # the old centroids stay for the next comparison
    B.btc_assign(st["vectors"], st["N"], st["v"], st["codebook"], st["K"], st["z"], st["dist2"])
    B.btc_update(st["vectors"], st["z"], st["N"], st["v"], st["new"], st["K"], st["ws"])
    B.btc_pack(st["s"], st["z"], st["packed"], st["ws_pack"])
    return dict(z=st["z"], dist2=st["dist2"], codebook=st["new"], packed=st["packed"])


# ---- what a pass cannot do without -------------------------------------------------------------------------------
def _weight_bytes(out, n_in, v, K):
    return out * (-(-_chunks(n_in, v) * _bits(K) // 32) * 4 + 8)


def work(case):
    c, kind = case, case["kind"]
    v, K = c["v"], c["K"]
    if kind in ("gemv", "groups"):
        out, n_in, rows = c["out"], c["in"], c.get("batch", 1)
        nbytes = _weight_bytes(out, n_in, v, K) + (4 << _bits(K)) + rows * (2 * n_in + SIZE[c["y"]] * out)
        if kind == "groups":
            nbytes += out * (-(-2 * n_in // 32) * 4 + 8 * (c["ngroups"] - 1))
        return dict(bytes=nbytes, flops=2 * rows * out * n_in)
    if kind == "cluster":
        N = c["out"] * _chunks(c["in"], v)
        # a vector read, its index and distance written; the indices packed; each different vector against each centroid
        return dict(bytes=12 * N + c["out"] * -(-_chunks(c["in"], v) * _bits(K) // 32) * 4 + 8 * K,
                    flops=2 * v * K * min(N, 1 << v))
    proj, n = _projections(c), _inputs(c)
    weights = sum(_weight_bytes(out, n_in, v, K) for out, n_in in proj)
    products = 2 * sum(out * n_in for out, n_in in proj)
    transforms = sum(2 * m * sum(factors(m)) for m in n) if c.get("transform") else 0
    per_transform = sum(m // 8 + 4 * sum(f * f for f in factors(m)) for m in n) if c.get("transform") else 0
    outs = sum(out for out, _ in proj)
    if kind == "decode":
        return dict(bytes=c["layers"] * (weights + 2 * sum(n) + 2 * outs + per_transform) + (4 << _bits(K)),
                    flops=c["layers"] * (products + transforms))
    M = c["rows"]
    nbytes = weights + (4 << _bits(K)) + per_transform + M * (2 * sum(n) + SIZE[c["y"]] * outs)
    if kind == "act":
        nbytes += M * (sum(n) + 32) + 4 * outs      # the codes, offsets and steps written; the row sums of the weights
    return dict(bytes=nbytes, flops=M * (products + transforms))


def tolerance(case):
    """fp32 results are sums of exact products in fp32; 16-bit results are those rounded once.  Behind a transform the
    activations themselves are rounded to 16 bits, where two correct sums can fall on different sides."""
    if case["kind"] == "cluster":
        return "exact"
    y = case.get("y", "f16")
    rel = {"f32": 1e-5, "f16": 1e-3, "bf16": 1e-2}[y]
    if case.get("transform"):
        rel = max(rel, {"f16": 1e-3, "bf16": 4e-3}[case.get("x", "f16")])
    return {"rel": rel}
