"""The work that users of this library have it do, as cases that can be timed and checked.

Every case goes through the public binding ``paper_2406_05981_amd.shiftadd``.
Three kinds of program use it:

* an inference program: one call per linear layer on weights that were packed
  once (``layer``), or, for a token step, the projections of a decoder layer
  captured in a HIP graph and replayed (``decoder``);
* the offline reparameterization: fp32 weights to packed planes (``quantize``);
* the bit allocation: the criterion of a layer from its calibration
  activations (``criterion``).

Inputs follow the synthetic layers of ``workloads``: fair-coin planes,
exponents uniform over the workload's range, N(0, 1) activations with 1% of the
channels x20, weights N(0, 0.02^2) with a per-row log-normal factor.
"""
import math

import torch

import paper_2406_05981_amd.shiftadd as sa

DEV = "cuda"

# The projections of one decoder layer with the bit widths of the mixed 7B layer
# set: (rows, columns, planes, index of the input it reads).  q, k and v read
# one activation, up and gate another.
DECODER = (
    (4096, 4096, 2, 0), (4096, 4096, 2, 0), (4096, 4096, 4, 0), (4096, 4096, 4, 1),
    (11008, 4096, 3, 2), (11008, 4096, 3, 2), (4096, 11008, 3, 3),
)


def _layer(name, N, K, q, B, layout="row", G=128, f16=False, row_block=0, terms=0, lo=-10):
    return dict(name=name, kind="layer", layout=layout, N=N, K=K, q=q, B=B, G=G, f16=f16,
                row_block=row_block, terms=terms, exp_lo=lo, exp_hi=-3)


def listed():
    return [
        # a token step of a small model: one projection, a launch's latency
        _layer("proj_768_b1", 768, 768, 3, 1, lo=-8),
        # a token step of a 7B model: an attention projection
        _layer("attn_4096_b1", 4096, 4096, 3, 1),
        # a decoder layer's seven projections in one replayed graph, as a serving
        # loop runs them: a single sequence, and sixteen decoded together
        dict(name="decoder_b1", kind="decoder", B=1, G=128),
        dict(name="decoder_b16", kind="decoder", B=16, G=128),
        # the two MLP projections of a 70B model: one token, and eight sequences
        # with binary16 outputs
        _layer("mlp_up_70b_b1", 28672, 8192, 3, 1, lo=-12),
        _layer("mlp_down_70b_b8_f16", 8192, 28672, 3, 8, f16=True, lo=-12),
        # a chunk of a prompt near the largest batch the library takes, ragged rows
        _layer("prompt_b250", 11003, 4096, 3, 250),
        # the other scale layouts: column-wise factors for a few sequences,
        # block-wise factors (the paper's N/8 rows) for one token, additive factors
        # of two terms for a decoding batch
        _layer("colwise_attn_b4", 4096, 4096, 3, 4, layout="col"),
        _layer("blockwise_up_b1", 11008, 4096, 2, 1, layout="blk", row_block=1376),
        _layer("terms_down_b16", 4096, 11008, 2, 16, layout="terms", terms=2),
        # reparameterization of one projection: planes, exponents, packed planes
        dict(name="quantize_attn_q3", kind="quantize", N=4096, K=4096, q=3, G=128, cycles=2,
             terms=0),
        # the criterion of one projection over 128 calibration sequences of 2048
        dict(name="criterion_attn", kind="criterion", N=4096, K=4096, T=262144),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["layer"] * 7 + ["decoder", "quantize", "criterion"])
    if kind == "decoder":
        return dict(kind="decoder", B=rng.randint(2, 15), G=rng.choice([128, 128, 256]))
    if kind == "quantize":
        return dict(kind="quantize", N=_log_uniform(rng, 512, 4000),
                    K=128 * _log_uniform(rng, 4, 32), q=rng.choice([2, 3, 4]), G=128,
                    cycles=rng.choice([1, 2, 3]), terms=rng.choice([0, 0, 2]))
    if kind == "criterion":
        return dict(kind="criterion", N=_log_uniform(rng, 512, 4096),
                    K=128 * _log_uniform(rng, 4, 32), T=32 * _log_uniform(rng, 64, 4096))
    layout = rng.choice(["row"] * 4 + ["col", "blk", "terms"])
    G = rng.choice([128, 128, 128, 256]) if layout in ("row", "terms") else 128
    # rows of every residue; columns a multiple of the group
    while True:
        N = _log_uniform(rng, 200, 28672)
        K = G * _log_uniform(rng, 512 // G, 28672 // G)
        if N * K <= 28672 * 8192:
            break
    if rng.random() < 0.5:
        N = 16 * max(N // 16, 1)
    B = rng.choice([1, 1, _log_uniform(rng, 2, 16), _log_uniform(rng, 2, 16),
                    _log_uniform(rng, 17, 256)])
    while B > 16 and N * K * B > 28672 * 8192 * 16:
        B //= 2
    q = rng.choice([2, 3, 3, 4])
    row_block = rng.choice([-(-N // 8), 8, 64, 256]) if layout == "blk" else 0
    terms = rng.choice([1, 2, 2, 3]) if layout == "terms" else 0
    c = _layer("", N, K, q, B, layout=layout, G=G, f16=layout == "row" and rng.random() < 0.3,
               row_block=row_block, terms=terms, lo=rng.choice([-8, -10, -12]))
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(0x5A11 + int(seed))
    return g


def _signs(g, q, N, K):
    s = torch.randint(0, 2, (q, N, K), dtype=torch.int8, device=DEV, generator=g)
    return s.mul_(2).sub_(1)


def _exps(g, shape, lo, hi):
    return torch.randint(lo, hi + 1, shape, dtype=torch.int8, device=DEV, generator=g)


def _x(g, B, K):
    """fp16 activations: N(0, 1), the same 1% of channels x20 in every row."""
    x = torch.randn((B, K), device=DEV, generator=g)
    out = torch.randperm(K, device=DEV, generator=g)[:round(0.01 * K)]
    x[:, out] *= 20.0
    return x.to(torch.float16)


def _layer_weights(c, g):
    """Planes and factors of one layer, as the reparameterization hands them over."""
    q, N, K = c["q"], c["N"], c["K"]
    signs = _signs(g, q, N, K)
    lo, hi = c["exp_lo"], c["exp_hi"]
    if c["layout"] == "col":
        return signs, _exps(g, (q, K), lo, hi), None
    if c["layout"] == "blk":
        return signs, _exps(g, (q, -(-N // c["row_block"]), K // 8), lo, hi), None
    if c["layout"] == "terms":
        # a greedy expansion: each term 1 to 3 binades below the one before, later
        # terms of either sign, one in eight absent
        T, shape = c["terms"], (q, N, K // c["G"])
        e = [_exps(g, shape, lo, hi)]
        ts = [torch.ones(shape, dtype=torch.int8, device=DEV)]
        for _ in range(1, T):
            e.append(e[-1] - _exps(g, shape, 1, 3))
            sg = _exps(g, shape, 0, 1) * 2 - 1
            ts.append(sg * (_exps(g, shape, 0, 7) > 0).to(torch.int8))
        return signs, torch.stack(e, -1).contiguous(), torch.stack(ts, -1).contiguous()
    return signs, _exps(g, (q, N, K // c["G"]), lo, hi), None


def _decoder_layers(c, g):
    """(N, K, q, planes, exponents, activation) of each projection in turn."""
    xs = [_x(g, c["B"], K) for K in (4096, 4096, 4096, 11008)]
    for N, K, q, i in DECODER:
        yield N, K, q, _signs(g, q, N, K), _exps(g, (q, N, K // c["G"]), -10, -3), xs[i]


def _fp_weights(g, N, K):
    rows = torch.exp(0.25 * torch.randn((N, 1), device=DEV, generator=g))
    w = torch.randn((N, K), device=DEV, generator=g) * (0.02 * rows)
    w[torch.rand((N, K), device=DEV, generator=g) < 1e-3] *= 10.0
    return w


def _calibration(c, g):
    """fp16 [K][T]: one row per channel, some channels larger than others."""
    x = torch.randn((c["K"], c["T"]), device=DEV, dtype=torch.float16, generator=g)
    return x.mul_(torch.exp(0.5 * torch.randn((c["K"], 1), device=DEV, generator=g)).half())


def prepare(case, seed):
    c, g = case, _gen(seed)
    s = dict(c)
    if c["kind"] == "layer":
        signs, s["exps"], s["tsg"] = _layer_weights(c, g)
        s["packed"] = sa.pack_weights(signs)
        s["x"] = _x(g, c["B"], c["K"])
        s["y"] = torch.empty((c["B"], c["N"]), device=DEV,
                             dtype=torch.float16 if c["f16"] else torch.float32)
    elif c["kind"] == "decoder":
        s["layers"] = []
        for N, K, q, signs, exps, x in _decoder_layers(c, g):
            y = torch.empty((c["B"], N), dtype=torch.float32, device=DEV)
            s["layers"].append((x, sa.pack_weights(signs), exps, q, N, K, c["G"], c["B"], y))
        # the step is captured once and replayed for every token; the activations
        # and outputs keep their buffers
        torch.cuda.synchronize()
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            for a in s["layers"]:
                sa.sa_shiftadd_gemm(*a)
        stream.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"], stream=stream):
            for a in s["layers"]:
                sa.sa_shiftadd_gemm(*a)
    elif c["kind"] == "quantize":
        s["w"] = _fp_weights(g, c["N"], c["K"])
    else:
        s["w"] = _fp_weights(g, c["N"], c["K"])
        s["x"] = _calibration(c, g)
    return s


def run(s):
    if s["kind"] == "layer":
        q, N, K, B, y = s["q"], s["N"], s["K"], s["B"], s["y"]
        if s["layout"] == "col":
            sa.sa_shiftadd_gemm_colwise(s["x"], s["packed"], s["exps"], q, N, K, B, y)
        elif s["layout"] == "blk":
            sa.sa_shiftadd_gemm_blockwise(s["x"], s["packed"], s["exps"], q, N, K, s["row_block"],
                                          B, y)
        elif s["layout"] == "terms":
            sa.sa_shiftadd_gemm_terms(s["x"], s["packed"], s["exps"], s["tsg"], q, N, K, s["G"],
                                      s["terms"], B, y)
        elif s["f16"]:
            sa.sa_shiftadd_gemm_f16(s["x"], s["packed"], s["exps"], q, N, K, s["G"], B, y)
        else:
            sa.sa_shiftadd_gemm(s["x"], s["packed"], s["exps"], q, N, K, s["G"], B, y)
        return y
    if s["kind"] == "decoder":
        s["graph"].replay()
        return [a[-1] for a in s["layers"]]
    if s["kind"] == "quantize":
        if s["terms"]:
            signs, exps, tsg = sa.quantize_bcq_terms(s["w"], s["q"], s["G"], s["cycles"], s["terms"])
            return signs, exps, tsg, sa.pack_weights(signs)
        signs, exps = sa.quantize_bcq(s["w"], s["q"], s["G"], s["cycles"])
        return signs, exps, sa.pack_weights(signs)
    C, norm, std, d = sa.bit_criterion(s["w"], s["x"])
    return C, norm, std, d


# ------------------------------------------------------------------ what a pass cannot do without

def _layer_work(q, N, K, B, factor_bytes, out_bytes=4):
    """Packed planes, factors, activations and outputs once; the multiply-adds
    of one product with the summed weight."""
    return q * N * K // 8 + factor_bytes + 2 * B * K + out_bytes * B * N, 2 * N * K * B


def work(case):
    c = case
    if c["kind"] == "layer":
        q, N, K, B = c["q"], c["N"], c["K"], c["B"]
        if c["layout"] == "col":
            fb = q * K
        elif c["layout"] == "blk":
            fb = q * -(-N // c["row_block"]) * (K // 8)
        elif c["layout"] == "terms":
            fb = 2 * c["terms"] * q * N * (K // c["G"])
        else:
            fb = q * N * (K // c["G"])
        b, f = _layer_work(q, N, K, B, fb, 2 if c["f16"] else 4)
        return {"bytes": b, "flops": f}
    if c["kind"] == "decoder":
        w = [_layer_work(q, N, K, c["B"], q * N * (K // c["G"])) for N, K, q, _ in DECODER]
        return {"bytes": sum(b for b, _ in w), "flops": sum(f for _, f in w)}
    N, K = c["N"], c["K"]
    if c["kind"] == "quantize":
        q, T = c["q"], c["cycles"]
        fb = q * N * K // c["G"] * (2 * c["terms"] if c["terms"] else 1)
        # greedy residuals, then per cycle B^T w and the nearest of 2^q values
        return {"bytes": 4 * N * K + q * N * K + q * N * K // 8 + fb,
                "flops": N * K * (2 * q + T * (q + 2 ** (q + 1)))}
    T = c["T"]
    return {"bytes": 2 * K * T + 4 * N * K + 8 * K,
            "flops": K * (K + 1) * T + K ** 3 // 3 + 4 * N * K}


# ------------------------------------------------------------------ the same in 64 bits

def _pow2(e):
    return torch.exp2(e.double())


def _matmul64(x, signs, factor_of):
    """sum over planes of x (signs * factor)^T, rows in slices."""
    q, N, K = signs.shape
    y = torch.zeros((x.shape[0], N), dtype=torch.float64, device=DEV)
    x = x.double()
    step = max(1, (1 << 27) // K)
    for n in range(0, N, step):
        for i in range(q):
            w = signs[i, n:n + step].double() * factor_of(i, n, min(n + step, N))
            y[:, n:n + step] += torch.matmul(x, w.t().contiguous())
    return y


def exact(case, seed):
    c, g = case, _gen(seed)
    if c["kind"] == "layer":
        signs, exps, tsg = _layer_weights(c, g)
        x = _x(g, c["B"], c["K"])
        if c["layout"] == "col":
            f = lambda i, a, b: _pow2(exps[i])[None, :]  # noqa: E731
        elif c["layout"] == "blk":
            f = lambda i, a, b: _pow2(exps[i]).index_select(  # noqa: E731
                0, torch.arange(a, b, device=DEV) // c["row_block"]).repeat_interleave(8, 1)
        elif c["layout"] == "terms":
            f = lambda i, a, b: (_pow2(exps[i, a:b]) * tsg[i, a:b].double()).sum(  # noqa: E731
                -1).repeat_interleave(c["G"], 1)
        else:
            f = lambda i, a, b: _pow2(exps[i, a:b]).repeat_interleave(c["G"], 1)  # noqa: E731
        return _matmul64(x, signs, f)
    if c["kind"] == "decoder":
        return [_matmul64(x, signs,
                          lambda i, a, b, e=exps: _pow2(e[i, a:b]).repeat_interleave(c["G"], 1))
                for N, K, q, signs, exps, x in _decoder_layers(c, g)]
    if c["kind"] == "quantize":
        return None  # planes and exponents: whole numbers
    w = _fp_weights(g, c["N"], c["K"]).double()
    x = _calibration(c, g)
    H = torch.zeros((c["K"], c["K"]), dtype=torch.float64, device=DEV)
    for t in range(0, c["T"], 16384):
        xt = x[:, t:t + 16384].double()
        H += torch.matmul(xt, xt.t().contiguous())
    H += 0.01 * H.diagonal().mean() * torch.eye(c["K"], dtype=torch.float64, device=DEV)
    # the diagonal of the Cholesky factor of the inverse, from the factor of the
    # matrix with rows and columns reversed: reciprocals in reverse order
    L = torch.linalg.cholesky(H.flip(0, 1).contiguous())
    d = 1.0 / L.diagonal().flip(0)
    s = w / d[None, :]
    norm, std = float(s.square().sum().sqrt()), float(s.std(correction=0))
    return norm * std * std, norm, std, d


def tolerance(case):
    if case["kind"] == "quantize":
        # fp64 decisions: a residual or a scale on a boundary may fall either way
        return {"rel": 0.0, "differ": 1e-6}
    if case["kind"] == "criterion":
        # the Gram matrix is summed in fp32 over up to 262144 tokens
        return {"rel": 2e-5, "max": 2e-4}
    if case["kind"] == "layer" and case["f16"]:
        # the result rounded to binary16: another order of the fp32 sums moves a
        # value by one unit in the last place here and there
        return {"rel": 2e-4, "max": 2e-3}
    # fp32 sums of exact products over up to q * K terms
    return {"rel": 2e-6, "max": 2e-5}
