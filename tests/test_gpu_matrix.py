"""GPU parity of the layer's matrix-core forms at the sizes where their tiling
can go wrong, against the CPU oracle.

Bound: the binary16 form's products are exact and the fp8 split is off by at
most 2^-28 of the largest of 32 columns per activation, so 2 * 2^-24 of
sum|terms|; the fp32 additions of one output form chains of at most
q * K / 128 + 32 terms of which each rounds by 2^-24 of a partial sum."""
import sys

import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():  # pragma: no cover - CPU-only environment
    pytest.skip("no GPU", allow_module_level=True)
sa = pytest.importorskip("paper_2406_05981_amd.shiftadd")


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# kernels of sa_plan_gemm_matrix: block-scaled; binary16, columns shared; activations shared
MX, SPLIT, TILE = 1, 2, 3


def runs(c, kernel, row_tiles=None, col_tiles=None, shares=None):
    """The call runs this kernel (with this geometry)."""
    p = sa.sa_plan_gemm_matrix(c["q"], c["N"], c["K"], c["G"], c["B"], c.get("T", 0))
    say(f"  {p}")
    assert p["kernel"] == kernel
    for name, want in (("row_tiles", row_tiles), ("col_tiles", col_tiles),
                       ("column_shares", shares)):
        assert want in (None, p[name]), name
    return c


def layer(c, exps=None):
    y = torch.full((c["B"], c["N"]), float("nan"), dtype=torch.float32, device="cuda")
    sa.sa_shiftadd_gemm(dev(c["x"]), sa.pack_weights(dev(c["signs"])),
                        dev(c["exps"]) if exps is None else exps, c["q"], c["N"], c["K"], c["G"],
                        c["B"], y)
    torch.cuda.synchronize()
    return y.cpu().numpy().astype(np.float64)


def check(y, c, what):
    y_ref, a_ref = oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], c["G"])
    bound = (64 + c["q"] * c["K"] / 128) * 2.0 ** -24
    worst = float((np.abs(y - y_ref) / np.where(a_ref > 0, a_ref, 1)).max())
    say(f"  {what}: max |y-y_ref|/sum|terms| = {worst:.3e} (bound {bound:.1e})")
    assert np.isfinite(y).all() and worst <= bound, what
    assert (y[a_ref == 0] == 0).all(), what


def norm_error(y, ref):
    return float(np.sqrt(np.square(y - ref).sum() / np.square(ref).sum()))


def table_batch(c):
    """The layer on the batch table kernel, by the block-wise entry point with
    blocks of one row."""
    q, N, K, B = c["q"], c["N"], c["K"], c["B"]
    blk = np.repeat(c["exps"], c["G"] // 8, axis=2)
    y = torch.full((B, N), float("nan"), dtype=torch.float32, device="cuda")
    sa.sa_shiftadd_gemm_blockwise(dev(c["x"]), sa.pack_weights(dev(c["signs"])), dev(blk), q, N, K,
                                  1, B, y)
    torch.cuda.synchronize()
    return y.cpu().numpy().astype(np.float64)


# (q, N, K, G, B), row tiles of a wave, waves that share the columns: partial
# 512-column groups (1 to 3 blocks), fewer groups than waves with one and several
# row sets, one and several groups a wave, ragged row and 64-row tiles, 1 to 8 row
# tiles, every batch that fills a column tile in part
SMALL = [
    ((4, 1, 1152, 128, 2), 1, 4), ((1, 15, 3328, 128, 2), 1, 8), ((1, 16, 3200, 128, 2), 1, 8),
    ((4, 17, 3328, 128, 3), 1, 8), ((3, 300, 4096, 4096, 4), 1, 8),
    ((4, 4150, 256, 128, 2), 1, 1), ((2, 9597, 384, 128, 2), 1, 1),
    ((1, 43317, 384, 128, 2), 2, 1), ((4, 8366, 768, 128, 2), 1, 2),
    ((3, 4157, 1152, 128, 2), 1, 4), ((3, 5000, 4096, 256, 4), 2, 8),
    ((3, 4170, 2176, 128, 5), 2, 8), ((4, 2244, 5248, 128, 6), 1, 8),
    ((4, 8102, 1280, 128, 5), 1, 4), ((3, 11019, 1408, 1408, 7), 2, 4),
    ((2, 36083, 768, 128, 5), 3, 2), ((3, 44555, 512, 128, 5), 2, 1),
    ((4, 2300, 8320, 128, 8), 1, 8), ((4, 2300, 12288, 12288, 8), 1, 8),
    ((1, 33186, 1152, 128, 8), 5, 4), ((2, 12001, 2304, 256, 7), 3, 8),
    ((1, 29508, 2176, 128, 8), 8, 8),
]


@pytest.mark.parametrize("shape,tiles,shares", SMALL)
def test_small_batch(shape, tiles, shares):
    q, N, K, G, B = shape
    say(f"matrix form q={q} N={N} K={K} G={G} B={B}")
    c = workloads.random_case(q, N, K, G, B, seed=31, exp_range=(-12, -3), outlier_fraction=0.01)
    runs(c, MX, tiles, 1 if B <= 4 else 2, shares)
    check(layer(c), c, c["name"])


# (q, N, K, G, B), kernel, row tiles, column tiles, column shares.  Columns shared by
# waves: 1 to 4 row tiles, 1 to 8 shares, a partial last group, several groups a
# wave, ragged rows and batch; activations shared in LDS: 1, 2 and 4 column tiles, 4
# and 2 row tiles, every plane count of 4 column tiles, exponents that load as a word
# (G = 128, K % 512 == 0) and by the byte, a last group of one block.
LARGE = [
    ((3, 4090, 4096, 128, 16), SPLIT, 1, 1, 8), ((4, 4096, 4224, 128, 16), SPLIT, 1, 1, 8),
    ((3, 4097, 8320, 128, 15), SPLIT, 1, 1, 8), ((1, 15556, 640, 128, 9), SPLIT, 1, 1, 2),
    ((2, 2876, 1152, 128, 9), SPLIT, 1, 1, 4), ((1, 23643, 512, 128, 9), SPLIT, 1, 1, 1),
    ((2, 7601, 2560, 128, 13), SPLIT, 2, 1, 8), ((3, 6000, 1664, 128, 17), SPLIT, 2, 1, 4),
    ((4, 5474, 2560, 128, 9), SPLIT, 2, 1, 8), ((3, 4100, 4096, 128, 32), SPLIT, 3, 1, 8),
    ((3, 6001, 4096, 256, 30), SPLIT, 3, 1, 8), ((1, 9000, 4096, 128, 13), SPLIT, 3, 1, 8),
    ((4, 5000, 4096, 4096, 20), SPLIT, 3, 1, 8), ((3, 4096, 4096, 128, 64), SPLIT, 4, 1, 8),
    ((2, 12730, 2688, 128, 9), SPLIT, 4, 1, 8), ((1, 13276, 1152, 128, 18), SPLIT, 4, 1, 4),
    ((2, 1509, 128, 128, 9), TILE, 4, 1, 1), ((4, 1384, 128, 128, 10), TILE, 4, 1, 1),
    ((2, 12001, 1152, 128, 16), TILE, 2, 1, 2), ((3, 2783, 256, 128, 9), TILE, 2, 1, 2),
    ((1, 3001, 1280, 128, 256), TILE, 4, 2, 1), ((3, 2000, 640, 128, 255), TILE, 4, 2, 1),
    ((4, 8001, 512, 128, 60), TILE, 4, 2, 1), ((2, 8000, 4480, 640, 17), TILE, 2, 2, 2),
    ((2, 2100, 4224, 384, 129), TILE, 2, 2, 2), ((3, 2300, 2048, 256, 250), TILE, 2, 2, 2),
    ((4, 4100, 1664, 128, 130), TILE, 2, 2, 2), ((1, 26486, 768, 128, 33), TILE, 4, 4, 1),
    ((2, 11007, 1024, 1024, 128), TILE, 4, 4, 1), ((3, 5003, 4096, 128, 250), TILE, 4, 4, 1),
    ((3, 11003, 1408, 128, 250), TILE, 4, 4, 1), ((4, 8000, 1152, 128, 100), TILE, 4, 4, 1),
]


@pytest.mark.parametrize("shape,kernel,row_tiles,col_tiles,shares", LARGE)
def test_large_batch(shape, kernel, row_tiles, col_tiles, shares):
    q, N, K, G, B = shape
    say(f"matrix form q={q} N={N} K={K} G={G} B={B}")
    c = workloads.random_case(q, N, K, G, B, seed=36, exp_range=(-12, -3), outlier_fraction=0.01)
    runs(c, kernel, row_tiles, col_tiles, shares)
    check(layer(c), c, c["name"])


# (q, N, K, G, B) that stay on the batch table kernel, its row-tile height: 32 and 64
# rows over one, two and three pieces at 1 to 5 planes, a wide plane count, ragged
# rows, eight batch quads
KEPT = [
    ((1, 4100, 128, 128, 2), 32), ((1, 5374, 1152, 128, 2), 32), ((2, 4952, 256, 256, 2), 32),
    ((2, 4218, 2432, 128, 2), 32), ((3, 4100, 2304, 128, 3), 32), ((4, 2547, 256, 128, 6), 32),
    ((1, 11297, 256, 128, 2), 64), ((2, 8977, 1152, 128, 3), 64), ((2, 4590, 2176, 128, 5), 64),
    ((3, 8323, 1152, 384, 3), 64), ((4, 8603, 640, 128, 3), 64), ((7, 4099, 1152, 128, 9), 64),
    ((5, 8201, 256, 128, 32), 64),
]


@pytest.mark.parametrize("shape,rows", KEPT)
def test_table_kernel_kept(shape, rows):
    q, N, K, G, B = shape
    say(f"table form q={q} N={N} K={K} G={G} B={B}")
    c = workloads.random_case(q, N, K, G, B, seed=43, exp_range=(-12, -3), outlier_fraction=0.01)
    runs(c, 0)
    assert sa.sa_plan_gemm(q, N, K, G, B)["rows_per_wg"] == rows
    check(layer(c), c, c["name"])


def terms_layer(c, shift=0):
    y = torch.full((c["B"], c["N"]), float("nan"), dtype=torch.float32, device="cuda")
    e, s = dev(c["exps"]).reshape(-1), dev(c["term_signs"]).reshape(-1)
    if shift:  # 2-byte aligned, not 8-byte
        be = torch.zeros(e.numel() + shift, dtype=torch.int8, device="cuda")
        bs = torch.zeros_like(be)
        be[shift:], bs[shift:] = e, s
        e, s = be[shift:], bs[shift:]
    sa.sa_shiftadd_gemm_terms(dev(c["x"]), sa.pack_weights(dev(c["signs"])), e, s, c["q"], c["N"],
                              c["K"], c["G"], c["T"], c["B"], y)
    torch.cuda.synchronize()
    return y.cpu().numpy().astype(np.float64)


# block-scaled: 1 to 4 terms, groups of several blocks, misaligned factors; binary16:
# 1 to 4 terms, 1 and 2 row tiles, 1 to 8 column shares, factors that load as
# words (two terms, G = 128, K % 512 == 0, aligned) and by the term's bytes
@pytest.mark.parametrize("q,N,K,G,B,T,shift,kernel,row_tiles", [
    (3, 1000, 4096, 128, 4, 2, 0, MX, 1), (4, 300, 2688, 384, 4, 3, 0, MX, 1),
    (2, 12000, 4096, 128, 2, 4, 4, MX, 3), (2, 9000, 4096, 128, 7, 1, 1, MX, 3),
    (4, 300, 7296, 384, 8, 3, 0, MX, 1), (4, 10800, 4096, 128, 5, 4, 0, MX, 3),
    (2, 4000, 4096, 128, 16, 2, 0, SPLIT, 1), (2, 4000, 4096, 128, 16, 2, 2, SPLIT, 1),
    (4, 1500, 8192, 128, 16, 2, 0, SPLIT, 1), (4, 5448, 1152, 128, 9, 2, 0, SPLIT, 1),
    (1, 12001, 4096, 256, 33, 2, 0, SPLIT, 2), (1, 16411, 384, 128, 18, 2, 0, SPLIT, 2),
    (3, 9000, 1408, 128, 16, 2, 0, SPLIT, 2), (3, 4170, 3200, 128, 16, 2, 2, SPLIT, 2),
    (1, 300, 3200, 128, 33, 1, 1, SPLIT, 1), (3, 4170, 384, 384, 140, 1, 0, SPLIT, 2),
    (2, 5003, 128, 128, 40, 3, 0, SPLIT, 1), (2, 4170, 384, 128, 140, 4, 4, SPLIT, 2)])
def test_additive(q, N, K, G, B, T, shift, kernel, row_tiles):
    say(f"additive matrix form q={q} N={N} K={K} G={G} B={B} T={T} shift={shift}")
    c = runs(workloads.terms_case(q, N, K, G, B, T, seed=37), kernel, row_tiles)
    c["exps"][0, 0, 0, -1], c["term_signs"][0, 0, 0, -1] = 127, 0  # no term, whatever its exponent
    y_ref, a_ref = oracle.shiftadd_gemm_terms(c["x"], c["signs"], c["exps"], c["term_signs"], G)
    bound = (64 + T * q * K / 128) * 2.0 ** -24
    y = terms_layer(c, shift)
    worst = float((np.abs(y - y_ref) / a_ref).max())
    say(f"  max |y-y_ref|/sum|terms| = {worst:.3e} (bound {bound:.1e})")
    assert np.isfinite(y).all() and worst <= bound


@pytest.mark.parametrize("q,N,K,B,kernel", [(2, 4096, 4096, 16, SPLIT),
                                           (2, 2300, 640, 250, TILE)])
def test_large_batch_extremes(q, N, K, B, kernel):
    """Not finite activations, subnormals, the int8 range of exponents."""
    say(f"large batch extremes q={q} N={N} K={K} B={B}")
    c = workloads.random_case(q, N, K, 128, B, seed=38, exp_range=(-128, 127))
    runs(c, kernel)
    x = c["x"].astype(np.float64) * 2.0 ** -12
    x[3] = 2.0 ** -24
    c["x"] = x.astype(np.float16)
    check(layer(c), c, "int8 range, subnormals")
    c["exps"] = np.clip(c["exps"], -10, -3)
    ref = oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], 128)[0]
    c["x"][0, 5] = np.nan
    c["x"][1, 600] = np.inf
    y = layer(c)
    s = np.where(c["signs"][:, :, 600] > 0, 1.0, -1.0).sum(0)
    assert np.isnan(y[0]).all()
    assert np.array_equal(np.isnan(y[1]), s == 0) and np.isinf(y[1][s != 0]).all()
    assert np.array_equal(y[1][s != 0] > 0, s[s != 0] > 0)
    assert np.abs(y[2:] - ref[2:]).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("B", [2, 4, 8])
def test_activation_ranges(B):
    """Block maxima from the smallest subnormal to the largest binary16 value,
    zero blocks, and wide ranges inside one block of 32 columns."""
    say(f"activation ranges B={B}")
    c = runs(workloads.random_case(3, 4500, 4096, 128, B, seed=32, exp_range=(-10, -2)), MX)
    x = c["x"].astype(np.float64)
    x[0, :32] = 2.0 ** -24
    x[0, 32:64] = 0.0
    x[0, 64:96] *= 2.0 ** -15
    x[0, 96:128] *= 2.0 ** -10
    x[0, 96] = 60000.0
    x[B - 1, 256:288] = np.linspace(-63000, 63000, 32)
    x[B - 1, 512:1024] *= 1e-6
    c["x"] = x.astype(np.float16)
    check(layer(c), c, "ranges")
    x[1, 2000] = 65504.0
    x[1, 2001] = -64000.0
    c["x"] = x.astype(np.float16)
    check(layer(c), c, "top of the range")


@pytest.mark.parametrize("B", [3, 8])
def test_not_finite_activations(B):
    """An infinity or NaN reaches every output of its batch row, and no other."""
    say(f"not finite B={B}")
    c = runs(workloads.random_case(2, 9000, 4096, 128, B, seed=33, exp_range=(-10, -2)), MX)
    x = c["x"].copy()
    x[0, 700] = np.inf
    x[1, 5] = np.nan
    x[2, 9], x[2, 4000] = np.inf, -np.inf
    ref = oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], 128)[0]
    c["x"] = x
    y = layer(c)
    s = np.where(c["signs"][:, :, 700] > 0, 1.0, -1.0).sum(0)  # two planes: both signs or neither
    assert np.array_equal(np.isnan(y[0]), s == 0)
    assert (y[0][s > 0] == np.inf).all() and (y[0][s < 0] == -np.inf).all()
    assert np.isnan(y[1]).all()
    p = c["signs"][:, :, 9] * np.array(1, np.int8), -c["signs"][:, :, 4000]
    t = np.concatenate(p).sum(0)  # four terms of +-inf
    assert np.array_equal(np.isnan(y[2]), np.abs(t) != 4)
    assert np.abs(y[3:] - ref[3:]).max(initial=0.0) <= 1e-4 * np.abs(ref).max()


@pytest.mark.parametrize("B", [2, 7])
def test_exponent_range(B):
    """Every int8 exponent, 127 and -128 among them, at an odd address."""
    say(f"exponent range B={B}")
    c = runs(workloads.random_case(3, 4500, 4096, 128, B, seed=34, exp_range=(-128, 127)), MX)
    c["x"] = (c["x"].astype(np.float64) * 2.0 ** -12).astype(np.float16)
    flat = c["exps"].reshape(-1)
    buf = torch.zeros(flat.size + 1, dtype=torch.int8, device="cuda")
    buf[1:] = dev(flat)
    check(layer(c, exps=buf[1:]), c, "int8 range")
    c["exps"] = np.minimum(c["exps"], np.int8(126))
    check(layer(c), c, "up to 126")
    c["exps"] = np.clip(c["exps"], -100, -90)
    check(layer(c), c, "small")


@pytest.mark.parametrize("q,N,K,G,B,kernel", [
    (3, 1000, 4096, 128, 4, MX), (4, 2300, 8448, 384, 8, MX), (3, 4090, 4096, 128, 16, SPLIT),
    (2, 2100, 4224, 384, 129, TILE), (3, 5003, 4096, 128, 250, TILE)])
def test_half_output_and_graph(q, N, K, G, B, kernel):
    """binary16 outputs are the fp32 ones rounded; replays of a captured call on
    new activations equal direct calls."""
    say(f"half output and graph q={q} N={N} K={K} B={B}")
    c = runs(workloads.random_case(q, N, K, G, B, seed=35, exp_range=(-10, -2)), kernel)
    packed, e = sa.pack_weights(dev(c["signs"])), dev(c["exps"])
    x = dev(c["x"])
    y32 = torch.empty((B, N), dtype=torch.float32, device="cuda")
    y16 = torch.empty((B, N), dtype=torch.float16, device="cuda")
    out = torch.empty((B, N), dtype=torch.float32, device="cuda")
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        sa.sa_shiftadd_gemm(x, packed, e, q, N, K, G, B, out)
    for rep in range(3):
        x.copy_(torch.randn((B, K), device="cuda").to(torch.float16))
        graph.replay()
        sa.sa_shiftadd_gemm(x, packed, e, q, N, K, G, B, y32)
        sa.sa_shiftadd_gemm_f16(x, packed, e, q, N, K, G, B, y16)
        torch.cuda.synchronize()
        assert torch.equal(out, y32)
        assert torch.equal(y16, y32.to(torch.float16))


@pytest.mark.parametrize("N,K,B", [(40, 4096, 2), (9000, 8192, 4), (24001, 2176, 7)])
@pytest.mark.parametrize("scale", [0, 3, -1])
def test_small_beside_large_is_exact(N, K, B, scale):
    """Activations of 11 bits at 2^-13 of the largest of their 32 columns: every
    partial sum fits fp32, so the layer is exact."""
    say(f"small beside large B={B} scale=2^{scale}")
    c = runs(workloads.random_case(1, N, K, 128, B, seed=51, exp_range=(0, 0)), MX)
    rng = np.random.default_rng(52)
    x = np.zeros((B, K))
    for b in range(B):
        at = 32 * int(rng.integers(0, K // 32))
        x[b, at:at + 32] = rng.choice([-1.0, 1.0], 32) * 2.0 ** -13 * (1 + 2.0 ** -10)
        x[b, at + int(rng.integers(0, 32))] = 1.0
    c["x"] = (x * 2.0 ** scale).astype(np.float16)
    assert (c["x"].astype(np.float64) == x * 2.0 ** scale).all()
    ref = oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], 128)[0]
    y = layer(c)
    say(f"  max |y-y_ref| = {np.abs(y - ref).max():.3e}")
    assert np.array_equal(y, ref)


@pytest.mark.parametrize("B", [2, 4, 8])
@pytest.mark.parametrize("outlier", [20.0, 1000.0, 8000.0, 16000.0])
def test_massive_outliers(B, outlier):
    """Four channels far above the rest: no further from 64 bits than the fp32
    tables of binary16 activations (1.1: the two add in different orders; dropped
    bits of the activations showed as a factor of 2)."""
    say(f"massive outliers x{outlier} B={B}")
    c = runs(workloads.random_case(3, 4170, 4096, 128, B, seed=53, exp_range=(-10, -3)), MX)
    x = np.random.default_rng(54).standard_normal((B, 4096))
    x[:, [7, 1030, 2111, 4000]] = outlier * np.sign(x[:, [7, 1030, 2111, 4000]])
    c["x"] = x.astype(np.float16)
    ref = oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], 128)[0]
    e, er = norm_error(layer(c), ref), norm_error(table_batch(c), ref)
    say(f"  error {e:.3e}, table kernel {er:.3e}")
    assert e <= 1.1 * er


@pytest.mark.parametrize("q,N,K,B,kernel", [
    (4, 8001, 512, 60, TILE), (3, 2000, 640, 255, TILE), (3, 5003, 4096, 250, TILE),
    (3, 4096, 4096, 16, SPLIT), (1, 15556, 640, 9, SPLIT), (3, 4170, 4096, 8, MX)])
def test_error_as_the_table_kernel(q, N, K, B, kernel):
    """Ordinary activations with 1% of the channels x20: no further from 64 bits
    than the fp32 tables (1.1: the two add in different orders)."""
    say(f"error q={q} N={N} K={K} B={B}")
    c = workloads.random_case(q, N, K, 128, B, seed=60, exp_range=(-10, -3),
                              outlier_fraction=0.01)
    runs(c, kernel)
    ref = oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], 128)[0]
    e, er = norm_error(layer(c), ref), norm_error(table_batch(c), ref)
    say(f"  error {e:.3e}, table kernel {er:.3e}")
    assert e <= 1.1 * er


@pytest.mark.parametrize("q,N,B,T", [(4, 2300, 4, 4), (3, 4170, 8, 2), (3, 4170, 2, 2)])
@pytest.mark.parametrize("outlier", [20.0, 1000.0, 30000.0])
def test_massive_outliers_additive(q, N, B, T, outlier):
    """Every term adds the activations again: the chains of fp32 additions stay as
    short as the table kernel's, whose errors at these sizes are 0.9e-7 to 1.5e-7
    (with chains over the terms up to 2.9e-7)."""
    say(f"massive outliers x{outlier}, additive q={q} B={B} T={T}")
    c = runs(workloads.terms_case(q, N, 4096, 128, B, T, seed=53), MX)
    x = np.random.default_rng(54).standard_normal((B, 4096))
    x[:, [7, 1030, 2111, 4000]] = outlier * np.sign(x[:, [7, 1030, 2111, 4000]])
    c["x"] = x.astype(np.float16)
    ref = oracle.shiftadd_gemm_terms(c["x"], c["signs"], c["exps"], c["term_signs"], 128)[0]
    e = norm_error(terms_layer(c), ref)
    say(f"  error {e:.3e}")
    assert e <= 1.6e-7


@pytest.mark.parametrize("q,N,K,G,B", [(3, 300, 4096, 128, 2), (3, 300, 4096, 4096, 4),
                                       (2, 9000, 8192, 128, 8)])
def test_top_of_the_range_leaves_other_rows(q, N, K, G, B):
    """Finite activations of any size run the same arithmetic: the other batch
    rows keep their bits, and the row itself is a layer like any other."""
    say(f"top of the range q={q} N={N} K={K} G={G} B={B}")
    c = runs(workloads.random_case(q, N, K, G, B, seed=55, exp_range=(-10, -3)), MX)
    clean = layer(c)
    c["x"][1, 100], c["x"][1, K - 1], c["x"][1, 64:96] = 65504.0, -63500.0, np.float16(63488.0)
    y = layer(c)
    others = [b for b in range(B) if b != 1]
    assert np.array_equal(y[others], clean[others])
    check(y, c, "top of the range")
    # 2^15 times a row of ordinary values is 2^15 times its result, bit for bit
    c["x"][0] = np.clip(c["x"][0], -1.999, 1.999)
    small = layer(c)[0]
    c["x"][0] = (c["x"][0].astype(np.float64) * 2.0 ** 15).astype(np.float16)
    assert np.array_equal(layer(c)[0], small * 2.0 ** 15)


@pytest.mark.parametrize("N,B", [(300, 2), (2300, 3), (5003, 8)])
@pytest.mark.parametrize("T", [0, 2])
def test_sums_that_cancel_before_the_shift(N, B, T):
    """A group's sum is small where its terms cancel: nothing overflows before the
    factor, up to 2^126, is applied."""
    say(f"cancelling group B={B} T={T}")
    q, K = 3, 4096
    x = np.zeros((B, K))
    x[:, 128:192], x[:, 192:256], x[:, 255] = 4.0, -4.0, -3.75
    x[:, 1000] = 1.0
    signs = np.ones((q, N, K), np.int8)
    signs[:, :, 1000] = np.where(np.arange(N) % 2, 1, -1)
    exps = np.zeros((q, N, K // 128), np.int8)
    exps[0, :, 1] = 77 + np.arange(N) % 50
    c = dict(x=x.astype(np.float16), signs=signs, exps=exps, q=q, N=N, K=K, G=128, B=B)
    if T:
        ts = np.ones((q, N, K // 128, T), np.int8)
        ts[..., 1] = 0  # no second term, whatever its exponent
        c.update(T=T, exps=np.stack([exps, np.full_like(exps, 127)], -1), term_signs=ts)
        y = terms_layer(runs(c, MX))
        ref = oracle.shiftadd_gemm_terms(c["x"], signs, c["exps"], ts, 128)[0]
    else:
        y, ref = layer(runs(c, MX)), oracle.shiftadd_gemm(c["x"], signs, exps, 128)[0]
    assert np.array_equal(y, ref.astype(np.float32).astype(np.float64))


@pytest.mark.parametrize("N,B,kernel", [(200, 2, MX), (4170, 8, MX), (4096, 16, SPLIT),
                                       (5003, 250, TILE)])
def test_smallest_exponents(N, B, kernel):
    """Results about 2^-126 keep the spacing 2^-149 of fp32 subnormals, also where
    one row of the same tile has the largest factor."""
    say(f"smallest exponents B={B}")
    q, K = 3, 4096
    c = runs(workloads.random_case(q, N, K, 128, B, seed=58, exp_range=(-128, -124)), kernel)
    c["x"] = (c["x"].astype(np.float64) * 2.0 ** -9).astype(np.float16)
    for row in (None, 33):
        if row is not None:
            c["exps"][0, row, 7] = 127
        y, (ref, a_ref) = layer(c), oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], 128)
        # one rounding per plane and 128 columns, to fp32 or to a multiple of 2^-149
        bound = (64 + q * K / 128) * 2.0 ** -24 * a_ref + q * K / 128 * 2.0 ** -149
        say(f"  max |y-y_ref| / bound = {(np.abs(y - ref) / bound).max():.2e}")
        assert (np.abs(y - ref) <= bound).all()


@pytest.mark.parametrize("q,N,K,G,B,T", [(3, 300, 4096, 128, 2, 0), (3, 300, 4096, 4096, 4, 0),
                                         (2, 9000, 8192, 128, 8, 0), (2, 40000, 384, 128, 2, 0),
                                         (4, 300, 7296, 384, 8, 3), (4, 300, 2688, 384, 4, 3)])
def test_not_finite_leaves_other_rows(q, N, K, G, B, T):
    """Infinities and NaNs of a batch row reach its outputs as the oracle says
    (absent terms take none); the other rows keep their bits."""
    say(f"not finite, other rows q={q} N={N} K={K} G={G} B={B} T={T}")
    if T:
        c = workloads.terms_case(q, N, K, G, B, T, seed=56)
        # group 0: one term in every second row, none in row 5
        c["term_signs"][1:, ::2, 0], c["term_signs"][0, ::2, 0, 1:] = 0, 0
        c["term_signs"][:, 5, 0] = 0
    else:
        c = workloads.random_case(q, N, K, G, B, seed=56, exp_range=(-10, -3))

    runs(c, MX)

    def both():
        with np.errstate(invalid="ignore"):
            if T:
                return terms_layer(c), oracle.shiftadd_gemm_terms(c["x"], c["signs"], c["exps"],
                                                                  c["term_signs"], G)[0]
            return layer(c), oracle.shiftadd_gemm(c["x"], c["signs"], c["exps"], G)[0]

    clean = both()[0]
    c["x"][1, 77] = np.inf
    c["x"][B - 1, 5], c["x"][B - 1, K - 3] = -np.inf, np.inf
    y, ref = both()
    others = [b for b in range(B) if b not in (1, B - 1)]
    assert np.array_equal(y[others], clean[others])
    assert np.array_equal(np.isnan(y), np.isnan(ref))
    inf = np.isinf(ref)
    assert (inf[1].any() or B == 2) and np.array_equal(y[inf], ref[inf])
    fin = np.isfinite(ref)
    assert np.abs(y[fin] - ref[fin]).max() <= 1e-5 * np.abs(clean).max()
    c["x"][0], c["x"][1, 77] = np.nan, 1.0
    y = layer(c) if not T else terms_layer(c)
    assert np.isnan(y[0]).all()
    assert np.array_equal(y[others[1:]], clean[others[1:]])
