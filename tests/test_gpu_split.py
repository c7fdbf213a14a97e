"""GPU parity of rrq_linear's split form (more than 16 tokens: groups of 32
and 64, and groups of 128 with 3 or 4 stages), through the C ABI, against the
oracle's Eq. 20 product in float64.

* exact: power-of-two scales, integer or dyadic zero-points and
  small-integer activations make every intermediate exactly representable
  (the weight is a multiple of 2^-4 below 4, so its first two bfloat16
  operands hold it), so the sampled outputs must equal the exact value bit for bit:
  every tile shape, ragged rows, tokens and last chunks, quarters of unequal
  length and empty ones, every stage count and format;
* bounded: realistic packages, and scales and activations whose ranges move
  by many binades along a row, all tokens alike or each its own way, and
  between the groups of one chunk, with the scales' range against the
  activations' or near the ends of binary32's, stay within the bound of
  include/rrq.h, as do rows longer than 8192 inputs in every way of splitting
  a row over waves;
* the results do not depend on the tile shape a call takes (rows of up to
  2048 inputs), nor a token's on the other tokens;
* a token holding an infinity or a NaN does not touch the others.
Packages come from the oracle or a seeded generator, never from the GPU.
"""

import math
import sys

import numpy as np
import pytest

import oracle
from oracle import rrq_oracle as npo
from test_dispatch import form

pytestmark = pytest.mark.gpu
U = 2.0 ** -24


def _log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def _run(gpu, codes, s_raw, z, rows, cols, G, k, xb, zp="int", sd="f32"):
    import torch
    M = xb.size // cols
    c = torch.from_numpy(codes.view(np.int32).copy()).cuda()
    sc = torch.from_numpy(s_raw.copy()).cuda()
    ze = None if z is None else torch.from_numpy(z.copy()).cuda()
    X = torch.from_numpy(xb.view(np.int16).reshape(M, cols).copy()).cuda().view(torch.bfloat16)
    Y = torch.full((M, rows), float("nan"), dtype=torch.float32, device="cuda")
    gpu.rrq_linear_format(c, sc, ze, rows, cols, G, codes.shape[0], gpu.ZERO_POINTS[zp],
                          gpu.SCALE_TYPES[sd], k, X, M, Y)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


def _exact(rows, cols, G, M, seed):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, 2 ** 32, (4, rows * cols // 16), dtype=np.uint64).astype(np.uint32)
    s = (2.0 ** rng.integers(-4, -1, (4, rows * cols // G))).astype(np.float32)
    z = rng.integers(0, 4, (4, rows * cols // G)).astype(np.float32)
    xb = npo.f32_to_bf16_bits(rng.integers(-4, 5, (M, cols)).astype(np.float32))
    return codes, s, z, xb


def _sample(rows, seed):
    if rows <= 320:
        return np.arange(rows)
    rng = np.random.default_rng(seed)
    return np.unique(np.concatenate([np.arange(32), np.arange(rows - 32, rows),
                                     rng.choice(rows, 96, replace=False)]))


# On 256 compute units: 256-, 128- and 64-token tiles of 128 rows for 4090
# rows at 2043, 1021 and 490 tokens, a quarter per wave with 64-, 32- and
# 32-token tiles of 32, 32 and 64 rows for 4090 rows at 121 tokens, 250 or
# fewer rows, and 12290 rows at 30 tokens. Rows of 1 to 9 chunks of 128 inputs,
# partial last chunks with the smaller groups.
EXACT = [
    (4090, 320, 64, 2043), (4090, 448, 64, 1021), (4090, 64, 64, 490), (4090, 576, 64, 121),
    (250, 1088, 64, 140), (4090, 608, 32, 1021), (4090, 32, 32, 490), (4090, 1120, 32, 121),
    (35, 96, 32, 67), (1, 32, 32, 130), (4090, 384, 128, 2043), (4090, 1152, 128, 1021),
    (4090, 128, 128, 1021), (1023, 640, 128, 127), (70, 128, 128, 66),
    (4090, 352, 32, 2043), (12290, 160, 32, 30), (12290, 192, 64, 30), (12290, 128, 128, 30),
    (16700, 128, 128, 50), (4090, 256, 128, 100),
    # row tiles no multiple of 8: with a pitch that is one, and where that would
    # take another round
    (2100, 192, 64, 2043), (2680, 128, 128, 79),
]


@pytest.mark.parametrize("rows,cols,G,M", EXACT)
@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_split_exact(gpu, rows, cols, G, M, k):
    if G == 128 and k < 3:
        pytest.skip("groups of 128 take the split form from 3 stages")
    _log(f"split exact rows={rows} cols={cols} G={G} M={M} k={k}")
    codes, s, z, xb = _exact(rows, cols, G, M, rows + cols + M + k)
    y = _run(gpu, codes, s, z, rows, cols, G, k, xb)
    idx = _sample(rows, cols)
    ref = npo.linear(codes, s, z, rows, cols, G, k, xb, row_index=idx)
    bad = np.argwhere(y[:, idx].astype(np.float64) != ref)
    assert bad.size == 0, f"{len(bad)} outputs differ, first {bad[:3]}"
    assert not np.any(np.isnan(y)), "unwritten outputs"


@pytest.mark.parametrize("zp,sd", [("sym", "f16"), ("real", "f32"), ("int", "bf16"), ("sym", "f32")])
@pytest.mark.parametrize("rows,cols,G,M,k", [(310, 416, 32, 70, 2), (310, 704, 64, 140, 4),
                                             (4090, 192, 64, 500, 3), (310, 640, 128, 70, 4)])
def test_split_exact_formats(gpu, zp, sd, rows, cols, G, M, k):
    _log(f"split exact format {zp}/{sd} rows={rows} cols={cols} G={G} M={M}")
    codes, s, z, xb = _exact(rows, cols, G, M, 17)
    if zp == "sym":
        zz, zv = None, np.full_like(s, 2.0)
    elif zp == "real":
        zz = (np.random.default_rng(5).integers(0, 13, s.shape) * 0.25).astype(np.float32)
        zv = zz
    else:
        zz = zv = z
    s_raw = (s.astype(np.float16).view(np.uint16) if sd == "f16"
             else (s.view(np.uint32) >> 16).astype(np.uint16) if sd == "bf16" else s)
    y = _run(gpu, codes, s_raw, zz, rows, cols, G, k, xb, zp, sd)
    idx = _sample(rows, 3)
    ref = npo.linear(codes, s, zv, rows, cols, G, k, xb, row_index=idx)
    assert np.array_equal(y[:, idx].astype(np.float64), ref)


def _bound(s, z, rows, cols, G, k, xb, idx):
    x = np.abs(npo.bf16_bits_to_f32(xb).reshape(-1, cols).astype(np.float64))
    T = x.reshape(x.shape[0], cols // G, G).sum(axis=2)
    A = sum(T @ (np.abs(s[t].astype(np.float64)) * (11 + np.abs(z[t].astype(np.float64))))
            .reshape(rows, cols // G)[idx].T for t in range(k))
    p = cols // G
    n = k * (min(p, 4 * math.ceil(p / 16)) + 1)
    return 1.05 * U * A * (G + 2 * n + 24) + 1e-300


@pytest.mark.parametrize("rows,cols,G,M", [(300, 2048, 64, 140), (4096, 1024, 64, 500),
                                           (300, 1536, 32, 40), (300, 2048, 128, 72),
                                           (2048, 512, 128, 2048)])
@pytest.mark.parametrize("ranges", ["realistic", "moving"])
def test_split_within_bound(gpu, rows, cols, G, M, ranges):
    """moving: the scales of a row's groups and the activations of a token's
    chunks each wander over 2^+-24, every chunk another power of two, and a
    token and a chunk are all zeros."""
    rng = np.random.default_rng(rows + cols + G)
    w = (rng.standard_normal(rows * cols) * 0.02).astype(np.float32)
    w = np.where(rng.random(w.size) < 1e-3, w * 20, w).astype(np.float32)
    codes, s, z = oracle.c_construct(npo.f32_to_bf16_bits(w), G, 4)
    x = rng.standard_normal((M, cols)).astype(np.float32)
    if ranges == "moving":
        chunks = -(-cols // 128)
        f = 2.0 ** rng.integers(-24, 25, (M, chunks))
        f[:, chunks // 2] = 0
        x = (x * np.repeat(f, 128, axis=1)[:, :cols]).astype(np.float32)
        x[3] = 0
        g = 2.0 ** rng.integers(-24, 25, (rows, chunks))
        g = np.repeat(g, 128 // G, axis=1)[:, :cols // G].reshape(-1)
        s = (s * g[None]).astype(np.float32)
    xb = npo.f32_to_bf16_bits(x)
    idx = _sample(rows, 1)
    for k in (3, 4) if G == 128 else (1, 2, 4):
        y = _run(gpu, codes, s, z, rows, cols, G, k, xb)
        ref = npo.linear(codes, s, z, rows, cols, G, k, xb, row_index=idx)
        tol = _bound(s, z, rows, cols, G, k, xb, idx)
        err = np.abs(y[:, idx].astype(np.float64) - ref)
        assert np.all(err <= tol), f"k={k}: {np.max(err / tol)}"
        _log(f"split {ranges} G={G} M={M} k={k}: max err / bound = {np.max(err / tol):.3g}")


@pytest.mark.parametrize("G,k", [(64, 2), (32, 4), (128, 4)])
def test_split_same_results_in_every_shape(gpu, G, k):
    """The same token gives the same bits whatever the tile shape: 2048 tokens
    (the largest tiles that fill the chip), the first 1024 and, in calls of
    127, the first 254 (a quarter of the row per wave)."""
    rows, cols = 4096, 1152
    rng = np.random.default_rng(G)
    w = (rng.standard_normal(rows * cols) * 0.02).astype(np.float32)
    codes, s, z = oracle.c_construct(npo.f32_to_bf16_bits(w), G, 4)
    xb = npo.f32_to_bf16_bits(rng.standard_normal((2048, cols)).astype(np.float32))
    y = _run(gpu, codes, s, z, rows, cols, G, k, xb)
    for m0, m1 in ((0, 1024), (0, 127), (127, 254)):
        part = _run(gpu, codes, s, z, rows, cols, G, k, xb.reshape(2048, cols)[m0:m1].reshape(-1))
        assert np.array_equal(part.view(np.uint32), y[m0:m1].view(np.uint32)), (m0, m1)


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3e38, 1e-38])
def test_split_extreme_token(gpu, value):
    """One extreme activation in one token: the other tokens' outputs keep
    their bits; an infinity or a NaN gives that token non-finite outputs."""
    rows, cols, G, M, k = 96, 640, 64, 140, 4
    rng = np.random.default_rng(9)
    w = (rng.standard_normal(rows * cols) * 0.02).astype(np.float32)
    codes, s, z = oracle.c_construct(npo.f32_to_bf16_bits(w), G, 4)
    x = rng.standard_normal((M, cols)).astype(np.float32)
    plain = _run(gpu, codes, s, z, rows, cols, G, k, npo.f32_to_bf16_bits(x))
    bits = npo.f32_to_bf16_bits(x).reshape(M, cols).copy()
    bits[7, 200] = np.float32(value).view(np.uint32) >> 16
    y = _run(gpu, codes, s, z, rows, cols, G, k, bits.reshape(-1))
    others = np.arange(M) != 7
    assert np.array_equal(y[others].view(np.uint32), plain[others].view(np.uint32))
    if not math.isfinite(value):
        assert not np.any(np.isfinite(y[7]))
    else:
        ref = npo.linear(codes, s, z, rows, cols, G, k, bits.reshape(-1))
        tol = _bound(s, z, rows, cols, G, k, bits.reshape(-1), np.arange(rows))
        assert np.all(np.abs(y[7].astype(np.float64) - ref[7]) <= tol[7])


# Which waves take a row's chunks: each quarter its own (60 and 72 tokens, 300
# rows) or all in turn (1000 tokens, 4090 rows).
_SPLITS = [(300, 60), (300, 72), (4090, 1000)]


def _ranged(rows, cols, G, M, fx, fs, seed):
    """A package and activations with chunk or group factors fx (of the
    inputs) and fs (of the groups), both powers of two along the row."""
    rng = np.random.default_rng(seed)
    w = (rng.standard_normal(rows * cols) * 0.02).astype(np.float32)
    codes, s, z = oracle.c_construct(npo.f32_to_bf16_bits(w), G, 4)
    x = rng.standard_normal((M, cols)).astype(np.float32)
    with np.errstate(over="raise"):
        x = (x.astype(np.float64) * fx[None]).astype(np.float32)
        s = (s.reshape(4, rows, cols // G).astype(np.float64) * fs[None, None]).astype(np.float32)
    return codes, s.reshape(4, -1), z, npo.f32_to_bf16_bits(x)


def _check_bound(gpu, codes, s, z, rows, cols, G, k, xb, what):
    assert form(rows, cols, k, xb.size // cols, G) == "split"
    idx = _sample(rows, 1)
    y = _run(gpu, codes, s, z, rows, cols, G, k, xb)
    ref = npo.linear(codes, s, z, rows, cols, G, k, xb, row_index=idx)
    tol = _bound(s, z, rows, cols, G, k, xb, idx)
    worst = np.max(np.abs(y[:, idx].astype(np.float64) - ref) / tol)
    _log(f"split {what}: max err / bound = {worst:.3g}")
    assert worst <= 1, f"{what}: {worst}"
    return y


@pytest.mark.parametrize("rows,M", _SPLITS)
@pytest.mark.parametrize("G", [32, 64, 128])
@pytest.mark.parametrize("R", [24, 34, 36, 60])
def test_split_ranges_drop_along_a_row(gpu, rows, M, G, R):
    """The first chunk of every quarter is 2^R larger in the activations and
    2^R smaller in the scales (all tokens and rows alike)."""
    cols, k = 2048, 4
    chunk = np.where(np.arange(16) % 4 == 0, 2.0 ** R, 1.0)
    pkg = _ranged(rows, cols, G, M, np.repeat(chunk, 128), np.repeat(1 / chunk, 128 // G), R)
    _check_bound(gpu, *pkg[:3], rows, cols, G, k, pkg[3], f"drop 2^{R} G={G} M={M}")


@pytest.mark.parametrize("rows,M", _SPLITS)
def test_split_ranges_drop_after_zero_weights(gpu, rows, M):
    """A first chunk of large activations whose weights are all zero."""
    cols, G, k = 1024, 128, 4
    fx = np.repeat(np.where(np.arange(8) % 2 == 0, 2.0 ** 40, 1.0), 128)
    fs = np.where(np.arange(8) % 2 == 0, 0.0, 1.0)
    pkg = _ranged(rows, cols, G, M, fx, fs, 5)
    _check_bound(gpu, *pkg[:3], rows, cols, G, k, pkg[3], f"zero weights M={M}")


@pytest.mark.parametrize("rows,M", _SPLITS)
@pytest.mark.parametrize("G", [32, 64])
@pytest.mark.parametrize("R", [12, 22, 30, 40, 80])
def test_split_ranges_between_groups_of_a_chunk(gpu, rows, M, G, R):
    """Neighbouring groups 2^R apart, the activations one way and the scales
    the other; and the large activations over groups of scale 0."""
    cols, k = 640, 2
    far = np.arange(cols // G) % 2 == 0
    fx = np.repeat(np.where(far, 2.0 ** R, 1.0), G)
    pkg = _ranged(rows, cols, G, M, fx, np.where(far, 2.0 ** -R, 1.0), R + G)
    _check_bound(gpu, *pkg[:3], rows, cols, G, k, pkg[3], f"in-chunk 2^{R} G={G} M={M}")
    pkg = _ranged(rows, cols, G, M, fx, np.where(far, 0.0, 1.0), R + G)
    _check_bound(gpu, *pkg[:3], rows, cols, G, k, pkg[3], f"in-chunk 2^{R}, zero scales G={G} M={M}")


@pytest.mark.parametrize("rows,M", _SPLITS)
@pytest.mark.parametrize("G", [32, 128])
@pytest.mark.parametrize("scale", [2.0 ** 104, 2.0 ** 90, 2.0 ** -60, 2.0 ** -72, 2.0 ** -115, "moving"])
def test_split_ranges_near_the_ends(gpu, rows, M, G, scale):
    """Scales near binary32's ends with activations that bring the products
    back, and a row that goes through all of them."""
    cols, k = 1024, 4
    f = (np.array([1, 2.0 ** 104, 2.0 ** -115, 2.0 ** -70, 0, 2.0 ** 90, 2.0 ** -60, 2.0 ** -1])
         if scale == "moving" else np.full(8, scale))
    inv = np.where(f == 0, 1, 1 / np.where(f == 0, 1, f))
    pkg = _ranged(rows, cols, G, M, np.repeat(inv, 128), np.repeat(f, 128 // G), G)
    y = _check_bound(gpu, *pkg[:3], rows, cols, G, k, pkg[3], f"scale {scale} G={G} M={M}")
    assert np.all(np.isfinite(y))


@pytest.mark.parametrize("rows,M", _SPLITS)
@pytest.mark.parametrize("G,cols,k", [(128, 9216, 4), (128, 20608, 3), (64, 8896, 2), (32, 10272, 1)])
def test_split_long_rows_within_bound(gpu, rows, M, G, cols, k):
    pkg = _ranged(rows, cols, G, M, np.ones(cols), np.ones(cols // G), cols)
    _check_bound(gpu, *pkg[:3], rows, cols, G, k, pkg[3], f"cols={cols} G={G} M={M}")


@pytest.mark.parametrize("G,R", [(128, 35), (64, 35), (32, 20)])
def test_split_token_does_not_depend_on_the_others(gpu, G, R):
    """A token whose ranges drop along the row keeps its bits whether the
    other tokens of its tile do as it does, or not, and wherever it stands."""
    rows, cols, M, k = 300, 2048, 72, 4
    chunk = np.where(np.arange(16) % 4 == 0, 2.0 ** R, 1.0)
    assert form(rows, cols, k, M, G) == "split"
    codes, s, z, xb = _ranged(rows, cols, G, M, np.repeat(chunk, 128), np.repeat(1 / chunk, 128 // G), 3)
    y = _run(gpu, codes, s, z, rows, cols, G, k, xb)
    rng = np.random.default_rng(4)
    other = npo.f32_to_bf16_bits((rng.standard_normal((M, cols)) *
                                  2.0 ** rng.integers(-40, 41, (M, cols // 128)).repeat(128, axis=1)
                                  ).astype(np.float32)).reshape(M, cols)
    for at in (0, 17, 71):
        mixed = other.copy()
        mixed[at] = xb.reshape(M, cols)[17]
        ym = _run(gpu, codes, s, z, rows, cols, G, k, mixed.reshape(-1))
        assert np.array_equal(ym[at].view(np.uint32), y[17].view(np.uint32)), at


@pytest.mark.parametrize("rows,cols,G,M,k", [(300, 1088, 64, 40, 2), (4090, 384, 128, 1021, 4)])
def test_split_graph_replays(gpu, rows, cols, G, M, k):
    import torch
    assert form(rows, cols, k, M, G) == "split"
    codes, s, z, xb = _exact(rows, cols, G, M, 7)
    want = _run(gpu, codes, s, z, rows, cols, G, k, xb)
    c, sc, ze = (torch.from_numpy(a).cuda() for a in (codes.view(np.int32).copy(), s, z))
    X = torch.from_numpy(xb.view(np.int16).reshape(M, cols).copy()).cuda().view(torch.bfloat16)
    Y = torch.empty((M, rows), device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        gpu.linear(X, c, sc, ze, rows, cols, G, k, out=Y)
    for _ in range(3):
        Y.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(Y.cpu().numpy().view(np.uint32), want.view(np.uint32))
