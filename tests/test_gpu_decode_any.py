"""GPU parity of rrq_linear's decode form on rows that are no multiple of 4096
inputs (groups of 128; up to 4 tokens on up to 30720 inputs, 5 to 8 on up to 12288) against the
oracle's Eq. 20 product in float64.

* exact: power-of-two scales, integer zero-points and small-integer
  activations make every intermediate exactly representable, so the sampled
  outputs must equal the exact value bit for bit: 1 to 60 sets of 4 groups
  (waves with one set, with 4 or 5 of 5, uneven shares), a last set of 1 to 4
  groups, ragged row tiles, every stage count and format, and the neighbours
  of the rule's edges;
* a row whose scales are infinite or NaN leaves the other rows' bits alone
  (the missing groups of a row's last set lie in the next row's memory);
* a captured call replays to the eager result.
"""

import numpy as np
import pytest

from oracle import rrq_oracle as npo
from test_gpu_decode import G, _log, _run, _sample_rows

pytestmark = pytest.mark.gpu


def _package(rows, cols, M, seed):
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, 2 ** 32, (4, rows * cols // 16), dtype=np.uint64).astype(np.uint32)
    s = (2.0 ** rng.integers(-4, -1, (4, rows * cols // G))).astype(np.float32)
    z = rng.integers(0, 4, (4, rows * cols // G)).astype(np.float32)
    xb = npo.f32_to_bf16_bits(rng.integers(-4, 5, (M, cols)).astype(np.float32))
    return codes, s, z, xb


@pytest.mark.parametrize("rows,cols,M", [
    (4097, 128, 1), (4103, 256, 4), (4099, 384, 2), (5000, 512, 3), (4098, 640, 1), (515, 1920, 4),
    (1025, 5120, 1), (5120, 5120, 4), (300, 5888, 2), (257, 6144, 1), (258, 6272, 3),
    (1027, 7680, 1), (259, 10240, 4), (130, 12416, 2), (1024, 20480, 1), (1100, 25600, 1),
    (130, 30592, 3), (67, 30720, 4), (1, 20608, 1),
    # the rule's edges: short rows up to 4096 of them, rows past the longest
    # 5 to 8 tokens, up to 12288 inputs; their edges
    (5000, 128, 8), (4097, 640, 5), (1025, 1152, 6), (1024, 5120, 8), (5121, 5888, 7), (516, 6272, 8),
    (1027, 8192, 5), (1022, 12288, 8), (300, 12416, 6), (1030, 1920, 8), (1030, 2048, 7),
    # between the batch form and the general kernel
    (1024, 3072, 8), (1025, 3072, 5), (2047, 2688, 6), (2049, 3968, 7), (5117, 2048, 8), (5117, 2432, 5),
    (4096, 640, 2), (2049, 1024, 1), (2049, 1152, 1), (67, 30848, 2), (1025, 12800, 1),
])
@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_decode_any_exact(gpu, rows, cols, M, k):
    _log(f"decode any exact rows={rows} cols={cols} M={M} k={k}")
    codes, s, z, xb = _package(rows, cols, M, rows + cols + M + k)
    y = _run(gpu, codes, s, z, rows, cols, k, xb)
    idx = _sample_rows(rows, k)
    ref = npo.linear(codes, s, z, rows, cols, G, k, xb, row_index=idx)
    assert np.all(np.abs(ref) < 2.0 ** 20)
    assert np.array_equal(y[:, idx].astype(np.float64), ref)
    assert not np.any(np.isnan(y)), "unwritten outputs"


@pytest.mark.parametrize("zp,sd", [("sym", "f16"), ("real", "f32"), ("int", "bf16")])
@pytest.mark.parametrize("rows,cols,k,M", [(1022, 1664, 3, 3), (517, 10368, 4, 3), (130, 25600, 2, 3),
                                           (1022, 1664, 4, 7), (517, 10368, 4, 6)])
def test_decode_any_exact_formats(gpu, zp, sd, rows, cols, k, M):
    _log(f"decode any format {zp}/{sd} rows={rows} cols={cols}")
    codes, s, z, xb = _package(rows, cols, M, 5)
    z = None if zp == "sym" else z * 0.25 if zp == "real" else z
    s_raw = (s.astype(np.float16).view(np.uint16) if sd == "f16"
             else (s.view(np.uint32) >> 16).astype(np.uint16) if sd == "bf16" else s)
    y = _run(gpu, codes, s, z, rows, cols, k, xb, zp, sd, s_raw)
    idx = _sample_rows(rows, k)
    ref = npo.linear(codes, s, np.full_like(s, 2.0) if z is None else z, rows, cols, G, k, xb,
                     row_index=idx)
    assert np.array_equal(y[:, idx].astype(np.float64), ref)


@pytest.mark.parametrize("cols", [1152, 5248, 10368, 25728])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_decode_any_rows_are_apart(gpu, cols, value):
    rows, M, k = 97, 2, 4
    codes, s, z, xb = _package(rows, cols, M, 3)
    plain = _run(gpu, codes, s, z, rows, cols, k, xb)
    for bad in (1, 50, 96):
        s2 = s.reshape(4, rows, cols // G).copy()
        s2[:, bad] = value
        z2 = z.reshape(4, rows, cols // G).copy()
        z2[:, bad] = value
        y = _run(gpu, codes, s2.reshape(4, -1), z2.reshape(4, -1), rows, cols, k, xb)
        others = np.arange(rows) != bad
        assert np.array_equal(y[:, others].view(np.uint32), plain[:, others].view(np.uint32))
        assert not np.any(np.isfinite(y[:, bad]))


def test_decode_any_graph_replays(gpu):
    import torch
    rows, cols, M, k = 1030, 2688, 2, 4
    codes, s, z, xb = _package(rows, cols, M, 9)
    want = _run(gpu, codes, s, z, rows, cols, k, xb)
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
