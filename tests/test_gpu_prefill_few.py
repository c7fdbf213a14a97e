"""GPU parity of rrq_linear's prefill form with 17 to 127 tokens
against the oracle's Eq. 20 product in float64: power-of-two scales,
integer zero-points and small-integer activations make every intermediate
exactly representable, so the sampled outputs must equal the exact value bit
for bit. Shapes on both sides of the rule that picks the form (256 compute
units): one 64 x 64 tile per compute unit, two that share their codes, two row
tiles, more than one round, 128- and 256-row tiles, ragged rows and tokens; and a row or token that is
not finite stays by itself."""

import numpy as np
import pytest

from oracle import rrq_oracle as npo
from test_gpu_decode import _log, _run, _sample_rows
from test_gpu_decode_any import _package

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,cols,M", [
    (12288, 256, 48), (12290, 128, 64), (8200, 384, 65), (8190, 256, 64), (5121, 640, 100),
    (16385, 128, 40), (16384, 256, 127), (25600, 128, 33), (25601, 256, 64), (33000, 128, 127),
    # 128 x 128 tiles in one round; 256 x 128 at one stage, and not for half a tile of tokens
    (16448, 256, 80), (24448, 128, 127), (65537, 128, 100), (65537, 128, 48),
    # the general kernel's side
    (12288, 128, 17), (4096, 384, 64), (300, 1152, 100),
])
@pytest.mark.parametrize("k", [1, 2, 3, 4])
def test_few_tokens_exact(gpu, rows, cols, M, k):
    _log(f"few tokens rows={rows} cols={cols} M={M} k={k}")
    codes, s, z, xb = _package(rows, cols, M, rows + cols + M + k)
    y = _run(gpu, codes, s, z, rows, cols, k, xb)
    idx = _sample_rows(rows, k)
    ref = npo.linear(codes, s, z, rows, cols, 128, k, xb, row_index=idx)
    assert np.array_equal(y[:, idx].astype(np.float64), ref)
    assert not np.any(np.isnan(y)), "unwritten outputs"


@pytest.mark.parametrize("zp,sd", [("sym", "f16"), ("real", "f32"), ("int", "bf16")])
def test_few_tokens_formats(gpu, zp, sd):
    rows, cols, M, k = 12300, 384, 50, 2
    _log(f"few tokens format {zp}/{sd}")
    codes, s, z, xb = _package(rows, cols, M, 5)
    z = None if zp == "sym" else z * 0.25 if zp == "real" else z
    s_raw = (s.astype(np.float16).view(np.uint16) if sd == "f16"
             else (s.view(np.uint32) >> 16).astype(np.uint16) if sd == "bf16" else s)
    y = _run(gpu, codes, s, z, rows, cols, k, xb, zp, sd, s_raw)
    idx = _sample_rows(rows, k)
    ref = npo.linear(codes, s, np.full_like(s, 2.0) if z is None else z, rows, cols, 128, k, xb,
                     row_index=idx)
    assert np.array_equal(y[:, idx].astype(np.float64), ref)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_few_tokens_stay_apart(gpu, value):
    rows, cols, M, k = 12290, 256, 50, 2
    codes, s, z, xb = _package(rows, cols, M, 3)
    plain = _run(gpu, codes, s, z, rows, cols, k, xb)
    bits = xb.reshape(M, cols).copy()
    bits[49, 200] = np.float32(value).view(np.uint32) >> 16
    s2 = s.reshape(4, rows, cols // 128).copy()
    s2[:, 12289, 1] = value
    y = _run(gpu, codes, s2.reshape(4, -1), z, rows, cols, k, bits.reshape(-1))
    assert np.array_equal(y[:49, :12289].view(np.uint32), plain[:49, :12289].view(np.uint32))
    assert not np.any(np.isfinite(y[49])) and not np.any(np.isfinite(y[:, 12289]))
