"""The linear layer's rules for which kernel and tile serve a call, called on
the CPU through the library's internal functions (256 compute units). form()
tells the other tests which kernel they run."""

import ctypes

import pytest

import paper_2608_04048_amd as rrq

CUS = 256
I64, I32 = ctypes.c_int64, ctypes.c_int
SMALL, LARGE, WIDE = range(3)


def _function(name, *args, restype=ctypes.c_bool):
    f = getattr(rrq.load_library(), name)
    f.argtypes, f.restype = args, restype
    return f


def prefill_fits(rows, cols, k, tokens, G=128):
    f = _function("_ZN10rrq_detail19linear_prefill_fitsElliili", I64, I64, I32, I32, I64, I32)
    return f(rows, cols, G, k, tokens, CUS)


def decode_fits(rows, cols, k, tokens, G=128):
    f = _function("_ZN10rrq_detail18linear_decode_fitsElliil", I64, I64, I32, I32, I64)
    return f(rows, cols, G, k, tokens)


def batch_fits(rows, cols, k, tokens, G=128):
    f = _function("_ZN10rrq_detail17linear_batch_fitsElliil", I64, I64, I32, I32, I64)
    return f(rows, cols, G, k, tokens)


def split_fits(rows, cols, k, tokens, G=128):
    f = _function("_ZN10rrq_detail17linear_split_fitsElliili", I64, I64, I32, I32, I64, I32)
    return f(rows, cols, G, k, tokens, CUS)


def split_shape(rows, cols, tokens, k, G=128):
    f = _function("_ZN10rrq_detail11split_shapeElliiliPl", I64, I64, I32, I32, I64, I32,
                  ctypes.POINTER(I64), restype=I32)
    return "ABCDEF"[f(rows, cols, G, k, tokens, CUS, ctypes.byref(I64()))]


def form(rows, cols, k, tokens, G=128):
    """The kernel that serves a call (the order of the C ABI's dispatch)."""
    for name, fits in (("decode", decode_fits), ("batch", batch_fits), ("split", split_fits),
                       ("prefill", prefill_fits)):
        if fits(rows, cols, k, tokens, G):
            return name
    return "general"


def prefill_tile(rows, tokens, k):
    f = _function("_ZN10rrq_detail12prefill_tileElliiPl", I64, I64, I32, I32,
                  ctypes.POINTER(I64), restype=I32)
    cost = I64(-1)
    return f(rows, tokens, k, CUS, ctypes.byref(cost)), cost.value


@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("tokens", [80, 127])
def test_prefill_rule_charges_the_tile_that_runs(k, tokens):
    """One more row tile than compute units: the cost stays between one round
    of the cheaper tile and two, and one and two stages stay with the form."""
    _, full = prefill_tile(16384, tokens, k)
    _, more = prefill_tile(16448, tokens, k)
    _, large = prefill_tile(32768, tokens, k)      # one round of 128 x 128 tiles
    assert full <= more <= min(2 * full, large)
    if k <= 2:
        assert prefill_fits(16384, 2048, k, tokens) and prefill_fits(16448, 2048, k, tokens)


@pytest.mark.parametrize("rows", [65281, 70000, 100000, 152064])
def test_prefill_few_tokens_take_no_padded_tile(rows):
    """Up to 64 tokens the 128-token tiles would be half padding; above,
    one-stage calls on so many rows take the wide one."""
    for tokens in (17, 48, 64):
        for k in (1, 2, 3, 4):
            assert prefill_tile(rows, tokens, k)[0] == SMALL
    assert prefill_tile(rows, 100, 1)[0] == WIDE
    assert prefill_tile(rows, 128, 1)[0] == WIDE


def test_decode_rule_leaves_the_batch_form_only_what_it_takes():
    """5 to 8 tokens on rows of 2048 to 4096 inputs: small packages, which the
    batch form does not take, go to the decode form where it is ahead."""
    for tokens in (5, 8):
        for rows, cols, k in ((1024, 3072, 4), (512, 2048, 3), (1000, 2560, 2), (2048, 2560, 4),
                              (5120, 2048, 4), (5120, 2048, 2)):
            assert not batch_fits(rows, cols, k, tokens)
            assert decode_fits(rows, cols, k, tokens), (rows, cols, k)
        for rows, cols, k in ((3000, 2560, 4), (2048, 2560, 3), (1024, 2048, 2), (4096, 3968, 4),
                              (12288, 3072, 3)):
            assert not decode_fits(rows, cols, k, tokens), (rows, cols, k)


def test_split_tests_reach_every_tile_shape():
    from test_gpu_split import EXACT
    seen = {(G, split_shape(rows, cols, M, k, G)) for rows, cols, G, M in EXACT for k in (1, 2, 3, 4)
            if form(rows, cols, k, M, G) == "split"}
    assert seen == {(G, s) for G in (32, 64, 128) for s in "ABCDEF"}


def test_prefill_tests_run_the_prefill_form():
    import test_gpu_prefill as t
    for rows, cols, M in (*t.EXACT, *t.LARGE):
        assert all(form(rows, cols, k, M) == "prefill" for k in (1, 2, 3, 4)), (rows, cols, M)
    rows, cols, M = t.WIDE
    assert form(rows, cols, 1, M) == "prefill" and prefill_tile(rows, M, 1)[0] == WIDE
    for rows, cols, M, k in t.SAME_ORDER:
        assert form(rows, cols, k, M) == "prefill"
        assert all(form(rows, cols, k, min(32, M - m)) == "general" for m in range(0, M, 32))


def test_split_rule_on_many_rows():
    """Rows whose package lines outgrow the L2: calls of few tokens leave the
    64- and 32-token tiles that would read them with every chunk."""
    for rows in (25600, 28672, 32000):
        assert split_shape(rows, 4096, 24, 4, 128) != "C" and split_shape(rows, 4096, 24, 4, 64) == "E"
    for rows, cols in ((16384, 8192), (16000, 6144)):
        assert form(rows, cols, 4, 24) == "prefill"
    for rows, cols, k, G in ((10922, 12288, 3, 128), (8192, 12288, 4, 128), (10885, 8192, 4, 64),
                             (16384, 8192, 2, 64)):
        assert form(rows, cols, k, 24, G) == "general"
    for rows, cols, k, G in ((10885, 8192, 3, 128), (10885, 5120, 4, 64), (8192, 8192, 4, 128)):
        assert form(rows, cols, k, 24, G) == "split"
