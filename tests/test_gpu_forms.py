"""The two forms of the Group-GEMM launch (planned tiles, and the narrow items
that launches with few tiles are cut into) against the oracle, at the edges of
their tiles: rows around 16 / 32 / 64 / 128, channels around the item widths
(64, 128) and the tile widths (256, 512), reductions with and without slices."""

import pytest

from paper_2505_05799_amd import workloads as W
from tests.gpuhelp import say
from tests.stagewise import check_forward
from tests.test_gpu_forward import run_block
from tests.test_gpu_kernels import _check_linear, _linear_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", W.ALL_SCHEMES, ids=lambda s: s.name)
@pytest.mark.parametrize("m,n,k", [(1, 528, 1536), (16, 144, 640), (17, 1040, 512), (33, 656, 1536),
                                   (64, 272, 384), (97, 400, 1536), (129, 784, 256)])
def test_narrow_linear(scheme, m, n, k):
    """At most 512 tiles: the narrow form (the rows' halves and the channels'
    quarters past the edges hold no work)."""
    for act in ("bf16", "fp16"):
        q, a, got, _ = _linear_case(scheme, act, m, n, k, m + n + k)
        _check_linear(q, a, got, act)


@pytest.mark.parametrize("scheme", W.ALL_SCHEMES, ids=lambda s: s.name)
@pytest.mark.parametrize("m", [4133, 7201])
def test_wide_linear(scheme, m):
    """(1 + m / 64) tile rows of 9 (m = 4133) or 5 channel tiles are more than
    512 tiles of few weight bytes each: the planned tiles themselves."""
    n = 2064 if m == 4133 else 1040
    for act in ("bf16", "fp16"):
        q, a, got, _ = _linear_case(scheme, act, m, n, 384, m + n)
        _check_linear(q, a, got, act)


BLOCKS = [
    [(W.W4G128,) * 3, (W.W8A8, W.W8A8, W.W2G128), (W.W4A4,) * 3, (W.W16, W.W16, W.W3G128), (W.W3G128,) * 3,
     (W.W8G128, W.W8G128, W.W4A4), (W.W2G128, W.W2G128, W.W8A8)],
    [(W.MXFP4,) * 3, (W.FP8,) * 3, (W.W4A4G128,) * 3, (W.W4A4F6, W.W4A4F6, W.W4G128), (W.FP8, W.FP8, W.MXFP4),
     (W.W4A4G128, W.W4A4G128, W.W4A4F6), (W.W4G128, W.W4G128, W.FP8)],
]


@pytest.mark.parametrize("act", ["bf16", "fp16"])
@pytest.mark.parametrize("mix", [0, 1])
@pytest.mark.parametrize("T", [41, 3000])   # narrow; 594 and more gate|up tiles: wide
def test_block_forms(T, mix, act):
    blk = W.random_small_block(31 + T, T=T, H=256, F=768, E=6, k=2, n_shared=1, F_shared=384, act=act,
                               schemes=BLOCKS[mix], skew=1.0)
    mb, y = run_block(blk)
    rep = check_forward(mb, blk, y)
    say(f"T={T} mix {mix} {act}: {rep.line()}")
