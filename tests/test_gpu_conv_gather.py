"""The image loads of the convolution kernels that gather through VGPRs, where
their two loads per chunk can go wrong: filter rows of just under, exactly and
just over a chunk, image rows shorter than a chunk, padding wider than a chunk
and than the image, chunks over both edges of an image row, the first and last
pixels of the image, K ends inside a chunk.

Integer-valued operands, so every result is exact and compared bit for bit."""
import pytest

import oracle
from oracle import tolerance
from paper_2409_01075_amd import inputs as I
from paper_2409_01075_amd import vx

from .test_gpu_conv import run_conv

pytestmark = pytest.mark.gpu

CASES = [
    # N, H, W, Cin, KH, KW, stride, pad, dil
    (1, 5, 9, 3, 2, 2, (1, 1), (0, 0), (1, 1)),      # filter rows of 6: below a 16-bit chunk, above a 32-bit one
    (2, 4, 7, 1, 3, 7, (1, 1), (1, 3), (1, 1)),      # filter and image rows of 7
    (2, 4, 8, 1, 3, 8, (1, 1), (1, 4), (1, 1)),      # filter and image rows of 8: exactly a chunk
    (1, 5, 9, 1, 4, 9, (1, 1), (2, 4), (1, 1)),      # rows of 9: nearly every chunk crosses
    (1, 1, 3, 3, 3, 7, (1, 1), (1, 9), (1, 1)),      # padding wider than the image and a chunk, one image row
    (3, 6, 5, 11, 3, 3, (2, 1), (2, 2), (1, 1)),     # odd channels, stride, padding past the first tap
    (2, 9, 6, 7, 3, 3, (1, 1), (2, 1), (3, 1)),      # rows of the filter three image rows apart
    (2, 7, 9, 5, 3, 3, (1, 2), (1, 2), (1, 2)),      # dilated along the width: element gathers
    (1, 6, 7, 16, 3, 3, (1, 1), (1, 1), (1, 1)),     # whole chunks of channels
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("code", [I.F32, I.F16, I.BF16])
def test_gathered_chunks_exact(code, case):
    N, H, W, Cin, KH, KW, st, pd, dl = case
    g = I.rng(1260 + code)
    picked = {}
    for i in range(vx.vx_registry_count()):
        k = vx.vx_registry_get(i)
        if k.op == 1 and k.dtype == code and k.enabled and not k.align & 1:
            picked.setdefault((k.family, k.align, k.stages, k.threads), k)
    assert picked
    x = I.small_int(g, (N, H, W, Cin), code, -3, 3)
    for k in picked.values():
        for split in (1, 2):
            if split * k.kb > KH * KW * Cin + k.kb - 1:
                continue
            w = I.small_int(g, (KH, KW, Cin, 24), code, -3, 3)
            ref = oracle.conv2d(x, w, code, st, pd, dl, with_mag=False)
            assert vx.vx_force_plan(k.id, split) == 0
            try:
                y = run_conv(x, w, code, st, pd, dl)
            finally:
                vx.vx_force_plan(-1, 0)
            tolerance.check_exact(y, ref, code, "conv kernel %d split %d %s" % (k.id, split, case))
