"""Both sides of the rule that shares the frames of a loss out over a block's waves; every
oversampling and the kernel per pixel among those that are shared.

A block covers 256 pixels. Frames are shared from six on up to 256 blocks and from eight on up to 512.
Bounds as in test_gpu_loss_frames.py: sums of doubles to 1e-13 of their magnitudes, the residual to one rounding.
"""
import pytest

from tests.test_gpu_loss_frames import (test_fused_seed_of_several_frames_matches_the_separate_calls as fused_seed,
                                        test_loss_of_several_frames_matches_float64 as plain_loss)

pytestmark = pytest.mark.gpu


# 5 and 6 frames; 7 and 8 past 256 blocks (256^2 pixels); 512 blocks (362^2) and 515 (363^2)
@pytest.mark.parametrize("kind", ["poisson", "chi2"])
@pytest.mark.parametrize("nd,frames", [(33, 5), (33, 6), (256, 6), (257, 7), (257, 8), (362, 9), (363, 9), (181, 16)])
def test_loss_alone_on_both_sides(nd, frames, kind):
    plain_loss(nd, frames, kind)


# q = 1 .. 5 and a kernel per pixel, shared; the same limits
@pytest.mark.parametrize("q,nd,frames,per_pixel", [(1, 17, 6, False), (2, 9, 6, False), (3, 21, 6, False), (4, 16, 7, False),
                                                   (5, 7, 6, False), (1, 30, 7, True), (3, 11, 9, True), (4, 10, 16, True),
                                                   (2, 33, 5, False), (1, 257, 7, False), (1, 257, 8, False),
                                                   (1, 362, 17, False), (1, 363, 8, False)])
def test_fused_seed_on_both_sides(q, nd, frames, per_pixel):
    fused_seed(q, nd, frames, per_pixel)
