"""Both sides of the rules that share the frames of a loss out over a block's waves, and that give a lane four
pixels of the integer-dither seeds; every oversampling and the kernel per pixel among those that are shared.

A block covers 256 pixels. Frames are shared from six on up to 256 blocks and from eight on up to 512.
Bounds as in test_gpu_loss_frames.py: sums of doubles to 1e-13 of their magnitudes, the residual to one rounding.
"""
import numpy as np
import pytest

from synth import make_dithered_workload, make_workload
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


# planes of 2070 and 2025 blocks with two stars, 4096 and 4032 with one (a star's last wave is partial)
@pytest.mark.parametrize("nd,n_sources", [(720, 2), (712, 2), (1016, 1), (1008, 1), (720, 5), (61, 17)])
def test_integer_dither_seeds_on_both_sides(nd, n_sources):
    """dlx_psf_backward's fluxes against their definition sum_p h bs, h = sum_f flat r in window f, from the same
    plan's single-star images; positions by the same seed weights."""
    from tests.gpu_helpers import dev
    from tests.test_gpu_dither import plan_for
    print(f"dither seeds nd={nd} stars={n_sources}", flush=True)
    margin = 4
    w = make_dithered_workload(n_pupil=16, n_det=nd, oversample=1, margin=margin, n_sources=n_sources,
                               det_pixel_mas=100.0, wavelengths=(600e-9,), dithers=((0, 0), (4, -3), (-2, 1)),
                               flux=(1e6, 1e7))
    rng = np.random.default_rng(nd)
    p = w.eval_params()
    flat = rng.normal(1.0, 0.05, (nd, nd)).astype(np.float32)
    r = rng.normal(size=(3, nd, nd)).astype(np.float32)
    plan = plan_for(w)
    args = (dev(p["coeffs"]), None, dev(p["sources"]), dev(flat))
    plan.forward(*args)
    gs = plan.backward(*args, dev(r))[2].cpu().numpy()
    # star s alone with unit flux: its image on the detector, frame by frame
    for s in {0, n_sources - 1}:
        one = np.array(p["sources"])
        one[..., 2] = 0.0
        one[..., s, 2] = 1.0
        b, _ = plan.forward(args[0], None, dev(one), args[3])
        b = b.cpu().numpy().astype(np.float64)
        want = np.sum(flat * r * b)
        size = np.sum(np.abs(flat * r) * b)
        # h is an FP32 sum of up to three products, b is rounded to FP32: 5 roundings of 2^-24
        assert abs(gs.reshape(-1, 3)[s, 2] - want) <= 5 * 2.0 ** -24 * size
    assert plan.sync() == 0
    plan.close()
