"""Stars outside the region that a PSF table's launches are sized for: only the blocks of the table that some star
reaches are transformed, and a star beyond the sampled field has its own at every wavelength.

Against the same plan's dense per-star form; and what the blocks that are left out still hold from an earlier
evaluation, finite or not, must not come back.
"""
import functools

import numpy as np
import pytest

import oracle as O
from synth import make_workload
from tests.helpers import oracle_problem
from tests.test_gpu_table import _against_per_star_form

pytestmark = pytest.mark.gpu


@functools.lru_cache(maxsize=None)
def workload(q=3, n_pupil=97, n_focal=177, n_wl=32, frames=8):
    return make_workload("c3", n_pupil=n_pupil, n_focal=n_focal, oversample=q, n_wavelengths=n_wl, n_frames=frames,
                         noll=tuple(range(2, 8)))


def with_counts(w, src):
    """Counts of the images that the truth's coefficients and flat give for these positions."""
    return w.with_data(O.forward(oracle_problem(w), w.coeffs_true, None, src, w.flat_true)[1])


def reach(w):
    P = w.problem
    return float(np.min(P.wavelengths)) * P.n_pupil / (2 * P.diameter)


# positions in units of half the sampled field: alone and together, along one axis and both, up to its edge and past it
PLACES = {"x": [(0, 0, 0.7, 0)], "y": [(2, 1, 0, -0.8)], "corner": [(1, 0, 0.99, -0.99)], "several": [(0, 0, 0.6, 0.1), (3, 1, -0.9, 0.5),
          (7, 0, 0.2, 0.95)], "far x": [(4, 1, 1.4, 0.0)], "far both": [(5, 0, -2.7, 3.3)],
          "far and near": [(0, 0, 1.05, 0.3), (2, 1, 0.8, 0.8), (6, 0, -2.0, 0.01), (6, 1, 1.3, -1.3)]}


@pytest.mark.parametrize("place", list(PLACES))
@pytest.mark.parametrize("q,n_pupil,n_focal,n_wl", [(3, 97, 177, 32), (1, 128, 128, 70)])
def test_outlying_stars_match_the_per_star_form(place, q, n_pupil, n_focal, n_wl):
    print(f"outlying stars {place} q={q}", flush=True)
    w = workload(q, n_pupil, n_focal, n_wl)
    src, true, half = np.array(w.sources), np.array(w.sources_true), reach(w)
    for f, s, x, y in PLACES[place]:
        src[f, s, :2] += (x * half, y * half)
        true[f, s, :2] += (x * half, y * half)
    _against_per_star_form(with_counts(w, true.astype(np.float32)), src.astype(np.float32), 1e-5)


def test_blocks_left_out_hold_nothing_of_earlier_evaluations():
    """Everything is NaN after an evaluation with a coefficient that is not finite; the next ones, in the graph and
    out of it, near, outlying, far and near again, give the bits of a plan that never saw it."""
    import torch
    from paper_2406_08703_amd import CapturedEval
    from tests.gpu_helpers import dev, make_plan, run_eval
    print("outlying stars after NaN", flush=True)
    w = workload()
    w = with_counts(w, w.sources_true)
    p, half = w.eval_params(), reach(w)
    places = [np.array(w.sources)]
    for x, y in ((0.8, -0.5), (1.3, 0.4), (0.0, 0.0)):
        src = np.array(w.sources)
        src[3, 0, :2] += (x * half, y * half)
        places.append(src)
    clean = make_plan(w)
    want = [run_eval(w, params=dict(p, sources=s), kind="chi2", plan=clean) for s in places]
    clean.close()
    plan = make_plan(w)
    everywhere = np.array(w.sources)
    everywhere[0, 0, :2] = (0.99 * half, 0.99 * half)   # the whole table in use
    everywhere[1, 0, :2] = (1.9 * half, -1.7 * half)
    bad = np.array(p["coeffs"])
    bad[2] = np.nan
    held = dev(p["sources"])
    cap = CapturedEval(plan, dev(p["coeffs"]), None, held, dev(p["flat"]), dev(w.data), "chi2", w.prior_mu, w.prior_sigma)
    for replay in (False, True):
        for src, ref in zip(places, want):
            run_eval(w, params=dict(p, coeffs=bad, sources=everywhere), kind="chi2", plan=plan)
            if replay:
                held.copy_(dev(src))
                o = cap.replay()
                torch.cuda.synchronize()
                got = dict(model=o.model, r=o.r, grad_flat=o.grad_flat, grad_sources=o.grad_sources,
                           grad_coeffs=o.grad_zernike[:w.problem.n_zernike])
                got = {k: v.cpu().numpy() for k, v in got.items()}
            else:
                got = run_eval(w, params=dict(p, sources=src), kind="chi2", plan=plan)
            for k in ("model", "r", "grad_flat", "grad_sources", "grad_coeffs"):
                assert np.all(np.isfinite(ref[k]))
                np.testing.assert_array_equal(got[k], ref[k])
    plan.close()
