"""Nyquist pixels with one sample each, on a shared PSF table: the coarsest focal grids, whose interpolation takes
the longest windows that are compiled (72 and 80 table samples here), against the FP64 oracle.

The chi-squared data term: at these sizes the faintest of the two million pixels hold 1e-9 of the brightest, where
an error of eta sqrt(m m_max) in the model, which one FP32 transform per star leaves as well, is 1e-5 and more of
1 - d / m; (m - d) / max(d, 1) does not divide by the model.
"""
import pytest

import oracle as O
from synth import make_workload
from tests.helpers import oracle_problem
from tests.test_gpu_table import transforms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("band,frames,n_wl", [((545e-9, 645e-9), 8, 10), ((450e-9, 700e-9), 8, 10)])
def test_nyquist_pixels_without_oversampling_match_the_oracle(band, frames, n_wl):
    from tests.gpu_helpers import make_plan, run_eval
    from tests.test_gpu_parity import compare
    print(f"table Q=1 Nyquist {band}", flush=True)
    w = make_workload("c5", n_pupil=384, n_focal=512, oversample=1, band=band, centre=0.5 * sum(band),
                      n_wavelengths=n_wl, n_frames=frames, noll=tuple(range(2, 12)), n_map=0)
    prob = oracle_problem(w)
    w = w.with_data(O.forward(prob, w.coeffs_true, None, w.sources_true, w.flat_true)[1])
    p = w.eval_params()
    ref = O.value_and_grad(prob, p["coeffs"], None, p["sources"], p["flat"], w.data, "chi2", w.prior_mu,
                           w.prior_sigma)
    plan = make_plan(w)
    n, got = transforms(plan, lambda: run_eval(w, kind="chi2", plan=plan))
    plan.close()
    assert n == n_wl   # one transform per wavelength: the plan is on a table
    assert got["status"] == 0
    compare(got, ref, q=1, kind="chi2")
