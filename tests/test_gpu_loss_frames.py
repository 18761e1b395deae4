"""The loss terms and seed weights of several frames, shared out over the waves of a block.

Detector sizes around the 256 pixels of a block and the 1024 blocks from which one wave runs its frames
alone; frame counts around the 16 waves of a block. Against NumPy in float64: every sum has positive and
negative terms of known size, so it is held to 1e-13 of the sum of their magnitudes (2^-53 per addition of
at most a few hundred per partial, 1 ulp of the logarithm); the residual is rounded to float32 once.
"""
import numpy as np
import pytest

from synth import make_workload

pytestmark = pytest.mark.gpu


def terms(m, b, d, flat, kind, mu, sigma):
    m, b, d, flat = (np.asarray(a, np.float32).astype(np.float64) for a in (m, b, d, flat))
    if kind == "poisson":
        ell, r = m - np.where(d != 0, d * np.log(m), 0.0), 1.0 - d / m
    else:
        wt = np.maximum(d, 1.0)
        ell, r = 0.5 * (m - d) ** 2 / wt, (m - d) / wt
    prior, dprior = 0.5 * ((flat - mu) / sigma) ** 2, (flat - mu) / sigma ** 2
    return (ell.sum() + prior.sum(), np.abs(ell).sum() + prior.sum(), r, (r * b).sum(0) + dprior,
            np.abs(r * b).sum(0) + np.abs(dprior))


@pytest.mark.parametrize("kind", ["poisson", "chi2"])
@pytest.mark.parametrize("nd,frames", [(5, 2), (16, 3), (17, 16), (33, 17), (47, 40), (511, 2), (512, 3)])
def test_loss_of_several_frames_matches_float64(nd, frames, kind):
    from paper_2406_08703_amd import PsfPlan
    from tests.gpu_helpers import dev, geometry
    print(f"loss nd={nd} frames={frames} {kind}", flush=True)
    w = make_workload("c3", n_pupil=16, n_focal=nd, oversample=1, n_wavelengths=1, n_frames=frames,
                      noll=(2, 3))
    plan = PsfPlan(geometry(w), dev(w.transmission), dev(w.zbasis), None, None)
    rng = np.random.default_rng(nd * frames)
    shape = (frames, nd, nd)
    m, b = rng.uniform(0.5, 300.0, shape).astype(np.float32), rng.uniform(0.5, 300.0, shape).astype(np.float32)
    d = rng.poisson(100.0, shape).astype(np.float32) * (rng.uniform(size=shape) > 0.1)
    flat = rng.normal(1.0, 0.05, (nd, nd)).astype(np.float32)
    L, r, gF = plan.loss_grad(dev(m), dev(b), dev(d), dev(flat), kind, 1.0, 0.1)
    assert plan.sync() == 0
    plan.close()
    loss, size, rr, g, gsize = terms(m, b, d, flat, kind, 1.0, 0.1)
    assert abs(float(L[0]) - loss) <= 1e-13 * size
    np.testing.assert_allclose(r.cpu().numpy(), rr.astype(np.float32), rtol=2.0 ** -23, atol=2.0 ** -52)
    assert np.all(np.abs(gF.cpu().numpy() - g) <= 1e-13 * gsize)


@pytest.mark.parametrize("q,nd,frames,per_pixel", [(1, 17, 3, False), (2, 9, 17, False), (3, 21, 2, False),
                                                   (3, 11, 5, True), (4, 16, 2, False), (5, 7, 18, False)])
def test_fused_seed_of_several_frames_matches_the_separate_calls(q, nd, frames, per_pixel):
    """dlx_eval's seed weights and flux partials against dlx_loss_grad and dlx_psf_backward, which form them one
    pixel per thread: the same seed weights, so the same optics gradients; the fluxes' sums differ in order."""
    from paper_2406_08703_amd import PsfPlan, evaluate
    from tests.gpu_helpers import dev, geometry
    print(f"seed q={q} nd={nd} frames={frames} per_pixel={per_pixel}", flush=True)
    w = make_workload("c3", n_pupil=24, n_focal=q * nd, oversample=q, n_wavelengths=2, n_frames=frames,
                      noll=(2, 3, 4))
    rng = np.random.default_rng(q)
    k = 1.0 + 0.1 * rng.normal(size=(nd, nd, q, q) if per_pixel else (q, q))
    plan = PsfPlan(geometry(w), dev(w.transmission), dev(w.zbasis), None, dev(k), pixel_kernel=per_pixel)
    p = w.eval_params()
    data = rng.poisson(50.0, (frames, nd, nd))
    args = (dev(p["coeffs"]), None, dev(p["sources"]), dev(p["flat"]))
    got = evaluate(plan, *args, dev(data), "chi2", w.prior_mu, w.prior_sigma)
    b, m = plan.forward(*args)
    L, r, gF = plan.loss_grad(m, b, dev(data), args[3], "chi2", w.prior_mu, w.prior_sigma)
    gz, _, gs = plan.backward(*args, r)
    assert plan.sync() == 0
    plan.close()
    np.testing.assert_array_equal(got.r.cpu().numpy(), r.cpu().numpy())
    np.testing.assert_array_equal(got.grad_flat.cpu().numpy(), gF.cpu().numpy())
    np.testing.assert_array_equal(got.grad_zernike.cpu().numpy()[:3], gz.cpu().numpy())
    gs, ge = gs.cpu().numpy(), got.grad_sources.cpu().numpy()
    np.testing.assert_array_equal(ge[..., :2], gs[..., :2])
    # flux: sums of at most nd^2 doubles whose magnitudes add up to no more than sum |flat r| max(bs)
    size = np.abs(p["flat"] * r.cpu().numpy()).sum() * (b.cpu().numpy().max() / p["sources"][..., 2].min())
    assert np.all(np.abs(ge[..., 2] - gs[..., 2]) <= 1e-13 * size)


@pytest.mark.parametrize("q,nd,L,frames,per_pixel", [(1, 13, 9, 2, True), (2, 11, 11, 3, True), (2, 11, 9, 2, False),
                                                     (3, 9, 5, 2, True), (4, 8, 3, 2, False), (4, 8, 5, 2, True)])
def test_intrapixel_gradient_past_the_wavelengths_loaded_at_once(q, nd, L, frames, per_pixel):
    """Wavelength counts that leave a remainder of the 8, 8, 4 and 2 that kgrad_kernel loads together for
    Q = 1 .. 4, and pixels past the last whole wave; held, as the other intra-pixel tests are, to 1e-5 of the
    gradient's own scale sum |F r| B / Q^2 (per pixel with one kernel per pixel)."""
    import oracle as O
    from paper_2406_08703_amd import PsfPlan, evaluate
    from tests.gpu_helpers import dev, geometry
    from tests.helpers import oracle_problem
    print(f"intra-pixel gradient q={q} L={L} per_pixel={per_pixel}", flush=True)
    w = make_workload("c3", n_pupil=24, n_focal=q * nd, oversample=q, n_wavelengths=L, n_frames=frames, noll=(2, 3, 4))
    rng = np.random.default_rng(L)
    k = 1.0 + 0.05 * rng.normal(size=(nd, nd, q, q) if per_pixel else (q, q))
    import dataclasses
    w = dataclasses.replace(w, intrapixel=k.astype(np.float32))
    prob = oracle_problem(w)
    p = w.eval_params()
    data = rng.poisson(50.0, (frames, nd, nd)).astype(np.float64)
    ref = O.value_and_grad(prob, p["coeffs"], None, p["sources"], p["flat"], data, "chi2", w.prior_mu, w.prior_sigma)
    want = O.intrapixel_grad(prob, p["coeffs"], None, p["sources"], p["flat"], ref["r"])
    plan = PsfPlan(geometry(w), dev(w.transmission), dev(w.zbasis), None, dev(w.intrapixel), pixel_kernel=per_pixel)
    got = evaluate(plan, dev(p["coeffs"]), None, dev(p["sources"]), dev(p["flat"]), dev(data), "chi2", w.prior_mu,
                   w.prior_sigma, intrapixel_grad=True).grad_intrapixel.cpu().numpy()
    assert plan.sync() == 0
    plan.close()
    size = np.abs(np.asarray(p["flat"], np.float64)[None] * ref["r"]) * ref["binned"]
    scale = size.sum(0).max() if per_pixel else size.sum()
    assert np.max(np.abs(got - want)) / (scale / (q * q)) < 1e-5
