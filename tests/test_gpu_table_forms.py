"""Which form a plan takes, a shared PSF table or one transform per star, where the flags meet."""
import numpy as np
import pytest

from synth import make_workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("frames", [(8,), (8, 1), (1, 1)])
def test_the_grouped_flag_changes_nothing_where_it_does_not_apply(frames):
    """DLX_FLAG_GROUPED runs problems of one frame together, each star with its own transforms. With a problem of
    several frames it does not apply: every problem takes the form it takes without the flag, to the bit."""
    import torch
    from paper_2406_08703_amd import BatchPlan
    from paper_2406_08703_amd import dlx as C
    from tests.gpu_helpers import geometry
    print(f"grouped flag, frames {frames}", flush=True)
    ws = [make_workload("c3", n_pupil=97, n_focal=177, n_wavelengths=32, n_frames=f, noll=(2, 3, 4)) for f in frames]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32))
    got = []
    for grouped in (False, True):
        bp = BatchPlan([geometry(w) for w in ws], [t(w.transmission) for w in ws], [t(w.zbasis) for w in ws],
                       intrapixels=[t(w.intrapixel) for w in ws], grouped=grouped)
        p = [w.eval_params() for w in ws]
        d = bp.pack("images", [torch.full((w.problem.n_frames, 59, 59), 50.0) for w in ws])
        out = bp.buffers()
        a = bp.eval_args(bp.pack("zernike_coeffs", [t(e["coeffs"]) for e in p]), None,
                         bp.pack("sources", [t(e["sources"]) for e in p]), bp.pack("flat", [t(e["flat"]) for e in p]), d, out,
                         "chi2", 1.0, 0.05)
        C.dlx_plan_profile(bp.plan, True)
        bp.evaluate(a)
        assert bp.sync() == 0
        n = C.dlx_plan_stage_times(bp.plan)["F1"][2]
        got.append((n, {k: v.cpu().numpy() for k, v in out.items() if v is not None}))
        bp.close()
    (n0, a), (n1, b) = got
    # 32 wavelengths on a table, 2 stars of 32 wavelengths of one frame
    assert n0 == n1 == sum(32 if f > 1 else 64 for f in frames)
    if max(frames) > 1:
        for k in a:
            np.testing.assert_array_equal(a[k], b[k])
    else:   # the flag applies: the same images, sums in another order
        np.testing.assert_array_equal(a["binned"], b["binned"])
