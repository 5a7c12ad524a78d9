"""max_rel_h where its denominator changes sign: rays that hover at the horizon (no
capture buffer, steps in s), where Delta is a rounding error of either sign.  A ratio
replaces the running one where Kabs > running * D: with D > 0 a larger one does, with
D < 0 and a negative running one a ratio of larger magnitude.  So among values of one
sign the magnitude never falls along a ray."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("a", [0.9, -0.7])
def test_running_ratio_at_the_horizon(a):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2202_00086_amd import kerrtrace as K
    print("[gpu-case] max_rel_h at the horizon", a, flush=True)
    sys.stdout.flush()
    params = dict(M=1.0, a=a, r_obs=4.0, incl=1.2, fov_x=1.5, fov_y=1.5, nx=16, ny=12, method=0, h_fixed=1.0 / 8,
                  cap_buffer=0.0, r_escape=40.0)
    before, falls, negative = None, 0, 0
    # one more step per render
    for budget in range(1, 1200):
        r = K.Renderer(device="cuda:0", want=("fate", "max_rel_h"), stats=False, **dict(params, max_steps=budget))
        out = r.render()["max_rel_h"].cpu().numpy()
        if before is not None:
            with np.errstate(invalid="ignore"):
                falls += int(((np.sign(out) == np.sign(before)) & (np.abs(out) < np.abs(before) * (1 - 1e-15))).sum())
        negative += int((out < 0).sum())
        before = out
    print(f"[max_rel_h] {negative} negative values, {falls} falls", flush=True)
    assert negative > 0 and falls == 0
