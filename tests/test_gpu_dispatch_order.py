"""The dispatch order's key does not depend on the unit of length: an image whose
lengths are all scaled by a power of two has the same bins."""
import sys

import numpy as np
import pytest

from paper_2202_00086_amd import workloads as W

pytestmark = pytest.mark.gpu

LENGTHS = ("M", "a", "r_obs", "fov_x", "fov_y", "h_init", "cap_buffer", "r_escape", "r_src", "r_in", "r_out")


def _bins(K, params):
    """The bins of the last render, from its workspace (256-byte aligned parts:
    the parameters up to byte 2048, 8 bytes per ray, 4 bytes per ray, 1025
    counts, 2 bytes per ray)."""
    import torch
    r = K.Renderer(device="cuda:0", want=("fate",), stats=False, launch=K.kt_launch(1, 256, 1, 4), **params)
    r.render()
    torch.cuda.synchronize()
    at = 2048
    for part in (8 * r.n, 4 * r.n, 4 * 1025):
        at = (at + part + 255) // 256 * 256
    return r.ws[at:at + 2 * r.n].cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("a,incl", [(0.9, 1.05), (-0.98, 1.57), (1.0, 0.3), (0.0, 1.4)])
@pytest.mark.parametrize("power", [-40, -3, 20, 45, 62])
def test_bins_do_not_depend_on_the_unit_of_length(power, a, incl):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2202_00086_amd import kerrtrace as K
    print("[gpu-case] dispatch bins", power, a, incl, flush=True)
    sys.stdout.flush()
    params = dict(W.kerr_ring(a, n=64), incl=incl, nx=72, ny=57, max_steps=2000)
    want = _bins(K, params)
    scaled = dict(params, **{k: params[k] * 2.0 ** power for k in LENGTHS if k in params})
    scaled["atol"] *= min(1.0, 2.0 ** power)
    assert want.max() < 1024 and np.unique(want).size > 50
    np.testing.assert_array_equal(_bins(K, scaled), want)
