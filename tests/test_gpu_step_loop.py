"""The edges of the trace kernels' step loop, of the default launch's rule and
of the adjoint's stored forward passes: images of a wave, a block and one ray
more, budgets that end inside a refill, disks seen edge on, spheres inside and
outside the camera's, against the oracle (the parity rules' own 1e-8); and
launches on both sides of each line of the rule, which must agree bit for bit;
and the adjoint with step counts that are too small, too large or missing."""
import ctypes as C
import math
import sys

import numpy as np
import pytest

import oracle as O
from paper_2202_00086_amd import workloads as W
from tests import parity as P
from tests.test_gpu_adjoint import _assert_split_close

pytestmark = pytest.mark.gpu


def _announce(*what):
    print("[gpu-case]", *what, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def K():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2202_00086_amd import kerrtrace
    return kerrtrace


def _render(K, params, launch=None):
    import torch
    r = K.Renderer(device="cuda:0", launch=launch, **params)
    out = r.render()
    torch.cuda.synchronize()
    return {k: v.cpu().numpy() for k, v in out.items() if k != "stats"}


def _same(a, b, what):
    for key in a:
        np.testing.assert_array_equal(a[key].view(np.uint8), b[key].view(np.uint8), err_msg=f"{what} {key}")


RING = dict(W.kerr_ring(0.9, n=8))
DISK = dict(W.schwarzschild_disk(n=8))
SHAPES = {
    "one wave": dict(RING, nx=8, ny=8),
    "one wave and a ray": dict(RING, nx=13, ny=5),
    "a block and a ray": dict(RING, nx=257, ny=1),
    "one ray, edge on": dict(DISK, nx=1, ny=1, incl=math.pi / 2),
    "edge on, a row in the disk plane": dict(DISK, nx=31, ny=9, incl=math.pi / 2),
    "source inside the camera's sphere": dict(RING, nx=19, ny=11, r_src=0.5 * RING["r_obs"]),
    "source at the escape radius": dict(RING, nx=19, ny=11, r_src=1.1 * RING["r_obs"], r_escape=1.1 * RING["r_obs"]),
    "source and disk": dict(RING, nx=19, ny=11, disk_on=1, r_in=3.0, r_out=20.0),
    "Bulirsch-Stoer, a wave and a ray": dict(RING, nx=13, ny=5, method=4),
    "rational Bulirsch-Stoer, a disk": dict(DISK, nx=17, ny=15, method=5),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_edges_match_the_oracle(K, name):
    params = SHAPES[name]
    nx, ny = params["nx"], params["ny"]
    _announce("step loop", name, nx, ny)
    g = _render(K, params)
    o = O.trace_pixels(O.Setup(**params))
    P.check_fates(g["fate"], o["fate"], nx, ny, min_allowed=1)
    m = P.value_mask(g, o, nx, ny)
    for key in ("deflection", "r_hit", "g"):
        if key in g:
            P.check_values(g, o, key, m, rtol=1e-8)


@pytest.mark.parametrize("method", [0, 1, 4])
@pytest.mark.parametrize("budget", [1, 2, 63])
def test_budgets_end_every_ray_alike(K, method, budget):
    """A ray ends after `budget` accepted steps or 16 `budget` evaluations,
    whichever comes first, on every launch shape."""
    params = dict(RING, nx=33, ny=21, method=method, max_steps=budget, r_src=4.0 * RING["r_obs"],
                  r_escape=4.0 * RING["r_obs"], h_fixed=1.0 / 128)
    _announce("budget", method, budget)
    g = _render(K, params)
    o = O.trace_pixels(O.Setup(**params))
    P.check_fates(g["fate"], o["fate"], 33, 21, min_allowed=1)
    for end in (o, g):
        over = end["fate"] == O.MAXSTEPS
        assert ((end["n_steps"] == budget) | (end["n_evals"] >= 16 * budget))[over].all()
    by_evals = (o["fate"] == O.MAXSTEPS) & (g["fate"] == O.MAXSTEPS) & (o["n_steps"] < budget) & (g["n_steps"] < budget)
    np.testing.assert_array_equal(g["n_evals"][by_evals], o["n_evals"][by_evals])
    _same(g, _render(K, params, K.kt_launch(1, 64, 1, 1)), "one block per CU")
    _same(g, _render(K, params, K.kt_launch(1, 256, 3, 4)), "three waves")


# rays per lane of one wave per SIMD at which the default changes, and one row more
@pytest.mark.parametrize("nx,ny,method", [(512, 512, 1), (512, 513, 1), (2048, 1023, 1), (2048, 1024, 1),
                                          (768, 768, 4), (768, 769, 4)])
def test_default_launch_on_both_sides_of_its_lines(K, nx, ny, method):
    params = dict(RING, nx=nx, ny=ny, method=method)
    _announce("default launch", nx, ny, method)
    g = _render(K, params)
    _same(g, _render(K, params, K.kt_launch(1, 256, 2, 16)), "two waves")


def _adjoint(K, torch, r, out, cot, integ, n_steps):
    nbytes = K.kt_adjoint_workspace_bytes(r.cam, integ)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
    grads = [torch.full((r.n,), 7.0, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    stats = torch.empty(4, dtype=torch.int64, device="cuda:0")
    code = K.kt_adjoint(r.cam, r.st, r.disk, integ, out["fate"].data_ptr(), out["r_hit"].data_ptr(), cot.data_ptr(),
                        grads[0].data_ptr(), grads[1].data_ptr(), grads[2].data_ptr(), stats.data_ptr(),
                        ws.data_ptr(), nbytes, C.c_void_p(torch.cuda.current_stream().cuda_stream),
                        n_steps.data_ptr() if n_steps is not None else None, None)
    assert code == K.KT_OK, K.kt_last_error()
    torch.cuda.synchronize()
    return [g.cpu().numpy() for g in grads], stats.cpu().numpy()


@pytest.mark.parametrize("nx,ny", [(1, 1), (8, 8), (65, 1), (33, 31)])
def test_stored_passes_equal_the_one_lane_path(K, nx, ny):
    """The stored passes and their sweep give the one-lane path's gradients, to
    the bound of the split sweeps (the two kernels' multiply-adds are fused
    differently), with the render's step counts and with counts that are too
    small for some rays, too large, or beyond what the checkpoints cover; where
    no ray finds room or none has a bin, the one-lane path runs them all and
    the gradients are the same bits."""
    import torch
    params = dict(W.differentiable_disk(n=8), nx=nx, ny=ny)
    _announce("stored passes", nx, ny)
    r = K.Renderer(device="cuda:0", want=("fate", "r_hit", "n_cross", "n_steps"), stats=False, **params)
    out = r.render()
    torch.cuda.synchronize()
    cot = torch.linspace(-1.0, 2.0, r.n, dtype=torch.float64, device="cuda:0")
    n = out["n_steps"]
    base, base_st = _adjoint(K, torch, r, out, cot,
                             K.make_structs(**dict(params, checkpoint_every=64, split_above=-1))[4], None)
    assert base_st[1:].tolist() == [0, 0, 0]
    counts = {"the render's": n, "none": torch.zeros_like(n), "half": n // 2, "double": 2 * n, "negative": -n,
              "every third too small": torch.where(torch.arange(r.n, device=n.device) % 3 == 0, n // 4, n),
              "long": torch.full_like(n, 3000), "beyond the list's bins": torch.full_like(n, 1 << 20)}
    for every in (1, 64):
        integ = K.make_structs(**dict(params, checkpoint_every=every, split_above=1 << 20))[4]
        for what, steps in counts.items():
            _announce("  step counts", every, what)
            maps, st = _adjoint(K, torch, r, out, cot, integ, steps.contiguous())
            assert st.tolist() == base_st.tolist(), (every, what)
            for a, b in zip(maps, base):
                if base_st[0] > 0:
                    _assert_split_close(a, b)
                if what not in ("none", "negative", "beyond the list's bins"):
                    continue
                np.testing.assert_array_equal(a.view(np.uint8), b.view(np.uint8), err_msg=f"{every} {what}")


@pytest.mark.parametrize("n,incl_deg,a", [(96, 60.0, 0.5), (420, 25.0, 0.9), (360, 45.0, 0.7)])
def test_sweeps_do_not_depend_on_who_runs_them(K, n, incl_deg, a):
    """The waves of the forward pass sweep rays of their own (360x360, 96x96) or
    none (420x420, nearly face on: every lane has enough to do).  Where a sweep
    is cut and who goes on with it changes from run to run, the gradients do
    not, and they equal the one-lane path's to the bound of the split sweeps."""
    import torch
    params = W.differentiable_disk(n=n, incl_deg=incl_deg, a=a)
    _announce("sweeps", n, incl_deg, a)
    r = K.Renderer(device="cuda:0", want=("fate", "r_hit", "n_cross", "n_steps"), stats=False, **params)
    out = r.render()
    torch.cuda.synchronize()
    cot = torch.linspace(-1.0, 2.0, r.n, dtype=torch.float64, device="cuda:0")
    first, first_st = _adjoint(K, torch, r, out, cot, r.integ, out["n_steps"])
    for _ in range(3):
        maps, st = _adjoint(K, torch, r, out, cot, r.integ, out["n_steps"])
        assert st.tolist() == first_st.tolist()
        for x, y in zip(maps, first):
            np.testing.assert_array_equal(x.view(np.uint8), y.view(np.uint8))
    lane, lane_st = _adjoint(K, torch, r, out, cot, K.make_structs(**dict(params, split_above=-1))[4], out["n_steps"])
    assert lane_st.tolist() == first_st.tolist() and lane_st[1:].tolist() == [0, 0, 0]
    for x, y in zip(first, lane):
        _assert_split_close(x, y)


SPHERE = dict(src_on=1, r_src=700.0)
THIN = dict(disk_on=1, r_in=6.0, r_out=30.0)
SKY = dict(sky_on=1, grid_deg=6.0, line_deg=0.25)


@pytest.mark.parametrize("method,options", [(1, {}), (1, SPHERE), (1, THIN), (1, SKY), (1, dict(SPHERE, **THIN)),
                                            (1, dict(SPHERE, **SKY)), (1, dict(THIN, **SKY)),
                                            (1, dict(SPHERE, **THIN, **SKY)), (0, {}), (0, dict(SPHERE, **THIN))],
                         ids=str)
@pytest.mark.parametrize("waves", [1, 3])
def test_spin_zero_equals_the_general_right_hand_side(K, method, options, waves):
    """A spin of 1e-200 takes the general right-hand side, and its terms vanish
    against the others in every sum: the same bits as a spin of 0, which takes
    the right-hand side without them."""
    params = dict(W.schwarzschild_disk(n=8), disk_on=0, nx=38, ny=27, method=method, h_fixed=1.0 / 64, r_obs=900.0,
                  r_escape=990.0)
    params.update(options)
    _announce("spin 0", method, options, waves)
    launch = K.kt_launch(1, 256, waves, 4)
    _same(_render(K, dict(params, a=0.0), launch), _render(K, dict(params, a=1e-200), launch), "a = 0")
