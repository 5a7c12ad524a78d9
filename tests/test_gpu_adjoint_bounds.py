"""kt_adjoint's stored passes where a bound of theirs takes effect: the step
budget, the store's room, the records and the segment items.  The one-lane path
(split_above -1) decides there, so both must count the same rays and give the
same gradients, to the bound of the split sweeps."""
import ctypes as C
import sys

import numpy as np
import pytest

from paper_2202_00086_amd import workloads as W
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


def _forward(K, params):
    import torch
    r = K.Renderer(device="cuda:0", want=("fate", "r_hit", "n_cross", "n_steps"), stats=False, **params)
    out = r.render()
    torch.cuda.synchronize()
    return r, out


def _adjoint(K, r, out, integ, n_steps, more=0):
    """Gradient maps, stats and the workspace's counters (uint32 from byte 16 on)."""
    import torch
    nbytes = K.kt_adjoint_workspace_bytes(r.cam, integ) + more
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda:0")
    cot = torch.linspace(-1.0, 2.0, r.n, dtype=torch.float64, device="cuda:0")
    grads = [torch.full((r.n,), 7.0, dtype=torch.float64, device="cuda:0") for _ in range(3)]
    stats = torch.empty(4, dtype=torch.int64, device="cuda:0")
    code = K.kt_adjoint(r.cam, r.st, r.disk, integ, out["fate"].data_ptr(), out["r_hit"].data_ptr(), cot.data_ptr(),
                        grads[0].data_ptr(), grads[1].data_ptr(), grads[2].data_ptr(), stats.data_ptr(),
                        ws.data_ptr(), nbytes, C.c_void_p(torch.cuda.current_stream().cuda_stream),
                        n_steps.data_ptr(), None)
    assert code == K.KT_OK, K.kt_last_error()
    torch.cuda.synchronize()
    return [g.cpu().numpy() for g in grads], stats.cpu().numpy(), ws[16:64].cpu().numpy().view(np.uint32)


@pytest.mark.parametrize("every", [1, 64])
@pytest.mark.parametrize("max_steps", [1, 100, 200, 500])
def test_budget_smaller_than_the_renders(K, max_steps, every):
    """max_steps bounds the adjoint's attempts (16 times as many) and its
    checkpoints, not the accepted steps: a ray that takes more than max_steps of
    them but fits the checkpoints has its gradient, stored or not."""
    params = W.differentiable_disk(n=33)
    _announce("adjoint budget", max_steps, every)
    r, out = _forward(K, params)
    small = dict(params, max_steps=max_steps, checkpoint_every=every)
    want, want_st, _ = _adjoint(K, r, out, K.make_structs(**dict(small, split_above=-1))[4], out["n_steps"])
    got, st, _ = _adjoint(K, r, out, K.make_structs(**small)[4], out["n_steps"])
    assert st.tolist() == want_st.tolist()
    steps = out["n_steps"].cpu().numpy()[out["fate"].cpu().numpy() == K.DISK]
    assert want_st.sum() == steps.size
    if every == 64 and max_steps in (100, 200):
        assert want_st[0] > (steps <= max_steps).sum()  # rays over the budget within the checkpoints
    for a, b in zip(got, want):
        if want_st[0] > 0:
            _assert_split_close(a, b)
