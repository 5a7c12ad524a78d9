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


def _compare(K, r, out, params, n_steps, more, split_above):
    """The stored passes' counters, after comparing them with the one-lane path."""
    want, want_st, _ = _adjoint(K, r, out, K.make_structs(**dict(params, split_above=-1))[4], out["n_steps"])
    got, st, c = _adjoint(K, r, out, K.make_structs(**dict(params, split_above=split_above))[4], n_steps, more)
    assert st.tolist() == want_st.tolist() and want_st[1:].tolist() == [0, 0, 0]
    for a, b in zip(got, want):
        _assert_split_close(a, b)
    listed, split, stored = int(want_st[0]), int(c[0]), int(c[4]) - int(c[3])
    print(f"[adjoint] listed {listed} stored {stored} split {split} store {c[1]} items {c[2]} redone {c[7]}", flush=True)
    return listed, stored, split, int(c[3])


@pytest.mark.parametrize("split_above", [0, 1, 400, 1 << 20])
@pytest.mark.parametrize("inflate", [1500, 2500, 3700])
def test_store_that_holds_some_of_the_rays(K, inflate, split_above):
    """Step counts of every second ray so much too large that the store is full
    before the shorter bins: those take the one-lane path, in the memory that the
    store had."""
    import torch
    params = W.differentiable_disk(n=33)
    _announce("adjoint part of the rays stored", inflate, split_above)
    r, out = _forward(K, params)
    n = out["n_steps"]
    steps = torch.where(torch.arange(r.n, device=n.device) % 2 == 0, n + inflate, n).contiguous()
    listed, stored, _, _ = _compare(K, r, out, params, steps, 0, split_above)
    assert 0 < stored < listed


def test_store_that_holds_too_few_of_the_rays_is_left_empty(K):
    """Every ray's count at the store's bin limit: it would hold a quarter of them."""
    import torch
    params = W.differentiable_disk(n=33)
    _announce("adjoint store left empty")
    r, out = _forward(K, params)
    listed, stored, split, _ = _compare(K, r, out, params, torch.full_like(out["n_steps"], 4080), 0, 0)
    assert stored == split == 0


@pytest.mark.parametrize("every", [1, 64, 1024])
def test_longest_rays_ahead_of_the_stored_ones(K, every):
    """Counts beyond the bins' range (4092 steps) for every third ray: those take the
    one-lane path and the stored rays start behind them in the list."""
    import torch
    params = dict(W.differentiable_disk(n=33), checkpoint_every=every)
    _announce("adjoint long rays ahead", every)
    r, out = _forward(K, params)
    n = out["n_steps"]
    steps = torch.where(torch.arange(r.n, device=n.device) % 3 == 0, torch.full_like(n, 5000), n).contiguous()
    listed, stored, _, first = _compare(K, r, out, params, steps, 64 << 20, 0)
    assert first > 0 and first + stored == listed


def test_items_for_some_of_the_splits(K):
    """A threshold that asks for more segments than there is room for: the longest
    rays are split, the others swept whole (the longest ray's count is beyond the bins)."""
    import torch
    params = W.differentiable_disk(n=33)
    _announce("adjoint segment items")
    r, out = _forward(K, params)
    listed, stored, split, _ = _compare(K, r, out, params, out["n_steps"] + 3500, 128 << 20, 1)
    assert 0 < split < stored == listed - 1


def test_more_rays_than_records(K):
    """1024x1024 at 20 degrees: 600 thousand rays, of which 524288 have a record,
    with a workspace that holds every pass."""
    params = dict(W.differentiable_disk(n=1024, incl_deg=20.0))
    _announce("adjoint more rays than records")
    r, out = _forward(K, params)
    least = K.kt_adjoint_workspace_bytes(r.cam, r.integ)
    listed, stored, _, _ = _compare(K, r, out, params, out["n_steps"], K.adjoint_room(r.cam, r.integ) - least, 0)
    assert listed > 524288 >= stored > 400000
