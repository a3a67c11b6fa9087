"""A handle that is configured again: what a call reports is read from its own
solve, whatever the handle's earlier calls needed."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_common import say

pytestmark = pytest.mark.gpu


def _setup():
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    return torch, P


def _configure(P, box, prec, rtol, max_iter, max_batch):
    """Another configuration on a live handle, bound to the box's own workspace."""
    from paper_1712_06758_amd import _abi
    L = _abi.lib()
    _abi.check(L.spde_configure(box._hh.h, prec, rtol, max_iter, max_batch))
    assert L.spde_workspace_bytes(box._hh.h) <= box._ws.numel()
    _abi.check(L.spde_bind_workspace(box._hh.h, C.c_void_p(box._ws.data_ptr()), box._ws.numel()))


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [16, 32])
@pytest.mark.parametrize("max_iter", [1, 7, 20])
def test_a_smaller_cap_is_reported(n, precision, max_iter):
    torch, P = _setup()
    say(f"reconfigured handle n={n} {precision} max_iter={max_iter}")
    prec = P.SPDE_FP64 if precision == "fp64" else P.SPDE_MIXED
    xi = torch.randn(3, n ** 3, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda",
                     dtype=torch.float64)
    box = P.Box(n, 10.0, precision=precision, max_batch=3)
    first = box.sample(xi[:2].contiguous(), u_box=True)
    assert first["status"] == P.SPDE_OK and first["iters"].min() > 24
    _configure(P, box, prec, box.rtol, max_iter, 3)
    fresh = P.Box(n, 10.0, precision=precision, max_batch=3, max_iter=max_iter)
    want = fresh.sample(xi, u_box=True, allow_notconv=True)
    for _ in range(2):              # the second call meets what the first one left in the handle
        got = box.sample(xi, u_box=True, allow_notconv=True)
        assert got["status"] == P.SPDE_ENOTCONV
        assert np.array_equal(got["iters"], np.full(3, max_iter))
        assert torch.equal(got["u_box"], want["u_box"])
    # and back: the whole solve again
    _configure(P, box, prec, box.rtol, 1000, 3)
    again = box.sample(xi[:2].contiguous(), u_box=True)
    assert again["status"] == P.SPDE_OK and np.array_equal(again["iters"], first["iters"])
    assert torch.equal(again["u_box"], first["u_box"])


def test_a_breakdown_is_reported_after_reconfiguring():
    torch, P = _setup()
    n = 32
    say("reconfigured handle, a sample that breaks down")
    xi = torch.randn(2, n ** 3, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda",
                     dtype=torch.float64)
    box = P.Box(n, 10.0, precision="mixed", max_batch=2)
    box.sample(xi, u_box=True)
    _configure(P, box, P.SPDE_MIXED, box.rtol, 7, 2)
    xi[1, 5] = float("nan")
    out = box.sample(xi, u_box=True, allow_notconv=True, allow_failed=True)
    assert out["status"] == P.SPDE_EFAILED
    assert torch.isnan(out["u_box"][1]).all() and not torch.isnan(out["u_box"][0]).any()


def _launched(box, call):
    """The call's result and the iterations that it enqueued (operator launches)."""
    box.timing(-1)
    box.timing(1)
    try:
        out = call()
        return out, box.timing_report()["operator"]["launches"]
    finally:
        box.timing(0)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("change", ["coefficients", "face", "warm"])
def test_no_iterations_beyond_a_poll(precision, change):
    """A call that needs fewer iterations than the one before, because the coefficients,
    the face block or the kind of start changed, stops at the next poll."""
    torch, P = _setup()
    n, poll = 32, 8
    say(f"idle iterations after a change of {change}, {precision}")
    g = torch.Generator(device="cuda").manual_seed(4)
    xi = torch.randn(2, n ** 3, generator=g, device="cuda", dtype=torch.float64)
    box = P.Box(n, 10.0, precision=precision, max_batch=2)
    box.set_poll_interval(poll)
    if change == "coefficients":
        rough = 10.0 * torch.exp(0.6 * torch.randn(n ** 3, generator=g, device="cuda", dtype=torch.float64))
        box.set_coefficients(kappa=rough, kappa_ref=10.0)
        before = box.sample(xi, u_box=True)["iters"]
        box.set_coefficients()
        out, count = _launched(box, lambda: box.sample(xi, u_box=True))
    elif change == "face":
        box.set_face_preconditioner(0)
        before = box.sample(xi, u_box=True)["iters"]
        box.set_face_preconditioner(1)
        out, count = _launched(box, lambda: box.sample(xi, u_box=True))
    else:
        # a load that the coarse grid holds exactly: the warm start has next to nothing left to do
        before = box.sample(xi, u_box=True)["iters"]
        flat = torch.ones(2, n ** 3, device="cuda", dtype=torch.float64)
        u = box.sample(flat, u_box=True)["u_box"]
        box.sample(xi, u_box=True)
        uc = u[:, : (n // 2) ** 3].contiguous()
        out, count = _launched(box, lambda: box.sample_warm(flat, uc, u_box=True))
    say(f"  iterations {before} before, {out['iters']} now, {count} enqueued")
    most = -(-(int(out["iters"].max()) + 1) // poll) * poll
    assert before.max() >= most
    assert count <= most
