"""Boxes of 8^3 and 16^3, whose MINRES iterations run whole in one launch:
fields and fluxes against the oracle, independence of the batch and of how the
iterations are cut into launches, zero and failing loads, refinement, the cell-wise
load and both face blocks."""
import numpy as np
import pytest

from oracle import spectral as S
from tests.gpu_common import gval, oracle_u, rel_l2, say

pytestmark = pytest.mark.gpu


def _setup():
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    return torch, P


# the solvers' default tolerances hold these bars at every size (fp64, mixed)
BARS = {"fp64": 1e-10, "mixed": 1e-7}


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n,batch", [(8, 1), (8, 300), (16, 1), (16, 37)])
def test_small_boxes_match_oracle(n, batch, precision, kind):
    torch, P = _setup()
    say(f"small box n={n} batch={batch} {precision} face block {kind}")
    kappa = 12.0
    xi = np.random.default_rng(n + batch).standard_normal((batch, n ** 3))
    xd = torch.tensor(xi, device="cuda")
    box = P.Box(n, kappa, precision=precision, max_batch=batch)
    box.set_face_preconditioner(kind)
    out = box.sample(xd, u_box=True, relres=True)
    u = out["u_box"].cpu().numpy()
    ref = oracle_u(n, kappa, gval(kappa), xi)
    assert max(rel_l2(u[b], ref[b]) for b in range(batch)) <= BARS[precision]
    # each sample alone gives the same bits, and so does a second call, which
    # knows how many iterations to expect
    one = P.Box(n, kappa, precision=precision, max_batch=1)
    one.set_face_preconditioner(kind)
    b = batch - 1
    assert torch.equal(one.sample(xd[b:b + 1].contiguous(), u_box=True)["u_box"][0], out["u_box"][b])
    again = box.sample(xd, u_box=True)
    assert torch.equal(again["u_box"], out["u_box"])
    assert np.array_equal(again["iters"], out["iters"])
    # timed calls and single-iteration launches too
    box.timing(1)
    assert torch.equal(box.sample(xd, u_box=True)["u_box"], out["u_box"])
    box.timing(0)
    assert box.timing_report()["iterations_small"]["launches"] > 0
    box.set_poll_interval(1)
    box.set_graphs(False)
    assert torch.equal(box.sample(xd, u_box=True)["u_box"], out["u_box"])


@pytest.mark.parametrize("n", [8, 16])
def test_small_boxes_zero_and_failing_samples(n):
    torch, P = _setup()
    say(f"small box n={n} zero and NaN loads")
    xi = np.random.default_rng(1).standard_normal((4, n ** 3))
    xi[1] = 0.0
    xi[2, 5] = np.nan
    box = P.Box(n, 10.0, precision="mixed", max_batch=4)
    out = box.sample(torch.tensor(xi, device="cuda"), u_box=True, allow_failed=True)
    u = out["u_box"].cpu().numpy()
    assert out["status"] == P.SPDE_EFAILED
    assert np.all(u[1] == 0.0) and np.all(np.isnan(u[2]))
    for b in (0, 3):
        alone = box.sample(torch.tensor(xi[b:b + 1], device="cuda"), u_box=True)["u_box"].cpu().numpy()[0]
        assert np.array_equal(alone, u[b])
        assert rel_l2(u[b], S.solve_u(n, 10.0, gval(10.0), xi[b])) <= 1e-7


@pytest.mark.parametrize("n", [8, 16])
def test_small_boxes_refined_and_cellwise(n):
    torch, P = _setup()
    say(f"small box n={n} refinement, cell-wise coefficients")
    kappa = 10.0
    rng = np.random.default_rng(9)
    xi = rng.standard_normal((3, n ** 3))
    xd = torch.tensor(xi, device="cuda")
    box = P.Box(n, kappa, precision="mixed", max_batch=3)
    box.set_refinement(1e-11)
    out = box.sample(xd, u_box=True, relres=True)
    assert out["relres"].max() <= 1e-11
    ref = oracle_u(n, kappa, gval(kappa), xi)
    u = out["u_box"].cpu().numpy()
    assert max(rel_l2(u[b], ref[b]) for b in range(3)) <= 1e-10
    # a cell-wise load keeps the constant operator; a kappa field takes the other kernels
    g = rng.uniform(0.5, 2.0, n ** 3)
    box = P.Box(n, kappa, g=1.0, precision="fp64", max_batch=3)
    box.set_coefficients(g=g)
    u = box.sample(xd, u_box=True)["u_box"].cpu().numpy()
    ref = oracle_u(n, kappa, 1.0, xi * g)
    assert max(rel_l2(u[b], ref[b]) for b in range(3)) <= 1e-10
    box.set_coefficients(kappa=np.full(n ** 3, kappa), g=g)
    u = box.sample(xd, u_box=True)["u_box"].cpu().numpy()
    assert max(rel_l2(u[b], ref[b]) for b in range(3)) <= 1e-10
