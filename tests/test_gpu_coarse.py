"""The V-cycle, levels from the finest down to the exact solve on 4^3, against the
same cycle in numpy (boxes above 16^3: the persistent kernel's top is 16^3)."""
import numpy as np
import pytest

from tests.gpu_common import rel_l2, say

pytestmark = pytest.mark.gpu


def nbrs(x):
    """Sum over the 7-point stencil's neighbours inside the box."""
    p = np.pad(x, [(0, 0)] + [(1, 1)] * 3)
    i = slice(1, -1)
    return (p[:, :-2, i, i] + p[:, 2:, i, i] + p[:, i, :-2, i] + p[:, i, 2:, i] + p[:, i, i, :-2] +
            p[:, i, i, 2:])


def vcycle(kappa, b):
    """Two Chebyshev steps on [lmax/4, lmax] from zero before and after, sums over
    2x2x2 children down, injection up, exact on 4^3; b: [batch, m, m, m]."""
    m = b.shape[1]
    H = 1.0 / m
    k2, a = kappa ** 2 * H ** 3, 1.5 * H
    d = k2 + a * nbrs(np.ones((1, m, m, m)))
    A = lambda x: d * x - a * nbrs(x)
    if m == 4:
        M = A(np.eye(64).reshape(64, 4, 4, 4)).reshape(64, 64)
        return np.linalg.solve(M, b.reshape(-1, 64).T).T.reshape(b.shape)
    lmax = min(2.0, (k2 + 12 * a) / (k2 + 6 * a))
    th, dl = 0.625 * lmax, 0.375 * lmax
    r0 = dl / th
    r1 = 1.0 / (2.0 / r0 - r0)

    def smooth(r):
        y = r / d / th
        return y + r1 * r0 * y + 2 * r1 / dl * (r - A(y)) / d

    x = smooth(b)
    r = b - A(x)
    e = vcycle(kappa, r.reshape(-1, m // 2, 2, m // 2, 2, m // 2, 2).sum((2, 4, 6)))
    x = x + e.repeat(2, 1).repeat(2, 2).repeat(2, 3)
    return x + smooth(b - A(x))


# a chain of some fifty roundings from b to z: 50 eps of each level precision
@pytest.mark.parametrize("precision,bar", [("fp64", 50 * 2.0 ** -53), ("mixed", 50 * 2.0 ** -24)])
@pytest.mark.parametrize("n,batch", [(8, 2), (16, 3), (32, 1), (32, 5), (64, 2)])
def test_vcycle_matches_numpy(n, batch, precision, bar):
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    say(f"V-cycle n={n} batch={batch} {precision}")
    kappa = 10.0
    r = np.random.default_rng(n + batch).standard_normal((batch, n ** 3))
    box = P.Box(n, kappa, precision=precision, max_batch=batch)
    z = box.apply_vcycle(torch.tensor(r, device="cuda")).cpu().numpy()
    ref = vcycle(kappa, r.reshape(batch, n, n, n)).reshape(batch, -1)
    assert max(rel_l2(z[b], ref[b]) for b in range(batch)) <= bar


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("precision,shapes", [("fp64", (1, 4, 5)), ("mixed", (0, 1, 2, 3, 4, 5))])
def test_samples_with_3d_tiles(precision, shapes, kind):
    """The partial sums of the finest up kernel: every 3-D tile shape reaches the
    oracle, with constant kappa and with a cell-wise one (constant multigrid)."""
    from tests.gpu_common import gval, oracle_u
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    n, kappa, batch = 32, 12.0, 3
    bar = {"fp64": 1e-10, "mixed": 1e-7}[precision]
    rng = np.random.default_rng(31 + kind)
    xi = rng.standard_normal((batch, n ** 3))
    xd = torch.tensor(xi, device="cuda")
    ref = oracle_u(n, kappa, gval(kappa), xi)
    kc = kappa * (1.0 + 0.2 * rng.random(n ** 3))
    box = P.Box(n, kappa, precision=precision, max_batch=batch)
    box.set_face_preconditioner(kind)
    var = P.Box(n, kappa, precision=precision, max_batch=batch)
    var.set_face_preconditioner(kind)
    var.set_coefficients(kc, None, kappa_ref=kappa)
    var.set_tiles(10, 10)
    want = var.sample(xd, u_box=True)["u_box"].cpu().numpy()
    for shape in shapes:
        say(f"3-D tile {shape} {precision} face block {kind}")
        box.set_tiles(shape, shape)
        u = box.sample(xd, u_box=True)["u_box"].cpu().numpy()
        assert max(rel_l2(u[b], ref[b]) for b in range(batch)) <= bar
        var.set_tiles(shape, shape)
        u = var.sample(xd, u_box=True)["u_box"].cpu().numpy()
        assert max(rel_l2(u[b], want[b]) for b in range(batch)) <= 2 * bar
