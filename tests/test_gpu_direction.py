"""Deferred direction and solution updates: the fields do not depend on how many
iterations a direction pass takes (every update is one fused chain per cell, so
the values are the same bit for bit), and captured slot steps replay any number
of times."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_common import gval, oracle_u, rel_l2, say

pytestmark = pytest.mark.gpu


def _setup():
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    return torch, P


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-10), ("mixed", 1e-7)])
@pytest.mark.parametrize("n,batch", [(4, 3), (16, 2), (64, 2)])
def test_fields_independent_of_pass_grouping(n, batch, precision, bar):
    torch, P = _setup()
    say(f"direction grouping n={n} batch={batch} {precision}")
    kappa = 10.0
    xi = np.random.default_rng(5).standard_normal((batch, n ** 3))
    xd = torch.tensor(xi, device="cuda")
    box = P.Box(n, kappa, precision=precision, max_batch=batch)
    base = box.sample(xd, u_box=True)
    u = base["u_box"].cpu().numpy()
    ref = oracle_u(n, kappa, gval(kappa), xi)
    assert max(rel_l2(u[b], ref[b]) for b in range(batch)) <= bar
    capped = P.Box(n, kappa, precision=precision, max_batch=batch, max_iter=7)
    for lvl, (d, s) in enumerate(base["tiles"]):
        capped.set_tiles(d, s, level=lvl)
    cap0 = capped.sample(xd, u_box=True, allow_notconv=True)["u_box"]
    for poll in (1, 3, 16, 40):     # passes of 16, 15, 16 and 16 iterations, and a remainder
        for bx, want in ((box, base["u_box"]), (capped, cap0)):
            bx.set_poll_interval(poll)
            got = bx.sample(xd, u_box=True, allow_notconv=True)["u_box"]
            assert torch.equal(got, want), poll


def test_captured_slot_steps_replay():
    torch, P = _setup()
    from paper_1712_06758_amd import _abi
    say("captured slot steps")
    n, slots = 16, 2
    L = _abi.lib()
    box = P.Box(n, 10.0, precision="mixed", max_batch=slots)
    box.set_graphs(False)
    st = torch.cuda.Stream()
    sp = C.c_void_p(st.cuda_stream)

    def start():
        _abi.check(L.spde_slots_reset(box._hh.h, slots, sp))
        for s in range(slots):
            _abi.check(L.spde_slot_start_seeded(box._hh.h, s, 7, s, 0, sp))

    def finish():
        u = torch.empty(slots, n ** 3, dtype=torch.float64, device="cuda")
        for s in range(slots):
            _abi.check(L.spde_slot_finish(box._hh.h, s, C.c_void_p(u[s].data_ptr()), sp))
        st.synchronize()
        return u

    start()
    _abi.check(L.spde_slots_step(box._hh.h, slots, 60, sp))
    want = finish()
    start()
    _abi.check(L.spde_slots_step(box._hh.h, slots, 3, sp))   # leaves updates waiting
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        _abi.check(L.spde_slots_step(box._hh.h, slots, 19, C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    for _ in range(3):
        with torch.cuda.stream(st):
            g.replay()
        st.synchronize()
    assert torch.equal(finish(), want)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", [0, 1])
def test_operator_blocks_of_every_depth_agree(precision, kind):
    """The operator pass takes blocks of 2, 4 or 16 planes by the size of the
    launch (64^3: 1, 4 and 13 samples); a sample's result is the same bit for bit."""
    torch, P = _setup()
    say(f"operator block depths {precision} face block {kind}")
    n = 64
    g = torch.Generator(device="cuda").manual_seed(3)
    xs = torch.randn(13, 3 * n * n * (n + 1), generator=g, device="cuda", dtype=torch.float64)
    xu = torch.randn(13, n ** 3, generator=g, device="cuda", dtype=torch.float64)
    box = P.Box(n, 10.0, precision=precision, max_batch=13)
    box.set_face_preconditioner(kind)
    ys, yu = box.apply_operator_precond(xs, xu)
    for b in (1, 4):
        s, u = box.apply_operator_precond(xs[:b].contiguous(), xu[:b].contiguous())
        assert torch.equal(s, ys[:b]) and torch.equal(u, yu[:b]), b


@pytest.mark.parametrize("n", [32, 64])
def test_samples_keep_their_bits_in_every_block_order(n):
    """Blocks are dealt out to the XCDs by slot, in turns of eight and a remainder:
    every sample of batches around those edges is what it is alone."""
    torch, P = _setup()
    say(f"block orders n={n}")
    xi = torch.randn(17, n ** 3, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda",
                     dtype=torch.float64)
    box = P.Box(n, 10.0, precision="mixed", max_batch=17)
    want = box.sample(xi, u_box=True)["u_box"]
    for b in (7, 8, 9, 16):
        assert torch.equal(box.sample(xi[:b].contiguous(), u_box=True)["u_box"], want[:b]), b
    assert torch.equal(box.sample(xi[16:].contiguous(), u_box=True)["u_box"][0], want[16])
