"""The ring of waiting updates at every depth (16, 8, 4 and 2 iterations, chosen by
the workspace that is bound): the same fields bit for bit, through every way that
iterations are enqueued."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_common import gval, oracle_u, rel_l2, say

pytestmark = pytest.mark.gpu


def _setup():
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    from paper_1712_06758_amd import _abi
    return torch, P, _abi


def _bind(box, abi, ring):
    """The box's own workspace, of which the handle is told what a ring of `ring` takes."""
    L, h = abi.lib(), box._hh.h
    most, least = L.spde_workspace_bytes(h), L.spde_workspace_bytes_min(h)
    assert least < most <= box._ws.numel()
    # 14 entries lie between; the pieces of the workspace are padded to 256 bytes
    nbytes = most if ring == 16 else least + (ring - 2) * (most - least) // 14 + 512 * (ring > 2)
    abi.check(L.spde_bind_workspace(h, C.c_void_p(box._ws.data_ptr()), nbytes))


def _passes(box, call):
    """Direction passes of a call."""
    box.timing(-1)
    box.timing(1)
    try:
        out = call()
        return out, box.timing_report()["direction"]["launches"]
    finally:
        box.timing(0)


def test_smaller_workspaces_are_refused():
    torch, P, abi = _setup()
    say("workspace below the least")
    L = abi.lib()
    box = P.Box(16, 10.0, max_batch=2)
    h, p = box._hh.h, C.c_void_p(box._ws.data_ptr())
    least = L.spde_workspace_bytes_min(h)
    assert L.spde_bind_workspace(h, p, least - 1) == abi.SPDE_ENOMEM
    assert L.spde_bind_workspace(h, p, least) == abi.SPDE_OK
    assert L.spde_workspace_bytes_min(h) == least and L.spde_workspace_bytes(h) == box._ws.numel()


@pytest.mark.parametrize("precision,bar", [("fp64", 1e-10), ("mixed", 1e-7)])
@pytest.mark.parametrize("n,batch", [(4, 2), (16, 3), (32, 9), (64, 2)])
def test_samples_keep_their_bits(n, batch, precision, bar):
    torch, P, abi = _setup()
    say(f"ring depths n={n} batch={batch} {precision}")
    kappa = 10.0
    xi = np.random.default_rng(6).standard_normal((batch, n ** 3))
    xd = torch.tensor(xi, device="cuda")
    box = P.Box(n, kappa, precision=precision, max_batch=batch)
    base = box.sample(xd, u_box=True)
    for lvl, (d, s) in enumerate(base["tiles"]):
        box.set_tiles(d, s, level=lvl)
    ref = oracle_u(n, kappa, gval(kappa), xi)
    u = base["u_box"].cpu().numpy()
    assert max(rel_l2(u[b], ref[b]) for b in range(batch)) <= bar
    tiles = base["tiles"]
    for ring in (2, 4, 8, 16):
        _bind(box, abi, ring)
        for lvl, (d, s) in enumerate(tiles):        # a bind plans the levels anew
            box.set_tiles(d, s, level=lvl)
        out, passes = _passes(box, lambda: box.sample(xd, u_box=True))
        assert torch.equal(out["u_box"], base["u_box"]), ring
        its = int(out["iters"].max())
        assert passes >= -(-its // ring) and (ring == 16 or passes > -(-its // (2 * ring)))
        for poll in (1, 3, 8, 40):
            box.set_poll_interval(poll)
            for split in (1, 2):
                box.set_split(split)
                assert torch.equal(box.sample(xd, u_box=True)["u_box"], base["u_box"]), (ring, poll, split)
        box.set_poll_interval(8)
        box.set_split(1)


@pytest.mark.parametrize("ring", [2, 4, 8])
@pytest.mark.parametrize("n,precision", [(16, "mixed"), (32, "mixed"), (32, "fp64")])
def test_refined_and_warm_calls_keep_their_bits(n, precision, ring):
    torch, P, abi = _setup()
    say(f"ring of {ring}: refinement and warm start n={n} {precision}")
    g = torch.Generator(device="cuda").manual_seed(n)
    xi = torch.randn(2, n ** 3, generator=g, device="cuda", dtype=torch.float64)
    uc = torch.randn(2, (n // 2) ** 3, generator=g, device="cuda", dtype=torch.float64)
    kap = 10.0 * torch.exp(0.3 * torch.randn(n ** 3, generator=g, device="cuda", dtype=torch.float64))

    def calls(box):
        out = [box.sample_warm(xi, uc, u_box=True)["u_box"]]
        box.set_refinement(1e-12)
        out.append(box.sample(xi, u_box=True)["u_box"])
        box.set_refinement(0.0)
        box.set_coefficients(kappa=kap)
        out.append(box.sample(xi, u_box=True)["u_box"])
        box.set_coefficients()
        return out

    box = P.Box(n, 10.0, precision=precision, max_batch=2)
    want = calls(box)
    tiles = box.info()["tiles"]
    _bind(box, abi, ring)
    for lvl, (d, s) in enumerate(tiles):
        box.set_tiles(d, s, level=lvl)
    for a, b in zip(calls(box), want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("ring", [2, 4, 8, 16])
@pytest.mark.parametrize("n,precision", [(16, "fp64"), (32, "mixed")])
def test_slots_keep_their_bits(n, precision, ring):
    """Steps of every length over a short ring, eager and captured."""
    torch, P, abi = _setup()
    say(f"ring of {ring}: slots n={n} {precision}")
    L, slots = abi.lib(), 3
    xi = P.noise(n, 7, batch=slots)
    box = P.Box(n, 10.0, precision=precision, max_batch=slots)
    base = box.sample(xi, u_box=True)
    torch.cuda.synchronize()
    _bind(box, abi, ring)
    for lvl, (d, s) in enumerate(base["tiles"]):
        box.set_tiles(d, s, level=lvl)
    h, st = box._hh.h, torch.cuda.Stream()
    sp = C.c_void_p(st.cuda_stream)

    def start():
        abi.check(L.spde_slots_reset(h, slots, sp))
        for s in range(slots):
            abi.check(L.spde_slot_start_seeded(h, s, 7, s, 0, sp))

    def finish():
        u = torch.empty(slots, n ** 3, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        for s in range(slots):
            abi.check(L.spde_slot_finish(h, s, C.c_void_p(u[s].data_ptr()), sp))
        st.synchronize()
        return u

    for poll in (1, 4, 40):
        box.set_poll_interval(poll)
        for iters in (1, 3, 7, 60):
            start()
            for _ in range(-(-60 // iters)):
                abi.check(L.spde_slots_step(h, slots, iters, sp))
            assert torch.equal(finish(), base["u_box"]), (poll, iters)
    box.set_poll_interval(8)
    start()
    abi.check(L.spde_slots_step(h, slots, 1, sp))
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        abi.check(L.spde_slots_step(h, slots, 11, sp))
    for _ in range(2):
        for _ in range(3):
            with torch.cuda.stream(st):
                g.replay()
            abi.check(L.spde_slots_step(h, slots, 3, sp))
        with torch.cuda.stream(st):
            g.replay()
            g.replay()
        assert torch.equal(finish(), base["u_box"])
        start()


def test_a_box_fits_where_only_the_least_is_free():
    """Device memory for the least workspace, but not for the one it runs fastest with."""
    torch, P, abi = _setup()
    say("box in little memory")
    n, batch = 64, 32
    xi = torch.randn(batch, n ** 3, device="cuda", dtype=torch.float64)
    box = P.Box(n, 10.0, max_batch=batch)
    base = box.sample(xi, u_box=True)
    most = box._ws.numel()
    L = abi.lib()
    least = L.spde_workspace_bytes_min(box._hh.h)
    box._ws = box = None
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (most + least) // 2) / total)
        small = P.Box(n, 10.0, max_batch=batch)
        assert small.info()["workspace_bytes"] == least
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    for lvl, (d, s) in enumerate(base["tiles"]):
        small.set_tiles(d, s, level=lvl)
    assert torch.equal(small.sample(xi, u_box=True)["u_box"], base["u_box"])
