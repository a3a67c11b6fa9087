"""The slots of a handle beside its other calls: a finished slot's field is final
whatever runs before it is fetched, and a running one is not disturbed."""
import ctypes as C

import pytest

from tests.gpu_common import say

pytestmark = pytest.mark.gpu


def _setup():
    torch = pytest.importorskip("torch")
    import paper_1712_06758_amd as P
    from paper_1712_06758_amd import _abi
    return torch, P, _abi


class Slots:
    """A handle's slots on one stream, started from the events 0, 1, ... of one seed."""

    def __init__(self, n, precision, slots, busy=None):
        self.torch, P, self.abi = _setup()
        self.L, self.n, self.slots = self.abi.lib(), n, slots
        self.box = P.Box(n, 10.0, precision=precision, max_batch=slots)
        self.box.set_poll_interval(4)
        self.h = self.box._hh.h
        self.st = self.torch.cuda.Stream()
        self.sp = C.c_void_p(self.st.cuda_stream)
        self.start(range(slots if busy is None else busy))

    def start(self, which):
        self.check(self.L.spde_slots_reset(self.h, self.slots, self.sp))
        for s in which:
            self.check(self.L.spde_slot_start_seeded(self.h, s, 7, s, 0, self.sp))

    def check(self, status):
        self.abi.check(status)

    def step(self, iters):
        self.check(self.L.spde_slots_step(self.h, self.slots, iters, self.sp))

    def states(self):
        st, it = (C.c_int * self.slots)(), (C.c_int * self.slots)()
        self.check(self.L.spde_slots_poll(self.h, self.slots, st, it, self.sp))
        return list(st)

    def run(self, iters, want=1):
        """Steps until `want` slots have left the active state; those slots."""
        for _ in range(400):
            self.step(iters)
            done = [s for s, v in enumerate(self.states()) if v == 1]
            if len(done) >= want:
                return done
        raise AssertionError("no slot finished")

    def finish(self, slot, stream=None):
        u = self.torch.full((self.n ** 3,), float("nan"), dtype=self.torch.float64, device="cuda")
        self.torch.cuda.synchronize()
        self.check(self.L.spde_slot_finish(self.h, slot, C.c_void_p(u.data_ptr()),
                                           self.sp if stream is None else C.c_void_p(stream.cuda_stream)))
        return u


def _call(box, torch, name, batch):
    n = box.n
    g = torch.Generator(device="cuda").manual_seed(9)
    xs = torch.randn(batch, 3 * n * n * (n + 1), generator=g, device="cuda", dtype=torch.float64)
    xu = torch.randn(batch, n ** 3, generator=g, device="cuda", dtype=torch.float64)
    if name == "vcycle":
        box.apply_vcycle(xu)
    elif name == "operator":
        box.apply_operator(xs, xu)
    elif name == "operator_precond":
        box.apply_operator_precond(xs, xu)
    elif name == "sample":
        box.sample(xu[: batch - 1].contiguous(), u_box=True)
    torch.cuda.synchronize()


@pytest.mark.parametrize("call", ["operator", "operator_precond", "vcycle"])
@pytest.mark.parametrize("iters", [1, 3, 16])
@pytest.mark.parametrize("n,precision", [(16, "mixed"), (32, "mixed"), (32, "fp64")])
def test_finished_field_survives_other_calls(n, precision, iters, call):
    """Whatever uses the handle's buffers between the end of a slot and its fetch."""
    torch, P, _ = _setup()
    say(f"finished slot, then {call}: n={n} {precision} steps of {iters}")
    S = Slots(n, precision, 3)
    done = S.run(iters)
    want = [S.finish(s) for s in done]
    S.st.synchronize()
    S.start(range(3))
    assert S.run(iters) == done
    _call(S.box, torch, call, 3)
    got = [S.finish(s) for s in done]
    S.st.synchronize()
    for a, b in zip(got, want):
        assert torch.equal(a, b)


@pytest.mark.parametrize("n,precision", [(16, "mixed"), (32, "mixed"), (64, "fp64")])
def test_sample_leaves_the_other_slots(n, precision):
    """A sampling call takes the slots of its batch and leaves the slots above as they are."""
    torch, P, _ = _setup()
    say(f"sampling beside a running slot n={n} {precision}")
    S = Slots(n, precision, 3)
    S.run(5, want=3)
    want = S.finish(2)
    S.st.synchronize()
    S.start(range(3))
    S.step(12)
    S.st.synchronize()
    _call(S.box, torch, "sample", 3)
    S.run(5, want=3)
    got = S.finish(2)
    S.st.synchronize()
    assert torch.equal(got, want)


def test_fetch_under_capture_leaves_the_running_slots():
    """Capturing a fetch runs nothing: the updates that wait for a slot that goes on
    wait still, and the captured fetch gives the field when it is replayed."""
    torch, P, _ = _setup()
    say("fetch captured beside a running slot")
    S = Slots(32, "mixed", 2, busy=1)
    S.run(4)
    want = S.finish(0)
    S.st.synchronize()
    S.start([0])
    S.step(12)                               # updates of twelve iterations wait
    S.st.synchronize()
    u = torch.zeros(32 ** 3, dtype=torch.float64, device="cuda")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=S.st):
        S.check(S.L.spde_slot_finish(S.h, 1, C.c_void_p(u.data_ptr()), S.sp))
    S.step(12)
    S.run(4)
    assert torch.equal(S.finish(0), want)
    # the other way round: a captured fetch of a slot that goes on iterating
    S.start([0])
    S.step(4)
    S.st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=S.st):
        S.check(S.L.spde_slot_finish(S.h, 0, C.c_void_p(u.data_ptr()), S.sp))
    S.run(4)
    S.st.synchronize()
    with torch.cuda.stream(S.st):
        g.replay()
    S.st.synchronize()
    assert torch.equal(u, want)


@pytest.mark.parametrize("n,precision", [(16, "mixed"), (64, "mixed"), (64, "fp64")])
def test_fetch_on_a_second_stream(n, precision):
    """A finished slot is fetched on another stream while the others' steps run."""
    torch, P, _ = _setup()
    say(f"fetch on a second stream n={n} {precision}")
    slots = 6
    S = Slots(n, precision, slots)
    S.run(4, want=slots)
    want = [S.finish(s) for s in range(slots)]
    S.st.synchronize()
    second = torch.cuda.Stream()
    S.start([0])
    S.step(20)                               # slot 0 is ahead of the others
    for s in range(1, slots):
        S.check(S.L.spde_slot_start_seeded(S.h, s, 7, s, 0, S.sp))
    done = S.run(3)
    assert 0 in done and len(done) < slots
    out = {s: torch.empty(n ** 3, dtype=torch.float64, device="cuda") for s in done}
    torch.cuda.synchronize()
    for _ in range(4):
        S.step(3)
    for s in done:                           # while those steps run
        S.check(S.L.spde_slot_finish(S.h, s, C.c_void_p(out[s].data_ptr()), C.c_void_p(second.cuda_stream)))
    second.synchronize()
    S.run(3, want=slots - len(done))
    for s in range(slots):
        u = out[s] if s in out else S.finish(s)
        S.st.synchronize()
        assert torch.equal(u, want[s]), s


@pytest.mark.parametrize("n,precision", [(16, "mixed"), (32, "mixed"), (64, "mixed"), (32, "fp64")])
@pytest.mark.parametrize("iters", [3, 12, 16])
def test_vcycle_leaves_running_slots(n, precision, iters):
    """The V-cycle check between the steps of running slots, called and replayed."""
    torch, P, _ = _setup()
    say(f"V-cycle beside running slots n={n} {precision} after {iters}")
    S = Slots(n, precision, 2)
    S.run(4, want=2)
    want = [S.finish(s) for s in range(2)]
    r = torch.randn(2, n ** 3, generator=torch.Generator(device="cuda").manual_seed(9), device="cuda",
                    dtype=torch.float64)
    torch.cuda.synchronize()
    z0 = S.box.apply_vcycle(r)
    torch.cuda.synchronize()
    z = torch.empty_like(r)
    g = torch.cuda.CUDAGraph()               # captured while nothing waits
    with torch.cuda.graph(g, stream=S.st):
        S.check(S.L.spde_apply_vcycle(S.h, 2, C.c_void_p(r.data_ptr()), C.c_void_p(z.data_ptr()), S.sp))
    for how in ("called", "replayed"):
        S.start(range(2))
        S.step(iters)
        S.st.synchronize()
        if how == "called":
            z.copy_(S.box.apply_vcycle(r))
        else:
            z.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(S.st):
                g.replay()
        torch.cuda.synchronize()
        assert torch.equal(z, z0)
        S.run(4, want=2)
        got = [S.finish(s) for s in range(2)]
        S.st.synchronize()
        for a, b in zip(got, want):
            assert torch.equal(a, b), how


@pytest.mark.parametrize("n,precision", [(32, "mixed"), (64, "mixed"), (64, "fp64")])
def test_filling_and_emptying_keeps_the_bits(n, precision):
    """The operator's block order changes with the share of busy slots (7/8 of them,
    from 64^3 up): slots that live through both orders give what they give alone."""
    torch, P, _ = _setup()
    say(f"engine filled and emptied n={n} {precision}")
    slots = 17
    S = Slots(n, precision, slots, busy=0)
    xi = P.noise(n, 7, batch=slots)
    torch.cuda.synchronize()                 # the slots use the handle's buffers on another stream
    want = S.box.sample(xi, u_box=True)["u_box"]
    torch.cuda.synchronize()
    S.start([])
    for s in range(slots):                   # filled one by one, emptied as they finish
        S.check(S.L.spde_slot_start_seeded(S.h, s, 7, s, 0, S.sp))
        S.step(4 if s == 15 else 1)
    left = set(range(slots))
    while left:
        for s in [t for t in S.run(3, want=1) if t in left]:
            got = S.finish(s)
            S.st.synchronize()
            assert torch.equal(got, want[s]), s
            left.remove(s)


@pytest.mark.parametrize("face", [0, 1])
@pytest.mark.parametrize("n,precision", [(16, "mixed"), (32, "fp64"), (64, "mixed"), (64, "fp64")])
def test_cellwise_slots(n, precision, face):
    """Slots of a box with a kappa field, in every operator form: finished in the step
    that finds them so, with the fields of a sampling call."""
    torch, P, _ = _setup()
    say(f"cell-wise slots n={n} {precision} face block {face}")
    S = Slots(n, precision, 2, busy=0)
    S.box.set_face_preconditioner(face)
    g = torch.Generator(device="cuda").manual_seed(n)
    S.box.set_coefficients(kappa=10.0 * torch.exp(0.3 * torch.randn(n ** 3, generator=g, device="cuda",
                                                                    dtype=torch.float64)))
    xi = P.noise(n, 7, batch=2)
    torch.cuda.synchronize()
    want = S.box.sample(xi, u_box=True)["u_box"]
    torch.cuda.synchronize()
    for iters in (1, 4):
        S.start(range(2))
        S.run(iters, want=2)
        _call(S.box, torch, "operator", 2)
        for s in range(2):
            got = S.finish(s)
            S.st.synchronize()
            assert torch.equal(got, want[s]), (iters, s)
