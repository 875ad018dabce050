"""lbm_step_noalloc takes nothing from what is in its static array: a sequence
of calls over storage forms, collisions, budgets and lattice sizes (one and
several sweep workgroups, the FP64-solve list, D1Q3), in an order in which each
call finds another configuration's contents, then with the whole array
overwritten before each call, and as captured calls replayed over such an
array.  Each against lbm_step from a fresh context, bit for bit."""
import ctypes

import pytest
import torch

from paper_1110_0270_amd import lbm as B
from tests.parity_util import make_sim, random_state

pytestmark = pytest.mark.gpu

E = dict(ehrenfest=True, ehr_delta=0.0)
CALLS = [
    ("f64", dict(lattice="D2Q9", nx=70, ny=37, bc="periodic", ehr_k=9, positivity=True, **E)),
    ("f32", dict(lattice="D2Q9", nx=300, ny=90, bc="cavity", u_lid=0.1, ehr_k=60, positivity=True, **E)),
    ("f32", dict(lattice="D2Q9", nx=300, ny=13, bc="periodic", collision="elbm")),
    ("f16s", dict(lattice="D2Q9", nx=512, ny=300, bc="periodic", ehr_k=150, **E)),
    ("f32", dict(lattice="D2Q9", nx=70, ny=37, bc="cavity", u_lid=0.1, collision="elbm", ehr_k=30, **E)),
    ("f64", dict(lattice="D1Q3", nx=800, ny=1, bc="bounceback", ehr_k=4, **E)),
    ("f64", dict(lattice="D2Q9", nx=301, ny=300, bc="couette", u_lid=0.1, ehr_k=90, **E)),
    ("f32", dict(lattice="D2Q9", nx=70, ny=37, bc="periodic", ehr_k=0, **E)),
    ("bf16s", dict(lattice="D2Q9", nx=130, ny=66, bc="periodic", collision="mrt", ehr_k=10**6, **E)),
    ("f64", dict(lattice="D2Q9", nx=1, ny=1, bc="periodic", ehr_k=1, **E)),
    ("f32", dict(lattice="D2Q9", nx=260, ny=70, bc="periodic", median=True, med_delta=1e-4, ehr_k=20,
                 **E)),
    ("f32", dict(lattice="D2Q9", nx=90, ny=50, bc="periodic", ehr_k=40, sel_action="mrt", **E)),
    ("f16s", dict(lattice="D1Q3", nx=70000, ny=1, bc="periodic", ehr_k=70, **E)),
    # every site eligible at one Delta S: the budget falls inside one tie
    ("f64", dict(lattice="D2Q9", nx=200, ny=150, bc="periodic", ehr_k=300, ties=True, **E)),
]


class _Call:
    def __init__(self, i):
        storage, p = CALLS[i]
        p = dict(p)
        ties = p.pop("ties", False)
        kind = "entropic" if p.get("collision") == "elbm" else "poly"
        if kind == "entropic":
            p["equilibrium"] = "entropic"
        p["nu"] = 1e-3
        f0 = random_state(p, 40 + i, amp=0.3, kind=kind).cuda()
        if ties:
            f0 = f0[:, :1, :1].expand_as(f0).contiguous()
        Q, ny, nx = f0.shape
        self.cfg = B.make_config(**{**p, "storage": storage})
        self.dtype = {"f64": torch.float64, "f32": torch.float32, "f16s": torch.float16,
                      "bf16s": torch.bfloat16}[storage]
        w1 = torch.tensor((1 / 6, 2 / 3, 1 / 6), dtype=torch.float64, device="cuda")
        w = w1 if Q == 3 else (w1.view(3, 1) * w1.view(1, 3)).reshape(9)
        self.shift = w.view(Q, 1, 1) * (0.0 if storage == "f64" else 1.0)
        sim = make_sim(p, storage)
        sim.set_populations(f0)
        # both from the state as the library has stored it
        self.src = (sim.populations() - self.shift).to(self.dtype)
        sim.step(1)
        self.want = sim.populations()
        self.dst = torch.empty_like(self.src)

    def run(self):
        self.dst.fill_(float("nan"))
        B.lbm_step_noalloc(self.cfg, self.src, self.dst)

    def check(self, what):
        got = self.dst.to(torch.float64) + self.shift
        assert torch.equal(got, self.want), (what, float((got - self.want).abs().max()))


def _fill_scratch(word):
    """Every 32-bit word of the array set to `word`."""
    with open("/proc/self/maps") as f:      # the runtime that this process has loaded
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    ptr = ctypes.c_void_p()
    assert B.library()._ZN3lbm15scratch_addressEiPPv(torch.cuda.current_device(), ctypes.byref(ptr)) == 0
    torch.cuda.synchronize()
    assert hip.hipMemsetD32(ptr, ctypes.c_int(word), ctypes.c_size_t(B.NOALLOC_SCRATCH_BYTES // 4)) == 0
    torch.cuda.synchronize()


@pytest.fixture(scope="module")
def calls():
    return [_Call(i) for i in range(len(CALLS))]


def test_sequence_of_configurations(calls):
    for i in list(range(len(calls))) + list(range(len(calls) - 1, -1, -1)):
        calls[i].run()
        calls[i].check(i)


def test_array_overwritten_before_each_call(calls):
    for i, c in enumerate(calls):
        _fill_scratch(1)
        c.run()
        c.check(i)


def test_captured_calls_over_an_overwritten_array(calls):
    graphs = []
    for c in calls:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            B.lbm_step_noalloc(c.cfg, c.src, c.dst)
        graphs.append(g)
    for rep in range(2):
        for i, (c, g) in enumerate(zip(calls, graphs)):
            if rep == 0:
                _fill_scratch(1)
            c.dst.fill_(float("nan"))
            g.replay()
            c.check((rep, i))
            calls[(i + 5) % len(calls)].run()       # eager work of another configuration
