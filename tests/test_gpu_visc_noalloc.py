"""The viscous form without allocation: one eager call with the term, in either precision, leaves
a plan with its tables that a call of the other precision finds, without allocation and under
stream capture; both equal an eager call of that precision bit for bit."""
import numpy as np
import pytest

import sesynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _case(name):
    m = (sesynth.tiny_mesh("fan100") if name == "fan" else
         sesynth.planar_grid(*{"2k": (61, 37), "33k": (193, 171), "70k": (301, 233)}[name], 1500.0,
                             1400.0, jitter=0.3, r=sesynth.rng(5)))
    return sesynth.random_case(m, seed=6, nsub=9, tau=0.2 if name == "fan" else 20.0)


def _params(case, prec):
    from paper_2311_08241_amd import Params
    return Params(g=case["g"], theta=case["theta"], precision=prec, visc=(5.0, 0.1))


class _Step:
    def __init__(self, mesh, case, prec):
        from paper_2311_08241_amd import device_inputs
        self.mesh, self.p = mesh, _params(case, prec)
        self.d = device_inputs(mesh, case, self.p)
        self.Uavg = torch.empty((mesh.ne, 2), dtype=torch.float64, device="cuda:0")
        self.kw = dict(R=self.d["R"], f=self.d["f"], H0=self.d["H0"], nsub=case["nsub"],
                       dt=case["tau"], params=self.p, Uavg=self.Uavg)

    def out(self):
        torch.cuda.synchronize()
        assert self.mesh.check_faults() == 0
        return [t.cpu().numpy() for t in (self.d["eta"], self.d["U"], self.Uavg)]


def _eager(mesh, case, prec):
    s = _Step(mesh, case, prec)
    s.mesh.subcycle(s.d["eta"], s.d["U"], **s.kw)
    return s.out()


@pytest.mark.parametrize("call", ["noalloc", "capture"])
@pytest.mark.parametrize("name", ["fan", "2k", "33k", "70k"])
@pytest.mark.parametrize("first,second", [("f32", "f64"), ("f64", "f32")])
def test_viscous_call_of_the_other_precision_finds_tables(first, second, name, call):
    from paper_2311_08241_amd import Mesh
    case = _case(name)
    ref = _eager(Mesh.from_dict(case, device=0), case, second)
    m = Mesh.from_dict(case, device=0)
    _eager(m, case, first)
    s = _Step(m, case, second)
    if call == "noalloc":
        m.subcycle_noalloc(s.d["eta"], s.d["U"], **s.kw)
        for x, y in zip(ref, s.out()):
            assert np.array_equal(x, y)
        return
    e0, u0 = s.d["eta"].clone(), s.d["U"].clone()
    ws = m.workspace(s.p, case["nsub"])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.subcycle(s.d["eta"], s.d["U"], workspace=ws, **s.kw)
    for _ in range(3):
        s.d["eta"].copy_(e0)
        s.d["U"].copy_(u0)
        graph.replay()
        for x, y in zip(ref, s.out()):
            assert np.array_equal(x, y)
