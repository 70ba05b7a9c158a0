"""Default plans: chosen from the mesh size per form of the subcycle at its first call.

The plan does not change results (the same IEEE operations in the same order for every
plan), so each form on its default plan must equal the same form on a plan set by the
caller bit for bit, volumes (summed per tile) to rounding; a call that may not allocate
finds a plan once any form has made its default.
"""
import numpy as np
import pytest

import sesynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FORMS = [("f64", "se", False), ("f32", "se", False), ("f64", "sesm", False),
         ("f32", "sesm", False), ("f64", "se", True), ("f32", "se", True)]


def _mesh(name):
    if name == "two":
        return sesynth.tiny_mesh("two")
    if name == "fan":
        return sesynth.tiny_mesh("fan100")
    nx, ny = {"2k": (61, 37), "16k": (128, 129), "33k": (193, 171), "70k": (301, 233)}[name]
    return sesynth.planar_grid(nx, ny, 1500.0, 1400.0, jitter=0.3, r=sesynth.rng(5))


def _params(case, prec, scheme, visc):
    from paper_2311_08241_amd import Params
    return Params(g=case["g"], theta=case["theta"], precision=prec, scheme=scheme,
                  visc=(5.0, 0.1) if visc else None)


def _run(mesh, case, p, call="subcycle"):
    from paper_2311_08241_amd import device_inputs
    d = device_inputs(mesh, case, p)
    Uavg = torch.empty((mesh.ne, 2), dtype=torch.float64, device="cuda:0")
    vol = torch.empty(case["nsub"] + 1, dtype=torch.float64, device="cuda:0")
    getattr(mesh, call)(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=case["nsub"],
                        dt=case["tau"], params=p, Uavg=Uavg, volume=vol)
    torch.cuda.synchronize()
    assert mesh.check_faults() == 0
    return d["eta"].cpu().numpy(), d["U"].cpu().numpy(), Uavg.cpu().numpy(), vol.cpu().numpy()


@pytest.mark.parametrize("name", ["two", "fan", "2k", "16k", "33k", "70k"])
def test_default_plans_equal_a_set_plan(name):
    from paper_2311_08241_amd import Mesh
    # (the fan's 60 m triangles need substeps of a few hundredths of a second)
    case = sesynth.random_case(_mesh(name), seed=3, nsub=11, tau=0.2 if name == "fan" else 24.0)
    ref, dflt = Mesh.from_dict(case, device=0), Mesh.from_dict(case, device=0)
    ref.set_plan(64, 2, 256)
    area = dflt.geometry()[0]
    for prec, scheme, visc in FORMS:
        p = _params(case, prec, scheme, visc)
        a, b = _run(ref, case, p), _run(dflt, case, p)
        for x, y in zip(a[:3], b[:3]):
            assert np.array_equal(x, y), (name, prec, scheme, visc)
        # volumes: the same terms in another order, at most nv roundings of the largest sum
        tol = area.size * np.finfo(float).eps * float((area * np.abs(case["eta0"])).sum() + 1.0)
        assert np.abs(a[3] - b[3]).max() <= tol


@pytest.mark.parametrize("first", [0, 1])
def test_calls_that_may_not_allocate_find_a_default(first):
    """One call of one form makes a plan that every form can run on: without allocation, and
    under stream capture (replayed, against the eager result)."""
    from paper_2311_08241_amd import Mesh, device_inputs
    case = sesynth.random_case(_mesh("33k"), seed=4, nsub=9)
    ref, m = Mesh.from_dict(case, device=0), Mesh.from_dict(case, device=0)
    _run(m, case, _params(case, *FORMS[first]))
    for prec, scheme, visc in FORMS[:4]:
        p = _params(case, prec, scheme, visc)
        a = _run(ref, case, p)
        for x, y in zip(a[:3], _run(m, case, p, "subcycle_noalloc")[:3]):
            assert np.array_equal(x, y), (prec, scheme)
        d = device_inputs(m, case, p)
        e0, u0 = d["eta"].clone(), d["U"].clone()
        ws = m.workspace(p, case["nsub"])
        fresh = Mesh.from_dict(case, device=0)
        _run(fresh, case, _params(case, *FORMS[1 - first]))
        Uavg = torch.empty((m.ne, 2), dtype=torch.float64, device="cuda:0")
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fresh.subcycle(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=case["nsub"],
                           dt=case["tau"], params=p, Uavg=Uavg, workspace=ws)
        for _ in range(3):
            d["eta"].copy_(e0)
            d["U"].copy_(u0)
            graph.replay()
            torch.cuda.synchronize()
            for x, y in zip(a[:3], (d["eta"], d["U"], Uavg)):
                assert np.array_equal(x, y.cpu().numpy()), (prec, scheme)
