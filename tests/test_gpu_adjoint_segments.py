"""The adjoint on a tile plan keeps the forward elevations of the whole step where they fit
the workspace of the call's ckpt_every, and recomputes segments where they do not.  Both equal
the per-substep path (no plan on the mesh), whose segments always have ckpt_every substeps, bit
for bit."""
import pytest

import sesynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 1, 2: one launch, a remainder of one; 30, 37: whole step kept, any interval; 400: the
# elevations of 400 substeps exceed the workspace of ckpt_every 14 (28 substeps at a time) but
# not that of 1 (a checkpoint per substep)
@pytest.mark.parametrize("nsub,ckpt", [(2, 1), (30, 1), (30, 7), (37, 36), (400, 14), (400, 1)])
@pytest.mark.parametrize("precision,plan", [("f64", (128, 5, 256)), ("f32", (96, 8, 512))])
def test_whole_trajectory_and_segments_equal_the_per_substep_path(precision, plan, nsub, ckpt):
    from paper_2311_08241_amd import Mesh, Params, device_inputs
    case = sesynth.adjoint_c5(n=64)
    out = []
    for tiles in (False, True):
        mesh = Mesh.from_dict(case, device=0)
        if tiles:
            assert mesh.plan_stats(*plan)["ok_" + precision]
            mesh.set_plan(*plan)
        p = Params(precision=precision, eta_ref=case["eta_ref"] if precision == "f32" else 0.0)
        d = device_inputs(mesh, case, p)
        gen = torch.Generator(device="cpu").manual_seed(5)
        rnd = lambda *s, dt=p.dtype: torch.randn(*s, generator=gen, dtype=torch.float64).to(dt).cuda()
        lam = rnd(mesh.nv), rnd(mesh.ne, 2), rnd(mesh.ne, 2, dt=torch.float64)
        ws = mesh.workspace(p, nsub, ckpt)
        ws.view(torch.uint8).fill_(255)   # NaN in every unwritten entry
        out.append(mesh.adjoint(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=nsub,
                                dt=case["tau"], params=p, ckpt_every=ckpt, lam_eta=lam[0],
                                lam_U=lam[1], lam_Uavg=lam[2], workspace=ws))
        torch.cuda.synchronize()
        assert mesh.check_faults() == 0
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and torch.equal(a, b)


# one tile per 64 vertices, one tile per CU, 1024-thread tiles of two rounds (FP64) or one
@pytest.mark.parametrize("n", [64, 250, 360])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_default_plan_of_the_adjoint_equals_the_per_substep_path(precision, n):
    from paper_2311_08241_amd import Mesh, Params, device_inputs
    case = sesynth.adjoint_c5(n=n)
    out = []
    for planned in (False, True):
        mesh = Mesh.from_dict(case, device=0)
        p = Params(precision=precision, eta_ref=case["eta_ref"] if precision == "f32" else 0.0)
        d = device_inputs(mesh, case, p)
        if planned:   # a forward step makes the mesh's default plans
            mesh.subcycle(d["eta"].clone(), d["U"].clone(), R=d["R"], f=d["f"], H0=d["H0"],
                          nsub=4, dt=case["tau"] / 8, params=p)
        lam = torch.linspace(0.5, 1.5, mesh.nv, dtype=p.dtype, device="cuda:0")
        out.append(mesh.adjoint(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=13,
                                dt=case["tau"] / 4, params=p, ckpt_every=5, lam_eta=lam))
        torch.cuda.synchronize()
        assert mesh.check_faults() == 0
    for a, b in zip(*out):
        assert torch.isfinite(a).all() and torch.equal(a, b)
