"""Default plans when the device has no room for another one: a form that has not run yet takes
the plan that runs every form, with the same fields, and keeps it."""
import pytest

import sesynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _fill(room):
    """Tensors that hold the device's memory but for about `room` bytes."""
    held = []
    free, _ = torch.cuda.mem_get_info()
    for size in (free - (1 << 30), 256 << 20, room):
        for _ in range(32):
            try:
                held.append(torch.empty(size, dtype=torch.uint8, device="cuda:0"))
            except torch.cuda.OutOfMemoryError:
                break
    held.pop()
    torch.cuda.empty_cache()
    return held


def test_form_without_room_for_its_own_plan_runs_on_the_every_form_plan():
    from paper_2311_08241_amd import Mesh, Params, device_inputs
    case = sesynth.random_case(sesynth.planar_grid(1100, 900, 1500.0, 1400.0, jitter=0.3,
                                                   r=sesynth.rng(5)), seed=4, nsub=7)
    forms = {f: Params(g=case["g"], theta=case["theta"], precision=f) for f in ("f32", "f64")}
    out = []
    for scarce in (False, True):
        mesh = Mesh.from_dict(case, device=0)
        state = {f: device_inputs(mesh, case, p) for f, p in forms.items()}
        ws = {f: mesh.workspace(p, case["nsub"]) for f, p in forms.items()}

        def step(f):
            d = state[f]
            mesh.subcycle(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=case["nsub"],
                          dt=case["tau"], params=forms[f], workspace=ws[f])
            torch.cuda.synchronize()
        step("f32")
        filler = _fill(32 << 20) if scarce else []   # the tables of one more plan: over 80 MiB
        step("f64")
        step("f64")
        assert mesh.check_faults() == 0
        out.append([state["f64"][k].clone() if not scarce else state["f64"][k] for k in ("eta", "U")])
        del filler
        torch.cuda.empty_cache()
    for x, y in zip(*out):
        assert torch.equal(x, y)
