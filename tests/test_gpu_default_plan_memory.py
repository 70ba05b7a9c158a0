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


# per local triangle its record, id, geometry and area, per local vertex its id, area and row offset
@pytest.mark.parametrize("first,second,plan,tri_bytes,vtx_bytes", [
    ("f64", "f32", (448, 4, 512), 8 + 4 + 16 + 4, 4 + 4 + 2),
    ("f32", "f64", (320, 4, 512), 8 + 4 + 32 + 8, 4 + 8 + 2)])
def test_own_plan_of_a_form_holds_one_precision(first, second, plan, tri_bytes, vtx_bytes):
    """The first call of a further form adds the tables of its precision alone, those of every
    tile as long as the largest tile's."""
    from paper_2311_08241_amd import Mesh, Params, device_inputs
    case = sesynth.random_case(sesynth.planar_grid(1100, 900, 1500.0, 1400.0, jitter=0.3,
                                                   r=sesynth.rng(5)), seed=4, nsub=3)
    mesh = Mesh.from_dict(case, device=0)
    used = None
    for f in (first, second):
        p = Params(g=case["g"], theta=case["theta"], precision=f)
        d, ws = device_inputs(mesh, case, p), mesh.workspace(p, case["nsub"])
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        mesh.subcycle(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=case["nsub"],
                      dt=case["tau"], params=p, workspace=ws)
        torch.cuda.synchronize()
        used = before - torch.cuda.mem_get_info()[0]
    st = mesh.plan_stats(*plan)   # the default of this size; nine arrays in 2 MiB pages
    tile = tri_bytes * (st["max_tri"] + 32) + vtx_bytes * (st["max_vtx"] + 32) + 128
    assert used <= st["ntiles"] * tile + 9 * (2 << 20)
