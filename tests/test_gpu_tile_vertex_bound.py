"""Tiles of more local vertices than a fixed-width record's 13 bits: thousands of triangles that
share nothing but the centres of small stars, their outer vertices far apart in the mesh order.
Such plans take compact rows; the tile path equals the per-substep path bit for bit."""
import numpy as np
import pytest

import sesynth
from paper_2311_08241_amd import Mesh

T, DEG = 682, 6


def _stars(n=T, deg=DEG):
    """n stars of deg triangles; along the mesh order (the quadrants of the plane along the
    Hilbert curve) first one outer vertex of n of the triangles, then the n centres, then the
    other outer vertices, so that the second tile holds every star."""
    r = sesynth.rng(3)
    corner = np.array([(0, 0), (1, 0), (1, 1), (0, 1)], float)
    xy, tri = [], []

    def put(quadrant):
        xy.append((corner[quadrant] + r.uniform(0.05, 0.45, 2)) * 1e4)
        return len(xy) - 1
    for i in range(n):
        c = put(1)
        for j in range(deg):
            a, b = put(0 if i * deg + j < n else 2), put(3)
            p, q, s = xy[c], xy[a], xy[b]
            left = (q[0] - p[0]) * (s[1] - p[1]) > (s[0] - p[0]) * (q[1] - p[1])
            tri.append((c, a, b) if left else (c, b, a))
    x, y = np.array(xy).T.copy()
    return dict(x=x, y=y, tri=np.array(tri, np.int32), periodic_x=False, periodic_y=False,
                period_x=0.0, period_y=0.0, spherical=False, radius=0.0, nx=x.size, ny=1, dx=1e4,
                dy=1e4)


def _lds_f32(nv, nvu, entries, block=512):
    off = 0
    for b in (4 * nv, 4 * nv, 4 * nvu, 4 * nvu, 8 * (block // 64) * 9, 4 * 18, 4 * (entries + 64),
              2 * (nvu + 4)):
        off = (off + b + 15) & ~15
    return off


@pytest.mark.parametrize("tile", [T, T - 60])
def test_plans_beyond_the_bound_take_compact_rows(tile):
    case = sesynth.random_case(_stars(), seed=2)
    st = Mesh.from_dict(case, device=-1).plan_stats(tile, 1, 512)
    assert st["ok_f32"] and (st["max_vtx"] > 8192) == (tile == T)
    # (a row of DEG triangles: DEG deposits, or the fixed width of 7)
    width = DEG if st["max_vtx"] > 8192 else 7
    assert st["lds_f32"] == _lds_f32(st["max_vtx"], tile, width * tile)


@pytest.mark.gpu
@pytest.mark.parametrize("tile", [T, T - 60])
def test_tile_path_beyond_the_bound_equals_the_per_substep_path(tile):
    torch = pytest.importorskip("torch")
    from paper_2311_08241_amd import Params, device_inputs
    case = sesynth.random_case(_stars(), seed=2, nsub=5, tau=2.0, U_amp=0.1)
    mesh = Mesh.from_dict(case, device=0)
    mesh.set_plan(tile, 1, 512)
    p = Params(g=case["g"], theta=case["theta"], precision="f32")
    out = []
    for plain in (True, False):
        d = device_inputs(mesh, case, p)
        Uavg = torch.empty((mesh.ne, 2), dtype=torch.float64, device="cuda:0")
        mesh.subcycle(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=case["nsub"],
                      dt=case["tau"], params=p, Uavg=Uavg, plain=plain)
        torch.cuda.synchronize()
        assert mesh.check_faults() == 0
        out.append((d["eta"], d["U"], Uavg))
    for x, y in zip(*out):
        assert torch.isfinite(x).all() and torch.equal(x, y)
