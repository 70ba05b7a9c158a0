"""Tile tables of the trim/z* consumer: kept for every class of layer counts, so that a call
finds those of its class whatever ran in between (a captured call, which may not build any,
included); and used for rows of up to 126 triangles (up to 24 layers), 94 (25 to 32) and 62, as
far as their vertices fit a tile."""
import ctypes

import numpy as np
import pytest

import sesynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _inputs(mesh, K, seed=1):
    g = torch.Generator().manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, dtype=torch.float64).cuda()
    H0 = 1000.0 + 50.0 * rnd(mesh.nv)
    h0 = (H0[:, None] / K).expand(-1, K).contiguous()
    return dict(H0=H0, eta_new=0.3 * rnd(mesh.nv), Uavg=rnd(mesh.ne, 2), Ustar=rnd(mesh.ne, K, 2),
                hn=h0 + 0.001 * rnd(mesh.nv, K), h0=h0, tau=100.0)


def _three_launches(mesh, inp):   # in place: the form without tiles
    U = inp["Ustar"].clone()
    return mesh.trim_zstar(**dict(inp, Ustar=U), U=U)


def test_classes_of_layer_counts_keep_their_tables():
    from paper_2311_08241_amd import Mesh
    mesh = Mesh.from_dict(sesynth.channel_c2(nx=96, ny=40, nsteps=1), device=0)
    inp = {K: _inputs(mesh, K) for K in (5, 12, 20, 28, 40, 60)}
    ref = {K: _three_launches(mesh, i) for K, i in inp.items()}
    out = {K: mesh.trim_zstar(**i) for K, i in inp.items()}   # builds each class's tables
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for K, i in inp.items():
            mesh.trim_zstar(**i, U=out[K][0], hnew=out[K][1], w=out[K][2])
    for _ in range(2):
        for o in out.values():
            for t in o:
                t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for K in inp:
            for a, b in zip(out[K], ref[K]):
                assert torch.equal(a, b), K


def _hub(deg):
    """A planar grid with a vertex far below it, joined to deg edges of the lowest row."""
    m = sesynth.planar_grid(150, 24, 1500.0, 1400.0)
    x, y, tri = m["x"], m["y"], m["tri"]
    south = np.argsort(y, kind="stable")[:150]
    south = south[np.argsort(x[south])][:deg + 1]
    hub = np.full(deg, x.size)
    x, y = np.append(x, x[south].mean()), np.append(y, y.min() - 50000.0)
    return dict(m, x=x, y=y, tri=np.concatenate([tri, np.stack([hub, south[1:], south[:-1]], -1)
                                                 .astype(np.int32)]))


def _kernels(fn):
    """Kernel launches that fn makes, from the nodes of a captured graph."""
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fn()
    n = ctypes.c_size_t()
    with open("/proc/self/maps") as maps:   # the runtime that is loaded
        lib = ctypes.CDLL(next(line.split()[-1] for line in maps if "libamdhip64" in line))
    assert lib.hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(n)) == 0
    return n.value


# (an open fan of n triangles has n + 2 vertices; a tile holds as many as triangles)
# a row at the edges of the two tile sizes of a layer count, and beyond the larger one
@pytest.mark.parametrize("K,deg,launches", [
    (17, 94, 1), (17, 95, 1), (24, 110, 1), (24, 126, 1), (24, 127, 3), (25, 62, 1), (25, 63, 1),
    (32, 80, 1), (32, 94, 1), (32, 95, 3), (40, 62, 1), (40, 63, 3), (16, 126, 1), (16, 127, 3)])
def test_rows_near_the_tile_sizes(K, deg, launches):
    from paper_2311_08241_amd import Mesh
    mesh = Mesh.from_dict(sesynth.random_case(_hub(deg), seed=1), device=0)
    assert int(np.diff(mesh.csr()[1]).max()) == deg
    inp = _inputs(mesh, K)
    ref = _three_launches(mesh, inp)
    out = mesh.trim_zstar(**inp)
    for a, b in zip(out, ref):
        assert torch.equal(a, b)
    assert _kernels(lambda: mesh.trim_zstar(**inp, U=out[0], hnew=out[1], w=out[2])) == launches
