"""Tile tables of the trim/z* consumer: kept for every class of layer counts, so that a call
finds those of its class whatever ran in between (a captured call, which may not build any,
included)."""
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
