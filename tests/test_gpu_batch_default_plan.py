"""Default plan of a batch: one per precision.  A call gives the same bits, volumes (summed tile
by tile) among them, whether or not the batch ran in the other precision before; alternating
precisions, graphs and eager calls keep their own tables."""
import numpy as np
import pytest

import sesynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _batch(cases):
    from paper_2311_08241_amd import Batch, Mesh
    return Batch([Mesh.from_dict(c, device=0) for c in cases])


def _run(batch, cases, prec, use_graph, stream):
    from paper_2311_08241_amd import Params, batch_inputs
    p = Params(g=9.81, theta=0.14, precision=prec)
    nsub = [c["nsub"] for c in cases]
    with torch.cuda.stream(stream):
        d = batch_inputs(batch, cases, p)
        Uavg = torch.empty((batch.ne, 2), dtype=torch.float64, device="cuda:0")
        vol = torch.empty(batch.volume_size(p, nsub), dtype=torch.float64, device="cuda:0")
        batch.subcycle(d["eta"], d["U"], R=d["R"], f=d["f"], H0=d["H0"], nsub=nsub,
                       dt=[c["tau"] for c in cases], params=p, Uavg=Uavg, volume=vol,
                       use_graph=use_graph, stream=stream)
    stream.synchronize()
    assert batch.check_faults(stream=stream) == 0
    return d, (d["eta"].cpu().numpy(), d["U"].cpu().numpy(), Uavg.cpu().numpy(), vol.cpu().numpy())


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("n,lo,hi", [(5, 800, 6000), (10, 9000, 20000)])
def test_results_do_not_depend_on_the_precisions_run_before(n, lo, hi, use_graph):
    cases = sesynth.batch_c4(seed=3, nmembers=n, nv_lo=lo, nv_hi=hi, m_lo=5, m_hi=23)
    s = torch.cuda.Stream()
    alone = {prec: _run(_batch(cases), cases, prec, use_graph, s)[1] for prec in ("f32", "f64")}
    for order in (("f32", "f64", "f32", "f64"), ("f64", "f32", "f64")):
        batch = _batch(cases)
        for prec in order:
            for x, y in zip(alone[prec], _run(batch, cases, prec, use_graph, s)[1]):
                assert np.array_equal(x, y), (order, prec)
