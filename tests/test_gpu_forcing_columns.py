"""The forcing kernel's rounds: layer counts at the edges of its blocks of eight layers and of its
rounds (one of up to five blocks, then four at a time), with three to none of the layer arrays,
against the oracle within the bound of test_gpu_forcing."""
import numpy as np
import pytest

import sesynth
from test_gpu_forcing import _bound, _gpu, _orc

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


@pytest.mark.parametrize("drop", [(), ("RA",), ("RA", "RP"), ("RA", "RP", "RhV")])
@pytest.mark.parametrize("K", [8, 9, 17, 32, 33, 40, 41, 64, 65])
def test_forcing_rounds(K, drop):
    from paper_2311_08241_amd import Mesh
    case = sesynth.random_case(sesynth.tiny_mesh("chan54"), seed=5, nsub=4)
    d = sesynth.column_forcing(case, K=K, seed=K)
    mesh = Mesh.from_dict(case, device=0)
    for args in (drop, drop + ("nlev",)):
        full = d if "nlev" not in args else dict(d, nlev=np.full(d["nlev"].size, K, np.int32))
        assert np.all(np.abs(_gpu(mesh, d, drop=args) - _orc(full, drop=drop)) <= _bound(full))
    assert mesh.check_faults() == 0
