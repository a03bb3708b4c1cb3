"""The block tables built on the device: element maps over them against the oracle where the
tables can go wrong (a ragged last block, one block, the largest blocks, wide corner slots, a
vertex shared by more blocks than the fixed-width halo rows hold, vertices with no tet)."""
import numpy as np
import pytest
import torch

import oracle
from paper_1506_07577_amd import meshgen as mg

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1506_07577_amd import ebbx
else:  # collected on a CPU host only to be deselected
    ebbx = None


def _fan(nt, isolated):
    """nt tets that share vertex `isolated` and nothing else, with that many vertices without a
    tet before them and as many after."""
    rng = np.random.default_rng(7)
    base = rng.uniform(0.5, 1.0, size=(nt, 3)) * rng.choice([-1.0, 1.0], size=(nt, 3))
    own = base[:, None, :] + 0.2 * rng.uniform(-1.0, 1.0, size=(nt, 3, 3))
    det = np.linalg.det(own)
    own[det < 0] = own[det < 0][:, ::-1]
    own[np.abs(det) < 0.01] = np.eye(3)
    lone = np.ones((isolated, 3))
    X = np.concatenate([lone, np.zeros((1, 3)), own.reshape(-1, 3), lone])
    tets = np.empty((nt, 4), dtype=np.int32)
    tets[:, 0] = isolated
    tets[:, 1:] = isolated + 1 + np.arange(3 * nt).reshape(nt, 3)
    return mg.Mesh(X=X, tets=tets, pinned=np.zeros(len(X), dtype=np.uint8), n=0, h=0.1)


MESHES = {
    "one_tet": lambda: mg.single_tet(),
    "ragged": lambda: mg.jitter(mg.kuhn_cube(5), 0.01, seed=0),   # 750 tets
    "scrambled": lambda: mg.scramble(mg.jitter(mg.kuhn_cube(7), 0.01, seed=0), seed=1)[0],
    "fan": lambda: _fan(1500, 3),
}


@pytest.mark.parametrize("bt", [64, 192, 256, 320, 1024])
@pytest.mark.parametrize("name", sorted(MESHES))
def test_block_tables(name, bt):
    m = MESHES[name]()
    mesh = ebbx.FemMesh(m.X, m.tets, m.pinned, model=ebbx.STVK, elem_prec=ebbx.F64, E=1e5, nu=0.3,
                        strategy=ebbx.STRAT_BLOCK, block=bt)
    ref = oracle.FEM.create(ebbx.STVK, m.X, m.tets, 1e5, 0.3, pinned=m.pinned)
    d, u = mg.perturbed_state(m, 0.02, seed=10), mg.direction(m, 11)
    for got, want in ((mesh.fem.forces(mesh.to_dev(d)), ref.forces(d)),
                      (mesh.fem.kmul(mesh.to_dev(d), mesh.to_dev(u)), ref.kmul(d, u))):
        got = mesh.from_dev(got)
        assert np.abs(got - want).max() <= 1e-10 * np.abs(want).max()
        assert not got[~np.isin(np.arange(m.nv), m.tets)].any()   # vertices with no tet get exactly zero
    # the tables are rebuilt for another size, and the sums stay reproducible
    f = mesh.fem.forces(mesh.to_dev(d))
    mesh.fem.set_strategy(ebbx.STRAT_BLOCK, 128)
    mesh.fem.forces(mesh.to_dev(d))
    mesh.fem.set_strategy(ebbx.STRAT_BLOCK, bt)
    assert torch.equal(f, mesh.fem.forces(mesh.to_dev(d)))
