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


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("model", [0, 1])
def test_tables_in_a_locality_order(model, prec):
    """A scrambled mesh, whose rows' order has no locality: the tables follow an order of their own,
    and so must everything per tet that the block kernels read (rest shapes, a material that
    changes), through changes of strategy.  Normwise 1e-10 (FP64) and 1e-5 (FP32 elements)."""
    m, _, _ = mg.scramble(mg.jitter(mg.kuhn_cube(11), 0.01, seed=0), seed=1)
    bound = 1e-10 if prec == "f64" else 1e-5
    rng = np.random.default_rng(3)
    E = [1e5 * np.exp(0.5 * rng.standard_normal(m.nt)) for _ in range(2)]
    d, u, w = mg.perturbed_state(m, 0.02, seed=10), mg.direction(m, 11), mg.direction(m, 12)
    mesh = ebbx.FemMesh(m.X, m.tets, m.pinned, model=model, elem_prec=ebbx.F64 if prec == "f64" else ebbx.F32,
                        E=1e5, nu=0.3, strategy=ebbx.STRAT_BLOCK)
    fem, dd, du, dw = mesh.fem, *(mesh.to_dev(a) for a in (d, u, w))

    def check(ref):
        err = lambda got, want: np.abs(mesh.from_dev(got) - want).max() / np.abs(want).max()
        assert err(fem.forces(dd), ref.forces(d)) <= bound
        assert err(fem.kmul(dd, du), ref.kmul(d, u)) <= bound
        assert err(fem.tmul(dd, du, dw), ref.tmul(d, u, w)) <= bound
        assert err(fem.jacobi_diag(dd, 1e-3), ref.jacobi_diag(d, 1e-3)) <= bound
        x, v = mesh.to_dev(d), mesh.to_dev(0.01 * u)
        st = fem.implicit_step(x, v, 1e-3, maxit=12)
        assert ebbx.stats_fetch(st).status == 0
        _d1, v1, _dv, _s = ref.implicit_step(d, 0.01 * u, 1e-3, maxit=12)
        assert err(v, v1) <= 10 * bound

    check(oracle.FEM.create(model, m.X, m.tets, 1e5, 0.3, pinned=m.pinned))
    for Et, how in zip(E, ((ebbx.STRAT_LANES, 128), (ebbx.STRAT_SEG, 0))):
        fem.set_material(E_tet=mesh.tet_to_dev(Et), nu=0.3)
        ref = oracle.FEM.create(model, m.X, m.tets, Et, 0.3, pinned=m.pinned)
        check(ref)
        fem.set_strategy(*how)
        check(ref)
        fem.set_strategy(ebbx.STRAT_BLOCK, 256)
        check(ref)
        fem.set_strategy(ebbx.STRAT_BLOCK_LDS, 128)
        check(ref)
        fem.set_strategy(ebbx.STRAT_BLOCK, 512 | ebbx.BLOCK_TPT2)
        check(ref)


@pytest.mark.parametrize("n,bt,morton", [(13, 64, False), (13, 64, True), (13, 256, True), (20, 64, False)])
def test_halo_rows(n, bt, morton):
    """Halo rows of one width (lattice order in blocks of 64 tets: a third of the shared vertices lie in
    more than 4 blocks) and of two, through the maps and a step.  Normwise 1e-10, FP64."""
    m = mg.jitter(mg.kuhn_cube(n), 0.01, seed=0)
    mesh = ebbx.FemMesh(m.X, m.tets, m.pinned, model=1, elem_prec=ebbx.F64, E=1e5, nu=0.3,
                        strategy=ebbx.STRAT_BLOCK, block=bt, morton=morton)
    ref = oracle.FEM.create(1, m.X, m.tets, 1e5, 0.3, pinned=m.pinned)
    d, u = mg.perturbed_state(m, 0.02, seed=10), mg.direction(m, 11)
    dd, du = mesh.to_dev(d), mesh.to_dev(u)
    err = lambda got, want: np.abs(mesh.from_dev(got) - want).max() / np.abs(want).max()
    assert err(mesh.fem.forces(dd), ref.forces(d)) <= 1e-10
    assert err(mesh.fem.kmul(dd, du), ref.kmul(d, u)) <= 1e-10
    x, v = mesh.to_dev(d), mesh.to_dev(0.01 * u)
    mesh.fem.implicit_step(x, v, 1e-3, tol=0.0, maxit=12)
    _d1, v1, _dv, _s = ref.implicit_step(d, 0.01 * u, 1e-3, tol=0.0, maxit=12)
    assert err(v, v1) <= 1e-10
