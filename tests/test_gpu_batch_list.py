"""The block lists of batches at the edges of the workgroups that form them by themselves: one mesh per
thread of the block kernel, up to 256, against the oracle mesh by mesh; more meshes take the list of a
kernel of its own.  Every batch has meshes that share blocks, ones that finish before the first
iteration (fully pinned) and ones that finish apart.

Tolerance (normwise per mesh): 1e-9, FP64 elements, both solves run to 1e-12."""
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


@pytest.mark.parametrize("meshes,block", [(2, 256), (64, 64), (65, 64), (65, 256), (128, 128), (255, 256),
                                          (256, 256), (257, 256), (256, 512)])
def test_lists(meshes, block):
    rng = np.random.default_rng(meshes + block)
    ms = [mg.jitter(mg.kuhn_cube(int(n)), 0.01, seed=100 + i) for i, n in enumerate(rng.integers(1, 4, meshes))]
    E, nu = 10.0 ** rng.uniform(4.0, 6.0, meshes), rng.uniform(0.3, 0.45, meshes)
    still = set(int(i) for i in rng.choice(meshes, meshes // 8, replace=False))
    for i in still:
        ms[i].pinned[:] = 1
    un = mg.union(ms)
    d0, v0 = 0.002 * rng.uniform(-1, 1, (un.nv, 3)), 0.05 * rng.uniform(-1, 1, (un.nv, 3))
    d0[un.pinned == 1] = 0.0
    v0[un.pinned == 1] = 0.0
    bm = ebbx.BatchMesh(un, E, nu, model=ebbx.NH, elem_prec=ebbx.F64, strategy=ebbx.STRAT_BLOCK, block=block)
    d, v = bm.to_dev(d0), bm.to_dev(v0)
    st = ebbx.stats_parse(bm.batch.implicit_step(d, v, 1e-3, tol=1e-12, maxit=400))
    got = bm.from_dev(v)
    for i, m in enumerate(ms):
        a, b = un.vptr[i], un.vptr[i + 1]
        assert st[i].status == ebbx.OK, i
        if i in still:
            assert st[i].iters == 0 and np.all(got[a:b] == 0.0), i
            continue
        ref = oracle.FEM.create(ebbx.NH, m.X, m.tets, E[i], nu[i], pinned=m.pinned)
        _d, want, _dv, _s = ref.implicit_step(d0[a:b], v0[a:b], 1e-3, tol=1e-12, maxit=400)
        assert np.abs(got[a:b] - want).max() <= 1e-9 * np.abs(want).max(), i
    bm.batch.close()
