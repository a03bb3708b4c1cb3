"""A change of strategy that fails half-way for want of memory: calls that need the tables it was
replacing are refused (E_STATE), never launched over them, until a strategy is set again; where the
old tables are still whole the results stay right.  The allocator hook fails at every allocation of
the change in turn."""
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


class _Memory:
    """The library's allocator hook (torch's allocator), out of memory from the n-th allocation on."""

    def __init__(self, n):
        self.n, self.count = n, 0
        self.alloc, self.free = ebbx._ALLOC_T(self._alloc), ebbx._FREE_T(ebbx._torch_free)

    def _alloc(self, nbytes, ctx, stream):
        self.count += 1
        return None if self.count > self.n else ebbx._torch_alloc(nbytes, ctx, stream)

    def __enter__(self):
        ebbx._check(ebbx.lib().ebbx_set_allocator(self.alloc, self.free, None))
        return self

    def __exit__(self, *exc):
        ebbx.use_torch_allocator(True)


_keep = []   # buffers are released through the hook that made them: the hooks live as long as the process


def _failing(n):
    _keep.append(_Memory(n))
    return _keep[-1]


CHANGES = {   # from, to
    "block_block": ((0, 256), (0, 128)),
    "block_pipe": ((0, 256), (1, 2)),
    "pipe_block": ((1, 2), (0, 256)),
    "owner_owner": ((2, 64), (2, 128)),
    "block_lanes": ((0, 256), (3, 128)),
}


@pytest.mark.parametrize("name", sorted(CHANGES))
def test_failed_change_of_strategy(name):
    kinds = (ebbx.STRAT_BLOCK, ebbx.STRAT_PIPE, ebbx.STRAT_OWNER, ebbx.STRAT_LANES)
    (k0, b0), (k1, b1) = CHANGES[name]
    m = mg.jitter(mg.kuhn_cube(11), 0.01, seed=0)
    if name in ("block_block", "block_lanes"):   # tables in a locality order of their own
        m, _, _ = mg.scramble(m, seed=1)
    ref = oracle.FEM.create(ebbx.STVK, m.X, m.tets, 1e5, 0.3, pinned=m.pinned)
    d, u = mg.perturbed_state(m, 0.02, seed=10), mg.direction(m, 11)
    want_f, want_y = ref.forces(d), ref.kmul(d, u)
    _d1, want_v, _dv, _s = ref.implicit_step(d, 0.01 * u, 1e-3, maxit=4)
    mesh = ebbx.FemMesh(m.X, m.tets, m.pinned, model=ebbx.STVK, elem_prec=ebbx.F64, E=1e5, nu=0.3)
    dd, du = mesh.to_dev(d), mesh.to_dev(u)

    def step():
        x, v = mesh.to_dev(d), mesh.to_dev(0.01 * u)
        mesh.fem.implicit_step(x, v, 1e-3, maxit=4)
        return v

    calls = ((lambda: mesh.fem.forces(dd), want_f), (lambda: mesh.fem.kmul(dd, du), want_y), (step, want_v))
    refused = failed = n = 0
    while True:
        mesh.fem.set_strategy(kinds[k0], b0)
        for call, want in calls:   # the domain is whole again
            assert np.abs(mesh.from_dev(call()) - want).max() <= 1e-10 * np.abs(want).max()
        torch.cuda.synchronize()
        try:
            with _failing(n):
                mesh.fem.set_strategy(kinds[k1], b1)
        except ebbx.EbbxError as e:
            assert e.code == ebbx.E_OOM
        else:
            break
        failed += 1
        assert mesh.fem.get_strategy() == (kinds[k0], b0)
        for call, want in calls:
            try:
                got = call()
            except ebbx.EbbxError as e:
                assert e.code == ebbx.E_STATE
                refused += 1
            else:
                assert np.abs(mesh.from_dev(got) - want).max() <= 1e-10 * np.abs(want).max()
        torch.cuda.synchronize()
        n += 1
    assert failed >= 3 and refused >= 3
    for call, want in calls:
        assert np.abs(mesh.from_dev(call()) - want).max() <= 1e-10 * np.abs(want).max()
    mesh.fem.close()
