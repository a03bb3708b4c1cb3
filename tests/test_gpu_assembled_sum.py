"""The assembled blocks are sums of whole tet blocks: each tet's corner block is formed first and
then added, once, in ascending tet order (in FP64, FP32 elements' blocks rounded to FP32 before).

So an edge's block is, bit for bit, the sum over the tets of the blocks that each tet gives when it
is assembled alone, in every configuration of vertices per workgroup."""
import numpy as np
import pytest
import torch

from paper_1506_07577_amd import meshgen as mg

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1506_07577_amd import ebbx
else:  # collected on a CPU host only to be deselected
    ebbx = None


def _blocks(X, tets, d, model, prec):
    mesh = ebbx.FemMesh(X, tets, np.zeros(len(X), dtype=np.uint8), model=model,
                        elem_prec=ebbx.F64 if prec == "f64" else ebbx.F32, E=1e5, nu=0.35, strategy=ebbx.STRAT_BLOCK,
                        morton=False)
    mesh.fem.assemble(mesh.to_dev(d))
    row, col, blk = (a.cpu().numpy() for a in mesh.fem.edges())
    mesh.fem.close()
    tail = np.repeat(np.arange(len(X)), np.diff(row))
    return {(int(i), int(j)): blk[:, e] for e, (i, j) in enumerate(zip(tail, col))}


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("model", [0, 1])
def test_blocks_are_sums_of_whole_tet_blocks(model, prec):
    m = mg.jitter(mg.kuhn_cube(3), 0.01, seed=0)
    d = mg.perturbed_state(m, 0.02, seed=10)
    got = _blocks(m.X, m.tets, d, model, prec)
    want = {}
    for t in m.tets:   # ascending
        # the tet alone, its corners in the order of their vertices' numbers
        v = np.sort(t)
        local = np.searchsorted(v, t).astype(np.int32)[None]
        for (i, j), b in _blocks(m.X[v], local, d[v], model, prec).items():
            key = (int(v[i]), int(v[j]))
            want[key] = want.get(key, np.zeros(9)) + b
    assert got.keys() == want.keys()
    for key, b in want.items():
        b = b.astype(np.float32).astype(np.float64) if prec == "f32" else b
        assert np.array_equal(got[key], b), key
