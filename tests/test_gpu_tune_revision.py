"""Tuning caches of earlier builds: a choice is taken only if it was made among the kernels and tables
that are there now; other entries of the file are kept and the domain is timed again."""
import json

import numpy as np
import pytest
import torch

from paper_1506_07577_amd import meshgen as mg

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1506_07577_amd import ebbx
else:  # collected on a CPU host only to be deselected
    ebbx = None


def test_choices_of_an_earlier_build_are_timed_again(tmp_path):
    m, _, _ = mg.scramble(mg.jitter(mg.kuhn_cube(11), 0.01, seed=0), seed=1)
    path = tmp_path / "tune.json"
    mesh = ebbx.FemMesh(m.X, m.tets, m.pinned, model=ebbx.STVK, elem_prec=ebbx.F64, E=1e5, nu=0.3,
                        E_tet=np.full(m.nt, 1e5), strategy=ebbx.STRAT_BLOCK)
    assert len(mesh.fem.autotune(cache=str(path))) >= 8
    (key,) = json.loads(path.read_text())
    # the same domain as a build without the revision named it
    old = "|".join(p for p in key.split("|") if not (p[0] in "ro" and p[1:].isdigit()))
    assert old != key
    path.write_text('{\n"%s": {"strategy": %d, "block": 64, "us": 1.000}\n}\n' % (old, ebbx.STRAT_ATOMIC))
    assert len(mesh.fem.autotune(cache=str(path))) >= 8   # timed, not taken
    choice = mesh.fem.get_strategy()
    assert choice != (ebbx.STRAT_ATOMIC, 64)
    data = json.loads(path.read_text())
    assert set(data) == {old, key}
    assert (data[key]["strategy"], data[key]["block"]) == choice
    assert mesh.fem.autotune(cache=str(path)) == [] and mesh.fem.get_strategy() == choice
    # a batch of this one mesh, whose tables keep the rows' order, is another entry
    un = mg.union([m])
    bm = ebbx.BatchMesh(un, np.array([1e5]), np.array([0.3]), model=ebbx.STVK, elem_prec=ebbx.F64, strategy=ebbx.STRAT_BLOCK)
    assert len(bm.fem.autotune(cache=str(path))) >= 8
    assert len(json.loads(path.read_text())) == 3
    bm.batch.close()
    mesh.fem.close()
