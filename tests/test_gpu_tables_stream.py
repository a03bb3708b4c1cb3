"""Block tables built on a stream that the null stream does not wait for."""
import json
import threading

import pytest
import torch

from paper_1506_07577_amd import meshgen as mg

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_1506_07577_amd import ebbx
else:  # collected on a CPU host only to be deselected
    ebbx = None


def test_locality_order_on_a_stream_of_its_own(tmp_path):
    """Tables built on a non-blocking stream (a tuning cache's hit, which takes the caller's stream)
    while another stream keeps the device busy: the same order, so the same sums, bit for bit, as
    those that set_strategy builds on the null stream."""
    m, _, _ = mg.scramble(mg.jitter(mg.kuhn_cube(30), 0.01, seed=0), seed=1)
    mesh = ebbx.FemMesh(m.X, m.tets, m.pinned, model=ebbx.STVK, elem_prec=ebbx.F64, E=1e5, nu=0.3,
                        strategy=ebbx.STRAT_BLOCK)
    d, u = mesh.to_dev(mg.perturbed_state(m, 0.02, seed=10)), mesh.to_dev(mg.direction(m, 11))
    path = tmp_path / "tune.json"
    mesh.fem.autotune(d, u, cache=str(path))
    (entry,) = json.loads(path.read_text()).values()
    key = path.read_text().split('"')[1]
    entry.update(strategy=ebbx.STRAT_BLOCK, block=256)   # the strategy whose tables take that order
    path.write_text('{\n"%s": %s\n}\n' % (key, json.dumps(entry)))
    mesh.fem.set_strategy(ebbx.STRAT_LANES, 64)
    mesh.fem.set_strategy(ebbx.STRAT_BLOCK, 256)
    want = mesh.fem.kmul(d, u)
    busy, side = torch.cuda.Stream(), torch.cuda.Stream()
    a = torch.randn(4096, 4096, device="cuda")
    torch.cuda.synchronize()
    stop = threading.Event()

    def load():
        with torch.cuda.stream(busy):
            while not stop.is_set():
                for _ in range(4):
                    torch.mm(a, a)
                busy.synchronize()

    t = threading.Thread(target=load)
    t.start()
    try:
        for _ in range(8):
            mesh.fem.set_strategy(ebbx.STRAT_LANES, 64)   # the rows' own order
            with torch.cuda.stream(side):
                assert mesh.fem.autotune(d, u, cache=str(path)) == []
                got = mesh.fem.kmul(d, u)
            side.synchronize()
            assert mesh.fem.get_strategy() == (ebbx.STRAT_BLOCK, 256)
            assert torch.equal(got, want)
    finally:
        stop.set()
        t.join()
