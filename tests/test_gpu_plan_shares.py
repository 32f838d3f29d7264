"""Shares of the LDS that a launch plan may ask for, sweeps of any row width:
every share that leaves 24 KiB beside x and the tables is taken, down to a ring
of one segment, and the bits stay the same."""
import numpy as np
import pytest

import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")

ICT = dict(b_fact="ict", c_fact="ict", b_order="mindeg", droptol=1e-4)
CHOL = dict(b_fact="chol", c_fact="chol")


@pytest.mark.parametrize("name,over,kw,most", [
    ("lap2d_64", dict(N=16), CHOL, 6),
    ("lap2d_64", dict(N=40), CHOL, 5),
    ("lap2d_64", dict(N=64), CHOL, 4),
    ("lap2d_64", dict(N=64), dict(CHOL, fact_prec="fp32", uk_prec="fp32"), 4),
    ("lap3d_64", dict(N=20, boxes=2), ICT, 5),
    ("lap3d_64", dict(N=20, boxes=2), dict(ICT, fact_prec="fp32", uk_prec="fp32"), 5),
    ("lap3d_64", dict(N=30, boxes=2), dict(ICT, b_fact="ildlt"), 3),
    ("lap3d_64", dict(N=26, boxes=2), dict(b_order="mindeg", refactor=True), 4),
], ids=lambda v: str(v))
def test_every_share_is_accepted(name, over, kw, most):
    print(name, over, kw, flush=True)
    pr = si.make_config(name, **over)
    slr = P.SLR(pr.csr, pr.part, pr.nparts, k=4, lanczos_steps=20, v0=pr.v0(), **kw)
    rn = np.random.Generator(np.random.PCG64(5)).uniform(-1, 1, (7, pr.n))
    r = torch.tensor(rn, dtype=torch.float64, device="cuda").t()
    one, all7 = slr.apply(r[:, 0].contiguous()), slr.apply(r)
    slots = []
    for div in range(1, most + 1):
        for persistent in (0, 2):
            slr.set_bsolve_plan(False, 512, div)
            slr.set_bsolve_plan(True, 256, div, 7, persistent)
            slots.append(slr.forms()["b_slots"])
            print("share 1 /", div, "slots", slots[-1], flush=True)
            assert torch.equal(slr.apply(r[:, 0].contiguous()), one)
            assert torch.equal(slr.apply(r), all7)
    assert min(slots) >= 1 and max(slots) >= 3
    # a serialised setup keeps the plan
    again = P.SLR.import_setup(slr.export_setup())
    assert again.forms()["b_slots"] == slots[-1]
    assert torch.equal(again.apply(r), all7) and torch.equal(again.apply(r[:, 0].contiguous()), one)


def test_a_ring_of_one_segment():
    pr = si.make_config("lap2d_64", N=64)
    slr = P.SLR(pr.csr, pr.part, pr.nparts, k=4, lanczos_steps=20, v0=pr.v0(), **CHOL)
    slr.set_bsolve_plan(False, 512, 4)
    assert slr.forms()["b_slots"] == 1
