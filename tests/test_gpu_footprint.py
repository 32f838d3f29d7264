"""slr_analyze's estimate of the device footprint against what a setup holds
(without the apply's scratch): rows of fixed and of any width, exact, threshold
and zero-fill factors, interface factors by blocks and by their own launches,
and the recursive interface solver."""
import pytest

import slr_inputs as si

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1505_04340_amd")

ICT = dict(b_fact="ict", c_fact="ict", b_order="mindeg", droptol=1e-4)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name,over,kw", [
    ("lap2d_64", dict(N=64), dict(b_fact="chol", c_fact="chol")),
    ("lap3d_64", dict(N=20, boxes=2), ICT),
    ("lap3d_64", dict(N=33, boxes=3), dict(ICT, c_order="hid")),
    ("lap3d_64", dict(N=36, boxes=3), dict(c_order="multicolor")),
    ("lap3d_64", dict(N=36, boxes=3), dict(c_order="subdomain")),
    ("lap3d_64", dict(N=36, boxes=3), dict(c_fact="ict", c_order="hid", c_levels=2, k2=4, droptol=1e-4)),
], ids=lambda v: str(v))
def test_estimate(name, over, kw, prec):
    print(name, over, kw, prec, flush=True)
    pr = si.make_config(name, **over)
    kw = dict(kw, k=4, lanczos_steps=20, fact_prec=prec, uk_prec=prec)
    est = P.analyze(pr.csr, pr.part, pr.nparts, **kw)[0]["device_bytes"]
    slr = P.SLR(pr.csr, pr.part, pr.nparts, v0=pr.v0(), **kw)
    slr.trim()
    q = slr.query()
    scratch = 8 * (2 * q["s"] + max(512, q["lr_chunks"]) * 4)
    held = q["device_bytes"] - scratch
    print(est, held, est / held, flush=True)
    assert 0.8 * held <= est <= 1.25 * held
