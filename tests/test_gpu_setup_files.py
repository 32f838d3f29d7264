"""Serialised setups of deep interface factors: the file holds the block form
(import does not build it again and holds no second copy of the factor), and
files of the form before, which hold the schedules only."""
import os

import numpy as np
import pytest

import oracle as O
import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")

GOLDEN = os.path.join(os.path.dirname(__file__), "golden")


def _vectors(n, c):
    r = np.random.Generator(np.random.PCG64(5)).uniform(-1, 1, (c, n))
    return torch.tensor(r, dtype=torch.float64, device="cuda").t()


@pytest.mark.parametrize("name,N,more,lead", [
    ("chol_fp64", 12, dict(b_fact="chol", c_fact="chol"), False),
    ("hid_fp32", 26, dict(b_fact="ict", c_fact="ict", b_order="mindeg", c_order="hid", fact_prec="fp32",
                          droptol=1e-4), True),
])
def test_a_file_with_the_schedules_only(name, N, more, lead):
    pr = si.make_config("lap2d_64", N=N)
    with open(os.path.join(GOLDEN, f"setup_v3_lap2d_{name}.bin"), "rb") as f:
        old = P.SLR.import_setup(f.read())
    ex = old.export()
    lr = (ex["U"], ex["lambda"], ex["theta"])
    new = P.SLR(pr.csr, pr.part, pr.nparts, k=4, lowrank=lr, **more)
    assert old.forms() == new.forms() and new.forms()["c_deep"] == 1 and (new.forms()["c_lead"] > 0) == lead
    r = _vectors(pr.n, 5)
    z = old.apply(r)
    assert torch.equal(z, new.apply(r))
    again = P.SLR.import_setup(old.export_setup())
    assert again.forms() == old.forms() and torch.equal(again.apply(r), z)
    zo = O.setup(pr.scipy(), pr.part, pr.nparts, 4, lowrank=lr, **more).apply(r[:, 0].cpu().numpy())
    tol = 1e-5 if more.get("fact_prec") == "fp32" else 1e-12
    assert np.linalg.norm(z[:, 0].cpu().numpy() - zo) <= tol * np.linalg.norm(zo)


@pytest.mark.parametrize("order", ["hid", "subdomain"])
def test_an_import_is_the_context_that_was_exported(order):
    pr = si.make_config("lap3d_64", N=16, boxes=2)
    kw = dict(b_fact="ict", c_fact="ict", b_order="mindeg", c_order=order, droptol=1e-4)
    a = P.SLR(pr.csr, pr.part, pr.nparts, k=4, lanczos_steps=20, v0=pr.v0(), **kw)
    blob = a.export_setup()
    b = P.SLR.import_setup(blob)
    assert a.forms()["c_deep"] == 1 and b.forms() == a.forms()
    assert b.export_setup() == blob
    r = _vectors(pr.n, 3)
    assert torch.equal(a.apply(r), b.apply(r))
    # one copy of C's factor: its entries in the block form only
    A = P.analyze(pr.csr, pr.part, pr.nparts, k=4, **kw)[0]
    assert a.query()["s"] == A["s"]
    for ctx in (a, b):
        ctx.trim()
    assert b.query()["device_bytes"] <= a.query()["device_bytes"]
    # files cut short or changed are refused
    for bad in (blob[:-1], blob[:40], blob[:7] + b"5" + blob[8:], blob[:-9] + bytes([blob[-9] ^ 1]) + blob[-8:]):
        with pytest.raises(P.SLRError) as e:
            P.SLR.import_setup(bad)
        assert e.value.code == P.SLR_ERR_ARG
