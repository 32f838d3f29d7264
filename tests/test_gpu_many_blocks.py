"""More blocks than compute units, rows of any width: several workgroups share
a compute unit (subdomains), and connectors are solved by workgroups whose
solver waves take columns of their own.  Bars: FP64 apply <= 1e-12 relative
per column against the oracle on the same stored data, FP32 <= 1e-5; a
column's bits do not depend on the columns beside it."""
import numpy as np
import pytest

import oracle as O
import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")


def _check(pr, part, p, kw, prec, counts):
    kw = dict(kw, fact_prec=prec, uk_prec=prec)
    G = P.SLR(pr.csr, part, p, k=4, lanczos_steps=20, v0=pr.v0(), **kw)
    rn = np.random.Generator(np.random.PCG64(5)).uniform(-1, 1, (max(counts), pr.n))
    r = torch.tensor(rn, dtype=torch.float64, device="cuda").t()
    alone = torch.stack([G.apply(r[:, i].contiguous()) for i in range(max(counts))], 1)
    for c in counts:
        assert torch.equal(G.apply(r[:, :c]), alone[:, :c]), c
    ex = G.export()
    low = dict(lowrank=(ex["U"], ex["lambda"], ex["theta"]))
    if kw.get("c_levels") == 2:
        ei = G.export_inner()
        low["lowrank2"] = (ei["U"], ei["lambda"], ei["theta"])
    ref = O.setup(pr.csr, part, p, 4, v0=pr.v0(), **low, **kw)
    z = ref.apply(rn[1])
    assert np.linalg.norm(alone[:, 1].cpu().numpy() - z) <= (1e-12 if prec == "fp64" else 1e-5) * np.linalg.norm(z)
    return G


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("bf,bo", [("chol", "natural"), ("ict", "mindeg")])
def test_subdomains(bf, bo, prec):
    print(bf, bo, prec, flush=True)
    pr = si.make_config("lap2d_64", N=170)
    part = si.box_partition_2d(170, 17, 17)
    _check(pr, part, 289, dict(b_fact=bf, b_order=bo, c_fact="ic0", c_order="multicolor", droptol=1e-4), prec,
           (2, 5, 9))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("tau", [1e-2, 1e-5])
def test_connectors(tau, prec):
    print(tau, prec, flush=True)
    pr = si.make_config("lap3d_64", N=36, boxes=6)
    G = _check(pr, pr.part, pr.nparts,
               dict(c_fact="ict", c_order="hid", c_levels=2, k2=4, droptol=tau), prec, (2, 3, 4, 7))
    assert G.forms()["c1_slots"] >= 2
