"""Sweeps of any row width (exact and threshold factors): chains, panels and
pieces at their edges, every number of columns that changes how the waves
share the work, few ring slots, and setups serialised in the previous form.

Bars: FP64 apply <= 1e-12 relative per column against the oracle on the same
stored data, FP32 <= 1e-5 (as the other parity tests); a column's bits do not
depend on the columns beside it nor on the launch shape."""
import os

import numpy as np
import pytest

import oracle as O
import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")

GOLDEN = os.path.join(os.path.dirname(__file__), "golden")

# name, size, factors, order, drop tolerance: interiors of 9, 16, 81 and 361
# rows in one chain run, threshold factors with wide levels before the run
CASES = [
    ("lap2d_64", dict(N=8), "chol", "chol", "natural", 0.0),
    ("lap2d_64", dict(N=10), "chol", "chol", "natural", 0.0),
    ("lap2d_64", dict(N=20), "chol", "chol", "natural", 0.0),
    ("lap2d_64", dict(N=40), "chol", "chol", "natural", 0.0),
    ("lap3d_64", dict(N=20, boxes=2), "ict", "ict", "mindeg", 1e-4),
    ("shifted3d_128", dict(N=26, boxes=2, neg=4), "ildlt", "ict", "mindeg", 1e-5),
]


def _setup(name, over, bf, cf, bo, tau, prec="fp64", **more):
    pr = si.make_config(name, **over)
    kw = dict(k=4, lanczos_steps=20, b_fact=bf, c_fact=cf, b_order=bo, droptol=tau, fact_prec=prec, uk_prec=prec)
    kw.update(more)
    return pr, kw, P.SLR(pr.csr, pr.part, pr.nparts, v0=pr.v0(), **kw)


def _vectors(n, c):
    r = np.random.Generator(np.random.PCG64(5)).uniform(-1, 1, (c, n))
    return torch.tensor(r, dtype=torch.float64, device="cuda").t()


def _oracle(pr, kw, slr):
    ex = slr.export()
    kw = {k: v for k, v in kw.items() if k not in ("k", "lanczos_steps")}
    return O.setup(pr.scipy(), pr.part, pr.nparts, slr.info["k"], lowrank=(ex["U"], ex["lambda"], ex["theta"]), **kw)


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]['N']}-{c[2]}")
def test_apply_matches_the_oracle_at_every_column_count(case, prec, tol):
    print(case, prec, flush=True)
    pr, kw, slr = _setup(*case, prec=prec)
    r = _vectors(pr.n, 17)
    alone = torch.stack([slr.apply(r[:, i].contiguous()) for i in range(17)], 1)
    ref = _oracle(pr, kw, slr)
    for i in (0, 16):
        z = ref.apply(r[:, i].cpu().numpy())
        assert np.linalg.norm(alone[:, i].cpu().numpy() - z) <= tol * np.linalg.norm(z)
    for c in (2, 3, 4, 6, 7, 17):
        assert torch.equal(slr.apply(r[:, :c]), alone[:, :c]), c


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 1e-5)])
@pytest.mark.parametrize("name,over,order,cf", [
    ("lap3d_64", dict(N=16, boxes=2), "hid", "ict"),        # connectors, small remainder
    ("lap3d_64", dict(N=33, boxes=3), "hid", "ict"),        # uneven boxes
    ("lap3d_64", dict(N=20, boxes=2), "subdomain", "ict"),  # one block, wide rows
    ("lap3d_64", dict(N=24, boxes=3), "subdomain", "ic0"),  # one block, fixed width
])
def test_deep_interface_factor(name, over, order, cf, prec, tol):
    print(name, over, order, cf, prec, flush=True)
    pr, kw, slr = _setup(name, over, "ic0", cf, "natural", 1e-4, prec=prec, c_order=order)
    assert slr.info["c_levels"] > 8
    r = _vectors(pr.n, 17)
    alone = torch.stack([slr.apply(r[:, i].contiguous()) for i in range(17)], 1)
    ref = _oracle(pr, kw, slr)
    z = ref.apply(r[:, 3].cpu().numpy())
    assert np.linalg.norm(alone[:, 3].cpu().numpy() - z) <= tol * np.linalg.norm(z)
    for c in (3, 5, 17):
        assert torch.equal(slr.apply(r[:, :c]), alone[:, :c]), c
    assert torch.equal(P.SLR.import_setup(slr.export_setup()).apply(r), alone)


def test_few_ring_slots_and_a_resident_grid_keep_the_bits():
    pr, kw, slr = _setup("lap3d_64", dict(N=20, boxes=2), "ict", "ict", "mindeg", 1e-4)
    r = _vectors(pr.n, 5)
    one, five = slr.apply(r[:, 0].contiguous()), slr.apply(r)
    done = 0
    for div in range(2, 9):
        try:
            slr.set_bsolve_plan(False, 512, div)
            slr.set_bsolve_plan(True, 256, div, 2, 1)
        except P.SLRError as e:
            assert e.code == P.SLR_ERR_ARG
            continue
        print("share of the LDS: 1 /", div, flush=True)
        assert torch.equal(slr.apply(r[:, 0].contiguous()), one)
        assert torch.equal(slr.apply(r), five)
        done += 1
    assert done >= 2


@pytest.mark.parametrize("name,over,more", [
    ("chol_fp64", dict(N=16), dict(b_fact="chol", c_fact="chol")),
    ("ict_fp32", dict(N=22), dict(b_fact="ict", c_fact="ict", b_order="mindeg", fact_prec="fp32", droptol=1e-4)),
])
def test_setup_serialised_in_the_previous_form(name, over, more):
    pr = si.make_config("lap2d_64", **over)
    with open(os.path.join(GOLDEN, f"setup_v2_lap2d_{name}.bin"), "rb") as f:
        old = P.SLR.import_setup(f.read())
    ex = old.export()
    new = P.SLR(pr.csr, pr.part, pr.nparts, k=4, lowrank=(ex["U"], ex["lambda"], ex["theta"]), **more)
    r = _vectors(pr.n, 5)
    z = old.apply(r)
    assert torch.equal(z, new.apply(r))
    assert torch.equal(P.SLR.import_setup(old.export_setup()).apply(r), z)
    ref = O.setup(pr.scipy(), pr.part, pr.nparts, 4, lowrank=(ex["U"], ex["lambda"], ex["theta"]), **more)
    zo = ref.apply(r[:, 0].cpu().numpy())
    tol = 1e-5 if more.get("fact_prec") == "fp32" else 1e-12
    assert np.linalg.norm(z[:, 0].cpu().numpy() - zo) <= tol * np.linalg.norm(zo)


def test_a_value_that_is_not_finite():
    """An infinite entry makes the chain solve again under masks; the next
    call is as before."""
    pr, kw, slr = _setup("lap2d_64", dict(N=20), "chol", "chol", "natural", 0.0)
    r = _vectors(pr.n, 1)[:, 0].contiguous()
    z = slr.apply(r)
    bad = r.clone()
    bad[int(slr.export()["perm"][0])] = float("inf")
    assert not bool(torch.isfinite(slr.apply(bad)).all())
    assert torch.equal(slr.apply(r), z)
