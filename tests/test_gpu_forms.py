"""Which form a context's solves take: a test of a form asks that it was taken.

The interface factor by blocks (leading blocks and a remainder, one block, or
the schedule's own launches), and the refactorisation by blocks or level by
level.  The choices depend on sizes and patterns only."""
import ctypes

import pytest

import slr_inputs as si

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1505_04340_amd")


def _slr(name, over, **kw):
    pr = si.make_config(name, **over)
    return pr, P.SLR(pr.csr, pr.part, pr.nparts, v0=pr.v0(), **dict(dict(k=4, lanczos_steps=20, droptol=1e-4), **kw))


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name,over,order,cf,form", [
    ("lap3d_64", dict(N=16, boxes=2), "hid", "ict", "split"),        # connectors and a remainder
    ("lap3d_64", dict(N=33, boxes=3), "hid", "ict", "split"),
    ("lap2d_64", dict(N=200), "hid", "ic0", "split"),                # the same in rows of fixed width
    ("lap3d_64", dict(N=20, boxes=2), "subdomain", "ict", "one"),    # one block
    ("lap3d_64", dict(N=24, boxes=3), "subdomain", "ic0", "one"),
    ("lap3d_64", dict(N=64, boxes=4), "subdomain", "ic0", "own"),    # 67,032 rows: no workgroup's LDS holds them
    ("lap3d_64", dict(N=24, boxes=3), "multicolor", "ic0", "own"),   # a few wide levels
])
def test_form_of_the_interface_factor(name, over, order, cf, form, prec):
    print(name, over, order, cf, prec, flush=True)
    pr, slr = _slr(name, over, c_order=order, c_fact=cf, fact_prec=prec, uk_prec=prec)
    f = slr.forms()
    assert f["c_deep"] == (form != "own")
    if form == "split":
        # pieces of 128 rows or more, a remainder that is not empty
        assert 0 < f["c_lead"] < slr.info["s"] and 1 < f["c_blocks"] <= f["c_lead"] // 128 + 1
    else:
        assert (f["c_lead"], f["c_blocks"]) == (0, 0)


@pytest.mark.parametrize("name,over,order,blocks", [
    ("lap3d_64", dict(N=26, boxes=2), "natural", True),    # 3 entries a row at most
    ("lap2d_64", dict(N=40), "mindeg", True),              # 4 at most: the limit
    ("lap3d_64", dict(N=26, boxes=2), "mindeg", False),    # rows of 5 and 6 among them: level by level
])
def test_form_of_the_refactorisation(name, over, order, blocks):
    pr, slr = _slr(name, over, b_order=order, refactor=True)
    assert slr.forms()["refactor_blocks"] == (pr.nparts if blocks else 0)


@pytest.mark.parametrize("name,over,kw", [
    ("lap2d_64", dict(N=40), dict(b_fact="chol", c_fact="chol")),
    ("lap3d_64", dict(N=20, boxes=2), dict(b_fact="ict", c_fact="ict", b_order="mindeg")),
    ("lap3d_64", dict(N=24, boxes=3), dict(c_fact="ict", c_order="hid", c_levels=2, k2=4)),
])
def test_levels_are_those_of_the_schedules(name, over, kw):
    pr, slr = _slr(name, over, **kw)
    info = P.analyze(pr.csr, pr.part, pr.nparts, **dict(dict(k=4, droptol=1e-4), **kw))[0]
    assert slr.info["b_levels_max"] == info["b_levels_max"] and slr.info["c1_levels"] == info["c1_levels"]


def test_layout():
    assert ctypes.sizeof(P.slr_forms) == 48 and P.slr_forms.c_deep.offset == 16
