"""The apply in the caller's order: bit for bit the apply in the internal
order between two permutations, for every form of the B solves that gathers
and scatters, also in place and where the two vectors overlap."""
import ctypes

import numpy as np
import pytest

import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")


@pytest.mark.parametrize("plan", [None, (512, 1, 4, 1), (1024, 1, 16, 2)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("N,boxes,more", [
    (9, 2, {}),                                        # fewer rows than lanes in a subdomain
    (33, 2, {}),                                       # more rows than one batch of loads
    (20, 2, dict(b_fact="chol")),
    (26, 2, dict(b_order="mindeg")),
    (24, 2, dict(c_levels=2, c_order="hid")),
])
def test_apply_in_the_callers_order(N, boxes, more, prec, plan):
    print(N, boxes, more, prec, plan, flush=True)
    pr = si.make_config("lap3d_64", N=N, boxes=boxes)
    slr = P.SLR(pr.csr, pr.part, pr.nparts, v0=pr.v0(), k=4, lanczos_steps=20, fact_prec=prec, uk_prec=prec, **more)
    if plan:
        slr.set_bsolve_plan(False, *plan)
        slr.set_bsolve_plan(True, *plan)
    perm = torch.tensor(slr.export()["perm"], device="cuda")
    n = pr.n
    x = np.random.Generator(np.random.PCG64(2)).uniform(-1, 1, (7, n))
    r = torch.tensor(x, dtype=torch.float64, device="cuda")
    for c in (1, 2, 7):
        dd = slr.apply_dd(r[:c, perm].contiguous().t())
        want = torch.empty_like(r[:c])
        want[:, perm] = dd.t()
        assert torch.equal(slr.apply(r[:c].t()), want.t()), c

        def call(src, dst):
            P._check(P.slr_apply(slr._h, ctypes.c_void_p(src.data_ptr()), ctypes.c_void_p(dst.data_ptr()), c,
                                 P._stream(None)), "slr_apply")

        same = r[:c].clone()
        call(same, same)
        assert torch.equal(same, want), c
        # the result starts 3 entries into the input
        buf = torch.empty(c * n + 3, dtype=torch.float64, device="cuda")
        buf[:c * n] = r[:c].reshape(-1)
        call(buf, buf[3:])
        assert torch.equal(buf[3:].view(c, n), want), c
