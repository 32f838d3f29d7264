"""The built-in launch shape of the B solves of several columns is not far
from the best one: the columns go into as many groups as the compute units hold
in one round, whatever the number of subdomains."""
import pytest

import slr_inputs as si

pytestmark = pytest.mark.gpu

P = pytest.importorskip("paper_1505_04340_amd")


@pytest.mark.parametrize("q,N,counts", [(12, 480, (3, 4, 6)), (10, 400, (5, 7)), (8, 320, (4, 8)), (4, 160, (5,))])
def test_columns_a_workgroup(q, N, counts):
    pr = si.make_config("lap2d_64", N=N)
    part = si.box_partition_2d(N, q, q)
    slr = P.SLR(pr.csr, part, q * q, k=4, lanczos_steps=8, c_order="multicolor", fact_prec="fp32", uk_prec="fp32")
    for c in counts:
        def us():
            return min(slr.time_kernel("bsolve2", c, 20) for _ in range(3)) * 1e3
        slr.set_bsolve_plan(True, 0)
        mine, other = us(), {}
        for R in range(1, c + 1):
            slr.set_bsolve_plan(True, 1024, 1, R, 0)
            other[R] = us()
        print(q * q, "subdomains", c, "columns", mine, other, flush=True)
        assert mine <= 1.25 * min(other.values())
