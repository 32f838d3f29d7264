"""CG iterations on several columns: tiles of columns at their edges and row
counts that leave threads, blocks or a whole launch row idle.  A column's
iterates do not depend on the columns beside it (to the bit), and its true
residual meets the tolerance."""
import numpy as np
import pytest

import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")


@pytest.mark.parametrize("method", ["pcg", "fcg"])
@pytest.mark.parametrize("N,boxes", [(6, 2), (13, 2), (36, 3), (84, 6)])
def test_columns_beside_each_other(N, boxes, method):
    print(N, boxes, method, flush=True)
    pr = si.make_config("lap3d_64", N=N, boxes=boxes)
    slr = P.SLR(pr.csr, pr.part, pr.nparts, v0=pr.v0(), k=4, lanczos_steps=20)
    rng = np.random.Generator(np.random.PCG64(7))
    x = rng.uniform(-1, 1, (9, pr.n))
    x[3] = 0.0                                  # a column that is done at once
    b = torch.tensor(x, dtype=torch.float64, device="cuda").t()
    A = pr.scipy()
    base = {}
    for c in (2, 3, 4, 5, 8, 9):
        sol, info = slr.solve(b[:, :c], method=method, rtol=1e-8, maxit=200)
        sol = sol.cpu().numpy()
        for i in range(c):
            if i in base:
                assert np.array_equal(sol[:, i], base[i]), (c, i)
            else:
                base[i] = sol[:, i].copy()
                res = np.linalg.norm(x[i] - A @ sol[:, i])
                assert res <= 1.1e-8 * np.linalg.norm(x[i]), (c, i)
