"""Refactorisation by blocks: levels wider than a workgroup's threads, blocks
of few rows, minimum degree orders, and patterns whose rows subtract products
(level by level as before).  The apply equals that of a fresh refactorable
setup with the new values bit for bit (a setup that is not refactorable may
solve a deep interface schedule by blocks, in another order of summation)."""
import numpy as np
import pytest
import scipy.sparse as sp

import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")


def _values(A, seed):
    """A's pattern with new symmetric values, diagonally dominant"""
    n = A[3]
    M = sp.csr_matrix((A[2], A[1], A[0]), shape=(n, n))
    rng = np.random.default_rng(seed)
    d = rng.uniform(0.5, 1.5, n)
    M = (sp.diags(d) @ M @ sp.diags(d)).tocsr()
    M = ((M + M.T) * 0.5).tocsr()
    M.sort_indices()
    return M.indptr.astype(A[0].dtype), M.indices.astype(A[1].dtype), M.data, n


@pytest.mark.parametrize("b_fact", ["ic0", "ildlt0"])
@pytest.mark.parametrize("name,over,order", [
    ("lap3d_64", dict(N=6, boxes=2), "natural"),       # a level or two of one row
    ("lap3d_64", dict(N=42, boxes=2), "natural"),      # levels of more than 256 rows
    ("lap3d_64", dict(N=26, boxes=2), "mindeg"),
    ("lap2d_64", dict(N=40), "natural"),
    ("nine", dict(N=33), "natural"),                   # products: level by level
])
def test_blocks_equal_a_fresh_setup(name, over, order, b_fact):
    print(name, over, order, b_fact, flush=True)
    if name == "nine":
        N = over["N"]
        L = sp.diags([np.ones(N - 1), 3.0 * np.ones(N), np.ones(N - 1)], [-1, 0, 1])
        M = (10.0 * sp.eye(N * N) - sp.kron(L, L) * 0.5 + 3.0 * sp.eye(N * N)).tocsr()
        M.sort_indices()
        A = (M.indptr.astype(np.int64), M.indices.astype(np.int32), M.data, N * N)
        g = np.arange(N * N)
        part, p = ((g // N >= N // 2) * 2 + (g % N >= N // 2)).astype(np.int32), 4
    else:
        pr = si.make_config(name, **over)
        A, part, p = pr.csr, pr.part, pr.nparts
    kw = dict(b_fact=b_fact, b_order=order, c_fact="ic0")
    G = P.SLR(A, part, p, k=4, lanczos_steps=20, refactor=True, **kw)
    ex = G.export()
    r = torch.tensor(np.random.default_rng(5).uniform(-1, 1, (A[3], 2)), dtype=torch.float64, device="cuda")
    for seed in (1, 2):
        A2 = _values(A, seed)
        G.refactor(A2)
        F = P.SLR(A2, part, p, lowrank=(ex["U"], ex["lambda"], ex["theta"]), refactor=True, **kw)
        assert torch.equal(G.apply(r), F.apply(r))
