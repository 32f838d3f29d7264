"""Values that are not finite, sweeps of any row width: an infinite entry
reaches the rows that depend on it and no others, and stays an infinity there.

The matrix holds a piece that couples to nothing else, in the same subdomain
as the rest, so its rows share levels, chains and panels with rows that do not
depend on it.  All couplings are negative and all pivots positive: every row
of the piece that the entry reaches, and no other, comes out as +Inf, as a
solve that skips structural zeros gives it."""
import numpy as np
import pytest
import scipy.sparse as sp

import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")


def _problem(N, piece):
    """2-D Laplacian in 2 x 2 boxes and, in the first box's subdomain, pieces of their own."""
    A, part = si.laplacian_2d(N), si.box_partition_2d(N, 2, 2)
    A = sp.csr_matrix((A[2], A[1], A[0]), shape=(A[3], A[3]))
    # (a lone row first: the first row of a subdomain also pads its rows of E^T)
    M = sp.block_diag([A, sp.eye(1) * 2.0] + piece).tocsr()
    M.sort_indices()
    part = np.concatenate([part, np.zeros(M.shape[0] - N * N, dtype=part.dtype)])
    return (M.indptr.astype(np.int64), M.indices.astype(np.int32), M.data, M.shape[0]), part


def _band(n, w):
    return sp.diags([np.full(n - abs(o), -1.0 if o else 2.0 * w + 1.0) for o in range(-w, w + 1)],
                    list(range(-w, w + 1)))


def _star(n):
    """rows that depend on the first one only: one wide level"""
    S = sp.lil_matrix((n, n))
    S.setdiag(float(n))
    S[0, 1:] = S[1:, 0] = -1.0
    return S


CASES = {
    "diagonal": [sp.eye(70) * 2.0],            # rows without entries
    "band1": [_band(40, 1)],                   # rows of one entry: padded to two
    "band7": [_band(90, 7)],                   # a chain and panels beside the box's own
    "star": [_star(80)],                       # a row of 79 entries backwards: lanes that share a row
    "mixed": [sp.eye(9) * 2.0, _band(33, 3), _star(20)],
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("bf,bo", [("chol", "natural"), ("ict", "mindeg"), ("ildlt", "mindeg")])
@pytest.mark.parametrize("name", sorted(CASES))
def test_infinities_stay_where_they_belong(name, bf, bo, prec):
    print(name, bf, bo, prec, flush=True)
    A, part = _problem(20, CASES[name])
    n, base = A[3], 401
    slr = P.SLR(A, part, 4, k=4, lanczos_steps=20, b_fact=bf, b_order=bo, c_fact="chol", droptol=0.0,
                fact_prec=prec, uk_prec=prec)
    assert slr.forms()["b_slots"] > 0
    M = sp.csr_matrix((A[2], A[1], A[0]), shape=(n, n))
    _, comp = sp.csgraph.connected_components(M)
    r = torch.tensor(np.random.default_rng(5).uniform(0.5, 1.0, n), dtype=torch.float64, device="cuda")
    clean = slr.apply(r)
    assert bool(torch.isfinite(clean).all())
    for at in (base, base + (n - base) // 2, n - 1):
        bad = r.clone()
        bad[at] = float("inf")
        hit = torch.tensor(comp == comp[at], device="cuda")
        for nrhs in (1, 5):
            z = slr.apply(bad if nrhs == 1 else torch.stack([r, bad, r, bad, r], 1))
            z = z if nrhs == 1 else z[:, 3]
            assert bool((z[hit] == float("inf")).all()), (at, nrhs)
            assert torch.equal(z[~hit], clean[~hit]), (at, nrhs)
    assert torch.equal(slr.apply(r), clean)
