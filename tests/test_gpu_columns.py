"""Column counts around the fill of the compute units: the B solves split the
columns over workgroups by it.  A column's bits do not depend on the columns beside it; FP64 <= 1e-12
relative per column against the oracle on the same stored data."""
import numpy as np
import pytest

import oracle as O
import slr_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
P = pytest.importorskip("paper_1505_04340_amd")


@pytest.mark.parametrize("boxes,fact", [(2, "ic0"), (4, "ic0"), (7, "ic0"), (4, "chol")])
def test_columns_around_the_fill(boxes, fact):
    N = 2 * boxes + 5 if boxes < 7 else 22   # uneven boxes
    print(N, boxes, fact, flush=True)
    pr = si.make_config("lap3d_64", N=N, boxes=boxes)
    slr = P.SLR(pr.csr, pr.part, pr.nparts, v0=pr.v0(), k=4, lanczos_steps=20, b_fact=fact)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    edge = max(1, cu // pr.nparts)
    most = min(3 * edge + 1, 130)
    r = np.random.Generator(np.random.PCG64(3)).uniform(-1, 1, (most, pr.n))
    t = torch.tensor(r, dtype=torch.float64, device="cuda").t()
    alone = torch.stack([slr.apply(t[:, i].contiguous()) for i in range(most)], 1)
    ex = slr.export()
    ref = O.setup(pr.scipy(), pr.part, pr.nparts, slr.info["k"], b_fact=fact,
                  lowrank=(ex["U"], ex["lambda"], ex["theta"]))
    for i in (0, most - 1):
        z = ref.apply(r[i])
        assert np.linalg.norm(alone[:, i].cpu().numpy() - z) <= 1e-12 * np.linalg.norm(z)
    for c in sorted({2, edge - 1, edge, edge + 1, 2 * edge + 1, most}):
        if 1 < c <= most:
            assert torch.equal(slr.apply(t[:, :c]), alone[:, :c]), c
