"""Source iteration in one launch an iteration against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import sn_workloads as sw

pytestmark = pytest.mark.gpu

# (K, N, L, regions): one cell and a ragged last tile; fewer moment
# columns than angles, angles below and at a padded width; the largest number of
# tiles that takes one launch and one more
CASES = [(1, 8, 7, 1), (37, 8, 3, 3), (130, 10, 9, 2), (515, 16, 15, 4), (257, 16, 1, 2), (300, 34, 33, 2),
         (97, 48, 10, 3), (515, 64, 63, 5), (4096, 16, 15, 2), (4097, 16, 15, 2)]


# 1e-11 of the moments: both sides iterate in FP64 from the same start, and a
# contraction does not amplify rounding (1e-16) a hundred thousand times
@pytest.mark.parametrize("source", ["random", "none"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "K%dN%dL%dR%d" % c)
def test_si_step(case, source):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    K, N, L, regions = case
    p = sw.random_slab(700 + K, K=K, N=N, L=L, regions=regions, kernel="hg", source="random", c_range=(0.3, 0.6))
    if source == "none":
        p.q[...] = 0.0
    S = snfpsa.SlabSolver([p])
    q = None if source == "none" else torch.from_numpy(np.ascontiguousarray(p.q).ravel()).cuda()
    for cap in (1, 2, 200):  # both iterate buffers, and to convergence
        print("si step", case, source, cap, flush=True)
        pe = torch.zeros(N, dtype=torch.float64, device="cuda")
        r = S.solve("si", tol=1e-9, max_iter=cap, q_ext=q, psi_exit=pe)
        ro = oracle.solve(p, "si", tol=1e-9, max_iter=cap)
        err = np.abs(r["phi"].cpu().numpy().reshape(ro["phi"].shape) - ro["phi"]).max()
        assert r["iters"][0] == ro["iters"] and err <= 1e-11 * np.abs(ro["phi"]).max()
        ex = np.concatenate([ro["psi"][0, 0, : N // 2], ro["psi"][-1, 1, N // 2:]])
        assert np.abs(pe.cpu().numpy() - ex).max() <= 1e-11 * np.abs(ex).max()
    S.close()
