"""Slabs of a batched FP64 solve that stop iterating before the others."""
import numpy as np
import pytest

import sn_workloads as sw

pytestmark = pytest.mark.gpu


# Slabs from a fast to a slow contraction: each result within tol of the
# slab-by-slab solve at tol / 1e3 (its change is below tol / 64 and the rates
# below 0.98, so what is left is below tol / 64 * 0.98 / 0.02 < tol), the
# iteration counts those of the slab-by-slab solve, and after a limit of
# iterations that none or some slabs need, the same iterates.
@pytest.mark.parametrize("method,scheme,N", [("si", "none", 16), ("fpsa", "wfd", 16), ("fpsa", "mpd", 70), ("fpsa", "wfd", 128)])
def test_early_stop(method, scheme, N):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    probs = [sw.random_slab(40 + i, K=20 + 13 * i, N=N, regions=1, kernel="hg", source="random", c_range=(c, c + 0.01))
             for i, c in enumerate((0.05, 0.5, 0.9, 0.7, 0.3))]
    S = snfpsa.SlabSolver(probs, fp_scheme=scheme)
    q = torch.from_numpy(np.concatenate([p.q.ravel() for p in probs])).cuda()
    tol = 1e-8

    def solve(batched, tol, max_iter):
        print("early stop", method, scheme, N, batched, tol, max_iter, flush=True)
        S.set_batched_solve(batched)
        pe = torch.zeros(S.exit_len, dtype=torch.float64, device="cuda")
        r = S.solve(method, tol=tol, max_iter=max_iter, q_ext=q, psi_exit=pe)
        return r["iters"], r["phi"].cpu().numpy(), pe.cpu().numpy(), r["status"]

    its, phi, ex, status = solve(True, tol, 500)
    its1, _, _, _ = solve(False, tol, 500)
    _, ref, refx, _ = solve(False, tol / 1e3, 800)
    assert status == 0 and list(its) == list(its1) and len(set(its)) > 2
    assert np.abs(phi - ref).max() < tol and np.abs(ex - refx).max() < tol
    for cap in (3, int(sorted(its)[2])):
        itc, phic, exc, sc = solve(True, tol, cap)
        it1, phi1, ex1, s1 = solve(False, tol, cap)
        assert sc == s1 != 0 and list(itc) == list(it1)
        late = [b for b in range(len(probs)) if its[b] > cap]
        off = np.concatenate([[0], np.cumsum([2 * p.K * (p.L + 1) for p in probs])])
        for b in late:
            a, z = phic[off[b]:off[b + 1]], phi1[off[b]:off[b + 1]]
            assert np.abs(a - z).max() <= 1e-12 * np.abs(z).max()
    S.close()
