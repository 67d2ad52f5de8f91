"""What a batched FP64 solve returns: every slab iterated as often as the
slowest, whatever passed its test before."""
import numpy as np
import pytest

import sn_workloads as sw

pytestmark = pytest.mark.gpu


def slabs(N, K, shared):
    """Slabs from a fast to a slow contraction; shared: of equal sizes, widths
    and mean coefficients (one factorisation), the moments past the first
    those of the kernel or none."""
    if not shared:
        return [sw.random_slab(40 + i, K=K + 13 * i, N=N, regions=1, kernel="hg", source="random", c_range=(c, c + 0.01))
                for i, c in enumerate((0.05, 0.5, 0.95, 0.7, 0.3))]
    out = []
    for i, keep in enumerate((2, N, 3, N // 2)):
        p = sw.random_slab(90 + i, K=K, N=N, regions=1, kernel="hg", source="random")
        p.sigma_t = np.ones(K)
        p.sigma_s = np.tile(0.99 * 0.93 ** np.arange(N), (K, 1))
        p.sigma_s[:, keep:] = 0.0
        out.append(p)
    return out


# The reference of a slab: the slab-by-slab solve run for as many iterations
# as the slowest slab needed.  The batched result is no further from the
# converged moments (more iterations of a contraction; 1e-12 of the largest
# moment for rounding).  The last two cases run the eliminations, the second
# of them with factors that the slabs share.
@pytest.mark.parametrize("method,scheme,coef,N,K,shared", [
    ("si", "none", "cell", 16, 20, False), ("fpsa", "wfd", "cell", 16, 20, False), ("fpsa", "mpd", "mean", 64, 90, True),
    ("fpsa", "wfd", "cell", 116, 70, False), ("fpsa", "wfd", "mean", 116, 80, True)])
def test_as_far_as_the_slowest(method, scheme, coef, N, K, shared):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    probs = slabs(N, K, shared)
    S = snfpsa.SlabSolver(probs, fp_scheme=scheme, fp_coefficients=coef)
    q = torch.from_numpy(np.concatenate([p.q.ravel() for p in probs])).cuda()

    def solve(batched, tol, max_iter):
        print("converged", method, scheme, coef, N, batched, tol, max_iter, flush=True)
        S.set_batched_solve(batched)
        pe = torch.zeros(S.exit_len, dtype=torch.float64, device="cuda")
        r = S.solve(method, tol=tol, max_iter=max_iter, q_ext=q, psi_exit=pe, history=True)
        return r["iters"], r["phi"].cpu().numpy(), pe.cpu().numpy(), r["hist"]

    tol = 1e-6
    its, phi, ex, hist = solve(True, tol, 300)
    its1, _, _, hist1 = solve(False, tol, 300)
    assert list(its) == list(its1) and max(its) > min(its) + 1 and max(its) < 300
    _, full, fullx, _ = solve(False, 1e-13, 600)
    _, ref, refx, _ = solve(False, 0.0, int(max(its)))
    off = offx = 0
    for b, p in enumerate(probs):
        n = its[b]
        assert np.abs(hist[b][:n] - hist1[b][:n]).max() <= 1e-11 * np.abs(hist1[b][:n]).max()
        m = 2 * p.K * (p.L + 1)
        for a, r, z in ((phi[off:off + m], ref[off:off + m], full[off:off + m]),
                        (ex[offx:offx + N], refx[offx:offx + N], fullx[offx:offx + N])):
            e, e1, scale = np.abs(a - z).max(), np.abs(r - z).max(), np.abs(z).max()
            print(b, n, "off by %.2e, slab by slab %.2e" % (e, e1))
            assert e <= e1 + 1e-12 * scale
        off += m
        offx += N
    S.close()
