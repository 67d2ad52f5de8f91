"""The Fokker-Planck correction by the doubling tree against the FP64 oracle,
at the edges of its cut into stages, chunks, passes and column tiles."""
import numpy as np
import pytest

import oracle
import sn_workloads as sw

pytestmark = pytest.mark.gpu

# (K, N, L, regions, scheme): no level, one, a ragged last node; a pass of 16
# rows and one more; columns and moments below, at and past tiles of 16; one
# chunk at its largest, one cell past it; two and three stages; regions that
# cut passes; more than 64 angles, both sides of the eliminations' range; no
# two cells alike
CASES = [
    (1, 4, 3, 1, "wfd"), (2, 8, 7, 1, "mpd"), (5, 2, 1, 2, "wfd"), (17, 16, 15, 1, "wfd"), (33, 64, 63, 1, "wfd"),
    (128, 10, 9, 3, "mpd"), (256, 8, 7, 1, "wfd"), (257, 8, 4, 1, "mpd"), (515, 24, 15, 5, "mpd"), (130, 64, 40, 3, "wfd"),
    (1100, 6, 5, 4, "wfd"), (4097, 14, 13, 2, "wfd"), (2049, 64, 63, 3, "wfd"), (70, 66, 65, 1, "mpd"), (130, 112, 111, 1, "wfd"),
    (130, 114, 113, 3, "wfd"), (90, 128, 127, 4, "mpd"), (33, 256, 200, 2, "wfd"),
    (50, 16, 15, 50, "wfd"), (520, 64, 63, 520, "wfd"),
]


# 1e-10 of the correction, as for the eliminations: both compose the cells'
# responses in FP64 with inverses of I - R R', R below one
@pytest.mark.parametrize("case", CASES, ids=lambda c: "K%dN%dL%dR%d%s" % c)
def test_fp_tree(case):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    K, N, L, regions, scheme = case
    print("fp tree", case, flush=True)
    p = sw.random_slab(500 + K, K=K, N=N, L=L, regions=regions, kernel="hg", source="random", c_range=(0.9, 0.99))
    S = snfpsa.SlabSolver([p], fp_scheme=scheme)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64).ravel()).cuda()
    ph, po = sw.random_vectors(10 + K, K, 2, L + 1), sw.random_vectors(20 + K, K, 2, L + 1)
    out = S.fpsa_correct(dev(ph), dev(po))
    ref, _ = oracle.fpsa_correct(p, ph, po, scheme)
    got = out.cpu().numpy().reshape(ref.shape)
    assert np.abs((got - ph) - (ref - ph)).max() < 1e-10 * np.abs(ref - ph).max()
    out2 = S.fpsa_correct_noalloc(dev(ph), dev(po), S.phi_tensor())
    assert torch.equal(out, out2)
    if K <= 600:
        r = S.solve("fpsa", tol=1e-11, max_iter=500, q_ext=dev(p.q))
        ro = oracle.solve(p, "fpsa", scheme, tol=1e-11, max_iter=500)
        err = np.abs(r["phi"].cpu().numpy().reshape(ro["phi"].shape) - ro["phi"]).max() / np.abs(ro["phi"]).max()
        assert r["status"] == 0 and r["iters"][0] == ro["iters"] and err < 1e-10
    S.close()
