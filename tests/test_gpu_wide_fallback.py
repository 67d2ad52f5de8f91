"""The 256-wide classes of batched handles where the kernels in BF16 pieces
cannot be held: the kernels that stand in for them against the FP64 oracle."""
import copy

import numpy as np
import pytest

import oracle
import sn_workloads as sw

pytestmark = pytest.mark.gpu


# A solve with another source goes first, so that a source left where it was
# would be that solve's.  2e-5 (split-BF16 source 1e-4) of the largest moment,
# as the other solves of these precisions.
@pytest.mark.parametrize("precision,bound", [("f32", 2e-5), ("bf16x3", 1e-4)])
@pytest.mark.parametrize("graphs", [True, False])
@pytest.mark.parametrize("N,L", [(132, 131), (256, 255), (200, 3)])
def test_without_pieces(N, L, graphs, precision, bound):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    print("wide class without pieces", N, L, graphs, precision, flush=True)
    probs = [sw.random_slab(700 + K, K=K, N=N, L=L, regions=min(3, K), kernel="hg", source="random",
                            c_range=(0.3, 0.35)) for K in (1, 17, 33, 70)]
    S = snfpsa.SlabSolver(probs, fp_scheme="none", precision=precision)
    S.set_graph_replay(graphs)
    q = torch.from_numpy(np.concatenate([p.q.ravel() for p in probs]).astype(np.float32)).cuda()
    for pieces, factor in ((1, 1.0), (0, -2.0), (1, 0.5)):
        snfpsa._check(snfpsa.load_library().sn_diag_set_piece_gemms(S.handle, pieces))
        shifted = []
        for p in probs:
            p = copy.copy(p)
            p.q = factor * p.q
            shifted.append(p)
        ref = [oracle.solve(p, "si", tol=1e-12) for p in shifted]
        scale = max(float(np.abs(r["phi"]).max()) for r in ref)
        r = S.solve("si", tol=1e-6 * scale, max_iter=500, q_ext=factor * q)
        assert r["status"] == 0
        phi, off = r["phi"].cpu().numpy(), 0
        for p, z in zip(probs, ref):
            n = 2 * p.K * (p.L + 1)
            e = np.abs(phi[off:off + n] - z["phi"].ravel()).max() / np.abs(z["phi"]).max()
            print(pieces, p.K, "rel err %.2e" % e)
            assert e < bound
            off += n
    S.close()
