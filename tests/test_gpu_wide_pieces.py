"""The 256-wide class GEMMs in BF16 pieces against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import sn_workloads as sw

pytestmark = pytest.mark.gpu

# slabs of one class (N, L): a single cell, one below, at and past a 32-row
# unit and a 64-row tile, and one of several; angle and moment counts at both
# ends of the width, moments far fewer than angles
CASES = [(132, 131), (256, 255), (200, 3), (252, 127)]


# 2e-5 as the FP32 solves' other tests: FP32 sweeps, sources and moments
@pytest.mark.parametrize("qext", ["random", "none"])
@pytest.mark.parametrize("N,L", CASES)
def test_wide_class(N, L, qext):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    print("wide class", N, L, qext, flush=True)
    probs = [sw.random_slab(900 + K, K=K, N=N, L=L, regions=min(3, K), kernel="hg", source="random",
                            c_range=(0.2 + 0.05 * i, 0.25 + 0.05 * i)) for i, K in enumerate((1, 15, 16, 17, 32, 33, 200))]
    S = snfpsa.SlabSolver(probs, fp_scheme="none", precision="f32")
    q = None
    if qext == "random":
        q = torch.from_numpy(np.concatenate([p.q.ravel() for p in probs]).astype(np.float32)).cuda()
    ref = [oracle.solve(p, "si", tol=1e-12, q_ext="problem" if qext == "random" else None) for p in probs]
    scale = max(float(np.abs(r["phi"]).max()) for r in ref)
    r = S.solve("si", tol=1e-6 * scale, max_iter=500, q_ext=q)
    assert r["status"] == 0 and len(set(r["iters"])) > 1
    phi, off = r["phi"].cpu().numpy(), 0
    for p, z in zip(probs, ref):
        n = 2 * p.K * (p.L + 1)
        e = np.abs(phi[off:off + n] - z["phi"].ravel()).max() / np.abs(z["phi"]).max()
        print(p.K, "rel err %.2e" % e)
        assert e < 2e-5
        off += n
    S.close()
