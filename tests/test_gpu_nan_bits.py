"""A NaN of any bits in a source or a first iterate ends a batched solve with
an error, as every other NaN does."""
import numpy as np
import pytest

import sn_workloads as sw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [0x7fffffff, 0xffffffff, 0x7fff8000, 0x7fc00000])
@pytest.mark.parametrize("precision", ["f32", "bf16x3"])
@pytest.mark.parametrize("N,L", [(16, 15), (64, 63), (128, 127), (200, 3), (256, 255), (30, 29)])
def test_nan_in_source(N, L, precision, bits):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    print("nan bits", N, L, precision, hex(bits), flush=True)
    probs = [sw.random_slab(60 + K, K=K, N=N, L=L, regions=1, kernel="hg", source="random") for K in (5, 40)]
    S = snfpsa.SlabSolver(probs, fp_scheme="none", precision=precision)
    q = np.ones(S.psi_len, dtype=np.float32)
    q[-5] = np.array([bits], dtype=np.uint32).view(np.float32)[0]
    for fused in ((True, False) if S.fused_iteration()["available"] else (False,)):
        if S.fused_iteration()["available"]:
            S.set_fused_iteration(fused)
        with pytest.raises(snfpsa.SnError) as e:
            S.solve("si", tol=1e-5, max_iter=50, q_ext=torch.from_numpy(q.view(np.int32).copy()).cuda().view(torch.float32))
        assert e.value.status == -4, fused
    S.close()
