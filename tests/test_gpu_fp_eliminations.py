"""The Fokker-Planck correction by the eliminations' kernels, in the sizes that
keep them and at the edges of those, against the FP64 oracle."""
import copy

import numpy as np
import pytest

import oracle
import sn_workloads as sw

pytestmark = pytest.mark.gpu


def _gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1907_13013_amd as snfpsa
    return torch, snfpsa


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64).ravel()).cuda()


def _ran(S, call):
    S.set_kernel_timing(True)
    r = call()
    names = {k for k, v in S.kernel_timing().items() if v[0]}
    S.set_kernel_timing(False)
    return r, names


# (K, N, L, regions, coefficients, tree): one type with its source formed in
# the additive-term kernel, several types with a source GEMM each; widths and
# cells at the edges of the rule and one past them; half-widths that fill the
# kernels' 64 and that do not.  1e-10 of the correction.
CASES = [
    (65, 106, 105, 1, "cell", False), (65, 106, 20, 1, "mean", False), (64, 128, 30, 1, "cell", True),
    (150, 128, 127, 1, "cell", False), (97, 116, 60, 1, "mean", False), (65, 98, 97, 2, "cell", False),
    (66, 96, 95, 2, "cell", True), (120, 128, 31, 2, "cell", False), (90, 128, 127, 3, "cell", False),
    (90, 124, 50, 3, "cell", True), (90, 126, 50, 3, "mean", False), (700, 114, 9, 2, "cell", False),
    (701, 114, 9, 2, "cell", True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "K%dN%dL%dR%d%s-%s" % c)
def test_correction(case):
    torch, snfpsa = _gpu()
    K, N, L, regions, coef, tree = case
    print("eliminations", case, flush=True)
    p = sw.random_slab(800 + K, K=K, N=N, L=L, regions=1, kernel="hg", source="random", c_range=(0.9, 0.99))
    st = 1.0 + 0.4 * (np.arange(K) * regions // K)
    f = p.sigma_s[0] / p.sigma_s[0, 0]
    p.sigma_t, p.sigma_s = st, 0.97 * st[:, None] * f[None, :]
    if coef == "mean":  # the operator of the rounded means is the oracle's of such a slab
        p.sigma_t = np.ones(K)
        p.sigma_s = np.tile(np.r_[0.9, 0.9 * 0.8, 0.5 * 0.6 ** np.arange(L - 1)], (K, 1))
    S = snfpsa.SlabSolver([p], fp_scheme="wfd", fp_coefficients=coef)
    ph, po = sw.random_vectors(10 + K, K, 2, L + 1), sw.random_vectors(20 + K, K, 2, L + 1)
    out, names = _ran(S, lambda: S.fpsa_correct(_dev(torch, ph), _dev(torch, po)))
    assert any(n.startswith("fp_tree") for n in names) == tree, names
    assert ("fp_chain" in names) == (not tree), names
    ref, _ = oracle.fpsa_correct(p, ph, po, "wfd")
    got = out.cpu().numpy().reshape(ref.shape)
    err = np.abs((got - ph) - (ref - ph)).max() / np.abs(ref - ph).max()
    print("rel err %.2e" % err, sorted(names))
    assert err < 1e-10
    out2 = S.fpsa_correct_noalloc(_dev(torch, ph), _dev(torch, po), S.phi_tensor())
    assert torch.equal(out, out2)
    S.close()


# Handles of a few slabs, which keep the eliminations all or take the tree all:
# (K, N, regions) of each slab; equal ones share their cells, and with slab-mean
# coefficients one factorisation.  As many iterations as the slab-by-slab solve,
# moments within 1e-10 (slab by slab) and 1e-9 (oracle) of the largest.
HANDLES = {
    "wide": ([(80, 116, 1), (80, 116, 1), (80, 116, 1), (70, 128, 1)], False),
    "regions": ([(60, 66, 2), (90, 128, 5), (60, 66, 2)], False),
    "narrow": ([(60, 64, 4), (90, 50, 5)], False),
    "mixed": ([(80, 116, 1), (80, 116, 1), (60, 64, 4)], True),
}


@pytest.mark.parametrize("coef", ["cell", "mean"])
@pytest.mark.parametrize("name", list(HANDLES))
def test_few_slabs(name, coef):
    torch, snfpsa = _gpu()
    shapes, tree = HANDLES[name]
    if coef == "mean" and name == "narrow":
        tree = True  # one run: the coefficients are the slab's
    if coef == "mean" and name == "regions":
        tree = True
    probs = []
    for i, (K, N, regions) in enumerate(shapes):
        p = copy.deepcopy(sw.random_slab(500 + N, K=K, N=N, regions=regions, kernel="hg", source="random", c_range=(0.6, 0.9)))
        f = p.sigma_s[0] / p.sigma_s[0, 0]
        p.sigma_t = 1.0 + 0.2 * (np.arange(K) * regions // K)
        p.sigma_s = 0.8 * p.sigma_t[:, None] * f[None, :]
        p.q = np.random.default_rng(i).uniform(0.0, 2.0, size=p.q.shape)
        probs.append(p)
    S = snfpsa.SlabSolver(probs, fp_scheme="wfd", fp_coefficients=coef)
    q = torch.from_numpy(np.concatenate([p.q.ravel() for p in probs])).cuda()
    res = {}
    for batched in (True, False):
        print("few slabs", name, coef, batched, flush=True)
        S.set_batched_solve(batched)
        r, names = _ran(S, lambda: S.solve("fpsa", tol=1e-12, max_iter=2000, q_ext=q))
        assert r["status"] == 0 and ("fp_chain" in names) == (not tree) and ("fp_tree_update" in names) == tree, names
        again = S.solve("fpsa", tol=1e-12, max_iter=2000, q_ext=q)  # by replay
        assert list(again["iters"]) == list(r["iters"])
        res[batched] = (list(r["iters"]), again["phi"].cpu().numpy())
    assert res[True][0] == res[False][0]
    assert np.abs(res[True][1] - res[False][1]).max() <= 1e-10 * np.abs(res[False][1]).max()
    off = 0
    for p in probs:
        ref = oracle.solve(p, "fpsa", "wfd", tol=1e-13, max_iter=3000)["phi"].ravel()
        assert np.abs(res[True][1][off:off + ref.size] - ref).max() < 1e-9 * np.abs(ref).max(), (p.K, p.N)
        off += ref.size
    S.close()


# The path of a slab whose tree cannot be built, at every padded half-width
# (2, 4, .. 128, below and at each), one region and several, slab by slab and
# in batched launches.
@pytest.mark.parametrize("N,L,K,regions", [
    (2, 1, 30, 1), (4, 3, 41, 3), (6, 5, 25, 1), (8, 7, 64, 2), (12, 11, 33, 1), (16, 3, 50, 4), (20, 19, 40, 1),
    (32, 31, 45, 2), (50, 20, 30, 1), (64, 63, 37, 3), (80, 79, 21, 1), (128, 127, 19, 2), (130, 129, 12, 1), (256, 100, 9, 2)])
def test_every_width(N, L, K, regions, monkeypatch):
    torch, snfpsa = _gpu()
    print("eliminations, width", N, L, K, regions, flush=True)
    lib = snfpsa.load_library()
    monkeypatch.setattr(lib, "sn_setup", lib.sn_diag_setup_eliminations)
    probs = [sw.random_slab(70 + N + i, K=K + 5 * i, N=N, L=L, regions=regions, kernel="hg", source="random", c_range=(0.8, 0.95))
             for i in range(2)]
    for S, group in ((snfpsa.SlabSolver(probs[:1], fp_scheme="mpd" if N == 12 else "wfd"), probs[:1]),
                     (snfpsa.SlabSolver(probs, fp_scheme="wfd"), probs)):
        scheme = S.fp_scheme
        phs = [sw.random_vectors(10 + i, p.K, 2, L + 1) for i, p in enumerate(group)]
        pos = [sw.random_vectors(20 + i, p.K, 2, L + 1) for i, p in enumerate(group)]
        cat = lambda v: _dev(torch, np.concatenate([a.ravel() for a in v]))
        out, names = _ran(S, lambda: S.fpsa_correct(cat(phs), cat(pos)))
        assert "fp_chain" in names and not any(n.startswith("fp_tree") for n in names), names
        q = cat([p.q for p in group])
        r = S.solve("fpsa", tol=1e-11, max_iter=500, q_ext=q)
        assert r["status"] == 0
        got, phi, off = out.cpu().numpy(), r["phi"].cpu().numpy(), 0
        for p, a, b, it in zip(group, phs, pos, r["iters"]):
            ref, _ = oracle.fpsa_correct(p, a, b, scheme)
            n = ref.size
            d = got[off:off + n].reshape(ref.shape) - a
            assert np.abs(d - (ref - a)).max() < 1e-10 * np.abs(ref - a).max(), (p.K, N)
            z = oracle.solve(p, "fpsa", scheme, tol=1e-11, max_iter=500)
            assert it == z["iters"]
            assert np.abs(phi[off:off + n] - z["phi"].ravel()).max() < 1e-9 * np.abs(z["phi"]).max()
            off += n
        S.close()
