"""The benchmark's roofline line names the kernel that takes the most time
(CPU only)."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)

import bench  # noqa: E402
import sn_workloads as sw  # noqa: E402

snfpsa = pytest.importorskip("paper_1907_13013_amd")

# launches and total ms of one solve of the workload, by kernel
TIMING = {"sweep_aggregate": (22, 0.271), "sweep_apply": (22, 0.274), "fp_tree_up": (22, 0.193), "fp_tree_mid": (66, 0.746),
          "fp_tree_update": (22, 0.289), "krylov": (0, 0.0), "exit_flux": (1, 0.002)}


def test_dominant_kernel_of_the_workload():
    p = sw.srk_slab_2000()
    stages = snfpsa.diag_fp_tree(p.K, p.N, p.L, p.h, p.sigma_t, p.sigma_s)
    assert len(stages) == 3 and stages[0]["n"] == p.K and stages[-1]["chunks"] == 1
    per_iter = bench.algorithmic_bytes_per_iteration(p.K, p.N, p.L + 1, stages)
    # every launch of an iteration is in the model, as often as it runs
    for name, (n, _) in TIMING.items():
        if n >= 22:
            assert per_iter[name][1] * 22 == n, name
    kernels, dom = bench.rooflines(TIMING, per_iter)
    assert dom == "fp_tree_mid" == kernels[dom]["kernel"] and set(kernels) == set(per_iter)
    assert kernels[dom]["algorithmic_bytes_per_launch"] * 3 == 8 * p.N * (
        4 * (stages[1]["n"] + 1) + 2 * (stages[2]["n"] + 1))
    assert bench.rooflines({**TIMING, "sweep_apply": (22, 2.0)}, per_iter)[1] == "sweep_apply"


def test_tree_stages_and_eliminations():
    p = sw.random_slab(3, K=240, N=128, L=5, regions=1, kernel="hg")
    assert snfpsa.diag_fp_tree(p.K, p.N, p.L, p.h, p.sigma_t, p.sigma_s) == []
    p = sw.random_slab(3, K=515, N=24, L=5, regions=5, kernel="hg")
    one = snfpsa.diag_fp_tree(p.K, p.N, p.L, p.h, p.sigma_t, p.sigma_s)
    for a, b in zip(one, one[1:]):
        assert b["n"] == a["chunks"] == -(-a["n"] // a["c"]) and a["c"] == 1 << a["levels"] and a["classes"] > 0
