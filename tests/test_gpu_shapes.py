"""Shared-tile launch shapes of SHAP values around the planner's lines, each against
Algorithm 1 on a ragged row count, with the rows and waves the planner gives."""
import numpy as np
import pytest

from paper_2010_13972_amd import gts, synth
from parity import assert_parity
from test_gpu_shap import chain_tree

pytestmark = pytest.mark.gpu

# (features, dtype, longest path, rows per tile, waves)
SHAPES = [
    # 64 rows in double: two workgroups of 12 or 8 waves a CU, one of 16
    (80, "f32", 8, 64, 12), (81, "f32", 8, 64, 8), (95, "f32", 8, 64, 16), (102, "f32", 8, 64, 16),
    (103, "f32", 8, 32, 8), (81, "f32", 11, 64, 8), (95, "f32", 11, 64, 16),
    (102, "f32", 16, 64, 16), (102, "f32", 20, 32, 8), (103, "f32", 11, 32, 8),
    # 32 rows: the same
    (166, "f32", 11, 32, 8), (167, "f32", 11, 32, 16), (186, "f32", 16, 32, 16),
    (186, "f32", 20, 16, 16),
    # 16 rows: the same, beyond 12 features
    (333, "f32", 13, 16, 16), (334, "f32", 13, 16, 16), (373, "f32", 20, 16, 16),
    (334, "f32", 12, 8, 16), (374, "f32", 13, 8, 16),
    # 8 rows: 16 and 12 waves in double, then in float
    (1337, "f32", 11, 8, 16), (1338, "f32", 11, 8, 12), (1429, "f32", 16, 8, 12),
    (1430, "f32", 16, 8, 16),
    (2007, "f32", 20, 8, 16), (2008, "f32", 11, 8, 12),
    # short paths: 12 waves twice a CU, on 16 and 8 rows in double, then in float
    (167, "f32", 8, 16, 12), (287, "f32", 8, 16, 12), (288, "f32", 8, 8, 12),
    (373, "f32", 8, 8, 12), (576, "f32", 8, 8, 12), (577, "f32", 8, 8, 12),
    (1000, "f32", 8, 8, 16), (1100, "f32", 8, 8, 16),
    # fp64: 8 waves on 64 and 32 rows
    (40, "f64", 8, 64, 8), (68, "f64", 8, 64, 8), (69, "f64", 8, 32, 8), (81, "f64", 9, 64, 8),
    (82, "f64", 9, 32, 8), (142, "f64", 12, 32, 8),
    (160, "f64", 8, 16, 16), (300, "f64", 8, 8, 16), (635, "f64", 8, 8, 16),
    # fp64: 16 waves to 10 features, then 12, whose registers hold a path
    (160, "f64", 9, 16, 16), (300, "f64", 10, 8, 16), (160, "f64", 11, 16, 12),
    (285, "f64", 12, 16, 12), (300, "f64", 12, 8, 12),
    (635, "f64", 16, 8, 12), (784, "f64", 20, 8, 12), (1300, "f64", 12, 8, 8),
    (1500, "f64", 16, 4, 12),
]


@pytest.mark.parametrize("M,dtype,q,rows,waves", SHAPES)
def test_shape(orc, M, dtype, q, rows, waves):
    import torch
    rng = np.random.default_rng(M + q)
    m = min(M, 63)
    ens = synth.ensemble_from_lists([chain_tree(q, m, rng), chain_tree(max(1, q - 3), m, rng)], M=M)
    X = rng.random((71, M)).astype(np.float32)
    model = gts.prepare(ens, dtype)
    assert model.desc.max_path_len == q + 1
    cfg = gts.launch_config(model, 71)
    print("shape", M, dtype, q, cfg, flush=True)
    assert (cfg["rows_per_tile"], cfg["waves"], cfg["private_tiles"]) == (rows, waves, 0)
    got = gts.shap(model, torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    assert_parity(got, orc.treeshap(ens, X), dtype, what=f"M={M} {dtype} {q} features")


# (trees, depth, groups, rows): more bins than a workgroup's 4 waves in a group
FEW = [(4, 5, 1, 13), (10, 7, 10, 9), (16, 7, 10, 47)]


@pytest.mark.parametrize("trees,depth,groups,rows", FEW)
def test_no_wave_takes_two_of_few_bins(orc, trees, depth, groups, rows):
    """Slices enough that no wave has a second bin, also in a group of twice the mean."""
    import torch
    w = synth.random_workload(trees, num_trees=trees, max_depth=depth, p_split=0.85, M=20,
                              num_groups=groups, n_bg=200, rows=rows)
    model = gts.prepare(w.ensemble, "f32")
    cfg = gts.launch_config(model, rows)
    mean = model.desc.num_bins / groups
    print("few bins", trees, groups, model.desc.num_bins, cfg, flush=True)
    assert cfg["private_tiles"] == 1 and cfg["waves"] == 4 and mean > 4
    assert cfg["slices"] * 4 >= (mean if groups == 1 else 2 * int(mean))
    got = gts.shap(model, torch.from_numpy(w.X).cuda()).cpu().numpy().astype(np.float64)
    assert_parity(got, orc.treeshap(w.ensemble, w.X), "f32", what=f"{trees} trees")
