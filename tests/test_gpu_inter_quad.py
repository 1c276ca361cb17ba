"""Interaction values of models whose longest path holds 9 to 16 features (the
quadrature kernel), against the oracle's conditioning route: chains at every
path length around its padded variants, and one model per tile shape, with
shorter paths, zero covers, ties, several groups, ragged rows, a pruned model
and rows that are not finite."""
import numpy as np
import pytest

from paper_2010_13972_amd import gts, synth
from parity import assert_parity
from test_gpu_shap import chain_tree

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def run(torch, model, X):
    out = gts.shap_interactions(model, torch.from_numpy(np.ascontiguousarray(X)).cuda())
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("depth", [9, 10, 11, 13, 15, 16])
def test_chains(torch, orc, depth, dtype):
    """The chain's leaves give paths of every length from 1 to depth."""
    rng = np.random.default_rng(depth)
    ens = synth.ensemble_from_lists([chain_tree(depth, 16, rng), chain_tree(9, 16, rng)], M=16)
    X = rng.random((19, 16)).astype(np.float32)
    print("chain", depth, dtype, flush=True)
    got = run(torch, gts.prepare(ens, dtype), X)
    assert_parity(got, orc.interactions(ens, X), dtype, 2, what=f"chain {depth}")


# (M, dtype, rows per tile and waves of the launch): in fp32 tiles of 16, 8 and 4 rows
# in double, then of 8 and 4 rows in float
SHAPES = [(12, "f32", 16, 16), (50, "f32", 8, 16), (70, "f32", 4, 16), (80, "f32", 8, 12),
          (110, "f32", 4, 16), (116, "f32", 4, 8),
          (20, "f64", 16, 8), (50, "f64", 8, 8), (75, "f64", 4, 8)]


@pytest.mark.parametrize("M,dtype,rw,waves", SHAPES)
def test_tile_shapes(torch, orc, M, dtype, rw, waves):
    w = synth.random_workload(900 + M, num_trees=9, max_depth=16, p_split=0.75, M=M, num_groups=3,
                              n_bg=60, rows=37, max_leaves=200)
    print("shape", M, dtype, rw, flush=True)
    model = gts.prepare(w.ensemble, dtype)
    assert 9 <= model.desc.max_path_len - 1 <= 16
    cfg = gts.launch_config(model, 37, interactions=True)
    assert (cfg["rows_per_tile"], cfg["waves"]) == (rw, waves)
    want = orc.interactions(w.ensemble, w.X)
    assert_parity(run(torch, model, w.X), want, dtype, 2, what=f"M={M}")
    X = torch.from_numpy(w.X).cuda()
    pruned = gts.shap_interactions(gts.prune(model, X), X)
    assert_parity(pruned.cpu().numpy().astype(np.float64), want, dtype, 2, what=f"pruned M={M}")


@pytest.mark.parametrize("M", [12, 30, 50, 56, 70, 77, 80, 110, 116])
def test_no_further_from_fp64_than_the_runtime_length_code(torch, orc, M):
    """The runtime-length code takes a path of 9 features and more in fp64 and rounds
    once for each addition to a float tile.  Here the same blob runs through it when
    the descriptor states a longest path beyond the quadrature's; the quadrature's
    distance from the oracle is no larger."""
    w = synth.random_workload(900 + M, num_trees=30, max_depth=16, p_split=0.85, M=M, num_groups=1,
                              n_bg=300, rows=40, max_leaves=150)
    model = gts.prepare(w.ensemble, "f32")
    assert 9 <= model.desc.max_path_len - 1 <= 16
    want = orc.interactions(w.ensemble, w.X)
    quad = run(torch, model, w.X)
    model.desc.max_path_len = 18
    general = run(torch, model, w.X)
    errs = [float(np.linalg.norm(x - want) / np.linalg.norm(want)) for x in (quad, general)]
    print("distance", M, errs, flush=True)
    assert not np.array_equal(quad, general)
    assert errs[0] <= errs[1]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("rows", [40, 100, 300])
def test_slices_of_one_round(torch, rows, dtype):
    """A CU's registers hold one workgroup: the slices of a model with bins enough come
    to one workgroup for each CU at most."""
    w = synth.random_workload(12, num_trees=60, max_depth=14, p_split=0.9, M=12, n_bg=500, rows=1,
                              max_leaves=256)
    model = gts.prepare(w.ensemble, dtype)
    assert 9 <= model.desc.max_path_len - 1 <= 16
    cfg = gts.launch_config(model, rows, interactions=True)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert model.desc.num_bins // cfg["waves"] * (-(-rows // 16)) > cus   # bins for more
    assert cus // 2 < cfg["workgroups"] <= cus


def test_a_value_that_is_not_finite_is_in_no_range(torch):
    """NaN and +inf fail every element's range test: a row of either gives what
    the other gives, finite everywhere, and the rows beside it are unchanged."""
    w = synth.random_workload(77, num_trees=6, max_depth=15, p_split=0.8, M=14, n_bg=60, rows=18,
                              max_leaves=150)
    model = gts.prepare(w.ensemble, "f64")
    assert 9 <= model.desc.max_path_len - 1 <= 16
    base = run(torch, model, w.X)
    outs = []
    for bad in (np.nan, np.inf):
        X = w.X.copy()
        X[5, 3] = bad
        outs.append(run(torch, model, X))
    assert np.isfinite(outs[0]).all()
    np.testing.assert_allclose(outs[0], outs[1], rtol=0, atol=1e-12)
    keep = np.arange(18) != 5
    np.testing.assert_allclose(outs[0][keep], base[keep], rtol=0, atol=1e-12)
