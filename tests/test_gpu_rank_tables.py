"""The bin-wide dead-pair test from rank tables of the row tile (private-tile
launches of at most 16 features, one path per wave) against Algorithm 1, on batches
of so many rows that every workgroup takes a whole group's bins: the largest and a
small feature count, paths within one scan of four and of five steps, several
groups, bins dead for a whole tile, ties and ragged rows; and the same models just
below the rule, where the per-path test finds the dead pairs."""
import numpy as np
import pytest

from paper_2010_13972_amd import gts, synth
from parity import assert_parity
from test_gpu_shap import spine_tree

pytestmark = pytest.mark.gpu

ROWS = 64 * 4096 - 29   # 4096 row tiles, the last ragged: one slice


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def has_tables(cfg, other, M):
    """Whether a launch holds the tables that the other one, the same but for them, lacks."""
    return cfg["lds_bytes"] - other["lds_bytes"] >= M * 65 * 12


def check(torch, orc, ens, X, dtype, what):
    model = gts.prepare(ens, dtype)
    M = ens.num_features
    few = gts.launch_config(model, 70)
    many = gts.launch_config(model, ROWS)
    print(what, dtype, "bins", model.desc.num_bins, many, flush=True)
    for cfg in (few, many):
        assert cfg["rows_per_tile"] == 64 and cfg["private_tiles"] == 1
    assert has_tables(many, few, M)
    got = gts.shap(model, torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    sel = np.unique(np.concatenate([np.arange(150), np.arange(ROWS - 70, ROWS),
                                    np.random.default_rng(1).integers(0, ROWS, 150)]))
    want = orc.treeshap(ens, X[sel])
    assert_parity(got[sel], want, dtype, what=f"{what}, tables")
    # the first rows alone: without tables
    got = gts.shap(model, torch.from_numpy(X[:70]).cuda()).cpu().numpy().astype(np.float64)
    assert_parity(got, want[:70], dtype, what=f"{what}, no tables")
    return got


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("M,groups,trees", [(16, 1, 60), (16, 3, 180), (4, 1, 20)])
def test_zero_covers_and_ties(torch, orc, M, groups, trees, dtype):
    w = synth.random_workload(70 + M, num_trees=trees, max_depth=7, M=M, num_groups=groups,
                              n_bg=30, rows=1)
    X = np.random.default_rng(M).integers(0, 4, size=(ROWS, M)).astype(np.float32)
    check(torch, orc, w.ensemble, X, dtype, f"M={M} G={groups}")


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("longest", [12, 16])
def test_long_paths(torch, orc, longest, dtype):
    """Zero-fraction elements anywhere on paths of up to 12 and of 16 features."""
    rng = np.random.default_rng(longest)
    trees = []
    for t in range(90):
        n = longest - 3 + t % 4
        zero = set(rng.choice(n, size=1 + t % 4, replace=False).tolist())
        trees.append(spine_tree(rng.permutation(16)[:n], rng, zero))
    ens = synth.ensemble_from_lists(trees, M=16)
    X = rng.random((ROWS, 16), dtype=np.float32)
    check(torch, orc, ens, X, dtype, f"longest {longest}")


def test_bins_dead_for_a_tile(torch, orc):
    """Right subtrees of zero cover that rows with x0 < 0.5 do not reach: their longer
    paths fill bins of their own, dead for all but the last tiles."""
    rng = np.random.default_rng(7)
    trees = []
    for t in range(600):
        f1 = 1 + t % 7
        trees.append([(1, 2, 0, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 10.0, float(rng.normal())),
                      (3, 4, f1, 0.25 + 0.5 * rng.random(), 0.0, 0.0),
                      (-1, -1, -1, 0, 0.0, float(rng.normal())),
                      (-1, -1, -1, 0, 0.0, float(rng.normal()))])
    ens = synth.ensemble_from_lists(trees, M=8)
    X = rng.random((ROWS, 8), dtype=np.float32) * np.float32(0.5)
    X[-100:, 0] += np.float32(0.5)
    for dtype in ("f32", "f64"):
        got = check(torch, orc, ens, X, dtype, "dead bins")
        assert np.all(got[:, 0, 1:8] == 0.0)
