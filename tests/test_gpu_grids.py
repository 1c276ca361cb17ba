"""Launches of more than 2^32 work-items in all, which a grid holds in several rows:
more than 2^26 rows in the interaction kernel's largest workgroups (1024 threads
for 16 rows) and more than 2^26 trees in device extraction (256 threads a tree, a
wave a tree for the sums)."""
import numpy as np
import pytest

from paper_2010_13972_amd import gts, synth
from test_gpu_shap import chain_tree, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def test_interactions_of_many_rows(torch):
    """64 rows repeated 2^20 + 1 times: every block holds what the first does, up to
    the order in which waves add to a tile (about 10 paths, each sum of at most 10
    terms of the block's magnitude, rounded to 2^-24)."""
    rng = np.random.default_rng(9)
    model = gts.prepare(synth.ensemble_from_lists([chain_tree(9, 9, rng)], M=9), "f32")
    blocks = (1 << 20) + 1
    rows = 64 * blocks
    cfg = gts.launch_config(model, rows, interactions=True)
    say("many rows", rows, cfg)
    assert cfg["workgroups"] * cfg["waves"] * 64 >= 1 << 32
    base = torch.from_numpy(rng.random((64, 9)).astype(np.float32)).cuda()
    want = gts.shap_interactions(model, base).double()
    assert float(want.abs().max()) > 0
    out = gts.shap_interactions(model, base.repeat(blocks, 1)).view(blocks, 64, 10, 10)
    bound = 10 * 2.0 ** -24 * float(want.abs().max()) * 10
    first = want.float().view(1, 64, 10, 10)
    step = 1 << 16
    for a in range(0, blocks, step):
        assert float((out[a:a + step] - first).abs().max()) <= bound


def test_extraction_of_many_trees(torch):
    """2^26 + 5 trees of one leaf each: one root element per tree, and the bias is
    the sum of the leaf values (small integers, so exact in any order)."""
    T = (1 << 26) + 5
    i = torch.arange(T, device="cuda")
    value = ((i % 7) - 3).double()
    none = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    d = gts.DeviceEnsemble.__new__(gts.DeviceEnsemble)
    d.tensors = {"off": torch.arange(T + 1, device="cuda"), "left": none, "right": none,
                 "feat": none, "group": torch.zeros(T, dtype=torch.int32, device="cuda"),
                 "thr": torch.zeros(T, device="cuda"), "value": value,
                 "cover": torch.ones(T, dtype=torch.float64, device="cuda")}
    t = d.tensors
    d.num_trees = d.num_nodes = T
    d.num_groups = 1
    d.struct = gts._Ensemble(1, 1, T, T, *(t[k].data_ptr() for k in (
        "off", "group", "left", "right", "feat", "thr", "cover", "value")))
    say("many trees", T)
    raw, paths, bias = gts.extract_paths_device(d)
    assert paths == T and raw.numel() == 40 * T
    assert bias.cpu().tolist() == [float(value.sum())]
    el = raw.view(torch.int32).view(T, 10)
    assert bool((raw.view(torch.int64).view(T, 5)[:, 0] == i).all())        # path_idx
    assert bool((el[:, 2] == -1).all()) and bool((el[:, 3] == 0).all())     # feature, group
    assert bool((raw.view(torch.float64).view(T, 5)[:, 4] == value).all())  # v
