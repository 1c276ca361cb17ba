"""gts_extract_paths_device (Sections 3.1-3.2 on the GPU) against the
oracle's independent extraction (or_extract_paths) and against the host
extraction gts_extract_paths: every element field and the bias compare as raw
bytes.  Malformed ensembles, which the oracle does not validate, compare the
error status with the host call's."""
import ctypes

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


def device_extract(torch, ens):
    dens = gts.DeviceEnsemble(ens)
    raw, npaths, bias = gts.extract_paths_device(dens)
    torch.cuda.synchronize()
    return gts.elements_from_device(raw), npaths, bias.cpu().numpy()


FIELDS = ("path_idx", "feature_idx", "group", "lower", "upper", "zero_fraction", "v")


def assert_same(torch, orc, ens, what):
    d_el, d_npaths, d_bias = device_extract(torch, ens)
    oel, onpaths, obias = orc.extract_paths(ens)
    assert d_npaths == onpaths, what
    assert len(d_el) == len(oel), what
    for f in FIELDS:
        assert np.ascontiguousarray(d_el[f]).tobytes() == np.ascontiguousarray(oel[f]).tobytes(), \
            (what, f)
    assert d_bias.tobytes() == np.ascontiguousarray(obias, np.float64).tobytes(), what
    el, npaths, bias = gts.extract_paths(ens)
    assert d_npaths == npaths, what
    assert d_el.tobytes() == el.tobytes(), what
    assert d_bias.tobytes() == bias.tobytes(), what


@pytest.mark.parametrize("name", ["tiny", "covtype_med", "deep", "wide"])
def test_workload_models_bitwise(torch, orc, name):
    w = synth.workload(name, rows=1)
    say("device extraction", name)
    assert_same(torch, orc, w.ensemble, name)


@pytest.mark.parametrize("seed", range(10))
def test_random_edge_case_ensembles_bitwise(torch, orc, seed):
    """Repeated features, ties, zero-cover nodes, several output groups."""
    w = synth.random_workload(seed, num_trees=20, max_depth=9, M=5, num_groups=3, n_bg=30,
                              rows=1)
    say("device extraction random", seed)
    assert_same(torch, orc, w.ensemble, f"random{seed}")


def full_tree(nodes, M):
    """A full tree of the largest 2^k - 1 <= nodes nodes, then leaves split one by one."""
    inner = (1 << ((nodes + 1).bit_length() - 2)) - 1
    res = [(2 * n + 1, 2 * n + 2, n % M, 0.5, 1024.0, 0.0) for n in range(inner)]
    res += [(-1, -1, -1, 0.0, 1.0, 0.25 * (n % 9)) for n in range(inner + 1)]
    n = len(res) - 1
    while len(res) < nodes:
        res[n] = (len(res), len(res) + 1, n % M, 0.5, 1.0, 0.0)
        res += [(-1, -1, -1, 0.0, 1.0, -1.0), (-1, -1, -1, 0.0, 0.0, 2.0)]
        n -= 1
    assert len(res) == nodes
    return res


# One workgroup a tree where all have at most 4096 nodes; a larger one anywhere sends the
# ensemble through the kernels of a thread a node.  The larger tree comes first, so a
# fault of another tree is not node 0's of tree 0.
BOTH = pytest.mark.parametrize("larger", [[], [4097]], ids=["tree", "node"])


@BOTH
def test_special_trees_bitwise(torch, orc, larger):
    rng = np.random.default_rng(4)
    leaf = [(-1, -1, -1, 0.0, 10.0, 2.5)]
    stump = [(1, 2, 1, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 3.0, -1.0), (-1, -1, -1, 0, 7.0, 4.0)]
    dup = [(1, 2, 0, 0.8, 16, 0), (3, 4, 0, 0.6, 12, 0), (-1, -1, -1, 0, 4, 1.0),
           (5, 6, 0, 0.3, 7, 0), (-1, -1, -1, 0, 5, 2.0), (-1, -1, -1, 0, 3, 3.0),
           (-1, -1, -1, 0, 4, 4.0)]
    # children stored before their parents, and a node no parent refers to
    shuffled = [(2, 1, 0, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 6.0, 1.5), (-1, -1, -1, 0, 4.0, -0.5),
                (-1, -1, -1, 0, 1.0, 9.0)]
    trees = [leaf, stump, dup, chain_tree(63, 63, rng), shuffled, leaf]
    trees += [full_tree(n, 7) for n in larger]
    ens = synth.ensemble_from_lists(trees, M=63, num_groups=2)
    say("device extraction special trees")
    assert_same(torch, orc, ens, "special trees")


@BOTH
def test_cycle_apart_from_the_tree(torch, larger):
    """Two nodes that are each other's child, with leaves, which no path from the root
    reaches: not part of the tree, as on the host (the oracle takes no such input)."""
    tree = [(1, 2, 1, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 3.0, -1.0), (-1, -1, -1, 0, 7.0, 4.0),
            (4, 5, 2, 0.5, 4.0, 0.0), (3, 6, 3, 0.5, 4.0, 0.0),
            (-1, -1, -1, 0, 1.0, 3.0), (-1, -1, -1, 0, 1.0, 7.0)]
    ens = synth.ensemble_from_lists([full_tree(n, 5) for n in larger] + [tree], M=5)
    say("device extraction cycle", larger)
    el, paths, bias = gts.extract_paths(ens)
    d_el, d_paths, d_bias = device_extract(torch, ens)
    assert d_paths == paths and d_el.tobytes() == el.tobytes()
    assert d_bias.tobytes() == bias.tobytes()


@BOTH
def test_errors_match_the_host(torch, larger):
    good = [(1, 2, 0, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 4.0, 1.0), (-1, -1, -1, 0, 6.0, 2.0)]
    cases = {
        "child out of range": [(1, 5, 0, 0.5, 10.0, 0.0)] + good[1:],
        "feature out of range": [(1, 2, 7, 0.5, 10.0, 0.0)] + good[1:],
        "NaN threshold": [(1, 2, 0, float("nan"), 10.0, 0.0)] + good[1:],
        "negative cover": [good[0], (-1, -1, -1, 0, -4.0, 1.0), good[2]],
        "shared child": [(1, 1, 0, 0.5, 10.0, 0.0)] + good[1:],
        "cycle to the root": [(1, 2, 0, 0.5, 10.0, 0.0), (0, 2, 1, 0.5, 4.0, 0.0),
                              (-1, -1, -1, 0, 6.0, 2.0)],
        "leaf value": [good[0], (-1, -1, -1, 0, 4.0, float("inf")), good[2]],
    }
    for what, tree in cases.items():
        ens = synth.ensemble_from_lists([full_tree(n, 2) for n in larger] + [good, tree], M=2)
        say("device extraction error", what, larger)
        with pytest.raises(gts.GtsError) as host:
            gts.extract_paths(ens)
        with pytest.raises(gts.GtsError) as dev:
            device_extract(torch, ens)
        assert dev.value.status == host.value.status == gts.GTS_EINVAL, what


def doubled_chain(depth, below):
    """A chain whose every node has the next one as both of its children, above a
    full tree: a leaf's count of the leaves to its left grows past the number of
    nodes, since every doubled link counts the whole tree once more."""
    res = [(d + 1, d + 1, 0, 0.5, 16.0, 0.0) for d in range(depth)]
    inner = (1 << below) - 1
    for n in range(2 * inner + 1):
        a = depth + 2 * n + 1
        res.append((a, a + 1, 1, 0.5, 16.0, 0.0) if n < inner else (-1, -1, -1, 0.0, 1.0, 1.0))
    ranks = depth * (inner + 1)
    assert ranks > 8 * len(res)
    return res


@BOTH
def test_ranks_of_a_malformed_tree_are_not_used(torch, larger):
    """The ranks of such a tree would index far past the workspace: the call
    reports the error as the host does, and a buffer allocated behind the
    workspace keeps its bytes."""
    ens = synth.ensemble_from_lists([full_tree(n, 2) for n in larger] + [doubled_chain(200, 8)],
                                    M=2)
    dens = gts.DeviceEnsemble(ens)
    size = ctypes.c_int64(0)
    assert gts.lib().gts_extract_workspace_bytes(ens.num_trees, ens.num_nodes,
                                                 ctypes.byref(size)) == 0
    need = size.value
    both = torch.full((need + (1 << 21),), 0x5a, dtype=torch.uint8, device="cuda")
    say("device extraction doubled chain", ens.num_nodes, need)
    with pytest.raises(gts.GtsError) as host:
        gts.extract_paths(ens)
    with pytest.raises(gts.GtsError) as dev:
        gts.extract_paths_device(dens, workspace=both[:need])
    assert dev.value.status == host.value.status == gts.GTS_EINVAL
    assert bool((both[need:] == 0x5a).all())


@BOTH
def test_too_long_merged_path(torch, larger):
    """64 distinct features on one path cannot fill a 64-lane bin."""
    rng = np.random.default_rng(1)
    ens = synth.ensemble_from_lists([full_tree(n, 64) for n in larger] + [chain_tree(64, 64, rng)],
                                    M=64)
    with pytest.raises(gts.GtsError) as dev:
        device_extract(torch, ens)
    assert dev.value.status == gts.GTS_EPATHLEN


@BOTH
@pytest.mark.parametrize("splits", [256, 257])
def test_deepest_path(torch, orc, splits, larger):
    """256 splits on a path are taken, on 5 features; 257 are refused."""
    rng = np.random.default_rng(splits)
    ens = synth.ensemble_from_lists([full_tree(n, 5) for n in larger] + [chain_tree(splits, 5, rng)],
                                    M=5)
    say("device extraction deep", splits, larger)
    if splits == 256:
        assert_same(torch, orc, ens, "256 splits")
        return
    with pytest.raises(gts.GtsError) as dev:
        device_extract(torch, ens)
    assert dev.value.status == gts.GTS_EINVAL
    assert "256" in str(dev.value)


@pytest.mark.parametrize("M", [5, 90])
@pytest.mark.parametrize("nodes", [4095, 4097])
def test_trees_at_one_workgroups_limit(torch, orc, M, nodes):
    trees = [full_tree(n, M) for n in (1, 3, nodes, 7)]
    say("device extraction nodes", nodes, M)
    assert_same(torch, orc, synth.ensemble_from_lists(trees, M=M), f"{nodes} nodes")


@pytest.mark.parametrize("M", [5, 90])
@pytest.mark.parametrize("depth", [11, 12])
def test_trees_around_one_workgroup(torch, M, depth):
    """Full trees of 4095 and 8191 nodes, on both sides of the 4096 nodes one
    workgroup holds, beside small ones, with at most and more than 64 features:
    the host's elements and bias, byte for byte."""
    w = synth.random_workload(40 + M, num_trees=2, max_depth=depth, p_split=1.0, M=M,
                              num_groups=2, n_bg=300, rows=1)
    small = synth.random_workload(41 + M, num_trees=9, max_depth=4, M=M, num_groups=2, n_bg=300,
                                  rows=1)
    a, b = w.ensemble, small.ensemble
    cat = {k: np.concatenate([getattr(a, k), getattr(b, k)])
           for k in ("tree_group", "left", "right", "feature", "threshold", "cover", "value")}
    off = np.concatenate([a.tree_node_offsets, a.num_nodes + b.tree_node_offsets[1:]])
    ens = synth.Ensemble(num_features=M, num_groups=2, tree_node_offsets=off, **cat)
    assert np.diff(off).max() == (1 << (depth + 1)) - 1
    raw, npaths, bias = gts.extract_paths_device(gts.DeviceEnsemble(ens))
    el, want_paths, want_bias = gts.extract_paths(ens)
    assert npaths == want_paths
    assert raw.cpu().numpy().tobytes() == el.tobytes()
    assert bias.cpu().numpy().tobytes() == want_bias.tobytes()
