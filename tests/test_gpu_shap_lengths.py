"""SHAP values of paths of 9 to 16 features in every launch shape (private and
shared 64-row tiles, 32, 16, 8 and 4 rows, tiles of doubles and of floats)
against Algorithm 1: the quadrature at every number of nodes and the chains'
shorter paths beside them, on ragged rows."""
import dataclasses

import numpy as np
import pytest

from paper_2010_13972_amd import gts, synth
from parity import assert_parity
from test_gpu_shap import chain_tree

pytestmark = pytest.mark.gpu

# (M, rows per tile, private tiles)
SHAPES = [(16, 64, 1), (60, 64, 0), (120, 32, 0), (300, 16, 0), (700, 8, 0), (3500, 4, 0)]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("M,rw,priv", SHAPES)
def test_path_lengths_in_every_shape(orc, M, rw, priv, dtype):
    import torch
    if dtype == "f64" and M == 3500:
        M = 2500
    rng = np.random.default_rng(M)
    X = rng.random((71, M)).astype(np.float32)
    for depth in (9, 12, 13, 16):
        ens = synth.ensemble_from_lists([chain_tree(depth, min(M, 63), rng),
                                         chain_tree(7, min(M, 63), rng)], M=M)
        model = gts.prepare(ens, dtype)
        cfg = gts.launch_config(model, 71)
        print("shape", M, dtype, depth, cfg, flush=True)
        if dtype == "f32":
            assert (cfg["rows_per_tile"], cfg["private_tiles"]) == (rw, priv)
        got = gts.shap(model, torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
        assert_parity(got, orc.treeshap(ens, X), dtype, what=f"M={M} {dtype} depth {depth}")


@pytest.mark.parametrize("M", [16, 60, 700])
@pytest.mark.parametrize("depth", [8, 12, 16])
def test_small_leaf_values(M, depth):
    """Leaves scaled by 2^-60: the values scale with them.  An fp32 node weight
    of a long path times such a leaf would not be a normal number.  Both sides
    round each of at most 33 paths' values to about 40 x 2^-24."""
    import torch
    rng = np.random.default_rng(depth)
    X = torch.from_numpy(rng.random((65, M)).astype(np.float32)).cuda()
    ens = synth.ensemble_from_lists([chain_tree(depth, min(M, 63), rng)], M=M)
    out = []
    for scale in (1.0, 2.0 ** -60):
        e = dataclasses.replace(ens, value=ens.value * scale)
        print("leaves", M, depth, scale, flush=True)
        out.append(gts.shap(gts.prepare(e, "f32"), X).cpu().numpy().astype(np.float64) / scale)
    np.testing.assert_allclose(out[1], out[0], rtol=0, atol=5e-6 * np.abs(out[0]).max())
