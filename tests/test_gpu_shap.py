"""gts_shap on the GPU against the fp64 CPU oracle (SHAP values, Eq. 2).

Small cases compare every output element; the full-size workloads run in the
benchmark's launch configuration and compare every row (the wide model: a
2000-row prefix and the tail) with the oracle's Algorithm 1, plus, for every
row, local accuracy (Eq. 1: the explanation sums to the model output).
"""
import numpy as np
import pytest

from paper_2010_13972_amd import gts, synth
from parity import assert_parity, sum_tolerance

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return torch


def run_shap(torch, ens, X, dtype, ld_pad=0):
    model = gts.prepare(ens, dtype)
    Xd = torch.zeros((X.shape[0], X.shape[1] + ld_pad), dtype=torch.float32, device="cuda")
    Xd[:, :X.shape[1]] = torch.from_numpy(np.ascontiguousarray(X, np.float32))
    phi = gts.shap(model, Xd)
    torch.cuda.synchronize()
    return phi.cpu().numpy().astype(np.float64)


def say(*a):
    print(*a, flush=True)


# --------------------------------------------------------------------------
# small inputs: every element
# --------------------------------------------------------------------------

@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_tiny_ensemble_all_rows_vs_brute_force(torch, orc, dtype):
    w = synth.workload("tiny")
    say("tiny", dtype, w.X.shape)
    got = run_shap(torch, w.ensemble, w.X, dtype)
    want = orc.brute_shap(w.ensemble, w.X)
    assert_parity(got, want, dtype, what="tiny vs Eq. 2")
    assert_parity(got, orc.treeshap(w.ensemble, w.X), dtype, what="tiny vs Algorithm 1")


@pytest.mark.parametrize("seed", range(8))
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_random_edge_case_ensembles(torch, orc, seed, dtype):
    """Repeated features, ties x == t, zero-cover nodes, three output groups,
    ragged row counts."""
    w = synth.random_workload(seed, num_trees=12, max_depth=7, M=6, num_groups=3,
                              n_bg=40, rows=37 + 29 * seed)
    say("random", seed, dtype, w.X.shape)
    got = run_shap(torch, w.ensemble, w.X, dtype)
    assert_parity(got, orc.treeshap(w.ensemble, w.X), dtype, what=f"random{seed}")


@pytest.mark.parametrize("rows", [1, 2, 63, 64, 65, 130])
def test_ragged_row_counts_and_strided_X(torch, orc, rows):
    w = synth.workload("tiny")
    X = np.concatenate([w.X] * 2)[:rows]
    say("ragged", rows)
    got = run_shap(torch, w.ensemble, X, "f64", ld_pad=3)
    assert_parity(got, orc.treeshap(w.ensemble, X), "f64", what=f"rows={rows}")


def test_zero_rows_is_a_no_op(torch):
    w = synth.workload("tiny")
    model = gts.prepare(w.ensemble, "f32")
    X = torch.zeros((0, 8), dtype=torch.float32, device="cuda")
    out = gts.shap(model, X)
    torch.cuda.synchronize()
    assert tuple(out.shape) == (0, 1, 9)


def test_side_streams_and_concurrent_models(torch):
    """Launches on two non-default streams at once (two models, one of them
    with interaction values) give the default stream's results: no result
    depends on an earlier call.  (Not bit for bit: the order in which waves
    add to a tile entry varies from run to run.)"""
    wa, wb = synth.workload("covtype_med"), synth.workload("tiny")
    ma, mb = gts.prepare(wa.ensemble, "f32"), gts.prepare(wb.ensemble, "f64")
    Xa = torch.from_numpy(wa.X[:3000]).cuda()
    Xb = torch.from_numpy(wb.X).cuda()
    ref_a = gts.shap(ma, Xa)
    ref_b = gts.shap_interactions(mb, Xb)
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    outs = []
    for _ in range(3):
        with torch.cuda.stream(s1):
            oa = gts.shap(ma, Xa)
        with torch.cuda.stream(s2):
            ob = gts.shap_interactions(mb, Xb)
        outs.append((oa, ob))
    torch.cuda.synchronize()
    ra = ref_a.cpu().numpy().astype(np.float64)
    rb = ref_b.cpu().numpy().astype(np.float64)
    for oa, ob in outs:
        assert_parity(oa.cpu().numpy(), ra, "f32", what="side stream, SHAP")
        assert_parity(ob.cpu().numpy(), rb, "f64", 2, what="side stream, interactions")


def chain_tree(depth, M, rng):
    """A spine of `depth` splits on distinct features (the left child
    continues the spine), so the deepest path has `depth` features."""
    res = []
    cover = 1000.0
    for d in range(depth):
        base = len(res)
        res.append((base + 2, base + 1, d % M, np.float32(0.5 + 0.01 * d), cover, 0.0))
        cl = max(1.0, float(int(cover * 0.8)))
        res.append((-1, -1, -1, 0.0, cover - cl, float(rng.normal())))
        cover = cl
    res.append((-1, -1, -1, 0.0, cover, float(rng.normal())))
    return res


@pytest.mark.parametrize("depth", [1, 15, 16, 17, 31, 63])
def test_long_paths(torch, orc, depth):
    """Path lengths around the unrolled-variant boundary and the wave64
    maximum (63 features + root = 64 elements)."""
    rng = np.random.default_rng(depth)
    M = 63
    trees = [chain_tree(depth, M, rng), chain_tree(max(1, depth // 2), M, rng)]
    ens = synth.ensemble_from_lists(trees, M=M)
    X = rng.uniform(0.4, 1.2, size=(70, M)).astype(np.float32)
    say("long paths", depth)
    for dtype in ("f64", "f32"):
        got = run_shap(torch, ens, X, dtype)
        assert_parity(got, orc.treeshap(ens, X), dtype, what=f"depth={depth}")


def test_special_models(torch, orc):
    """Single-leaf trees (bias only), stumps, and a path whose feature is
    repeated at every level (merged into one element)."""
    leaf = [(-1, -1, -1, 0.0, 10.0, 2.5)]
    stump = [(1, 2, 1, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 3.0, -1.0), (-1, -1, -1, 0, 7.0, 4.0)]
    dup = [(1, 2, 0, 0.8, 16, 0), (3, 4, 0, 0.6, 12, 0), (-1, -1, -1, 0, 4, 1.0),
           (5, 6, 0, 0.3, 7, 0), (-1, -1, -1, 0, 5, 2.0), (-1, -1, -1, 0, 3, 3.0),
           (-1, -1, -1, 0, 4, 4.0)]
    ens = synth.ensemble_from_lists([leaf, stump, dup, leaf], M=3)
    X = np.random.default_rng(0).uniform(0, 1, size=(50, 3)).astype(np.float32)
    X[:5, 0] = [0.3, 0.6, 0.8, 0.0, 1.0]  # exact ties with thresholds
    for dtype in ("f64", "f32"):
        got = run_shap(torch, ens, X, dtype)
        want = orc.treeshap(ens, X)
        assert_parity(got, want, dtype, what="special models")
        assert np.all(got[:, 0, 2] == 0.0)  # feature 2 never used


@pytest.mark.parametrize("M", [16, 17])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_rank_table_feature_limit(torch, orc, M, dtype):
    """One-path-per-wave launches with private tiles test each path for dead
    (row, path) pairs on a batch this small (test_gpu_rank_tables.py has the
    test by rank tables, which serves M <= 16): 16 and 17 features, zero-cover
    splits and rows tied on four values, 150 rows (three 64-row tiles, the last
    ragged)."""
    w = synth.random_workload(60 + M, num_trees=14, max_depth=7, M=M, n_bg=30, rows=150)
    model = gts.prepare(w.ensemble, dtype)
    cfg = gts.launch_config(model, 150)
    say("rank tables", M, dtype, cfg)
    assert cfg["rows_per_tile"] == 64 and cfg["private_tiles"] == 1
    got = run_shap(torch, w.ensemble, w.X, dtype)
    assert_parity(got, orc.treeshap(w.ensemble, w.X), dtype, what=f"M={M} {dtype}")


def spine_tree(feats, rng, zero_right):
    """A spine of splits on the distinct features `feats` (the left child
    continues the spine) with a leaf on every right; right leaves at the
    spine positions in `zero_right` have zero cover, so their paths end in a
    zero-fraction element that rows going left never reach."""
    res, cover = [], 1000.0
    for d, f in enumerate(feats):
        base = len(res)
        right = 0.0 if d in zero_right else max(1.0, float(int(cover * 0.15)))
        res.append((base + 2, base + 1, int(f), np.float32(rng.uniform(0.25, 0.75)), cover, 0.0))
        res.append((-1, -1, -1, 0.0, right, float(rng.normal())))
        cover -= right
    res.append((-1, -1, -1, 0.0, cover, float(rng.normal())))
    return res


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_sixteen_feature_paths(torch, orc, dtype):
    """Paths of 12 to 16 features on a 16-feature model: the variant
    unrolled for at most 16 features, and in fp32 the one-path-per-wave launch
    with private tiles; 150 rows (three 64-row tiles, the last ragged)."""
    rng = np.random.default_rng(16)
    M = 16
    trees = []
    for t in range(24):
        n = 12 + t % 5
        zero = set(rng.choice(n, size=1 + t % 4, replace=False).tolist())
        trees.append(spine_tree(rng.permutation(M)[:n], rng, zero))
    ens = synth.ensemble_from_lists(trees, M=M)
    X = rng.uniform(0.0, 1.0, size=(150, M)).astype(np.float32)
    model = gts.prepare(ens, dtype)
    cfg = gts.launch_config(model, 150)
    say("sixteen-feature paths", dtype, cfg)
    assert model.desc.max_path_len == 17  # 16 features and the root
    if dtype == "f32":
        assert cfg["rows_per_tile"] == 64 and cfg["private_tiles"] == 1
    got = run_shap(torch, ens, X, dtype)
    assert_parity(got, orc.treeshap(ens, X), dtype, what=f"16-feature paths {dtype}")


def test_bins_without_live_paths(torch, orc):
    """Trees whose right subtree has zero cover: its paths carry two
    zero-fraction elements, and rows with x0 < 0.5 reach none of them, so
    all of these (longer) paths of whole bins are dead for whole tiles; the left
    paths (cover 10 of 10) stay live.  Rows with x0 >= 0.5 in
    a later tile make some of them live there."""
    rng = np.random.default_rng(7)
    trees = []
    for t in range(60):
        f1 = 1 + t % 7
        trees.append([(1, 2, 0, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 10.0, float(rng.normal())),
                      (3, 4, f1, 0.25 + 0.5 * rng.random(), 0.0, 0.0),
                      (-1, -1, -1, 0, 0.0, float(rng.normal())),
                      (-1, -1, -1, 0, 0.0, float(rng.normal()))])
    ens = synth.ensemble_from_lists(trees, M=8)
    X = rng.uniform(0, 0.5, size=(200, 8)).astype(np.float32)
    X[128:, 0] = rng.uniform(0.5, 1.0, size=72)   # the third and fourth tiles reach the right subtrees
    for dtype in ("f32", "f64"):
        got = run_shap(torch, ens, X, dtype)
        want = orc.treeshap(ens, X)
        assert_parity(got, want, dtype, what="dead bins")
        assert np.all(got[:128, 0, 1:8] == 0.0)  # no live path splits on f1..f7 there


def empty_ensemble(M, G):
    return synth.Ensemble(
        num_features=M, num_groups=G, tree_node_offsets=np.zeros(1, np.int64),
        tree_group=np.zeros(0, np.int32), left=np.zeros(0, np.int32),
        right=np.zeros(0, np.int32), feature=np.zeros(0, np.int32),
        threshold=np.zeros(0, np.float32), cover=np.zeros(0), value=np.zeros(0))


def test_empty_model_and_unfed_groups(torch, orc):
    """A model without trees, and a model whose middle output group no tree
    feeds: phi is exactly 0 there (no path, bias 0); the fed groups match
    Algorithm 1."""
    X = np.random.default_rng(1).uniform(0, 1, size=(70, 3)).astype(np.float32)
    for dtype in ("f64", "f32"):
        say("empty model", dtype)
        got = run_shap(torch, empty_ensemble(3, 2), X, dtype)
        assert got.shape == (70, 2, 4) and np.all(got == 0.0)
    stump = [(1, 2, 1, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 3.0, -1.0), (-1, -1, -1, 0, 7.0, 4.0)]
    stump0 = [(1, 2, 0, 0.25, 8.0, 0.0), (-1, -1, -1, 0, 2.0, 1.5), (-1, -1, -1, 0, 6.0, -0.5)]
    leaf = [(-1, -1, -1, 0.0, 10.0, 2.5)]
    ens = synth.ensemble_from_lists([stump, leaf, stump0], M=3, num_groups=3,
                                    tree_group=[0, 2, 0])
    for dtype in ("f64", "f32"):
        say("unfed group", dtype)
        got = run_shap(torch, ens, X, dtype)
        assert_parity(got, orc.treeshap(ens, X), dtype, what="unfed group")
        assert np.all(got[:, 1, :] == 0.0)


# (M, dtype, rows per tile the launch policy picks): a private tile per wave,
# and shared tiles of 64, 32, 16 and 4 rows (8 is the wide workload's)
SHAPES = [(8, "f32", 64), (63, "f32", 64), (150, "f32", 32), (250, "f32", 16),
          (150, "f64", 16), (3000, "f32", 4)]


@pytest.mark.parametrize("M,dtype,rw", SHAPES, ids=[f"M{m}-{d}" for m, d, _ in SHAPES])
def test_launch_shapes(torch, orc, M, dtype, rw):
    """Every tile height of the launch policy, checked through
    gts_launch_config, against Algorithm 1 on a ragged row count."""
    w = synth.random_workload(7 + M, num_trees=10, max_depth=6, M=M, num_groups=2, n_bg=40,
                              rows=70)
    model = gts.prepare(w.ensemble, dtype)
    cfg = gts.launch_config(model, 70)
    say("launch shape", M, dtype, cfg)
    assert cfg["rows_per_tile"] == rw
    assert cfg["private_tiles"] == (1 if M == 8 else 0)
    assert cfg["lds_bytes"] <= 160 * 1024
    assert cfg["workgroups"] == -(-70 // rw) * 2 * cfg["slices"]
    got = run_shap(torch, w.ensemble, w.X, dtype)
    assert_parity(got, orc.treeshap(w.ensemble, w.X), dtype, what=f"M={M} {dtype}")


# --------------------------------------------------------------------------
# full-size workloads, in the launch configuration bench.py times: every row
# (or a long prefix and the tail) element by element against Algorithm 1
# --------------------------------------------------------------------------

def sample_rows(n, k=24, seed=0):
    rng = np.random.default_rng(seed)
    rows = set(range(min(4, n))) | set(range(max(0, n - 4), n))
    rows |= set(rng.choice(n, size=min(k, n), replace=False).tolist())
    return np.array(sorted(rows))


# (workload, dtype, rows compared: None = all)
FULL = [("covtype_med", "f32", None), ("deep", "f32", None), ("deep", "f64", None),
        ("wide", "f32", 2000), ("tiny", "f64", None)]


@pytest.mark.parametrize("name,dtype,prefix", FULL, ids=[f"{n}-{d}" for n, d, _ in FULL])
def test_full_size_workloads(torch, orc, name, dtype, prefix):
    w = synth.workload(name)
    n = w.X.shape[0]
    say("full size", name, dtype, w.X.shape, "paths", int((w.ensemble.left < 0).sum()))
    got = run_shap(torch, w.ensemble, w.X, dtype)
    rows = np.arange(n) if prefix is None else \
        np.unique(np.concatenate([np.arange(prefix), np.arange(n - 65, n), sample_rows(n)]))
    say("  oracle on", len(rows), "rows")
    want = orc.treeshap(w.ensemble, w.X[rows])
    assert_parity(got[rows], want, dtype, what=f"{name} {dtype}, {len(rows)} rows")
    # Eq. 1 on every row, scaled by the oracle's magnitudes (the largest
    # explanation among the compared rows)
    f = orc.predict(w.ensemble, w.X)
    err = np.abs(got.sum(-1) - f)
    scale = float(sum_tolerance(np.abs(want), dtype).max())
    assert np.all(err <= scale), float(err.max() / scale)


@pytest.mark.parametrize("name,rows", [("covtype_med", 1 << 20), ("deep", 1 << 16)])
def test_large_row_counts(torch, orc, name, rows):
    """The largest batches the rows sweep times (2^20 rows of the
    covtype-shaped model, 2^16 of the deep one): 1024 rows spread over the
    batch (and its tail) element by element against Algorithm 1; every row
    against Eq. 1, with a bound scaled by the oracle's magnitudes on the
    compared rows."""
    w = synth.workload(name, rows=1)
    X = synth.sweep_rows(name, rows)
    say("large batch", name, X.shape)
    got = run_shap(torch, w.ensemble, X, "f32")
    sel = np.unique(np.concatenate([np.arange(0, rows, rows // 1024), np.arange(rows - 65, rows),
                                    sample_rows(rows, k=16, seed=3)]))
    want = orc.treeshap(w.ensemble, X[sel])
    assert_parity(got[sel], want, "f32", what=f"{name} {rows} rows, {len(sel)} compared")
    f = orc.predict(w.ensemble, X)
    err = np.abs(got.sum(-1) - f)
    scale = 2 * float(sum_tolerance(np.abs(want), "f32").max())
    assert np.all(err <= scale), float(err.max() / scale)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("inter", [False, True])
def test_largest_feature_count(torch, orc, dtype, inter):
    """The widest phi row a workgroup's LDS holds (4 rows per tile): the
    largest M that gts_launch_config accepts runs and matches the oracle;
    one more feature is GTS_EINVAL from the launch call, before any launch."""
    def stump(M):
        return [(1, 2, M - 1, 0.5, 10.0, 0.0), (-1, -1, -1, 0, 3.0, -1.0), (-1, -1, -1, 0, 7.0, 4.0)]

    def fits(M):
        model = gts.prepare(synth.ensemble_from_lists([stump(M)], M=M), dtype)
        try:
            gts.launch_config(model, 8, inter)
            return True
        except gts.GtsError as e:
            assert e.status == gts.GTS_EINVAL
            return False

    lo, hi = 2, 1 << 14
    assert fits(lo) and not fits(hi)
    while lo + 1 < hi:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if fits(mid) else (lo, mid)
    say("largest M", dtype, inter, lo)
    rng = np.random.default_rng(lo)
    fn = gts.shap_interactions if inter else gts.shap
    want = orc.interactions if inter else orc.treeshap
    for M, good in ((lo, True), (lo + 1, False)):
        ens = synth.ensemble_from_lists([stump(M), [(-1, -1, -1, 0.0, 5.0, 0.25)]], M=M)
        X = rng.uniform(0, 1, size=(9, M)).astype(np.float32)
        model = gts.prepare(ens, dtype)
        Xd = torch.from_numpy(X).cuda()
        if good:
            got = fn(model, Xd)
            torch.cuda.synchronize()
            assert_parity(got.cpu().numpy().astype(np.float64), want(ens, X), dtype,
                          2 if inter else 1, f"M={M}")
        else:
            with pytest.raises(gts.GtsError) as err:
                fn(model, Xd)
            assert err.value.status == gts.GTS_EINVAL


@pytest.mark.parametrize("dtype,largest", [("f32", 17), ("f64", 11)])
def test_one_path_per_wave_boundary(torch, orc, dtype, largest):
    """The host keeps a path's elements (after its zero-fraction ones) in
    feature order, without the collision-avoiding rotation, exactly for the
    models whose every launch runs one path per wave: M <= 17 in fp32 and
    M <= 11 in fp64.  gts_launch_config must agree (64-row tiles for SHAP and
    interaction values up to that M, fewer rows for interaction values one
    feature above), and the results match the oracle on both sides."""
    for M in (largest, largest + 1):
        w = synth.random_workload(50 + M, num_trees=6, max_depth=6, M=M, num_groups=1,
                                  n_bg=40, rows=40)
        model = gts.prepare(w.ensemble, dtype)
        shap_rw = gts.launch_config(model, 40)["rows_per_tile"]
        inter_rw = gts.launch_config(model, 40, interactions=True)["rows_per_tile"]
        say("one path per wave", dtype, M, shap_rw, inter_rw)
        assert shap_rw == 64
        assert (inter_rw == 64) == (M == largest)
        got = run_shap(torch, w.ensemble, w.X, dtype)
        assert_parity(got, orc.treeshap(w.ensemble, w.X), dtype, what=f"M={M}")
        Xd = torch.from_numpy(w.X).cuda()
        inter = gts.shap_interactions(model, Xd)
        torch.cuda.synchronize()
        assert_parity(inter.cpu().numpy().astype(np.float64), orc.interactions(w.ensemble, w.X),
                      dtype, 2, f"interactions M={M}")
