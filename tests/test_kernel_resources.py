"""The compiler's resource report of the SHAP and interaction kernels
(written by the build into _build/kernel_resources.txt): the variants built
for paths of at most 8, 12 or 16 features hold no runtime-length path code and
no per-lane path arrays; only the long-path variants do."""
import os
import re

import pytest

REPORT = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                      "paper_2010_13972_amd", "_build", "kernel_resources.txt")
# shap_kernel<T, RW, INTER, WAVES, PRIV, QMAX, WIDE> in the mangled name
KERNEL = re.compile(r"shap_kernelI([fd])Li(\d+)ELb(\d)ELi(\d+)ELb(\d)ELi(\d+)ELb(\d)E")


def variants():
    if not os.path.exists(REPORT):
        pytest.skip("library not built (the report comes from the build)")
    out = []
    with open(REPORT) as f:
        for line in f:
            d = dict(kv.split("=", 1) for kv in line.rstrip("\n").split("\t"))
            m = KERNEL.search(d["name"])
            if m:
                t, rw, inter, waves, priv, qmax, wide = m.groups()
                out.append(dict(dtype=t, rw=int(rw), inter=inter == "1", waves=int(waves),
                                priv=priv == "1", qmax=int(qmax), wide=wide == "1",
                                scratch=int(d["ScratchSize [bytes/lane]"]),
                                vgprs=int(d["VGPRs"])))
    return out


def planned(dtype, inter, qmax):
    """The launch shapes the planner gives a variant: (rows, waves, private, double)."""
    def of(rows, waves, wide=False):
        return {(rows, w, False, wide) for w in waves}
    out = {(64, 4, True, False)}
    if inter:
        return out | of(64, [8]) | of(32, [8]) | of(16, [8, 16]) | of(8, [8, 16]) | of(4, [8, 16])
    if dtype == "d":
        low = [8, 12, 16] if qmax <= 12 else [8, 12]
        out |= of(8, low) | of(4, low) | of(64, [8]) | of(32, [8])
        return out | of(16, {8: [16], 12: [12, 16]}.get(qmax, [12]))
    out |= of(8, [8, 12, 16]) | of(4, [8, 12, 16])
    if qmax == 8:
        return (out | of(64, [8, 12, 16], True) | of(32, [8], True) | of(16, [12], True) |
                of(8, [12], True))
    out |= of(16, [16], True) | of(8, [12, 16], True)
    tall = [8] if qmax == 64 else [8, 16]
    return out | of(64, tall, True) | of(32, tall, True)


def test_every_variant_is_built():
    v = variants()
    for dtype in "fd":
        for inter, lengths in ((False, (8, 12, 16, 64)), (True, (8, 64))):
            for qmax in lengths:
                built = [(x["rw"], x["waves"], x["priv"], x["wide"]) for x in v
                         if (x["dtype"], x["inter"], x["qmax"]) == (dtype, inter, qmax)]
                assert sorted(built) == sorted(planned(dtype, inter, qmax)), (dtype, inter, qmax)
    assert {x["qmax"] for x in v if not x["inter"]} == {8, 12, 16, 64}
    assert {x["qmax"] for x in v if x["inter"]} == {8, 64}


# registers per lane a wave may hold when a workgroup of `waves` waves must
# fit on a CU (4 SIMDs, 512 registers per SIMD lane, granule 8)
VGPR_CAP = {4: 256, 8: 256, 12: 168, 16: 128}


def test_short_path_variants_hold_no_path_arrays():
    for x in variants():
        if x["qmax"] == 64:
            # the runtime-length code keeps 64-entry arrays per lane
            assert x["scratch"] >= 64 * 8, x
        elif x["scratch"]:
            # only register spills of a variant at its launch bound's cap
            assert x["vgprs"] == VGPR_CAP[x["waves"]] and x["scratch"] < (1024 if x["inter"] else 256), x
            assert x["inter"] or x["dtype"] == "d", x


def test_fp32_shap_variants_of_unrolled_paths_use_no_scratch():
    """Paths of at most 16 features, every launch shape."""
    for x in variants():
        if x["dtype"] == "f" and not x["inter"] and x["qmax"] <= 16:
            assert x["scratch"] == 0, x


# inter_quad_kernel<T, C, A, RW, LPR, WAVES> in the mangled name: model, arithmetic and
# tile type, rows, lanes a row, waves
QUAD = re.compile(r"inter_quad_kernelI([fd])([fd])([fd])Li(\d+)ELi(\d+)ELi(\d+)E")
# registers and scratch bytes a lane may hold (one workgroup a CU)
QUAD_CAPS = {("f", "f", "d", 16, 4, 16): (128, 32), ("f", "f", "d", 8, 8, 16): (128, 0),
             ("f", "f", "d", 4, 8, 16): (128, 0), ("f", "d", "f", 8, 8, 12): (168, 32),
             ("f", "d", "f", 4, 8, 16): (128, 192), ("f", "d", "f", 4, 8, 8): (256, 0),
             ("d", "d", "d", 16, 4, 8): (256, 0), ("d", "d", "d", 8, 8, 8): (256, 0),
             ("d", "d", "d", 4, 8, 8): (256, 0)}


def test_interaction_quadrature_kernels():
    """Every launch shape of the interaction quadrature, and no other, within its
    registers; what spills is a few words a lane."""
    if not os.path.exists(REPORT):
        pytest.skip("library not built (the report comes from the build)")
    seen = {}
    with open(REPORT) as f:
        for line in f:
            d = dict(kv.split("=", 1) for kv in line.rstrip("\n").split("\t"))
            m = QUAD.search(d["name"])
            if m:
                t, c, a, rw, lpr, waves = m.groups()
                seen[t, c, a, int(rw), int(lpr), int(waves)] = (
                    int(d["VGPRs"]), int(d["ScratchSize [bytes/lane]"]))
    assert set(seen) == set(QUAD_CAPS)
    for k, (vgprs, scratch) in seen.items():
        assert vgprs <= QUAD_CAPS[k][0] and scratch <= QUAD_CAPS[k][1], (k, vgprs, scratch)


def test_headline_variants_fit_their_occupancy():
    """The fp32 SHAP kernels for paths of at most 8 features with 64-row
    tiles: the shared-tile variant (covtype-shaped workload) stays within 64
    registers (8 waves per SIMD); the private-tile variant (deep and tiny
    workloads), whose rank tables hold a workgroup to 24 KB of LDS and so a
    CU to 6 workgroups of 4 waves, within 80 (6 waves per SIMD)."""
    seen = 0
    for x in variants():
        if x["dtype"] == "f" and not x["inter"] and x["qmax"] == 8 and x["rw"] == 64:
            cap = 80 if x["priv"] else 64
            assert x["vgprs"] <= cap and x["scratch"] == 0, x
            seen += 1
    assert seen == 4   # the private tile; shared ones of 8, 12 and 16 waves


def test_prune_kernels_use_no_private_memory():
    """The batch-pruning kernels (key sort, search, plan, copy) keep their
    arrays in registers and LDS: no scratch."""
    if not os.path.exists(REPORT):
        pytest.skip("library not built (the report comes from the build)")
    names = ("sort_keys", "mark_paths", "plan_pruned", "copy_paths")
    seen = set()
    with open(REPORT) as f:
        for line in f:
            d = dict(kv.split("=", 1) for kv in line.rstrip("\n").split("\t"))
            for n in names:
                if n in d["name"]:
                    seen.add(n)
                    assert d["ScratchSize [bytes/lane]"] == "0", d
    assert seen == set(names)


def test_device_build_kernels_use_no_private_memory():
    """The kernels that write a model blob from a host plan keep every path's
    merged feature ranges and fractions in registers: no scratch."""
    if not os.path.exists(REPORT):
        pytest.skip("library not built (the report comes from the build)")
    names = ("k_build_paths", "k_plan_tree_sums", "k_plan_bias", "k_plan_bins", "k_zero_gaps")
    seen = set()
    with open(REPORT) as f:
        for line in f:
            d = dict(kv.split("=", 1) for kv in line.rstrip("\n").split("\t"))
            for n in names:
                if n in d["name"]:
                    seen.add(n)
                    assert d["ScratchSize [bytes/lane]"] == "0", d
    assert seen == set(names)
