"""bench.matrix_products, the matrix instructions the step's kernels issue, at degree 4 in FP32 against the
hardware counter's figures per element or face (profiles/step_kernels_n4_311k.md), and the parts that can be
counted by hand."""
import os
import re

import pytest

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_degree_4_matches_the_counter():
    txt = open(os.path.join(ROOT, "profiles", "step_kernels_n4_311k.md")).read()
    got = {k: sum(v.values()) for k, v in bench.matrix_products(4, "fp32").items()}
    for name, kernel in (("k_ck", "predict"), ("k_update", "volume"), ("k_face", "face_flux")):
        row = re.search(rf"`dgd::{name}<[^|]*\|[^|]*\|\s*(\d+)\s*\|[^|]*\|[^|]*\|[^|]*\|", txt)
        assert int(row.group(1)) == got[kernel], name


def test_degree_1():
    """One tile of 4 modes, 8 points in a chunk, 2 tiles of derivative columns."""
    p = bench.matrix_products(1, "fp64")
    assert p["predict"]["fp64"] == 4 + 3 + 9                        # nodal values, K^e, mixing
    assert p["volume"]["fp64"] == 4 + 8 + 16 + 9                    # lift, evaluation, projection and stiffness, mixing
    assert p["face_flux"]["fp64"] == 2 * 2 + 1
    assert all(v["bf16"] == 0 for v in p.values())


@pytest.mark.parametrize("N", [1, 2, 3, 4])
def test_bf16_handles_issue_the_fp32_step(N):
    assert bench.matrix_products(N, "bf16") == bench.matrix_products(N, "fp32")
