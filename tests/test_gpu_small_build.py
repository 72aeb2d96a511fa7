"""Builds around the sizes where the small-scene sort (one workgroup, 1024 or 4096 points) and the wave that
finishes the clustering (64 clusters) begin and end, with many equal codes: bit-exact against the CPU reference."""

import numpy as np
import pytest
import torch

from oracle import oracle as O
from synthetic import scenes
from tests.test_gpu_bvh import _build

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("same", [False, True])
@pytest.mark.parametrize("n", [2, 63, 64, 65, 130, 1023, 1024, 1025, 2049, 4095, 4096, 4097])
def test_small_build_bit_exact(n, same):
    print("case small build", n, same, flush=True)
    sc = scenes.random_scene(300 + n, n)
    if same:
        sc.mean[::2] = sc.mean[0]  # equal codes keep the order of their indices
    got, status = _build(sc)
    assert status == 0
    codes, lo, hi = O.morton_codes(sc.mean)
    sorted_codes, perm = O.sort_codes(codes)
    np.testing.assert_array_equal(got["bounds"][:3], lo)
    np.testing.assert_array_equal(got["bounds"][3:], hi)
    np.testing.assert_array_equal(got["codes"], sorted_codes)
    np.testing.assert_array_equal(got["perm"], perm)
    lb = O.leaf_boxes(sc.mean, sc.scale, sc.quat, perm)
    child, boxes, _ = O.ploc(lb)
    np.testing.assert_array_equal(got["child"], child)
    np.testing.assert_array_equal(got["boxes"], boxes)
