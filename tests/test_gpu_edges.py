"""Kernels at the edges of their tiles and ranges, against the oracle."""
import pytest

from tests.test_gpu_cluster import test_cluster_parity as _cluster_parity

pytestmark = pytest.mark.gpu


# The eigensolver and the Cholesky factor hold d <= 64 and d <= 128 matrices in
# 4 x 4 register blocks: the smallest sizes, and one to each side of a block
# edge and of the switch between the two kernels.
@pytest.mark.parametrize("dt,d,xf", [
    ("f32", 2, "pca"), ("f32", 3, "metric"), ("f32", 5, "adaptive"),
    ("f32", 17, "metric"), ("f32", 63, "metric"), ("bf16", 65, "metric"), ("f32", 96, "pca"),
    ("f32", 127, "metric"), ("f32", 128, "adaptive"),
])
def test_transform_edges(dt, d, xf):
    _cluster_parity(dt, 900, d, 32, xf)
