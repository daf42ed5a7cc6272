"""The column walk on walked axes with two segments of 64 rows on each side of
lag 0 (lags beyond 95), d = 3 and 4: the checks of the other edges."""
import pytest

import test_gpu_cols as edges

pytestmark = pytest.mark.gpu

SHAPES = [[3, 100, 5], [2, 170, 20], [2, 3, 100, 4]]


@pytest.mark.parametrize("M", SHAPES, ids=lambda m: "x".join(map(str, m)))
def test_two_segments_a_side(kf, gpu, M):
    edges.test_column_walk_edges(kf, gpu, M)


@pytest.mark.parametrize("M", SHAPES, ids=lambda m: "x".join(map(str, m)))
def test_two_segments_a_side_derivatives(kf, gpu, M):
    edges.test_derivative_families_edges(kf, gpu, M)
