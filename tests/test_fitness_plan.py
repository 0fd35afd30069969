"""Launch plans of the float32 fitness (host code, no GPU needed)."""
import pytest

from fitness_plan import plan


@pytest.mark.parametrize("NP,N,P,cols", [(6199, 28, 777, 128), (10933, 30, 404, 128),
                                         (18553, 20, 851, 128), (12365, 32, 194, 64)])
def test_trigonometric_degree_1_avoids_narrow_tiles(NP, N, P, cols):
    """Shapes that wider tiles run 5 to 18 % faster than 32-chromosome ones."""
    assert plan(NP, N, 1, P, basis=3).cols == cols
