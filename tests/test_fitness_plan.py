"""Launch plans of the float32 fitness (host code, no GPU needed)."""
import pytest

from fitness_plan import REACHES, plan, reached, resident


@pytest.mark.parametrize("NP,N,P,cols", [(6199, 28, 777, 128), (10933, 30, 404, 128),
                                         (18553, 20, 851, 128), (12365, 32, 194, 64)])
def test_trigonometric_degree_1_avoids_narrow_tiles(NP, N, P, cols):
    """Shapes that wider tiles run 5 to 18 % faster than 32-chromosome ones."""
    assert plan(NP, N, 1, P, basis=3).cols == cols


@pytest.mark.parametrize("case,fits", [
    # (NP, N, d, P, options), one workgroup / two launches in us a generation:
    # 5.0 / 8.2, 8.4 / 9.6, 7.9 / 11.4, 9.0 / 10.0
    ((2100, 8, 1, 23, dict(basis=2, error_fn=2)), True), ((1000, 5, 3, 50, {}), True),
    ((300, 6, 4, 32, dict(basis=3)), True), ((512, 7, 4, 50, {}), True),
    # 9.1 / 8.5, 10.6 / 9.3, 9.2 / 8.8, 8.5 / 8.4, 11.7 / 10.5
    ((2000, 8, 1, 64, dict(basis=2)), False), ((1024, 16, 1, 64, dict(basis=2, error_fn=2)), False),
    ((1500, 8, 1, 64, dict(basis=2, error_fn=2)), False), ((2000, 4, 2, 50, {}), False),
    ((1209, 4, 2, 64, dict(basis=2, error_fn=2, selection=1)), False),
    # the best kept need the order too
    ((1209, 4, 2, 64, dict(basis=2, error_fn=2, elite_mode=1)), False)])
def test_one_workgroup_runs_where_it_is_faster(case, fits):
    assert resident(*case[:4], **case[4]) is fits


@pytest.mark.parametrize("name", list(REACHES))
def test_shapes_of_the_gpu_tests_reach_their_kernels(name):
    for basis in (0, 1, 2):
        reached(name, basis)
