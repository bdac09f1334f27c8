"""Host: which kernel the library's default takes, seen from the calls that report it."""
import pytest

from paper_1008_2865_amd import binding as B


@pytest.mark.parametrize("storage", [B.LB_F32, B.LB_F16DEV])
@pytest.mark.parametrize("n, tile", [(256, (64, 16)), (512, (128, 32)), (800, (256, 16)), (1000, (256, 32)), (1000, (128, 8))])
def test_a_tile_shape_of_the_callers_keeps_two_steps_per_launch(n, tile, storage):
    # One step per launch with the same tiles takes 1.1 to 1.3 times as long.
    p = B.make_params(n, n, storage=storage, tile_x=tile[0], tile_y=tile[1], rho_ref=0.7)
    assert B.lb_two_step_shape(p)[:2] == tile
    # Tiles lower than eight rows and double precision run one step per launch.
    low = B.make_params(n, n, storage=storage, tile_x=tile[0], tile_y=4, rho_ref=0.7)
    assert B.lb_two_step_shape(low)[0] == 0
    assert B.lb_two_step_shape(B.make_params(n, n, storage=B.LB_F64, tile_x=tile[0], tile_y=tile[1]))[0] == 0
