"""Tile and parts of the grad_h_s product, at sizes where the one taken measured at least 4 % ahead of the tile height named beside
it (product and gradh_finish, microseconds a call)."""
import pytest

from paper_2603_01875_amd import kdloss as K


@pytest.mark.parametrize("T, H_t, H_s, V, plan", [
    (4096, 4096, 1024, 151936, (128, 2)),          # 1123; 256 rows 1213
    (4096, 512, 256, 151936, (128, 8)),            # 403; 256 rows 485
    (256, 4096, 1024, 151936, (128, 32)),          # 119; 64 rows 134, 256 rows 141
    (512, 4096, 1024, 151936, (256, 32)),          # 159; 128 rows 167
    (16384, 4096, 1024, 128256, (256, 1)),         # 3363; 128 rows 3898
    (32768, 5120, 4096, 151936, (256, 1))])
def test_grad_h_takes_the_faster_tile(T, H_t, H_s, V, plan):
    assert K.kd_loss_plan_grad_h(K.make_params(T, H_t, H_s, V)) == plan
