"""tests/test_gpu_product_tiles.py reaches every tile of the grad_h_s product, asked on the host."""
from paper_2603_01875_amd import kdloss as K
from tests.test_gpu_product_tiles import CASES, _params


def test_every_tile_is_reached():
    seen = set()
    for T, keep, H_s, V, hv, chunk, grad, rows, parts in CASES:
        p = _params(T, H_s, V, hv, chunk, grad)
        assert K.kd_loss_plan_grad_h(p) == (rows, parts), (T, H_s, V, hv, chunk)
        seen.add((hv, rows, K.kd_loss_plan_info(p)[0] < V, parts > 1))
    assert {(hv, rows) for hv, rows, _, _ in seen} == {(hv, rows) for hv in (False, True) for rows in (64, 128, 192, 256)}
    for hv in (False, True):       # chunks: one, several; parts: one, several
        assert {(several, split) for order, rows, several, split in seen if order == hv and rows == 256} >= \
            {(False, True), (True, False), (True, True)}
