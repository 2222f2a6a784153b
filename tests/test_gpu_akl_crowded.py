"""AKL on the strip loop where many entries share one cell at the border: their token tile takes a third search pass, the others find
the border in the row pass.  Crowded rows: one entry of 0.9 % of the mass above V - 1 equal ones, which lie on one side of the border,
the tail's.  Beside them, and in the other token tiles, the rows of test_gpu_akl_border.py, whose split is known exactly."""
import numpy as np
import pytest

from oracle import kd_oracle as O
from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G
from tests.test_gpu_akl_border import MU, ROWS, _teachers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("crowded", [range(0), range(300, 304), range(200, 600)])
@pytest.mark.parametrize("V, layout", [(16200, K.W_VH), (16192, K.W_HV)])
def test_crowded_tiles(V, layout, crowded):
    T, H_t, H_s = 600, 2816, 128
    assert K.kd_loss_plan_loop(K.make_params(T, H_t, H_s, V, I.AKL, beta=MU, w_layout=layout)) == 1
    rng = np.random.default_rng(V)
    coarse, fine, head = _teachers(V, rng, True)
    flat = np.zeros((1, V))
    flat[0, 77] = 5.0
    coarse, fine, head = np.vstack([coarse, flat]), np.vstack([fine, 0 * flat]), np.vstack([head, flat > 0])
    row = rng.permutation(T) % ROWS
    row[list(crowded)] = ROWS
    W_t, h_t = np.zeros((V, H_t)), np.zeros((T, H_t))
    W_t[:, 0:2 * ROWS + 2:2], W_t[:, 1:2 * ROWS + 2:2] = coarse.T, fine.T
    h_t[np.arange(T), 2 * row], h_t[np.arange(T), 2 * row + 1] = 1.0, 1.0 / 1024
    h_s, W_s = (I.round_to_bf16(rng.standard_normal(s).astype(np.float32) * k) for s, k in (((T, H_s), 1.0), ((V, H_s), 0.05)))
    z_t = (coarse + fine / 1024)[row]
    z_s = h_s.astype(np.float64) @ W_s.astype(np.float64).T
    p_t, p_s = (np.exp(O.log_softmax(z, 1.0)) for z in (z_t, z_s))
    gap = np.abs(p_t - p_s)
    w_f = (gap * head[row]).sum(1) / gap.sum(1)
    l_f, l_r = O.divergence_rows(z_t, z_s, 1.0, O.FKL)[0], O.divergence_rows(z_t, z_s, 1.0, O.RKL)[0]
    order = (lambda x: np.ascontiguousarray(x.T)) if layout == K.W_HV else (lambda x: x)
    run = lambda: K.kd_loss_fwd_bwd(*[G.to_device(x.astype(np.float32), I.BF16) for x in (h_t, order(W_t), h_s, order(W_s))], None,
                                    kind=I.AKL, beta=MU, w_layout=layout)
    out, again = run(), run()
    np.testing.assert_allclose(G.to_host(out["per_token_loss"]), w_f * l_f + (1 - w_f) * l_r, rtol=1e-4)
    for k in ("per_token_loss", "grad_h_s", "grad_W_s"):
        assert (G.to_host(out[k]) == G.to_host(again[k])).all(), k
