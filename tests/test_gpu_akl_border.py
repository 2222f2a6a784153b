"""Where AKL's border between head and tail lies: on a grid, one cell above the entry that passes mu.  Entries of one cell lie on one
side.  The eight-wave loop's grid has 17^4 cells from 40 below a token's largest base-2 teacher log-probability to 1e-3 above
it; the strip loop's 44^3, from log2((1 - mu) / V) - 1 where that is higher.  The teachers here have two entries close together at
the border, each of several per cent of the mass, so a border on another grid shows in the token's loss; on rows whose entries
stay clear of a cell's edge (fp32 rounding of log-probabilities: 1e-5 at 40, a fiftieth of a cell; 2e-6 at 16, a seventieth) the split
is known exactly."""
import numpy as np
import pytest

from oracle import kd_oracle as O
from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

ROWS, ENTRIES, MU = 60, 24, 0.5


def _teachers(V, rng, strip):
    """Logits [ROWS, V] as the sum of a coarse and a fine part / 1024, both bf16 values, and the split on the grid."""
    coarse, fine, head = np.zeros((ROWS, V)), np.zeros((ROWS, V)), np.zeros((ROWS, V), bool)
    bf16 = lambda x: I.round_to_bf16(np.asarray(x, np.float32)).astype(np.float64)
    done = 0
    while done < ROWS:
        c, f = np.full(V, -20.0), np.zeros(V)
        at = rng.permutation(V)[:ENTRIES]
        c[at], f[at] = bf16(rng.uniform(3.0, 5.0, ENTRIES)), bf16(rng.uniform(-64, 64, ENTRIES))
        z = c + f / 1024
        # the entry that passes mu moves to just below the last one of the head
        order = np.argsort(-z)
        p = np.exp(O.log_softmax(z[None], 1.0)[0])
        k = int((np.cumsum(p[order]) <= MU).sum())
        c[order[k]] = c[order[k - 1]]
        f[order[k]] = bf16([f[order[k - 1]] - rng.uniform(0.02, 0.9) * 4.8e-4 * np.log(2) * 1024])[0]
        z = c + f / 1024
        lt = O.log_softmax(z[None], 1.0)[0] / np.log(2)
        p = 2.0 ** lt
        order = np.argsort(-z)
        low = max(lt.max() - 40, np.log2((1 - MU) / V) - 1) if strip else lt.max() - 40
        at_cell = (lt - low) / ((lt.max() + 1e-3 - low) / (44 ** 3 if strip else 17 ** 4))
        mass = np.cumsum(p[order])
        k = int((mass <= MU).sum())                    # entry k passes mu
        near = np.abs(at_cell[at] - np.round(at_cell[at])).min() < 0.05 or np.abs(mass - MU).min() < 1e-3
        if near or z[order[k - 1]] - z[order[k]] > 4.8e-4 or k < 3:
            continue
        cut = np.floor(at_cell)
        coarse[done], fine[done], head[done] = c, f, cut > cut[order[k]]
        done += 1
    return coarse, fine, head


@pytest.mark.parametrize("loop, T, H_t, H_s, V, layout", [
    (0, 300, 128, 64, 2000, K.W_VH), (0, 200, 128, 64, 1984, K.W_HV), (1, 600, 2816, 128, 16200, K.W_VH),
    (1, 600, 2816, 128, 16192, K.W_HV)])
def test_border_lies_on_the_grid(loop, T, H_t, H_s, V, layout):
    import torch
    assert K.kd_loss_plan_loop(K.make_params(T, H_t, H_s, V, I.AKL, beta=MU, w_layout=layout)) == loop
    rng = np.random.default_rng(V)
    coarse, fine, head = _teachers(V, rng, loop == 1)
    row = rng.permutation(T) % ROWS                    # token -> row of the teacher
    W_t, h_t = np.zeros((V, H_t)), np.zeros((T, H_t))
    W_t[:, 0:2 * ROWS:2], W_t[:, 1:2 * ROWS:2] = coarse.T, fine.T
    h_t[np.arange(T), 2 * row], h_t[np.arange(T), 2 * row + 1] = 1.0, 1.0 / 1024
    h_s, W_s = (I.round_to_bf16(rng.standard_normal(s).astype(np.float32) * k) for s, k in (((T, H_s), 1.0), ((V, H_s), 0.05)))
    z_t = (coarse + fine / 1024)[row]
    z_s = h_s.astype(np.float64) @ W_s.astype(np.float64).T
    gap = np.abs(np.exp(O.log_softmax(z_t, 1.0)) - np.exp(O.log_softmax(z_s, 1.0)))
    w_f = (gap * head[row]).sum(1) / gap.sum(1)
    l_f, l_r = O.divergence_rows(z_t, z_s, 1.0, O.FKL)[0], O.divergence_rows(z_t, z_s, 1.0, O.RKL)[0]
    order = (lambda x: np.ascontiguousarray(x.T)) if layout == K.W_HV else (lambda x: x)
    out = K.kd_loss_fwd_bwd(*[G.to_device(x.astype(np.float32), I.BF16) for x in (h_t, order(W_t), h_s, order(W_s))], None,
                            kind=I.AKL, beta=MU, w_layout=layout)
    ptl = G.to_host(out["per_token_loss"])
    ref = w_f * l_f + (1 - w_f) * l_r
    # an entry on the other side moves w_f by a few per cent and the loss by that much of the difference of the two KLs
    share = np.where(head[row], gap, 0).max(1) / gap.sum(1)
    assert np.median(share * np.abs(l_f - l_r) / ref) > 0.01
    np.testing.assert_allclose(ptl, ref, rtol=1e-4)
