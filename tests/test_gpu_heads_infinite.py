"""An infinite weight belongs to its own vocabulary row.  bf16 heads as [V, H] off the 64-element grid that are read in place: the last
k-step of a row runs on behind the row's end, and what lies there, the first elements of the next row, must not count, whatever it
is (0 x infinity is not 0).  Teacher entries at minus infinity have probability 0, which TVD and the skewed reverse KL give finite losses
and gradients for; infinite student entries finite losses.  Both logit loops, few tokens, hidden sizes 8 to 56 past the grid and
below one k-step, rows at the edges of tiles.  Against the fp64 oracle with the tolerances of the other parity tests."""
import numpy as np
import pytest
import torch

from oracle import kd_oracle as O
from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

SIZES = [(20, 584, 1016, 6008, 0), (300, 1000, 520, 5000, 0), (257, 56, 40, 50264, 0), (768, 2824, 136, 16200, 1), (768, 2872, 200, 16136, 1),
         (512, 40, 2504, 33000, 1)]


def _with_infinities(data, side, H, V):
    """Weights of minus infinity among the first elements of some rows, where the hidden states are positive."""
    h, W = data["h_" + side].copy(), data["W_" + side].copy()
    at = [0, 7, min(8, H - 1), (64 - H % 64) - 1 if H > 64 else H - 1]
    h[:, at] = np.abs(h[:, at]) + 0.125
    for row, k in zip((0, 1, 63, 64, 127, 128, 192, 384, 1000, 1001, V // 2, V - 1), 3 * at):
        W[row, k] = -np.inf
    return dict(data, **{"h_" + side: I.round_to_bf16(h), "W_" + side: W})


@pytest.mark.parametrize("kind", [I.TVD, I.SKEW_RKL])
@pytest.mark.parametrize("T, H_t, H_s, V, loop", SIZES)
def test_infinite_teacher_entries(T, H_t, H_s, V, loop, kind):
    assert K.kd_loss_plan_loop(K.make_params(T, H_t, H_s, V, kind, beta=0.5)) == loop
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, kind=kind, beta=0.5, w_t_std=0.05, mask="ones")
    data = _with_infinities(I.generate(cfg), "t", H_t, V)
    with np.errstate(invalid="ignore"):
        ref = G.run_oracle(cfg, data)
        allow = G.tvd_tie_allowance(cfg, data) if kind == I.TVD else None
    assert np.isfinite(ref["per_token_loss"]).all() and np.isfinite(ref["grad_W_s"]).all()
    G.check(G.run_gpu(cfg, data), ref, "infinite teacher entries", allow)


@pytest.mark.parametrize("T, H_t, H_s, V, loop", SIZES)
def test_infinite_student_entries(T, H_t, H_s, V, loop):
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, kind=I.TVD, w_t_std=0.05, mask="ones")
    data = _with_infinities(I.generate(cfg), "s", H_s, V)
    want = O.divergence_rows(*(data["h_" + s].astype(np.float64) @ data["W_" + s].astype(np.float64).T for s in "ts"), 1.0, O.TVD)[0]
    assert np.isfinite(want).all()
    got = K.kd_loss_fwd(*[G.to_device(data[k], I.BF16) for k in ("h_t", "W_t", "h_s", "W_s")], None, kind=I.TVD)["per_token_loss"]
    np.testing.assert_allclose(G.to_host(got), want, rtol=2e-3, atol=5e-7)


@pytest.mark.parametrize("T, H_t, H_s, V, hv", [(20, 584, 1016, 6008, False), (300, 1000, 520, 5000, False), (300, 512, 256, 1024, True),
                                                (600, 2824, 136, 16200, False), (600, 2816, 128, 16200, False), (600, 2816, 128, 16192, True)])
def test_infinite_teacher_entries_beside_padding(T, H_t, H_s, V, hv):
    """Masked tokens and the rest of the last token tile, which the copies of the hidden states fill up: their dL/dz is 0 there, too."""
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, kind=I.SKEW_RKL, beta=0.5, w_t_std=0.05, mask="bernoulli10")
    data = _with_infinities(I.generate(cfg), "t", H_t, V)
    with np.errstate(invalid="ignore"):
        ref = G.run_oracle(cfg, data)
    head = (lambda x: np.ascontiguousarray(x.T)) if hv else (lambda x: x)
    d = [G.to_device(x, I.BF16) for x in (data["h_t"], head(data["W_t"]), data["h_s"], head(data["W_s"]))]
    out = K.kd_loss_fwd_bwd(*d, torch.from_numpy(data["mask"]).cuda(), tau=cfg.tau, kind=cfg.kind, beta=0.5, w_layout=K.W_HV if hv else K.W_VH)
    if hv:
        out["grad_W_s"] = out["grad_W_s"].t()
    G.check(out, ref, "beside padding")
