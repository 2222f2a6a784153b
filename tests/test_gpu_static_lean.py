"""The static entry point near the limit of its array, where it falls back to its smallest plan: eight ranges of the
vocabulary per token tile, copies with the rows that there are.  Against the fp64 oracle on the tokens that count, with the
tolerances of the other parity tests."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T, H_t, H_s, V, kind, hv, fp8, chunk, keep", [
    (1060, 44216, 64, 240, I.RKL, True, False, 0, 1060), (12687, 576, 448, 11520, I.AKL, True, False, 0, 300),
    (47615, 512, 128, 3720, I.RKL, False, True, 0, 520), (32768, 256, 256, 32000, I.FKL, False, False, 0, 290),
    (2, 320, 8696, 7112, I.SKEW_RKL, False, False, 256, 2)])
def test_smallest_plan_of_the_static_entry_point(T, H_t, H_s, V, kind, hv, fp8, chunk, keep):
    import torch
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, kind=kind, w_t_std=0.1)
    data, few, idx = G.few_tokens(cfg, keep)
    kw = {}
    if fp8:
        q = G.fp8_teacher(data)
        few.update(h_t=q["h_t"][idx], W_t=q["W_t"])
        kw = dict(flags=K.FLAG_TEACHER_FP8, teacher_scale=q["teacher_scale"])
    lay = lambda w: np.ascontiguousarray(w.T) if hv else w
    h_t, W_t = ((torch.from_numpy(q["q_" + k]).cuda() for k in ("h_t", "W_t")) if fp8 else
                (G.to_device(data["h_t"], I.BF16), G.to_device(lay(data["W_t"]), I.BF16)))
    h_s, W_s = G.to_device(data["h_s"], I.BF16), G.to_device(lay(data["W_s"]), I.BF16)
    p = K.make_params(T, H_t, H_s, V, kind, cfg.tau, cfg.beta, w_layout=K.W_HV if hv else K.W_VH, vocab_chunk=chunk, **kw)
    out = dict(loss=torch.full((1,), 7.0, device="cuda"), per_token_loss=torch.full((T,), 7.0, device="cuda"),
               grad_h_s=torch.full((T, H_s), 7.0, device="cuda", dtype=torch.bfloat16),
               grad_W_s=torch.full(W_s.shape, 7.0, device="cuda", dtype=torch.bfloat16))
    K.kd_loss_fwd_bwd_static_raw(p, h_t, W_t, h_s, W_s, torch.from_numpy(data["mask"]).cuda(), out["loss"],
                                 out["per_token_loss"], out["grad_h_s"], out["grad_W_s"])
    torch.cuda.synchronize()
    extra = None
    if kind == I.AKL:
        extra = G.spread_tokens(G.akl_allowance(cfg, few), idx, T)
    ref = G.spread_tokens(G.run_oracle(cfg, few), idx, T)
    if hv:
        out["grad_W_s"] = out["grad_W_s"].t()
    G.check(out, ref, f"T={T} H={H_t},{H_s} V={V} kind={kind}", extra)
