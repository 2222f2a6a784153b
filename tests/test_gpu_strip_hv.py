"""The strip loop on heads kept as [H, V] and read in place: one k-step and odd numbers of k-steps, last vocabulary tiles of
64, 128 and 192 rows, chunks that 192 does not divide, one token more or less than a token tile, every kind of epilogue, the
adding form.  Against the fp64 oracle on the tokens that count, with the tolerances of the other parity tests."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G
from tests.test_gpu_strip_reach import _device_hidden

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T, keep, H_t, H_s, V, kind, chunk", [
    (65536, 300, 1216, 64, 192, I.FKL, 0), (65536, 257, 640, 128, 192, I.JSD, 0), (65536, 511, 2112, 192, 320, I.FKL, 256),
    (16384, 513, 704, 64, 576, I.RKL, 512), (16384, 300, 1088, 320, 768, I.TVD, 512), (513, 513, 960, 192, 16192, I.SKEW_FKL, 4864),
    (16000, 270, 1024, 64, 704, I.SKEW_RKL, 256), (600, 600, 2816, 128, 16192, I.AKL, 0), (257, 257, 576, 64, 24192, I.RKL, 0)])
def test_strip_loop_on_hidden_major_heads(T, keep, H_t, H_s, V, kind, chunk):
    import torch
    assert K.kd_loss_plan_loop(K.make_params(T, H_t, H_s, V, kind, beta=0.5, vocab_chunk=chunk, w_layout=K.W_HV)) == 1
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=keep, H_t=H_t, H_s=H_s, V=V, kind=kind, w_t_std=0.1)
    few = I.generate(cfg)
    few["mask"] = np.ones(keep, dtype=np.uint8)
    idx = np.unique(np.linspace(0, T - 1, keep).astype(np.int64))
    assert len(idx) == keep
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    mask[torch.from_numpy(idx).cuda()] = 1
    heads = [G.to_device(few[k], I.BF16).t().contiguous() for k in ("W_t", "W_s")]
    out = K.kd_loss_fwd_bwd(_device_hidden(few["h_t"], idx, T, I.BF16), heads[0], _device_hidden(few["h_s"], idx, T, I.BF16),
                            heads[1], None if keep == T else mask, tau=cfg.tau, kind=kind, beta=cfg.beta, vocab_chunk=chunk,
                            w_layout=K.W_HV)
    out["grad_W_s"] = out["grad_W_s"].t()
    extra = G.tvd_tie_allowance(cfg, few) if kind == I.TVD else G.akl_allowance(cfg, few) if kind == I.AKL else None
    if extra is not None:
        extra = G.spread_tokens(dict(extra, per_token_loss=extra.get("per_token_loss", np.zeros(keep))), idx, T)
    G.check(out, G.spread_tokens(G.run_oracle(cfg, few), idx, T),
            f"T={T} kept={keep} H={H_t},{H_s} V={V} kind={kind} chunk={chunk}", extra)


def test_strip_loop_on_hidden_major_heads_adds_teachers():
    import torch
    T, H_t, H_s, V = 300, 1024, 64, 24000
    assert K.kd_loss_plan_loop(K.make_params(T, H_t, H_s, V, vocab_chunk=8704, w_layout=K.W_HV)) == 1
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, w_t_std=0.1)
    data = I.generate(cfg)
    h_t, h_s = G.to_device(data["h_t"], I.BF16), G.to_device(data["h_s"], I.BF16)
    W_t, W_s = (G.to_device(data[k], I.BF16).t().contiguous() for k in ("W_t", "W_s"))
    out = K.kd_loss_fwd_bwd_multi([h_t] * 2, [W_t] * 2, [0.5, 0.5], h_s, W_s, torch.from_numpy(data["mask"]).cuda(),
                                  vocab_chunk=8704, w_layout=K.W_HV)
    out["grad_W_s"] = out["grad_W_s"].t()
    G.check(out, G.run_oracle(cfg, data), "two halves of one teacher")
