"""The strip loop at the edges of the sizes that the library gives to it: one k-step and odd numbers of k-steps, last
vocabulary tiles of 8 .. 192 rows, chunks that 192 does not divide, one token more or less than a token tile, token tiles
that fours do not divide, fp32 and padded operands, the adding form, whole tiles strided over the workgroups (29 token tiles
x 43 vocabulary tiles).  Neighbouring sizes on the other side of the line run the eight-wave loop.  Against the fp64 oracle
on the tokens that count, with the tolerances of the other parity tests."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _device_hidden(x, idx, T, dtype):
    import torch
    full = torch.zeros(T, x.shape[1], dtype=torch.float32 if dtype == I.F32 else torch.bfloat16, device="cuda")
    full[torch.from_numpy(idx).cuda()] = G.to_device(x, dtype)
    return full


def _run(T, keep, H_t, H_s, V, kind, chunk, dtype, loop):
    """T tokens of which `keep` count (the first, the last, the rest evenly between); the others are zeros and masked."""
    import torch
    from paper_2603_01875_amd import kdloss as K
    p = K.make_params(T, H_t, H_s, V, kind, beta=0.5, in_dtype=K.F32 if dtype == I.F32 else K.BF16, vocab_chunk=chunk)
    assert K.kd_loss_plan_loop(p) == loop
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=keep, H_t=H_t, H_s=H_s, V=V, kind=kind, w_t_std=0.1, dtype=dtype)
    few = I.generate(cfg)
    few["mask"] = np.ones(keep, dtype=np.uint8)
    idx = np.unique(np.linspace(0, T - 1, keep).astype(np.int64))
    assert len(idx) == keep
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    mask[torch.from_numpy(idx).cuda()] = 1
    out = K.kd_loss_fwd_bwd(_device_hidden(few["h_t"], idx, T, dtype), G.to_device(few["W_t"], dtype),
                            _device_hidden(few["h_s"], idx, T, dtype), G.to_device(few["W_s"], dtype),
                            None if keep == T else mask, tau=cfg.tau, kind=kind, beta=cfg.beta, vocab_chunk=chunk)
    extra = (G.tvd_tie_allowance(cfg, few) if kind == I.TVD else G.akl_allowance(cfg, few) if kind == I.AKL else None)
    if extra is not None:
        extra = G.spread_tokens(dict(extra, per_token_loss=extra.get("per_token_loss", np.zeros(keep))), idx, T)
    G.check(out, G.spread_tokens(G.run_oracle(cfg, few), idx, T),
            f"T={T} kept={keep} H={H_t},{H_s} V={V} kind={kind} chunk={chunk}", extra)


@pytest.mark.parametrize("T, keep, H_t, H_s, V, kind, chunk, dtype", [
    (65536, 300, 1216, 64, 184, I.FKL, 0, I.BF16), (65536, 257, 640, 128, 136, I.JSD, 0, I.BF16),
    (65536, 3, 1216, 64, 192, I.RKL, 0, I.BF16), (65536, 511, 2112, 192, 264, I.FKL, 256, I.BF16),
    (16384, 513, 704, 64, 584, I.FKL, 512, I.BF16), (16384, 300, 1088, 320, 768, I.TVD, 512, I.BF16),
    (16000, 1300, 1000, 72, 712, I.SKEW_RKL, 256, I.BF16), (512, 512, 1024, 64, 24008, I.FKL, 8192, I.BF16),
    (257, 257, 576, 64, 24200, I.RKL, 0, I.BF16), (513, 513, 960, 192, 16200, I.SKEW_FKL, 4864, I.BF16),
    (600, 600, 2816, 128, 16200, I.AKL, 0, I.BF16), (511, 511, 520, 136, 24392, I.FKL, 0, I.F32),
    (16384, 270, 1024, 72, 616, I.JSD, 256, I.F32), (7400, 7400, 1024, 64, 8256, I.FKL, 0, I.BF16)])
def test_strip_loop_at_its_edges(T, keep, H_t, H_s, V, kind, chunk, dtype):
    _run(T, keep, H_t, H_s, V, kind, chunk, dtype, 1)


@pytest.mark.parametrize("T, keep, H_t, H_s, V, kind", [
    (65536, 300, 1216, 64, 128, I.FKL), (16384, 513, 320, 64, 584, I.FKL), (512, 512, 1024, 64, 16384, I.FKL),
    (256, 256, 1024, 64, 24008, I.JSD), (600, 600, 64, 128, 16328, I.AKL), (7400, 520, 256, 128, 8256, I.RKL)])
def test_eight_wave_loop_beside_the_line(T, keep, H_t, H_s, V, kind):
    _run(T, keep, H_t, H_s, V, kind, 0, I.BF16, 0)


def test_strip_loop_adds_teachers_at_its_edges():
    """The gradient kernel's adding form on chunks that 192 does not divide: two halves of one teacher."""
    import torch
    from paper_2603_01875_amd import kdloss as K
    T, H_t, H_s, V = 300, 1024, 64, 24008
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, w_t_std=0.1)
    assert K.kd_loss_plan_loop(K.make_params(T, H_t, H_s, V, vocab_chunk=8704)) == 1
    data = I.generate(cfg)
    d = {k: G.to_device(data[k], I.BF16) for k in ("h_t", "W_t", "h_s", "W_s")}
    out = K.kd_loss_fwd_bwd_multi([d["h_t"]] * 2, [d["W_t"]] * 2, [0.5, 0.5], d["h_s"], d["W_s"],
                                  torch.from_numpy(data["mask"]).cuda(), vocab_chunk=8704)
    G.check(out, G.run_oracle(cfg, data), "two halves of one teacher")
