"""Small sizes at the edges of the strip loop's tiles (192 x 256 logit tiles): one k-step and odd numbers of k-steps
per phase, last vocabulary tiles of 8 .. 192 rows, chunks that 192 does not divide, one row more or less than a token tile,
token tiles that fours do not divide, fewer vocabulary tiles than splits, fp32 and padded operands.  As small as they are,
the library gives them to the eight-wave loop; test_gpu_strip_reach.py has the same edges at sizes that reach the strip loop.
Against the fp64 oracle with the tolerances of the other parity tests."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T, H_t, H_s, V, kind, chunk, dtype", [
    (400, 64, 64, 8, I.FKL, 0, I.BF16), (257, 64, 192, 184, I.FKL, 256, I.BF16), (511, 192, 64, 192, I.JSD, 256, I.BF16),
    (513, 320, 128, 200, I.RKL, 256, I.BF16), (7400, 64, 64, 968, I.FKL, 512, I.BF16), (600, 128, 320, 1160, I.FKL, 512, I.BF16),
    (1290, 192, 192, 776, I.TVD, 256, I.BF16), (300, 72, 200, 2056, I.SKEW_RKL, 768, I.BF16),
    (520, 256, 64, 3848, I.AKL, 1024, I.BF16), (2100, 64, 64, 584, I.SKEW_FKL, 256, I.BF16),
    (330, 24, 40, 392, I.FKL, 256, I.F32), (270, 136, 64, 1544, I.JSD, 512, I.F32)])
def test_strip_loop_edges(T, H_t, H_s, V, kind, chunk, dtype):
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, kind=kind, w_t_std=0.1, dtype=dtype,
                   mask="bernoulli10")
    data = I.generate(cfg)
    data["mask"][0] = 1
    if H_t == H_s == 64 and T < 1000:
        data["mask"][3:] = 0                     # three tokens left of two token tiles
    extra = G.tvd_tie_allowance(cfg, data) if kind == I.TVD else G.akl_allowance(cfg, data) if kind == I.AKL else None
    ref = G.run_oracle(cfg, data)
    G.check(G.run_gpu(cfg, data, vocab_chunk=chunk), ref, f"T={T} H={H_t},{H_s} V={V} kind={kind} chunk={chunk}", extra)


def test_strip_loop_adds_the_teachers_of_a_call():
    """The gradient kernel's adding form, on chunks that 192 does not divide: two equal halves of one teacher."""
    from paper_2603_01875_amd import kdloss as K
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=300, H_t=128, H_s=64, V=1096, w_t_std=0.1)
    data = I.generate(cfg)
    d = {k: I.to_device(data[k], I.BF16) for k in ("h_t", "W_t", "h_s", "W_s")}
    import torch
    mask = torch.from_numpy(data["mask"]).cuda()
    out = K.kd_loss_fwd_bwd_multi([d["h_t"]] * 2, [d["W_t"]] * 2, [0.5, 0.5], d["h_s"], d["W_s"], mask, vocab_chunk=512)
    G.check(out, G.run_oracle(cfg, data), "two halves of one teacher")
    assert np.isfinite(G.to_host(out["grad_W_s"])).all()
