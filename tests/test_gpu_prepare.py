"""Operands that are re-packed before the logit passes: hidden sizes off the 64-element grid on both sides of the
512-element blocks of the copy, row counts that 16 and 64 do not divide, fp32 splits, [H,V] heads through the
transposing copy.  Against the fp64 oracle with the tolerances of the other parity tests."""
import numpy as np
import pytest

from oracle import kd_oracle as O
from paper_2603_01875_amd import inputs as I
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["vh", "hv"])
@pytest.mark.parametrize("T, H_t, H_s, V, dtype", [(33, 8, 520, 72, I.BF16), (300, 504, 72, 1032, I.BF16),
                                                   (17, 168, 8, 264, I.F32), (270, 64, 176, 520, I.F32)])
def test_repacked_operands(T, H_t, H_s, V, dtype, layout):
    import torch
    from paper_2603_01875_amd import kdloss as K
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, w_t_std=0.1, dtype=dtype,
                   mask="bernoulli10")
    data = I.generate(cfg)
    data["mask"][0] = 1
    if layout == "vh":
        G.check(G.run_gpu(cfg, data), G.run_oracle(cfg, data), "vh")
        return
    hv = {k: np.ascontiguousarray(data[k].T) for k in ("W_t", "W_s")}
    ref = O.kd_loss_fwd_bwd(data["h_t"], hv["W_t"], data["h_s"], hv["W_s"], data["mask"], cfg.tau, cfg.kind, cfg.beta,
                            O.W_HV)
    ref["per_token_loss"] = ref["per_token_loss"] * (data["mask"] != 0)
    dev = lambda x: G.to_device(x, dtype)
    out = K.kd_loss_fwd_bwd(dev(data["h_t"]), dev(hv["W_t"]), dev(data["h_s"]), dev(hv["W_s"]),
                            torch.from_numpy(data["mask"]).cuda(), w_layout=K.W_HV)
    G.check(out, ref, "hv")
