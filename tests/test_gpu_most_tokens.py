"""The largest token count that the library takes (2^22), nearly all tokens masked, through the packed hidden states of
the strip loop: 65536 panels of 64 tokens, more than a grid has along its second axis.  Against the fp64 oracle on the
tokens that count."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1 << 22, (1 << 21) + 1])
def test_most_tokens(T):
    import torch
    from paper_2603_01875_amd import kdloss as K
    keep, H_t, H_s, V = 300, 1280, 64, 192
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=keep, H_t=H_t, H_s=H_s, V=V, w_t_std=0.1)
    few = I.generate(cfg)
    few["mask"] = np.ones(keep, dtype=np.uint8)
    idx = np.unique(np.concatenate([[0, T - 1], np.linspace(1, T - 2, keep - 2).astype(np.int64)]))
    assert len(idx) == keep
    at = torch.from_numpy(idx).cuda()

    def hidden(x):
        full = torch.zeros(T, x.shape[1], dtype=torch.bfloat16, device="cuda")
        full[at] = G.to_device(x, I.BF16)
        return full
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    mask[at] = 1
    out = K.kd_loss_fwd_bwd(hidden(few["h_t"]), G.to_device(few["W_t"], I.BF16), hidden(few["h_s"]),
                            G.to_device(few["W_s"], I.BF16), mask)
    assert torch.count_nonzero(out["per_token_loss"]) <= keep and torch.count_nonzero(out["grad_h_s"][mask == 0]) == 0
    out["per_token_loss"], out["grad_h_s"] = out["per_token_loss"][at], out["grad_h_s"][at]
    G.check(out, G.run_oracle(cfg, few), f"T={T}")
