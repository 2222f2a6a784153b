"""grad_h_s by every tile height (64, 128, 192, 256 hidden rows) in both head orders: hidden sizes on and off the height, vocabulary
tails off a k-step ([V, H]), one chunk and several (the sums are read again), one part and several, two and three token tiles of
many.  Which tile a case takes is asked of the plan.  Against the fp64 oracle on the tokens that count, with the tolerances of the
other parity tests."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G
from tests.test_gpu_strip_reach import _device_hidden

pytestmark = pytest.mark.gpu

# T, tokens that count, H_s, V, [H, V] heads, the caller's chunk, gradients; tile rows, parts
CASES = [
    (1000, 300, 1104, 664, False, 0, K.BF16, 64, 1), (520, 520, 120, 2704, False, 1024, K.F32, 64, 2),
    (8192, 300, 968, 2296, False, 256, K.F32, 128, 1), (4096, 513, 576, 2720, False, 0, K.BF16, 128, 3),
    (8192, 257, 1048, 2952, False, 256, K.BF16, 192, 1), (7728, 300, 272, 3752, False, 0, K.F32, 192, 4),
    (16384, 300, 928, 2328, False, 0, K.BF16, 256, 1), (32768, 300, 392, 2264, False, 1024, K.F32, 256, 1),
    (3000, 513, 2040, 31992, False, 0, K.BF16, 256, 5), (5406, 513, 392, 13984, False, 8192, K.F32, 256, 5),
    (520, 300, 64, 384, True, 0, K.BF16, 64, 1), (300, 300, 320, 2624, True, 1024, K.F32, 64, 2),
    (8192, 300, 1024, 1728, True, 1024, K.BF16, 128, 1), (4096, 513, 576, 2368, True, 0, K.F32, 128, 3),
    (16384, 300, 704, 1088, True, 256, K.F32, 192, 1), (8192, 257, 576, 3264, True, 0, K.BF16, 192, 2),
    (32768, 300, 448, 2368, True, 1024, K.BF16, 256, 1), (16384, 513, 1024, 1408, True, 512, K.F32, 256, 1),
    (3000, 513, 2048, 32000, True, 0, K.BF16, 256, 5), (5406, 513, 768, 20928, True, 8192, K.F32, 256, 3)]


def _params(T, H_s, V, hv, chunk, grad):
    return K.make_params(T, 128, H_s, V, w_layout=K.W_HV if hv else K.W_VH, vocab_chunk=chunk, grad_dtype=grad)


@pytest.mark.parametrize("T, keep, H_s, V, hv, chunk, grad, rows, parts", CASES)
def test_every_tile_of_grad_h(T, keep, H_s, V, hv, chunk, grad, rows, parts):
    import torch
    assert K.kd_loss_plan_grad_h(_params(T, H_s, V, hv, chunk, grad)) == (rows, parts)
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=keep, H_t=128, H_s=H_s, V=V, w_t_std=0.1)
    few = I.generate(cfg)
    few["mask"] = np.ones(keep, dtype=np.uint8)
    idx = np.unique(np.linspace(0, T - 1, keep).astype(np.int64))
    assert len(idx) == keep
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    mask[torch.from_numpy(idx).cuda()] = 1
    heads = [G.to_device(few[k], I.BF16) for k in ("W_t", "W_s")]
    if hv:
        heads = [w.t().contiguous() for w in heads]
    out = K.kd_loss_fwd_bwd(_device_hidden(few["h_t"], idx, T, I.BF16), heads[0], _device_hidden(few["h_s"], idx, T, I.BF16),
                            heads[1], None if keep == T else mask, w_layout=K.W_HV if hv else K.W_VH, vocab_chunk=chunk,
                            grad_dtype=grad)
    if hv:
        out["grad_W_s"] = out["grad_W_s"].t()
    G.check(out, G.spread_tokens(G.run_oracle(cfg, few), idx, T), f"T={T} kept={keep} H_s={H_s} V={V} hv={hv} chunk={chunk}")
