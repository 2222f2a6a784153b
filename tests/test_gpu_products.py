"""The backward products (csrc/kd_products.hip) at the edges of their tiles: hidden sizes around every tile height of grad_W_s and
the 16-row blocks (grad_h_s takes its 64-row tile at these sizes; its others: test_gpu_product_tiles.py), vocabulary chunks around 256 columns and around a 64-column k-step, one token tile and several, both head
orders, both gradient types, written and added to.  Against the fp64 oracle with the tolerances of the other parity tests."""
import numpy as np
import pytest
import torch

from oracle import kd_oracle as O
from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T, H_s, V, hv, grad, chunk", [
    (1, 8, 8, False, K.BF16, 0), (64, 64, 256, False, K.F32, 0), (65, 72, 264, False, K.BF16, 256),
    (257, 128, 520, False, K.BF16, 256), (255, 136, 1032, False, K.F32, 512), (300, 192, 776, False, K.BF16, 256),
    (513, 200, 4104, False, K.BF16, 2048), (260, 256, 1336, False, K.BF16, 768), (100, 264, 2056, False, K.F32, 0),
    (777, 520, 1160, False, K.F32, 512), (530, 1032, 712, False, K.BF16, 256), (129, 16, 16392, False, K.BF16, 0),
    (300, 64, 320, True, K.BF16, 256), (257, 192, 1088, True, K.F32, 512), (65, 256, 640, True, K.BF16, 256),
    (513, 576, 448, True, K.BF16, 0), (90, 72, 328, True, K.BF16, 256), (520, 1024, 832, True, K.F32, 256)])
def test_products_at_tile_edges(T, H_s, V, hv, grad, chunk):
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=max(128, H_s), H_s=H_s, V=V, w_t_std=0.1,
                   mask="bernoulli10" if T > 1 else "ones")
    data = I.generate(cfg)
    if data["mask"] is not None:
        data["mask"][0] = 1
    ref = G.run_oracle(cfg, data)
    head = (lambda x: np.ascontiguousarray(x.T)) if hv else (lambda x: x)
    if hv:
        ref["grad_W_s"] = ref["grad_W_s"].T
    d = [I.to_device(x, I.BF16) for x in (data["h_t"], head(data["W_t"]), data["h_s"], head(data["W_s"]))]
    mask = None if data["mask"] is None else torch.from_numpy(data["mask"]).cuda()
    kw = dict(tau=cfg.tau, kind=cfg.kind, w_layout=K.W_HV if hv else K.W_VH, grad_dtype=grad, vocab_chunk=chunk)
    what = f"T={T} H_s={H_s} V={V} hv={hv} grad={grad} chunk={chunk}"
    out = K.kd_loss_fwd_bwd(*d, mask, **kw)
    G.check(out, ref, what)
    # added to itself: one rounding behind the whole sum, so twice the gradient exactly where it is fp32
    twice = K.kd_loss_fwd_bwd(*d, mask, grad_W_s=out["grad_W_s"].clone(), accumulate_grad_W=True, **kw)["grad_W_s"]
    if grad == K.F32:
        assert torch.equal(twice, 2 * out["grad_W_s"]), what
    else:       # the stored gradient and the sum are each half a unit (2^-9) off
        assert torch.allclose(twice.float(), 2 * out["grad_W_s"].float(), rtol=2 ** -7, atol=0), what
