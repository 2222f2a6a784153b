"""grad_W_s with one token tile: one to four panels of 64 tokens, whole and ragged, tokens masked so that fewer are left; hidden rows off
the 64 of a wave and the 256 of a workgroup; fewer columns than a step of 32, a ragged last step, and enough of them that a workgroup
walks many; both head orders, both gradient types, written and added to.  Against the fp64 oracle with the tolerances of the
other parity tests."""
import numpy as np
import pytest
import torch

from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T, kept, H_s, V, hv, grad, chunk", [
    (1, 1, 8, 8, False, K.BF16, 0), (64, 64, 64, 40, False, K.F32, 0), (65, 65, 72, 264, False, K.BF16, 256),
    (128, 128, 256, 1000, False, K.BF16, 0), (192, 192, 264, 520, False, K.F32, 256), (256, 256, 1032, 16392, False, K.BF16, 0),
    (256, 256, 2056, 4104, False, K.F32, 0), (256, 10, 1032, 16392, False, K.BF16, 8192), (200, 129, 520, 6152, False, K.F32, 2048),
    (64, 64, 64, 64, True, K.BF16, 0), (129, 129, 192, 1088, True, K.F32, 512), (256, 256, 1088, 16384, True, K.BF16, 0),
    (250, 65, 320, 12352, True, K.F32, 0), (31, 31, 72, 328, True, K.BF16, 256),
    # more than 128 MiB of bf16: stored past the last-level cache
    (64, 64, 1024, 66000, False, K.BF16, 0), (200, 129, 1032, 65544, False, K.BF16, 0)])
def test_grad_W_of_few_tokens(T, kept, H_s, V, hv, grad, chunk):
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=128, H_s=H_s, V=V, w_t_std=0.1, mask="ones")
    data = I.generate(cfg)
    data["mask"] = np.zeros(T, np.uint8)
    data["mask"][np.random.default_rng(T).permutation(T)[:kept]] = 1
    ref = G.run_oracle(cfg, data)
    head = (lambda x: np.ascontiguousarray(x.T)) if hv else (lambda x: x)
    ref["grad_W_s"] = head(ref["grad_W_s"])
    d = [I.to_device(x, I.BF16) for x in (data["h_t"], head(data["W_t"]), data["h_s"], head(data["W_s"]))]
    kw = dict(tau=cfg.tau, kind=cfg.kind, w_layout=K.W_HV if hv else K.W_VH, grad_dtype=grad, vocab_chunk=chunk)
    mask = torch.from_numpy(data["mask"]).cuda()
    out = K.kd_loss_fwd_bwd(*d, mask, **kw)
    G.check(out, ref, "written")
    start = torch.randn(out["grad_W_s"].shape, device="cuda").to(out["grad_W_s"].dtype) * float(np.abs(ref["grad_W_s"]).max())
    added = K.kd_loss_fwd_bwd(*d, mask, grad_W_s=start.clone(), accumulate_grad_W=True, **kw)["grad_W_s"]
    # the same sums as above: rounded once when they are added (fp32), or once there and once here (bf16)
    start, written, added = (x.double() for x in (start, out["grad_W_s"], added))
    unit = 2.0 ** -24 if grad == K.F32 else 2.0 ** -8
    allow = unit * (1 + 2.0 ** -6) * (start.abs() + (1 if grad == K.F32 else 2) * written.abs())
    assert bool(((added - (start + written)).abs() <= allow + 1e-37).all())
