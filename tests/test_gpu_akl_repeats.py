"""AKL on the strip loop, whose search adds by atomics in LDS: the same bits from call to call, in both head orders.  Nearly flat
teachers, so that the lanes of a token meet in a few bins."""
import pytest

from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("std, layout, V", [(0.001, K.W_VH, 16200), (0.02, K.W_VH, 16200), (0.02, K.W_HV, 16192)])
def test_akl_repeats_bit_by_bit(std, layout, V):
    import torch
    assert K.kd_loss_plan_loop(K.make_params(600, 2816, 128, V, I.AKL, beta=0.5, w_layout=layout)) == 1
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=600, H_t=2816, H_s=128, V=V, kind=I.AKL, beta=0.5, w_t_std=std)
    data = I.generate(cfg)
    d = {k: G.to_device(data[k], I.BF16) for k in ("h_t", "W_t", "h_s", "W_s")}
    if layout == K.W_HV:
        d.update({k: d[k].t().contiguous() for k in ("W_t", "W_s")})
    mask = torch.from_numpy(data["mask"]).cuda()
    run = lambda: K.kd_loss_fwd_bwd(d["h_t"], d["W_t"], d["h_s"], d["W_s"], mask, kind=I.AKL, beta=0.5, w_layout=layout)
    first = run()
    for _ in range(3):
        again = run()
        for k in ("loss", "per_token_loss", "grad_h_s", "grad_W_s"):
            assert torch.equal(first[k], again[k]), k
