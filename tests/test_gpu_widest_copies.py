"""The most tokens that the library takes with wide hidden states: packed copies of 2^35 elements and more (64 GiB), or 2^34 of
grad_h_s, whose blocks are more than a grid has threads for along one axis.  Nearly all tokens masked; against the fp64 oracle on
the others.  The quantiser at such sizes, against itself on a piece."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype, H_t, H_s, V", [(I.BF16, 8192, 64, 192), (I.F32, 2736, 64, 192), (I.BF16, 8192, 64, 128), (I.BF16, 64, 4096, 64)])
def test_widest_copies(dtype, H_t, H_s, V):
    import torch
    T, keep = 1 << 22, 300
    p = K.make_params(T, H_t, H_s, V, in_dtype=K.F32 if dtype == I.F32 else K.BF16)
    assert K.kd_loss_plan_loop(p) == (V == 192)
    torch.cuda.empty_cache()
    es = 4 if dtype == I.F32 else 2
    if torch.cuda.mem_get_info()[0] < K.kd_loss_workspace_size(p) + T * (H_t + 2 * H_s) * es + (4 << 30):
        pytest.skip("not enough memory on this GPU")
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=keep, H_t=H_t, H_s=H_s, V=V, w_t_std=0.1, dtype=dtype)
    few = I.generate(cfg)
    few["mask"] = np.ones(keep, dtype=np.uint8)
    idx = np.unique(np.concatenate([[0, T - 1], np.linspace(1, T - 2, keep - 2).astype(np.int64)]))
    assert len(idx) == keep
    at = torch.from_numpy(idx).cuda()

    def hidden(x):
        x = G.to_device(x, dtype)
        full = torch.empty(T, x.shape[1], dtype=x.dtype, device="cuda")     # (masked rows are never read)
        full[at] = x
        return full
    mask = torch.zeros(T, dtype=torch.uint8, device="cuda")
    mask[at] = 1
    out = K.kd_loss_fwd_bwd(hidden(few["h_t"]), G.to_device(few["W_t"], dtype), hidden(few["h_s"]), G.to_device(few["W_s"], dtype),
                            mask)
    out.pop("workspace", None)
    assert torch.count_nonzero(out["per_token_loss"]) <= keep
    assert sum(int(torch.count_nonzero(rows.any(1))) for rows in out["grad_h_s"].split(1 << 18)) <= keep
    out["per_token_loss"], out["grad_h_s"] = out["per_token_loss"][at], out["grad_h_s"][at]
    G.check(out, G.run_oracle(cfg, few), f"T={T} H_t={H_t} dtype={dtype} V={V}")
    del out
    torch.cuda.empty_cache()


def test_quantiser_beyond_one_axis():
    import torch
    torch.cuda.empty_cache()
    piece, n = 1 << 24, (1 << 35) + (1 << 24)
    if torch.cuda.mem_get_info()[0] < 3 * n + (4 << 30):
        pytest.skip("not enough memory on this GPU")
    x = torch.randn(piece, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3)).to(torch.bfloat16)
    code = K.quantize_e4m3(x, 0.01)
    q = K.quantize_e4m3(x.repeat(n // piece), 0.01)
    assert all(torch.equal(part, code) for part in q.split(piece))
    del q
    torch.cuda.empty_cache()
