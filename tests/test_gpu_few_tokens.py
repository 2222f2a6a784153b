"""At most 192 tokens: waves whose 64 tokens of the tile are not there only load.  Token counts around the 64 of a wave pair, masks that
leave fewer, one or none, every divergence, both head orders, fp32, the fp8 teacher, two teachers, several chunks and ranges of several
tiles; a workspace full of NaNs, so that nothing may be read that no wave has written.  Against the fp64 oracle with the tolerances of
the other parity tests."""
import numpy as np
import pytest
import torch

from oracle import kd_oracle as O
from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _nan_workspace(n):
    return torch.full((n,), 0xff, dtype=torch.uint8, device="cuda")


@pytest.mark.parametrize("T, kept, H_t, H_s, V, kind, hv, dtype, chunk", [
    (1, 1, 64, 64, 264, I.FKL, False, I.BF16, 0), (64, 64, 128, 64, 4104, I.JSD, False, I.BF16, 1024), (65, 65, 192, 128, 1000, I.RKL, False, I.BF16, 0),
    (127, 63, 128, 72, 2056, I.TVD, False, I.BF16, 256), (128, 128, 256, 64, 40008, I.FKL, False, I.BF16, 0), (129, 1, 96, 40, 520, I.SKEW_FKL, False, I.F32, 0),
    (192, 192, 128, 64, 2440, I.AKL, False, I.BF16, 512), (150, 0, 128, 64, 1544, I.FKL, False, I.BF16, 512), (191, 100, 128, 64, 1984, I.AKL, True, I.BF16, 0),
    (64, 64, 192, 128, 2048, I.SKEW_RKL, True, I.BF16, 512), (100, 30, 64, 64, 8192, I.JSD, True, I.BF16, 0), (192, 0, 64, 64, 640, I.JSD, False, I.F32, 256)])
def test_few_tokens(T, kept, H_t, H_s, V, kind, hv, dtype, chunk):
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, kind=kind, beta=0.5, w_t_std=0.05, mask="ones", dtype=dtype)
    data = I.generate(cfg)
    data["mask"] = np.zeros(T, np.uint8)
    data["mask"][np.random.default_rng(T).permutation(T)[:kept]] = 1
    head = (lambda x: np.ascontiguousarray(x.T)) if hv else (lambda x: x)
    d = [G.to_device(x, dtype) for x in (data["h_t"], head(data["W_t"]), data["h_s"], head(data["W_s"]))]
    layout = K.W_HV if hv else K.W_VH
    p = K.make_params(T, H_t, H_s, V, kind, cfg.tau, 0.5, w_layout=layout, vocab_chunk=chunk, in_dtype=K.F32 if dtype == I.F32 else K.BF16,
                      grad_dtype=K.F32)
    out = K.kd_loss_fwd_bwd(*d, torch.from_numpy(data["mask"]).cuda(), tau=cfg.tau, kind=kind, beta=0.5, w_layout=layout, vocab_chunk=chunk,
                            grad_dtype=K.F32, workspace=_nan_workspace(K.kd_loss_workspace_size(p) + 256))
    if kept == 0:
        assert not any(bool(out[k].any()) for k in ("loss", "per_token_loss", "grad_h_s", "grad_W_s"))
        return
    if hv:
        out["grad_W_s"] = out["grad_W_s"].t()
    allow = G.akl_allowance(cfg, data) if kind == I.AKL else G.tvd_tie_allowance(cfg, data) if kind == I.TVD else None
    G.check(out, G.run_oracle(cfg, data), "few tokens", allow)


def test_few_tokens_fp8_teacher_and_two_teachers():
    T, H_s, V = 70, 128, 4104
    base = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_s=H_s, V=V, mask="ones")
    ds = [I.generate(I.scaled(base, H_t=h, seed=700 + h)) for h in (256, 384)]
    dev = lambda x: G.to_device(x, I.BF16)
    ref = O.kd_loss_multi([d["h_t"] for d in ds], [d["W_t"] for d in ds], (0.6, 0.4), ds[0]["h_s"], ds[0]["W_s"], np.ones(T, np.uint8),
                          base.tau, base.kind, 0.5, O.W_VH)
    out = K.kd_loss_fwd_bwd_multi([dev(d["h_t"]) for d in ds], [dev(d["W_t"]) for d in ds], (0.6, 0.4), dev(ds[0]["h_s"]),
                                  dev(ds[0]["W_s"]), None, tau=base.tau, kind=base.kind, vocab_chunk=1024)
    G.check(out, ref, "two teachers")
    cfg, data = I.scaled(base, H_t=256), dict(ds[0])
    codes, scales = [], []
    for k in ("h_t", "W_t"):
        scales.append(float(np.abs(data[k]).max()) / 448)
        codes.append(K.quantize_e4m3(dev(data[k]), scales[-1]))
        data[k] = codes[-1].view(torch.float8_e4m3fn).float().cpu().numpy() * np.float32(scales[-1])
    out = K.kd_loss_fwd_bwd(*codes, dev(data["h_s"]), dev(data["W_s"]), None, flags=K.FLAG_TEACHER_FP8, teacher_scale=scales[0] * scales[1])
    G.check(out, G.run_oracle(cfg, data), "fp8 teacher")
