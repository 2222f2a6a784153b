"""Vocabulary chunks as the library chooses them below 4096 tokens: several chunks of a width that depends on the token
count and the hidden sizes, a last one of another width.  The fp64 oracle runs on the tokens that count alone (masked
ones must come out as zeros), so the vocabularies can be as large as the choice needs; tolerances are those of the
other parity tests."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


def _chunks(cfg):
    from paper_2603_01875_amd import kdloss as K
    vc, _ = K.kd_loss_plan_info(K.make_params(cfg.T, cfg.H_t, cfg.H_s, cfg.V, cfg.kind, cfg.tau, cfg.beta))
    assert vc % 256 == 0 and vc * 2 * -(-cfg.T // 256) * 256 <= 208 << 20
    return -(-cfg.V // vc)


@pytest.mark.parametrize("T, H_t, H_s, V, keep, kind", [
    (600, 64, 64, 151936, 70, I.FKL), (1300, 128, 192, 90008, 290, I.JSD), (2048, 192, 64, 60000, 513, I.RKL),
    (3333, 64, 128, 40008, 300, I.SKEW_FKL), (3840, 136, 72, 33000, 260, I.FKL), (2048, 2048, 1024, 60000, 257, I.FKL),
    (3585, 1024, 960, 40008, 130, I.SKEW_RKL)])
def test_chosen_widths(T, H_t, H_s, V, keep, kind):
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_t, H_s=H_s, V=V, kind=kind, w_t_std=0.1)
    assert _chunks(cfg) > 1
    data, few, idx = G.few_tokens(cfg, keep)
    ref = G.spread_tokens(G.run_oracle(cfg, few), idx, T)
    G.check(G.run_gpu(cfg, data), ref, f"T={T} H={H_t},{H_s} V={V}")


@pytest.mark.parametrize("T, V, H_s, H_ts", [(3072, 50264, 128, (1024, 256)), (3072, 40008, 64, (64, 256, 128)),
                                             (2100, 80008, 256, (256, 768))])
def test_teachers_of_different_width_in_chosen_chunks(T, V, H_s, H_ts):
    """One width for the whole call where each teacher alone would get another; narrow and wide teacher first."""
    from paper_2603_01875_amd import kdloss as K
    import torch
    base = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H_ts[0], H_s=H_s, V=V, w_t_std=0.1)
    weights = [0.5, 0.3, 0.2][:len(H_ts)]
    weights[-1] = 1.0 - sum(weights[:-1])
    data, few, idx = G.few_tokens(base, 90)
    h_t, W_t, ref = [], [], None
    for k, H in enumerate(H_ts):
        cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=H, H_s=H_s, V=V, w_t_std=0.1)
        assert _chunks(cfg) > 1
        d = I.generate(cfg)
        h_t.append(G.to_device(d["h_t"], I.BF16))
        W_t.append(G.to_device(d["W_t"], I.BF16))
        r = G.run_oracle(cfg, dict(few, h_t=d["h_t"][idx], W_t=d["W_t"]))
        part = {n: weights[k] * r[n] for n in ("loss", "per_token_loss", "grad_h_s", "grad_W_s")}
        ref = part if ref is None else {n: ref[n] + part[n] for n in part}
    dev = lambda k: G.to_device(data[k], I.BF16)
    ref = G.spread_tokens(ref, idx, T)
    mask = torch.from_numpy(data["mask"]).cuda()
    h_s, W_s = dev("h_s"), dev("W_s")
    for order in (slice(None), slice(None, None, -1)):
        out = K.kd_loss_fwd_bwd_multi(h_t[order], W_t[order], weights[order], h_s, W_s, mask)
        G.check(out, ref, f"teachers {H_ts[order]}")
