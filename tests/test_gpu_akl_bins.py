"""AKL's threshold search by bins (strip loop): head masses at both ends, teachers from nearly flat to nearly one-hot (the
interval that the search starts from is 1 to 40 wide), a short last tile, tokens masked so that whole token tiles have nothing
to search.  Against the fp64 oracle, with the allowance of the other AKL tests."""
import pytest

from paper_2603_01875_amd import inputs as I
from paper_2603_01875_amd import kdloss as K
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mu, std, V, kept", [(0.2, 0.02, 16200, 600), (0.9, 0.02, 16136, 600), (0.5, 0.001, 16200, 600),
                                              (0.8, 0.3, 16200, 600), (0.5, 0.1, 16256, 3), (0.999, 0.05, 16200, 257)])
def test_akl_search_by_bins(mu, std, V, kept):
    assert K.kd_loss_plan_loop(K.make_params(600, 2816, 128, V, I.AKL, beta=mu)) == 1
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=600, H_t=2816, H_s=128, V=V, kind=I.AKL, beta=mu, w_t_std=std)
    data = I.generate(cfg)
    data["mask"][:] = 0
    data["mask"][:kept] = 1
    G.check(G.run_gpu(cfg, data), G.run_oracle(cfg, data), f"mu={mu} std={std} V={V} kept={kept}", G.akl_allowance(cfg, data))
