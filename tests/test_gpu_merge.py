"""The kernels that merge the partial sums of a token, at the numbers of parts where their shape changes: 1024 parts
(one token tile), a few hundred (masked down to fewer tiles than planned), 128 and fewer; rows at the edges of their
8- and 32-token blocks.  Against the fp64 oracle with the tolerances of the other parity tests."""
import numpy as np
import pytest

from paper_2603_01875_amd import inputs as I
from tests import gpu_util as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [I.FKL, I.RKL, I.JSD, I.AKL])
@pytest.mark.parametrize("T, V, keep", [(1, 32776, 1), (9, 32776, 9), (255, 32768, 250), (520, 33000, 33),
                                        (3841, 4104, 3841), (4096, 4104, 3585)])
def test_merge_of_the_partial_sums(T, V, keep, kind):
    cfg = I.scaled(I.workload("fkl_bf16"), batch=1, seq=T, H_t=64, H_s=64, V=V, kind=kind, w_t_std=0.1)
    data = I.generate(cfg)
    data["mask"] = np.zeros(T, dtype=np.uint8)
    data["mask"][np.random.default_rng(T).permutation(T)[:keep]] = 1
    extra = G.akl_allowance(cfg, data) if kind == I.AKL else None
    out = G.run_gpu(cfg, data)
    G.check(out, G.run_oracle(cfg, data), f"T={T} V={V} kept={keep} kind={kind}", extra)
