"""Width of the vocabulary chunk with many tokens: 16384 columns while the staging buffer of dL/dz_s is within 512 MiB, then halved."""
import pytest

from paper_2603_01875_amd import kdloss as K


@pytest.mark.parametrize("T, width", [(4096, 16384), (6000, 16384), (16384, 16384), (16385, 8192), (32768, 8192), (32769, 4096), (262144, 1024),
                                      (1 << 22, 1024)])
def test_chunk_of_many_tokens(T, width):
    for V in (151936, 128256):
        assert K.kd_loss_plan_info(K.make_params(T, 512, 256, V))[0] == width
    assert K.kd_loss_plan_info(K.make_params(T, 512, 256, 1000))[0] == min(width, 1024)


@pytest.mark.parametrize("T, H_t, H_s, width", [(4096, 4096, 4096, 16384), (6656, 8192, 2048, 16384), (6657, 8192, 2048, 16384),
                                                (16384, 8192, 4096, 16384), (32768, 5120, 4096, 8192)])
@pytest.mark.parametrize("kw", [{}, {"kind": K.AKL}, {"in_dtype": K.F32}, {"w_layout": K.W_HV}])
def test_chunk_whatever_is_contracted(T, H_t, H_s, width, kw):
    assert K.kd_loss_plan_info(K.make_params(T, H_t, H_s, 128256, **kw))[0] == width
