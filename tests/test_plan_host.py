"""Which calls the library accepts and what their plans have in common, asked on the host: every call here is stopped
by a NULL pointer before anything is launched, so its status tells whether the plan itself was refused."""
import ctypes

import pytest

from paper_2603_01875_amd import kdloss as K

OK, NULL = 0, 1
FAKE = [ctypes.c_void_p(0x1000 * (i + 3)) for i in range(8)]         # aligned, never dereferenced


def _multi_status(p, H_t):
    """Status of a call with one teacher more than H_t, whose hidden states are NULL: it is reached only if the plans
    of all the others agree."""
    n = len(H_t) + 1
    H = (ctypes.c_int64 * n)(*H_t, H_t[0])
    hidden = (ctypes.c_void_p * n)(*[0x1000] * len(H_t), None)
    heads = (ctypes.c_void_p * n)(*[0x2000] * n)
    weights = (ctypes.c_float * n)(*[1.0 / n] * n)
    scales = (ctypes.c_float * n)(*[1.0] * n)
    return K.lib().kd_loss_fwd_bwd_multi(ctypes.byref(p), n, hidden, heads, H, weights, scales, *FAKE,
                                         ctypes.c_size_t(1 << 60), None)


def _multi_size(p, H_t):
    n = ctypes.c_size_t(0)
    H = (ctypes.c_int64 * len(H_t))(*H_t)
    return K.lib().kd_loss_workspace_size_multi(ctypes.byref(p), len(H_t), H, ctypes.byref(n)), n.value


@pytest.mark.parametrize("kw", [dict(), dict(kind=K.AKL), dict(w_layout=K.W_HV), dict(in_dtype=K.F32),
                                dict(flags=K.FLAG_TEACHER_FP8), dict(w_layout=K.W_HV, flags=K.FLAG_TEACHER_FP8)])
def test_teachers_of_different_width_share_one_plan(kw):
    """Vocabulary chunk, loop and student buffers are the call's, whatever the teachers' hidden sizes."""
    for T in (8, 257, 512, 777, 1024, 1500, 2048, 2600, 3000, 3072, 3584, 4096, 9000):
        for V in (2048, 32000, 128256, 151936):
            for H_s in (64, 896, 1024):
                for H_t in ((4096, 2048), (2048, 4096), (4096, 8192, 1024), (512, 3584, 128)):
                    p = K.make_params(T, H_t[0], H_s, V, beta=0.5, **kw)
                    assert _multi_status(p, H_t) == NULL, (T, V, H_s, H_t)
                    status, size = _multi_size(p, H_t)
                    assert status == OK and size > 0, (T, V, H_s, H_t)


def test_one_teacher_plans_as_the_plain_call():
    for T, V in ((100, 4096), (700, 50264), (2048, 151936), (8192, 32000)):
        p = K.make_params(T, 2048, 512, V)
        assert _multi_size(p, (2048,))[1] == K.kd_loss_workspace_size(p)


# T, H_t, H_s, V, kind, [H,V] heads, fp32, fp8 teacher, the caller's chunk
FIT_THE_STATIC_ARRAY = [
    (6144, 3584, 768, 32000, 6, 0, 0, 0, 0), (8192, 2048, 512, 128256, 6, 0, 0, 0, 0), (10934, 2176, 704, 115968, 0, 0, 0, 0, 0),
    (32768, 256, 256, 32000, 0, 0, 0, 0, 0), (32768, 64, 64, 32000, 6, 0, 0, 0, 0), (257, 65536, 24576, 256, 0, 0, 0, 0, 0),
    (31234, 128, 16, 89272, 4, 1, 0, 0, 256), (28889, 192, 128, 7144, 2, 0, 0, 0, 1024), (1060, 44216, 64, 240, 1, 1, 0, 0, 0),
    (61676, 24, 24, 6560, 5, 1, 0, 0, 256), (41261, 64, 48, 26536, 0, 0, 1, 0, 0), (28652, 640, 192, 114192, 0, 0, 0, 0, 256),
    (17295, 2048, 232, 13808, 2, 0, 0, 1, 1024), (11477, 768, 1024, 145928, 0, 0, 0, 1, 256), (52484, 256, 24, 11480, 5, 0, 0, 1, 0),
    (59165, 384, 24, 11168, 1, 1, 0, 1, 0), (31648, 256, 128, 28064, 1, 1, 0, 0, 0), (1429, 32, 10768, 296, 3, 0, 0, 0, 256),
    (28, 52408, 96, 224, 3, 0, 1, 0, 0), (1, 56368, 128, 1112, 0, 0, 0, 0, 0), (7, 62568, 3344, 784, 4, 0, 0, 0, 0),
    (20, 1536, 192, 66672, 0, 1, 0, 1, 1024), (9137, 128, 1088, 6696, 1, 1, 0, 1, 1024), (3775, 1832, 1920, 80, 5, 1, 1, 0, 0),
    (612, 160, 12048, 416, 1, 0, 1, 0, 256), (12687, 576, 448, 11520, 6, 1, 0, 0, 0), (19162, 32, 16, 33128, 6, 0, 1, 0, 256),
]


@pytest.mark.parametrize("T, H_t, H_s, V, kind, hv, f32, fp8, chunk", FIT_THE_STATIC_ARRAY)
def test_calls_that_fit_the_static_array(T, H_t, H_s, V, kind, hv, f32, fp8, chunk):
    """Sizes near the limit of the static array, where only the smallest partial sums and copies fit: many tokens, or
    few tokens of wide hidden states; every layout and type."""
    p = K.make_params(T, H_t, H_s, V, kind, beta=0.5, w_layout=K.W_HV if hv else K.W_VH, in_dtype=K.F32 if f32 else K.BF16,
                      flags=K.FLAG_TEACHER_FP8 if fp8 else 0, teacher_scale=1.0 if fp8 else 0.0, vocab_chunk=chunk)
    args = [None] + FAKE
    assert K.lib().kd_loss_fwd_bwd_static(ctypes.byref(p), *args, None) == NULL


@pytest.mark.parametrize("kw", [dict(), dict(kind=K.AKL), dict(w_layout=K.W_HV), dict(flags=K.FLAG_TEACHER_FP8, teacher_scale=1.0)])
def test_few_tokens_need_few_rows(kw):
    """Below a token tile the copies of the hidden states have the rows that there are, not a tile's."""
    n = [K.kd_loss_workspace_size(K.make_params(T, 65536, 64, 256, beta=0.5, **kw)) for T in (1, 101, 201)]
    es = 1 if "flags" in kw else 2
    assert n[1] - n[0] >= 100 * 65536 * es and n[2] - n[1] >= 100 * 65536 * es and n[0] < 4 << 20


# Which loop makes the logit tiles, at sizes where one of them measured at least 4 % ahead of the other.  (Three of them on an earlier
# state: the strip loop is 27 and 35 % ahead now at AKL's two sizes among EIGHT_WAVES, which only hold the line where it is, and 1 % at
# T = 256.)
EIGHT_WAVES = [   # T, H_t, H_s, V, kind
    (257, 2048, 1024, 512, 0), (512, 8192, 512, 512, 0), (4096, 8192, 512, 512, 0), (8192, 8192, 512, 256, 0),
    (1024, 2048, 1024, 4096, 0), (2048, 2048, 1024, 4096, 0), (4096, 2048, 1024, 2048, 0), (300, 4096, 1024, 32000, 0),
    (512, 2048, 1024, 16384, 0), (4096, 256, 128, 151936, 0), (16384, 256, 128, 151936, 0), (777, 1000, 520, 50264, 4),
    (2048, 512, 256, 65536, 2), (4096, 2048, 1024, 4096, 2), (1024, 1024, 512, 65536, 6), (4096, 1024, 512, 128256, 6),
    (256, 4096, 1024, 151936, 0), (1, 4096, 1024, 151936, 2)]
STRIPS = [
    (4096, 4096, 1024, 151936, 0), (4096, 4096, 1024, 151936, 2), (8192, 8192, 2048, 128256, 0), (32768, 5120, 4096, 151936, 2),
    (1003, 4096, 2048, 128256, 1), (2048, 4096, 1024, 151936, 6), (512, 4096, 1024, 20000, 0), (300, 4096, 1024, 24576, 0),
    (2048, 8192, 512, 6144, 0), (4096, 8192, 512, 3072, 0), (2048, 2048, 1024, 100000, 0), (1024, 8192, 2048, 151936, 2)]


@pytest.mark.parametrize("sizes, loop", [(s, 0) for s in EIGHT_WAVES] + [(s, 1) for s in STRIPS])
def test_the_faster_loop_is_taken(sizes, loop):
    T, H_t, H_s, V, kind = sizes
    assert K.kd_loss_plan_loop(K.make_params(T, H_t, H_s, V, kind, beta=0.5)) == loop
    # ... and the teachers of a call share one, whatever each alone would take
    assert _multi_status(K.make_params(T, H_t, H_s, V, kind, beta=0.5), (H_t, 64, 8 * H_t if H_t <= 8192 else H_t)) == NULL
