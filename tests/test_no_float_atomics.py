"""Results are the same bits from call to call: no kernel of the built library adds, or takes a minimum or maximum, in floating
point by an atomic, in LDS or in memory, where the order of the operands would be the hardware's."""
import re
import subprocess

from paper_2603_01875_amd import kdloss as K
from tests.test_strip_hazards import LLVM, _code_objects

FLOAT_ATOMIC = re.compile(r"^\s+((?:ds|global|flat|buffer)_\S*?(?:add|sub|min|max)\S*_(?:pk_)?(?:f16|bf16|f32|f64))\s")


def float_atomics(text):
    return [m[1] for m in map(FLOAT_ATOMIC.match, text.splitlines()) if m]


def test_no_floating_point_atomic_in_the_library(tmp_path):
    K.lib()
    objects = list(_code_objects(K._LIB_PATH, str(tmp_path)))
    assert objects
    seen = 0
    for obj in objects:
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", obj], check=True, capture_output=True,
                              text=True).stdout
        assert float_atomics(text) == []
        seen += text.count("ds_add_u64")
    assert seen >= 2 * 192            # AKL's bins: both head orders, every entry of a tile


def test_the_pattern_sees_them():
    for op in ("ds_add_f32", "ds_add_rtn_f32", "ds_pk_add_rtn_bf16", "ds_min_f64", "global_atomic_add_f32", "global_atomic_pk_add_f16",
               "buffer_atomic_max_f64", "flat_atomic_add_f64"):
        assert float_atomics(f"\t{op} v1, v2 // 0") == [op]
    for op in ("ds_add_u64", "ds_min_u64", "global_atomic_add_x2", "v_add_f32_e32", "v_pk_max_f16", "ds_read_b32"):
        assert float_atomics(f"\t{op} v1, v2 // 0") == []
