"""The hazards of test_strip_hazards.py and test_product_hazards.py in the strip kernels that read [H, V] heads in place: their
MFMAs and their transposing LDS reads are both inline assembly."""
import re
import subprocess

from paper_2603_01875_amd import kdloss as K
from tests.test_product_hazards import early_uses
from tests.test_strip_hazards import LLVM, _code_objects, hazards, parse


def test_no_hazard_in_the_hidden_major_kernels(tmp_path):
    K.lib()
    kernels = {}
    for obj in _code_objects(K._LIB_PATH, str(tmp_path)):
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", obj], check=True, capture_output=True,
                              text=True).stdout
        for m in re.finditer(r"^([0-9a-f]+) <(\S*strip_hv\S*)>:\n((?:\t.*\n)+)", text, re.M):
            kernels[m[2]] = parse(m[3].splitlines(), int(m[1], 16))
    assert len(kernels) == 17                 # statistics x 4, rows x 5, gradient x 7, the AKL search
    for name, code in kernels.items():
        assert sum(c.op.startswith("v_mfma") for c in code) >= 4 * 48, name
        assert sum("ds_read_b64_tr" in c.op for c in code) >= 2 * 24, name
        assert hazards(code) == [], name
        assert early_uses(code) == [], name
