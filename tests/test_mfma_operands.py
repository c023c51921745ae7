"""No matrix product of the prompt passes writes its result over one of its operands: such a
placement once gave wrong scores, and the compiler makes it where an operand ends at a product
with a zero addend.  Read from the assembly of the built source."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2412_03131_amd import build

PRODUCT = re.compile(r"^\s+v_mfma_\S+\s+([av])\[(\d+):(\d+)\], ([av])\[(\d+):(\d+)\], ([av])\[(\d+):(\d+)\],")


@pytest.mark.skipif(not shutil.which(build.HIPCC), reason="no hipcc")
def test_no_product_over_its_operands(tmp_path):
    out = str(tmp_path / "k_prompt.s")
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    subprocess.run([build.HIPCC, "-x", "hip", "-S", "--cuda-device-only",
                    os.path.join(build.CSRC, "k_prompt.hip"), "-o", out] + flags, check=True, capture_output=True)
    products, over = 0, []
    with open(out) as f:
        for line in f:
            m = PRODUCT.match(line)
            if not m:
                continue
            products += 1
            kind, lo, hi = m.group(1), int(m.group(2)), int(m.group(3))
            for i in (4, 7):
                if m.group(i) == kind and int(m.group(i + 1)) <= hi and int(m.group(i + 2)) >= lo:
                    over.append(line.strip())
    assert products >= 500
    assert not over, over[:4]
