"""The rows of records that the accumulate pass requests unconditionally (csrc/bwd_record.hpp: load_from) keep their whole offset in
the vector operand of the buffer load, which the buffer's bound covers; the scalar operand, which the compiler's documentation
leaves out of the bounds check, is 0.  Read from the assembly, no GPU."""
import os
import re
import subprocess

from paper_2201_05989_amd.build import CSRC, HIPCC_FLAGS, INCLUDE, hipcc

HERE = os.path.dirname(os.path.abspath(__file__))


def test_the_buffers_bound_covers_a_rows_whole_offset(tmp_path):
    out = str(tmp_path / "load.s")
    flags = [f for f in HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([hipcc(), *flags, "--cuda-device-only", "-S", f"-I{INCLUDE}", f"-I{CSRC}", os.path.join(HERE, "record_load_check.hip"),
                    "-o", out], check=True, capture_output=True)
    with open(out) as f:
        loads = re.findall(r"^\s*buffer_load_\w+ (.+)$", f.read(), re.M)
    assert len(loads) == 3 * (1 + 1 + 1 + 2 + 1 + 3)  # records of 3, 3, 4, 6, 4 and 10 words, four words a load at most
    for operands in loads:
        scalar_offset = operands.split(",")[3].split()[0]
        assert scalar_offset == "0" and " offen" in operands, operands
