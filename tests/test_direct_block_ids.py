"""Block ids of the one-launch decode form: only slots in use are read, and the ids of a batch of rows are asked for
together, in front of its rows (checked on the kernel's own slot function and on the code hipcc emits; no GPU)."""
import os
import re
import subprocess

from paper_2402_14808_amd import build
from test_codegen import _device_asm

PROGRAM = """
#include "decode_direct.hip"
#include <cstdio>
int main() {
    for (int bsl = 0; bsl <= 7; ++bsl)
        for (int s : {0, 1, 15, 64, 300})
            for (int c : {1, 2, 7, 8, 9, 31, 32, 33, 127, 128, 129, 500}) {
                const int used = (c + (1 << bsl) - 1) >> bsl;
                for (int row = 0; row < s + c; ++row) {
                    const int slot = ra::used_slot(row, s, bsl);
                    if (slot < 0 || slot >= used || (row >= s && slot != (row - s) / (1 << bsl))) {
                        printf("row %d of %d + %d, block size %d: slot %d\\n", row, s, c, 1 << bsl, slot);
                        return 1;
                    }
                }
            }
    return 0;
}
"""


def test_no_slot_behind_the_used_ones(tmp_path):
    (tmp_path / "slots.hip").write_text(PROGRAM)
    exe = str(tmp_path / "slots")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    r = subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")] + flags +
                       ["-I", build.CSRC, str(tmp_path / "slots.hip"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_block_ids_of_a_batch_in_front_of_its_rows():
    """Four ids a batch: an id between two rows, which are 16-byte loads, is waited for together with the rows before it."""
    kernels = re.split(r"\n(?=_ZN\S+decode_direct_kernel\S+:)", _device_asm("decode_direct"))[1:]
    assert len(kernels) == 6
    for text in kernels:
        loads = re.findall(r"^\s+global_load_dword(x4)? ", text, re.M)
        ids = re.findall("I+", "".join("R" if x else "I" for x in loads))
        assert len(ids) >= 3 and all(len(run) == 4 for run in ids), (text.split(":")[0], ids)
