"""Rules of the instruction set that the compiler does not keep for inline asm,
checked in the device assembly of the library's own sources (no GPU)."""
import os
import re
import subprocess

from paper_2609_04663_amd import build as B


def test_wait_states_after_16_byte_stores(tmp_path):
    """A VALU instruction may overwrite the data of a store of more than 8 bytes
    only two wait states after it; the replay's stores are inline asm."""
    out = str(tmp_path / "split.s")
    subprocess.run([B.HIPCC, *B.FLAGS, "-S", "--cuda-device-only",
                    os.path.join(B.CSRC, "split.hip"), "-o", out], check=True)
    with open(out) as f:
        asm = f.read()
    blocks = re.findall(r";;?#ASMSTART\s*\n(.*?);;?#ASMEND", asm, re.S)
    stores = [b for b in blocks if "global_store_dwordx4" in b]
    assert len(stores) >= 12        # six levels, packed by rows and by columns
    for b in stores:
        m = re.search(r"global_store_dwordx4[^\n]* sc1\s*\n\s*s_nop (\d+)", b)
        assert m and int(m.group(1)) >= 1, b
