"""Absorbed-weight path: the k loop of the weighted sums (csrc/apt_absorb_pv16.hip) as it was compiled."""
import re
import subprocess

import pytest

from tests.test_abi_host import _code_objects

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


def test_last_k_tiles_do_not_wait_for_the_copies_behind_them(tmp_path):
    """A k-tile waits for its own copies only, those of the S - 2 k-tiles behind it stay in flight; the last ones, behind which fewer are in
    flight, too.  So the largest count of a kernel's waits is there twice, in the full loop and in the last iterations."""
    try:
        subprocess.run([OBJDUMP, "--version"], capture_output=True, check=True)
    except OSError:
        pytest.skip("no llvm-objdump")
    seen = 0
    for n, elf in enumerate(_code_objects()):
        if b"apt_absorb_pv16_kernel" not in elf:
            continue
        obj = tmp_path / f"{n}.o"
        obj.write_bytes(elf)
        text = subprocess.run([OBJDUMP, "-d", str(obj)], capture_output=True, text=True, check=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\w*apt_absorb_pv16_kernel\w*)>:\n(.*?)(?=^$|\Z)", text, flags=re.M | re.S):
            waits = [int(c) for c in re.findall(r"s_waitcnt vmcnt\((\d+)\)", body)]
            assert max(waits) > 0 and waits.count(max(waits)) >= 2, (name, waits)
            seen += 1
    assert seen >= 16
