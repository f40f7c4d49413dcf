"""The probe reads X once: on planes of whole cache lines its 16-bit kernel loads with the non-temporal hint, on others without.
Both kinds of load have to be in the built code: a compiler that sees the same load in the two arms of the choice keeps one of
them, without the hint, and no result shows it.  Host only (reads the library built here)."""
import os
import re
import shutil
import subprocess
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2106_06998_amd", "libxconv.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
# dtype, blocks of 16 probe columns, pixels per lane, split Z, channels-last
KERNEL = re.compile(r"<_ZN2xc15probe_16_kernelILi(\d)ELi(\d)ELi(\d)ELb(\d)ELb(\d)E\S*>:")


def loads_of(text):
    """(kernel, hinted, plain) of the vector loads of every probe_16_kernel in a disassembly."""
    parts = re.split(r"\n[0-9a-f]+ (?=<)", text)
    for f in parts:
        m = KERNEL.match(f)
        if m:
            lines = re.findall(r"global_load_dwordx[24] .*", f)
            hinted = sum(bool(re.search(r"\bnt\b", l)) for l in lines)
            yield m.groups(), hinted, len(lines) - hinted


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump not installed")
def test_both_kinds_of_load_are_there():
    assert os.path.exists(LIB)
    tmp = tempfile.mkdtemp(prefix="xconv_hints_")
    try:
        shutil.copy(LIB, os.path.join(tmp, "lib.so"))
        subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp, check=True, stdout=subprocess.DEVNULL)
        seen = 0
        for name in sorted(os.listdir(tmp)):
            # the probe's code object is the one that holds its symbols
            if "amdgcn" not in name or b"_ZN2xc15probe_16_kernel" not in open(os.path.join(tmp, name), "rb").read():
                continue
            text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", name], cwd=tmp, check=True, stdout=subprocess.PIPE, text=True).stdout
            for key, hinted, plain in loads_of(text):
                seen += 1
                if key[4] == "1":                       # channels-last rows: always hinted
                    assert hinted > 0, key
                else:                                   # planes: each load in both kinds (plain besides: Z in fragment order)
                    assert hinted >= 32 and hinted <= plain <= hinted + 8, (key, hinted, plain)
        assert seen >= 80
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
