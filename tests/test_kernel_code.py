"""The compiled kernels keep the shape that their launch bounds were chosen
for: a model evaluation is part of its kernel, not a function called from it
(a call passes the kernel's arguments through scratch memory and reads LDS by
flat accesses), and the two-component fits keep nothing of their loops in
scratch.  Read from the code object's notes and symbols; needs no GPU."""
import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2404_07780_amd", "lib", "libgmfit.so")
LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """(kernel -> bytes of scratch per lane, names of the other device functions) of libgmfit.so."""
    if not os.path.exists(LIB):
        from paper_2404_07780_amd import build

        build.build()
    tmp = tmp_path_factory.mktemp("code")
    elf = str(tmp / "k.elf")
    data = open(LIB, "rb").read()
    kernels, functions, pos = {}, set(), data.find(MAGIC)
    while pos >= 0:
        n, o = struct.unpack_from("<Q", data, pos + 24)[0], pos + 32
        for _ in range(n):
            off, size, tl = struct.unpack_from("<QQQ", data, o)
            target = data[o + 24:o + 24 + tl].decode()
            o += 24 + tl
            if not (target.endswith("gfx950") and size):
                continue
            open(elf, "wb").write(data[pos + off:pos + off + size])
            notes = subprocess.run([LLVM + "/llvm-readelf", "--notes", elf], capture_output=True, text=True).stdout
            here = dict(zip(re.findall(r"\.symbol:\s+'?(\w+)\.kd", notes),
                            map(int, re.findall(r"\.private_segment_fixed_size:\s+(\d+)", notes))))
            kernels.update(here)
            syms = subprocess.run([LLVM + "/llvm-readelf", "-sW", elf], capture_output=True, text=True).stdout
            functions |= {l.split()[-1] for l in syms.splitlines() if " FUNC " in l} - set(here)
        pos = data.find(MAGIC, pos + 24)
    assert len(kernels) > 100
    return kernels, functions


def test_evaluation_is_part_of_its_kernel(code):
    for part in ("evaluate", "eval_prologue", "fill_region", "fit_errors"):
        name = f"{len(part)}{part}"
        assert not [f for f in code[1] if name in f], part


def test_two_component_kernels_use_little_scratch(code):
    pairs = {k: v for k, v in code[0].items() if "FamPair" in k and ("lm_fit_kernel" in k or "errors_kernel" in k)}
    assert len(pairs) >= 16
    for k, v in pairs.items():
        assert v <= 128, (k, v)


def test_one_component_fits_use_little_scratch(code):
    """At a PSF side without a kernel of its own."""
    fits = {k: v for k, v in code[0].items() if "FamSingle" in k and "lm_fit_kernel" in k and "ELi0E" in k}
    assert len(fits) >= 16
    for k, v in fits.items():
        assert v <= 128, (k, v)
