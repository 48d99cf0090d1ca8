"""The built library's own gfx950 code, read for wait states that the compiler
cannot insert: it looks for hazards between instructions it emits, not inside
an asm block."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2607_01237_amd import kara

OBJDUMP = shutil.which("llvm-objdump", path=os.environ.get("ROCM_PATH", "/opt/rocm") + "/llvm/bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: its instructions in order}"""
    assert OBJDUMP, "llvm-objdump is part of the ROCm toolchain that builds the library"
    if not os.path.exists(kara.LIB_PATH):
        from paper_2607_01237_amd import build
        build.build()
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(kara.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=d)
    out, name = {}, None
    for f in sorted(p for p in d.iterdir() if p.name.endswith("gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(f)], check=True,
                              capture_output=True, text=True).stdout
        for line in text.splitlines():
            m = re.match(r"(?:[0-9a-f]+ )?<(.*)>:$", line)
            if m:
                name = m.group(1)
                out[name] = []
            elif name and line.startswith(("\t", " ")):
                ins = line.split("//")[0].strip()
                if ins:
                    out[name].append(ins)
    return out


def test_every_kernel_is_listed(kernels):
    for part in ("score1_kernel", "score_kernel", "score_res_kernel", "attn_kernel", "decode_split_kernel", "select_kernel"):
        assert any(part in k and v for k, v in kernels.items()), part


def test_lds_copies_wait_for_m0(kernels):
    # a load into LDS takes its address from M0 and needs one wait state after
    # a scalar write of it
    copies, early = 0, {}
    for name, code in kernels.items():
        for prev, ins in zip(code, code[1:]):
            if "_load_lds_" in ins:
                copies += 1
                if re.match(r"s_\w+ m0,", prev):
                    early[name] = early.get(name, 0) + 1
    assert copies > 1000
    assert not early, early
