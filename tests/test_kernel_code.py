"""What the built kernels must not contain: loads through flat pointers (each is waited for together with everything in
flight, which undoes a pipelined loop) and registers spilled to memory in the loops that are bound by latency.  Reads the
listing of the library built here; needs no GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2404_06910_amd import binding as B

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel name: its instructions}"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    at = tmp_path_factory.mktemp("code")
    shutil.copy(B.lib_path(), at / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=at, check=True, stdout=subprocess.DEVNULL)
    found, name = {}, None
    for f in sorted(os.listdir(at)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", f], cwd=at, check=True, capture_output=True, text=True).stdout
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(\w+)>:", line)
            if m:
                name = m.group(1)
                found[name] = []
            elif name and line.strip():
                found[name].append(line.split("//")[0].strip())
    return found


def _named(kernels, part):
    some = {n: c for n, c in kernels.items() if part in n}
    assert some, part
    return some


def test_decode_loads_are_global(kernels):
    for name, code in _named(kernels, "decode").items():
        assert not [c for c in code if c.startswith("flat_load")], name
        # K and V of the next batch (or V of this one) stay in flight across the first products
        assert any(re.match(r"s_waitcnt vmcnt\([1-9]", c) for c in code), name


def test_decode_keeps_its_registers(kernels):
    for name, code in _named(kernels, "decode").items():
        assert not [c for c in code if c.startswith("scratch_")], name


def test_fp32_prefill_keeps_its_registers(kernels):
    for name, code in _named(kernels, "prefill_f32").items():
        assert not [c for c in code if c.startswith(("scratch_", "flat_load"))], name


def test_wide_prefill_keeps_its_registers(kernels):
    for name, code in _named(kernels, "prefill_wide").items():
        assert not [c for c in code if c.startswith(("scratch_", "flat_"))], name
