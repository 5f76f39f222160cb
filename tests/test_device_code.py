"""What the hand-written loads of the decode kernel rely on, looked up in the device code of the built library.  Runs without a GPU."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_23294_amd import _lib


def _objdump():
    for path in (shutil.which("llvm-objdump"), "/opt/rocm/llvm/bin/llvm-objdump"):
        if path and os.path.exists(path):
            return path
    pytest.skip("llvm-objdump is needed to list the device code")


def _scalars(text):
    text = text.strip().split()[0]
    m = re.fullmatch(r"s\[(\d+):(\d+)\]", text)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.fullmatch(r"s(\d+)", text)
    return {int(m[1])} if m else set()


def test_wait_states_and_m0_of_the_loads_to_shared_memory(tmp_path):
    """A load to shared memory takes m0, a resource and an offset from scalar registers.  Behind the last wait of five states in
    its block no vector instruction writes one of these, and m0 is what the load's own statement put there."""
    tool = _objdump()
    lib = shutil.copy(_lib.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([tool, "--offloading", str(lib)], cwd=tmp_path, check=True, capture_output=True)
    loads = 0
    for obj in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([tool, "-d", "--no-show-raw-insn", str(obj)], check=True, capture_output=True, text=True).stdout
        code = [line.split("//")[0].strip() for line in text.splitlines()]
        code = [line for line in code if line]
        for i, line in enumerate(code):
            if "m0" in re.split(r"[\s,]+", line) and not re.match(r"s_mov(k_i32|_b32) m0,", line):
                raise AssertionError(f"{obj.name}: another use of m0: {line}")
            if not (line.startswith("buffer_load") and line.endswith(" lds")):
                continue
            loads += 1
            _, resource, offset = line.split(None, 1)[1].split(",")
            uses = _scalars(resource) | _scalars(offset)
            assert len(uses) >= 4, line
            assert re.match(r"s_mov(k_i32|_b32) m0,", code[i - 2]) and code[i - 1].startswith("s_nop"), code[i - 3:i + 1]
            for back in range(i - 1, -1, -1):
                prev = code[back]
                if re.match(r"s_nop [4-9]", prev):
                    break
                assert not prev.endswith(":") and not prev.startswith(("s_branch", "s_cbranch")), f"no wait before: {code[back:i + 1]}"
                if prev.startswith("v_"):
                    assert not _scalars(prev.split(None, 1)[1].split(",")[0]) & uses, (prev, line)
    assert loads > 0


def test_no_kernel_for_short_contexts_that_no_plan_asks_for():
    """Five to eight heads per wave take a staged block per iteration and nothing else; the others one unit or several: group sizes 32, 64 and (at
    head_dim 128) 128, with and without INT8."""
    tool = shutil.which("llvm-nm") or next((p for p in ("/opt/rocm/llvm/bin/llvm-nm",) if os.path.exists(p)), None) or shutil.which("nm")
    if not tool:
        pytest.skip("nm is needed to list the kernels")
    names = subprocess.run([tool, "-C", _lib.LIB_PATH], check=True, capture_output=True, text=True).stdout
    kernels = set(re.findall(r"cocktail::(?:__device_stub__)?(decode_short_\w+_kernel<[^>]*>)", names))
    count = {kind: sum(k.startswith(f"decode_short_{kind}_") for k in kernels) for kind in ("heads", "quads", "tiles")}
    assert count == {"heads": 5 * 2 * 2, "quads": 5 * 2 * 2, "tiles": 5 * 2}
