"""What the compiler made of the kernels' barriers, read from the assembly of the library that was built here (no GPU).

While loads that write LDS may be on their way, the compiler has a wavefront wait for all of its loads at every barrier.  In a kernel
with a loop over jobs they stay so as far as the compiler can see, if their wait depends on a condition of its own: every barrier of the loop
then waits for the next activation tile, or for the codes of the next piece."""
import os
import re
import subprocess

import pytest

import paper_2509_22951_amd as tq

BIN = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if not all(os.path.exists(os.path.join(BIN, t)) for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-objdump")):
        pytest.skip("needs the ROCm binary tools")
    tq.load()
    folder = tmp_path_factory.mktemp("code")
    fat, code = str(folder / "fat"), str(folder / "code")
    subprocess.run([f"{BIN}/llvm-objcopy", f"--dump-section=.hip_fatbin={fat}", tq.binding.lib_path(), "/dev/null"], check=True)
    subprocess.run([f"{BIN}/clang-offload-bundler", "--unbundle", "--type=o", f"--input={fat}", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    f"--output={code}"], check=True)
    text = subprocess.run([f"{BIN}/llvm-objdump", "-d", "--no-show-raw-insn", code], check=True, capture_output=True, text=True).stdout
    kernels, lines = {}, None
    for line in text.splitlines():
        head = re.match(r"^[0-9a-f]+ <(\w+)>:$", line)
        if head:
            lines = kernels.setdefault(head.group(1), [])
        elif lines is not None and line.strip():
            lines.append(line.split("//")[0].split())
    return kernels


@pytest.mark.parametrize("what,name,number", [
    ("products of up to 16 rows", r"_ZN2tq13k_matvec_ringI", 8),
    ("staged steps", r"_ZN2tq8k_matvecILi\d+ELi\d+ELb[01]ELi[12]ELb0ELb1E", 6),
])
def test_barriers_of_kernels_with_a_loop_wait_for_no_loads(assembly, what, name, number):
    found = {k: v for k, v in assembly.items() if re.match(name, k)}
    assert len(found) >= number, sorted(assembly)
    for kernel, lines in found.items():
        assert any(i[0] == "s_barrier" for i in lines)
        drained = [a for a, b in zip(lines, lines[1:]) if b[0] == "s_barrier" and a[0] == "s_waitcnt" and "vmcnt(0)" in a and "lgkmcnt(0)" in a]
        assert not drained, (what, kernel, len(drained))
