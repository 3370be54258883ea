"""Properties of the kernels' sources and of the code built from them that no
result shows (CPU only: no kernel runs)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1906_11367_amd", "csrc")
LIB = os.path.join(ROOT, "paper_1906_11367_amd", "libboxconv.so")


def test_asm_names_the_registers_it_writes():
    """An asm statement that writes m0 says so: the compiler may otherwise keep
    a value of its own there across it."""
    found = 0
    for name in sorted(os.listdir(CSRC)):
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        for stmt in re.findall(r"\basm\s+(?:volatile\s*)?\((.*?)\);", text, re.S):
            if re.search(r"\bs_mov_b32\s+m0\b", stmt):
                found += 1
                assert '"m0"' in stmt.rsplit(":", 1)[1], f"{name}: {stmt}"
    assert found


def _tool(name):
    for path in (shutil.which(name), f"/opt/rocm/llvm/bin/{name}"):
        if path and os.path.exists(path):
            return path
    pytest.skip(f"{name} not found")


@pytest.fixture(scope="module")
def device_code(tmp_path_factory):
    """The gfx950 code objects of the built library, one file each."""
    objdump = _tool("llvm-objdump")
    if not os.path.exists(LIB):
        pytest.skip("the library is not built")
    d = str(tmp_path_factory.mktemp("code"))
    lib = shutil.copy(LIB, d)
    subprocess.run([objdump, "--offloading", os.path.basename(lib)], cwd=d, check=True, capture_output=True)
    return [os.path.join(d, f) for f in sorted(os.listdir(d)) if f.endswith("gfx950")]


def _kernels(device_code, pattern):
    """(code object, mangled name) of the kernels whose mangled name matches."""
    readelf = _tool("llvm-readelf")
    out = []
    for obj in device_code:
        table = subprocess.run([readelf, "-sW", obj], check=True, capture_output=True, text=True).stdout
        out += [(obj, name) for name in {line.split()[-1] for line in table.splitlines() if " FUNC " in line}
                if re.search(pattern, name)]
    assert out, pattern
    return out


# fp32 storage, both operands aligned: forward, data gradient without and with
# the ReLU's mask, weight gradient, as (A contiguous along the reduction,
# masked; B contiguous along it, masked)
@pytest.mark.parametrize("a,b", [((1, 0), (0, 0)), ((0, 0), (0, 0)), ((0, 0), (0, 1)), ((1, 0), (1, 0))])
@pytest.mark.parametrize("tile", [64, 128])
def test_mix_loads_stay_in_flight(device_code, a, b, tile):
    """The next K-step's loads of the fp32 mix are not waited for before the
    matrix instructions of the current one."""
    (obj, name), = _kernels(device_code, rf"k_mix_gemmILb0ELi1ELb{a[0]}ELb{a[1]}ELi1ELb{b[0]}ELb{b[1]}ELi{tile}ELb1ELb1EE")
    text = subprocess.run([_tool("llvm-objdump"), "-d", f"--disassemble-symbols={name}", obj], check=True,
                          capture_output=True, text=True).stdout.splitlines()
    first_mfma = next(i for i, line in enumerate(text) if "v_mfma" in line)
    loads = [i for i in range(first_mfma) if "buffer_load_dwordx4" in text[i]]
    # the loop's loads are the last ones before its matrix instructions
    waits = [line for line in text[loads[-1]:first_mfma] if "vmcnt" in line]
    assert loads and not waits, waits


# (kernels, registers that leave the waves they are built for, bytes in memory):
# blocks of 512 threads of the streaming backward, two per CU (but for the ring
# that calls of few maps take); the backward from tables in memory, four waves per
# SIMD, two registers of the masked one spilled; the mix, two waves or three and
# nothing in memory, where a load in flight would be waited for; the forward of
# maps smaller than an item, eight waves
STREAM = r"k_box_bwd_streamILi64E(Li[24]ELi8E|Li3ELi8ELb1E|Li3ELi8ELb\dELb\dELb\dELb0E)"


@pytest.mark.parametrize("pattern,registers,spilled", [(STREAM, 128, 0), (r"k_box_bwd_gatherI", 128, 8), (r"k_mix_gemmI", 256, 0),
                                                       (r"k_box_fwd_ldsI\w+?Li\d+ELb\dELb\dELi0ELi3ELi0ELb1E", 64, 0)])
def test_waves_per_simd(device_code, pattern, registers, spilled):
    readelf = _tool("llvm-readelf")
    seen = 0
    for obj in device_code:
        notes = subprocess.run([readelf, "--notes", obj], check=True, capture_output=True, text=True).stdout
        for kernel in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", kernel).group(1)
            if not re.search(pattern, name):
                continue
            seen += 1
            assert int(re.search(r"\.vgpr_count:\s+(\d+)", kernel).group(1)) <= registers, name
            assert int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", kernel).group(1)) <= spilled, name
    assert seen
