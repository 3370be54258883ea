"""Properties of the kernels' sources and of the code built from them that no
result shows (CPU only: no kernel runs)."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1906_11367_amd", "csrc")


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
