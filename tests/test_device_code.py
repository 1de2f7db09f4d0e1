"""What the built device code has to keep and no run shows reliably: read from the library's own gfx950 code, no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2407_20761_amd.binding import LIB_PATH

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """{kernel: [(instruction, operands), ...]} of every device image in the library"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("needs llvm-objdump")
    here = tmp_path_factory.mktemp("images")
    lib = shutil.copy(LIB_PATH, here)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True, cwd=here)
    kernels, name = {}, None
    for image in sorted(p for p in here.iterdir() if p.name.endswith("gfx950") and p.stat().st_size):
        out = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", str(image)], check=True, capture_output=True, text=True).stdout
        for line in out.splitlines():
            head = re.match(r"<(\w+)>:$", line.strip())
            if head:
                name = head.group(1)
                kernels[name] = []
            elif name and line.startswith(("\t", " ")):
                text = line.split("//")[0].strip()
                if text:
                    op, _, rest = text.partition(" ")
                    kernels[name].append((op, rest.strip()))
    return kernels


def test_loads_to_lds_keep_their_distances(code):
    """The loads to LDS of dK / dV are inline assembly, whose neighbours the compiler does not look at: by itself the block of a load has
    one wait state after the write of m0 and, in front of its first load, five in which nothing can write the descriptor."""
    kernels = {n: c for n, c in code.items() if "attn_bwd_dkv" in n and "f32" not in n}
    assert len(kernels) >= 9      # (the bf16 ones)
    for name, instructions in kernels.items():
        is_load = lambda op, rest: op.startswith("buffer_load_dword") and rest.endswith(" lds")
        loads = [i for i, pair in enumerate(instructions) if is_load(*pair)]
        assert loads, name
        for at in loads:
            states, after_m0, i = 0, None, at - 1
            while states < 5:
                op, rest = instructions[i]
                own = op == "s_nop" or op in ("s_mov_b32", "s_add_i32") and rest.startswith("m0,") or is_load(op, rest)
                assert own, (name, instructions[i:at + 1])
                if rest.startswith("m0,") and after_m0 is None:
                    after_m0 = states
                states += int(rest, 0) + 1 if op == "s_nop" else 1
                i -= 1
            assert after_m0 is not None and after_m0 >= 1, (name, instructions[i:at + 1])
