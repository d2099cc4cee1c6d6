"""Where the shading code of the render kernels lies: its eight-byte vector
instructions run a few per cent faster from addresses of 4 modulo 8, and an
edit anywhere in a kernel can move them by four bytes.  Read from the
disassembly of the library built here."""
import os
import re
import subprocess

import pytest

from paper_2302_12249_amd import merf

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel: [(address, bytes, text)]} of the render kernels."""
    d = tmp_path_factory.mktemp("objects")
    os.symlink(merf.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)
    found = {}
    for f in sorted(os.listdir(d)):
        if "gfx950" not in f:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--demangle", f], cwd=d, check=True, capture_output=True, text=True).stdout
        code = None
        for line in text.splitlines():
            if m := re.match(r"^[0-9a-f]+ <(.*)>:$", line):
                k = re.search(r"(k_render\w*<.*>)\(", m.group(1))
                code = found.setdefault(k.group(1), []) if k else None
            elif code is not None and (m := re.match(r"^\s+(\S.*?)\s*//\s*([0-9A-F]+):((?: [0-9A-F]{8})+)", line)):
                code.append((int(m.group(2), 16), 4 * len(m.group(3).split()), m.group(1)))
    return found


@pytest.mark.parametrize("feat", [0, 1])
def test_shading_starts_at_four_modulo_eight(kernels, feat):
    names = [f"k_render<0, {m}, {feat}, false>" for m in range(3)]
    names += [f"{k}<{m}, {feat}, false>" for k in ("k_render_served", "k_render_parts") for m in range(3)]
    for name in names:
        code = kernels[name]
        # the shading pass runs at priority 2, the compositing at 1
        first = next(i for i, c in enumerate(code) if c[2].startswith("s_setprio 2"))
        last = next(i for i, c in enumerate(code) if i > first and c[2].startswith("s_setprio 1"))
        wide = [a for a, n, t in code[first:last] if n == 8 and t.startswith("v_")][-200:]
        share = sum(a % 8 == 4 for a in wide) / len(wide)
        assert len(wide) == 200 and share > 0.9, (name, share)
