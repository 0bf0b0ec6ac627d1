"""Hand-counted waits, checked on the built library's gfx950 code (no GPU needed).

gemm_big_kernel and vectors_cols_kernel wait for a stage's copies into LDS with s_waitcnt vmcnt(n):
what was issued before the newest n loads has landed. The first stage's four copies are therefore
safe to read only if at least n loads are issued between the last of them and that wait.
"""
import os
import re
import shutil
import subprocess

import pytest

import paper_2608_20530_amd as L

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def functions(tmp_path_factory):
    """Kernel symbol -> its instructions, over every gfx950 code object of the library."""
    assert os.path.exists(L.LIB_PATH), "the library is not built"
    d = tmp_path_factory.mktemp("code")
    lib = shutil.copy(L.LIB_PATH, d)
    subprocess.run([OBJDUMP, "--offloading", lib], cwd=d, check=True, stdout=subprocess.DEVNULL)
    out = {}
    for obj in sorted(d.glob("*gfx950")):
        if not re.search(rb"gemm_big_kernel|vectors_cols_kernel", obj.read_bytes()):
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(obj)], cwd=d, check=True,
                              capture_output=True, text=True).stdout
        for line in text.splitlines():
            if m := re.match(r"[0-9a-f]+ <(.+)>:", line):
                body = out.setdefault(m.group(1), [])
            elif line.startswith("\t"):
                body.append(line.split("//")[0].strip())
    return out


def loads_after_first_stage(code, n):
    """Loads issued after the fourth copy into LDS and before the first vmcnt(n) at a barrier."""
    end = next(i for i, (a, b) in enumerate(zip(code, code[1:]))
               if a == f"s_waitcnt vmcnt({n})" and b == "s_barrier")
    loads = [i for i in code[:end] if re.match(r"(buffer|global)_load", i)]
    copies = [k for k, i in enumerate(loads) if re.search(r"\blds\b", i)]
    return len(loads) - 1 - copies[3]


@pytest.mark.parametrize("kernel,n,instances", [("gemm_big_kernel", 20, 3),
                                                ("vectors_cols_kernel", 16, 1)])
def test_first_stage_is_covered(functions, kernel, n, instances):
    found = {k: v for k, v in functions.items() if kernel in k}
    assert len(found) == instances
    for name, code in found.items():
        assert loads_after_first_stage(code, n) >= n, name


def test_an_early_weight_load_is_noticed():
    copy, weight = "buffer_load_dwordx4 v1, s[0:3], 0 offen lds", "buffer_load_dwordx4 v[0:3], v4, s[0:3], 0 offen"
    wait = ["s_waitcnt vmcnt(16)", "s_barrier"]
    assert loads_after_first_stage([copy] * 8 + [weight] * 12 + wait, 16) == 16
    assert loads_after_first_stage([weight] + [copy] * 8 + [weight] * 11 + wait, 16) == 15
