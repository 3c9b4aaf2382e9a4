"""The order of the memory requests that gemm_duo_kernel's waits count on, in the library as it was built: a wait for all but N
requests has landed a stage only if exactly N were issued behind it."""
import os
import re
import subprocess

import pytest

from paper_2501_06589_amd import ladder

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
X = 4     # direct-to-LDS loads of activations per wavefront and stage


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    if not os.path.exists(ladder.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    at = tmp_path_factory.mktemp("code")
    lib = at / "lib.so"
    lib.symlink_to(ladder.LIB_PATH)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], cwd=at, check=True, capture_output=True)
    return sorted(str(f) for f in at.iterdir() if "gfx950" in f.name)


def spans(text):
    """Per stretch of code that ends at a barrier: its requests ("x" to LDS, "w" to registers) and the count waited for in front of it."""
    out, ops, count = [], "", None
    for line in text.splitlines():
        m = re.match(r"\s+(\S+)\s*(.*?)(//|$)", line)
        if not m:
            continue
        op, args = m.group(1), m.group(2)
        if op.startswith(("buffer_load", "global_load", "flat_load", "scratch_load")):
            ops += "x" if re.search(r"\blds\b", args) else "w"
        elif op == "s_waitcnt" and "vmcnt" in args:
            count = int(re.search(r"vmcnt\((\d+)\)", args).group(1))
        elif op == "s_barrier":
            out.append((ops, count))
            ops, count = "", None
    return out


def landed(found, jt):
    """The first three barriers: X(0) has landed behind the prologue's, X(s + 1) behind the others."""
    issued = ""
    for n, (ops, count) in enumerate(found[:3]):
        issued += ops
        at = -1
        for _ in range((n + 1) * X):      # the last load of stage n
            at = issued.index("x", at + 1)
        if count is None or count > len(issued) - 1 - at:
            return False
    return len(found) >= 3 and issued.startswith("x" * X + "w" * jt)


@pytest.mark.parametrize("jt", [2, 3, 4])
def test_stages_have_landed_where_they_are_read(code_objects, jt):
    name = f"_Z15gemm_duo_kernelILi{jt}EEv8GemmArgs"
    text = "".join(subprocess.run([OBJDUMP, "-d", "--disassemble-symbols=" + name, f], check=True, capture_output=True, text=True).stdout
                   for f in code_objects)
    found = spans(text)
    assert landed(found, jt), found[:4]
    # weights requested in front of the first activations (the wait then lets stage 0 be read before it is there): not accepted
    ops, count = found[0]
    assert not landed([("w" * ops.count("w") + "x" * ops.count("x"), count)] + found[1:], jt)
    assert not landed([("w" * jt + "x" * X + ops[X + jt:], count)] + found[1:], jt)
