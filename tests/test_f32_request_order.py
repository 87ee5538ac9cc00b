"""The fp32 products wait for a chunk of W in LDS by counting the requests behind it, so the built code has to issue them in that order: on every path through
a kernel, no LDS read may follow a barrier that a request of W passed without having landed.  Read from the device code in the library (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2509_22681_amd import build as build_mod

LLVM = "/opt/rocm/llvm/bin"
pytestmark = pytest.mark.skipif(not os.path.exists(f"{LLVM}/llvm-objdump"), reason="needs llvm-objdump")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Packed instances with counted waits: name -> [(address, instruction, branch target)]"""
    tmp = tmp_path_factory.mktemp("code")
    lib = shutil.copy(build_mod.LIB, tmp)
    subprocess.run([f"{LLVM}/llvm-objdump", "--offloading", lib], cwd=tmp, check=True, capture_output=True)
    found = {}
    for part in sorted(tmp.glob("*gfx950*")):
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", part], check=True, capture_output=True, text=True).stdout
        for m in re.finditer(r"^[0-9a-f]+ <(\S*15gemm_f32_kernelI(?:Li\d+E){5}Lb1ELb1E\S*)>:\n(.*?)(?=^[0-9a-f]+ <\S+>:\n|\Z)", text, re.S | re.M):
            code = []
            base = None
            for line in m.group(2).splitlines():
                i = re.match(r"\s*(.*?)\s*// ([0-9A-F]+):(?:.*<\S+?\+0x([0-9a-f]+)>)?", line)
                if i:
                    addr = int(i.group(2), 16)
                    base = addr if base is None else base
                    code.append((addr, i.group(1), base + int(i.group(3), 16) if i.group(3) else None))
            found[m.group(1)] = code
    return found


def unlanded_reads(code):
    """Addresses of LDS reads that some path reaches with a request of W pending from before the last barrier.  Pending requests, oldest first: "w" for W
    by LDS-DMA, "W" once a barrier has been passed, "l" for any other."""
    at = {a: i for i, (a, _, _) in enumerate(code)}
    seen, todo, bad = set(), [(0, "")], set()
    while todo:
        i, pending = todo.pop()
        while i < len(code) and (i, pending) not in seen:
            seen.add((i, pending))
            addr, text, target = code[i]
            op = text.split()[0]
            if op.startswith("global_load_lds"):
                pending += "w"
            elif op.startswith(("global_", "flat_", "scratch_", "buffer_load", "buffer_store")):
                pending += "l"
            elif op == "s_waitcnt" and "vmcnt" in text:
                n = int(re.search(r"vmcnt\((\d+)\)", text).group(1))
                pending = pending[len(pending) - n:] if n < len(pending) else pending
            elif op == "s_barrier":
                pending = pending.replace("w", "W")
            elif op.startswith("ds_read") and "W" in pending:
                bad.add(hex(addr))
                break
            if "W" not in pending and "w" not in pending:
                pending = ""                       # (only what stands behind a request of W counts)
            pending = pending[-63:]
            if op == "s_endpgm":
                break
            if op.startswith(("s_branch", "s_cbranch")):
                assert target in at, text
                if op == "s_branch":
                    i = at[target]
                    continue
                todo.append((at[target], pending))
            i += 1
    return sorted(bad)


def split_groups(code):
    """Addresses of requests of W that another request stands between and the one before them: the count behind a chunk of W begins with its last request."""
    bad, state = [], ""
    for addr, text, _ in code:
        op = text.split()[0]
        if op.startswith("global_load_lds"):
            if state == "wl":
                bad.append(hex(addr))
            state = "w"
        elif op.startswith("global_load") and state:
            state = "wl"
        elif op == "s_barrier" or "vmcnt" in text:
            state = ""
    return bad


def test_requests_of_w_have_landed_before_they_are_read(kernels):
    assert len(kernels) >= 8, sorted(kernels)
    for name, code in kernels.items():
        assert any(t.startswith("global_load_lds") for _, t, _ in code), name
        assert split_groups(code) == [], name
        assert unlanded_reads(code) == [], name


@pytest.mark.parametrize("order,ok", [("w l l vmcnt(2)", True), ("w l l vmcnt(3)", False), ("l w l vmcnt(2)", False), ("w w l l l vmcnt(2)", True)])
def test_the_check_itself(order, ok):
    ops = {"w": "global_load_lds_dwordx4 v1, s[0:1]", "l": "global_load_dwordx4 v[0:3], v1, s[0:1]"}
    text = [ops.get(o, f"s_waitcnt {o}") for o in order.split()] + ["s_barrier", "ds_read_b128 v[0:3], v0", "s_endpgm"]
    assert (unlanded_reads([(8 * i, t, None) for i, t in enumerate(text)]) == []) == ok
