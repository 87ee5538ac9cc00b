"""Properties of the launch code that need no GPU to check."""
import ctypes
import re
import subprocess
import sys
from pathlib import Path

import pytest

from paper_2509_22681_amd import build as build_mod

CSRC = Path(build_mod.CSRC)


def constants(source, pattern):
    return {k: int(v) for k, v in re.findall(pattern + r" = (\d+)(?=[,;])", (CSRC / source).read_text())}


# Limits of the key-ordered attention, as the source has them
KEY_ORDERED = constants("attn_mfma.hip", r"\bkAttnSeq(\w+)")


def library():
    """The library's own rules (internal symbols: the launches call them)."""
    from paper_2509_22681_amd import binding
    return binding._lib


def key_ordered(grid, n_items, n_cand, longest):
    f = library()._ZN5flame16attn_key_orderedEiiii
    f.restype = ctypes.c_bool
    return f(grid, n_items, n_cand, longest)


def layer_fused(d):
    f = library()._ZN5flame11layer_fusedEi
    f.restype = ctypes.c_bool
    return f(d)


def test_layer_kernel_runs_for_its_widths():
    """By width alone, at every size of a launch: this is the whole rule (test_gpu_layer_kernel.py counts the launches)."""
    assert [d for d in range(32, 1025, 32) if layer_fused(d)] == [128, 192, 256]
    call = re.search(r"const bool fused = (.*?);", (CSRC / "api.cpp").read_text()).group(1)
    assert re.findall(r"\w+_fused\w*\([^)]*\)", call) == ["layer_fused(d)"]


# (shortest and longest history of the row, limit where history tiles prevail)
@pytest.mark.parametrize("lo,hi,limit", [("History", "LongHistory", "Workgroups"), ("LongHistory", "LongerHistory", "LongWorkgroups"), ("LongerHistory", None, "LongerWorkgroups")])
def test_key_ordered_attention_runs_up_to_its_limits(lo, hi, limit):
    k = KEY_ORDERED
    assert len(k) == 6
    n = k[limit]
    for longest in (k[lo], k[hi] - 1 if hi else 1 << 20):
        assert key_ordered(n, n, n // 2, longest) and not key_ordered(n + 1, n + 1, (n + 1) // 2, longest)
        m = k["Workgroups"]                      # candidate tiles prevail
        assert key_ordered(m, m, m // 2 + 1, longest) and not key_ordered(m + 1, m + 1, m // 2 + 2, longest)
    assert not key_ordered(1, 1, 0, k["History"] - 1)


def test_the_plane_that_the_layer_kernel_overwrites_is_not_restrict():
    """The layer kernel reads U of its layer and writes U of the next to the same plane: a promise that U does not change would be a false one."""
    params = re.search(r"void layer_kernel\((.*?)\)\s*\{", (CSRC / "layer_mfma.hip").read_text(), re.S).group(1)
    by_name = {p.split()[-1].lstrip("*"): p for p in params.split(",")}
    assert "__restrict__" not in by_name["U"] and "__restrict__" in by_name["O"]


RUNTIME = r"""
// the two runtime calls behind the limit, recorded: device, kernel, bytes
static int device = 0, calls = 0, fail = 0, log_[64][2];
static const void *kernels[64];
extern "C" void stub_device(int d) { device = d; }
extern "C" void stub_fail(int n) { fail = n; }
extern "C" int stub_calls() { return calls; }
extern "C" int stub_log(int i, int what) { return log_[i][what]; }
extern "C" const void *stub_kernel(int i) { return kernels[i]; }
extern "C" int hipGetDevice(int *d) { *d = device; return 0; }
extern "C" int hipFuncSetAttribute(const void *f, int, int bytes) {
  if (fail > 0) { --fail; return 1; }
  kernels[calls] = f; log_[calls][0] = device; log_[calls][1] = bytes; ++calls;
  return 0;
}
"""

DRIVE = r"""
import ctypes as C, sys
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)       # in front of the library, so that its calls come here
lib = C.CDLL(sys.argv[2])
stub.stub_kernel.restype = C.c_void_p
class Shape(C.Structure):
    _fields_ = [(n, C.c_int) for n in "d H dh n_layers n_buckets D".split()] + [("eps", C.c_float), ("alpha", C.c_float), ("ws_rows", C.c_int64),
                ("softmax", C.c_int), ("latency", C.c_int)]
def shape(dh, softmax, latency):
    return Shape(2 * dh, 2, dh, 1, 16, 64, 1e-6, 1.0, 512, softmax, latency)
setups = [lambda s=shape(dh, sm, lat): lib._ZN5flame10attn_setupERKNS_5ShapeE(C.byref(s)) for dh in (32, 64) for sm in (0, 1) for lat in (0, 1)]
setups += [lambda d=d: lib._ZN5flame11layer_setupEi(d) for d in (128, 192, 256)]
for i, device in enumerate((0, 1, 63, 64, 1, 0)):
    stub.stub_device(device)
    if i == 1:
        stub.stub_fail(1)                            # one failure: reported, and made good by the next call
        assert [f() for f in setups].count(1) == 1
    assert all(f() == 0 for f in setups)
seen = {}
for i in range(stub.stub_calls()):
    seen.setdefault(stub.stub_log(i, 0), []).append((stub.stub_kernel(i), stub.stub_log(i, 1)))
want = sorted(seen[0])
# pointwise attention: 2 head widths x (throughput, two latency configurations); softmax: 2 x two latency ones; three widths of the layer kernel
assert len(want) == len(set(k for k, _ in want)) == 13, want
for device in (1, 63):
    assert sorted(seen[device]) == want, device
assert set(seen[64]) == set(want)                    # past the bits: every time
"""


def test_lds_limits_are_raised_on_every_device(tmp_path):
    """A kernel's limit belongs to one device: handles on a second one raise it there too, and a failure is not remembered."""
    stub = tmp_path / "libstub.so"
    subprocess.run(["g++", "-shared", "-fPIC", "-x", "c++", "-", "-o", stub], input=RUNTIME, text=True, check=True)
    r = subprocess.run([sys.executable, "-c", DRIVE, stub, build_mod.LIB], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
