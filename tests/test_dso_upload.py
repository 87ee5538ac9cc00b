"""Micro-batches of the request orchestrator without a GPU: the runtime and the forward are stand-ins, "device" memory is host memory.  What reaches the forward is whole and in place
however a batch was uploaded and whatever flushed it; short requests share their uploads; a failed upload ahead of the flush is not an error of the submit that made it."""
import re
import subprocess
import sys

from paper_2509_22681_amd import build as build_mod

STAND_INS = r"""
#include <cstdlib>
#include <cstring>
#include <cstdint>
static int copies = 0, fail = 0, last_error = 0;
extern "C" {
void stub_fail(int n) { fail = n; }
int stub_copies() { const int n = copies; copies = 0; return n; }
int hipGetLastError() { const int e = last_error; last_error = 0; return e; }
const char *hipGetErrorString(int) { return "made to fail"; }
int hipMalloc(void **p, size_t n) { *p = calloc(n ? n : 1, 1); return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = calloc(n ? n : 1, 1); return 0; }
int hipFree(void *p) { free(p); return 0; }
int hipHostFree(void *p) { free(p); return 0; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *) {
  if (kind == 1) {                                   // to the device
    if (fail > 0) { --fail; return last_error = 1; }
    ++copies;
  }
  memcpy(d, s, n);
  return 0;
}
int hipStreamCreateWithFlags(void **s, unsigned) { *s = malloc(1); return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamDestroy(void *s) { free(s); return 0; }
int hipEventCreateWithFlags(void **s, unsigned) { *s = malloc(1); return 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventSynchronize(void *) { return 0; }
int hipEventDestroy(void *s) { free(s); return 0; }
int hipDeviceSynchronize() { return 0; }
// a handle that knows its width; the score of a candidate: the sum of its row and of its request's history (fp32 rows)
int flame_gr_create(const int32_t *cfg, void **out) { *out = malloc(1); return 0; }
int flame_gr_destroy(void *h) { free(h); return 0; }
const char *flame_gr_last_error(const void *) { return ""; }
int flame_gr_forward(void *, const void *, const float *h, const int32_t *ho, const float *c, const int32_t *co, int32_t n, float *out, void *) {
  if (hipGetLastError() != 0) return -3;             // as the launches of the real one ask
  const int d = 64;
  for (int r = 0; r < n; ++r) {
    float hist = 0.f;
    for (int64_t i = (int64_t)ho[r] * d; i < (int64_t)ho[r + 1] * d; ++i) hist += h[i];
    for (int k = co[r]; k < co[r + 1]; ++k) {
      float s = hist;
      for (int i = 0; i < d; ++i) s += c[(int64_t)k * d + i];
      out[k] = s;
    }
  }
  return 0;
}
}
"""

DRIVE = r"""
import ctypes as C, sys
import numpy as np
stub = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)       # in front of the library, so that its calls come here
sys.path.insert(0, sys.argv[2])
piece = int(sys.argv[3])
from paper_2509_22681_amd import binding as B
d, batch, top, hmax = 64, 6, 64, 3 * piece // 256
rng = np.random.default_rng(0)

def request(n, m):
    # small whole numbers, of which few are not zero: the sums are exact in any order
    h, c = np.zeros((n, d), np.float32), rng.integers(-8, 8, (m, d)).astype(np.float32)
    if n: h[rng.integers(0, n, 64), rng.integers(0, d, 64)] = rng.integers(-100, 100, 64)
    return h, c, np.full(m, np.nan, np.float32), h.sum() + c.sum(1)

dso = B.flame_dso_create(B.make_config(1, d, 2, 16, 64, "f32"), B.flame_gr_weights(), hmax, [16, top], 2, explicit_shapes=2, max_batch=batch)

def submit(r):
    return B.flame_dso_submit_jagged(dso, r[0], r[1], r[2])

def check(rs):
    for r in rs:
        assert np.array_equal(r[2], r[3]), (r[0].shape, r[2][:4], r[3][:4])

long, short = (piece + 255) // 256, 5
sizes = [[long, long, short], [short, long, short, long], [long + 7, 0, short, 0, long], [0, long], [short] * 6, [long] * 6, [short, 2 * long, short, short, short, short]]
for how in ("wait", "drain", "flush", "full"):
    for ns in sizes:
        if how == "full" and len(ns) < batch:        # a request of more candidates than the largest profile is split; the pieces fill the batch
            rs = [request(n, 17) for n in ns[:2]] + [request(ns[0], top * 4 + 3)]
        else:
            rs = [request(n, 1 + 7 * i) for i, n in enumerate(ns)]
        tickets = [submit(r) for r in rs]
        if how == "wait":
            for t in tickets: B.flame_dso_wait(dso, t)
        elif how == "flush":
            B.flame_dso_flush(dso)
            for t in tickets[::-1]: B.flame_dso_wait(dso, t)
        else:
            B.flame_dso_drain(dso)
        check(rs)

# copies of a batch: short requests two, however many they are; long ones two each, of rows there are
stub.stub_copies()
for ns, want in (([short] * 5, 2), ([0] * 5, 1), ([long] * 5, 10), ([long, short, short, short, short], 4)):
    rs = [request(n, 3) for n in ns]
    for r in rs: submit(r)
    B.flame_dso_drain(dso)
    check(rs)
    got = stub.stub_copies()
    assert got == want, (ns, got, want)

# an upload ahead of the flush fails: the submit still gives its ticket, nothing is lost, and no error stays behind for the forward
for n_fail in (1, 2):
    rs = [request(long, 9), request(long, 4), request(short, 2)]
    stub.stub_fail(n_fail)
    tickets = [submit(r) for r in rs]
    for t in tickets: B.flame_dso_wait(dso, t)
    check(rs)
# one that lasts is reported by the flush
r = request(long, 3)
stub.stub_fail(100)
t = submit(r)
try:
    B.flame_dso_wait(dso, t)
    raise SystemExit("the failure was not reported")
except B.FlameGRError as e:
    assert e.code == -3, e.code
stub.stub_fail(0)
stub.hipGetLastError()
B.flame_dso_destroy(dso)
"""


def test_batches_are_whole_however_they_were_uploaded(tmp_path):
    with open(f"{build_mod.CSRC}/dso.cpp") as f:
        m = re.search(r"kUploadBytes = \(size_t\)(\d+) << (\d+);", f.read())
    piece = int(m.group(1)) << int(m.group(2))
    stub = tmp_path / "libstandin.so"
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-x", "c++", "-", "-o", stub], input=STAND_INS, text=True, check=True)
    r = subprocess.run([sys.executable, "-c", DRIVE, stub, build_mod.HERE + "/..", str(piece)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
