"""What a preconditioner's setup does where device memory ends (CPU only): the library's HIP calls
go to a stand-in that hands out addresses up to a budget and runs nothing."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <map>
static size_t budget = ~(size_t)0, used = 0, peak = 0;
static std::map<uintptr_t, size_t> live;
static uintptr_t next_address = (uintptr_t)1 << 40;
static int last = 0;
static int take(void **p, size_t n) {
    if (n > budget - used) return last = 2;  // hipErrorOutOfMemory
    *p = (void *)next_address;
    live[next_address] = n;
    next_address += (n + 4095) / 4096 * 4096;
    used += n;
    if (used > peak) peak = used;
    return 0;
}
static int give(void *p) {
    if (!p) return 0;
    auto it = live.find((uintptr_t)p);
    if (it == live.end()) return last = 1;
    used -= it->second;
    live.erase(it);
    return 0;
}
extern "C" {
void standin_budget(size_t b) { budget = b, peak = used; }
size_t standin_used() { return used; }
size_t standin_peak() { return peak; }
int hipMalloc(void **p, size_t n) { return take(p, n); }
int hipMallocAsync(void **p, size_t n, void *) { return take(p, n); }
int hipFree(void *p) { return give(p); }
int hipFreeAsync(void *p, void *) { return give(p); }
int hipMemcpyAsync(void *dst, const void *, size_t n, int kind, void *) {
    if (kind == 2) memset(dst, 0, n);  // device to host: no zero pivots
    return 0;
}
int hipMemsetAsync(void *, int, size_t, void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { return *s = (void *)8, 0; }
int hipStreamDestroy(void *) { return 0; }
int hipStreamWaitEvent(void *, void *, unsigned) { return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { return *e = (void *)8, 0; }
int hipEventRecord(void *, void *) { return 0; }
int hipEventDestroy(void *) { return 0; }
int hipGetLastError() { const int e = last; last = 0; return e; }
int hipLaunchKernel(const void *, unsigned long, unsigned, unsigned long, unsigned, void **, size_t, void *) { return 0; }
int __hipPushCallConfiguration(unsigned long, unsigned, unsigned long, unsigned, size_t, void *) { return 0; }
int __hipPopCallConfiguration(void *, void *, size_t *, void **) { return 0; }
}
"""

CHILD = r"""
import ctypes, json, sys
standin = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
for f in ("standin_used", "standin_peak"):
    getattr(standin, f).restype = ctypes.c_size_t
sys.path.insert(0, sys.argv[2])
from paper_1709_08803_amd import bim as B
L = B.lib()
N, M, storage = int(sys.argv[3]), int(sys.argv[4]), int(sys.argv[5])
prob = B._Problem(N, M, -1.0 * N, 1.0, 0.0, 1.0, 1, 0.05, 1.2, 4096, 4096, 4096, 0.0)
out = []
budget = 2 ** 62
while True:
    standin.standin_budget(ctypes.c_size_t(budget))
    h = ctypes.c_void_p()
    rc = L.precond_setup_ex(ctypes.byref(prob), -1, storage, ctypes.byref(h), None)
    out.append(dict(rc=rc, bytes=L.precond_bytes(h) if rc == 0 else 0, peak=standin.standin_peak()))
    if rc == 0:
        L.precond_destroy(h)
    assert standin.standin_used() == 0, "memory left behind"
    if rc:
        break
    budget = standin.standin_peak() - 1  # one byte less than it just took
print(json.dumps(out))
"""


@pytest.mark.parametrize("N,M,storage,forms", [(90, 91, 0, 3), (600, 5, 0, 2), (40, 21, 0, 1), (90, 91, 1, 1)],
                         ids=["tables-and-groups", "tables", "blocks", "fp32"])
def test_setup_takes_the_fastest_form_that_fits(tmp_path, N, M, storage, forms):
    (tmp_path / "standin.cpp").write_text(STAND_IN)
    lib = str(tmp_path / "standin.so")
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-o", lib, str(tmp_path / "standin.cpp")])
    r = subprocess.run([sys.executable, "-c", CHILD, lib, ROOT, str(N), str(M), str(storage)], capture_output=True,
                       text=True)
    assert r.returncode == 0, r.stderr
    runs = json.loads(r.stdout.strip().splitlines()[-1])
    print(runs)
    # every form in turn as the budget falls below what the one before took; then out of memory
    assert [q["rc"] for q in runs] == [0] * forms + [-3]
    sizes = [q["bytes"] for q in runs[:-1]]
    assert sizes == sorted(sizes, reverse=True) and len(set(sizes)) == forms
    s = N + 1
    w = 2 * max(1, min(10, round(M / 6))) + 1
    blocks = 8 * (4 * M * s * s + 4 * M * w * s * s + (M * s) ** 2 + 4 * M * s)
    if storage == 0:  # the last form is the stored blocks alone (arrays rounded up to 256 bytes)
        assert 0 <= sizes[-1] - blocks < 10 * 256
