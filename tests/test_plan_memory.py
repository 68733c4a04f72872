"""Device memory of a plan, on the CPU: the library runs on a stand-in for the
HIP runtime that allocates host memory up to a limit, counts what is held and
launches nothing."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HIP = r"""
#include <stdlib.h>
#include <string.h>
#include <stddef.h>
enum { kOk = 0, kOutOfMemory = 2 };
typedef struct { size_t n; char pad[48]; } Head;
static size_t held;
static int last;
size_t fake_limit = (size_t)-1;             /* bytes held at most */
int fake_dead;                              /* the table kernels report that nothing fits */
size_t fake_held(void) { return held; }
int fake_last(void) { return last; }
int hipMalloc(void** p, size_t n) {
  *p = NULL;
  if (held + n > fake_limit) return last = kOutOfMemory;
  Head* h = calloc(1, n + sizeof(Head));
  if (!h) return last = kOutOfMemory;
  h->n = n;
  held += n;
  *p = h + 1;
  return kOk;
}
int hipFree(void* p) {
  if (p) { Head* h = (Head*)p - 1; held -= h->n; free(h); }
  return kOk;
}
int hipMemcpy(void* d, const void* s, size_t n, int kind) {
  memcpy(d, s, n);
  if (fake_dead && kind == 2 && n == 16) ((int*)d)[2] = 1000;
  return kOk;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { return hipMemcpy(d, s, n, k); }
int hipGetDevice(int* d) { *d = 0; return kOk; }
int hipDeviceGetAttribute(int* v, int a, int d) { *v = 256; return kOk; }
int hipDeviceSynchronize(void) { return kOk; }
int hipStreamSynchronize(void* s) { return kOk; }
int hipFuncSetAttribute(const void* f, int a, int v) { return kOk; }
int hipFuncGetAttributes(void* a, const void* f) { return kOk; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void* f, int b, size_t l) { *n = 1; return kOk; }
int hipGetLastError(void) { int e = last; last = kOk; return e; }
const char* hipGetErrorString(int e) { return "stand-in"; }
static char symbol[4096];
int hipGetSymbolAddress(void** p, const void* s) { *p = symbol; return kOk; }
int hipLaunchKernel(const void* f, ...) { return kOk; }
int __hipPushCallConfiguration() { return kOk; }
int __hipPopCallConfiguration() { return kOk; }
void* __hipRegisterFatBinary(const void* d) { static void* h[4]; return h; }
void __hipRegisterFunction() {}
void __hipRegisterVar() {}
void __hipUnregisterFatBinary(void* h) {}
"""

RUN = r"""
import ctypes, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import importlib.util
spec = importlib.util.spec_from_file_location("mbtp_binding", sys.argv[2] + "/paper_1307_5700_amd/_lib.py")
L = importlib.util.module_from_spec(spec); spec.loader.exec_module(L)
lib = L.lib()
hip.fake_held.restype = ctypes.c_size_t
limit, dead = ctypes.c_size_t.in_dll(hip, "fake_limit"), ctypes.c_int.in_dll(hip, "fake_dead")
r = L.RfiParams(); lib.mb_rfi_defaults(ctypes.byref(r))
d = L.PlanDesc(1024, 96, 398.0, 20.0 / 1024, 51.2e-6, 0.0, 0.2, L.DTYPES["u8"], 0, r)
def make(lim, not_fit=0):
    limit.value, dead.value = lim, not_fit
    h = ctypes.c_void_p()
    st = lib.dedisp_plan_create(ctypes.byref(d), ctypes.byref(h))
    held, last = hip.fake_held(), hip.fake_last()
    if st == 0:
        assert lib.dedisp_plan_destroy(h) == 0
    print(st, held, last, hip.fake_held())
plain = 3 * 4 * 1024 * 96                  # delays and two offset tables
make(1 << 40)
make(plain + 4096)
make(1 << 40, 1)
make(plain - 1)
"""


def test_matrix_core_tables_are_optional(tmp_path):
    """The tables are allocated once the delays are known to fit, and a plan
    whose tables do not is created all the same, with no error left behind and
    nothing held after it; so is one whose delays do not fit, which allocates
    no tables.  A plan without room for its delay table is refused."""
    if shutil.which("gcc") is None:
        pytest.skip("gcc not found")
    src, so = tmp_path / "hip.c", tmp_path / "hip.so"
    src.write_text(HIP)
    subprocess.run(["gcc", "-shared", "-fPIC", "-w", "-O1", str(src), "-o", str(so)], check=True)
    out = subprocess.run([sys.executable, "-c", RUN, str(so), ROOT], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    (st, held, last, left), short, unfit, refused = [tuple(map(int, l.split())) for l in out.stdout.splitlines()]
    tables = 2 * 1024 * 96                 # at least: two one-hot bytes per DM and channel
    plain = 3 * 4 * 1024 * 96              # delays and two offset tables
    assert (st, last, left) == (0, 0, 0) and held >= plain + tables
    for st, held, last, left in (short, unfit):
        assert (st, last, left) == (0, 0, 0) and plain <= held < plain + 1024
    assert refused[0] == 2 and refused[3] == 0
