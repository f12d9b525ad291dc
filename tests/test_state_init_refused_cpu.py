"""albireo_penalty_state_init where the runtime refuses the LDS of the bitmap kernel, or the device index is
past the table of devices: the call goes to the sort kernel, which serves every vocabulary.  The library's
host side runs here against stand-ins for the HIP calls it makes, loaded ahead of it into a process of its own;
they note the kernel that is launched."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_01927_amd", "libalbireo.so")

STANDINS = r"""
#include <stddef.h>
#include <string.h>
typedef struct { unsigned x, y, z; } dim3_t;
static struct { const void* fn; const char* name; } table[4096];
static int n_table, device, refuse, last_error;
static const char* launched = "";
static struct { dim3_t g, b; size_t lds; void* stream; } pushed;
void** __hipRegisterFatBinary(const void* d) { static void* h; (void)d; return &h; }
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* fn, char* dev, const char* name, unsigned lim, void* a, void* b,
                           void* c, void* d, int* w) {
  (void)h; (void)dev; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
  if (n_table < 4096) { table[n_table].fn = fn; table[n_table++].name = name; }
}
void __hipRegisterVar(void** h, void* v, char* a, char* b, int e, size_t s, int c, int g) {
  (void)h; (void)v; (void)a; (void)b; (void)e; (void)s; (void)c; (void)g;
}
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t lds, void* stream) {
  pushed.g = g; pushed.b = b; pushed.lds = lds; pushed.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* g, dim3_t* b, size_t* lds, void** stream) {
  *g = pushed.g; *b = pushed.b; *lds = pushed.lds; *stream = pushed.stream;
  return 0;
}
int hipGetDevice(int* d) { *d = device; return 0; }
int hipFuncSetAttribute(const void* f, int a, int v) {
  (void)f; (void)a; (void)v;
  if (refuse) last_error = 1;
  return refuse;
}
int hipGetLastError(void) { int e = last_error; last_error = 0; return e; }
int hipLaunchKernel(const void* fn, dim3_t g, dim3_t b, void** args, size_t lds, void* stream) {
  (void)g; (void)b; (void)args; (void)lds; (void)stream;
  launched = "?";
  for (int i = 0; i < n_table; ++i) if (table[i].fn == fn) launched = table[i].name;
  return 0;
}
void standin_setup(int d, int r) { device = d; refuse = r; launched = ""; }
const char* standin_launched(void) { return launched; }
"""

CHILD = r"""
import ctypes, json, sys
sys.path.insert(0, "")
stand = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
stand.standin_launched.restype = ctypes.c_char_p
class State(ctypes.Structure):
    _fields_ = [("cap", ctypes.c_int32)] + [(n, ctypes.c_void_p) for n in ("ids", "counts", "len", "flags")]
init = lib.albireo_penalty_state_init
init.argtypes = [ctypes.POINTER(State)] + [ctypes.c_int64] * 2 + [ctypes.c_void_p] * 2 + [ctypes.c_int64] + \
    [ctypes.c_void_p] * 2 + [ctypes.c_int64, ctypes.c_void_p]
st = State(64, 16, 16, 16, 16)  # never read: nothing is launched
got = []
for device, refuse, V in json.loads(sys.argv[3]):
    stand.standin_setup(device, refuse)
    rc = init(ctypes.byref(st), 4, V, None, None, 0, None, None, 0, None)
    got.append([rc, stand.standin_launched().decode()])
print(json.dumps(got))
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("standins")
    src, so = str(d / "standins.c"), str(d / "libstandins.so")
    with open(src, "w") as f:
        f.write(STANDINS)
    subprocess.check_call(["gcc", "-O1", "-shared", "-fPIC", src, "-o", so])

    def call(cases):
        out = subprocess.run([sys.executable, "-c", CHILD, so, LIB, json.dumps(cases)], capture_output=True, text=True,
                             timeout=120)
        assert out.returncode == 0, out.stderr
        return json.loads(out.stdout)

    return call


def _sort(name):
    return "k_state_init" in name and "bitmap" not in name


@pytest.mark.parametrize("V", [1, 32000, 128256, 393216])
def test_refused_lds_takes_the_sort_kernel(run, V):
    (rc, name), (rc64, name64), (rc_ok, name_ok) = run([[0, 1, V], [64, 0, V], [1, 0, V]])
    assert rc == 0 and _sort(name), (rc, name)
    assert rc64 == 0 and _sort(name64), (rc64, name64)
    assert rc_ok == 0 and "bitmap" in name_ok  # a device that allows it


def test_wide_vocabulary_takes_the_sort_kernel(run):
    (rc, name), = run([[0, 0, 393217]])
    assert rc == 0 and _sort(name), (rc, name)
