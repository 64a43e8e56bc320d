"""Which kernels a call enqueues, on a machine without a GPU: the library in a child process whose HIP runtime only writes down the launches.
The addresses that the calls get are made up; nothing reads them, as no kernel runs."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUNTIME = r"""
#include <cstring>
#include <map>
#include <string>
#include <vector>
struct dim { unsigned x, y, z; };
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static std::string &out() { static std::string s; return s; }
static dim grid, block;
static size_t shared;
static void *stream;
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *p; return &p; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *) { names()[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim g, dim b, size_t s, void *st) { grid = g; block = b; shared = s; stream = st; return 0; }
int __hipPopCallConfiguration(dim *g, dim *b, size_t *s, void **st) { *g = grid; *b = block; *s = shared; *st = stream; return 0; }
// of the kernels that a test asks for (watch): their first two arguments, which are addresses, behind the name
static std::string watched;
void watch(const char *part) { watched = part; }
int hipLaunchKernel(const void *f, dim, dim, void **args, size_t, void *) {
    const std::string &n = names()[f];
    out() += n;
    if (!watched.empty() && n.find(watched) != std::string::npos)
        for (int i = 0; i < 2; i++) out() += " " + std::to_string(*(size_t *)args[i]);
    out() += "\n";
    return 0;
}
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { out() += "hipMemcpyAsync\n"; return 0; }
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int *v, int, int) { *v = 256; return 0; }
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return ""; }
const char *recorded() { static std::string s; s = out(); out().clear(); return s.c_str(); }
}
"""

# t(bytes, offset): something with the address and the size of a tensor, `offset` bytes past a multiple of 256
CHILD = r"""
import ctypes, json, sys, types
rt = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
rt.recorded.restype = ctypes.c_char_p
sys.modules["torch"] = types.ModuleType("torch")
sys.path.insert(0, sys.argv[2])
from paper_2510_06710_amd import binding as vb
vb._stream = lambda stream: None
class t:
    at = 1 << 40
    def __init__(self, nbytes=1 << 20, offset=0):
        self.n, self.p = nbytes, t.at + offset
        t.at += (nbytes + 511) // 256 * 256
    data_ptr = lambda self: self.p
    numel = lambda self: self.n
    element_size = lambda self: 1
def model(cfg, prepack=True):
    names = [n for n, _ in vb.vla_layer_weights._fields_]
    m = vb.DeviceModel(cfg, t(), t(), t(), [{n: t() for n in names} for _ in range(cfg.n_layers)])
    size = vb.vla_prepack_bytes(cfg)
    if size and prepack:
        vb.vla_prepack(m.handle, t(size))
    launches()
    return m
def launches():
    return rt.recorded().decode().split("\n")[:-1]
def shape(n_layers, hidden, n_heads, ffn, dtype="bf16"):
    return types.SimpleNamespace(n_layers=n_layers, hidden=hidden, n_heads=n_heads, ffn=ffn, vocab=640, n_bins=256, dtype=dtype, rms_eps=1e-5, rope_theta=1e4)
"""


def record(code, tmp_path):
    """Runs `code`, which leaves its findings in `result` (plain values), in the child and returns them."""
    src, so = tmp_path / "runtime.cpp", tmp_path / "runtime.so"
    src.write_text(RUNTIME)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD + code + "\nprint(json.dumps(result))", str(so), ROOT], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout.splitlines()[-1])
