"""Which kernels a call of the library would launch, without a GPU: a stand-in for the handful of HIP functions that the
library calls, loaded in front of the real ones in a child process, writes every launch down instead of making it."""
from __future__ import annotations

import json
import os
import subprocess
import sys
from dataclasses import dataclass

from paper_2403_07816_amd import binding as B

STAND_IN = r"""
#include <cstdio>
#include <cstdlib>
#include <map>
#include <string>
#include <cxxabi.h>
struct dim3 { unsigned x, y, z; };
static std::map<const void*, std::string> names;
static std::string log_text;
static dim3 grid, block;
static size_t shared;
extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  int status = 0;
  char* plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  names[host] = plain ? plain : name;
  free(plain);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, void*) { grid = g; block = b; shared = s; return 0; }
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, void** stream) {
  *g = grid; *b = block; *s = shared; *stream = nullptr;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t s, void*) {
  char line[160];
  // first argument of a kernel, as a pointer: which part of a tensor a launch starts at
  std::snprintf(line, sizeof line, "%u %u %u %u %u %u %zu %llu ", g.x, g.y, g.z, b.x, b.y, b.z, s,
                *static_cast<unsigned long long*>(args[0]));
  log_text += line + names[f] + "\n";
  return 0;
}
int hipGetDevice(int* dev) { *dev = 0; return 0; }
int hipDeviceGetAttribute(int* value, int, int) { *value = 256; return 0; }   // compute units
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipGetLastError() { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = reinterpret_cast<void*>(0x1000); return 0; }
const char* taken() { static std::string out; out.swap(log_text); log_text.clear(); return out.c_str(); }
}
"""

CHILD = r"""
import ctypes, json, sys, time
log = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
log.taken.restype = ctypes.c_char_p
lib = ctypes.CDLL(sys.argv[2])
out = []
for name, args in json.load(sys.stdin):
    fn = getattr(lib, name)
    fn.restype = ctypes.c_size_t if name.endswith("bytes") else ctypes.c_int
    args = [(ctypes.c_float if isinstance(a[0], float) else ctypes.c_void_p).__mul__(len(a))(*a) if isinstance(a, list) else
            ctypes.c_float(a) if isinstance(a, float) else ctypes.c_int64(a) for a in args]
    start = time.perf_counter()
    rc = fn(*args)
    seconds = time.perf_counter() - start
    out.append((rc, log.taken().decode(), seconds))
print(json.dumps(out))
"""


@dataclass(frozen=True)
class Launch:
    kernel: str                # demangled name with its template arguments, without namespaces and parameters
    grid: tuple
    block: tuple
    lds: int
    first: int                 # the kernel's first argument, if that is a pointer


def _short(name):
    name = name.replace("(anonymous namespace)::", "").replace("btx::", "")
    name = name[5:] if name.startswith("void ") else name
    depth = 0
    for i, ch in enumerate(name):
        depth += (ch == "<") - (ch == ">")
        if ch == "(" and depth == 0:
            return name[:i]
    return name


def _recorded(calls, tmp_path):
    source, stand_in = os.path.join(tmp_path, "stand_in.cpp"), os.path.join(tmp_path, "stand_in.so")
    if not os.path.exists(stand_in):
        with open(source, "w") as f:
            f.write(STAND_IN)
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", source, "-o", stand_in], check=True)
    r = subprocess.run([sys.executable, "-c", CHILD, stand_in, B.LIB_PATH], input=json.dumps(calls), capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


def host_seconds(call, tmp_path):
    """The least that a call takes on the host."""
    return min(seconds for _, _, seconds in _recorded([call] * 50, tmp_path))


def launches(calls, tmp_path):
    """calls: (entry point, arguments) with pointers as integers, floats as floats and host arrays as lists; per call its status
    and its launches."""
    result = []
    for rc, text, _ in _recorded(calls, tmp_path):
        found = []
        for line in text.splitlines():
            *numbers, name = line.split(" ", 8)
            v = [int(n) for n in numbers]
            found.append(Launch(_short(name), tuple(v[:3]), tuple(v[3:6]), v[6], v[7]))
        result.append((rc, found))
    return result


P = 0x100000                   # where every tensor is said to lie: aligned, never looked at
PLENTY = 1 << 62


def forward_call(T, d, f, E, k, dtype, p=P, stride=None, save=True):
    s = stride or d * f
    return ("btx_moe_ff_forward", [p, p, p, p, dtype, s, s, T, d, f, E, k, p, p, p, p, 0, p, p if save else 0, p if save else 0,
                                   p, PLENTY, 0])


def backward_call(T, d, f, E, k, dtype, dW_dtype=None, dW2=P, stride=None):
    s, p = stride or d * f, P
    return ("btx_moe_ff_backward", [p] * 6 + [dtype, s, s, T, d, f, E, k, 0, 0, 0.0, 0.0, 0, 0, 1.0] + [p] * 11 +
            [p, p, p, p, p, dW2, dtype if dW_dtype is None else dW_dtype, p, PLENTY, 0])


def route_call(T, d, E, k, dtype, norm=False):
    lead = [P, dtype, P, 1e-5, 2 * P, P] if norm else [P, dtype]
    return ("btx_moe_norm_route" if norm else "btx_moe_route",
            lead + [P, 0, 0, T, d, E, k, 0, 0, 0.01, 1.0, 0.0] + [P] * 10 + [P, PLENTY, 0])


def adamw_call(n, dtype=B.BTX_BF16, lowp=P, master=P):
    return ("btx_adamw_step", [master, P, P, P, dtype, lowp, n, 3, 1e-4, 0.9, 0.95, 1e-8, 0.1, 0])
