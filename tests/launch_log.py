"""What libchai.so would launch, on a machine without a GPU: the library is loaded in a child process whose HIP runtime calls
are answered by a small stand-in that writes every launch down.  Kernels are named by their mangled names."""
import json
import os
import subprocess
import sys
import textwrap

from paper_2403_08058_amd import build

_STAND_IN = r"""
#include <stddef.h>
#include <stdint.h>
#include <map>
#include <string>
#include <vector>
struct dim3_ { uint32_t x, y, z; };
static std::map<const void *, std::string> &names() { static std::map<const void *, std::string> m; return m; }
static std::map<const void *, int> leave;
struct Launch { const char *name; unsigned long long grid, block, lds, allowed; };
static std::vector<Launch> seen;
extern "C" {
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names()[host] = name;
}
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void *f, int, int value) { leave[f] = value; return 0; }
int hipExtLaunchKernel(const void *f, dim3_ g, dim3_ b, void **, size_t lds, void *, void *, void *, int)
{
    seen.push_back({names()[f].c_str(), 1ull * g.x * g.y * g.z, 1ull * b.x * b.y * b.z, lds, leave.count(f) ? 1ull * leave[f] : 0ull});
    return 0;
}
size_t launches_count() { return seen.size(); }
const char *launches_name(size_t i) { return seen[i].name; }
unsigned long long launches_value(size_t i, int what) { const Launch &l = seen[i]; return what == 0 ? l.grid : what == 1 ? l.block : what == 2 ? l.lds : l.allowed; }
void launches_clear() { seen.clear(); }
}
"""

_CHILD = """
import ctypes, json, os
S = ctypes.CDLL(os.environ["CHAI_STAND_IN"], mode=ctypes.RTLD_GLOBAL)        # found before the runtime, which comes with the library
S.launches_count.restype = ctypes.c_size_t
S.launches_name.restype = ctypes.c_char_p
S.launches_name.argtypes = [ctypes.c_size_t]
S.launches_value.restype = ctypes.c_ulonglong
S.launches_value.argtypes = [ctypes.c_size_t, ctypes.c_int]
L = ctypes.CDLL(os.environ["CHAI_LIBRARY"])
P = ctypes.c_void_p(1 << 20)             # a pointer that is never followed
N = ctypes.c_size_t(1 << 60)

def launches():
    "kernel, workgroups, threads, dynamic LDS and the LDS that the kernel has leave for, of each launch since the last call"
    got = [(S.launches_name(i).decode(),) + tuple(S.launches_value(i, w) for w in range(4)) for i in range(S.launches_count())]
    S.launches_clear()
    return got
"""


def run(tmp_path, code):
    """What `code` assigns to `result` (plain values), run behind _CHILD."""
    src, lib = str(tmp_path / "stand_in.cpp"), str(tmp_path / "stand_in.so")
    with open(src, "w") as f:
        f.write(_STAND_IN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", src, "-o", lib], check=True)
    env = dict(os.environ, CHAI_STAND_IN=lib, CHAI_LIBRARY=build.LIB)
    done = subprocess.run([sys.executable, "-c", _CHILD + textwrap.dedent(code) + "\nprint(json.dumps(result))"], env=env,
                          capture_output=True, text=True)
    assert done.returncode == 0, done.stderr
    return json.loads(done.stdout)
