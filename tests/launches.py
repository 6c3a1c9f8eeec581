"""What the library asks of the HIP runtime, for tests of its launch rules: runs a script in a process of its
own in which hipLaunchKernel and hipGraphInstantiate pass through a small library that keeps count."""
import json
import os
import subprocess
import sys
import textwrap

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <dlfcn.h>
#include <cstring>
#include <string>
#include <vector>
struct Dim3 { unsigned x, y, z; };
static void* real = nullptr;
static std::vector<std::string> pushes;      // the particle kernels, in order, repeats dropped
static int graphs = 0;
template <class F> static F get(const char* name) { return reinterpret_cast<F>(dlsym(real, name)); }
extern "C" {
int observe(const char* path) { real = dlopen(path, RTLD_LAZY | RTLD_NOLOAD); return real != nullptr; }
int n_graphs() { return graphs; }
int n_pushes() { return (int)pushes.size(); }
const char* push_name(int i) { return pushes[i].c_str(); }
void forget() { pushes.clear(); graphs = 0; }
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void** args, size_t lds, void* stream) {
    static auto call = get<int (*)(const void*, Dim3, Dim3, void**, size_t, void*)>("hipLaunchKernel");
    static auto name = get<const char* (*)(const void*, void*)>("hipKernelNameRefByPtr");
    const char* n = name(f, stream);
    if (n && std::strstr(n, "k_push") && (pushes.empty() || pushes.back() != n)) pushes.push_back(n);
    return call(f, g, b, args, lds, stream);
}
int hipGraphInstantiate(void** exec, void* graph, void** node, char* log, size_t n) {
    static auto call = get<int (*)(void**, void*, void**, char*, size_t)>("hipGraphInstantiate");
    ++graphs;
    return call(exec, graph, node, log, n);
}
}
"""

PRELUDE = r"""
import ctypes, json, re, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
shim.push_name.restype = ctypes.c_char_p
sys.path.insert(0, sys.argv[2])
import numpy as np
import torch
path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
assert shim.observe(path.encode())
from paper_2609_17661_amd import Pic1D, workloads

def pushes():
    '''The particle kernels launched since the last call: (backend, particles per lane, window, parts).'''
    out = []
    for i in range(shim.n_pushes()):
        name = shim.push_name(i).decode()
        m = re.search(r"k_pushILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)", name) or \
            re.search(r"k_push<(\d+), (\d+), (\d+), (\d+), (\d+)>", name)
        b, ppt, ww, kind, sub = map(int, m.groups())
        out.append((b, ppt, ww, sub))
    shim.forget()
    return out
"""


def run(tmp_path, body):
    """Runs the script; what it assigns to `result` (JSON values) comes back."""
    src, lib, script = tmp_path / "shim.cpp", tmp_path / "libshim.so", tmp_path / "script.py"
    src.write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True)
    script.write_text(PRELUDE + textwrap.dedent(body) + "\nprint('RESULT ' + json.dumps(result), flush=True)\n")
    p = subprocess.run([sys.executable, "-u", str(script), str(lib), ROOT], capture_output=True, text=True, timeout=100)
    print(p.stdout[-3000:], p.stderr[-3000:], flush=True)
    assert p.returncode == 0
    return json.loads(next(l for l in p.stdout.splitlines() if l.startswith("RESULT "))[7:])
