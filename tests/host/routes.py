"""Runs the library's host code against the recorder of recording_hip.cpp, in a process of its own (no GPU, no torch).

`run(code)` executes `code` there with what PRELUDE defines and returns what it printed, as a list of lines."""
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))
LIB = os.environ.get("RMSNL_LIB") or os.path.join(ROOT, "paper_2405_05751_amd", "librmsnl.so")

PRELUDE = '''
import ctypes, re, sys, threading
rec = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
V, I, F, L, Z = ctypes.c_void_p, ctypes.c_int, ctypes.c_float, ctypes.c_int64, ctypes.c_size_t
rec.rec_capture.argtypes = [V, I]
rec.rec_take.restype = ctypes.c_char_p
rec.rec_malloc_bytes.restype = Z
for name in ("rmsnorm_linear", "rmsnorm_linear_noalloc", "rmsnorm_gated_mlp"):
    getattr(lib, name).argtypes = [V, V, V, F, V, L, L, L, I, V]
lib.rl_qknorm_attention.argtypes = [V] * 7 + [F, V] + [L] * 4 + [I, V]
lib.matmul.argtypes = [V, V, V, L, L, L, I, V]
lib.rl_workspace_bytes.argtypes = [L, L, L, I]
lib.rl_workspace_bytes.restype = Z
lib.rl_set_workspace.argtypes = [V, Z]
lib.rl_last_error.restype = ctypes.c_char_p
F16, BF16, F32 = 0, 1, 2
P = [V((i + 1) << 44) for i in range(8)]                 # buffers of the caller

def linear(M, K, N, dt=BF16, stream=0, fn="rmsnorm_linear"):
    return getattr(lib, fn)(P[0], P[1], P[2], 1e-5, P[3], M, K, N, dt, V(stream))

def qknorm(B, H, S, D, dt=BF16, stream=0):
    return lib.rl_qknorm_attention(*P[:7], 1e-5, P[7], B, H, S, D, dt, V(stream))

def last():
    v = [I(), I(), I(), I()]
    assert lib.rl_last_launch(*[ctypes.byref(x) for x in v]) == 0
    return tuple(x.value for x in v)                     # variant, columns, slabs, workgroups

class Launch:
    def __init__(self, line):
        words = line.split()
        self.name = re.match(r"_ZN5rmsnl(?:\\d+_GLOBAL__N_1)?(\\d+)(\\w+)", words[0])
        self.name = self.name.group(2)[:int(self.name.group(1))] if self.name else words[0]
        self.mangled = words[0]
        self.grid, self.block, self.lds, self.stream = map(int, words[1:5])
        self.words = list(map(int, words[5:]))           # of the argument a test watches

def launches():
    return [Launch(l) for l in rec.rec_take().decode().splitlines()]

def names():
    return [l.name for l in launches()]
'''


def run(code):
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "recording_hip.so")
        subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "recording_hip.cpp")], check=True)
        r = subprocess.run([sys.executable, "-c", PRELUDE + code, so, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    return r.stdout.splitlines()
