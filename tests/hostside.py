"""The library's host side without a GPU: libsats.so in a process of its own whose
HIP runtime is tests/fake_hip (allocations, launches, synchronisations and
captures are logged, nothing runs)."""
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FAKE = os.path.join(ROOT, "tests", "fake_hip", "fake_hip.cpp")

#: what a scenario may use: lib, fwd(n, d, d_ff, ...), log() and the fake's controls
PRELUDE = r"""
import ctypes, json, os, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
fake.fake_log.restype = ctypes.c_char_p
fake.fake_held.restype = ctypes.c_size_t
fake.fake_limit.argtypes = [ctypes.c_size_t]
lib.sats_last_error.restype = ctypes.c_char_p
P, I = ctypes.c_void_p, ctypes.c_int64
PTR = 1 << 32   # device arrays that nothing reads, 16-byte aligned
AUTO, MFMA, SPLIT, COMPACT = range(4)

def log():
    '''Lines of the log since the last call, split into words; launches by kernel name.'''
    out = [l.split() for l in fake.fake_log().decode().splitlines()]
    fake.fake_clear()
    return out

def launches(lines):
    return [l[1] for l in lines if l[0] == "launch"]

def fwd(n, d, dff, dtype="bf16", L=1, noalloc=False, lut=True, rank=0):
    a = [P(PTR * k) for k in range(1, 9)]
    x, ids, wg, wu, wd, thr, table, out = a
    sizes = [I(n), I(d), I(dff), I(L), P(0)]
    if rank:
        ad = [P(PTR * k) for k in range(9, 15)]
        f = lib.sats_mlp_forward_lora if dtype == "bf16" else lib.sats_mlp_forward_lora_f32
        return f(x, ids, wg, wu, wd, *ad, I(rank), ctypes.c_float(1.0), thr, table if lut else P(0), out, *sizes,
                 P(0), P(0), P(0), P(0))
    f = lib.sats_mlp_forward_noalloc if noalloc else lib.sats_mlp_forward if dtype == "bf16" else lib.sats_mlp_forward_f32
    return f(x, ids if lut else P(0), wg, wu, wd, thr, table if lut else P(0), out, *sizes)

def reserve(n, d, dff, esz=2, L=1):
    return lib.sats_reserve(I(n), I(d), I(dff), I(L), ctypes.c_int(esz), P(0))

def options(batch_path=0, single_token=0, dec_block_cols=0, lora_per_token=0):
    o = (ctypes.c_int * 4)(batch_path, single_token, dec_block_cols, lora_per_token)
    return lib.sats_set_options(ctypes.byref(o))
"""


def build_fake(folder):
    so = os.path.join(str(folder), "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, FAKE], check=True)
    return so


def run(fake_so, body, lib=None):
    """Run `body` after PRELUDE in a fresh process; what it prints as JSON on its last line."""
    import json
    lib = lib or os.environ.get("SATS_LIB") or os.path.join(ROOT, "paper_2607_08991_amd", "libsats.so")
    r = subprocess.run([sys.executable, "-c", PRELUDE + body, fake_so, lib], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return json.loads(r.stdout.strip().splitlines()[-1])
