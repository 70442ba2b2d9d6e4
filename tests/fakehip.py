"""Runs a piece of Python against libspdp's host code with the stand-in HIP
runtime of ``fake_hip.cpp`` (no GPU: launches are recorded, not run)."""

import json
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes, json, os, re, sys
import numpy as np
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
hip.fake_log.restype = ctypes.c_char_p
for f in (hip.fake_used, hip.fake_live):
    f.restype = ctypes.c_size_t
hip.fake_budget.argtypes = hip.fake_fail_new.argtypes = [ctypes.c_size_t]
import paper_2607_21985_amd as spdp
L = spdp.lib()
X, Y = 1 << 40, 1 << 44  # addresses that nothing reads

def log():
    out = [tuple(l.split()) for l in hip.fake_log().decode().splitlines()]
    hip.fake_clear()
    return out

def launches(entries=None):
    # (kernel, grid) of each launch
    return [(re.sub(r"^_ZN12_GLOBAL__N_1[0-9]+", "", l[1]), tuple(int(v) for v in l[2:5]))
            for l in (log() if entries is None else entries) if l[0] == "launch"]

def ones(rows, cols, tile, keep=1.0, seed=0):
    rng = np.random.default_rng(seed)
    w = np.ones((rows, cols), np.float16)
    if keep < 1.0:
        w[rng.random((rows, cols)) >= keep] = 0
    return spdp.encode(w, tile)

def spmm(m, n):
    return L.spdp_spmm(m._h, X, n, Y, None)

def many(mats, tokens, mask=0, thresholds=None):
    k = len(mats)
    hs = (ctypes.c_void_p * k)(*[m._h for m in mats])
    xs = (ctypes.c_void_p * k)(*([X] * k))
    ys = (ctypes.c_void_p * k)(*[Y + (i << 32) for i in range(k)])
    ts = (ctypes.c_float * k)(*(thresholds or [0.5] * k))
    return L.spdp_spmspv_many_mask(hs, k, xs, tokens, ts, mask, ys, None)

out = {}
"""


@pytest.fixture(scope="session")
def fake_hip(tmp_path_factory):
    """The stand-in's path, built once."""
    gxx = shutil.which("g++") or shutil.which("c++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    path = str(tmp_path_factory.mktemp("fakehip") / "libamdhip64.so.7")
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", "-Wl,-soname,libamdhip64.so.7", "-o", path,
                    os.path.join(HERE, "fake_hip.cpp")], check=True)
    return path


def run(fake, body, env=None):
    """``body`` fills the dict ``out``; returns it."""
    code = PRELUDE + textwrap.dedent(body) + "\nprint('RESULT ' + json.dumps(out))\n"
    e = {k: v for k, v in os.environ.items() if not k.startswith("SPDP_")}
    e.update(env or {}, PYTHONPATH=ROOT)
    r = subprocess.run([sys.executable, "-c", code, fake], capture_output=True, text=True, env=e, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    line = [l for l in r.stdout.splitlines() if l.startswith("RESULT ")][-1]
    return json.loads(line[len("RESULT "):])
