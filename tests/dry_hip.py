"""Runs the built library's host code without a GPU: a child interpreter with a
HIP runtime that only keeps a log (dry_hip.cpp) preloaded."""
from __future__ import annotations

import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes, json, re, sys
sys.path.insert(0, {root!r})
import numpy as np
dry = ctypes.CDLL({lib!r})
dry.dry_log.restype = ctypes.c_char_p
dry.dry_fail.argtypes = [ctypes.c_char_p]
from paper_2404_16208_amd import ranc as R
from paper_2404_16208_amd import workloads as W
from tests.test_gpu_feedforward import forward_net

def log():
    "(what, stream, kernel or event, ...) of everything queued since the last call"
    rows = [l.split() for l in dry.dry_log().decode().splitlines()]
    dry.dry_clear()
    short = lambda k: re.sub(r"^_ZN4ranc[0-9]+([a-z_0-9]*?)(IL|E).*$", r"\1", k)
    return [[r[0], int(r[1])] + [short(x) for x in r[2:]] for r in rows]

def kernels(rows=None):
    return [r[2] for r in (log() if rows is None else rows) if r[0] == "launch"]

held = []
def load(net, S, T, path, size=None):
    "a handle on a workspace in host memory (of `size` bytes, by default as many as asked for)"
    d = R.Desc(net)
    n = size or R.ranc_workspace_bytes(d, S, T, R.PATHS[path])
    ws = np.zeros(n + 256, np.uint8)
    held.append((d, ws))
    h = R.ranc_load_network(d, S, T, R.PATHS[path], -(-ws.ctypes.data // 256) * 256, n, 0)
    log()
    return h

def need(net, S, T, path):
    return R.ranc_workspace_bytes(R.Desc(net), S, T, R.PATHS[path])

def run(handles, T, flags=0, stream=0):
    R.ranc_run_ticks(handles if isinstance(handles, list) else [handles], None, flags, T, stream)
    return log()

{body}
print("DRY" + json.dumps(result))
"""


def build(tmp_path) -> str:
    out = os.path.join(str(tmp_path), "libdry_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", out, os.path.join(ROOT, "tests", "dry_hip.cpp")],
                   check=True)
    return out


def run(lib: str, body: str):
    """`result` as the child's code `body` leaves it."""
    env = dict(os.environ, LD_PRELOAD=lib)
    r = subprocess.run([sys.executable, "-c", CHILD.format(root=ROOT, lib=lib, body=body)], env=env, cwd=ROOT,
                       capture_output=True, text=True, timeout=300)
    lines = [l for l in r.stdout.splitlines() if l.startswith("DRY")]
    assert r.returncode == 0 and lines, f"{r.stdout[-2000:]}\n{r.stderr[-4000:]}"
    return json.loads(lines[-1][3:])
