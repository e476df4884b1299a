import collections
import ctypes
import functools
import json
import math
import os
import re
import shutil
import subprocess
import sys
import tempfile

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

GOLDEN = os.path.join(ROOT, "tests", "golden")


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs an MI355X (gfx950) GPU and the built HIP library")
    config.addinivalue_line("markers", "slow: full-size parity case (minutes of oracle time)")


@functools.lru_cache(maxsize=None)
def device_asm(source):
    """Lines of the gfx950 assembly of csrc/<source>, compiled once per run with
    the build's flags (needs no GPU); skips where hipcc is missing."""
    from paper_2606_10415_amd import build
    if not os.path.exists(build.HIPCC):
        pytest.skip("hipcc not available")
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "device.s")
        subprocess.run([build.HIPCC, *build.COMMON_FLAGS, "--cuda-device-only", "-S", "-x", "hip",
                        os.path.join(build.CSRC, source), "-o", out], check=True, capture_output=True)
        with open(out) as f:
            return f.read().split("\n")


@functools.lru_cache(maxsize=None)
def _plan_library():
    """The host-side plans (plan_query.cpp, plan.cpp), compiled once per run; skips where g++ is missing."""
    if shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("needs g++ and the HIP headers")
    with tempfile.TemporaryDirectory() as d:
        out = os.path.join(d, "plan_query.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                        "-I/opt/rocm/include", f"-I{ROOT}/include", os.path.join(ROOT, "tests", "plan_query.cpp"),
                        os.path.join(ROOT, "paper_2606_10415_amd", "csrc", "plan.cpp"), "-o", out], check=True)
        return ctypes.CDLL(out)


GemmPlan = collections.namedtuple("GemmPlan", "columns split_at head tail splits")


def gemm_plan(transA, transB, M, N, K, epi=0, reads_r=False, ws=False):
    """How a GEMM call with tight operands (leading dimensions rounded up to 8)
    is launched: `head` tiles up to column (columns) or row split_at, `tail`
    tiles behind it, the tail's K split `splits` ways.  N in output columns
    (gate columns for epi 1)."""
    out = (ctypes.c_int64 * 7)()
    up8 = lambda n: -(-n // 8) * 8
    lda, ldb = up8(M if transA else K), up8(K if transB else N)
    _plan_library().query_gemm_plan(int(transA), *(ctypes.c_int64(n) for n in (M, N, K)), epi, int(reads_r), int(ws),
                                    int((lda | ldb) & 63 != 0), out)
    return GemmPlan(bool(out[0]), out[1], (out[2], out[3]), (out[4], out[5]), out[6])


def attn_shares(B, S, Hq, Hkv, D, causal):
    """(key tile width, shares per key tile) of the attention backward's dK/dV pass."""
    n, tiles = (ctypes.c_int * 512)(), ctypes.c_int()
    ktile = _plan_library().query_attn_shares(B, S, Hq, Hkv, D, int(causal), n, ctypes.byref(tiles))
    return ktile, list(n[:tiles.value])


def load_golden(name):
    with open(os.path.join(GOLDEN, name)) as f:
        return json.load(f)


_LN = re.compile(r"ln(\d+)")


def golden_value(expr):
    """Evaluate a fixture expression such as '-2/9*ln2 - 30/169*ln3', '2**0.5/5'
    or '3*cos(1) + sin(1)' in float64."""
    names = {f"ln{n}": math.log(int(n)) for n in _LN.findall(expr)}
    names.update({"cos": math.cos, "sin": math.sin})
    if not re.fullmatch(r"([0-9+\-*/(). ]|ln\d+|cos|sin)*", expr):
        raise ValueError(f"unexpected token in fixture expression {expr!r}")
    return float(eval(expr, {"__builtins__": {}}, names))  # fixture-local arithmetic only


def rel_f(x, ref):
    """Relative Frobenius error ||x - ref|| / ||ref|| in float64."""
    x = np.asarray(x, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    den = np.linalg.norm(ref)
    return float(np.linalg.norm(x - ref) / (den if den > 0 else 1.0))


def row_err(x, ref):
    """Largest row error norm relative to the RMS row norm of ``ref``.

    x, ref: [rows, features].  max_i ||x_i - ref_i|| / sqrt(mean_i ||ref_i||^2):
    a per-row bound that a single wrong row cannot dilute, and that stays
    meaningful for rows whose reference is exactly zero."""
    x = np.asarray(x, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    rms = math.sqrt(float(np.mean(np.sum(ref * ref, axis=1))))
    worst = float(np.max(np.linalg.norm(x - ref, axis=1)))
    return worst / (rms if rms > 0 else 1.0)
