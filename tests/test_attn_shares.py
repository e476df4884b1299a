"""Shares of the key tiles' work in the attention backward's dK/dV pass.

CPU: for random shapes the shares cover every tile, no workgroup is empty, and
the partial rows fit the workspace that lt_attn_bwd_workspace_size asks for.
GPU: shapes whose tiles get unequal shares (several, one written directly, a
ragged last tile, one tile only; 256- and 128-key tiles) against a float64
reference, recomputed and saved P; the shares of each are asserted; bars as for the other backward tests (FP16 results of FP32 sums over
FP16 P and dS: 1e-2 of the gradient's norm).
"""

import math
import os
import shutil
import subprocess

import pytest

from conftest import attn_shares, rel_f

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"

PROGRAM = r"""
#include "@/csrc/kernels.hpp"
#include <cstdio>
#include <random>
using namespace lt;
int main() {
  std::mt19937 r(3);
  long bad = 0, split = 0, uneven = 0, single = 0, none = 0;
  for (int it = 0; it < 200000; ++it) {
    const int B = 1 + r() % 4, Hkv = 1 << (r() % 6), grp = 1 + r() % 8, D = r() % 2 ? 64 : 128;
    const int S = 1 + r() % (1u << (4 + r() % 10)), causal = r() % 2, Hq = Hkv * grp;
    const DkdvPlan p = attn_bwd_dkdv_plan(B, S, Hq, Hkv);
    DkdvShares s;
    if (!attn_bwd_shares(B, S, Hq, Hkv, D, causal, p, &s)) { ++none; continue; }
    ++split;
    const int n_kt = (S - 1) / p.ktile + 1, rows = p.ktile < S ? p.ktile : S;
    bool ok = p.nsplit > 1 && s.off[0] == 0 && s.off[n_kt] == s.m;
    int lo = 1 << 30, hi = 0;
    for (int j = 0; j < n_kt; ++j) {
      const int n = s.off[j + 1] - s.off[j];
      const int work = grp * ((S - 1) / 64 + 1 - (causal ? j * (p.ktile / 64) : 0));
      ok = ok && n >= 1 && n <= work;
      lo = n < lo ? n : lo;
      hi = n > hi ? n : hi;
    }
    uneven += lo != hi;
    single += lo == 1;
    const size_t need = (size_t)2 * B * Hkv * s.m * rows * D * sizeof(float);
    ok = ok && need <= attn_bwd_part_bytes(B, S, Hq, Hkv, D);
    bad += !ok;
  }
  std::printf("%ld split, %ld uneven, %ld with a tile of one share, %ld not split, %ld bad\n", split, uneven, single,
              none, bad);
  return bad || !split || !uneven || !single || !none;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(f"{ROCM}/include/hip"),
                    reason="needs g++ and the HIP headers")
def test_shares_cover_the_tiles_within_the_workspace(tmp_path):
    src, exe = tmp_path / "shares.cpp", tmp_path / "shares"
    src.write_text(PROGRAM.replace("@", f"{ROOT}/paper_2606_10415_amd"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include", str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]


# key tile width and shares per key tile of each GPU case
PLANNED = {
    (1, 1300, 10, 2, 128, True): (256, [7, 6, 5, 3, 2, 1]),
    (1, 700, 4, 4, 64, True): (128, [1] * 6),
    (2, 200, 8, 1, 64, True): (256, [16]),
    (1, 1024, 8, 2, 128, False): (256, [16] * 4),
    (4, 333, 16, 16, 64, False): (128, [1] * 3),
    (1, 1500, 4, 4, 128, True): (128, [3, 3, 3, 2, 2, 2, 2, 2, 1, 1, 1, 1]),
    (1, 1500, 4, 4, 64, True): (128, [3, 3, 3, 2, 2, 2, 2, 2, 1, 1, 1, 1]),
    (6, 884, 1, 1, 128, True): (128, [3, 2, 2, 2, 1, 1, 1]),
    (3, 2304, 1, 1, 64, False): (128, [2] * 18),
}


def test_planned_shares():
    for case, plan in PLANNED.items():
        assert attn_shares(*case) == plan, case


@pytest.mark.parametrize("B,S,Hq,Hkv,D,shares", [
    # a few percent of estimated gain is no reason to leave equal shares (of a
    # ragged last tile's own number): backward and forward in proportion 124
    # and 392 us, equal 115 and 374
    (1, 1636, 16, 16, 128, [2] * 12 + [1]),
    (1, 2975, 32, 8, 128, [4] * 11 + [2]),
    # 20%: 122 us equal, 107 in proportion
    (1, 2048, 40, 8, 128, [7, 6, 5, 4, 4, 3, 2, 1]),
])
def test_equal_shares_stay_unless_clearly_slower(B, S, Hq, Hkv, D, shares):
    assert attn_shares(B, S, Hq, Hkv, D, True)[1] == shares


@pytest.mark.gpu
@pytest.mark.parametrize("saved", [False, True], ids=["recomputed", "saved-P"])
@pytest.mark.parametrize("B,S,Hq,Hkv,D,causal", [
    (1, 1300, 10, 2, 128, True),     # 256-key tiles, ragged last tile, many shares for the first
    (1, 700, 4, 4, 64, True),        # 128-key tiles, not split
    (2, 200, 8, 1, 64, True),        # one tile only
    (1, 1024, 8, 2, 128, False),     # equal work, no mask
    (4, 333, 16, 16, 64, False),     # one workgroup per tile although the workspace has room
    (1, 1500, 4, 4, 128, True),      # 128-key tiles (query halves per wave pair), shares, ragged last tile
    (1, 1500, 4, 4, 64, True),
    (6, 884, 1, 1, 128, True),       # ... several batches
    (3, 2304, 1, 1, 64, False),      # ... no mask
])
def test_uneven_shares_against_float64(B, S, Hq, Hkv, D, causal, saved):
    import torch
    from paper_2606_10415_amd import lt

    assert attn_shares(B, S, Hq, Hkv, D, causal) == PLANNED[B, S, Hq, Hkv, D, causal]
    print(f"shares B={B} S={S} Hq={Hq} Hkv={Hkv} D={D} causal={causal} saved={saved}", flush=True)
    T, row, hd, scale, ca = B * S, (Hq + 2 * Hkv) * D, Hq * D, 1 / math.sqrt(D), int(causal)
    g = torch.Generator().manual_seed(5)
    qkv, do = torch.randn(T, row, generator=g).half().cuda(), torch.randn(T, hd, generator=g).half().cuda()
    O, LSE = torch.empty(T, hd, dtype=torch.float16, device="cuda"), torch.empty(B, Hq, S, device="cuda")
    dqkv = torch.full((T, row), float("nan"), dtype=torch.float16, device="cuda")

    def heads(t):
        p = t.data_ptr()
        return p, p + 2 * hd, p + 2 * (hd + Hkv * D)

    (q, k, v), (dq, dk, dv) = heads(qkv), heads(dqkv)
    if saved:
        n_p, n = lt.lt_attn_p_size(B, S, Hq, ca), lt.lt_attn_bwd_p_workspace_size(B, S, Hq, Hkv, D)
        P, ws = (torch.empty(x, dtype=torch.uint8, device="cuda") for x in (n_p, n))
        lt.lt_attn_fwd_p(q, k, v, row, row, O, hd, LSE, P, n_p, B, S, Hq, Hkv, D, scale, ca)
        lt.lt_attn_bwd_p(q, k, v, row, row, O, do, hd, LSE, P, n_p, dq, dk, dv, row, row, ws, n, B, S, Hq, Hkv, D,
                         scale, ca)
    else:
        n = lt.lt_attn_bwd_workspace_size(B, S, Hq, Hkv, D, ca)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        lt.lt_attn_fwd(q, k, v, row, row, O, hd, LSE, B, S, Hq, Hkv, D, scale, ca)
        lt.lt_attn_bwd(q, k, v, row, row, O, do, hd, LSE, dq, dk, dv, row, row, ws, n, B, S, Hq, Hkv, D, scale, ca)
    got = dqkv.cpu().double().view(B, S, -1, D)
    x, dob = qkv.cpu().double().view(B, S, -1, D), do.cpu().double().view(B, S, Hq, D)
    ref = torch.zeros_like(x)
    drop = torch.ones(S, S, dtype=torch.bool).triu(1)
    for b in range(B):
        for h in range(Hq):
            kv = Hq + h // (Hq // Hkv)
            qh, kh, vh, gh = x[b, :, h], x[b, :, kv], x[b, :, kv + Hkv], dob[b, :, h]
            s = qh @ kh.t() * scale
            p = torch.softmax(s.masked_fill(drop, -math.inf) if causal else s, 1)
            dp = gh @ vh.t()
            ds = p * (dp - (p * dp).sum(1, keepdim=True)) * scale
            ref[b, :, h] = ds @ kh
            ref[b, :, kv] += ds.t() @ qh
            ref[b, :, kv + Hkv] += p.t() @ gh
    for b in range(B):
        for i in range(Hq + 2 * Hkv):
            assert rel_f(got[b, :, i].numpy(), ref[b, :, i].numpy()) <= 1e-2, (b, i)
