"""Launch plans of the GEMM: which tiles a call runs as (host code), and the tiles on the GPU.

CPU: a plan's cut lies on a tile edge inside the output, for random sizes,
epilogues and layouts; split-K plans only where the workspace rule has one.
GPU: every tile in every layout and epilogue, by itself and behind whole rounds
of 256x256 tiles, at ragged sizes.  The plan of each is asserted, so that another
cost model cannot drop one silently.  Integer operands, whose FP32 sums are
exact, so the plain results equal the float64 product bit for bit; the SwiGLU
epilogues meet the bars of their parity test.
"""

import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
import test_gpu_swiglu_layer as fused
from conftest import gemm_plan
from paper_2606_10415_amd.synth import uniform_int_f16

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = "/opt/rocm"

PROGRAM = r"""
#include "../paper_2606_10415_amd/csrc/kernels.hpp"
#include <cstdio>
#include <random>
using namespace lt;
int main() {
  std::mt19937_64 r(1);
  long bad = 0, n = 0, kinds[kNumGemmTiles] = {}, split = 0, two = 0;
  auto size = [&](int hi) { return (int64_t)1 << (r() % hi); };
  for (int it = 0; it < 200000; ++it) {
    const int64_t M = 1 + r() % (size(15)), N = 1 + r() % (size(16)), K = 1 + r() % (size(15));
    const int tA = r() % 2, epi = tA ? 0 : (int)(r() % 3);
    const bool ws = r() % 2, rd = epi == 0 && r() % 2;
    const GemmPlan p = gemm_plan(tA, M, N, K, epi, rd, ws);
    ++n;
    bool ok = p.tail >= 0 && p.tail < kNumGemmTiles && p.split_at >= 0 && p.splits >= 1;
    const int64_t unit = p.columns ? (epi == 1 ? 128 : 256) : 256;
    if (p.split_at) ok = ok && p.head == kTile256 && p.split_at % unit == 0 && p.split_at < (p.columns ? N : M);
    SplitTail st;
    if (p.splits > 1)
      ok = ok && ws && epi == 0 && p.tail == kTile256 && gemm_splitk_tail(M, N, K, &st) && st.S == p.splits &&
           st.split_at == p.split_at && (!p.split_at || st.columns == p.columns);
    bad += !ok;
    ++kinds[p.tail];
    split += p.splits > 1;
    two += p.split_at > 0;
  }
  // the largest sizes the entry points accept
  for (int tA = 0; tA < 2; ++tA) {
    const GemmPlan p = gemm_plan(tA, (int64_t)1 << 30, (int64_t)1 << 30, (int64_t)1 << 30, 0, true, true);
    bad += p.tail != kTile256 || p.splits != 1;
  }
  bool all = split && two;
  for (int t = 0; t < kNumGemmTiles; ++t) all = all && kinds[t] > 0;
  std::printf("%ld plans, %ld bad, every kind %d\n", n, bad, (int)all);
  return bad || !all;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(f"{ROCM}/include/hip"),
                    reason="needs g++ and the HIP headers")
def test_plans_cover_the_output(tmp_path):
    src, exe = tmp_path / "plan_check.cpp", tmp_path / "plan_check"
    src.write_text(PROGRAM.replace("../paper_2606_10415_amd", f"{ROOT}/paper_2606_10415_amd"))
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                    "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include", f"-I{ROOT}/include", str(src),
                    os.path.join(ROOT, "paper_2606_10415_amd", "csrc", "plan.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", [(0, 1), (0, 0), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,ws", [
    (65, 72, 64, False),        # 64x64 tiles, one slice in the eight-stage ring
    (200, 328, 584, False),     # 64x64, more slices than stages, last slice 8 wide
    (1000, 4096, 328, False),   # 128x128
    (1237, 5120, 456, False),   # 256x128, one launch, ragged rows
    (2048, 4096, 1224, False),  # 256x128, one round
    (1237, 7168, 200, True),    # 256x256, workspace given, not taken
    (1104, 4120, 1237, False),  # K odd: 128x256 with whole k-rows for weight gradients, fix-up elsewhere
])
def test_plan_tiles_exact_integers(transA, transB, M, N, K, ws):
    run_exact(transA, transB, M, N, K, ws)


def run_exact(transA, transB, M, N, K, ws):
    import torch
    from paper_2606_10415_amd import lt

    print(f"gemm plan trans=({transA},{transB}) M={M} N={N} K={K} ws={ws}", flush=True)
    a, b = uniform_int_f16(41, (M, K), -2, 2), uniform_int_f16(42, (K, N), -2, 2)
    r = uniform_int_f16(43, (M, N), -8, 8)

    def stored(x, trans):
        st = np.ascontiguousarray(x.T if trans else x)
        out = np.full((st.shape[0], -(-st.shape[1] // 8) * 8), np.nan, np.float16)   # padding is never used
        out[:, :st.shape[1]] = st
        return torch.from_numpy(out).cuda()

    A, B, R = stored(a, transA), stored(b, transB), stored(r, False)
    ldc = -(-N // 8) * 8
    C = torch.full((M + 1, ldc), 777.0, dtype=torch.float16, device="cuda")         # a guard row, guard columns
    if ws:
        need = max(lt.lt_gemm_f16_workspace_size(transA, transB, M, N, K), 16)
        w = torch.empty(need, dtype=torch.uint8, device="cuda")
        lt.lt_gemm_f16_ws(transA, transB, M, N, K, 3.0, A, A.shape[1], B, B.shape[1], -2.0, R, ldc, None, C, ldc, w,
                          need)
    else:
        lt.lt_gemm_f16_res(transA, transB, M, N, K, 3.0, A, A.shape[1], B, B.shape[1], -2.0, R, ldc, C, ldc)
    got = C.cpu().numpy()
    rows = np.unique(np.concatenate([np.random.default_rng(0).choice(M, min(M, 96), replace=False), [0, M - 1]]))
    ref = oracle.gemm(0, 0, 3.0, a[rows], b, -2.0, r[rows]).astype(np.float16)
    assert np.array_equal(np.ascontiguousarray(got[rows, :N]).view(np.uint16), ref.view(np.uint16))
    assert (got[M] == 777.0).all() and (got[:, N:] == 777.0).all()


ONE, COLUMNS, ROWS = "one launch", "columns", "rows"


def planned(p):
    return (ONE if p.split_at == 0 else COLUMNS if p.columns else ROWS), p.tail


# more slices than the tile has LDS stages, a last slice of 8 columns; ragged
# rows, columns and packed columns
@pytest.mark.gpu
@pytest.mark.parametrize("transA,transB", [(0, 1), (0, 0), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K,plan", [
    (61, 200, 1000, (ONE, (64, 64))),
    (3003, 328, 328, (ONE, (128, 128))),
    (777, 4675, 328, (ONE, (128, 256))),
    (901, 4131, 328, (ONE, (256, 128))),
    (2600, 3083, 200, (ONE, (256, 256))),
    (4000, 4088, 8, (ONE, (256, 256))),            # a single 8-wide slice
    (3848, 5107, 328, (COLUMNS, (128, 128))),
    (5107, 3848, 328, (ROWS, (128, 128))),
    (2040, 8691, 264, (COLUMNS, (64, 64))),
    (8691, 2040, 264, (ROWS, (64, 64))),
])
def test_every_tile_and_layout(transA, transB, M, N, K, plan):
    assert planned(gemm_plan(transA, transB, M, N, K, reads_r=True)) == plan
    run_exact(transA, transB, M, N, K, False)


@pytest.mark.gpu
@pytest.mark.parametrize("T,H,F,gate_up,swiglu_bwd", [
    (56, 1000, 200, (ONE, (64, 64)), (ONE, (64, 64))),
    (200, 328, 4120, (ONE, (128, 128)), (ONE, (128, 128))),
    (1544, 328, 4680, (ONE, (128, 256)), (ONE, (128, 256))),
    (3000, 328, 712, (ONE, (256, 128)), (ONE, (128, 128))),
    (2600, 200, 1544, (ONE, (256, 256)), (ONE, (256, 128))),
    (4088, 328, 2600, (COLUMNS, (256, 128)), (ONE, (256, 256))),
    (3000, 328, 4088, (ROWS, (256, 128)), (ONE, (256, 256))),
    (3848, 328, 5112, (COLUMNS, (128, 256)), (COLUMNS, (128, 128))),
    (5112, 328, 3848, (COLUMNS, (256, 128)), (ROWS, (128, 128))),
    (2600, 328, 3848, (ROWS, (128, 256)), (ONE, (256, 256))),
    (2600, 1000, 3080, (ROWS, (64, 64)), (ONE, (256, 256))),
])
def test_every_tile_of_the_swiglu_epilogues(T, H, F, gate_up, swiglu_bwd):
    import torch
    from paper_2606_10415_amd import lt

    assert planned(gemm_plan(0, 1, T, F, H, epi=1)) == gate_up
    assert planned(gemm_plan(0, 0, T, F, H, epi=2)) == swiglu_bwd
    fused.test_fused_gemm_swiglu_parity((torch, lt), T, H, F)


@pytest.mark.parametrize("transA,transB,M,N,K,splits", [
    # rows that lie across memory lines: whole-K 64x64 tiles take 88, 51, 30
    # and 61 us, split ones 54, 33, 24 and 44
    (0, 1, 128, 5160, 10616, 8), (1, 0, 120, 3272, 6504, 8), (0, 0, 152, 952, 5712, 8), (0, 1, 312, 1072, 8344, 8),
    # rows on memory lines: 20 us whole, 29 us split
    (0, 1, 480, 976, 5760, 1),
])
def test_split_of_skinny_products(transA, transB, M, N, K, splits):
    assert gemm_plan(transA, transB, M, N, K, ws=True).splits == splits
