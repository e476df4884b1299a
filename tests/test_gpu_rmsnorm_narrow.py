"""RMSNorm backward of narrow rows: the row groups of one and two waves.

Rows up to 512 (1024) columns are taken by one (two) of a workgroup's four
waves, side by side; sizes at the edges of those ranges, and row counts that
leave some groups without a row, against the float64 oracle (bar: 5e-3 of the
gradient's norm, as for the wider rows)."""

import numpy as np
import pytest

import oracle
from conftest import rel_f
from paper_2606_10415_amd.synth import normal_f16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 5, 3001])
@pytest.mark.parametrize("H", [8, 512, 520, 1024, 1032, 2048, 2056])
def test_narrow_rows(T, H):
    import torch
    from paper_2606_10415_amd import lt

    print(f"rmsnorm narrow T={T} H={H}", flush=True)
    x, dy, r = (normal_f16(71 + i, (T, H)) for i in range(3))
    w = (1 + normal_f16(75, (H,), 0.1).astype(np.float32)).astype(np.float16)
    X, dY, R, W = (torch.from_numpy(a).cuda() for a in (x, dy, r, w))
    Y, dW = torch.empty_like(X), torch.empty_like(W)
    dX = torch.full((T + 1, H), 777.0, dtype=torch.float16, device="cuda")      # a guard row
    rstd = torch.empty(T, dtype=torch.float32, device="cuda")
    n = lt.lt_rmsnorm_bwd_workspace_size(T, H)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    lt.lt_rmsnorm_fwd(X, H, W, Y, H, rstd, T, H, 1e-5)
    lt.lt_rmsnorm_bwd(dY, H, X, H, W, rstd, R, H, dX, H, dW, ws, n, T, H)
    dx_ref, dw_ref = oracle.rmsnorm_bwd(dy, x, w, 1e-5)
    got = dX.cpu().numpy()
    assert rel_f(got[:T], dx_ref + r.astype(np.float64)) <= 5e-3
    assert (got[T] == 777.0).all()
    assert rel_f(dW.cpu().numpy(), dw_ref) <= 5e-3
