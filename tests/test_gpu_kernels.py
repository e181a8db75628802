"""Single kernels at the sizes where their tiling can go wrong, against fp64 evaluations of the same quantity."""
import numpy as np
import pytest
import torch

from gpu_util import f64, rel_fro, say
from paper_2112_02194_amd import binding as als

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(gpu_device):
    c = als.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_shared_factor_against_the_closed_form_of_one_entry_rows(ctx, gpu_device, d):
    """1, 2, 4 and 8 blocks of 16 columns.  A row with the single entry v solves to B^-1 v / (1 + v^T B^-1 v)
    (Sherman-Morrison), so every column of the shared factor's inverse shows in the result.  Tolerance: L^-1 and
    Z = V L^-T are fp32 with rounding errors amplified by sqrt(cond(B)) each, 4 sqrt(d cond) 2^-24 together, and the
    1 x 1 system is formed from operands cut to 16 bits (4 * 2^-16)."""
    say(f"shared factor d={d}")
    gen = torch.Generator().manual_seed(d)
    n, alpha, lam = 203, 0.1, 1e-3
    H = torch.randn((n, d), generator=gen, dtype=torch.float64) * torch.logspace(0, -2, d, dtype=torch.float64)
    Hf = H.float()
    G = (Hf.double().T @ Hf.double()).float()
    B = alpha * G.double().numpy() + lam * np.eye(d)
    ev = np.linalg.eigvalsh(B)
    Y = als.Csr(n, n, torch.arange(n + 1, device=gpu_device), torch.arange(n, device=gpu_device, dtype=torch.int32))
    X = torch.empty((n, d), device=gpu_device)
    als.als_solve_rows(ctx, Y, Hf.to(gpu_device), G.to(gpu_device), als.make_params(alpha, lam), X)
    als.als_status_sync(ctx)
    BiV = np.linalg.solve(B, f64(Hf).T).T
    ref = BiV / (1.0 + np.sum(f64(Hf) * BiV, axis=1, keepdims=True))
    assert rel_fro(f64(X), ref) <= 4 * np.sqrt(d * ev[-1] / ev[0]) * 2.0 ** -24 + 4 * 2.0 ** -16


@pytest.mark.parametrize("d", [16, 128])
def test_a_gramian_that_is_not_positive_definite_is_reported(ctx, gpu_device, d):
    Y = als.Csr(4, 4, torch.arange(5, device=gpu_device), torch.arange(4, device=gpu_device, dtype=torch.int32))
    V = torch.ones((4, d), device=gpu_device)
    G = torch.eye(d, device=gpu_device)
    G[d - 1, d - 1] = -1.0  # the last pivot of the last block
    als.als_solve_rows(ctx, Y, V, G, als.make_params(0.1, 1e-3), torch.empty((4, d), device=gpu_device))
    with pytest.raises(als.AlsError) as e:
        als.als_status_sync(ctx)
    assert e.value.status == als.ALS_ENOTSPD
    als.als_status_sync(ctx)  # reported once
