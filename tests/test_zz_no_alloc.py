"""GPU check of als_gramian_static, the entry point for callers that cannot allocate device memory.

It is called through the C ABI twice in a row, the second time on a smaller table (the static
workspace keeps the first call's partial sums), and compared with als_gramian on the same tables.
Both run the same kernels in the same order, so the results agree bit for bit; the oracle bounds
both (1e-5 of the largest entry, as for als_gramian).  Tables beyond the stated maximum are refused.
"""
import gc

import numpy as np
import pytest
import torch

import oracle
from gpu_util import f64, say
from paper_2112_02194_amd import binding as als
from synth import init_table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype", [(128, torch.float32), (64, torch.bfloat16), (16, torch.float32)])
def test_static_gramian_two_calls_in_a_row(gpu_device, d, dtype):
    say(f"als_gramian_static d={d} {dtype}: 200001 rows, then 4099 rows")
    torch.cuda.set_device(0)
    ctx = als.Context(0)
    big = (init_table(200001, d, seed=9, stream=41) * 10.0 + 0.01 * torch.arange(d)[None, :]).to(dtype).to(gpu_device)
    small = big[1234:1234 + 4099].clone()
    out = torch.full((d, d), 7.0, dtype=torch.float32, device=gpu_device)
    got = torch.empty_like(out)
    gc.collect()
    torch.cuda.synchronize()
    for V in (big, small):
        free_before = torch.cuda.mem_get_info()[0]  # what the driver has left: falls with every hipMalloc
        als.als_gramian_static(V, out)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free_before
        got.copy_(out)
        want = als.als_gramian(ctx, V)
        torch.cuda.synchronize()
        assert torch.equal(got, want)
        ref = oracle.gramian_matmul(f64(V))
        assert np.abs(f64(got) - ref).max() <= 1e-5 * np.abs(ref).max()
    ctx.close()


def test_static_gramian_refuses_what_does_not_fit(gpu_device):
    say("als_gramian_static: too many rows, wrong device")
    torch.cuda.set_device(0)
    lib = als.load_library()
    V = torch.zeros(262144 + 1, 16, device=gpu_device)
    out = torch.full((16, 16), 3.0, device=gpu_device)
    with pytest.raises(als.AlsError) as e:
        als.als_gramian_static(V, out)
    assert e.value.status == als.ALS_ESHAPE and "262144" in str(e.value)
    tv = als._table(V[:100])
    import ctypes
    assert lib.als_gramian_static(5000, ctypes.byref(tv), out.data_ptr(), None) == als.ALS_EHIP
    torch.cuda.synchronize()
    assert torch.all(out == 3.0)
    als.als_gramian_static(V[:262144], out)  # the largest table that fits
    torch.cuda.synchronize()
    assert torch.all(out == 0.0)


@pytest.mark.parametrize("d,dtype", [(16, torch.float32), (32, torch.bfloat16), (64, torch.float32), (128, torch.bfloat16), (128, torch.float32)])
@pytest.mark.parametrize("rows", [129, 2113, 8192, 200001, 262144])
def test_static_gramian_has_the_bits_of_als_gramian_where_the_order_shows(gpu_device, d, dtype, rows):
    """One to 128 partial sums.  A few rows, spread over the table, are 2^40 times the others and come in pairs that cancel in
    the products of an even and an odd column: what is left of such an entry depends on which partials were added first, in its
    leading digits, fp64 or not."""
    say(f"als_gramian_static bits d={d} {dtype} rows={rows}")
    torch.cuda.set_device(0)
    gen = torch.Generator().manual_seed(rows + d)
    V = torch.randint(-8, 9, (rows, d), generator=gen).float()
    big = torch.randperm(rows, generator=gen)[:64]
    V[big] = 2.0 ** 40
    V[big[::2], 1::2] = -2.0 ** 40
    V = V.to(dtype).to(gpu_device)
    ctx = als.Context(0)
    out = torch.empty((d, d), device=gpu_device)
    als.als_gramian_static(V, out)
    want = als.als_gramian(ctx, V)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    ctx.close()
