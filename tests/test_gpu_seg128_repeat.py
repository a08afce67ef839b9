"""Products on segments of 128 weights whose code pairs fit the bounded table:
the same call many times over, on matrices that fill the GPU with blocks, every
output within the float32 rounding of a sum of cols products of the float64
value and the same bits each time."""
import numpy as np
import pytest

from gen import random_bf16, random_x

pytestmark = pytest.mark.gpu
hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


@pytest.mark.parametrize("rows,cols", [(1000, 4096), (4096, 4096), (8200, 2048)])
@pytest.mark.parametrize("batch", [1, 16])
def test_repeated_products(torch, rows, cols, batch):
    print(f"S=128 {rows}x{cols} batch {batch}", flush=True)
    w = random_bf16((rows, cols), seed=rows)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=128, grp_rows=16))
    x = torch.from_numpy(random_x(batch, cols, seed=batch, dtype="bf16").view(np.int16)).view(torch.bfloat16).cuda()
    wd = torch.from_numpy(w.view(np.int16)).view(torch.bfloat16).cuda().double()
    ref, den = x.double() @ wd.t(), x.double().abs() @ wd.abs().t()
    ys = [dt.gemv(x) for _ in range(40)]
    wrong = [k for k, y in enumerate(ys) if not float(((y.double() - ref).abs() / den).max()) <= cols * 2.0 ** -24]
    assert not wrong, wrong
    assert all(torch.equal(y, ys[0]) for y in ys)
