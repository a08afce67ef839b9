"""Float16 products of matrices of 8 column blocks and two groups or more for
each wave of 8 a compute unit: on the non-persistent kernel where two of its
blocks fit a compute unit, on the persistent one where longer segments leave
room for one. Products within the float32 rounding of a sum of cols products of
the float64 value, decode bit-exact."""
import numpy as np
import pytest

from gen import random_fp16, random_x

pytestmark = pytest.mark.gpu
hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


# rare exponents in one segment: none, few (longer than two blocks have room
# for), many (longer than the persistent kernel takes); two row blocks a unit,
# one more and ragged
@pytest.mark.parametrize("rare,bits", [(0, (600, 834)), (40, (834, 898)), (64, (950, 1500))])
@pytest.mark.parametrize("rows", [8192, 8201])
def test_products(torch, rare, bits, rows):
    cols = 2048
    w = random_fp16((rows, cols), seed=rows + rare)
    w[rows // 2, 64:64 + rare] = (w[rows // 2, 64:64 + rare] & 0x83FF) | (1 << 10)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=64, grp_rows=16, fp16=True))
    print(f"fp16 {rows}x{cols}: longest segment {dt.view.max_seg_bits}", flush=True)
    assert bits[0] <= dt.view.max_seg_bits < bits[1], dt.view.max_seg_bits
    assert np.array_equal(dt.decode().cpu().numpy().view(np.uint16), w)
    wd = torch.from_numpy(w.view(np.int16)).view(torch.float16).cuda().double()
    for batch in (1, 3, 16):
        x = torch.from_numpy(random_x(batch, cols, seed=batch, dtype="f16").view(np.int16)).view(torch.float16).cuda()
        y = dt.gemv(x, torch.full((batch, rows), float("nan"), device="cuda"))
        ref, den = x.double() @ wd.t(), x.double().abs() @ wd.abs().t()
        assert float(((y.double() - ref).abs() / den).max()) <= cols * 2.0 ** -24
        assert torch.equal(dt.gemv_noalloc(x, torch.full_like(y, float("nan"))), y)
