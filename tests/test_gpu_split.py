"""Products of row blocks split over blocks (the non-persistent kernels): whole
up to 8 column blocks, then parts of about 4 that meet through the workspace,
eight parts at a time in the last sum. Bar: every output within the float32
rounding of a sum of cols products, taken in any order, of the oracle's
exactly rounded value (cols * 2**-24 of the sum of magnitudes)."""
import numpy as np
import pytest

from gen import random_bf16, random_fp16, random_x
from oracle import gemv as ogemv

pytestmark = pytest.mark.gpu
hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


# (rows, column blocks of 256): the largest whole row block, the smallest split
# (3 parts), a last part shorter than the others, exactly 8 parts, 9 and 10 (a
# second round of the last sum)
@pytest.mark.parametrize("rows,cb", [(37, 8), (53, 9), (16, 14), (20, 32), (7, 36), (40, 40)])
@pytest.mark.parametrize("xdt", ["bf16", "f32", "f16"])
def test_parts_of_a_row_block(torch, rows, cb, xdt):
    cols = 256 * cb
    f16 = xdt == "f16"
    w = (random_fp16 if f16 else random_bf16)((rows, cols), seed=rows + cb)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=64, grp_rows=16, fp16=f16))
    for batch in (1, 3, 16):
        print(f"parts {rows}x{cols} x={xdt} batch={batch}", flush=True)
        x = random_x(batch, cols, seed=batch + cb, dtype=xdt)
        y_ref, den = ogemv.gemv_rows(w, x, weights="fp16") if f16 else ogemv.gemv_rows(w, x)
        xd = torch.from_numpy(x.view(np.int16)).view(torch.bfloat16) if xdt == "bf16" else torch.from_numpy(x)
        xd = xd.cuda()
        y = dt.gemv(xd)
        first = y.cpu().numpy()
        assert np.max(ogemv.rel_err(first, y_ref, den)) <= cols * 2.0 ** -24
        # the arrival counters are back at zero and the parts added in order
        for _ in range(3):
            assert np.array_equal(dt.gemv(xd).cpu().numpy(), first)
