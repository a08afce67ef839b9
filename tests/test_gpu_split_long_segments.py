"""Vector-kernel products of long segments and large batches, whose wave
regions leave few waves: their row blocks are split over as many blocks as
shorten the product, also past one block per compute unit. Bar as for the other
split products: the float32 rounding of a sum of cols products, taken in any
order, of the oracle's value."""
import ctypes

import numpy as np
import pytest

from gen import random_bf16, random_x
from oracle import gemv as ogemv

hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


# (rows, cols, segment length, group rows): few row blocks and 2 waves a block;
# a ragged last group; between half and one row block per compute unit; more
# row blocks than compute units; 5 waves for 5 column blocks
SHAPES = [(500, 3072, 512, 64), (61, 2048, 256, 32), (2077, 10240, 256, 16), (300 * 64 - 5, 2048, 512, 64),
          (1000, 1000, 200, 64)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,S,GR", SHAPES)
@pytest.mark.parametrize("xdt", ["bf16", "f32"])
def test_parts_of_long_segments(torch, rows, cols, S, GR, xdt):
    w = random_bf16((rows, cols), seed=rows + cols)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=S, grp_rows=GR))
    sample = sorted({0, 1, rows // 2, rows - 65 if rows > 65 else 0, rows - 1})
    for batch in (16, 1, 5):
        print(f"long segments {rows}x{cols} S={S} GR={GR} x={xdt} batch={batch}", flush=True)
        x = random_x(batch, cols, seed=batch, dtype=xdt)
        xd = (torch.from_numpy(x.view(np.int16)).view(torch.bfloat16) if xdt == "bf16" else torch.from_numpy(x)).cuda()
        y = dt.gemv(xd, torch.full((batch, rows), float("nan"), device="cuda"))
        wd = torch.from_numpy(w.view(np.int16)).view(torch.bfloat16).cuda().double()
        ref, den = xd.double() @ wd.t(), xd.double().abs() @ wd.abs().t()
        assert float(((y.double() - ref).abs() / den).max()) <= cols * 2.0 ** -24
        y_ref, den = ogemv.gemv_rows(w, x, rows=sample)
        assert np.max(ogemv.rel_err(y.cpu().numpy()[:, sample], y_ref, den)) <= cols * 2.0 ** -24
        na = torch.full_like(y, float("nan"))
        assert torch.equal(dt.gemv_noalloc(xd, na), y) and torch.equal(dt.gemv(xd), y)
        small = torch.zeros(4, dtype=torch.uint8, device="cuda")  # no room for parts: one block per row block
        whole = dt.gemv(xd, workspace=small)
        assert float(((whole - y).double().abs() / (xd.double().abs() @ wd.abs().t())).max()) <= 2 * cols * 2.0 ** -24


def test_split_where_waves_are_few():
    # (no GPU: the size query) partial sums of at least `parts` parts are asked
    # for, and never more than the allocation-free product has
    import torch
    for rows, cols, S, GR, batch, parts in ((500, 3072, 512, 64, 1, 3), (500, 3072, 512, 64, 16, 6),
                                            (2500, 10240, 256, 16, 1, 3), (16, 131072 - 1024, 256, 16, 16, 2)):
        blob = torch.from_numpy(hl.encode(random_bf16((rows, cols), seed=1), seg_len=S, grp_rows=GR))
        buf = torch.zeros(blob.numel() + hl.LUT_BYTES + 32, dtype=torch.uint8)
        buf = buf[-buf.data_ptr() % 16:]
        buf[:blob.numel()] = blob
        view, lut = hl.TensorView(), buf.data_ptr() + (blob.numel() + 15) // 16 * 16
        assert hl.lib().hl_tensor_view(buf.data_ptr(), buf.data_ptr(), blob.numel(), lut, ctypes.byref(view)) == 0
        need = int(hl.lib().hl_gemv_workspace_bytes(ctypes.byref(view), batch))
        assert need >= parts * batch * rows * 4, (rows, cols, S, GR, batch, need)
