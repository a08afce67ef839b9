"""The workspace that a DeviceTensor keeps (no GPU: a view of a container in
host memory, which the size query does not read): whatever batch it was first
asked for, it holds what a later product of any allowed batch asks."""
import ctypes

import pytest

from gen import random_bf16

hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


def _tensor(rows, cols):
    import torch
    blob = torch.from_numpy(hl.encode(random_bf16((rows, cols), seed=1), seg_len=64, grp_rows=16))
    host = torch.zeros(blob.numel() + 16, dtype=torch.uint8)
    host = host[-host.data_ptr() % 16:][:blob.numel()].copy_(blob)
    dt = hl.DeviceTensor.__new__(hl.DeviceTensor)
    dt.blob, dt.lut, dt.view = host, torch.zeros(hl.LUT_BYTES // 4 + 4, dtype=torch.int32), hl.TensorView()
    lut = dt.lut.data_ptr() + -dt.lut.data_ptr() % 16
    assert hl.lib().hl_tensor_view(host.data_ptr(), host.data_ptr(), host.numel(), lut, ctypes.byref(dt.view)) == 0
    return dt


@pytest.mark.parametrize("first", [[], [1], [0], [17], [1 << 20], [3, 17, 1]])
def test_first_batch_asked_does_not_matter(first):
    dt = _tensor(100, 4096)  # split: partial sums in proportion to the batch
    for batch in first:
        dt.workspace(batch)
    for batch in (1, 3, hl.MAX_BATCH):
        need = int(hl.lib().hl_gemv_workspace_bytes(ctypes.byref(dt.view), batch))
        assert need > 0 and dt.workspace(batch).numel() >= need
    ws = dt.workspace()
    assert not ws.any() and dt.workspace(1) is ws and dt.workspace(hl.MAX_BATCH) is ws
