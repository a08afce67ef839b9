"""Decode of matrices whose groups the persistent kernel's waves take in turn
(at least two groups for each of its 2048 waves on 256 CUs): few or many row
blocks, few column blocks, whole rounds and partial last ones, ragged last
row blocks. Bit-exact, and nothing written past the matrix."""
import numpy as np
import pytest

from gen import random_bf16, random_fp16

pytestmark = pytest.mark.gpu
hl = pytest.importorskip("paper_2502_00922_amd.hufflm")

ENCODE = {"split": {}, "whole": {"whole_exponent": True}, "fp16": {"fp16": True}}


# groups of 16 rows x 4 segments: 4096 (two whole rounds of 2048 waves), 4095
# (the other kernel), 4097 (one more), 4100 in one column block, 5000 in 100
# row blocks, 6399 and 6401 (a last round of about one wave a block), and
# 32-weight segments
@pytest.mark.parametrize("rows,cols,S", [(32 * 16, 128 * 256, 64), (273 * 16 - 3, 15 * 256, 64),
                                         (241 * 16 - 5, 17 * 256, 64), (4100 * 16 - 9, 256, 64), (100 * 16, 50 * 256, 64),
                                         (711 * 16 - 1, 9 * 256, 64), (173 * 16, 37 * 256, 64), (4400 * 16 - 1, 128, 32),
                                         (401 * 16 - 15, 11 * 128, 32)])
@pytest.mark.parametrize("fmt", ["split", "whole", "fp16"])
def test_decode_turns(rows, cols, S, fmt):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"decode {fmt} {rows}x{cols} S={S}", flush=True)
    w = (random_fp16 if fmt == "fp16" else random_bf16)((rows, cols), seed=rows)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=S, grp_rows=16, **ENCODE[fmt]))
    buf = torch.full((rows * cols + 4096,), 0x5A5A, dtype=torch.int16, device="cuda")
    out = buf[:rows * cols].view(rows, cols)
    for _ in range(2):
        dt.decode(out)
        got = buf.cpu().numpy().view(np.uint16)
        assert np.array_equal(got[:rows * cols].reshape(rows, cols), w)
        assert (got[rows * cols:] == 0x5A5A).all()
        buf.fill_(0x5A5A)
