"""Prefill products of more than 64 tokens whose vendor algorithm would divide
the sums over blocks (few output tiles, long sums): they run without a GEMM
workspace, by another algorithm or the fused kernel, whose partial
sums fit the workspace. Every output within the float32 rounding of a sum of cols products of the float64 value."""
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


# 31 tiles of columns or more per row set, ragged rows, one to five chunks of
# 128 tokens, and a workspace of fewer ranges than the fused kernel would take
@pytest.mark.parametrize("rows,cols,S", [(40, 28672, 64), (288, 11008, 64), (301, 8192, 32)])
@pytest.mark.parametrize("tokens", [65, 100, 128, 129, 512, 600])
@pytest.mark.parametrize("whole", [False, True])
def test_few_tiles_long_sums(torch, rows, cols, S, tokens, whole):
    print(f"gemm {rows}x{cols} S={S} tokens={tokens} whole={whole}", flush=True)
    w = random_bf16((rows, cols), seed=rows)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=S, grp_rows=16, whole_exponent=whole))
    x = torch.from_numpy(random_x(tokens, cols, seed=tokens, dtype="bf16").view(np.int16)).view(torch.bfloat16).cuda()
    y = dt.gemm(x)
    wd = torch.from_numpy(w.view(np.int16)).view(torch.bfloat16).cuda().double()
    ref, den = x.double() @ wd.t(), x.double().abs() @ wd.abs().t()
    assert float(((y.double() - ref).abs() / den).max()) <= cols * 2.0 ** -24
    assert torch.equal(dt.gemm(x), y)
