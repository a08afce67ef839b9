"""Prefill products of more than 64 tokens whose vendor algorithm would divide
the sums over blocks (few output tiles, long sums): they run without a GEMM
workspace, by another algorithm or the fused kernel, whose partial
sums fit the workspace. Every output within the float32 rounding of a sum of cols products of the float64 value."""
import time

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


# a prompt length that was seen before, after a hundred others, costs no second
# question to the vendor's library (65 of a call's 81 us of host time; 17 without)
def test_choices_of_many_lengths_are_kept(torch):
    rows, cols = 2048, 2048
    dt = hl.DeviceTensor(hl.encode(random_bf16((rows, cols), seed=1), seg_len=64, grp_rows=16))
    x = torch.from_numpy(random_x(200, cols, seed=1, dtype="bf16").view(np.int16)).view(torch.bfloat16).cuda()
    y = torch.empty((200, rows), device="cuda")
    took = []
    for _ in range(3):
        took.append([])
        for tokens in range(70, 200):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            dt.gemm(x[:tokens], y[:tokens])
            took[-1].append(time.perf_counter() - t0)
        print(f"130 lengths: median {1e6 * np.median(took[-1]):.0f} us", flush=True)
    assert np.median(took[2]) < 0.35 * np.median(took[0]), [np.median(t) for t in took]
