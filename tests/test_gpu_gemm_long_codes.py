"""Prefill products of more than 64 tokens of a matrix with a segment of the
longest codes: its stream columns do not fit the fused kernel's LDS, so the
product must not depend on the vendor library having an algorithm for it.
Every output within the float32 rounding of a sum of cols products of the
float64 value."""
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


def _weights(rows, cols):
    """Six blocks of 16 exponents in use besides a trained matrix's two, each
    twice as often as the one before (codes of up to 7 bits), and one segment in
    the rarest of them with rare low exponent bits (13 bits)."""
    w = random_bf16((rows, cols), seed=rows, outliers=False)
    rng = np.random.default_rng(rows)
    for k in range(6):
        at = rng.integers(0, w.size, 64 << k)
        w.reshape(-1)[at] = (w.reshape(-1)[at] & 0x87FF) | (k << 11)
    w[rows // 2, 64:128] = np.tile(np.array([(e << 7) | 5 for e in (0x0C, 0x0D)], dtype=np.uint16), 32)
    return w


# sums that the vendor's algorithms divide over blocks, and shorter ones; tokens
# in whole and ragged batches of 16
@pytest.mark.parametrize("rows,cols", [(2605, 22784), (301, 2048)])
@pytest.mark.parametrize("tokens", [65, 128, 198, 402])
def test_long_segment(torch, rows, cols, tokens):
    print(f"gemm with a long segment {rows}x{cols} tokens={tokens}", flush=True)
    w = _weights(rows, cols)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=64, grp_rows=16, lmax=15, pair_max=0))
    assert dt.view.max_seg_bits > 64 * 16, dt.view.max_seg_bits
    x = torch.from_numpy(random_x(tokens, cols, seed=tokens, dtype="bf16").view(np.int16)).view(torch.bfloat16).cuda()
    y = dt.gemm(x, torch.full((tokens, rows), float("nan"), device="cuda"))
    wd = torch.from_numpy(w.view(np.int16)).view(torch.bfloat16).cuda().double()
    ref, den = x.double() @ wd.t(), x.double().abs() @ wd.abs().t()
    assert float(((y.double() - ref).abs() / den).max()) <= cols * 2.0 ** -24
    assert torch.equal(dt.gemm(x), y)
