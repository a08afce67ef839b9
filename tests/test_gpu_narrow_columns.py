"""Matrices of 8 to 15 column blocks and many row blocks on the persistent
kernel, whose blocks then have as many waves as there are column blocks (and
float16 products of 8, which stay off it): products of one to 64 activation
rows within the float32 rounding of a sum of cols products of the float64
value, decode bit-exact, grouped launches equal to single ones' values."""
import numpy as np
import pytest

from gen import random_bf16, random_fp16, random_x

pytestmark = pytest.mark.gpu
hl = pytest.importorskip("paper_2502_00922_amd.hufflm")

ENCODE = {"split": {}, "whole": {"whole_exponent": True}, "fp16": {"fp16": True}}


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


def _matrix(torch, rows, cols, fmt, S, seed):
    half = torch.float16 if fmt == "fp16" else torch.bfloat16
    w = (random_fp16 if fmt == "fp16" else random_bf16)((rows, cols), seed)
    return w, hl.DeviceTensor(hl.encode(w, seg_len=S, grp_rows=16, **ENCODE[fmt])), \
        torch.from_numpy(w.view(np.int16)).view(half).cuda().double()


def _x(torch, n, cols, fmt):
    x = random_x(n, cols, seed=n, dtype="f16" if fmt == "fp16" else "bf16")
    return torch.from_numpy(x.view(np.int16)).view(torch.float16 if fmt == "fp16" else torch.bfloat16).cuda()


def _close(y, x, wd):
    ref, den = x.double() @ wd.t(), x.double().abs() @ wd.abs().t()
    return float(((y.double() - ref).abs() / den).max()) <= wd.shape[1] * 2.0 ** -24


# 8 column blocks (the fewest), ones between, 15 (the last with fewer than 16
# waves), 17 and 18 (two rounds of 9 at most, in fours); ragged last row blocks
@pytest.mark.parametrize("rows,cols,S", [(9217, 2048, 64), (9001, 2304, 64), (8999, 3328, 64), (8195, 3840, 64),
                                         (6700, 4608, 64), (6001, 4352, 64), (9210, 1152, 32)])
@pytest.mark.parametrize("fmt", ["split", "whole", "fp16"])
def test_narrow(torch, rows, cols, S, fmt):
    print(f"narrow {fmt} {rows}x{cols} S={S}", flush=True)
    w, dt, wd = _matrix(torch, rows, cols, fmt, S, rows)
    assert np.array_equal(dt.decode().cpu().numpy().view(np.uint16), w)
    for batch in (1, 5, 16):
        x = _x(torch, batch, cols, fmt)
        assert _close(dt.gemv(x), x, wd)
    for tokens in (3, 17, 33, 64) if fmt != "fp16" else ():
        x = _x(torch, tokens, cols, fmt)
        assert _close(dt.gemm(x), x, wd)


@pytest.mark.parametrize("shapes", [((3072, 3072),) * 3, ((4100, 2304), (4100, 2304)), ((4096, 4096), (1024, 4096), (1024, 4096))])
@pytest.mark.parametrize("fmt", ["split", "whole"])
def test_narrow_grouped(torch, shapes, fmt):
    print(f"narrow grouped {fmt} {shapes}", flush=True)
    ms = [_matrix(torch, r, c, fmt, 64, k) for k, (r, c) in enumerate(shapes)]
    for batch in (1, 7):
        x = _x(torch, batch, shapes[0][1], fmt)
        for (_, _, wd), y in zip(ms, hl.gemv_multi([m[1] for m in ms], x)):
            assert _close(y, x, wd)
