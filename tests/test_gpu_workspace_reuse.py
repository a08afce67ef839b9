"""One workspace over calls of different batches and matrices: a split
product's arrival counters are zero for every call, whatever the calls before
it left in the workspace (tiled activations of a larger batch, partial sums of
another matrix). The outputs are NaN before each call and afterwards equal, bit
for bit, the outputs of the same call on a fresh zeroed workspace."""
import itertools

import numpy as np
import pytest

from gen import random_bf16, random_fp16, random_x

pytestmark = pytest.mark.gpu
hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


def _matrix(rows, cols, fp16=False, seed=0):
    w = (random_fp16 if fp16 else random_bf16)((rows, cols), seed=rows + cols + seed)
    return hl.DeviceTensor(hl.encode(w, seg_len=64, grp_rows=16, fp16=fp16))


def _x(torch, batch, cols, xdt):
    x = random_x(batch, cols, seed=batch, dtype=xdt)
    return (torch.from_numpy(x.view(np.int16)).view(torch.bfloat16) if xdt == "bf16" else torch.from_numpy(x)).cuda()


def _nan(torch, batch, dt):
    return torch.full((batch, dt.shape[0]), float("nan"), device="cuda")


def _fresh(torch, dt):
    return torch.zeros(max(4, dt.workspace().numel()), dtype=torch.uint8, device="cuda")


# more than 8 column blocks of 256 and at most 128 row blocks: split products
@pytest.mark.parametrize("rows,cols", [(1000, 4096), (16, 8192), (2048, 2304)])
@pytest.mark.parametrize("xdt", ["bf16", "f32", "f16"])
def test_batches_in_any_order(torch, rows, cols, xdt):
    dt = _matrix(rows, cols, fp16=xdt == "f16")
    kinds = ["bf16", "f32"] if xdt == "bf16" else [xdt]  # both kinds of a bf16 matrix share its workspace
    xs = {(k, b): _x(torch, b, cols, k) for k in kinds for b in (1, 3, 16)}
    ref = {key: dt.gemv(x, _nan(torch, key[1], dt), workspace=_fresh(torch, dt)).clone() for key, x in xs.items()}
    assert not any(bool(torch.isnan(r).any()) for r in ref.values())
    for a, b in itertools.permutations(xs, 2):
        print(f"workspace {rows}x{cols} x={xdt}: {a} then {b}", flush=True)
        for key in (a, b):
            assert torch.equal(dt.gemv(xs[key], _nan(torch, key[1], dt)), ref[key]), (a, b, key)


# matrices that are multiplied one after another (not enough row blocks for a
# grouped launch), the larger one's workspace shared, and a group of one launch
# whose small matrices are split when multiplied alone
@pytest.mark.parametrize("rows,cols", [((2048, 512), 4096), ((512, 2048), 4096), ((2048, 1024, 1024), 4096)])
def test_products_after_gemv_multi(torch, rows, cols):
    ts = [_matrix(r, cols, seed=k) for k, r in enumerate(rows)]
    for batch, then in itertools.product((1, 5, 16), (1, 16)):
        print(f"multi {rows}x{cols} batch {batch}, then each with {then}", flush=True)
        x, x1 = _x(torch, batch, cols, "bf16"), _x(torch, then, cols, "bf16")
        ref = [t.gemv(x1, _nan(torch, then, t), workspace=_fresh(torch, t)).clone() for t in ts]
        ys = [_nan(torch, batch, t) for t in ts]
        hl.gemv_multi(ts, x, ys)
        assert not any(bool(torch.isnan(y).any()) for y in ys)
        for t, r in zip(ts, ref):
            assert torch.equal(t.gemv(x1, _nan(torch, then, t)), r)
        # and the other way round: the workspace of a single product, then the group
        again = [_nan(torch, batch, t) for t in ts]
        hl.gemv_multi(ts, x, again)
        assert all(torch.equal(a, y) for a, y in zip(again, ys))


# one workspace, large enough for each, handed to matrices of different sizes
def test_one_workspace_for_several_matrices(torch):
    ts = [_matrix(r, c) for r, c in ((1000, 4096), (32, 16384), (2048, 3072), (4352, 4096))]
    ws = torch.zeros(max(t.workspace().numel() for t in ts), dtype=torch.uint8, device="cuda")
    for batch in (16, 1, 3, 16, 1):
        for t in ts:
            x = _x(torch, batch, t.shape[1], "bf16")
            ref = t.gemv(x, _nan(torch, batch, t), workspace=_fresh(torch, t))
            print(f"shared workspace {t.shape} batch {batch}", flush=True)
            assert torch.equal(t.gemv(x, _nan(torch, batch, t), workspace=ws), ref)
