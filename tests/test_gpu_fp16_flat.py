"""The float16 decode for flat mh codes (every mh code of 5 bits, what Huffman
coding leaves of uniform mantissa bits): one table for ml and e together, mh
by bit reversal, four weights per four column words. Decode is bit-exact with
codes longer than the joint window (the second table) and with quads of
weights around and past the 85 code bits a lane's words are sure to hold (the
bit-serial path); products agree with the oracle within the float32 rounding
of their sum."""
import numpy as np
import pytest

from gen import random_fp16, random_x
from oracle import codec, gemv as ogemv

pytestmark = pytest.mark.gpu
hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


def _weights(rows, cols, kind, seed):
    rng = np.random.default_rng(seed)
    n = rows * cols
    mh = rng.permutation(np.arange(n, dtype=np.uint32) % 32)
    if kind == "gaussian":
        return random_fp16((rows, cols), seed)
    if kind == "mh_alone":  # e and ml without stream bits
        e = np.full(n, 14, dtype=np.uint32)
        ml = np.full(n, 3, dtype=np.uint32)
    else:
        e, ml = (np.minimum(rng.geometric(0.4, n) - 1, 20).astype(np.uint32) for _ in range(2))
        # quads of four weights with rare values of both fields: most of them in some, all in others
        quads = rng.choice(n // 4, n // 500, replace=False)
        for k in range(4):
            for f in (e, ml):
                rare = rng.random(quads.size) < np.where(np.arange(quads.size) % 2, 1.0, 0.7)
                f[quads[rare] * 4 + k] = 29 - rng.integers(0, 18, np.count_nonzero(rare))
    return codec.join_fields16(rng.integers(0, 2, n), e, mh, ml).reshape(rows, cols)


def _flat_container(w, kind, **kw):
    cb = hl.build_codebook16(w)
    assert list(cb.mh.len) == [5] * 32
    e, ml = np.array(cb.e.len)[(w >> 10) & 31], np.array(cb.ml.len)[w & 31]
    bits = (e + ml + 5).reshape(-1, 4).sum(1)
    if kind == "long":
        assert (e + ml).max() > 12 and ((bits > 80) & (bits <= 85)).any() and (bits > 85).any()
    return hl.DeviceTensor(hl.encode(w, codebook=cb, fp16=True, **kw))


# generic kernels (every segment length of the matrix-core product, 32- and
# 64-row groups: decode only) and the persistent kernel (S = 64 and 32)
@pytest.mark.parametrize("shape,kw", [((96, 1024), dict(seg_len=s, grp_rows=16)) for s in (8, 16, 32, 64, 128)] +
                         [((70, 1024), dict(seg_len=64, grp_rows=32)), ((130, 1000), dict(seg_len=200)),
                          ((8200, 2304), {}), ((8200, 2048), dict(seg_len=32, grp_rows=16))])
@pytest.mark.parametrize("kind", ["gaussian", "long", "mh_alone"])
def test_flat_codes(torch, shape, kw, kind):
    print(f"flat fp16 {shape} {kw} {kind}", flush=True)
    w = _weights(*shape, kind, seed=shape[0] + shape[1])
    dt = _flat_container(w, kind, **kw)
    assert np.array_equal(dt.decode().cpu().numpy().view(np.uint16), w)
    if dt.view.grp_rows != 16:
        return
    rows = np.unique(np.r_[:16, shape[0] // 2 + np.arange(8), shape[0] - 16:shape[0]])
    wf = np.abs(ogemv.fp16_to_f64(w))
    for batch in (1, 16):
        x = random_x(batch, shape[1], seed=batch, dtype="f16")
        y = dt.gemv(torch.from_numpy(x).cuda()).cpu().numpy()
        y_ref, den = ogemv.gemv_rows(w, x, rows=rows, weights="fp16")
        assert np.max(ogemv.rel_err(y[:, rows], y_ref, den)) <= shape[1] * 2.0 ** -24
        every = x.astype(np.float64) @ ogemv.fp16_to_f64(w).T
        scale = np.abs(x).astype(np.float64) @ wf.T
        assert np.max(np.abs(y - every) / scale) <= shape[1] * 2.0 ** -24
