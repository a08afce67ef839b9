"""Runs of long code pairs (no joint limit: pairs of up to 22 bits, longer than
the decode tables' window), so that four of them do not fit one 64-bit window:
every kernel that decodes, bit for bit against the weights that were encoded,
and every product within the float32 rounding of a sum of cols products of the
float64 value."""
import numpy as np
import pytest

from gen import random_bf16, random_x
from oracle import codec

hl = pytest.importorskip("paper_2502_00922_amd.hufflm")


@pytest.fixture(scope="module")
def torch():
    import torch as t
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    hl.lib()
    return t


def _weights(rows, cols, runs, whole_segment=False):
    """Weights and their codebook. Seven blocks of 16 exponents in use besides a
    trained matrix's two, each twice as often as the one before; the codes are of
    these weights (high exponent bits up to 8 or 9, low ones up to 13). Then
    `runs` runs of 3 to 9 weights of the rarest blocks and low exponent bits,
    and with `whole_segment` one segment of 64 of them."""
    w = random_bf16((rows, cols), seed=rows + cols, outliers=False)
    rng = np.random.default_rng(rows)
    flat = w.reshape(-1)
    blocks = [0, 1, 2, 3, 4, 5, 8]
    for k, b in enumerate(blocks):
        at = rng.integers(0, flat.size, 8 << k)
        flat[at] = (flat[at] & 0x87FF) | (b << 11)
    cb = hl.build_codebook(w, 15, 0)
    low = np.argsort(cb.el.len, kind="stable")[-4:]

    def rare(n):
        return ((rng.choice(blocks[:3], n) << 4 | rng.choice(low, n)) << 7 | rng.integers(0, 128, n)).astype(np.uint16)

    for at in rng.integers(0, flat.size - 9, runs):
        n = int(rng.integers(3, 10))
        flat[at:at + n] = rare(n)
    if whole_segment:
        w[rows // 2, 64:128] = rare(64)
    return w, cb


def _pairs(w, cb):
    e = (w >> 7) & 0xFF
    return np.array(cb.eh.len)[e >> 4] + np.array(cb.el.len)[e & 15]


def test_runs_do_not_fit_a_window():
    import torch  # noqa: F401  its HIP runtime before the library's: the tests below share this process
    # (no GPU) the weights are what the tests below are about, and the container holds them
    w, cb = _weights(64, 2048, 200, True)
    bits = _pairs(w, cb).astype(int)
    first3, fourth = bits[:, :-3] + bits[:, 1:-2] + bits[:, 2:-1], bits[:, 3:]
    cut = (first3 > 62 - 13) & (first3 + fourth > 62) & (bits[:, 0:-3] > 13)
    assert cut.sum() > 100
    blob = hl.encode(w, seg_len=64, grp_rows=16, codebook=cb)
    assert np.array_equal(np.asarray(codec.decode(bytes(blob))).reshape(w.shape), w)


# the small matrix-core kernel and a segment too long for the persistent one;
# the persistent kernel (20 stream words, one and several rounds, ragged rows);
# shorter segments; the vector kernel's groups
CASES = [(301, 2048, 64, 16, 300, True), (4352, 4096, 64, 16, 600, False), (4101, 8192, 64, 16, 600, False),
         (4352, 4096, 32, 16, 300, False), (300, 1024, 128, 16, 200, True), (130, 1000, 200, 64, 100, True)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,cols,S,GR,runs,whole_segment", CASES)
def test_decode_and_products(torch, rows, cols, S, GR, runs, whole_segment):
    w, cb = _weights(rows, cols, runs, whole_segment)
    dt = hl.DeviceTensor(hl.encode(w, seg_len=S, grp_rows=GR, codebook=cb))
    print(f"long pairs {rows}x{cols} S={S} GR={GR}: decode", flush=True)
    out = dt.decode().cpu().numpy().view(np.uint16)
    assert np.array_equal(out, w), np.argwhere(out != w)[:8].tolist()
    wd = torch.from_numpy(w.view(np.int16)).view(torch.bfloat16).cuda().double()

    def check(what, x, y):
        ref, den = x.double() @ wd.t(), x.double().abs() @ wd.abs().t()
        err = float(((y.double() - ref).abs() / den).max())
        assert err <= cols * 2.0 ** -24, (what, err)

    for batch in (1, 3, 16):
        for xdt in ("bf16", "f32"):
            print(f"long pairs {rows}x{cols} S={S} GR={GR}: gemv {xdt} batch {batch}", flush=True)
            x = random_x(batch, cols, seed=batch, dtype=xdt)
            x = (torch.from_numpy(x.view(np.int16)).view(torch.bfloat16) if xdt == "bf16" else torch.from_numpy(x)).cuda()
            check((xdt, batch), x, dt.gemv(x, torch.full((batch, rows), float("nan"), device="cuda")))
    if GR == 16 and S in (32, 64) and not whole_segment:
        for tokens in (20, 50, 100):
            print(f"long pairs {rows}x{cols} S={S}: gemm {tokens} tokens", flush=True)
            x = torch.from_numpy(random_x(tokens, cols, seed=tokens, dtype="bf16").view(np.int16))
            x = x.view(torch.bfloat16).cuda()
            check(("gemm", tokens), x, dt.gemm(x, torch.full((tokens, rows), float("nan"), device="cuda")))
