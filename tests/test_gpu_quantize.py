"""Quantization at its rounding thresholds: weights on (q + 1/2) times the
stored scale and one binary32 step to either side of it, for every code, with
small, ordinary, large and subnormal binary16 scales of either sign.  Packed bytes
equal the oracle's, which decides on binary64 quotients."""
import numpy as np
import pytest
import torch

from paper_2607_02501_amd import workloads as W
from tests.gpu_helpers import QT

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eb():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_02501_amd import eb as m
    return m


def _near(points):
    p = np.asarray(points, dtype=np.float32)
    up, down = np.nextafter(p, np.float32(np.inf)), np.nextafter(p, np.float32(-np.inf))
    return np.concatenate([p, up, down])


def _threshold_blocks(size, extreme, lo, hi, sub=None):
    """Blocks of `size` weights whose first weight, extreme * d, fixes the scale d."""
    rng = np.random.default_rng(3)
    rows = []
    for bits in (0x0001, 0x0007, 0x03ff, 0x0400, 0x1234, 0x211d, 0x2c01, 0x3555, 0x3c00, 0x4a6b, 0x5bff):
        d = np.float32(np.uint16(bits).view(np.float16))
        for sign in (1.0, -1.0):
            for e in ((d,) if sub is None else [np.float32(d * s) for s in sub]):
                t = _near([(q + 0.5) * e for q in range(lo, hi)]) * np.float32(sign)
                t = rng.permutation(t)
                t = np.resize(t, (len(t) + size - 2) // (size - 1) * (size - 1)).reshape(-1, size - 1)
                rows.append(np.concatenate([np.full((len(t), 1), extreme * e * sign, np.float32), t], 1))
    return np.concatenate(rows)


@pytest.mark.parametrize("qtype,k", [("q8_0", 32), ("q8_0", 288), ("q4_0", 32), ("q4_0", 288),
                                     ("q6_s", 256), ("q6_s", 2304)])
def test_rounding_thresholds_bit_exact(eb, oracle, qtype, k):
    if qtype == "q8_0":
        b = _threshold_blocks(32, 127.0, -127, 127)
    elif qtype == "q4_0":
        b = _threshold_blocks(32, -8.0, -8, 7)
    else:  # sub-blocks of 16 with sub-scales of many sizes; one of 127 d fixes d16
        b = _threshold_blocks(16, -32.0, -32, 31, sub=(1, 2, 3, 31, 64, 99, 126, 127))
    flat = b.reshape(-1)
    n = -(-flat.size // k) + 1
    w = np.resize(flat, (n, k)).astype(np.float32)
    wt = torch.from_numpy(w)
    qw = eb.quantize(wt.cuda(), qtype)
    got = eb.to_canonical(qw).cpu().numpy()
    assert np.array_equal(got, oracle.quantize(QT[qtype], w))
    back = eb.from_canonical(torch.from_numpy(got).cuda(), qtype, n, k)
    assert torch.equal(back.buf, qw.buf)


@pytest.mark.parametrize("qtype,n,k", [("q8_0", 5, 32), ("q4_0", 3, 96), ("q4_0", 37, 1504),
                                       ("q6_s", 3, 256), ("q6_s", 67, 768)])
def test_canonical_at_any_byte_offset(eb, oracle, qtype, n, k):
    """Canonical bytes have no alignment requirement: both directions at every
    offset modulo 16 give the oracle's bytes."""
    w = W.normal((n, k), n + k, "cpu", W.WEIGHT_STD)
    ref = oracle.quantize(QT[qtype], w.numpy()).reshape(-1)
    qw = eb.quantize(w.cuda(), qtype)
    c, s = qw.c, torch.cuda.current_stream().cuda_stream
    for off in (0, 1, 2, 4, 8, 15):
        dst = torch.full((ref.size + 32,), 0xA5, dtype=torch.uint8, device="cuda")
        assert eb.lib.eb_qweights_to_canonical(c, dst.data_ptr() + off, s) == 0
        host = dst.cpu().numpy()
        assert np.array_equal(host[off:off + ref.size], ref), off
        assert (host[:off] == 0xA5).all() and (host[off + ref.size:] == 0xA5).all()
        out = eb.empty_qweights(qtype, n, k)
        assert eb.lib.eb_qweights_from_canonical(eb.QTYPES[qtype], dst.data_ptr() + off, n, k,
                                                 out.buf.data_ptr(), s) == 0
        assert torch.equal(out.buf, qw.buf)
