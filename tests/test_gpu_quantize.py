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


def _not_finite(n, k):
    """Ordinary weights with, by row: one NaN, infinities, a whole block of 32
    (and of 16) NaNs, a row of them, NaNs among zeros."""
    w = W.normal((n, k), n + k, "cpu", W.WEIGHT_STD).numpy().copy()
    w[0, 5] = np.nan
    w[1, 7], w[1, 70] = np.inf, -np.inf
    w[2, 32:64] = np.nan
    w[3, 16:32] = -np.nan
    w[4, :] = np.nan
    w[5, :] = 0.0
    w[5, 3] = np.nan
    return w


def _ieee_blocks(qtype, w):
    """The formats' definitions in IEEE arithmetic: comparisons and maxima pass
    NaNs by, and a quotient that is NaN takes the lowest code."""
    n, k = w.shape
    with np.errstate(invalid="ignore", divide="ignore", over="ignore"):
        if qtype == "q6_s":
            b = w.reshape(n, k // 256, 16, 16)
            mag = np.where(np.isnan(b), -1.0, np.abs(b))
            m = np.take_along_axis(b, mag.argmax(-1)[..., None], -1)
            m = np.where(mag.max(-1, keepdims=True) > 0, m, np.float32(0))
            s = m / np.float32(-32)
            d = (np.abs(s).max(2, keepdims=True) / np.float32(127)).astype(np.float16).astype(np.float64)
            sc = _nearest(s.astype(np.float64), d, -127, 127, away=True)
            e = d * sc
            return d, sc, _nearest(b.astype(np.float64), e, -32, 31, away=False)
        b = w.reshape(n, k // 32, 32)
        mag = np.where(np.isnan(b), -1.0, np.abs(b))
        m = np.take_along_axis(b, mag.argmax(-1)[..., None], -1)
        m = np.where(mag.max(-1, keepdims=True) > 0, m, np.float32(0))
        d32 = np.abs(m) / np.float32(127) if qtype == "q8_0" else m / np.float32(-8)
        d = d32.astype(np.float16).astype(np.float64)
        lo, hi = (-127, 127) if qtype == "q8_0" else (-8, 7)
        return d, None, _nearest(b.astype(np.float64), d, lo, hi, away=qtype == "q8_0")


def _nearest(v, d, lo, hi, away):
    t = v / d
    t = np.sign(t) * np.floor(np.abs(t) + 0.5) if away else np.floor(t + 0.5)
    return np.where(d == 0, 0, np.where(np.isnan(t), lo, np.clip(t, lo, hi)))


@pytest.mark.parametrize("qtype", ["q8_0", "q4_0", "q6_s"])
def test_weights_that_are_not_finite(eb, qtype):
    n, k = 7, 768
    w = _not_finite(n, k)
    got = eb.to_canonical(eb.quantize(torch.from_numpy(w).cuda(), qtype)).cpu().numpy()
    d, sc, q = _ieee_blocks(qtype, w)
    nb = k // (256 if qtype == "q6_s" else 32)
    assert np.array_equal(got[..., :2].copy().view(np.float16)[..., 0].astype(np.float64), d.reshape(n, nb))
    if qtype == "q8_0":
        assert np.array_equal(got[..., 2:].view(np.int8), q)
    elif qtype == "q4_0":
        codes = np.concatenate([got[..., 2:] & 15, got[..., 2:] >> 4], -1).astype(int) - 8
        assert np.array_equal(codes, q)
    else:
        assert np.array_equal(got[..., 2:18].view(np.int8), sc[..., 0])
        c = got[..., 18:].reshape(n, nb, 8, 24).astype(int)
        low = np.concatenate([c[..., :16] & 15, c[..., :16] >> 4], -1)
        top = np.concatenate([c[..., 16:] >> s & 3 for s in (0, 2, 4, 6)], -1)
        assert np.array_equal((low | top << 4).reshape(n, nb, 16, 16) - 32, q)
