"""The small-m matrix-core kernel (m <= 128, or little work; Q8_0 / Q4_0) at the edges of its
tiles: 16-row blocks of x and of the weights, one to four of either per
workgroup, k in steps of eight (lone) or four (long fused runs) 32-weight
blocks, splits of k.

The kernel multiplies the integer codes exactly and scales each block's sum in
fp32, so its error is that of fp32 sums: with 32 products per block, one
scaling and one addition per block and up to 8 partial tiles, at most
(32 + 2 k / 32 + 16) 2^-24 of sum |x||w_hat|."""
import pytest
import torch

from tests.gpu_helpers import QT, XT, assert_parity, bits16, oracle_reference
from paper_2607_02501_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module")
def eb():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2607_02501_amd import eb as m
    return m


def tol(k):
    return (32 + 2 * (k // 32) + 16) * 2.0 ** -24


FORMATS = [("q8_0", torch.bfloat16), ("q8_0", torch.float16), ("q4_0", torch.bfloat16),
           ("q4_0", torch.float16)]


@pytest.mark.parametrize("qtype,xdtype", FORMATS)
@pytest.mark.parametrize("m,n,k", [
    (2, 1, 32), (16, 15, 224), (17, 16, 256), (33, 17, 288), (48, 33, 544),   # fewer columns than CUs: split k
    (49, 3001, 1504), (64, 4097, 256), (65, 2049, 288), (77, 3008, 96),       # one or two row tiles
    (100, 8191, 288), (128, 8193, 224), (128, 16400, 64), (31, 20000, 64),    # wide tiles of the weights
    (129, 1000, 288), (300, 1025, 96), (816, 2560, 160), (700, 4097, 32),     # more rows, tiles of four waves
    (1100, 9, 96), (925, 237, 1056), (513, 150, 2080),                       # fewer columns of tiles than XCDs
])
def test_rows_lone(eb, oracle, qtype, xdtype, m, n, k):
    w = W.normal((n, k), 7 * n + k, "cpu", W.WEIGHT_STD)
    x = W.normal((m, k), 11 * m + k, "cpu").to(xdtype)
    qw = eb.quantize(w.to(DEV), qtype)
    _, y_ref, bound = oracle_reference(oracle, qtype, w.numpy(), x)
    xd = x.to(DEV)
    y = eb.qlinear(qw, xd, path="mfma")                      # with a workspace: k may be split
    assert_parity(y, y_ref, bound, tol(k), f"rows {qtype} m={m} n={n} k={k}")
    out = torch.full((m + 1, n), 7.0, device=DEV)            # without one; nothing past the last row
    op = eb.make_op(qw, xd, out[:m])
    import ctypes
    st = eb.lib.eb_qlinear_fused_ws(ctypes.byref(op), eb.EB_PATH_MFMA, None, 0,
                                    torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert_parity(out[:m], y_ref, bound, tol(k), f"rows_nows {qtype} m={m} n={n} k={k}")
    assert bool((out[m] == 7.0).all())


@pytest.mark.parametrize("qtype,xdtype", FORMATS)
@pytest.mark.parametrize("shapes", [
    # (m, n, k): few workgroups (narrow weight tiles), then enough for the widest ones
    [(50, 40, 1056), (3, 33, 32), (128, 17, 288)],
    [(50, 8200, 160), (16, 8190, 96), (33, 1024, 1056), (64, 65, 32)],
])
def test_rows_fused_run(eb, oracle, qtype, xdtype, shapes):
    entries, refs = [], []
    for i, (m, n, k) in enumerate(shapes):
        w = W.normal((n, k), 31 * i + n, "cpu", W.WEIGHT_STD)
        x = W.normal((m, k), 37 * i + m, "cpu").to(xdtype)
        _, y_ref, bound = oracle_reference(oracle, qtype, w.numpy(), x)
        entries.append((eb.quantize(w.to(DEV), qtype), x.to(DEV),
                        torch.full((m, n), 7.0, device=DEV)))
        refs.append((y_ref, bound, k))
    ops = eb.make_ops(entries)
    assert eb.stack_launches(ops) == 1
    for _ in range(2):  # the second call replays the recorded graph
        eb.qlinear_stack(ops)
        for (_, _, y), (y_ref, bound, k) in zip(entries, refs):
            assert_parity(y, y_ref, bound, tol(k), f"rows_fused {qtype} k={k}")
            y.fill_(7.0)
    eb.stack_cache_clear()


@pytest.mark.parametrize("qtype,xdtype", FORMATS)
@pytest.mark.parametrize("m,n,k", [
    (2, 4096, 4096), (2, 4097, 4064), (2, 12289, 64), (3, 8193, 4096), (4, 8192, 4128),  # both sides of the rule
    (3, 17, 32), (5, 1, 32), (7, 4099, 2080), (8, 33, 8192),
])
def test_gemv_of_several_rows(eb, oracle, qtype, xdtype, m, n, k):
    """The bandwidth path at 2 to 8 rows, on either side of the rule that
    takes it to this kernel, with no workspace and each epilogue."""
    w = W.normal((n, k), 5 * n + k, "cpu", W.WEIGHT_STD)
    x = W.normal((m, k), 13 * m + k, "cpu").to(xdtype)
    qw, xd = eb.quantize(w.to(DEV), qtype), x.to(DEV)
    _, y_ref, bound = oracle_reference(oracle, qtype, w.numpy(), x)
    y = eb.qlinear(qw, xd, path="gemv")
    assert_parity(y, y_ref, bound, tol(k), f"rows_gemv {qtype} m={m} n={n} k={k}")
    r = W.normal((m, n), 17 * n + m, "cpu")
    got = eb.qlinear_fused(qw, xd, epilogue="add", residual=r.to(DEV), path="gemv")
    # the epilogues act on the same fp32 sums, in one rounding each
    torch.testing.assert_close(got, y + r.to(DEV), rtol=0, atol=0)
    if n % 2 == 0:
        z = y.double()
        want = z[:, 0::2] / (1 + torch.exp(-z[:, 0::2])) * z[:, 1::2]
        got = eb.qlinear_fused(qw, xd, epilogue="glu", path="gemv")
        # silu and the product in fp32, the exponential to 2^-21: 2^-19 of the result covers both
        torch.testing.assert_close(got.double(), want, rtol=2.0 ** -19, atol=1e-30)


@pytest.mark.parametrize("qtype", ["q8_0", "q4_0"])
@pytest.mark.parametrize("m,n,k,path", [
    (50, 40, 1056, "mfma"),      # k split: partial sums
    (128, 8193, 224, "mfma"),    # wide tiles of the weights
    (300, 1025, 96, "mfma"),     # more rows
    (7, 257, 2080, "gemv"),      # the bandwidth path at several rows
])
def test_activations_beyond_the_range_of_a_block_sum(eb, oracle, qtype, m, n, k, path):
    """bfloat16 activations whose sums with the integer codes leave the range of
    fp32 before the block's scale brings the output back into it, between rows
    of ordinary ones; and blocks of scale zero with codes, which add nothing.
    Such outputs are fp32 sums over k of exact products: k 2^-24 of the bound,
    and as much again for the parts of a split."""
    w = W.normal((n, k), 3 * n + k, "cpu", W.WEIGHT_STD)
    x = W.normal((m, k), 19 * m + k, "cpu")
    x[::3] *= 2.0 ** 125                       # sums with the codes of 2^129 and more, outputs near 2^125
    x[1] = torch.where(x[1] < 0, -1.0, 1.0) * 3.38e38
    x = x.to(torch.bfloat16)
    blocks = oracle.quantize(QT[qtype], w.numpy())
    blocks[:, 1::3, :2] = 0
    # row 1 (the largest finite activations) meets scales of 2^-24
    small = blocks.copy()
    small[:, 0::3, 0], small[:, 0::3, 1] = 1, 0
    small[:, 2::3, 0], small[:, 2::3, 1] = 1, 0
    for b, rows in ((blocks, [i for i in range(m) if i != 1]), (small, [1])):
        qw = eb.from_canonical(torch.from_numpy(b).to(DEV), qtype, n, k)
        y_ref, bound = oracle.qlinear(QT[qtype], b, n, k, bits16(x[rows]), XT[x.dtype])
        bar = 2 * k * 2.0 ** -24 + tol(k)
        xd = x.to(DEV)
        y = eb.qlinear(qw, xd, path=path)[rows]
        assert_parity(y, y_ref, bound, bar, f"rows_range {qtype} m={m} n={n} k={k}")
        if m <= 128:  # as a fused run
            out = [torch.zeros(m, n, device=DEV) for _ in range(2)]
            eb.qlinear_stack(eb.make_ops([(qw, xd, o) for o in out]))
            for o in out:
                assert_parity(o[rows], y_ref, bound, bar, f"rows_range_fused {qtype} m={m} n={n} k={k}")
            eb.stack_cache_clear()
