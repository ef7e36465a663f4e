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

from tests.gpu_helpers import assert_parity, oracle_reference
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
