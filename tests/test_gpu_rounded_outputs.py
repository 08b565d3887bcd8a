"""Results in the storage type: the same numbers as the fp32 results of the general calls, rounded once.  Whole numbers make every
sum exact in any order, so the comparison is bit for bit."""
import numpy as np
import pytest

from paper_2506_22714_amd import binding as lb
from paper_2506_22714_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def whole(shape, dtype, seed, top=24):
    return torch.from_numpy(np.random.default_rng(seed).integers(-top, top + 1, size=shape).astype(np.float32)).to(dtype).cuda()


def matrix(seed=4):
    """Ragged row count, empty rows, rows that are decomposed, windows that are decomposed."""
    return wl.with_long_rows(wl.random_pattern(333, 260, 0.05, seed=seed, empty_rows=0.2), [7, 150, 332], 200, seed=5)


def plan(A, dtype, **opts):
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a.astype(np.int32))).cuda()
    val = whole(A.nnz, dtype, 6)
    return lb.Plan.from_device_csr(A.M, A.Kc, dev(A.rowptr), dev(A.col), val, resident=True, keep_host_copy=False, **opts)


@pytest.mark.parametrize("opts", [dict(), dict(cs=32, ts=1), dict(mode=lb.MODE_DENSE_ONLY, ts=2), dict(mode=lb.MODE_SCALAR_ONLY, cs=16),
                                  dict(flags=lb.FLAG_XCD_ORDER, cs=50), dict(flags=lb.FLAG_TWO_KERNELS, cs=50)], ids=str)
@pytest.mark.parametrize("dtype", list(DTYPES))
def test_spmm_rounded(dtype, opts):
    A, dt = matrix(), DTYPES[dtype]
    p = plan(A, dt, **opts)
    for N in (32, 64, 96, 128, 224, 256, 512):
        B = whole((A.Kc, N + 8), dt, N)[:, :N]               # a row stride of its own
        want = p.spmm(B)
        assert want.abs().max() > 2048                       # beyond what either type holds exactly: the rounding is part of the test
        got = p.spmm_rounded(B)
        assert got.dtype == dt and torch.equal(got, want.to(dt)), (N, opts)
    # what the fp32 call refuses is refused
    for bad in (B.float(), B[:, :40], B[1:]):
        with pytest.raises((ValueError, lb.LibraError)):
            p.spmm_rounded(bad)
    p.close()


@pytest.mark.parametrize("lds", [0, -1, 7, 64])
def test_spmm_rounded_without_scratch_memory(lds):
    """Rows with one writer need none, whatever its stride is given as; rows with several do."""
    A = wl.random_pattern(333, 260, 0.05, seed=4, empty_rows=0.2)
    p, q = plan(A, torch.float16), plan(matrix(), torch.float16, cs=50)
    assert p.stats()["spmm_zero_rows"] == 0 < q.stats()["spmm_zero_rows"]
    B = whole((A.Kc, 64), torch.float16, 3)
    out = torch.full((A.M, 64), float("nan"), dtype=torch.float16, device="cuda")
    call = lambda plan: lb.libra_spmm_rounded(plan.handle, B.data_ptr(), 64, 64, out.data_ptr(), 64, 0, lds, torch.cuda.current_stream().cuda_stream)
    call(p)
    assert torch.equal(out, p.spmm(B).half())
    with pytest.raises(lb.LibraError) as e:
        call(q)
    assert e.value.code == lb.ERR["NULL"]
    p.close()
    q.close()


def test_spmm_rounded_of_infinities_and_overflow():
    A = matrix()
    p = plan(A, torch.float16, cs=50)
    B = whole((A.Kc, 64), torch.float16, 9) * 128           # sums beyond the largest fp16 number
    B[3, 5], B[4, 6], B[11, 7] = float("inf"), float("-inf"), float("nan")
    want, got = p.spmm(B).to(torch.float16), p.spmm_rounded(B)
    assert torch.isinf(want).any() and torch.isnan(want).any()
    assert torch.equal(got.nan_to_num(1.0, 2.0, 3.0), want.nan_to_num(1.0, 2.0, 3.0)) and torch.equal(got.isnan(), want.isnan())
    p.close()


@pytest.mark.parametrize("K", [32, 64, 128])
@pytest.mark.parametrize("dtype", list(DTYPES))
def test_sddmm_pattern_rounded(dtype, K):
    A, dt = matrix(), DTYPES[dtype]
    X, Y = whole((A.M, K), dt, 1), whole((A.Kc, K), dt, 2)
    for opts in (dict(), dict(sddmm_min_blk_nnz=8), dict(mode=lb.MODE_SCALAR_ONLY), dict(sddmm_min_blk_nnz=8, flags=lb.FLAG_XCD_ORDER)):
        p = plan(A, dt, **opts)
        want = p.sddmm(X, Y, pattern_only=True)
        assert want.abs().max() > 2048
        got = p.sddmm_pattern_rounded(X, Y)
        assert got.dtype == dt and torch.equal(got, want.to(dt)), opts
        with pytest.raises((ValueError, lb.LibraError)):
            p.sddmm_pattern_rounded(X, Y[:, :16])
        p.close()


@pytest.mark.parametrize("dtype", list(DTYPES))
def test_edge_softmax_backward_of_a_rounded_gradient(dtype):
    """A 16-bit gradient is widened exactly: the result is that of the fp32 call on the widened one, bit for bit."""
    A, dt = wl.make("gat", small=True), DTYPES[dtype]        # rows of every length class
    p = plan(A, dt)
    g = torch.Generator(device="cuda").manual_seed(3)
    alpha = p.edge_softmax(torch.randn(A.nnz, device="cuda", generator=g), 0.7)
    d = torch.randn(A.nnz, device="cuda", generator=g).to(dt)
    assert torch.equal(p.edge_softmax_backward_rounded(alpha, d, 0.7), p.edge_softmax_backward(alpha, d.float(), 0.7))
    for bad in (d.float(), d[1:]):
        with pytest.raises(ValueError):
            p.edge_softmax_backward_rounded(alpha, bad, 0.7)
    p.close()


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("n", [1, 7, 8, 9, 4099, 1 << 20])
def test_value_products(dtype, n):
    """Groups of eight, remainders, and arrays that are only aligned to their elements.  The product is rounded from fp32, or (fp16, where one
    instruction does both) without that step between: where the two differ, which is rare, the result is nearer to the exact product."""
    dt = DTYPES[dtype]
    g = torch.Generator(device="cuda").manual_seed(n)
    for shift in ((0, 0), (1, 0), (0, 1), (3, 2)):
        vals = torch.randn(n + 8, device="cuda", generator=g).to(dt)[shift[0]:shift[0] + n]
        factors = (torch.randn(n + 8, device="cuda", generator=g) * 100)[shift[1]:shift[1] + n]
        out = torch.empty_like(vals)
        lb.libra_value_products(vals.data_ptr(), factors.data_ptr(), n, lb.F16 if dtype == "f16" else lb.BF16, out.data_ptr(),
                                torch.cuda.current_stream().cuda_stream)
        by_fp32, exact = (factors * vals.float()).to(dt), factors.double() * vals.double()
        other = out != by_fp32
        assert int(other.sum()) <= n * 2.0 ** -11, shift         # an fp32 product lies next to the middle of two fp16 numbers
        assert bool(((out.double() - exact).abs() < (by_fp32.double() - exact).abs())[other].all()), shift


# ---- numbers that are not whole: rows with one writer are summed in one order, so that the results are the same bits ----
@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("opts", [dict(), dict(mode=lb.MODE_DENSE_ONLY, ts=100), dict(mode=lb.MODE_SCALAR_ONLY)], ids=str)
def test_rounded_sums_of_any_numbers(dtype, opts):
    dt = DTYPES[dtype]
    A = wl.random_pattern(1333, 260, 0.1, seed=4, empty_rows=0.2)
    p = plan(A, dt, **opts)
    assert p.stats()["spmm_zero_rows"] == 0
    g = torch.Generator(device="cuda").manual_seed(2)
    p.set_values(torch.randn(A.nnz, device="cuda", generator=g).to(dt))
    for N in (32, 64, 128, 224):
        B = torch.randn(A.Kc, N, device="cuda", generator=g).to(dt)
        want = p.spmm(B)
        assert torch.equal(p.spmm(B), want) and torch.equal(p.spmm_rounded(B), want.to(dt))
    perm = torch.randperm(A.nnz, device="cuda", generator=g, dtype=torch.int32)
    vals = torch.randn(A.nnz, device="cuda", generator=g).to(dt)
    p.set_values(vals[perm].contiguous(), lb.OP_SPMM)
    want = p.spmm(B)
    p.set_values_ordered(vals, p.value_order(perm))
    assert torch.equal(p.spmm(B), want)
    for K in (32, 64, 128):
        X, Y = torch.randn(A.M, K, device="cuda", generator=g).to(dt), torch.randn(A.Kc, K, device="cuda", generator=g).to(dt)
        assert torch.equal(p.sddmm_pattern_rounded(X, Y), p.sddmm(X, Y, pattern_only=True).to(dt))
    p.close()


@pytest.mark.parametrize("dtype", list(DTYPES))
def test_rounded_sums_of_rows_with_several_writers(dtype):
    """Added up in any order: two calls are as far apart as the order of fp32 sums allows, and at most one rounding further."""
    dt = DTYPES[dtype]
    A = matrix()
    p = plan(A, dt, cs=16, ts=1)
    g = torch.Generator(device="cuda").manual_seed(2)
    vals, B = torch.randn(A.nnz, device="cuda", generator=g).to(dt), torch.randn(A.Kc, 64, device="cuda", generator=g).to(dt)
    p.set_values(vals)
    rows = torch.repeat_interleave(torch.arange(A.M), torch.from_numpy(np.diff(A.rowptr)).long()).cuda()
    terms = vals.double()[:, None] * B.double()[torch.from_numpy(A.col).long().cuda()]
    exact = torch.zeros(A.M, 64, dtype=torch.float64, device="cuda").index_add_(0, rows, terms)
    size = torch.zeros_like(exact).index_add_(0, rows, terms.abs())
    longest = int(np.diff(A.rowptr).max())
    fp32 = size * longest * 2.0 ** -24                            # of any order of additions
    ulp = 2.0 ** -(11 if dtype == "f16" else 8)
    assert bool(((p.spmm(B).double() - exact).abs() <= fp32).all())
    assert bool(((p.spmm_rounded(B).double() - exact).abs() <= fp32 * (1 + ulp) + exact.abs() * ulp + 2.0 ** -25).all())
    p.close()
