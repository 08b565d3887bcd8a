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


def test_spmm_rounded_of_infinities_and_overflow():
    A = matrix()
    p = plan(A, torch.float16, cs=50)
    B = whole((A.Kc, 64), torch.float16, 9) * 128           # sums beyond the largest fp16 number
    B[3, 5], B[4, 6], B[11, 7] = float("inf"), float("-inf"), float("nan")
    want, got = p.spmm(B).to(torch.float16), p.spmm_rounded(B)
    assert torch.isinf(want).any() and torch.isnan(want).any()
    assert torch.equal(got.nan_to_num(1.0, 2.0, 3.0), want.nan_to_num(1.0, 2.0, 3.0)) and torch.equal(got.isnan(), want.isnan())
    p.close()
