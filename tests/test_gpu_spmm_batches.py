"""The 16-bit SpMM task at the edges of its batches: windows with every combination of dense vectors around whole blocks and
pairs of blocks and residual nonzeros around whole batches, each row owned, split or shared, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2506_22714_amd import binding as lb
from paper_2506_22714_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DENSE = (0, 1, 16, 17, 32, 33, 49)          # vectors of three or more nonzeros per window
SINGLE = (0, 1, 31, 32, 33, 64, 65, 130)    # columns with one nonzero


def edge_windows(seed=5, Kc=400):
    rng = np.random.default_rng(seed)
    D = np.zeros((16 * len(DENSE) * len(SINGLE) - 5, Kc), dtype=np.float32)
    w = 0
    for d in DENSE:
        for r in SINGLE:
            rows = np.arange(16 * w, min(16 * w + 16, D.shape[0]))
            cols = rng.permutation(Kc)
            for c in cols[:d]:
                D[rng.choice(rows, size=rng.integers(3, rows.size + 1), replace=False), c] = 1.0
            one_row = rng.random() < 0.3        # every third window: all its single nonzeros in one row, which is then split
            D[rng.choice(rows) if one_row else rng.choice(rows, size=r), cols[d:d + r]] = 1.0
            w += 1
    A = wl.from_dense(D)
    return wl.Csr(A.M, A.Kc, A.rowptr, A.col, wl.uniform_values(rng, A.nnz))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("N", [32, 64, 128, 224])
def test_batch_edges(N, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    A = edge_windows()
    B = wl.dense_normal(A.Kc, N, seed=1, dtype=np.float32)
    if dtype == "bf16":
        B, val = wl.to_bf16_bits(B), wl.to_bf16_bits(A.val.astype(np.float32))
        Bd = torch.from_numpy(B.view(np.int16)).cuda().view(torch.bfloat16)
    else:
        B, val = B.astype(np.float16), A.val
        Bd = torch.from_numpy(B).cuda()
    ref, S = oracle.spmm(A.rowptr, A.col, val, B, bf16=dtype == "bf16")
    deg = np.diff(A.rowptr).astype(np.float64)
    limit = 16.0 * np.sqrt(deg.max()) * 2.0 ** -24      # exact products, deg - 1 fp32 additions
    for opts in (dict(), dict(flags=lb.FLAG_NO_FILL_PADDING), dict(flags=lb.FLAG_NO_FILL_PADDING, cs=40, ts=2),
                 dict(flags=lb.FLAG_TWO_KERNELS, cs=40), dict(mode=lb.MODE_SCALAR_ONLY), dict(mode=lb.MODE_DENSE_ONLY)):
        p = lb.Plan.from_csr(A, val=val, val_dtype=lb.BF16 if dtype == "bf16" else None, **opts).upload()
        C = torch.full((A.M, N), float("nan"), device="cuda")
        got = p.spmm(Bd, out=C).cpu().numpy()
        err = oracle.graded_error(got, ref, S, np.maximum(deg, 1)[:, None])
        assert err <= limit, f"{dtype} N={N} {opts}: {err:.3e} > {limit:.3e}"
        p.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("N", [32, 64, 128, 224])
def test_inf_and_nan_reach_only_the_rows_that_refer_to_them(N, dtype):
    """0 * Inf = NaN: an Inf or NaN in a row of B must not come into the sums through the empty places of a tile, nor subnormal
    numbers be lost in it."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    A = edge_windows(seed=6)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float16
    B = torch.from_numpy(wl.dense_normal(A.Kc, N, seed=1, dtype=np.float32)).to(tdt)
    B[::7] *= 2.0 ** (-130 if dtype == "bf16" else -16)           # subnormal
    B[3, 0], B[50, N - 1], B[111, 5], B[200, N // 2] = float("inf"), -float("inf"), float("nan"), float("inf")
    val = torch.from_numpy(A.val.astype(np.float32)).to(tdt)
    rows = np.repeat(np.arange(A.M), np.diff(A.rowptr))
    D = np.zeros((A.M, A.Kc))
    D[rows, A.col] = val.double().numpy()
    Bd = B.double().numpy()
    want, scale = D @ np.where(np.isfinite(Bd), Bd, 0.0), np.abs(D) @ np.abs(np.where(np.isfinite(Bd), Bd, 0.0))
    with np.errstate(invalid="ignore"):
        for r, c in np.argwhere(~np.isfinite(Bd)):
            hit = D[:, r] != 0
            want[hit, c] += D[hit, r] * Bd[r, c]
    finite = np.isfinite(want)
    deg = np.diff(A.rowptr)
    limit = deg.max() * 2.0 ** -24                                # deg - 1 fp32 additions of exact products
    limit_abs = deg.max() * 2.0 ** -149                           # and of products below the normal range
    for opts in (dict(), dict(flags=lb.FLAG_NO_FILL_PADDING), dict(cs=40, ts=2), dict(flags=lb.FLAG_TWO_KERNELS, cs=40),
                 dict(mode=lb.MODE_SCALAR_ONLY), dict(mode=lb.MODE_DENSE_ONLY)):
        p = lb.Plan.from_csr(A, val=val.view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else val.numpy(),
                             val_dtype=lb.BF16 if dtype == "bf16" else None, **opts).upload()
        got = p.spmm(B.cuda()).double().cpu().numpy()
        np.testing.assert_array_equal(np.isnan(got), np.isnan(want), err_msg=str(opts))
        np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)], err_msg=str(opts))
        assert np.all(np.abs(got[finite] - want[finite]) <= (limit * scale + limit_abs)[finite]), opts
        p.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("N", [32, 64, 128, 224])
def test_every_kind_of_product_with_an_inf_or_nan(N, dtype):
    """Values of A of every kind (numbers of both signs, stored zeros, infinities, NaNs) against rows of B full of Inf, -Inf and
    NaN: each output is the sum of its own products and of no others."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    A = edge_windows(seed=7)
    rng = np.random.default_rng(8)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float16
    inf, nan = np.inf, np.nan
    for special_rows, special_values in ((0.02, 0.0), (0.02, 0.05), (1.0, 0.05)):
        b = wl.dense_normal(A.Kc, N, seed=1, dtype=np.float32)
        hit = (rng.random(A.Kc) < special_rows)[:, None] & (rng.random(b.shape) < 0.2)
        b[hit] = rng.choice([inf, -inf, nan], size=int(hit.sum()))
        v = A.val.astype(np.float32)
        hit = rng.random(v.size) < special_values
        v[hit] = rng.choice([0.0, -0.0, inf, -inf, nan], size=int(hit.sum()))
        B, val = torch.from_numpy(b).to(tdt), torch.from_numpy(v).to(tdt)
        Bn, vn = B.double().numpy(), val.double().numpy()
        want, scale = np.zeros((A.M, N)), np.zeros((A.M, N))
        with np.errstate(invalid="ignore"):
            for i in range(A.M):
                s, e = A.rowptr[i], A.rowptr[i + 1]
                products = vn[s:e, None] * Bn[A.col[s:e]]
                want[i], scale[i] = products.sum(axis=0), np.abs(products).sum(axis=0)
        finite = np.isfinite(want)
        limit = np.diff(A.rowptr).max() * 2.0 ** -24              # deg - 1 fp32 additions of exact products
        for opts in (dict(), dict(cs=40, ts=2), dict(flags=lb.FLAG_TWO_KERNELS, cs=40), dict(mode=lb.MODE_SCALAR_ONLY), dict(mode=lb.MODE_DENSE_ONLY)):
            p = lb.Plan.from_csr(A, val=val.view(torch.int16).numpy().view(np.uint16) if dtype == "bf16" else val.numpy(),
                                 val_dtype=lb.BF16 if dtype == "bf16" else None, **opts).upload()
            got = p.spmm(B.cuda()).double().cpu().numpy()
            np.testing.assert_array_equal(np.isnan(got), np.isnan(want), err_msg=str(opts))
            np.testing.assert_array_equal(got[np.isinf(want)], want[np.isinf(want)], err_msg=str(opts))
            assert np.all(np.abs(got[finite] - want[finite]) <= limit * scale[finite]), opts
            p.close()


@pytest.mark.parametrize("N", [32, 64, 128])
def test_operands_full_of_inf_cost_a_few_times_finite_ones(N):
    """An overflowed step of a mixed-precision training sends every task over its rows a second time.  Medians of 20 calls; measured
    3.0 / 3.5 / 4.4 times the finite call at N = 32 / 64 / 128, with sums formed one nonzero at a time 17.7 / 11.6 / 9.3 times."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    A = wl.rmat(scale=15, avg_degree=16, seed=3)
    p = lb.Plan.from_csr(A).upload()
    B = torch.from_numpy(wl.dense_normal(A.Kc, N, seed=1)).cuda()
    C = torch.empty((A.M, N), device="cuda")

    def median_us(operand):
        ev = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(25)]
        for start, end in ev:
            start.record()
            p.spmm(operand, out=C)
            end.record()
        torch.cuda.synchronize()
        return float(np.median([s.elapsed_time(e) for s, e in ev[5:]])) * 1e3

    usual, full = median_us(B), median_us(torch.full_like(B, float("inf")))
    print(f"N={N}: finite {usual:.1f} us, all Inf {full:.1f} us, ratio {full / usual:.2f}", flush=True)
    assert full <= 6.5 * usual
    p.close()
