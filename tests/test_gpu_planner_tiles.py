"""The device planner's census sorts the nonzeros a tile at a time: the host planner's plan at the edges of tiles - windows that span
many tiles, tiles of thousands of nearly empty windows, sizes around whole tiles, vectors where a tile ends, the widest columns."""
import numpy as np
import pytest

from paper_2506_22714_amd import binding as lb
from paper_2506_22714_amd import workloads as wl
from test_gpu_planner import assert_same_plan, device_plan

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

STEP = 256 * 7 - 16         # places between the boundaries of two tiles

OPTIONS = [dict(), dict(spmm_min_vec_nnz=2, sddmm_min_blk_nnz=17, ts=2, cs=9), dict(mode=lb.MODE_DENSE_ONLY), dict(mode=lb.MODE_SCALAR_ONLY, cs=50),
           dict(sddmm_min_blk_nnz=20, sddmm_min_dense_pct=60)]


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def csr(M, Kc, rows, cols):
    keys = np.unique(rows.astype(np.int64) * Kc + cols.astype(np.int64))
    rowptr = np.zeros(M + 1, dtype=np.int32)
    np.cumsum(np.bincount(keys // Kc, minlength=M), out=rowptr[1:])
    return wl.Csr(M, Kc, rowptr, (keys % Kc).astype(np.int32), np.arange(1, keys.size + 1).astype(np.float16))


def spread(M, Kc, n, seed, rows=None):
    """n distinct places, in the given rows if there are any."""
    rng = np.random.default_rng(seed)
    rows = np.arange(M) if rows is None else np.asarray(rows)
    at = rng.choice(rows.size * Kc, size=n, replace=False)
    return csr(M, Kc, rows[at // Kc], at % Kc)


def cases():
    yield "one full window", csr(16, 700, *map(np.ravel, np.indices((16, 700))))                     # 16 of a column wherever a tile ends
    yield "fifteen full rows", csr(31, 900, *map(np.ravel, np.indices((15, 900))))
    for n in (1, STEP - 1, STEP, STEP + 1, 2 * STEP + 15, 256 * 7, 256 * 7 + 1):
        yield f"{n} places", spread(100, 90, n, n)
    yield "one row", spread(40, 9000, 4 * STEP + 3, 1, rows=[21])
    yield "two rows of a window", spread(40, 9000, 3 * STEP, 2, rows=[32, 39])
    # a nonzero or none per window: a tile of some 1,800 windows, more of them if most are empty
    rng = np.random.default_rng(3)
    M = 16 * 5000
    yield "one per window", csr(M, 60, np.arange(5000) * 16 + rng.integers(0, 16, 5000), rng.integers(0, 60, 5000))
    yield "mostly empty", csr(16 * 40_000, 60, rng.choice(16 * 40_000, 4000, replace=False), rng.integers(0, 60, 4000))
    # hub windows between sparse ones, sharing columns
    r = np.concatenate([np.repeat(np.arange(1600), 3), np.full(5000, 805), np.full(4000, 806), np.full(3000, 3)])
    yield "hubs", csr(1600, 12_000, r, np.concatenate([rng.integers(0, 12_000, 4800), rng.choice(12_000, 5000, replace=False),
                                                       rng.choice(12_000, 4000, replace=False), rng.choice(12_000, 3000, replace=False)]))
    # columns of 31 bits
    wide = 2**31 - 1
    c = np.concatenate([rng.integers(0, wide, 3000), np.repeat(rng.integers(0, wide, 200), 8), [0, wide - 1, wide - 1, wide - 2]])
    yield "wide", csr(300, wide, np.concatenate([rng.integers(0, 300, 3000), np.tile(np.arange(64, 72), 200), [5, 5, 6, 6]]), c)


@pytest.mark.parametrize("name,A", list(cases()), ids=lambda x: x if isinstance(x, str) else "")
def test_tile_edges(name, A):
    for kw in OPTIONS:
        ph, pd = lb.Plan.from_csr(A, **kw), device_plan(A, **kw)
        assert_same_plan(ph, pd)
        ph.close()
        pd.close()


@pytest.mark.parametrize("at", [0, STEP - 1, STEP, 5 * STEP + 7, -1])
def test_bad_columns_are_refused_wherever_they_lie(at):
    """Unsorted rows and columns out of range, in the first, an inner and the last tile."""
    A = spread(500, 400, 6 * STEP, 5)
    for what, code in (("range", "COLUMN"), ("negative", "COLUMN"), ("unsorted", "UNSORTED")):
        col = A.col.copy()
        p = at % A.nnz
        if what == "unsorted":                  # a row of at least two holds the place
            row = np.searchsorted(A.rowptr, p, side="right") - 1
            assert A.rowptr[row + 1] - A.rowptr[row] >= 2
            p = max(p, A.rowptr[row] + 1)
            col[p] = col[p - 1]
        else:
            col[p] = A.Kc if what == "range" else -5
        with pytest.raises(lb.LibraError) as e:
            device_plan(wl.Csr(A.M, A.Kc, A.rowptr, col, A.val))
        assert e.value.code in (lb.ERR[code], lb.ERR["COLUMN"])


MARKED = 1 << 15            # rows that the 2048 nonzeros of a chunk span before each of them is searched for


@pytest.mark.parametrize("span", [MARKED - 1, MARKED, MARKED + 1, 5 * MARKED + 77])
@pytest.mark.parametrize("at", [1, 1024, 2047])
def test_rows_of_nonzeros_far_apart(span, at):
    """A chunk with `at` nonzeros (one and three a row in turn) before a run of empty rows and the rest behind it, whole chunks before and
    after, empty rows at both ends of the matrix."""
    M = 1000 + span + 9000
    counts = np.zeros(M, dtype=np.int64)
    left, row = 2048 + at, 1000
    while left > 0:
        counts[row] = min(left, 1 + row % 2 * 2)
        left, row = left - counts[row], row + 1
    first = int(np.searchsorted(np.cumsum(counts), 2048, side="right"))         # the row of nonzero 2048
    counts[first + span:first + span + 3000] = 2
    rows = np.repeat(np.arange(M), counts)
    assert rows[2048] == first and rows[2048 + at] == first + span
    A = csr(M, 500, rows, np.concatenate([np.arange(c) * 7 + i % 400 for i, c in enumerate(counts) if c]))
    assert A.nnz == rows.size
    for opts in (dict(), dict(flags=lb.FLAG_NO_SPMM, sddmm_min_blk_nnz=17)):
        ph, pd = lb.Plan.from_csr(A, **opts), device_plan(A, **opts)
        assert_same_plan(ph, pd, opts.get("flags", 0))
        ph.close()
        pd.close()


def test_runs_of_empty_rows_take_no_more_time_than_empty_rows_everywhere():
    """6,000 rows of 33 nonzeros among 2^26, at both ends or evenly: a workgroup that walked the run alone took 100 ms."""
    M, n, per = 1 << 26, 6000, 33
    times = []
    for rows in (np.r_[0:n // 2, M - n // 2:M], np.arange(n) * (M // n)):
        counts = torch.zeros(M, dtype=torch.int32, device="cuda")
        counts[torch.from_numpy(rows).cuda()] = per
        rowptr = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
        rowptr[1:] = torch.cumsum(counts, 0)
        col = (torch.arange(per, device="cuda") * 100).int().repeat(n)
        val = torch.ones(col.numel(), dtype=torch.float16, device="cuda")
        best = 1e9
        for _ in range(4):
            p = lb.Plan.from_device_csr(M, 4096, rowptr, col, val, resident=True, keep_host_copy=False, flags=lb.FLAG_NO_SPMM)
            best = min(best, p.stats()["plan_seconds"])
            p.close()
        times.append(best)
    assert times[0] < 4 * times[1], times


@pytest.mark.parametrize("M,Kc,share", [(16, 200_000, 0.6), (40, 130_003, 0.9), (33, 2_000_000, 0.07)])
def test_windows_of_more_than_a_thousand_tiles(M, Kc, share):
    """Whole groups of tiles, and parts of them, between a tile and the first one of its window."""
    rng = np.random.default_rng(M)
    n = [min(Kc, int(Kc * share * s)) for s in rng.uniform(0.8, 1.2, M)]
    rows, cols = np.repeat(np.arange(M), n), np.concatenate([rng.choice(Kc, k, replace=False) for k in n])
    with np.errstate(over="ignore"):            # the later values are infinities
        A = csr(M, Kc, rows, cols)
    assert np.diff(A.rowptr[::16]).max(initial=A.rowptr[16]) >= 4 * 256 * STEP
    ph, pd = lb.Plan.from_csr(A, spmm_min_vec_nnz=3, sddmm_min_blk_nnz=40), device_plan(A, spmm_min_vec_nnz=3, sddmm_min_blk_nnz=40)
    assert_same_plan(ph, pd)
    ph.close()
    pd.close()


def test_a_window_of_all_nonzeros_takes_no_more_time_than_many_windows():
    """2^28 nonzeros in one window or in 1,024: with a sum over all earlier tiles in every tile the first took three times as long."""
    times = []
    for M in (1 << 4, 1 << 14):
        Kc = (1 << 28) // M
        rowptr = torch.arange(M + 1, dtype=torch.int32, device="cuda") * Kc
        col = torch.arange(Kc, dtype=torch.int32, device="cuda").repeat(M)
        val = torch.zeros(M * Kc, dtype=torch.float16, device="cuda")
        best = 1e9
        for _ in range(4):
            p = lb.Plan.from_device_csr(M, Kc, rowptr, col, val, resident=True, keep_host_copy=False, flags=lb.FLAG_NO_SDDMM)
            best = min(best, p.stats()["plan_seconds"])
            p.close()
        times.append(best)
    assert times[0] < 2 * times[1], times
