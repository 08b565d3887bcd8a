"""The device planner (the paper's GPU preprocessing, Section 4.5) against the host planner: the exported
plans must be identical array by array, for every option the kernels' window shape allows.  The host planner
itself is checked against the reference planner in the CPU tests, so equality here carries that parity over."""
import time

import numpy as np
import pytest

from paper_2506_22714_amd import binding as lb
from paper_2506_22714_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lb.lib()


def dev_val(val, dtype_code):
    if dtype_code == lb.BF16:
        return torch.from_numpy(np.ascontiguousarray(val).view(np.int16)).cuda().view(torch.bfloat16)
    return torch.from_numpy(np.ascontiguousarray(val)).cuda()


def device_plan(A, val=None, val_dtype=None, **kw):
    v = A.val if val is None else val
    code = val_dtype if val_dtype is not None else (lb.F16 if v.dtype == np.float16 else lb.F32)
    return lb.Plan.from_device_csr(A.M, A.Kc, torch.from_numpy(A.rowptr.astype(np.int32)).cuda(),
                                   torch.from_numpy(A.col.astype(np.int32)).cuda(), dev_val(v, code), **kw)


TIMES = ("plan_seconds", "device_seconds")


def assert_same_plan(ph, pd, flags=0):
    sh, sd = ph.stats(), pd.stats()
    for k in sh:
        if k not in TIMES:
            assert sh[k] == sd[k], (k, sh[k], sd[k])
    assert sd["device_seconds"] > 0 and sh["device_seconds"] == 0
    for which in (0, 1):
        if flags & (lb.FLAG_NO_SPMM if which == 0 else lb.FLAG_NO_SDDMM):
            continue
        eh, ed = ph.export(which), pd.export(which)
        assert eh.keys() == ed.keys()
        for k in eh:
            assert np.array_equal(eh[k], ed[k]), (which, k)


CASES = [
    dict(),
    dict(spmm_min_vec_nnz=3, sddmm_min_blk_nnz=20, ts=2, cs=7, sddmm_cs=33, sddmm_ts=3),
    dict(spmm_min_vec_nnz=2, sddmm_min_blk_nnz=17, ts=1, cs=2, short_len=4),
    dict(mode=lb.MODE_DENSE_ONLY, ts=3, sddmm_ts=1),
    dict(mode=lb.MODE_SCALAR_ONLY, cs=5),
    dict(flags=lb.FLAG_NO_FILL_PADDING, ts=1, cs=3),
    dict(flags=lb.FLAG_NATURAL_ORDER, ts=2, cs=6),
    dict(flags=lb.FLAG_NO_SDDMM | lb.FLAG_XCD_ORDER, spmm_min_vec_nnz=1),
    dict(flags=lb.FLAG_NO_SPMM | lb.FLAG_NO_XCD_ORDER, sddmm_min_blk_nnz=64),
    dict(spmm_min_vec_nnz=16, sddmm_min_blk_nnz=200),
    dict(sddmm_min_blk_nnz=20, sddmm_min_dense_pct=30),
    dict(sddmm_min_blk_nnz=20, sddmm_min_dense_pct=85),
    dict(sddmm_min_blk_nnz=17, ts=2**31 - 1, cs=2**31 - 1, sddmm_cs=2**31 - 1, sddmm_ts=2**31 - 1),      # nothing is cut
    dict(mode=lb.MODE_DENSE_ONLY, sddmm_ts=2**31 - 2),
]


def matrices():
    yield "random", wl.random_pattern(203, 150, 0.08, seed=5, empty_rows=0.15)
    yield "community", wl.community(n_blocks=6, seed=2)
    yield "rmat", wl.rmat(scale=9, avg_degree=8, seed=3)
    yield "longrows", wl.with_long_rows(wl.random_pattern(90, 400, 0.03, seed=7), [3, 17, 18, 64], 300, seed=8)
    yield "single_row", wl.random_pattern(1, 50, 0.5, seed=9)
    yield "ragged_tail", wl.random_pattern(1000, 300, 0.03, seed=10, empty_rows=0.3)
    yield "dense_rows", wl.random_pattern(40, 700, 0.6, seed=11)          # windows with many blocks
    yield "leading_empty_windows", wl.with_long_rows(wl.random_pattern(100, 64, 0.0, seed=12), [70, 99], 40, seed=13)


@pytest.mark.parametrize("case", range(len(CASES)))
def test_device_planner_equals_host_planner(case):
    kw = CASES[case]
    for name, A in matrices():
        print("case", case, name, flush=True)
        ph = lb.Plan.from_csr(A, **kw)
        pd = device_plan(A, **kw)
        assert_same_plan(ph, pd, kw.get("flags", 0))
        ph.close()
        pd.close()


@pytest.mark.parametrize("case", range(len(CASES)))
def test_device_planner_equals_reference_planner(case):
    """The device-built plan against the reference planner written from the paper (not against the host planner, with
    which it shares the code that orders the task tables): same blocks, bitmaps, residual arrays, tasks, cleared rows."""
    from test_plan_host import check_subplan, ref_opts
    from oracle import planner_ref as pr
    kw = CASES[case]
    fl = kw.get("flags", 0)
    for name, A in matrices():
        if A.nnz > 20000:
            continue                    # the reference planner walks Python dictionaries
        print("case", case, name, flush=True)
        pd = device_plan(A, **kw)
        o = ref_opts(kw)
        if not fl & lb.FLAG_NO_SPMM:
            check_subplan(A, pd.export(0), pr.plan_spmm(A.M, A.rowptr, A.col, o), spmm=True)
        if not fl & lb.FLAG_NO_SDDMM:
            check_subplan(A, pd.export(1), pr.plan_sddmm(A.M, A.rowptr, A.col, o), spmm=False)
        pd.close()


def test_device_planner_random_options():
    rng = np.random.default_rng(20250622)
    for it in range(40):
        M, Kc = int(rng.integers(1, 400)), int(rng.integers(1, 500))
        A = wl.random_pattern(M, Kc, float(rng.uniform(0, 0.4)), seed=int(rng.integers(1 << 30)), empty_rows=0.2)
        if M > 3 and Kc > 30 and it % 2:
            A = wl.with_long_rows(A, [M // 2], min(Kc, 200), seed=it)
        kw = dict(mode=int(rng.integers(0, 3)), spmm_min_vec_nnz=int(rng.integers(1, 8)), sddmm_min_blk_nnz=int(rng.integers(1, 80)),
                  ts=int(rng.integers(1, 6)), cs=int(rng.integers(1, 40)), short_len=int(rng.integers(1, 5)),
                  sddmm_cs=int(rng.integers(1, 60)), sddmm_ts=int(rng.integers(1, 9)), flags=int(rng.choice([0, 1, 8, 9, 16, 32, 256, 288])),
                  sddmm_min_dense_pct=int(rng.choice([0, 0, 25, 60, 100])))
        print("random case", it, M, Kc, A.nnz, kw, flush=True)
        ph = lb.Plan.from_csr(A, **kw)
        pd = device_plan(A, **kw)
        assert_same_plan(ph, pd)
        ph.close()
        pd.close()


def test_device_planner_value_types_and_results():
    A = wl.make("powerlaw", small=True)
    # fp32 values: forced onto the scalar path, 4-byte values travel
    v32 = A.val.astype(np.float32) * 1.25
    assert_same_plan(lb.Plan.from_csr(A, val=v32), device_plan(A, val=v32))
    # bfloat16 bit patterns
    vb = wl.to_bf16_bits(np.linspace(-2, 2, A.nnz, dtype=np.float32) + 0.3)
    assert_same_plan(lb.Plan.from_csr(A, val=vb, val_dtype=lb.BF16), device_plan(A, val=vb, val_dtype=lb.BF16))
    # a device-built plan runs like a host-built one
    B = wl.dense_normal(A.Kc, 64, seed=3)
    ph = lb.Plan.from_csr(A).upload()
    pd = device_plan(A).upload()
    Bd = torch.from_numpy(B).cuda()
    Ch, Cd = ph.spmm(Bd), pd.spmm(Bd)
    one_writer = torch.ones(A.M, dtype=torch.bool, device="cuda")
    one_writer[torch.from_numpy(ph.export(0)["zero_rows"]).cuda().long()] = False
    assert torch.equal(Ch[one_writer], Cd[one_writer])
    assert torch.allclose(Ch, Cd, rtol=1e-4, atol=1e-3)


def _run_all(p, A, B, X, Y):
    """Every compute call on a ready plan; SpMM rows with several writers are returned separately."""
    C1 = p.spmm(B)
    out = torch.full((p.nnz,), float("nan"), dtype=torch.float32, device="cuda")
    p.sddmm(X, Y, out=out)
    alpha = p.edge_softmax(out, 0.25)
    p.set_values(alpha)
    C2 = p.spmm(B)
    out2 = p.sddmm(X, Y)
    torch.cuda.synchronize()
    return C1, out, alpha, C2, out2


@pytest.mark.parametrize("keep_host_copy", [True, False])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_resident_device_plan_computes_like_an_uploaded_host_plan(dtype, keep_host_copy):
    """The plan's device copy written by the planner itself (no host round trip) against libra_plan + libra_plan_upload."""
    A = wl.make("powerlaw", small=True)
    N, K = 64, 32
    if dtype == "f32":
        val, code, tdt = A.val.astype(np.float32) * 0.75, lb.F32, torch.float32
        mk = lambda r, c, seed: torch.from_numpy(wl.dense_normal(r, c, seed=seed, dtype=np.float32)).cuda()
    elif dtype == "bf16":
        val, code, tdt = wl.to_bf16_bits(A.val.astype(np.float32) * 0.75), lb.BF16, torch.bfloat16
        mk = lambda r, c, seed: torch.from_numpy(wl.dense_normal(r, c, seed=seed, dtype=np.float32)).cuda().to(torch.bfloat16)
    else:
        val, code, tdt = A.val, lb.F16, torch.float16
        mk = lambda r, c, seed: torch.from_numpy(wl.dense_normal(r, c, seed=seed)).cuda()
    B, X, Y = mk(A.Kc, N, 1), mk(A.M, K, 2), mk(A.Kc, K, 3)
    kw = dict(cs=40, ts=2)
    ph = lb.Plan.from_csr(A, val=val, val_dtype=code, **kw).upload()
    pd = lb.Plan.from_device_csr(A.M, A.Kc, torch.from_numpy(A.rowptr.astype(np.int32)).cuda(), torch.from_numpy(A.col.astype(np.int32)).cuda(),
                                 dev_val(val, code), resident=True, keep_host_copy=keep_host_copy, **kw)
    assert lb.libra_plan_device_bytes(pd.handle) == lb.libra_plan_device_bytes(ph.handle) <= pd._buf.numel()
    if keep_host_copy:
        assert_same_plan(ph, pd)
    else:
        for call in (lambda: pd.export(0), lambda: pd.upload()):
            with pytest.raises(lb.LibraError) as e:
                call()
            assert e.value.code == lb.ERR["NOT_BUILT"]
        sh, sd = ph.stats(), pd.stats()
        assert all(sh[k] == sd[k] for k in sh if k not in TIMES)
    one_writer = torch.ones(A.M, dtype=torch.bool, device="cuda")
    one_writer[torch.from_numpy(ph.export(0)["zero_rows"]).cuda().long()] = False
    assert 0 < int(one_writer.sum()) < A.M
    rh, rd = _run_all(ph, A, B, X, Y), _run_all(pd, A, B, X, Y)
    for k in (1, 2, 4):                                     # SDDMM, softmax: one writer per output
        assert torch.equal(rh[k], rd[k]), k
    for k in (0, 3):
        assert torch.equal(rh[k][one_writer], rd[k][one_writer]), k
        assert torch.allclose(rh[k], rd[k], rtol=1e-3, atol=1e-3), k


def test_device_planner_rejects_what_the_host_planner_rejects():
    A = wl.random_pattern(64, 64, 0.2, seed=3)
    rp = torch.from_numpy(A.rowptr.astype(np.int32)).cuda()
    col = torch.from_numpy(A.col.astype(np.int32)).cuda()
    val = torch.from_numpy(A.val).cuda()

    def rc(M=A.M, Kc=A.Kc, rowptr=rp, c=col, **kw):
        try:
            lb.Plan.from_device_csr(M, Kc, rowptr, c, val, **kw).close()
            return 0
        except lb.LibraError as e:
            return e.code

    assert rc() == 0
    bad = col.clone(); bad[5] = A.Kc
    assert rc(c=bad) == lb.ERR["COLUMN"]
    bad = col.clone(); bad[3] = -1
    assert rc(c=bad) == lb.ERR["COLUMN"]
    s, e = int(A.rowptr[10]), int(A.rowptr[11])
    assert e - s >= 2
    bad = col.clone(); bad[s + 1] = bad[s]
    assert rc(c=bad) == lb.ERR["UNSORTED"]
    badrp = rp.clone(); badrp[7] = badrp[8] + 1
    assert rc(rowptr=badrp) == lb.ERR["ROWPTR"]
    assert rc(window_rows=8) == lb.ERR["UNSUPPORTED"]
    assert rc(mode=7) == lb.ERR["OPTION"]
    # a matrix without nonzeros
    z = torch.zeros(9, dtype=torch.int32, device="cuda")
    p = lb.Plan.from_device_csr(8, 5, z, col[:0], val[:0])
    assert p.stats()["nnz"] == 0 and p.stats()["spmm_tasks"] == 1
    p.close()


@pytest.mark.parametrize("name", ["powerlaw", "community", "gat", "irregular"])
def test_device_planner_full_configs(name):
    A = wl.make(name)
    t0 = time.perf_counter()
    ph = lb.Plan.from_csr(A)
    t_host = time.perf_counter() - t0
    rp, col, val = (torch.from_numpy(x).cuda() for x in (A.rowptr.astype(np.int32), A.col.astype(np.int32), A.val))
    lb.Plan.from_device_csr(A.M, A.Kc, rp, col, val).close()           # warm-up (module load, allocator)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    pd = lb.Plan.from_device_csr(A.M, A.Kc, rp, col, val)
    t_dev = time.perf_counter() - t0
    print(f"{name}: host planner {t_host:.3f} s, device planner {t_dev:.3f} s "
          f"(device passes {pd.stats()['device_seconds']:.4f} s)", flush=True)
    assert_same_plan(ph, pd)
    # plan + device copy: host planner + upload against the resident device plan without a host copy
    t0 = time.perf_counter()
    ph.upload()
    torch.cuda.synchronize()
    t_up = time.perf_counter() - t0
    lb.Plan.from_device_csr(A.M, A.Kc, rp, col, val, resident=True, keep_host_copy=False).close()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    pr = lb.Plan.from_device_csr(A.M, A.Kc, rp, col, val, resident=True, keep_host_copy=False)
    torch.cuda.synchronize()
    t_res = time.perf_counter() - t0
    print(f"{name}: ready to compute: host plan + upload {t_host + t_up:.3f} s, resident device plan {t_res:.4f} s", flush=True)
    B = torch.from_numpy(wl.dense_normal(A.Kc, 32, seed=5)).cuda()
    one_writer = torch.ones(A.M, dtype=torch.bool, device="cuda")
    one_writer[torch.from_numpy(ph.export(0)["zero_rows"]).cuda().long()] = False
    assert torch.equal(ph.spmm(B)[one_writer], pr.spmm(B)[one_writer])


ORDER_CASES = [
    dict(cs=8, sddmm_cs=8),                                                        # segments by column
    dict(cs=8, sddmm_cs=8, ts=2, spmm_min_vec_nnz=2, sddmm_min_blk_nnz=17, sddmm_ts=1),
    dict(cs=8, sddmm_cs=8, flags=lb.FLAG_XCD_ORDER, sddmm_min_blk_nnz=17, sddmm_ts=1),
    dict(cs=8, sddmm_cs=8, flags=lb.FLAG_NO_XCD_ORDER),
    dict(cs=8, sddmm_cs=8, flags=lb.FLAG_SEGMENTS_BY_COST),
    dict(cs=8, sddmm_cs=8, flags=lb.FLAG_NATURAL_ORDER),
    dict(cs=4, ts=1, flags=lb.FLAG_NO_SDDMM),
    dict(sddmm_cs=4, flags=lb.FLAG_NO_SPMM | lb.FLAG_XCD_ORDER),
    dict(mode=lb.MODE_SCALAR_ONLY, cs=1, sddmm_cs=1),
]


@pytest.mark.parametrize("name", ["rmat", "community", "short_rows", "hub_windows"])
def test_large_task_tables_are_ordered_like_on_the_host(name):
    """Tables of more than 8192 tasks are ordered on the GPU: the same tables as the host's, and a plan whose records never
    were on the host computes what an uploaded one does."""
    A = {"rmat": lambda: wl.rmat(scale=13, avg_degree=16, seed=3),
         "community": lambda: wl.community(n_blocks=500, seed=2),                  # the die-aware order fires
         "short_rows": lambda: wl.random_pattern(140_003, 300, 0.004, seed=4, empty_rows=0.3),   # no segments
         # windows whose rows are all decomposed: empty tasks of cost 0 at the table's end
         "hub_windows": lambda: wl.with_long_rows(wl.random_pattern(20_000, 2000, 0.003, seed=7), list(range(64, 96)) + [7], 1500, seed=8)}[name]()
    B = torch.from_numpy(wl.dense_small_int(A.Kc, 32, seed=1)).cuda()
    X = torch.from_numpy(wl.dense_small_int(A.M, 32, seed=2)).cuda()
    ones = np.ones(A.nnz, dtype=np.float16)          # whole numbers: every order of additions gives the same sums
    for kw in ORDER_CASES:
        print(name, A.nnz, kw, flush=True)
        fl = kw.get("flags", 0)
        ph, pd = lb.Plan.from_csr(A, val=ones, **kw), device_plan(A, val=ones, **kw)
        assert ph.stats()["spmm_tasks"] + ph.stats()["sddmm_tasks"] > 8192 + 100      # beside the few empty tasks of the die-aware order
        assert_same_plan(ph, pd, fl)
        pd.close()
        ph.upload()
        pr = device_plan(A, val=ones, resident=True, keep_host_copy=False, **kw)
        sh, sr = ph.stats(), pr.stats()
        assert all(sh[k] == sr[k] for k in sh if k not in TIMES)
        if not fl & lb.FLAG_NO_SPMM:
            assert torch.equal(ph.spmm(B), pr.spmm(B))
        if not fl & lb.FLAG_NO_SDDMM:
            assert torch.equal(ph.sddmm(X, B), pr.sddmm(X, B))
        ph.close()
        pr.close()


@pytest.mark.parametrize("sddmm_cs", [2**31 - 1, 2**31 - 2, 2**30, 204_356, 204_355])
def test_segments_longer_than_the_residual_list(sddmm_cs):
    """sddmm_cs may be anything up to 2^31 - 1 ("do not cut"): one segment, or two, over the whole residual list, in a table
    ordered on the GPU and (small matrix, two or three residual nonzeros) in one ordered on the host."""
    A = wl.rmat(scale=13, avg_degree=16, seed=3)
    assert A.nnz == 204_356
    ones = np.ones(A.nnz, dtype=np.float16)
    kw = dict(mode=lb.MODE_SCALAR_ONLY, cs=8, sddmm_cs=sddmm_cs)
    ph, pd = lb.Plan.from_csr(A, val=ones, **kw), device_plan(A, val=ones, **kw)
    assert ph.stats()["spmm_tasks"] > 8192 and ph.stats()["sddmm_tasks"] == 1 + (sddmm_cs < A.nnz)
    assert_same_plan(ph, pd)
    pd.close()
    ph.upload()
    pr = device_plan(A, val=ones, resident=True, keep_host_copy=False, **kw)
    X, Y = (torch.from_numpy(wl.dense_small_int(n, 32, seed=k)).cuda() for k, n in ((1, A.M), (2, A.Kc)))
    out = torch.full((A.nnz,), float("nan"), device="cuda")
    pr.sddmm(X, Y, out=out)
    assert torch.equal(out, ph.sddmm(X, Y))
    ph.close()
    pr.close()
    for nnz in (1, 2, 3, 4):
        S = wl.Csr(5, 9, np.minimum(np.arange(6), nnz).astype(np.int32), np.arange(nnz, dtype=np.int32), ones[:nnz])
        ph, pd = lb.Plan.from_csr(S, **kw), device_plan(S, **kw)
        assert_same_plan(ph, pd)
        ph.close()
        pd.close()


def test_rows_of_large_matrices_are_checked_and_listed_on_the_device():
    """From 2^17 rows on rowptr stays on the GPU (plans without a host copy): the row classes of the edge softmax at their edges
    (64, 65, 2048, 2049 nonzeros) against the host-planned result, and a broken rowptr is refused."""
    M, Kc = (1 << 17) + 3, 4096
    A = wl.random_pattern(M, 64, 0.03, seed=4, empty_rows=0.3)
    A = wl.Csr(M, Kc, A.rowptr, A.col, A.val)
    for k, n in enumerate((64, 65, 2048, 2049, 2600)):
        A = wl.with_long_rows(A, [0 if n == 2600 else 100 * k + 7, 70_000 + k, M - 1 - k], n, seed=k)
    ones = np.ones(A.nnz, dtype=np.float16)
    ph, pd = lb.Plan.from_csr(A, val=ones).upload(), device_plan(A, val=ones, resident=True, keep_host_copy=False)
    scores = torch.randn(A.nnz, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    ah, ad = ph.edge_softmax(scores, 0.5, out=torch.empty_like(scores)), pd.edge_softmax(scores, 0.5, out=torch.full_like(scores, float("nan")))
    assert torch.equal(ah, ad)
    dalpha = torch.randn(A.nnz, device="cuda", generator=torch.Generator("cuda").manual_seed(2))
    assert torch.equal(ph.edge_softmax_backward(ah, dalpha, 0.5), pd.edge_softmax_backward(ad, dalpha, 0.5))
    ph.close()
    pd.close()
    col, val = torch.from_numpy(A.col.astype(np.int32)).cuda(), torch.from_numpy(ones).cuda()
    for at, by in ((0, 1), (M // 2, 100_000), (M, -1)):
        rowptr = A.rowptr.astype(np.int32).copy()
        rowptr[at] += by
        with pytest.raises(lb.LibraError) as e:
            lb.Plan.from_device_csr(M, Kc, torch.from_numpy(rowptr).cuda(), col, val, resident=True, keep_host_copy=False)
        assert e.value.code == lb.ERR["ROWPTR"]


@pytest.mark.parametrize("flags", [lb.FLAG_NO_SPMM, lb.FLAG_NO_SDDMM, 0])
def test_rows_listed_on_the_device_beside_tables_ordered_on_the_host(flags):
    """Without the SpMM tables a matrix of 2^17 rows may have few tasks: the list of rows of 65 .. 2048 nonzeros, which is in device
    memory, then lies in the plan between arrays that come from the host.  Every list from none to some thousand rows arrives whole."""
    M, Kc = (1 << 17) + 3, 4096
    for medium in (0, 1, 3, 200, 1500):
        for longest in (64, 2500):
            counts = np.zeros(M, dtype=np.int64)
            counts[::64] = 1 + np.arange(counts[::64].size) % 40
            counts[5:5 + 80 * medium:80] = 65 + np.arange(medium) % 60
            counts[[17, M - 2]] = longest
            rowptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
            col = (np.arange(rowptr[-1]) - np.repeat(rowptr[:-1], counts)).astype(np.int32)
            A = wl.Csr(M, Kc, rowptr, col, np.ones(col.size, dtype=np.float16))
            pd = device_plan(A, resident=True, keep_host_copy=False, flags=flags)
            if flags == lb.FLAG_NO_SPMM:
                assert 0 < pd.stats()["sddmm_tasks"] < 8192
            g = torch.Generator("cuda").manual_seed(1)
            scores, dalpha = torch.randn(A.nnz, device="cuda", generator=g), torch.randn(A.nnz, device="cuda", generator=g)
            ph = lb.Plan.from_csr(A, flags=flags).upload()
            nan = lambda: torch.full_like(scores, float("nan"))
            ah, ad = ph.edge_softmax(scores, 0.5, out=nan()), pd.edge_softmax(scores, 0.5, out=nan())
            assert not ah.isnan().any() and torch.equal(ah, ad), (medium, longest)
            assert torch.equal(ph.edge_softmax_backward(ah, dalpha, 0.5, out=nan()), pd.edge_softmax_backward(ah, dalpha, 0.5, out=nan()))
            ph.close()
            pd.close()


@pytest.mark.parametrize("M,flags", [((1 << 27) + 1605, 0), ((1 << 30) + 37, lb.FLAG_NO_SPMM)])
def test_more_windows_than_one_launch_has_waves(M, flags):
    """A wave writes the tasks of a window; with more than 2^23 windows a wave takes several, and 2^30 rows at a wave per window
    would be more threads than a launch can have.  A few rows with nonzeros among many empty ones, the last row among them."""
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs some 40 GiB")
    nw = (M + 15) // 16
    rows = np.unique(np.array([0, 5, 16 * 70, (1 << 27) - 1, 1 << 27, (1 << 27) + 1600, M // 2, M - 18, M - 1]))
    rows = rows[rows < M]
    per_row = 20
    rowptr = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    for r in rows.tolist():
        rowptr[r + 1:] += per_row
    col = torch.arange(per_row, dtype=torch.int32, device="cuda").repeat(rows.size) * 3
    val = torch.ones(col.numel(), dtype=torch.float16, device="cuda")
    p = lb.Plan.from_device_csr(M, 64, rowptr, col, val, flags=flags | lb.FLAG_NATURAL_ORDER, sddmm_min_blk_nnz=16, sddmm_ts=1)
    windows = np.unique(rows // 16)
    tasks = p.export(1)["tasks"]                # blocks of 16 columns, the rest residual
    dense = tasks[tasks["kind"] == lb.TASK_WINDOW]
    assert np.array_equal(np.unique(dense["id"]), windows)
    st = p.stats()
    assert st["n_windows"] == nw and st["sddmm_dense_nnz"] + st["sddmm_res_nnz"] == st["nnz"] == per_row * rows.size
    if not flags & lb.FLAG_NO_SPMM:
        tasks = p.export(0)["tasks"]
        assert np.array_equal(tasks["id"], np.arange(nw))
        assert np.all(tasks["store_mask"][:-1] == 0xffff) and tasks["store_mask"][-1] == (1 << (M - 16 * (nw - 1))) - 1
        assert np.array_equal(np.flatnonzero(tasks["res_end"] > tasks["res_begin"]), windows)
    p.close()


@pytest.mark.parametrize("M", [(1 << 13) + 8, 1 << 14])
def test_plans_of_very_many_nonzeros(M):
    """Places of nonzeros are 32-bit numbers: more than 2^30 of them, of which two no longer add up in 32 bits, and 100
    fewer than 2^31, where the last tile of the census has places past the last one.  A full matrix, the last row short: every nonzero lies
    in a dense block and no row has a residual one."""
    Kc = 1 << 17
    nnz = M * Kc - 100
    o = lb.PlanOpts(flags=lb.FLAG_NO_SDDMM)
    ws_bytes, plan_bytes = lb.libra_plan_device_workspace(M, nnz, o), 8 * nnz
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < ws_bytes + plan_bytes + 6 * nnz + (3 << 30):
        pytest.skip("needs some 110 bytes of GPU memory per nonzero")
    rowptr = (torch.arange(M + 1, device="cuda") * Kc).clamp_(max=nnz).int()
    col = torch.arange(Kc, dtype=torch.int32, device="cuda").repeat(M)[:nnz]
    val = torch.zeros(nnz, dtype=torch.float16, device="cuda")
    ws, buf = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (ws_bytes, plan_bytes))
    handle = lb.libra_plan_device(M, Kc, nnz, rowptr.data_ptr(), col.data_ptr(), val.data_ptr(), lb.F16, o, ws.data_ptr(), ws_bytes,
                                  buf.data_ptr(), plan_bytes, False, torch.cuda.current_stream().cuda_stream)
    st = lb.libra_plan_stats(handle)
    lb.libra_plan_destroy(handle)
    del rowptr, col, val, ws, buf
    torch.cuda.empty_cache()
    windows = (M + 15) // 16
    assert st["n_vectors"] == st["spmm_dense_vectors"] == windows * Kc and st["n_vectors_nnz1"] == 0
    assert st["spmm_dense_nnz"] == nnz and st["spmm_blocks"] == windows * Kc // 16
    assert st["spmm_res_nnz"] == st["spmm_short_rows"] == st["spmm_long_rows"] == st["spmm_split_rows"] == 0


def test_sddmm_of_nearly_the_most_nonzeros():
    """The last window's output records lie next to 2^31, where a wave's next 256 of them do not count in 32 bits with a sign."""
    M, Kc, K = 1 << 14, 1 << 17, 32
    nnz = M * Kc - 66
    o = lb.PlanOpts(flags=lb.FLAG_NO_SPMM)
    ws_bytes, plan_bytes = lb.libra_plan_device_workspace(M, nnz, o), 13 * nnz
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < ws_bytes + plan_bytes + 6 * nnz + (3 << 30):
        pytest.skip("needs some 230 GiB")
    rowptr = (torch.arange(M + 1, device="cuda") * Kc).clamp_(max=nnz).int()
    col = torch.arange(Kc, dtype=torch.int32, device="cuda").repeat(M)[:nnz]
    val = torch.zeros(nnz, dtype=torch.float16, device="cuda")
    ws, buf = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (ws_bytes, plan_bytes))
    stream = torch.cuda.current_stream().cuda_stream
    handle = lb.libra_plan_device(M, Kc, nnz, rowptr.data_ptr(), col.data_ptr(), val.data_ptr(), lb.F16, o, ws.data_ptr(), ws_bytes,
                                  buf.data_ptr(), plan_bytes, False, stream)
    del rowptr, col, val, ws
    torch.cuda.empty_cache()
    assert lb.libra_plan_stats(handle)["sddmm_dense_nnz"] == nnz
    g = torch.Generator("cuda").manual_seed(1)
    X, Y = (torch.randint(-3, 4, (n, K), device="cuda", generator=g).half() for n in (M, Kc))
    out = torch.full((M * Kc,), float("nan"), device="cuda")
    lb.libra_sddmm_pattern(handle, X.data_ptr(), Y.data_ptr(), K, out.data_ptr(), stream)
    assert bool(out[nnz:].isnan().all())
    out = out.view(M, Kc)
    Yt = Y.float().T.contiguous()
    for r in range(0, M, 1024):
        want = X[r:r + 1024].float() @ Yt
        same = out[r:r + 1024] == want
        if r + 1024 == M:
            same[-1, Kc - 66:] = True
        assert bool(same.all()), r
    lb.libra_plan_destroy(handle)
    del out, buf, want, same
    torch.cuda.empty_cache()


@pytest.mark.parametrize("flags", [lb.FLAG_XCD_ORDER, lb.FLAG_NATURAL_ORDER])
def test_more_tasks_than_one_launch_has_waves(flags):
    """A launch has fewer than 2^32 threads, i.e. 2^26 waves with a task each: tables of more tasks (segments of one nonzero) take
    several launches.  Values and operands are whole numbers, so every order of additions gives the same sums."""
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs some 60 GiB")
    M, deg, N = (1 << 20) + 5, 65, 32
    nnz = M * deg
    assert nnz > 1 << 26
    rowptr = torch.arange(M + 1, dtype=torch.int32, device="cuda") * deg
    first = torch.arange(M, dtype=torch.int32, device="cuda") % 128                # row i: 65 consecutive columns
    col = (first[:, None] + torch.arange(deg, dtype=torch.int32, device="cuda")).reshape(-1)
    val = torch.ones(nnz, dtype=torch.float16, device="cuda")
    p = lb.Plan.from_device_csr(M, 192, rowptr, col, val, resident=True, keep_host_copy=False, mode=lb.MODE_SCALAR_ONLY, cs=1, sddmm_cs=1,
                                flags=flags, ts=1 << 20, sddmm_ts=1 << 20)
    st = p.stats()
    assert st["spmm_tasks"] > 1 << 26 and st["sddmm_tasks"] > 1 << 26
    gen = torch.Generator("cuda").manual_seed(1)
    B = torch.randint(-3, 4, (192, N), device="cuda", generator=gen).half()
    X = torch.randint(-3, 4, (M, N), device="cuda", generator=gen).half()
    C = torch.full((M, N), float("nan"), device="cuda")
    p.spmm(B, out=C)
    sums = torch.cat([torch.zeros((1, N), device="cuda"), B.float().cumsum(0)])
    f = first.long()
    assert torch.equal(C, sums[f + deg] - sums[f])
    out = torch.full((nnz,), float("nan"), device="cuda")
    p.sddmm(X, B, out=out)
    want = (X.float() @ B.float().T).gather(1, col.reshape(M, deg).long())
    assert torch.equal(out.reshape(M, deg), want)
    p.close()
