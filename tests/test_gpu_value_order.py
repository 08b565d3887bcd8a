"""Values that come in another order of the nonzeros: the plan's contents, and so every product, are those of set_values with the
permuted values.  Whole numbers make every sum exact in any order, so the comparison is bit for bit."""
import numpy as np
import pytest

from paper_2506_22714_amd import binding as lb

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}
PASSES_MIN = (5 << 20) // 2         # from this many 16-bit nonzeros on the values are permuted in two passes (fp32: half as many)


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def random_csr(M, Kc, nnz, seed, clustered):
    """nnz distinct places; clustered: most of them in few columns of each window, so that both paths hold many."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    keys = torch.zeros(0, dtype=torch.int64, device="cuda")
    while keys.numel() < nnz:
        r = torch.randint(M, (nnz,), device="cuda", generator=g)
        c = torch.randint(Kc, (nnz,), device="cuda", generator=g)
        if clustered:
            c = torch.where(torch.rand(nnz, device="cuda", generator=g) < 0.7, (r // 16 * 37 + c % 64) % Kc, c)
        keys = torch.unique(torch.cat([keys, r * Kc + c]))
    keys = keys[torch.randperm(keys.numel(), device="cuda", generator=g)[:nnz]].sort().values
    rowptr = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(keys // Kc, minlength=M), 0)
    return rowptr, (keys % Kc).int()


def values(n, dt, seed):
    return torch.randint(-4, 5, (n,), device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed)).to(dt)


@pytest.mark.parametrize("dtype", list(DTYPES))
@pytest.mark.parametrize("nnz", [1, 7, 1000, PASSES_MIN - 1, PASSES_MIN, PASSES_MIN + 32768 * 3 + 5])
def test_ordered_values_are_permuted_values(nnz, dtype):
    dt = DTYPES[dtype]
    nnz = nnz - PASSES_MIN // 2 if dtype == "f32" and nnz > 1000 else nnz
    M, Kc = (40, 50) if nnz < 1000 else (301, 203) if nnz == 1000 else (40_003, 30_011)
    B = values(Kc * 32, dt, 5).view(Kc, 32)
    for opts, clustered in ((dict(), True), (dict(mode=lb.MODE_SCALAR_ONLY), False), (dict(mode=lb.MODE_DENSE_ONLY), True)):
        rowptr, col = random_csr(M, Kc, nnz, nnz, clustered)
        p = lb.Plan.from_device_csr(M, Kc, rowptr, col, values(nnz, dt, 1), resident=True, keep_host_copy=False, flags=lb.FLAG_NO_SDDMM, **opts)
        if nnz >= 1000 and not opts:
            s = p.stats()
            assert s["spmm_dense_nnz"] > 0 and s["spmm_res_nnz"] > 0
        g = torch.Generator(device="cuda").manual_seed(2)
        for perm in (torch.randperm(nnz, device="cuda", generator=g), torch.arange(nnz - 1, -1, -1, device="cuda")):
            order = p.value_order(perm.int())
            for shift in (0, 1):                         # also an array that is only aligned to its elements
                vals = values(nnz + 1, dt, 3 + shift)[shift:shift + nnz]
                p.set_values(vals[perm].contiguous(), lb.OP_SPMM)
                want = p.spmm(B)
                p.set_values(torch.zeros_like(vals), lb.OP_SPMM)
                p.set_values_ordered(vals, order)
                assert torch.equal(p.spmm(B), want), (opts, shift)
        p.close()


def test_transposed_order_of_a_skewed_matrix():
    """The permutation of a transposition, rows and columns of very different lengths (empty tiles of a chunk, whole-chunk runs)."""
    M, Kc, nnz = 20_000, 70_001, PASSES_MIN + 12_345
    g = torch.Generator(device="cuda").manual_seed(7)
    keys = torch.zeros(0, dtype=torch.int64, device="cuda")
    while keys.numel() < nnz:
        r = (torch.rand(nnz, device="cuda", generator=g) ** 4 * M).long()
        c = (torch.rand(nnz, device="cuda", generator=g) ** 3 * Kc).long()
        keys = torch.unique(torch.cat([keys, r * Kc + c]))
    keys = keys[:nnz]
    rowptr = torch.zeros(M + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.cumsum(torch.bincount(keys // Kc, minlength=M), 0)
    col = (keys % Kc).int()
    rowptr_t, col_t, perm_t = lb.transpose_csr(M, Kc, rowptr, col)
    p = lb.Plan.from_device_csr(Kc, M, rowptr_t, col_t, values(nnz, torch.float16, 1), resident=True, keep_host_copy=False)
    vals, B = values(nnz, torch.float16, 2), values(M * 32, torch.float16, 3).view(M, 32)
    p.set_values(vals[perm_t.long()].contiguous(), lb.OP_SPMM)
    want = p.spmm(B)
    p.set_values_ordered(vals, p.value_order(perm_t))
    assert torch.equal(p.spmm(B), want)
    p.close()


@pytest.mark.parametrize("dtype,nnz", [("f16", 1 << 27), ("f32", (1 << 26) + 16_385), ("f32", 1 << 27), ("f32", (1 << 27) + 64)])
def test_ordered_values_of_very_large_matrices(dtype, nnz):
    """Where the runs of a chunk take more LDS than leaves room for two workgroups, up to the most nonzeros, and past it."""
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 64 << 30:
        pytest.skip("needs some 30 GiB")
    dt, per = DTYPES[dtype], 64
    M, Kc = (nnz + per - 1) // per, 1 << 16
    g = torch.Generator(device="cuda").manual_seed(2)
    rowptr = (torch.arange(M + 1, device="cuda") * per).clamp_(max=nnz).int()
    # a window's rows share few columns of some strata and hardly any of the others
    col = torch.randint(0, Kc // per, (M, per), device="cuda", generator=g, dtype=torch.int32)
    col[:, ::2] %= 6
    col = (col + torch.arange(per, device="cuda", dtype=torch.int32) * (Kc // per)).reshape(-1)[:nnz].contiguous()
    p = lb.Plan.from_device_csr(M, Kc, rowptr, col, torch.ones(nnz, dtype=dt, device="cuda"), resident=True, keep_host_copy=False, flags=lb.FLAG_NO_SDDMM)
    s = p.stats()
    assert s["spmm_dense_nnz"] > nnz // 20 and s["spmm_res_nnz"] > nnz // 20
    perm = torch.randperm(nnz, device="cuda", generator=g, dtype=torch.int32)
    order = p.value_order(perm)
    assert (order[1] > 0) == (nnz <= 1 << 27)               # scratch memory: the two passes
    vals, B = values(nnz, dt, 3), values(Kc * 32, dt, 5).view(Kc, 32)
    p.set_values(vals[perm], lb.OP_SPMM)
    want = p.spmm(B)
    p.set_values(torch.zeros_like(vals), lb.OP_SPMM)
    p.set_values_ordered(vals, order)
    assert torch.equal(p.spmm(B), want)
    p.close()


@pytest.mark.parametrize("nnz", [1000, PASSES_MIN])
def test_orders_that_are_no_permutations_are_refused(nnz):
    M, Kc = (301, 203) if nnz == 1000 else (40_003, 30_011)
    rowptr, col = random_csr(M, Kc, nnz, 1, False)
    p = lb.Plan.from_device_csr(M, Kc, rowptr, col, values(nnz, torch.float16, 1), resident=True, keep_host_copy=False)
    good = torch.arange(nnz, dtype=torch.int32, device="cuda")
    p.value_order(good)
    for at, to in ((0, nnz), (nnz - 1, -1), (5, 6), (nnz - 1, nnz - 2)) + (((5, 40_000),) if nnz == PASSES_MIN else ()):
        bad = good.clone()
        bad[at] = to
        with pytest.raises(lb.LibraError) as e:
            p.value_order(bad)
        assert e.value.code == lb.ERR["SHAPE"]
    order = p.value_order(good)
    for vals in (values(nnz, torch.float32, 1), values(nnz - 1, torch.float16, 1)):
        with pytest.raises(ValueError):
            p.set_values_ordered(vals, order)
    p.close()


def test_orders_of_other_plans_are_refused():
    """Also where they are as long as an own one: the kernels take their places as they are."""
    plans, orders = [], []
    for i, opts in enumerate((dict(), dict(), dict(mode=lb.MODE_SCALAR_ONLY), dict(mode=lb.MODE_DENSE_ONLY))):
        rowptr, col = random_csr(301, 203, 1000 + 7 * (i == 1), 1, False)
        plans.append(lb.Plan.from_device_csr(301, 203, rowptr, col, torch.ones(col.numel(), dtype=torch.float16, device="cuda"), resident=True,
                                             keep_host_copy=False, **opts))
        orders.append(plans[i].value_order(torch.arange(col.numel(), dtype=torch.int32, device="cuda")))
    for i, p in enumerate(plans):
        vals = torch.ones(p.nnz, dtype=torch.float16, device="cuda")
        p.set_values_ordered(vals, orders[i])
        for bad in [o for k, o in enumerate(orders) if k != i] + [tuple(orders[i])]:
            with pytest.raises(ValueError):
                p.set_values_ordered(vals, bad)
    for p in plans:
        p.close()


def test_matrices_without_nonzeros_and_without_spmm():
    from paper_2506_22714_amd import autograd as ag
    empty = ag.SparseMatrix(40, 30, torch.zeros(41, dtype=torch.int32, device="cuda"), torch.zeros(0, dtype=torch.int32, device="cuda"))
    vals, B = torch.zeros(0, dtype=torch.float16, device="cuda"), torch.ones(30, 32, dtype=torch.float16, device="cuda", requires_grad=True)
    C = ag.spmm(empty, vals, B)
    C.sum().backward()
    assert torch.equal(C, torch.zeros_like(C)) and torch.equal(B.grad, torch.zeros_like(B))
    empty.close()
    rowptr, col = random_csr(301, 203, 1000, 1, False)
    sm = ag.SparseMatrix(301, 203, rowptr, col, flags=lb.FLAG_NO_SPMM)         # SDDMM alone: its values have a gradient
    vals = values(1000, torch.float16, 1).requires_grad_()
    X, Y = values(301 * 32, torch.float16, 2).view(301, 32), values(203 * 32, torch.float16, 3).view(203, 32)
    out = ag.sddmm(sm, vals, X, Y)
    out.sum().backward()
    want = (X.float()[torch.repeat_interleave(torch.arange(301, device="cuda"), rowptr.diff().long())] * Y.float()[col.long()]).sum(1)
    assert torch.equal(out.detach(), want * vals.detach().float()) and torch.equal(vals.grad, want.half())
    with pytest.raises(lb.LibraError):
        X2 = X.clone().requires_grad_()
        ag.sddmm(sm, vals, X2, Y).sum().backward()
    sm.close()


@pytest.mark.parametrize("nnz", [1000, PASSES_MIN + 77])
@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_training_calls_can_be_captured_in_a_graph(dtype, nnz):
    """They launch kernels on the caller's stream and nothing else: replays, with eager work between them and other values in place, give the
    eager result.  Both forms of an order; the order itself is made before."""
    dt = DTYPES[dtype]
    M, Kc, K = (301, 203, 64) if nnz == 1000 else (40_003, 30_011, 32)
    rowptr, col = random_csr(M, Kc, nnz, 3, True)
    p = lb.Plan.from_device_csr(M, Kc, rowptr, col, values(nnz, dt, 1), resident=True, keep_host_copy=False, cs=16)
    g = torch.Generator(device="cuda").manual_seed(2)
    order = p.value_order(torch.randperm(nnz, device="cuda", generator=g, dtype=torch.int32))
    vals, B, X = values(nnz, dt, 3), values(Kc * K, dt, 4).view(Kc, K), values(M * K, dt, 5).view(M, K)
    factors, alpha = values(nnz, torch.float32, 6), torch.rand(nnz, device="cuda", generator=g).to(dt)

    def step():
        p.set_values_ordered(p.value_products(vals, factors), order)
        dalpha = p.sddmm_pattern_rounded(X, B)
        return p.spmm_rounded(B), dalpha, p.edge_softmax_backward_rounded(alpha, dalpha, 0.5)

    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(graph, stream=side):
        outs = step()
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(4):
        vals.copy_(values(nnz, dt, 30 + rep))
        for o in outs:
            o.fill_(float("nan"))
        p.set_values(torch.zeros_like(vals))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [o.clone() for o in outs]
        want = step()
        assert all(torch.equal(x, y) for x, y in zip(got, want)), rep
    p.close()
