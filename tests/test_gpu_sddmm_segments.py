"""The SDDMM segment task at the places where it changes its path: 64 nonzeros whose rows lie within 16 consecutive rows or
just not, rows further apart than an entry can say, segments that end inside a batch, residual lists that are the whole
matrix (positions implied) and that are not, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2506_22714_amd import binding as lb
from paper_2506_22714_amd import workloads as wl

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def edge_rows(seed=3, Kc=700):
    """Row lengths: a long row; 4 per row, so that 64 nonzeros cover exactly 16 and then (one row of 3) 17 rows; single
    nonzeros with 29 .. 63 empty rows between them; a block dense enough for the matrix-unit path; one last nonzero."""
    lengths = [200] + [4] * 15 + [3] + [4] * 40
    for gap in (29, 30, 31, 32, 63):
        lengths += [0] * gap + [1]
    lengths += [0, 2] * 40 + [60] * 32 + [0] * 17 + [1]
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(120 if n == 60 else Kc, size=n, replace=False)) for n in lengths]
    rowptr = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    col = np.concatenate(cols).astype(np.int32)
    return wl.Csr(len(lengths), Kc, rowptr, col, wl.uniform_values(rng, col.size))


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("K", [32, 64, 128])
def test_segment_edges(K, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    A = edge_rows()
    assert A.M % 16 != 0 and A.nnz % 64 != 0
    tdt = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[dtype]
    bf16 = dtype == "bf16"

    def operand(rows, seed):
        a = wl.dense_normal(rows, K, seed=seed, dtype=np.float32)
        if bf16:
            a = wl.to_bf16_bits(a)
            return a, torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
        a = a if dtype == "f32" else a.astype(np.float16)
        return a, torch.from_numpy(a).cuda()

    def values(v):
        v = v.astype(np.float32)
        if bf16:
            v = wl.to_bf16_bits(v)
            return v, torch.from_numpy(v.view(np.int16)).cuda().view(torch.bfloat16)
        v = v if dtype == "f32" else v.astype(np.float16)
        return v, torch.from_numpy(v).cuda()

    (X, Xd), (Y, Yd) = operand(A.M, 1), operand(A.Kc, 2)
    val, vald = values(A.val)
    new, newd = values(wl.uniform_values(np.random.default_rng(9), A.nnz))
    one, _ = values(np.ones(A.nnz))
    rp, col = (torch.from_numpy(a).cuda() for a in (A.rowptr, A.col))
    limit = 16.0 * np.sqrt(K) * 2.0 ** -24      # products exact (f16, bf16) or rounded once, K - 1 fp32 additions
    refs = {k: oracle.sddmm(A.rowptr, A.col, v, X, Y, bf16=bf16) for k, v in (("val", val), ("new", new), ("one", one))}

    def check(got, which, what):
        ref, S = refs[which]
        err = oracle.graded_error(got.cpu().numpy(), ref, S, K)
        assert err <= limit, f"{what}: {err:.3e} > {limit:.3e}"

    for mode, cs in ((lb.MODE_SCALAR_ONLY, 50), (lb.MODE_SCALAR_ONLY, 64), (lb.MODE_SCALAR_ONLY, 65), (lb.MODE_HYBRID, 33), (lb.MODE_HYBRID, 128)):
        opts = dict(mode=mode, sddmm_cs=cs, sddmm_min_blk_nnz=64)
        plans = [lb.Plan.from_device_csr(A.M, A.Kc, rp, col, vald, resident=True, keep_host_copy=False, **opts),
                 lb.Plan.from_csr(A, val=val, val_dtype=lb.BF16 if bf16 else None, **opts).upload()]
        for p, who in zip(plans, ("device", "host")):
            assert (p.stats()["sddmm_dense_nnz"] > 0) == (mode == lb.MODE_HYBRID)
            what = f"{dtype} K={K} mode={mode} cs={cs} {who} plan"
            check(p.sddmm(Xd, Yd), "val", what)
            check(p.sddmm(Xd, Yd, pattern_only=True), "one", what + ", pattern only")
            p.set_values(newd)
            check(p.sddmm(Xd, Yd), "new", what + ", new values")
            p.close()
