"""GPU parity of the serving export (bit-packed codes, outliers as CSR)
against the oracle's reference layout: integer and byte work, so bit-exact."""
import numpy as np
import pytest
import torch

import synth
from parity import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [1, 2, 3, 4, 5, 7, 8])
@pytest.mark.parametrize("q,p", [(5, 29), (64, 4096), (3, 1)])
def test_pack_codes_bit_exact(qe, oracle, bits, q, p):
    codes = synth.integers((q, p), seed=bits * 10 + q, lo=0, hi=2 ** bits).astype(np.uint8)
    got = host(qe.pack_codes(dev(codes), bits))
    assert np.array_equal(got, oracle.pack_codes(codes, bits))


def test_outliers_csr_from_topk(qe, oracle):
    V = synth.gaussian((300, 257), seed=51)
    s = 2000
    out, sup, nnz = qe.topk_abs(dev(V), s)
    rowptr, cols, vals = qe.outliers_csr(out, sup, nnz)
    n = int(host(nnz)[0])
    ref_sup, ref_dense = oracle.topk_abs(V, s)
    r_rowptr, r_cols, r_vals = oracle.outliers_csr(ref_dense, ref_sup)
    assert np.array_equal(host(rowptr), r_rowptr)
    assert np.array_equal(host(cols)[:n], r_cols)
    assert np.array_equal(host(vals)[:n], r_vals)


def test_outliers_csr_empty(qe):
    H = torch.zeros((4, 6), dtype=torch.float32, device="cuda")
    sup = torch.zeros(3, dtype=torch.int64, device="cuda")
    nnz = torch.zeros(1, dtype=torch.int64, device="cuda")
    rowptr, _, _ = qe.outliers_csr(H, sup, nnz)
    assert not np.any(host(rowptr))


@pytest.mark.parametrize("bits", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("p", [31, 32, 33, 63, 65, 257])
def test_pack_codes_group_edges(qe, oracle, bits, p):
    """Rows that end inside, at and past a group of 32 codes, from a base one byte
    off; codes past 2^bits keep their low bits."""
    q = 7
    codes = synth.integers((q, p), seed=bits + p, lo=0, hi=256).astype(np.uint8)
    buf = torch.full((q * p + 33,), 255, dtype=torch.uint8, device="cuda")
    cd = buf[1:1 + q * p].view(q, p)
    cd.copy_(dev(codes))
    want = oracle.pack_codes(codes & np.uint8(2 ** bits - 1), bits)
    assert np.array_equal(host(qe.pack_codes(cd, bits)), want)


@pytest.mark.parametrize("q,p,n", [(1, 40, 17), (16, 33, 40), (4100, 64, 900), (300, 257, 1), (50, 20, 1000)])
def test_outliers_csr_row_search(qe, q, p, n):
    """Empty rows at both ends and in runs, one entry, every entry."""
    lin = np.sort(np.random.default_rng(q).choice(q * p, size=n, replace=False)).astype(np.int64)
    H = synth.gaussian((q, p), seed=q)
    rowptr, cols, vals = qe.outliers_csr(dev(H), dev(lin), dev(np.array([n], np.int64)))
    assert np.array_equal(host(rowptr), np.searchsorted(lin, np.arange(q + 1) * p))
    assert np.array_equal(host(cols), lin % p)
    assert np.array_equal(host(vals), H.reshape(-1)[lin])


def test_more_rows_than_one_grid_dimension(qe):
    """Row counts whose workgroups hold 2^32 threads and more: CSR row pointers (16
    lanes per row), the objective's row tiles (two forms of 128 rows each)."""
    q = 2 ** 28 + 7
    H = torch.zeros((q, 1), device="cuda")
    at = torch.tensor([5, q - 8, q - 1], device="cuda")
    H[at, 0] = torch.tensor([1.0, 2.0, 3.0], device="cuda")
    rowptr, cols, vals = qe.outliers_csr(H, at, torch.tensor([3], device="cuda"))
    assert [int(rowptr[i]) for i in (0, 5, 6, q - 8, q - 7, q - 1, q)] == [0, 0, 1, 1, 2, 2, 3]
    assert int(rowptr.double().sum()) == (q - 7 - 6) + 2 * 7 + 3
    assert host(vals).tolist() == [1.0, 2.0, 3.0] and not np.any(host(cols))
    del H, rowptr
    torch.cuda.empty_cache()
    q = 2 ** 30 + 5
    W, Wh = torch.ones((q, 1), device="cuda"), torch.full((q, 1), 3.0, device="cuda")
    out = qe.objective(W, Wh, torch.full((1, 1), 0.5, device="cuda"))
    assert host(out).tolist() == [2.0 * q, 0.5 * q]
    del W, Wh
    torch.cuda.empty_cache()
