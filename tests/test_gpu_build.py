"""Building a handle on the GPU machine: the checks of the uploaded CSR arrays, and blocks reused from handle to handle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _csr(N, D, per_row):
    rowptr = np.arange(N + 1, dtype=np.int64) * per_row
    col = (np.arange(N)[:, None] % (D - per_row) + np.arange(per_row)[None, :]).astype(np.int32).ravel()
    return rowptr, col, np.ones(N * per_row, np.float32)


@pytest.mark.parametrize("N", [1, 300, 200_003])  # one workgroup, a few, every workgroup with several rounds
@pytest.mark.parametrize("where", [0, -1])
@pytest.mark.parametrize("what,code", [("ok", 0), ("equal", -3), ("descending", -3), ("negative", -4), ("too large", -4),
                                       ("pointer", -3)])
def test_csr_rules_on_the_device(N, where, what, code):
    from paper_2004_13940_amd import binding as B
    D, k = 50, 3
    rowptr, col, val = _csr(N, D, k)
    i = 0 if where == 0 else N - 1
    if what == "equal":
        col[i * k + 1] = col[i * k]
    elif what == "descending":
        col[i * k + 2] = col[i * k]
    elif what == "negative":
        col[i * k] = -1
    elif what == "too large":
        col[i * k + 2] = D
    elif what == "pointer":
        if N == 1:
            pytest.skip("one row: both pointers are checked on the host")
        rowptr[i if i > 0 else 1] = N * k + 1
    if code == 0:
        B.Matrix(N, D, rowptr, col, val).close()
        return
    with pytest.raises(B.FMError) as e:
        B.Matrix(N, D, rowptr, col, val)
    assert e.value.code == code and (what == "pointer" or f" {i} " in str(e.value))


def test_handles_one_after_the_other_reuse_blocks_with_their_own_content():
    """Blocks above the pool's smallest size come back with an older handle's content."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(5)
    N, D, k, K = 40_000, 3_000, 12, 16
    w0, w = torch.zeros(1, device="cuda"), torch.from_numpy(rng.standard_normal(D).astype(np.float32)).cuda()
    V = torch.zeros(D * K, device="cuda")
    for shift in range(3):
        rowptr, col, val = _csr(N, D, k)
        val = (val * (1 + shift) + rng.random(N * k).astype(np.float32)).astype(np.float32)
        m = B.Matrix(N, D, rowptr, col, val)
        m.fm_build_csc()
        p = B.make_params(K, B.FM_LOSS_SQUARED, 0.0, 0.0, 0.1)
        a = torch.empty(N, device="cuda")
        m.fm_forward(p, None, w0, w, V, a=a)
        want = (val.reshape(N, k).astype(np.float64) * w.cpu().numpy().astype(np.float64)[col.reshape(N, k)]).sum(1)
        got = a.cpu().numpy()
        assert np.max(np.abs(got - want)) <= 1e-5 * np.max(np.abs(want))
        colptr, row, cval = m.fm_get_csc()
        order = np.argsort(col, kind="stable")
        assert np.array_equal(row, np.repeat(np.arange(N), k)[order]) and np.array_equal(cval, val[order])
        m.close()


def test_trim_gives_the_blocks_of_closed_handles_back():
    """What a closed handle leaves is kept for the next one until fm_trim; an open handle goes on working."""
    import torch
    from paper_2004_13940_amd import binding as B
    N, D, k, K = 400_000, 3_000, 12, 16
    y, w0, w = torch.ones(N, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(D, device="cuda")
    V = torch.full((D * K,), 0.01, device="cuda")
    p = B.make_params(K, B.FM_LOSS_SQUARED, 0.0, 0.0, 0.1, 1.0 / N)
    kept = B.Matrix(500, D, *_csr(500, D, k))
    before = kept.fm_evaluate(p, y[:500].clone(), w0, w, V)
    B.fm_trim()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    m = B.Matrix(N, D, *_csr(N, D, k))
    m.fm_build_csc()
    m.fm_sgd_epoch(p, y, w0.clone(), w.clone(), V.clone())
    m.close()
    assert torch.cuda.mem_get_info()[0] < free - (64 << 20)  # the matrix, its transpose and the aggregates
    B.fm_trim()
    assert torch.cuda.mem_get_info()[0] >= free - (8 << 20)  # the runtime keeps chunks of its own
    assert kept.fm_evaluate(p, y[:500].clone(), w0, w, V) == before
    kept.close()


@pytest.mark.parametrize("per_thread", [0, 1])
@pytest.mark.parametrize("N", [493_447, 493_448, 600_001])  # 16 columns: just below and from 64 MB on, where the upload is staged
def test_large_matrices_arrive_whole(N, per_thread):
    """Two threads open one each at the same time, on the default stream or on hipStreamPerThread (handle 2); a second round
    takes the blocks that the first left.  What a thread raises is raised here."""
    from concurrent.futures import ThreadPoolExecutor
    from types import SimpleNamespace
    from paper_2004_13940_amd import binding as B
    D = 16
    rowptr, col = np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N)
    vals = [np.random.default_rng(k).random((N, D), dtype=np.float32) for k in range(2)]
    stream = SimpleNamespace(cuda_stream=2) if per_thread else None
    print("large upload", N, per_thread, flush=True)

    def check(k):
        m = B.Matrix(N, D, rowptr, col, vals[k].ravel(), stream=stream)
        m.fm_build_csc(stream=stream)
        colptr, row, val = m.fm_get_csc()
        m.close()
        assert np.array_equal(colptr, np.arange(D + 1) * N)
        assert np.array_equal(row.reshape(D, N), np.broadcast_to(np.arange(N), (D, N)))
        assert np.array_equal(val.reshape(D, N), vals[k].T)
        return k

    with ThreadPoolExecutor(2) as threads:
        for _ in range(2):
            assert list(threads.map(check, range(2))) == [0, 1]
    B.fm_trim()


@pytest.mark.parametrize("P", [1, 3, 16, 300])  # one to nine bits of the stratum: one pass of the sort or two
@pytest.mark.parametrize("nnz", [1, 511, 512, 4095, 8191, 8192, 8193, 16_391])  # wavefronts and tiles of the sort, and one more
def test_transpose_and_strata_at_the_edges_of_the_sort(nnz, P):
    """Two thirds of the entries in a few full columns (equal digits side by side), rows and columns without entries between."""
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(nnz * 1000 + P)
    N, D = max(nnz // 3, 400), 1_000
    cells = set()
    while len(cells) < nnz:
        i = int(rng.integers(0, N))
        if 0.2 * N < i < 0.6 * N and nnz < N * 4 // 10:  # a long stretch of empty rows
            continue
        cells.add((i, int(rng.choice([0, 1, 2])) if rng.random() < 0.67 else int(rng.integers(600, D))))
    r, c = np.array(sorted(cells), np.int64).T
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=N))]).astype(np.int64)
    val = rng.standard_normal(nnz).astype(np.float32)
    print("sort edges", nnz, P, flush=True)
    m = B.Matrix(N, D, rowptr, c.astype(np.int32), val)
    m.fm_build_csc()
    order = np.argsort(c, kind="stable")
    colptr, row, cval = m.fm_get_csc()
    assert np.array_equal(colptr, np.concatenate([[0], np.cumsum(np.bincount(c, minlength=D))]))
    assert np.array_equal(row, r[order]) and np.array_equal(cval, val[order])
    m.fm_partition(P)
    rb, cb, cell = m.fm_get_block_index()
    p = np.searchsorted(rb, r, side="right") - 1
    s = (np.searchsorted(cb, c, side="right") - 1 - p) % P
    assert cell.sum() == nnz
    for t in range(P) if P < 300 else (0, 1, 150, 255, 256, 299):
        mine = np.nonzero(s == t)[0]
        ptr, col, v = m.fm_get_stratum_csr(t)
        assert np.array_equal(np.diff(ptr), np.bincount(r[mine], minlength=N))
        assert np.array_equal(col, c[mine]) and np.array_equal(v, val[mine])
        mine = order[s[order] == t]
        ptr, row, v = m.fm_get_stratum_csc(t)
        assert np.array_equal(np.diff(ptr), np.bincount(c[mine], minlength=D))
        assert np.array_equal(row, r[mine]) and np.array_equal(v, val[mine])
    m.close()
