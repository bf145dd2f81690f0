"""The column and row kernels at the edges of their rounds and items, against the oracle."""
import numpy as np
import pytest

from oracle import fm_oracle as O

from helpers import assert_close, dev_params, run_full_epochs, run_stratified_epochs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 2, 4, 12, 16, 28, 32, 60, 100, 256])  # every lane count, packed and planar rows
def test_columns_of_every_length_around_the_rounds_and_the_item(K):
    """Column j holds j entries, j = 0..100: rounds of 4, 8 and 16 entries, one and several items, all lengths mixed
    inside a wavefront; one column stores every row (summed by a whole workgroup)."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7000 + K)
    N, D = 6000, 102
    mask = np.zeros((N, D), bool)
    for j in range(101):
        mask[rng.choice(N, j, replace=False), j] = True
    mask[:, 101] = True
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    r = (rng.standard_normal(N) / N).astype(np.float32)
    G = rng.standard_normal((N, K)).astype(np.float32)
    w = (rng.standard_normal(D) * 0.1).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    print("columns of every length", K, len(col), flush=True)
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_build_csc()
    p = B.make_params(K, O.LOSS_SQUARED, 0.01, 0.02, 0.1)
    _, d_w, d_V = dev_params(np.float32(0), w, V)
    g0 = torch.full((1,), float("nan"), device="cuda")
    gw = torch.full((D,), float("nan"), device="cuda")
    gV = torch.full((D * K,), float("nan"), device="cuda")
    m.fm_gradient(p, to_dev(r), to_dev(G.ravel()), d_w, d_V, g0, gw, gV)
    torch.cuda.synchronize()
    X = O.make_matrix(N, D, rowptr, col, val)
    wg0, wgw, wgV = O.gradient(X, r, G, w, V, 0.01, 0.02)
    assert abs(g0.item() - wg0) <= 1e-5 * np.abs(r).sum()
    assert_close(gw.cpu().numpy(), wgw, "grad_w")
    assert_close(gV.cpu().numpy().reshape(D, K), wgV, "grad_V")
    m.close()


@pytest.mark.parametrize("K", [1, 2, 4, 8, 24, 64, 128, 256])  # every lane count of the finish
def test_table_whose_columns_are_all_summed_by_a_workgroup(K):
    """Every column has more items than a wavefront sums (128 of 32 entries), as in a table of some thousand rows."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7050 + K)
    N, D = 4200, 5
    rowptr, col = np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N)
    val = rng.standard_normal(N * D).astype(np.float32)
    y = rng.standard_normal(N).astype(np.float32)
    w = (rng.standard_normal(D) * 0.1).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    print("columns summed by a workgroup", K, flush=True)
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_build_csc()
    d_w0, d_w, d_V = dev_params(np.float32(0.1), w, V)
    m.fm_sgd_epoch(B.make_params(K, O.LOSS_SQUARED, 0.01, 0.02, 0.5, 1.0 / N), to_dev(y), d_w0, d_w, d_V)
    torch.cuda.synchronize()
    X = O.make_matrix(N, D, rowptr, col, val)
    w0_o, w_o, V_o, _ = O.full_epoch(X, y, float(np.float32(0.1)), w, V, loss=O.LOSS_SQUARED, s=1.0 / N, lambda_w=0.01,
                                     lambda_v=0.02, eta=0.5, update_w0=True)
    assert_close(d_w.cpu().numpy(), w_o, "w")
    assert_close(d_V.cpu().numpy().reshape(D, K), V_o, "V")
    assert abs(d_w0.item() - w0_o) <= 1e-5 * max(abs(w0_o), 0.1)
    m.close()


@pytest.mark.parametrize("N,K", [(1, 1), (1, 2), (2, 1), (5, 3), (17, 64), (300, 4), (1, 256)])
def test_evaluation_of_a_few_rows(N, K):
    """The row kernel leaves three doubles per block of rows for the metrics: at the smallest N and K they take more room
    than the aggregates do.  Another K follows on the same handle, which lays its storage out anew."""
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7100 + 10 * N + K)
    D = 6
    mask = rng.random((N, D)) < 0.6
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    y = np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32)
    X = O.make_matrix(N, D, rowptr, col, val)
    m = B.Matrix(N, D, rowptr, col, val)
    for k in (K, 1):
        print("evaluation of a few rows", N, k, flush=True)
        w = (rng.standard_normal(D) * 0.3).astype(np.float32)
        V = (rng.standard_normal((D, k)) * 0.3).astype(np.float32)
        got = m.fm_evaluate(B.make_params(k, O.LOSS_LOGISTIC, 0.0, 0.0, 0.1), to_dev(y), *dev_params(np.float32(0.1), w, V))
        yh = O.forward(X, float(np.float32(0.1)), w, V)[3]
        loss = O.loss_multiplier(O.LOSS_LOGISTIC, 1.0, yh, y)[0].mean()
        rmse = np.sqrt(np.mean((yh - y) ** 2))
        assert abs(got["mean_loss"] - loss) <= 1e-5 * loss
        assert abs(got["rmse"] - rmse) <= 1e-5 * rmse
        sure = np.abs(yh) > 1e-5
        right = (np.sign(yh) == y)[sure].sum() / N
        assert right - 1e-9 <= got["accuracy"] <= right + (~sure).sum() / N + 1e-9
    m.close()


@pytest.mark.parametrize("K", [1, 2, 6, 16, 28, 32, 60, 64, 128])  # every lane count of the row kernels, K that idles lanes
@pytest.mark.parametrize("P", [1, 3])
def test_refresh_of_rows_of_every_length_around_the_rounds(K, P):
    """Row i holds i mod 40 entries, so that a stratum's rows end in every place of a round, rows without entries among
    them; aggregates, multipliers and parameters after every stratum."""
    from types import SimpleNamespace
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7200 + 10 * K + P)
    N, D = 403, 61
    mask = np.zeros((N, D), bool)
    for i in range(N):
        mask[i, rng.choice(D, i % 40, replace=False)] = True
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    wl = SimpleNamespace(N=N, D=D, K=K, rowptr=rowptr, col=col, val=(rng.random(len(col)) + 0.2).astype(np.float32),
                         y=np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32), w0=np.float32(0.1),
                         w=(rng.standard_normal(D) * 0.2).astype(np.float32),
                         V=(rng.standard_normal((D, K)) * 0.2 / np.sqrt(K)).astype(np.float32), loss=O.LOSS_LOGISTIC,
                         lambda_w=0.01, lambda_v=0.02, eta=0.5, loss_scale=1.0 / N, update_w0=1)
    print("refresh of rows of every length", K, P, flush=True)
    X = O.make_matrix(N, D, rowptr, col, wl.val)
    m = B.Matrix(N, D, rowptr, col, wl.val)
    m.fm_build_csc()
    m.fm_partition(P)
    p = B.make_params(K, wl.loss, wl.lambda_w, wl.lambda_v, wl.eta, wl.loss_scale, 1)
    dev = (*dev_params(wl.w0, wl.w, wl.V), to_dev(wl.y))
    host = (float(wl.w0), wl.w.astype(np.float64), wl.V.astype(np.float64))
    run_stratified_epochs(B, wl, m, p, X, dev, host, 1, check_strata=True)
    m.close()


@pytest.mark.parametrize("N,P,K", [(65_535, 3, 8), (65_536, 3, 8), (70_001, 600, 16), (70_001, 600, 32), (66_000, 1, 4)])
def test_items_of_strata_and_batches_in_row_order(N, P, K):
    """Columns that are full, start late or end early, so that their items interleave by row; from 65,536 rows on they are
    worked on in that order; with 600 strata of 70,001 rows a stratum and a row no longer fit the sort key together and
    rows are taken in units of eight."""
    from types import SimpleNamespace
    from paper_2004_13940_amd import binding as B
    from test_gpu_parity import _run_minibatch_epochs
    rng = np.random.default_rng(7400 + N + K)
    D = max(P, 7)
    mask = rng.random((N, D)) < 2.0 / D
    for j, lo, hi in ((0, 0, N), (D // 3, 0, N), (D // 2, N // 3, N), (D - 2, 0, N // 2), (D - 1, 0, N)):
        mask[lo:hi, j] = True
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    wl = SimpleNamespace(N=N, D=D, K=K, P=P, rowptr=rowptr, col=col, val=rng.standard_normal(len(col)).astype(np.float32),
                         y=np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32), w0=np.float32(0.1),
                         w=(rng.standard_normal(D) * 0.2).astype(np.float32),
                         V=(rng.standard_normal((D, K)) * 0.2 / np.sqrt(K)).astype(np.float32), loss=O.LOSS_LOGISTIC,
                         lambda_w=0.01, lambda_v=0.02, eta=0.5, loss_scale=1.0 / N, update_w0=1, name="row order",
                         nnz=len(col))
    print("items in row order", N, P, K, flush=True)
    X = O.make_matrix(N, D, rowptr, col, wl.val)
    m = B.Matrix(N, D, rowptr, col, wl.val)
    m.fm_set_tuning(seg=16)
    m.fm_build_csc()
    m.fm_partition(P)
    p = B.make_params(K, wl.loss, wl.lambda_w, wl.lambda_v, wl.eta, wl.loss_scale, 1)
    dev = (*dev_params(wl.w0, wl.w, wl.V), to_dev(wl.y))
    host = (float(wl.w0), wl.w.astype(np.float64), wl.V.astype(np.float64))
    run_stratified_epochs(B, wl, m, p, X, dev, host, 1)
    m.close()
    wl.lambda_w = wl.lambda_v = 1e-5  # a batch is scored before its columns take their postponed regulariser steps
    m2, _, _ = _run_minibatch_epochs(B, wl, P, 1, update_w0=True, setup=lambda h: h.fm_set_tuning(seg=16))
    m2.close()


@pytest.mark.parametrize("D", [(1 << 19) - 1, 1 << 19])  # K = 256: empty columns behind the others and, from 2^27 floats, beside them
def test_empty_columns_of_a_large_factor_matrix(D):
    """Nearly all columns are empty.  Their gradient is lambda v and their step v (1 - eta lambda), exactly as rounded; the
    caller's next work on the same stream sees all of it."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7500 + D)
    N, K, lw, lv, eta = 300, 256, 0.01, 0.02, 0.5
    cols = np.sort(np.concatenate([[0, D - 1], rng.choice(np.arange(1, D - 1), 38, replace=False)])).astype(np.int32)
    mask = rng.random((N, 40)) < 0.4
    mask[0] = True  # every listed column has an entry
    mask[:, 7] = True
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    sub = np.nonzero(mask)[1].astype(np.int32)
    val = rng.standard_normal(len(sub)).astype(np.float32)
    r = (rng.standard_normal(N) / N).astype(np.float32)
    G = rng.standard_normal((N, K)).astype(np.float32)
    w, V = torch.rand(D, device="cuda"), torch.rand(D * K, device="cuda")
    print("empty columns", D, flush=True)
    m = B.Matrix(N, D, rowptr, cols[sub], val)
    m.fm_build_csc()
    p = B.make_params(K, O.LOSS_SQUARED, lw, lv, eta, 1.0 / N)
    at = torch.from_numpy(cols.astype(np.int64)).cuda()
    rest = torch.ones(D, dtype=torch.bool, device="cuda")
    rest[at] = False
    X = O.make_matrix(N, 40, rowptr, sub, val)
    _, wgw, wgV = O.gradient(X, r, G, w[at].cpu().numpy(), V.view(D, K)[at].cpu().numpy(), lw, lv)
    d_r, d_G, g0 = to_dev(r), to_dev(G.ravel()), torch.empty(1, device="cuda")
    for _ in range(3):
        gw, gV = torch.full((D,), float("nan"), device="cuda"), torch.full((D * K,), float("nan"), device="cuda")
        m.fm_gradient(p, d_r, d_G, w, V, g0, gw, gV)
        gw, gV = gw * 1.0, gV.view(D, K) * 1.0
        assert torch.equal(gw[rest], w[rest] * lw) and torch.equal(gV[rest], V.view(D, K)[rest] * lv)
        assert_close(gw[at].cpu().numpy(), wgw, "grad_w")
        assert_close(gV[at].cpu().numpy(), wgV, "grad_V")
    del gw, gV
    y, w1, V1, w0 = to_dev(rng.standard_normal(N)), w.clone(), V.clone(), torch.zeros(1, device="cuda")
    m.fm_sgd_epoch(p, y, w0, w1, V1)
    w2, V2 = w1 * 1.0, V1.view(D, K) * 1.0
    fw, fv = (float(np.float32(1) - np.float32(eta) * np.float32(x)) for x in (lw, lv))
    assert torch.equal(w2[rest], w[rest] * fw) and torch.equal(V2[rest], V.view(D, K)[rest] * fv)
    w0o, wo, Vo, _ = O.full_epoch(X, y.cpu().numpy(), 0.0, w[at].cpu().numpy(), V.view(D, K)[at].cpu().numpy(),
                                  loss=O.LOSS_SQUARED, s=1.0 / N, lambda_w=lw, lambda_v=lv, eta=eta, update_w0=True)
    assert_close(w2[at].cpu().numpy(), wo, "w")
    assert_close(V2[at].cpu().numpy(), Vo, "V")
    m.close()


def test_gradient_that_forks_for_its_empty_columns_replays_from_a_graph():
    """A caller may capture the call: the fork onto the side stream and the join are part of the graph."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7550)
    N, D, K = 200, 1 << 19, 256
    col = np.sort(rng.choice(D, (N, 6)), axis=1).astype(np.int32) // 6 * 6 + np.arange(6, dtype=np.int32)
    rowptr, val = np.arange(N + 1, dtype=np.int64) * 6, rng.standard_normal(N * 6).astype(np.float32)
    m = B.Matrix(N, D + 6, rowptr, col.ravel(), val)
    m.fm_build_csc()
    D += 6
    p = B.make_params(K, O.LOSS_SQUARED, 0.01, 0.02, 0.5, 1.0 / N)
    w, V, r, G = (torch.rand(n, device="cuda") for n in (D, D * K, N, N * K))
    g0, gw, gV = torch.empty(1, device="cuda"), torch.empty(D, device="cuda"), torch.empty(D * K, device="cuda")
    print("gradient from a graph", flush=True)
    m.fm_gradient(p, r, G, w, V, g0, gw, gV)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        m.fm_gradient(p, r, G, w, V, g0, gw, gV)
    for _ in range(4):
        r.add_(0.5)
        m.fm_gradient(p, r, G, w, V, g0, gw, gV)
        want = g0.clone(), gw.clone(), gV.clone()
        for t in (g0, gw, gV):
            t.fill_(float("nan"))
        graph.replay()
        assert torch.equal(g0, want[0]) and torch.equal(gw, want[1]) and torch.equal(gV, want[2])
    torch.cuda.synchronize()
    m.close()


@pytest.mark.parametrize("side_streams", [0, 1])
@pytest.mark.parametrize("K,planar", [(4, 0), (4, 1), (8, 0), (12, 0), (12, 1), (16, 0), (16, 1), (16, 2), (20, 1), (28, 0), (60, 0),
                                      (64, 0), (128, 0), (132, 0), (256, 0)])  # every lane count, K that idles lanes
def test_columns_staged_in_tiles(K, planar, side_streams):
    """Dense-ish columns beside sparse ones over five tiles of 64 rows and a ragged one, through the LDS-staged kernel on the
    launch stream or on its own; whole epochs one after the other, so that each needs the last one's step."""
    from types import SimpleNamespace
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7600 + K)
    N, D = 5 * 64 + 37, 45
    mask = rng.random((N, D)) < 0.02
    mask[:, 3] = True
    mask[:, 20] = rng.random(N) < 0.5
    mask[:, 21] = rng.random(N) < 0.15
    mask[64:128, 20] = False  # a dense-ish column without entries in one tile
    mask[:, 40] = rng.random(N) < 0.9
    mask[:, 30] = False
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    wl = SimpleNamespace(N=N, D=D, K=K, rowptr=rowptr, col=col, val=rng.standard_normal(len(col)).astype(np.float32),
                         y=np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32), w0=np.float32(0.1),
                         w=(rng.standard_normal(D) * 0.2).astype(np.float32),
                         V=(rng.standard_normal((D, K)) * 0.2 / np.sqrt(K)).astype(np.float32), loss=O.LOSS_LOGISTIC,
                         lambda_w=0.01, lambda_v=0.02, eta=0.5, loss_scale=1.0 / N, update_w0=1)

    def setup(m):
        m.fm_set_tuning(seg=16)
        m.fm_set_tile_tuning(tile_rows=64, min_per_tile=4, tile_seg=16)
        m.fm_set_option(B.FM_OPT_AUX_PLANAR, planar)
        m.fm_set_option(B.FM_OPT_SIDE_STREAMS, side_streams)

    print("columns staged in tiles", K, planar, side_streams, flush=True)
    m, p, _, dev, _ = run_full_epochs(B, wl, 3, setup=setup)
    m.fm_profile_enable(True)
    m.fm_sgd_epoch(p, dev[3], *dev[:3])
    assert m.fm_profile_read()["cols_tile"][0] == 1
    m.close()


@pytest.mark.parametrize("K,packed", [(1, 0), (2, 0), (3, 0), (4, 0), (8, 0), (12, 0), (16, 0), (28, 0), (32, 0),  # every lane count below 16
                                      (4, 2), (8, 2), (12, 2), (16, 2), (28, 2)])  # packed rows also where planar ones are the default
def test_columns_and_refresh_with_64_bit_addresses(K, packed, monkeypatch):
    """The same matrices through the form of the walk that large arrays take: slots without an entry read the run's last row
    again, empty runs row 0, and neither may count."""
    from paper_2004_13940_amd import binding as B
    build = B.Matrix.fm_build_csc

    def wide(m, *a, **k):
        m.fm_set_option(B.FM_OPT_WIDE_ADDRESSES, 1)
        m.fm_set_option(B.FM_OPT_AUX_PLANAR, packed)
        build(m, *a, **k)

    monkeypatch.setattr(B.Matrix, "fm_build_csc", wide)
    test_columns_of_every_length_around_the_rounds_and_the_item(K)
    for P in (1, 3):
        test_refresh_of_rows_of_every_length_around_the_rounds(K, P)


# packed rows of 128 bytes, the aggregates 4,096 bytes below 4 GiB and less, and more; the caller's G of 128 bytes a row,
# where the aggregates of 140 bytes a row decide
@pytest.mark.parametrize("N,K", [(33_554_300, 16), (33_554_500, 16), (30_678_300, 32), (30_678_400, 32)])
def test_gathers_at_offsets_of_two_to_four_gigabytes(N, K):
    """Columns whose entries lie in the first and the last rows and around 2 GiB: 32-bit offsets into the buffer up to its
    largest size, 64-bit addresses above."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7700 + K)
    edges = [0, 1, (1 << 24) - 2, (1 << 24) - 1, 1 << 24, (1 << 24) + 1, N - 2, N - 1]
    rows = np.unique(np.concatenate([edges, rng.choice(N, 300, replace=False)]))
    D = 5
    mask = rng.random((len(rows), D)) < 0.6
    mask[:, 0] = True
    counts = np.zeros(N, np.int64)
    counts[rows] = mask.sum(1)
    rowptr = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    sub = np.nonzero(mask)
    val = rng.standard_normal(len(sub[0])).astype(np.float32)
    gen = torch.Generator(device="cuda").manual_seed(K)
    G, r = torch.randn(N * K, generator=gen, device="cuda"), torch.randn(N, generator=gen, device="cuda")
    w = (rng.standard_normal(D) * 0.1).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    print("offsets of gigabytes", N, K, flush=True)
    m = B.Matrix(N, D, rowptr, sub[1].astype(np.int32), val)
    m.fm_build_csc()
    _, d_w, d_V = dev_params(np.float32(0), w, V)
    gw, gV = torch.full((D,), float("nan"), device="cuda"), torch.full((D * K,), float("nan"), device="cuda")
    m.fm_gradient(B.make_params(K, O.LOSS_SQUARED, 0.01, 0.02, 0.1), r, G, d_w, d_V, None, gw, gV)
    at = torch.from_numpy(rows).cuda()
    X = O.make_matrix(len(rows), D, np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64), sub[1].astype(np.int32), val)
    _, wgw, wgV = O.gradient(X, r[at].cpu().numpy(), G.view(N, K)[at].cpu().numpy(), w, V, 0.01, 0.02)
    assert_close(gw.cpu().numpy(), wgw, "grad_w")
    assert_close(gV.cpu().numpy().reshape(D, K), wgV, "grad_V")
    m.close()
    B.fm_trim()


@pytest.mark.parametrize("N,D,K", [(1, 1, 1), (31, 5, 4), (32, 32, 32), (33, 33, 33), (127, 31, 28), (129, 64, 3),
                                   (4097, 63, 17), (1000, 8, 64), (98_400, 33, 12), (99_000, 17, 40), (40_003, 64, 64), (33, 9, 8), (70, 40, 20)])
def test_dense_kernels_at_the_edges_of_their_tiles(N, D, K):
    """Tables whose rows, columns and latent dimensions end just before, at and after a tile of 32, one tile to a wavefront
    and more than eight (where its sums are set aside); packed and planar aggregates.  Forward, metrics, gradient, an epoch
    and a mini-batch epoch against the oracle; without the dense kernels, and with packed rows where planar ones are the default
    (K = 8 and more), the same entry points meet it too."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7900 + N + 100 * D + K)
    rowptr, col = np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N)
    val = rng.standard_normal(N * D).astype(np.float32)
    y = np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32)
    w0, w = np.float32(0.1), (rng.standard_normal(D) * 0.1).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.3 / np.sqrt(D * K)).astype(np.float32)
    X = O.make_matrix(N, D, rowptr, col, val)
    kw = dict(loss=O.LOSS_LOGISTIC, s=1.0 / N, lambda_w=0.01, lambda_v=0.02, eta=0.5)
    a, G, q, yhat = O.forward(X, float(w0), w, V)
    l, r = O.loss_multiplier(O.LOSS_LOGISTIC, 1.0 / N, yhat, y)
    want = dict(yhat=yhat, a=a, G=G, q=q, r=r)
    batches = min(N, 3)
    for dense, packed in ((1, 0), (0, 0)) + (((1, 2), (0, 2)) if K % 4 == 0 and 8 <= K <= 28 else ()):
        print("dense tiles", N, D, K, dense, packed, flush=True)
        m = B.Matrix(N, D, rowptr, col, val)
        m.fm_set_option(B.FM_OPT_DENSE_ROWS, dense)
        m.fm_set_option(B.FM_OPT_AUX_PLANAR, packed)
        p = B.make_params(K, O.LOSS_LOGISTIC, 0.01, 0.02, 0.5, 1.0 / N)
        d_w0, d_w, d_V = dev_params(w0, w, V)
        d_y = to_dev(y)
        out = {k: torch.full((N * (K if k == "G" else 1),), float("nan"), device="cuda") for k in want}
        loss_sum = m.fm_forward(p, d_y, d_w0, d_w, d_V, want_loss=True, **out)
        for k in want:
            assert_close(out[k].cpu().numpy().reshape(np.shape(want[k])), want[k], k)
        assert abs(loss_sum - l.sum()) <= 1e-5 * l.sum()
        met = m.fm_evaluate(p, d_y, d_w0, d_w, d_V)
        assert abs(met["rmse"] - np.sqrt(np.mean((yhat - y) ** 2))) <= 1e-5 * met["rmse"]
        m.fm_build_csc()
        gw = torch.full((D,), float("nan"), device="cuda")
        gV = torch.full((D * K,), float("nan"), device="cuda")
        g0 = torch.full((1,), float("nan"), device="cuda")
        m.fm_gradient(p, out["r"], out["G"], d_w, d_V, g0, gw, gV)
        wg0, wgw, wgV = O.gradient(X, r, G, w, V, 0.01, 0.02)
        assert abs(g0.item() - wg0) <= 1e-5 * np.abs(r).sum()
        assert_close(gw.cpu().numpy(), wgw, "grad_w")
        assert_close(gV.cpu().numpy().reshape(D, K), wgV, "grad_V")
        obj = m.fm_sgd_epoch(p, d_y, d_w0, d_w, d_V, want_objective=True)
        o0, ow, oV, oobj = O.full_epoch(X, y, float(w0), w, V, update_w0=True, **kw)
        assert abs(obj[0] - oobj[0]) <= 1e-5 * oobj[0] and abs(obj[1] - oobj[1]) <= 1e-5 * oobj[1]
        aux = {k: torch.full_like(out[k], float("nan")) for k in ("G", "r")}
        m.fm_get_aux(K, **aux)
        for k in aux:
            assert_close(aux[k].cpu().numpy().reshape(np.shape(want[k])), want[k], k + " held after the epoch")
        m.fm_partition_batches(batches)
        m.fm_minibatch_epoch(p, d_y, d_w0, d_w, d_V)
        o0, ow, oV, _ = O.minibatch_epoch(X, y, o0, ow, oV, B=batches, update_w0=True, reg_share=True, **kw)
        assert_close(d_w.cpu().numpy(), ow, "w")
        assert_close(d_V.cpu().numpy().reshape(D, K), oV, "V")
        assert abs(d_w0.item() - o0) <= 1e-4 * max(abs(o0), 1e-2)
        m.close()


@pytest.mark.parametrize("N,D,K", [(1, 1, 1), (1, 64, 64), (4, 33, 20), (5, 32, 32), (31, 8, 8), (33, 64, 33), (129, 7, 64)])
def test_dense_kernels_leave_what_lies_behind_the_last_row(N, D, K):
    """The last tile of a table has rows that do not exist: nothing is written behind the caller's G, r, a, q and scores, and
    the NaN that lie behind G and r do not reach the gradient."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7950 + N + D + K)
    rowptr, col = np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N)
    val = rng.standard_normal(N * D).astype(np.float32)
    y = rng.standard_normal(N).astype(np.float32)
    w0, w = np.float32(0.1), (rng.standard_normal(D) * 0.1).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    print("behind the last row", N, D, K, flush=True)
    X = O.make_matrix(N, D, rowptr, col, val)
    a, G, q, yhat = O.forward(X, float(w0), w, V)
    _, r = O.loss_multiplier(O.LOSS_SQUARED, 1.0, yhat, y)
    want = dict(yhat=yhat, a=a, G=G, q=q, r=r)
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_set_option(B.FM_OPT_DENSE_ROWS, 1)
    p = B.make_params(K, O.LOSS_SQUARED, 0.01, 0.02, 0.5, 1.0)
    d_w0, d_w, d_V = dev_params(w0, w, V)
    d_y = to_dev(y)
    out = {k: torch.full(((N + 64) * (K if k == "G" else 1),), float("nan"), device="cuda") for k in want}
    m.fm_forward(p, d_y, d_w0, d_w, d_V, **{k: t[:len(t) - 64 * (K if k == "G" else 1)] for k, t in out.items()})
    for k, t in out.items():
        n = want[k].size
        assert_close(t[:n].cpu().numpy().reshape(want[k].shape), want[k], k)
        assert torch.isnan(t[n:]).all(), k
    m.fm_build_csc()
    gw, gV, g0 = torch.zeros(D, device="cuda"), torch.zeros(D * K, device="cuda"), torch.zeros(1, device="cuda")
    m.fm_gradient(p, out["r"][:N], out["G"][:N * K], d_w, d_V, g0, gw, gV)
    _, wgw, wgV = O.gradient(X, r, G, w, V, 0.01, 0.02)
    assert_close(gw.cpu().numpy(), wgw, "grad_w")
    assert_close(gV.cpu().numpy().reshape(D, K), wgV, "grad_V")
    m.close()


@pytest.mark.parametrize("N,D,K", [(5_000, 64, 64), (40_000, 20, 8), (200_000, 32, 32), (230_000, 64, 32), (262_144, 64, 64),
                                   (300_000, 20, 8), (400_000, 64, 64), (500_000, 32, 64)])
def test_dense_gradient_adds_few_rows_in_fp32(N, D, K):
    """Sums over terms of one sign in the first half of the rows, of the other in the second: the total is small and its own
    rounding does not hide the error of the partial sums.  An fp32 sum of n terms makes n roundings of at most 2^-24 of the sum
    so far (rms 2^-24 / sqrt 3 of it), together sqrt(n / 3) of that; N / n such sums added exactly are off by
    2^-24 n / (3 sqrt N) of the sum of the magnitudes.  The bound is that of n = max(64, N / 4096) rows."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(7970)
    X, G, r = (rng.random(s, dtype=np.float32) + np.float32(0.5) for s in ((N, D), (N, K), N))
    r[N // 2:] *= -1
    print("rows to an fp32 sum", N, D, K, flush=True)
    m = B.Matrix(N, D, np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N), X.ravel())
    m.fm_set_option(B.FM_OPT_DENSE_ROWS, 1)
    m.fm_build_csc()
    p = B.make_params(K, O.LOSS_SQUARED, 0.0, 0.0, 0.5, 1.0)
    gw, gV, g0 = torch.zeros(D, device="cuda"), torch.zeros(D * K, device="cuda"), torch.zeros(1, device="cuda")
    m.fm_gradient(p, to_dev(r), to_dev(G.ravel()), torch.zeros(D, device="cuda"), torch.zeros(D * K, device="cuda"), g0, gw, gV)
    m.close()
    X, rG, r = X.astype(np.float64).T, G.astype(np.float64) * r[:, None], r.astype(np.float64)
    bound = 2.0 ** -24 * max(64, N / 4096) / (3 * np.sqrt(N))
    for got, want, size in ((gw.cpu().numpy(), X @ r, X @ np.abs(r)), (gV.cpu().numpy().reshape(D, K), X @ rG, X @ np.abs(rG))):
        assert np.sqrt(np.mean(((got - want) / size) ** 2)) <= bound


@pytest.mark.parametrize("N,D,K", [(2048, 60, 40), (2049, 60, 40), (8192, 33, 33), (8193, 33, 33), (8192, 20, 64), (8193, 40, 8), (4096, 40, 8), (4097, 40, 8)])
def test_tables_around_the_rows_that_the_dense_kernels_take(N, D, K):
    """Just up to and just beyond the numbers of rows from which the dense kernels take an epoch, a forward pass, a gradient
    and batches: every call against the oracle, and against the dense kernels whatever the number of rows."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8000 + N + D)
    rowptr, col = np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N)
    val = rng.standard_normal(N * D).astype(np.float32)
    y = np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32)
    w0, w = np.float32(0.1), (rng.standard_normal(D) * 0.1).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.3 / np.sqrt(D * K)).astype(np.float32)
    print("rows of the dense kernels", N, D, K, flush=True)
    X = O.make_matrix(N, D, rowptr, col, val)
    a, G, q, yhat = O.forward(X, float(w0), w, V)
    l, r = O.loss_multiplier(O.LOSS_LOGISTIC, 1.0 / N, yhat, y)
    _, wgw, wgV = O.gradient(X, r, G, w, V, 0.01, 0.02)
    kw = dict(loss=O.LOSS_LOGISTIC, s=1.0 / N, lambda_w=0.01, lambda_v=0.02, eta=0.5, update_w0=True)
    o0, ow, oV, oobj = O.full_epoch(X, y, float(w0), w, V, **kw)
    b0, bw, bV, _ = O.minibatch_epoch(X, y, o0, ow, oV, B=4, reg_share=True, **kw)
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.01, 0.02, 0.5, 1.0 / N)
    for option in (2, 1):
        m = B.Matrix(N, D, rowptr, col, val)
        m.fm_set_option(B.FM_OPT_DENSE_ROWS, option)
        d_w0, d_w, d_V = dev_params(w0, w, V)
        d_y = to_dev(y)
        dG, dr = torch.full((N * K,), float("nan"), device="cuda"), torch.full((N,), float("nan"), device="cuda")
        loss_sum = m.fm_forward(p, d_y, d_w0, d_w, d_V, G=dG, r=dr, want_loss=True)
        assert abs(loss_sum - l.sum()) <= 1e-5 * l.sum()
        assert_close(dG.cpu().numpy().reshape(N, K), G, "G")
        met = m.fm_evaluate(p, d_y, d_w0, d_w, d_V)
        assert abs(met["rmse"] - np.sqrt(np.mean((yhat - y) ** 2))) <= 1e-5 * met["rmse"]
        m.fm_build_csc()
        gw, gV, g0 = torch.zeros(D, device="cuda"), torch.zeros(D * K, device="cuda"), torch.zeros(1, device="cuda")
        m.fm_gradient(p, dr, dG, d_w, d_V, g0, gw, gV)
        assert_close(gw.cpu().numpy(), wgw, "grad_w")
        assert_close(gV.cpu().numpy().reshape(D, K), wgV, "grad_V")
        obj = m.fm_sgd_epoch(p, d_y, d_w0, d_w, d_V, want_objective=True)
        assert abs(obj[0] - oobj[0]) <= 1e-5 * oobj[0] and abs(obj[1] - oobj[1]) <= 1e-5 * oobj[1]
        assert_close(d_V.cpu().numpy().reshape(D, K), oV, "V")
        m.fm_partition_batches(4)
        m.fm_minibatch_epoch(p, d_y, d_w0, d_w, d_V)
        assert_close(d_w.cpu().numpy(), bw, "w after batches")
        assert_close(d_V.cpu().numpy().reshape(D, K), bV, "V after batches")
        m.close()


def test_captured_half_precision_pass_of_a_small_table_needs_no_copy_of_the_factors():
    """After a pass in fp32 the workspace is there; a first pass with half_gather is then captured, which a memory allocation
    would spoil, and replayed between eager passes."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8060)
    N, D, K = 700, 40, 36
    val = rng.standard_normal(N * D).astype(np.float32)
    m = B.Matrix(N, D, np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N), val)
    w0, w, V = dev_params(np.float32(0.1), (rng.standard_normal(D) * 0.1).astype(np.float32), (rng.standard_normal((D, K)) * 0.1).astype(np.float32))
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.0, 0.0, 0.5, 1.0 / N)
    ph = B.make_params(K, O.LOSS_LOGISTIC, 0.0, 0.0, 0.5, 1.0 / N, half_gather=1)
    out = torch.zeros(N, device="cuda")
    m.fm_forward(p, None, w0, w, V, yhat=out)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.fm_forward(ph, None, w0, w, V, yhat=out)
    eager = torch.zeros(N, device="cuda")
    for _ in range(3):
        out.zero_()
        g.replay()
        m.fm_forward(ph, None, w0, w, V, yhat=eager)
        torch.cuda.synchronize()
        assert torch.equal(out, eager)
    m.close()


@pytest.mark.parametrize("N,D,K", [(33, 5, 4), (4097, 33, 36), (40_003, 64, 32)])
def test_half_gather_of_dense_tables(N, D, K):
    """The dense kernel rounds the factors of the scores itself; the step is taken on the fp32 factors.  Metrics, scores and an
    epoch against the oracle: its forward on the rounded factors, its gradient on the factors as they are."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8050 + N)
    rowptr, col = np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N)
    val = rng.standard_normal(N * D).astype(np.float32)
    y = np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32)
    w0, w = np.float32(0.1), (rng.standard_normal(D) * 0.1).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.3 / np.sqrt(D * K)).astype(np.float32)
    X = O.make_matrix(N, D, rowptr, col, val)
    a, G, q, yhat = O.forward(X, float(w0), w, V.astype(np.float16).astype(np.float32))
    _, r = O.loss_multiplier(O.LOSS_LOGISTIC, 1.0 / N, yhat, y)
    _, gw, gV = O.gradient(X, r, G, w, V, 0.01, 0.02)
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_set_option(B.FM_OPT_DENSE_ROWS, 1)
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.01, 0.02, 0.5, 1.0 / N, half_gather=1)
    d_w0, d_w, d_V = dev_params(w0, w, V)
    d_y = to_dev(y)
    out = torch.full((N,), float("nan"), device="cuda")
    m.fm_forward(p, d_y, d_w0, d_w, d_V, yhat=out)
    assert_close(out.cpu().numpy(), yhat, "yhat")
    met = m.fm_evaluate(p, d_y, d_w0, d_w, d_V)
    assert abs(met["rmse"] - np.sqrt(np.mean((yhat - y) ** 2))) <= 1e-5 * met["rmse"]
    m.fm_build_csc()
    m.fm_sgd_epoch(p, d_y, d_w0, d_w, d_V)
    assert_close(d_w.cpu().numpy(), w - 0.5 * gw, "w")
    assert_close(d_V.cpu().numpy().reshape(D, K), V - 0.5 * gV, "V")
    m.close()


@pytest.mark.parametrize("N", [4096, 4098])  # blocks of 2,048 rows, the most whose columns are summed whole, and of one more
@pytest.mark.parametrize("K", [1, 2, 4, 6, 8, 16, 24, 28, 32, 64])  # every lane count, packed and planar rows
def test_long_columns_of_strata_and_batches_summed_whole(N, K):
    """Columns whose parts in the two row blocks have lengths around the item, the wavefront's and the workgroup's: strata,
    and batches with the bias step in the same launch."""
    from types import SimpleNamespace
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8100 + N + K)
    lengths = [0, 1, 31, 32, 33, 64, 127, 128, 129, 255, 256, 257, 300, 511, 1024, 1025, 2047, 2048]
    half, D = N // 2, 2 * len(lengths)
    mask = np.zeros((N, D), bool)
    for t, n in enumerate(lengths):
        mask[rng.choice(half, n, replace=False), 2 * t] = True
        mask[half + rng.choice(N - half, lengths[-1 - t], replace=False), 2 * t] = True
        mask[half + rng.choice(N - half, n, replace=False), 2 * t + 1] = True
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    wl = SimpleNamespace(N=N, D=D, K=K, rowptr=rowptr, col=col, val=rng.standard_normal(len(col)).astype(np.float32),
                         y=np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32), w0=np.float32(0.1),
                         w=(rng.standard_normal(D) * 0.2).astype(np.float32),
                         V=(rng.standard_normal((D, K)) * 0.2 / np.sqrt(K)).astype(np.float32), loss=O.LOSS_LOGISTIC,
                         lambda_w=0.01, lambda_v=0.02, eta=0.5, loss_scale=1.0 / N, update_w0=1)
    print("columns summed whole", N, K, flush=True)
    X = O.make_matrix(N, D, rowptr, col, wl.val)
    p = B.make_params(K, wl.loss, wl.lambda_w, wl.lambda_v, wl.eta, wl.loss_scale, 1)
    host = (float(wl.w0), wl.w.astype(np.float64), wl.V.astype(np.float64))
    m = B.Matrix(N, D, rowptr, col, wl.val)
    m.fm_build_csc()
    m.fm_partition(2)
    run_stratified_epochs(B, wl, m, p, X, (*dev_params(wl.w0, wl.w, wl.V), to_dev(wl.y)), host, 1, check_strata=True)
    m.fm_partition_batches(2)
    d_w0, d_w, d_V = dev_params(wl.w0, wl.w, wl.V)
    # a batch is scored before its columns take the regulariser steps they postponed: eta lambda below what is compared
    p = B.make_params(K, wl.loss, 1e-5, 2e-5, wl.eta, wl.loss_scale, 1)
    m.fm_minibatch_epoch(p, to_dev(wl.y), d_w0, d_w, d_V)
    o0, ow, oV, _ = O.minibatch_epoch(X, wl.y, *host, B=2, update_w0=True, reg_share=True, loss=wl.loss, s=1.0 / N,
                                      lambda_w=1e-5, lambda_v=2e-5, eta=0.5)
    assert_close(d_w.cpu().numpy(), ow, "w")
    assert_close(d_V.cpu().numpy().reshape(D, K), oV, "V")
    assert abs(d_w0.item() - o0) <= 1e-4 * max(abs(o0), 1e-2)
    m.close()


@pytest.mark.parametrize("row", [16, 17, 33, 50, 64, 65, 130])  # around the rounds of one, two and four groups
@pytest.mark.parametrize("K,half", [(1, 0), (2, 0), (4, 1), (6, 0), (8, 0), (16, 0), (16, 1), (24, 0)])  # every lane count
def test_forward_of_rows_shared_by_lane_groups(row, K, half):
    """Few rows of about `row` entries, shared by one, two or four lane groups; empty, short and twice as long rows among
    them.  Scores, aggregates, the sums of the loss and the gradient step that follow from them."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8200 + 10 * row + K)
    N, D = 203, 2 * row + 5
    lens = np.clip(rng.integers(row - 2, row + 3, N), 0, D)
    lens[::11], lens[5::17], lens[7::23] = 0, 1, 2 * row
    mask = np.zeros((N, D), bool)
    for i in range(N):
        mask[i, rng.choice(D, lens[i], replace=False)] = True
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    y = np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32)
    w0, w = np.float32(0.1), (rng.standard_normal(D) * 0.2).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    print("rows shared by lane groups", row, K, half, flush=True)
    X = O.make_matrix(N, D, rowptr, col, val)
    m = B.Matrix(N, D, rowptr, col, val)
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.01, 0.02, 0.5, 1.0 / N, half_gather=half)
    Vr = V.astype(np.float16).astype(np.float32) if half else V
    a, G, q, yhat = O.forward(X, float(w0), w, Vr)
    l, r = O.loss_multiplier(O.LOSS_LOGISTIC, 1.0 / N, yhat, y)
    want = dict(yhat=yhat, a=a, G=G, q=q, r=r)
    d_w0, d_w, d_V = dev_params(w0, w, V)
    d_y = to_dev(y)
    out = {k: torch.full((N * (K if k == "G" else 1),), float("nan"), device="cuda") for k in want}
    loss_sum = m.fm_forward(p, d_y, d_w0, d_w, d_V, want_loss=True, **out)
    for k in want:
        assert_close(out[k].cpu().numpy().reshape(np.shape(want[k])), want[k], k)
    assert abs(loss_sum - l.sum()) <= 1e-5 * l.sum()
    met = m.fm_evaluate(p, d_y, d_w0, d_w, d_V)
    assert abs(met["rmse"] - np.sqrt(np.mean((yhat - y) ** 2))) <= 1e-5 * met["rmse"]
    m.fm_build_csc()
    m.fm_sgd_epoch(p, d_y, d_w0, d_w, d_V)
    g0, gw, gV = O.gradient(X, r, G, w, V, 0.01, 0.02)
    assert_close(d_w.cpu().numpy(), w - 0.5 * gw, "w")
    assert_close(d_V.cpu().numpy().reshape(D, K), V - 0.5 * gV, "V")
    assert abs(d_w0.item() - (0.1 - 0.5 * g0)) <= 1e-5
    m.close()


@pytest.mark.parametrize("K", [20, 32])  # five and eight of the eight lanes of a group
@pytest.mark.parametrize("N,row", [(203, 3), (203, 17), (203, 40), (262_144, 5), (262_145, 5)])  # up to 2^21 lanes and beyond
def test_half_gather_of_eight_lane_groups(N, row, K):
    """Scores and aggregates from half-precision V, empty and short rows among them, in small and in large launches."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8250 + N + row + K)
    D = 2 * row + 5
    lens = rng.integers(0, row + 3, N)
    rowptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = np.concatenate([np.sort(rng.permutation(D)[:n]) for n in lens[:203]] + [np.arange(n) for n in lens[203:]]).astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    w0, w = np.float32(0.1), (rng.standard_normal(D) * 0.2).astype(np.float32)
    V = (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    print("half of eight lanes", N, row, K, flush=True)
    a, G, q, yhat = O.forward(O.make_matrix(N, D, rowptr, col, val), float(w0), w, V.astype(np.float16).astype(np.float32))
    m = B.Matrix(N, D, rowptr, col, val)
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.0, 0.0, 0.5, 1.0 / N, half_gather=1)
    out = {k: torch.full((N * (K if k == "G" else 1),), float("nan"), device="cuda") for k in ("yhat", "a", "G", "q")}
    m.fm_forward(p, None, *dev_params(w0, w, V), **out)
    for k, want in dict(yhat=yhat, a=a, G=G, q=q).items():
        assert_close(out[k].cpu().numpy().reshape(np.shape(want)), want, k)
    m.close()


def test_postponed_steps_start_from_zero_in_every_epoch():
    """Epochs with postponed steps follow one another on one handle: strata, batches, strata captured by the caller and
    replayed between eager epochs, and with the steps taken at once in between.  Each meets the same epoch on a new handle."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8300)
    N, D, K, P = 90, 70, 8, 6
    mask = rng.random((N, D)) < 0.06
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    y = to_dev(np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32))
    w, V = (rng.standard_normal(D) * 0.2).astype(np.float32), (rng.standard_normal((D, K)) * 0.2).astype(np.float32)
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.05, 0.1, 0.5, 1.0 / N, 1)

    def handle():
        m = B.Matrix(N, D, rowptr, col, val)
        m.fm_build_csc()
        m.fm_partition(P)
        m.fm_partition_batches(P)
        return m

    m = handle()
    m.fm_set_option(B.FM_OPT_GRAPH, 0)
    dev = dev_params(np.float32(0.1), w, V)
    new = dev_params(np.float32(0.1), w, V)
    first = [t.clone() for t in dev]
    m.fm_stratified_epoch(p, y, *dev)  # the workspace is there before the capture
    for a, b in zip(dev, first):
        a.copy_(b)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        m.fm_stratified_epoch(p, y, *dev)
    for step in ("strata", "batches", "replay", "strata", "at once", "replay", "batches", "replay", "strata"):
        h = handle()
        h.fm_set_option(B.FM_OPT_GRAPH, 0)
        for q, s, args in ((m, step, dev), (h, "strata" if step == "replay" else step, new)):
            if s == "replay":
                g.replay()
            elif s == "batches":
                q.fm_minibatch_epoch(p, y, *args)
            else:
                q.fm_set_option(B.FM_OPT_LAZY_REG, 0 if s == "at once" else 1)
                q.fm_stratified_epoch(p, y, *args)
                q.fm_set_option(B.FM_OPT_LAZY_REG, 1)
        torch.cuda.synchronize()
        h.close()
        for a, b, what in zip(dev, new, ("w0", "w", "V")):
            assert torch.equal(a, b), f"{what} after {step}"
    m.close()


@pytest.mark.parametrize("K", [4, 8, 12, 16, 20, 28])
def test_packed_rows_where_planar_ones_are_the_default(K, monkeypatch):
    """Aggregates forced into packed rows: small gradients and, at K = 16, strata and batches take planar ones by themselves."""
    from paper_2004_13940_amd import binding as B
    build = B.Matrix.fm_build_csc

    def packed(m, *a, **k):
        m.fm_set_option(B.FM_OPT_AUX_PLANAR, 2)
        build(m, *a, **k)

    monkeypatch.setattr(B.Matrix, "fm_build_csc", packed)
    test_columns_of_every_length_around_the_rounds_and_the_item(K)
    for P in (1, 3):
        test_refresh_of_rows_of_every_length_around_the_rounds(K, P)


@pytest.mark.parametrize("N", [199_999, 200_003])  # full epochs planar, packed; strata and small batches planar
def test_layouts_of_the_aggregates_follow_one_another_on_a_handle(N):
    import torch
    from types import SimpleNamespace
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(N)
    D, K, row = 40, 16, 3
    col = np.sort(np.argpartition(rng.random((N, D)), row, axis=1)[:, :row], axis=1).astype(np.int32).ravel()
    wl = SimpleNamespace(N=N, D=D, K=K, rowptr=np.arange(N + 1, dtype=np.int64) * row, col=col,
                         val=rng.standard_normal(N * row).astype(np.float32),
                         y=np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32), w0=np.float32(0.1),
                         w=(rng.standard_normal(D) * 0.2).astype(np.float32),
                         V=(rng.standard_normal((D, K)) * 0.2 / np.sqrt(K)).astype(np.float32), loss=O.LOSS_LOGISTIC,
                         lambda_w=0.01, lambda_v=0.02, eta=0.5, loss_scale=1.0 / N, update_w0=1)
    print("layouts one after the other", N, flush=True)
    m, p, X, dev, host = run_full_epochs(B, wl, 1)
    m.fm_partition(3)
    host = run_stratified_epochs(B, wl, m, p, X, dev, host, 1, check_strata=True)
    m.fm_partition_batches(4)
    m.fm_minibatch_epoch(p, dev[3], *dev[:3])
    host = O.minibatch_epoch(X, wl.y, *host, B=4, update_w0=True, reg_share=True, loss=wl.loss, s=wl.loss_scale,
                             lambda_w=wl.lambda_w, lambda_v=wl.lambda_v, eta=wl.eta)[:3]
    m.fm_sgd_epoch(p, dev[3], *dev[:3])
    host = O.full_epoch(X, wl.y, *host, update_w0=True, loss=wl.loss, s=wl.loss_scale, lambda_w=wl.lambda_w,
                        lambda_v=wl.lambda_v, eta=wl.eta)[:3]
    m.fm_stratified_begin(p, dev[3], *dev[:3])
    a, G, q, yhat = O.forward(X, *host)
    out = {k: torch.full((N * (K if k == "G" else 1),), float("nan"), device="cuda") for k in "aGqr"}
    m.fm_get_aux(K, **out)
    r = O.loss_multiplier(wl.loss, wl.loss_scale, yhat, wl.y)[1]
    for k, want in dict(a=a, G=G, q=q, r=r).items():
        assert_close(out[k].cpu().numpy().reshape(np.shape(want)), want, k)
    gw, gV = torch.full((D,), float("nan"), device="cuda"), torch.full((D * K,), float("nan"), device="cuda")
    m.fm_gradient(p, out["r"], out["G"], dev[1], dev[2], grad_w=gw, grad_V=gV)
    _, wgw, wgV = O.gradient(X, r, G, host[1], host[2], wl.lambda_w, wl.lambda_v)
    assert_close(gw.cpu().numpy(), wgw, "grad_w")
    assert_close(gV.cpu().numpy().reshape(D, K), wgV, "grad_V")
    with pytest.raises(B.FMError):  # a gradient takes the aggregates that strata go on from
        m.fm_stratified_step(p, 0, dev[3], *dev[:3])
    m.close()


@pytest.mark.parametrize("N,K", [(64_512, 8), (64_513, 8), (64_513, 64), (131_073, 16), (359_999, 12), (360_000, 12), (360_000, 36)])
def test_panels_and_tiles_where_their_rules_change(N, K):
    """Plain segments below 64,513 rows, panels from there on, LDS tiles from 360,000; columns of every density."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(N + K)
    density = np.array([0.6, 0.2, 0.05, 0.02, 0.01, 0.004, 0.001, 5e-4, 2e-4, 1e-4, 0.0])
    D = len(density)
    mask = rng.random((N, D)) < density
    rowptr = np.concatenate([[0], np.cumsum(mask.sum(1))]).astype(np.int64)
    col = np.nonzero(mask)[1].astype(np.int32)
    val = rng.standard_normal(len(col)).astype(np.float32)
    r = (rng.standard_normal(N) / N).astype(np.float32)
    G = rng.standard_normal((N, K)).astype(np.float32)
    w, V = (rng.standard_normal(D) * 0.1).astype(np.float32), (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    print("panels and tiles", N, K, len(col), flush=True)
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_build_csc()
    m.fm_profile_enable(True)
    _, d_w, d_V = dev_params(np.float32(0), w, V)
    gw, gV = torch.full((D,), float("nan"), device="cuda"), torch.full((D * K,), float("nan"), device="cuda")
    m.fm_gradient(B.make_params(K, O.LOSS_SQUARED, 0.01, 0.02, 0.1), to_dev(r), to_dev(G.ravel()), d_w, d_V, grad_w=gw, grad_V=gV)
    torch.cuda.synchronize()
    assert m.fm_profile_read()["cols_tile"][0] == (1 if N >= 360_000 and K <= 32 else 0)
    _, wgw, wgV = O.gradient(O.make_matrix(N, D, rowptr, col, val), r, G, w, V, 0.01, 0.02)
    assert_close(gw.cpu().numpy(), wgw, "grad_w")
    assert_close(gV.cpu().numpy().reshape(D, K), wgV, "grad_V")
    m.close()


@pytest.mark.parametrize("captured", ["epoch", "strata", "batches"])
def test_aggregates_of_a_replayed_pass_are_read_in_its_layout(captured):
    """K = 16, 200,003 rows: full epochs keep packed rows, strata and batches planar ones.  What a pass leaves is read in that
    pass's layout whichever call was enqueued last: a graph runs whenever it is launched, and a capture runs nothing."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8400)
    N, D, K, row = 200_003, 40, 16, 3
    col = np.sort(np.argpartition(rng.random((N, D)), row, axis=1)[:, :row], axis=1).astype(np.int32).ravel()
    val = rng.standard_normal(N * row).astype(np.float32)
    rowptr = np.arange(N + 1, dtype=np.int64) * row
    w, V = (rng.standard_normal(D) * 0.2).astype(np.float32), (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    y = to_dev(np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32))
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.0, 0.0, 0.0, 1.0 / N, 0)  # steps of length zero: G and r of the parameters as given
    want = {}
    X = O.make_matrix(N, D, rowptr, col, val)
    for scale in (1.0, 2.0):
        _, G, _, yhat = O.forward(X, 0.1 * scale, w * scale, V * scale)
        want[scale] = (G, O.loss_multiplier(O.LOSS_LOGISTIC, 1.0 / N, yhat, y.cpu().numpy())[1])
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_build_csc()
    m.fm_partition(3)
    m.fm_partition_batches(3)
    calls = dict(epoch=m.fm_sgd_epoch, strata=m.fm_stratified_epoch, batches=m.fm_minibatch_epoch)
    one, two = (dev_params(np.float32(0.1 * s), w * s, V * s) for s in (1.0, 2.0))
    G, r = torch.empty(N * K, device="cuda"), torch.empty(N, device="cuda")

    def check(scale, what):
        G.fill_(float("nan")), r.fill_(float("nan"))
        m.fm_get_aux(K, G=G, r=r)
        assert_close(G.cpu().numpy().reshape(N, K), want[scale][0], f"G {what}")
        assert_close(r.cpu().numpy(), want[scale][1], f"r {what}")

    for name in calls:
        print("layouts under capture", captured, name, flush=True)
        calls[captured](p, y, *two)  # the workspace is there before the capture
        calls[name](p, y, *one)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            calls[captured](p, y, *two)
        check(1.0, f"after {name}, {captured} only captured")
        for turn in range(2):
            g.replay()
            check(2.0, f"after replay {turn} of {captured}")
            calls[name](p, y, *one)
            check(1.0, f"after {name} behind replay {turn} of {captured}")
            g.replay()
            check(2.0, f"after replay {turn} of {captured} behind {name}")
    m.close()


@pytest.mark.parametrize("N,D,row", [(1, 3, 2), (257, 9, 9), (40_000, 30, 3), (40_001, 30, 3), (200_001, 20, 2), (9_001, 20, 20)])
@pytest.mark.parametrize("K,option", [(4, 0), (12, 0), (16, 0), (16, 2), (28, 0), (8, 1), (32, 0), (6, 0)])
def test_gradient_leaves_what_it_was_given_in_the_aggregates(N, D, row, K, option):
    """Where packed rows exist (K a multiple of four up to 28, not switched off), whichever layout and kernels the call takes."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(N + 100 * K + option)
    col = np.sort(np.argpartition(rng.random((N, D)), row - 1, axis=1)[:, :row], axis=1).astype(np.int32).ravel()
    m = B.Matrix(N, D, np.arange(N + 1, dtype=np.int64) * row, col, rng.standard_normal(N * row).astype(np.float32))
    m.fm_set_option(B.FM_OPT_AUX_PLANAR, option)
    m.fm_build_csc()
    p = B.make_params(K, O.LOSS_SQUARED, 0.01, 0.02, 0.1)
    _, w, V = dev_params(0.0, rng.standard_normal(D), rng.standard_normal((D, K)).ravel())
    for turn in range(2):
        r, G = to_dev(rng.standard_normal(N)), to_dev(rng.standard_normal(N * K))
        m.fm_gradient(p, r, G, w, V, grad_w=torch.empty(D, device="cuda"), grad_V=torch.empty(D * K, device="cuda"))
        gotr, gotG = torch.empty(N, device="cuda"), torch.empty(N * K, device="cuda")
        if option == 1 or K % 4 or K > 28:
            with pytest.raises(B.FMError):
                m.fm_get_aux(K, G=gotG, r=gotr)
            continue
        m.fm_get_aux(K, G=gotG, r=gotr)
        assert torch.equal(gotr, r) and torch.equal(gotG, G)
        with pytest.raises(B.FMError):
            m.fm_get_aux(K, a=gotr)
    m.close()


@pytest.mark.parametrize("N,batches", [(3, 5), (3, 1), (700, 3)])
@pytest.mark.parametrize("K", [4, 8, 32])
@pytest.mark.parametrize("dense", [0, 1])
def test_batches_of_a_table_leave_their_layout(N, batches, K, dense):
    """K = 4: gradients of the dense kernels keep planar rows, batches packed ones, and the first pass over rows writes the word
    for all, which is not the first batch's where that is empty.  K = 8 and 32: planar always, no word."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8500 + N + K)
    D = 5
    rowptr, col = np.arange(N + 1, dtype=np.int64) * D, np.tile(np.arange(D, dtype=np.int32), N)
    val = rng.standard_normal(N * D).astype(np.float32)
    y = rng.standard_normal(N).astype(np.float32)
    w, V = (rng.standard_normal(D) * 0.2).astype(np.float32), (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    _, wantG, _, yhat = O.forward(O.make_matrix(N, D, rowptr, col, val), 0.1, w, V)
    wantr = O.loss_multiplier(O.LOSS_SQUARED, 1.0 / N, yhat, y)[1]
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_set_option(B.FM_OPT_DENSE_ROWS, dense)
    m.fm_build_csc()
    m.fm_partition_batches(batches)
    p = B.make_params(K, O.LOSS_SQUARED, 0.0, 0.0, 0.0, 1.0 / N, 0)  # steps of length zero
    for turn in range(2):
        params = dev_params(np.float32(0.1), w, V)
        m.fm_gradient(p, to_dev(rng.standard_normal(N)), to_dev(rng.standard_normal(N * K)), *params[1:],
                      grad_w=torch.empty(D, device="cuda"), grad_V=torch.empty(D * K, device="cuda"))
        m.fm_minibatch_epoch(p, to_dev(y), *params)
        G, r = torch.empty(N * K, device="cuda"), torch.empty(N, device="cuda")
        m.fm_get_aux(K, G=G, r=r)
        assert_close(G.cpu().numpy().reshape(N, K), wantG, "G")
        assert_close(r.cpu().numpy(), wantr, "r")
    m.close()


def test_partial_sums_of_one_stratum_or_batch_are_held_at_a_time():
    """2,000 columns times strata of two items each where all columns have 65,000 as a whole: the workspace has rows for the
    larger of one stratum's and the whole matrix's items, and strata that reuse the rows step like the oracle's."""
    import torch
    from types import SimpleNamespace
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(8500)
    N, D, K, row, P = 200_000, 1_000, 64, 20, 96  # 2,083 rows to a block: not summed whole; 41 entries to a column and stratum
    col = (np.arange(row) * (D // row) + rng.integers(0, D // row, (N, row))).astype(np.int32).ravel()
    wl = SimpleNamespace(N=N, D=D, K=K, P=P, rowptr=np.arange(N + 1, dtype=np.int64) * row, col=col,
                         val=rng.standard_normal(N * row).astype(np.float32),
                         y=np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32), w0=np.float32(0.1),
                         w=(rng.standard_normal(D) * 0.2).astype(np.float32),
                         V=(rng.standard_normal((D, K)) * 0.02).astype(np.float32), loss=O.LOSS_LOGISTIC,
                         lambda_w=0.01, lambda_v=0.02, eta=0.5, loss_scale=1.0 / N, update_w0=1)
    m = B.Matrix(N, D, wl.rowptr, col, wl.val)
    m.fm_build_csc()
    m.fm_partition(P)
    m.fm_partition_batches(P)
    dev = (*dev_params(wl.w0, wl.w, wl.V), to_dev(wl.y))
    p = B.make_params(K, wl.loss, wl.lambda_w, wl.lambda_v, wl.eta, wl.loss_scale, 1)
    X = O.make_matrix(N, D, wl.rowptr, col, wl.val)
    torch.cuda.synchronize()
    B.fm_trim()
    free = torch.cuda.mem_get_info()[0]
    print("partial sums of one stratum", flush=True)
    host = run_stratified_epochs(B, wl, m, p, X, dev, (float(wl.w0), wl.w, wl.V), 1)
    held = free - torch.cuda.mem_get_info()[0]
    rows = N * (K + 3) * 4 + (row * N // 64 + D) * 96 * 4  # aggregates, and 96 floats for each item of the whole matrix
    assert held <= rows + (16 << 20), (held, rows)  # rows for all strata would be 190,000 x 384 bytes
    m.fm_minibatch_epoch(p, dev[3], *dev[:3])
    host = O.minibatch_epoch(X, wl.y, *host, B=P, update_w0=True, reg_share=True, loss=wl.loss, s=wl.loss_scale,
                             lambda_w=wl.lambda_w, lambda_v=wl.lambda_v, eta=wl.eta)[:3]
    assert_close(dev[1].cpu().numpy(), host[1], "w after batches")
    assert_close(dev[2].cpu().numpy().reshape(D, K), host[2], "V after batches")
    m.close()


@pytest.mark.parametrize("N,density", [(200_000, 0.05), (200_000, 0.005), (131_072, 0.02), (400_001, 0.0025), (70_000, 0.3)])
@pytest.mark.parametrize("K", [4, 8, 16, 28, 32, 60, 64, 128, 2])  # packed and planar rows, groups of up to eight lanes and wider ones
def test_sums_of_long_columns_are_rounded_a_few_times(N, density, K):
    """Sums of values of one sign whose products are exact: only additions round.  Items of n entries, at least 24 to a column (a
    panel each, up to 128 entries), are added up in fp32 by at most 16 entries, in fp64 from there on, and rounded once.  With u
    the rounding of one addition an item is off by u sqrt(1 + 16 / 3 / (n / 16)), the column by sqrt(items) less.  It shows in
    the share of results that are not the nearest float: sqrt(2 / pi) times that error in units of the last place, where u is
    0.31 of one (2^-23 / sqrt(12), on the average over the mantissas of partial and final sums).  Single chains of 128 would
    be at 0.13 to 0.18 in the first case, where the bound is 0.06 to 0.08."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(N + K)
    D = 48
    cols = [np.sort(rng.choice(N, int(N * density), replace=False)) for _ in range(D)]
    row = np.concatenate(cols)
    col = np.repeat(np.arange(D, dtype=np.int32), [len(c) for c in cols])
    order = np.argsort(row, kind="stable")
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=N))]).astype(np.int64)
    m = B.Matrix(N, D, rowptr, col[order], np.ones(len(row), np.float32))
    m.fm_set_tuning(seg=128)  # what matrices of 8e6 entries and more have
    m.fm_build_csc()
    G = (rng.random((N, K)) + 0.5).astype(np.float32)
    zero = torch.zeros(D * K, device="cuda")
    gV = torch.full((D * K,), float("nan"), device="cuda")
    print("rounding of long columns", N, density, K, flush=True)
    m.fm_gradient(B.make_params(K, O.LOSS_SQUARED, 0.0, 0.0, 0.1), torch.full((N,), 2.0 ** -10, device="cuda"), to_dev(G.ravel()),
                  torch.zeros(D, device="cuda"), zero, grad_V=gV)
    want = np.stack([G[c].astype(np.float64).sum(0) * 2.0 ** -10 for c in cols]).astype(np.float32)
    share = float(np.mean(gV.cpu().numpy().reshape(D, K) != want))
    items = 24 * -(-N * density // (24 * 128))
    rounds = max(N * density / items / 16, 1.0)
    want = np.sqrt(2 / np.pi) * 0.31 * np.sqrt((1 + 16 / 3 / rounds) / items)
    bound = 1.5 * want + 3 * np.sqrt(want / (D * K))  # items are not all of one length; D K results are a sample
    print("share", share, "bound", bound, flush=True)
    assert share <= bound
    m.close()


@pytest.mark.parametrize("call,N,parts", [("batches", 400_000, 1), ("batches", 400_001, 1), ("strata", 400_000, 1), ("strata", 400_001, 1),
                                          ("strata", 2_200_000, 2)])
def test_layouts_where_their_rules_change(call, N, parts):
    """K = 16: batches and a single block of strata of up to 400,000 rows planar, larger ones packed; several blocks planar at any size."""
    import torch
    from paper_2004_13940_amd import binding as B
    rng = np.random.default_rng(N)
    D, K, row = 30, 16, 2
    col = (np.arange(row) * (D // row) + rng.integers(0, D // row, (N, row))).astype(np.int32).ravel()
    rowptr, val = np.arange(N + 1, dtype=np.int64) * row, rng.standard_normal(N * row).astype(np.float32)
    y = np.where(rng.random(N) < 0.5, 1.0, -1.0).astype(np.float32)
    w, V = (rng.standard_normal(D) * 0.2).astype(np.float32), (rng.standard_normal((D, K)) * 0.1).astype(np.float32)
    m = B.Matrix(N, D, rowptr, col, val)
    m.fm_build_csc()
    p = B.make_params(K, O.LOSS_LOGISTIC, 0.01, 0.02, 0.5, 1.0 / N, 1)
    kw = dict(loss=O.LOSS_LOGISTIC, s=1.0 / N, lambda_w=0.01, lambda_v=0.02, eta=0.5)
    X = O.make_matrix(N, D, rowptr, col, val)
    dev, d_y = dev_params(np.float32(0.1), w, V), to_dev(y)
    print("layouts at their lines", call, N, parts, flush=True)
    if call == "batches":
        m.fm_partition_batches(parts)
        m.fm_minibatch_epoch(p, d_y, *dev)
        _, G, _, yhat = O.forward(X, 0.1, w, V)  # one batch: the aggregates that the only step was taken from
        host = O.minibatch_epoch(X, y, 0.1, w, V, B=parts, update_w0=True, reg_share=True, **kw)[:3]
    else:
        m.fm_partition(parts)
        m.fm_stratified_epoch(p, d_y, *dev)
        held = {}  # the aggregates as the last stratum refreshed them
        host = O.stratified_epoch(X, y, 0.1, w, V, P=parts, update_w0=True, final_objective=False,
                                  on_stratum=lambda s, st: held.update(G=st["G"].copy()), **kw)[:3]
        G = held["G"]
    G_dev = torch.full((N * K,), float("nan"), device="cuda")
    m.fm_get_aux(K, G=G_dev)
    assert_close(G_dev.cpu().numpy().reshape(N, K), G, "G")
    assert_close(dev[1].cpu().numpy(), host[1], "w")
    assert_close(dev[2].cpu().numpy().reshape(D, K), host[2], "V")
    m.close()
