"""GPU parity at the edges of the launch shapes: column counts that are no multiple of the columns a
lane owns, slices that end with a few columns, work lists at the edges of their blocks."""
import numpy as np
import pytest

import oracle
from paper_2307_05740_amd import binding, synth
from tests.test_gpu_parity import TOL, assert_within, csr_of, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,kc", [(5, 0), (9, 0), (63, 16), (65, 64), (66, 64), (67, 64), (127, 32), (257, 0), (259, 0)])
@pytest.mark.parametrize("fuse", [0, 1])
def test_last_lane_shares_columns(torch, k, kc, fuse):
    """The last lane of a row reaches back into its neighbour's columns; with separate levels the
    launches add to Y, where two slices must not both own a column."""
    w = synth.make_config(2, 8)
    X = synth.normal_matrix(w.n, k, seed=11)
    opt = binding.arrow_options_default(fuse_levels=fuse, kc=kc)
    op = binding.ArrowSpMM(*csr_of(w), w.b, options=opt)
    Y = torch.full((w.n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    Yref, B = oracle.spmm(*csr_of(w), X)
    assert_within(Y.cpu().numpy(), Yref, B)
    op.close()


@pytest.mark.parametrize("k", [5, 6, 7, 33, 261])
def test_shared_columns_count_once_in_dot_products(torch, k):
    """Infinite factors in the last columns stay infinite (a shared column is dropped, not multiplied by 0)."""
    w = synth.make_config(0, 2)
    U = synth.normal_matrix(w.n, k, seed=12)
    V = synth.normal_matrix(w.n, k, seed=13)
    V[::7, k - 1] = np.inf
    V[3::11, k - 3] = -np.inf
    op = binding.ArrowSpMM(*csr_of(w), w.b)
    S = op.sddmm(torch.from_numpy(U).cuda(), torch.from_numpy(V).cuda()).cpu().numpy()
    op.close()
    rows = np.repeat(np.arange(w.n), np.diff(w.rowptr))
    with np.errstate(invalid="ignore"):
        ref = w.vals.astype(np.float64) * np.einsum("ij,ij->i", U[rows].astype(np.float64), V[w.colidx].astype(np.float64))
    assert np.array_equal(np.isnan(S), np.isnan(ref)) and np.array_equal(np.isinf(S), np.isinf(ref))
    assert np.array_equal(S[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
    fin = np.isfinite(ref)
    bound = np.abs(w.vals[fin]) * np.einsum("ij,ij->i", np.abs(U[rows[fin]]), np.abs(V[w.colidx[fin]]))
    assert np.all(np.abs(S[fin] - ref[fin]) <= TOL * bound)


@pytest.mark.parametrize("n", [1, 7, 64, 65, 513, 20000])
@pytest.mark.parametrize("k", [1, 4, 16, 128])
def test_short_work_lists(torch, n, k):
    """Lists shorter than a workgroup's share, rows without entries in between, one row of middle length."""
    rng = np.random.default_rng(n)
    length = np.where(rng.random(n) < 0.4, 0, rng.integers(1, min(n, 5) + 1, n))
    length[n // 2] = min(n, 40)
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    colidx = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in length]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=14)
    op = binding.ArrowSpMM(rowptr, colidx, vals, max(1, n // 8))
    binding.arrow_self_check(op.h)
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)
    op.close()


@pytest.mark.parametrize("k", [1, 4, 16, 64, 68, 96, 128, 130, 200, 256])
def test_rows_shared_by_the_wavefronts_of_a_workgroup(torch, k):
    """Row lengths around what a lane group, a wavefront, a workgroup and several of them take."""
    n = 6000
    length = np.full(n, 3)
    for i, m in enumerate([0, 1, 16, 17, 48, 49, 255, 256, 257, 258, 511, 1023, 1024, 1025, 2047, 2048, 2049, 4096, 4097, n]):
        length[7 * i + 5] = m
    rng = np.random.default_rng(5)
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    colidx = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in length]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=15)
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    Xd = torch.from_numpy(X).cuda()
    for opt in (None, binding.arrow_options_default(chunk_nnz=40), binding.arrow_options_default(window_rows=1024)):
        op = binding.ArrowSpMM(rowptr, colidx, vals, 500, options=opt)
        binding.arrow_self_check(op.h)
        Y = torch.full((n, k), float("nan"), device="cuda")
        op.spmm(Xd, Y)
        assert_within(Y.cpu().numpy(), Yref, B)
        op.close()


@pytest.mark.parametrize("l", [1, 2, 3, 4, 5, 7])
@pytest.mark.parametrize("room", [False, True])
def test_chained_products_with_and_without_a_second_buffer(torch, l, room):
    w = synth.make_config(0, 3)
    op = binding.ArrowSpMM(*csr_of(w), w.b)
    X = synth.normal_matrix(w.n, 7, seed=16)
    Xl = X.copy()
    for _ in range(l):
        Xl = op.spmm(torch.from_numpy(Xl).cuda()).cpu().numpy()
    Xd = torch.from_numpy(X).cuda()
    nbytes = binding.arrow_workspace_bytes(op.h, 7) + (-(-w.n * 7 * 4 // 256) * 256 if room else 0)
    ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    binding.arrow_set_workspace(op.h, ws.data_ptr(), nbytes)
    binding.arrow_spmm_iter(op.h, Xd.data_ptr(), 7, l, torch.cuda.current_stream().cuda_stream)
    assert np.array_equal(Xd.cpu().numpy().view(np.uint32), Xl.view(np.uint32))
    op.close()


@pytest.mark.parametrize("k", [1, 5, 8, 16, 20, 33, 64, 65, 130])
@pytest.mark.parametrize("span", [96, 700, 2500, 4096])
@pytest.mark.parametrize("fuse", [0, 1])
def test_lds_windows(torch, k, span, fuse):
    """Windows from narrow to the widest allowed, rows of 0 to 100 entries inside them and 0 to 7 outside."""
    b, blocks = 4096, 3
    n = b * blocks
    rng = np.random.default_rng(span)
    rows, cols = [], []
    for i in range(b, n):
        m = int(rng.integers(0, 101)) if i % 50 else 0
        lo = min(max(i - span // 2, i // b * b), (i // b + 1) * b - span)
        c = np.union1d(lo + rng.choice(span, min(m, span), replace=False), rng.choice(b, int(rng.integers(0, 8)), replace=False))
        rows.append(np.full(len(c), i))
        cols.append(c)
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int64)
    vals = rng.uniform(-1, 1, len(cols)).astype(np.float32)
    opt = binding.arrow_options_default(window_span=4096, window_tile_rows=500, window_level_share=0.0, fuse_levels=fuse,
                                        bfs_tail=0, separators=0)
    opt.window_reuse = 0.5
    op = binding.ArrowSpMM(rowptr, cols.astype(np.int32), vals, b, options=opt)
    binding.arrow_self_check(op.h)
    assert sum(L["nnz_window"] for L in op.levels()) > 0
    X = synth.normal_matrix(n, k, seed=17)
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    Yref, B = oracle.spmm(rowptr, cols.astype(np.int32), vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)
    op.close()


@pytest.mark.parametrize("R", [1, 3, 4, 9, 32, 64, 130, 260])
@pytest.mark.parametrize("I", [3, 2046, 2300])
def test_mttkrp_fibre_lengths(torch, I, R):
    """Few slices (a workgroup per item) and many (a wavefront per item); fibres of 1 to 130 entries, equally
    long ones next to single ones, empty slices, a slice of several items."""
    rng = np.random.default_rng(I)
    J, K = 300, 140
    ti, tj, tk = [], [], []
    for i in range(I):
        if i % 5 == 4:
            continue
        for f in range(260 if i == 1 else int(rng.integers(1, 7))):
            j = f if i == 1 else int(rng.integers(0, J))
            m = [1, 1, 2, 3, 4, 5, 8, 9][int(rng.integers(0, 8))] if i != 2 else int(rng.integers(60, 131))
            ti += [i] * m
            tj += [j] * m
            tk += list(rng.integers(0, K, m))
    tv = rng.uniform(-1, 1, len(ti)).astype(np.float32)
    ti, tj, tk = (np.array(x, dtype=np.int32) for x in (ti, tj, tk))
    Bf, Cf = synth.normal_matrix(J, R, seed=18), synth.normal_matrix(K, R, seed=19)
    op = binding.Csf3Mttkrp((I, J, K), ti, tj, tk, tv)
    A = torch.full((I, R), float("nan"), device="cuda")
    op.mttkrp(torch.from_numpy(Bf).cuda(), torch.from_numpy(Cf).cuda(), A)
    Aref, E = oracle.mttkrp((I, J, K), ti, tj, tk, tv, Bf, Cf)
    assert_within(A.cpu().numpy(), Aref, E)
    op.close()


@pytest.mark.parametrize("k", [1, 6, 32, 72])
@pytest.mark.parametrize("n,full", [(1024 * 64, True), (1024 * 64 + 301, False), (4096 * 64 + 301, True), (300001, False)])
def test_many_batches_of_short_rows(torch, n, full, k):
    """Short rows only, enough of them for several batches per workgroup: batches that fill the staging
    buffer to the last entry, rows without entries, an incomplete last batch."""
    rng = np.random.default_rng(n)
    length = np.full(n, 16) if full else rng.integers(0, 17, n)
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    row = np.repeat(np.arange(n), length)
    step = 1 + rng.integers(0, 3, n)
    colidx = (np.clip(np.arange(n) - 20, 0, n - 64)[row] + (np.arange(len(row)) - rowptr[row]) * step[row]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=21)
    op = binding.ArrowSpMM(rowptr, colidx, vals, 4096)
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


@pytest.mark.parametrize("k", [1, 6, 32, 72])
@pytest.mark.parametrize("n,full", [(1024 * 64, True), (1024 * 64 + 1, True), (75011, False), (4096 * 64 + 301, True)])
def test_many_batches_of_short_rows_without_window_tiles(torch, n, full, k):
    """The same rows with the window tiles off, which take most of them above: at least as many short rows as the
    kernel that copies batches ahead begins at (1024 batches of 64)."""
    rng = np.random.default_rng(n)
    length = np.full(n, 16) if full else rng.integers(0, 17, n)
    assert np.count_nonzero(length) >= 1024 * 64
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    row = np.repeat(np.arange(n), length)
    step = 1 + rng.integers(0, 3, n)
    colidx = (np.clip(np.arange(n) - 20, 0, n - 64)[row] + (np.arange(len(row)) - rowptr[row]) * step[row]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=21)
    op = binding.ArrowSpMM(rowptr, colidx, vals, 4096, options=binding.arrow_options_default(window_span=0))
    level = op.levels()[0]
    assert level["short_rows"] == n and level["chunks"] == 0 and level["window_tiles"] == 0
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


@pytest.mark.parametrize("k", [33, 50, 64, 128, 200])
@pytest.mark.parametrize("n,pieces,short", [(60, 3, 20), (3000, 501, 1999), (11000, 2000, 8321), (15000, 4001, 8601)])
@pytest.mark.parametrize("fuse", [0, 1])
def test_pieces_of_a_wavefront_each(torch, n, pieces, short, k, fuse):
    """Rows of 17 to 48 entries that four lane groups share, or that they have one by one, beside short rows and rows without entries."""
    rng = np.random.default_rng(n + k)
    length = np.zeros(n, np.int64)
    length[:pieces] = rng.integers(17, 49, pieces)
    length[pieces:pieces + short] = rng.integers(1, 17, short)
    rng.shuffle(length)
    colidx = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in length]).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=34)
    op = binding.ArrowSpMM(rowptr, colidx, vals, max(1, n // 16), options=binding.arrow_options_default(fuse_levels=fuse))
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    assert_within(Y.cpu().numpy(), *oracle.spmm(rowptr, colidx, vals, X))
    op.close()


@pytest.mark.parametrize("k", [8, 20, 70])
@pytest.mark.parametrize("n,b", [(200, 64), (4000, 500), (17 * 256 + 3, 256)])
@pytest.mark.parametrize("fuse", [0, 1])
def test_tiles_shared_by_workgroups(torch, n, b, k, fuse):
    """Fewer window tiles than compute units: workgroups take parts of a tile's rows, some of them none."""
    rng = np.random.default_rng(n)
    rowptr = (np.arange(n + 1) * 30).astype(np.int64)
    lo = np.arange(n) // b * b
    hi = np.minimum(lo + b, n)
    colidx = np.concatenate([np.sort(rng.permutation(hi[i] - lo[i])[:30] + lo[i]) if hi[i] - lo[i] >= 30 else np.arange(30)
                             for i in range(n)]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=22)
    op = binding.ArrowSpMM(rowptr, colidx, vals, b, options=binding.arrow_options_default(fuse_levels=fuse))
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


@pytest.mark.parametrize("R", [14, 41, 128])
@pytest.mark.parametrize("I,longest", [(2047, 900), (2049, 60), (2049, 900), (4097, 900), (8190, 900)])
def test_mttkrp_items_of_unequal_length(torch, I, longest, R):
    """Slices of one entry beside one that is cut into several items of about the same length."""
    rng = np.random.default_rng(longest)
    J, K = 300, 200
    hub = rng.choice(J * K, longest, replace=False)
    ti = np.concatenate([np.arange(I), np.full(longest, I // 2)]).astype(np.int32)
    tj = np.concatenate([rng.integers(0, J, I), hub // K]).astype(np.int32)
    tk = np.concatenate([rng.integers(0, K, I), hub % K]).astype(np.int32)
    tv = rng.uniform(-1, 1, len(ti)).astype(np.float32)
    Bm, Cm = synth.normal_matrix(J, R, seed=23), synth.normal_matrix(K, R, seed=24)
    h = binding.Csf3Mttkrp((I, J, K), ti, tj, tk, tv, device="cuda:0")
    A = h.mttkrp(torch.from_numpy(Bm).cuda(), torch.from_numpy(Cm).cuda()).cpu().numpy()
    h.close()
    ref, bound = np.zeros((I, R)), np.zeros((I, R))
    term = tv[:, None].astype(np.float64) * Bm[tj] * Cm[tk]
    np.add.at(ref, ti, term)
    np.add.at(bound, ti, np.abs(term))
    assert_within(A, ref, bound)


@pytest.mark.parametrize("k", [4, 33, 64, 65, 128, 200, 300])
def test_dot_products_of_long_rows_shared_by_wavefronts(torch, k):
    """A few long rows of any length beside short ones: wavefronts share a chunk, some of them get nothing of it."""
    n = 700
    rng = np.random.default_rng(k)
    length = rng.integers(0, 4, n)
    length[:12] = [17, 18, 33, 49, 64, 100, 255, 256, 257, 511, 699, 700]
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    colidx = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in length]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    U, V = synth.normal_matrix(n, k, seed=25), synth.normal_matrix(n, k, seed=26)
    op = binding.ArrowSpMM(rowptr, colidx, vals, 64)
    S = op.sddmm(torch.from_numpy(U).cuda(), torch.from_numpy(V).cuda()).cpu().numpy()
    op.close()
    rows = np.repeat(np.arange(n), length)
    prod = U[rows].astype(np.float64) * V[colidx]
    assert_within(S, vals * prod.sum(1), np.abs(vals) * np.abs(prod).sum(1))


def window_operand(b=64, blocks=9):
    """Blocks of b rows with 1 to 33 entries inside the row's block and three anywhere."""
    n = b * blocks
    rng = np.random.default_rng(27)
    cols = []
    for i in range(n):
        inside = i // b * b + rng.choice(b, 1 + i % 33, replace=False)
        cols.append(np.union1d(inside, rng.integers(0, n, 3)))
    rowptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    colidx = np.concatenate(cols).astype(np.int32)
    return n, b, rowptr, colidx, rng.uniform(-1, 1, len(colidx)).astype(np.float32)


@pytest.mark.parametrize("k", [8, 24, 64, 70])
@pytest.mark.parametrize("fuse", [0, 1])
def test_non_finite_rows_of_a_window_stay_with_their_readers(torch, k, fuse):
    """The first row of every window (and another one) holds an infinity or NaN: rows without an entry
    in its column stay finite, however many of a batch's places they leave empty."""
    n, b, rowptr, colidx, vals = window_operand()
    opt = binding.arrow_options_default(window_level_share=0.0, fuse_levels=fuse)
    opt.window_reuse = 0.5
    op = binding.ArrowSpMM(rowptr, colidx, vals, b, options=opt)
    binding.arrow_self_check(op.h)
    levels = op.levels()
    assert levels[0]["window_tiles"] > 0 and (fuse or any(L["window_tiles"] for L in levels[1:]))
    X = synth.normal_matrix(n, k, seed=28)
    rng = np.random.default_rng(k)
    for level in range(len(levels)):
        perm, r, c, _ = binding.arrow_export_level(op.h, level)
        diag = c[(r >= b) & (c >= b) & (r // b == c // b)]
        for block in np.unique(diag // b):
            inside = diag[diag // b == block]
            for q, bad in ((inside.min(), np.inf), (rng.choice(inside), (-np.inf, np.nan)[block % 2])):
                X[perm[q], (q + level) % k] = bad
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Y = Y.cpu().numpy()
    with np.errstate(invalid="ignore"):
        term = vals[:, None].astype(np.float64) * X[colidx]
        ref = np.add.reduceat(term, rowptr[:-1])                  # no row is empty
    bound = np.add.reduceat(np.abs(np.where(np.isfinite(term), term, 0.0)), rowptr[:-1])
    fin = np.isfinite(ref)
    assert 0.5 < fin.mean() < 1.0
    assert np.array_equal(np.isnan(Y), np.isnan(ref)) and np.array_equal(Y[np.isinf(ref)], ref[np.isinf(ref)].astype(np.float32))
    assert np.all(np.abs(Y[fin] - ref[fin]) <= TOL * bound[fin])


@pytest.mark.parametrize("I,J,K,nnz,R", [
    (600, 1700, 1300, 700_000, 1), (600, 1700, 1300, 700_000, 2), (600, 1700, 1300, 700_000, 3),
    (600, 1700, 1300, 700_000, 4), (600, 1700, 1300, 700_000, 7), (513, 5000, 300, 700_000, 33),
    (520, 600, 9599, 1_900_000, 6), (520, 9899, 300, 1_200_000, 6), (520, 900, 900, 535_000, 130),
    (600, 700, 700, 600_000, 520), (600, 700, 700, 600_000, 1030), (230, 400, 1500, 260_000, 9)])
def test_mttkrp_factors_in_lds(torch, I, J, K, nnz, R):
    """The form for factors that fit the LDS, up to the last row of it (J + K + 1 = 10200): fibres of one entry
    and of more than a segment holds, a slice of several items (but for the smallest), slices of one entry and without any,
    rows of the factors that no entry refers to (infinite here), duplicates, entries in any order."""
    rng = np.random.default_rng(I + R)
    i = rng.integers(0, I, nnz)
    i[i % 97 == 5] = 1                                       # a hub slice, empty ones
    j, k = rng.integers(1, J - 1, nnz), rng.integers(1, K - 1, nnz)
    i[:300], j[:300] = 7, 1                                  # one fibre of five segments
    i[300:700], j[300:700], k[300:700] = 8, J - 2, K - 2     # a coordinate that repeats
    drop = (i >= 20) & (i < 23)
    i, j, k = i[~drop], j[~drop], k[~drop]
    only = np.flatnonzero(i == 30)[1:]                       # a slice of a single entry
    i[only] = 31
    v = rng.uniform(-1, 1, len(i)).astype(np.float32)
    i, j, k = (x.astype(np.int32) for x in (i, j, k))
    B, C = synth.normal_matrix(J, R, seed=31), synth.normal_matrix(K, R, seed=32)
    Aref, E = oracle.mttkrp((I, J, K), i, j, k, v, B, C)
    B[[0, -1]], C[[0, -1]] = np.inf, np.nan                  # what no entry refers to has no effect
    op = binding.Csf3Mttkrp((I, J, K), i, j, k, v)
    assert op.info["items"] == I - op.info["split_rows"] + op.info["partials"]
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_FACTORS_IN_LDS
    A = torch.full((I, R), float("nan"), device="cuda")
    op.mttkrp(torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda(), A)
    assert_within(A.cpu().numpy(), Aref, E)
    first = A.clone()
    op.mttkrp(torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda(), A)
    assert torch.equal(first, A)
    op.close()


@pytest.mark.parametrize("I,J,K,nnz,R", [
    (2000, 2549, 2550, 1_500_000, 57), (2000, 2549, 2551, 1_500_000, 57), (2100, 1500, 2000, 6_000_000, 8),
    (2000, 900, 1200, 1_500_000, 16), (1300, 1100, 700, 1_200_000, 63), (1300, 1100, 700, 1_200_000, 64), (600, 4000, 1500, 3_000_000, 1024),
    (200, 900, 800, 200_000, 6145)])
def test_mttkrp_factors_in_lds_eight_columns(torch, I, J, K, nnz, R):
    """The same form where eight columns at a time take less (not in the second and the last but one, whose rows do not fit so): up
    to the last row that fits (J + K + 1 = 5100), ranks that are no multiple of eight, more slices of columns than four rounds of workgroups."""
    rng = np.random.default_rng(I + R)
    i, j, k = (rng.integers(0, d, nnz).astype(np.int32) for d in (I, J, K))
    i[:9000] = 1                                             # a slice of several items
    j[:300], j[300:600], k[300:600] = J - 1, 0, K - 1        # a fibre of several segments, a coordinate that repeats
    v = rng.uniform(-1, 1, nnz).astype(np.float32)
    B, C = synth.normal_matrix(J, R, seed=31), synth.normal_matrix(K, R, seed=32)
    Aref, E = oracle.mttkrp((I, J, K), i, j, k, v, B, C)
    op = binding.Csf3Mttkrp((I, J, K), i, j, k, v)
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_FACTORS_IN_LDS and op.info["partials"] > 0
    A = torch.full((I, R), float("nan"), device="cuda")
    op.mttkrp(torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda(), A)
    assert_within(A.cpu().numpy(), Aref, E)
    first = A.clone()
    op.mttkrp(torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda(), A)
    assert torch.equal(first, A)
    op.close()


@pytest.mark.parametrize("lanes", [64, 61])
def test_mttkrp_steps_of_the_last_block(torch, lanes):
    """Items whose last block of eight steps has one to eight of them, with a factor whose first and last rows are infinite where
    no entry refers to them; eight columns at a time give the bits of four."""
    I, J, K, R = 2000, 1000, 900, 64
    rng = np.random.default_rng(lanes)
    length = 1 + np.arange(I) % 9                            # of the `lanes` fibres of a slice: 2 to 10 steps
    i = np.repeat(np.arange(I), lanes * length)
    j = np.concatenate([np.repeat(1 + rng.choice(J - 2, lanes, replace=False), n) for n in length])
    k = rng.integers(1, K - 1, len(i))
    v = rng.uniform(-1, 1, len(i)).astype(np.float32)
    i, j, k = (x.astype(np.int32) for x in (i, j, k))
    B, C = synth.normal_matrix(J, R, seed=41), synth.normal_matrix(K, R, seed=42)
    Aref, E = oracle.mttkrp((I, J, K), i, j, k, v, B, C)
    B[[0, -1]], C[[0, -1]] = np.inf, np.nan
    op = binding.Csf3Mttkrp((I, J, K), i, j, k, v)
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_FACTORS_IN_LDS and op.info["partials"] == 0
    A = torch.full((I, R), float("nan"), device="cuda")
    op.mttkrp(torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda(), A)
    assert_within(A.cpu().numpy(), Aref, E)
    four = op.mttkrp(torch.from_numpy(np.ascontiguousarray(B[:, :4])).cuda(), torch.from_numpy(np.ascontiguousarray(C[:, :4])).cuda())
    assert np.array_equal(four.cpu().numpy().view(np.uint32), A[:, :4].contiguous().cpu().numpy().view(np.uint32))
    op.close()


@pytest.mark.parametrize("k", [1, 6, 20, 33, 128, 260])
@pytest.mark.parametrize("fuse", [0, 1])
def test_rows_of_many_partial_vectors(torch, k, fuse):
    """Hub rows next to each other and far apart, long enough for the wavefronts of a workgroup to share their
    partial vectors (from 32 of them on at k = 128), beside split rows of a few."""
    n = 140001
    rng = np.random.default_rng(k)
    length = rng.integers(0, 3, n)
    length[[0, 1, 2, 3, 5, 70000]] = [140000, 30000, 100000, 9000, 139999, 60000]
    length[1000:1040] = 600
    rowptr = np.concatenate([[0], np.cumsum(length)]).astype(np.int64)
    colidx = np.concatenate([np.sort(rng.choice(n, m, replace=False)) for m in length]).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=33)
    op = binding.ArrowSpMM(rowptr, colidx, vals, 1024, options=binding.arrow_options_default(fuse_levels=fuse))
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


@pytest.mark.parametrize("I,J,K,R,offset", [
    (70001, 33001, 12000, 1, 0), (70001, 33001, 12000, 3, 0), (70001, 12000, 33001, 8, 0), (70001, 33001, 12000, 9, 4),
    (600000, 900, 1000, 12, 0), (600000, 1000, 900, 16, 0), (600000, 1000, 900, 16, 8), (330007, 33001, 12000, 17, 0),
    (70001, 33001, 12000, 32, 0), (70001, 33001, 12000, 32, 4), (600000, 900, 1000, 33, 0), (70001, 33001, 12000, 96, 0)])
def test_mttkrp_rows_summed_in_lds(torch, I, J, K, R, offset):
    """The form for many small slices: hub slices cut into pieces, slices of one entry and without any, more rows
    than fit the wavefronts of the chip at once (330007), factors whose rows are no whole lines or do not begin
    at one (`offset` floats), duplicates, rows that no entry refers to (infinite), entries in any order."""
    rng = np.random.default_rng(I + R)
    nnz = 2_300_000
    i = (I * rng.random(nnz) ** 1.5).astype(np.int64)
    i[:40000], i[40000:41000] = 11, I - 1
    j, k = rng.integers(1, J - 1, nnz), rng.integers(1, K - 1, nnz)
    i[-30:], j[-30:], k[-30:] = 77, 5, 6
    i[(i > 500) & (i < 600)] = 601
    v = rng.uniform(-1, 1, nnz).astype(np.float32)
    i, j, k = (x.astype(np.int32) for x in (i, j, k))
    B, C = synth.normal_matrix(J, R, seed=34), synth.normal_matrix(K, R, seed=35)
    Aref, E = oracle.mttkrp((I, J, K), i, j, k, v, B, C)
    B[[0, -1]], C[[0, -1]] = np.inf, np.nan
    op = binding.Csf3Mttkrp((I, J, K), i, j, k, v)
    assert op.info["items"] == I - op.info["split_rows"] + op.info["partials"] and op.info["split_rows"] > 0
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_SUMS_IN_LDS
    Bd, Cd = (torch.empty(M.size + 64, device="cuda")[offset:offset + M.size].view(M.shape).copy_(torch.from_numpy(M)) for M in (B, C))
    A = torch.full((I, R), float("nan"), device="cuda")
    op.mttkrp(Bd, Cd, A)
    assert_within(A.cpu().numpy(), Aref, E)
    first = A.clone()
    op.mttkrp(Bd, Cd, A)
    assert torch.equal(first, A)
    op.mttkrp(torch.ones((J, R + 1), device="cuda"), torch.ones((K, R + 1), device="cuda"))   # a larger workspace, then
    op.mttkrp(Bd, Cd, A)                                                                      # fewer columns again
    assert torch.equal(first, A)
    op.close()


def test_mttkrp_without_room_for_laid_out_factors(torch):
    """A workspace for the partial vectors alone: the factors are read where they are, with the last lanes of a row
    moved back, and every sum has the same terms in the same order."""
    I, J, K = 600000, 900, 1000
    rng = np.random.default_rng(41)
    i = rng.integers(0, I, 2_200_000)
    i[:9000] = 11
    i, j, k = (x.astype(np.int32) for x in (i, rng.integers(0, J, len(i)), rng.integers(0, K, len(i))))
    op = binding.Csf3Mttkrp((I, J, K), i, j, k, rng.uniform(-1, 1, len(i)).astype(np.float32))
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_SUMS_IN_LDS and op.info["split_rows"] > 0
    stream = torch.cuda.current_stream().cuda_stream
    for R, offset in ((1, 0), (3, 0), (7, 4), (8, 4), (9, 0), (15, 0), (16, 8), (17, 0), (31, 4), (32, 0), (32, 4), (33, 0), (50, 0), (100, 12)):
        Bd, Cd = (torch.randn(rows * R + 64, device="cuda")[offset:offset + rows * R].view(rows, R) for rows in (J, K))
        full = op.mttkrp(Bd, Cd)
        least = -(-op.info["partials"] * R * 4 // 256) * 256 + 256
        ws = torch.empty(least, dtype=torch.uint8, device="cuda")
        binding.csf3_set_workspace(op.h, ws.data_ptr(), least)
        A = torch.full((I, R), float("nan"), device="cuda")
        binding.csf3_mttkrp(op.h, Bd.data_ptr(), Cd.data_ptr(), A.data_ptr(), R, stream)
        assert torch.equal(A, full), (R, offset)
        with pytest.raises(binding.ArrowError) as e:
            binding.csf3_set_workspace(op.h, ws.data_ptr(), least - 256)
            binding.csf3_mttkrp(op.h, Bd.data_ptr(), Cd.data_ptr(), A.data_ptr(), R, stream)
        assert e.value.code == binding.ARROW_ETOOSMALL
        op._ws = None
    op.close()


@pytest.mark.parametrize("R", [32, 50])
def test_mttkrp_on_several_streams(torch, R):
    """Products of one tensor on two streams with factors of their own: they share the partial vectors of split slices and,
    at R = 50, the room for factors that are laid out anew."""
    I, J, K = 600000, 900, 1000
    rng = np.random.default_rng(43)
    i = rng.integers(0, I, 2_200_000)
    i[:9000] = 11
    i, j, k = (x.astype(np.int32) for x in (i, rng.integers(0, J, len(i)), rng.integers(0, K, len(i))))
    op = binding.Csf3Mttkrp((I, J, K), i, j, k, rng.uniform(-1, 1, len(i)).astype(np.float32))
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_SUMS_IN_LDS and op.info["split_rows"] > 0
    factors = [[torch.randn(rows, R, device="cuda") for rows in (J, K)] for _ in range(2)]
    want = [op.mttkrp(*f) for f in factors]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = [torch.full((I, R), float("nan"), device="cuda") for _ in range(6)]
    torch.cuda.synchronize()
    for n, A in enumerate(got):
        with torch.cuda.stream(streams[n % 2]):
            op.mttkrp(*factors[n % 2], A)
    torch.cuda.synchronize()
    assert all(torch.equal(A, want[n % 2]) for n, A in enumerate(got))
    op.close()


@pytest.mark.parametrize("k", [7, 20, 64, 128, 150])
@pytest.mark.parametrize("fuse", [0, 1])
def test_short_work_lists_beside_window_tiles(torch, k, fuse):
    """More rows than the wave list is ordered by rows for, nearly all of them in window tiles: what is left, chunks of
    long rows, pieces and short rows, goes into one launch."""
    n, b, m = 140001, 512, 14
    rng = np.random.default_rng(k)
    lo = np.arange(n) // b * b
    inside = lo[:, None] + (rng.random((n, m)) * np.minimum(b, n - lo)[:, None]).astype(np.int64)
    hub = rng.choice(64, 5, replace=False)
    far = np.concatenate([np.stack([np.full(c, h), rng.choice(n, c, replace=False)], 1) for h, c in zip(hub, (3000, 1500, 900, 600, 400))])
    key = np.unique(np.concatenate([(np.arange(n)[:, None] * n + inside).ravel(), far[:, 0] * n + far[:, 1]]))
    row, colidx = key // n, (key % n).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int64)
    vals = rng.uniform(-1, 1, len(key)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=36)
    op = binding.ArrowSpMM(rowptr, colidx, vals, b, options=binding.arrow_options_default(fuse_levels=fuse))
    level = op.levels()[0]
    assert level["window_tiles"] > 200 and 0 < level["chunks"] <= 2048 and level["short_rows"] <= 16384
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


@pytest.mark.parametrize("k", [7, 16, 32, 128])
def test_only_chunks_beside_window_tiles(torch, k):
    """All that window tiles leave is long rows, a few chunks of them: those keep a kernel of their own."""
    n, b, m = 140001, 512, 62
    rng = np.random.default_rng(3)
    lo = np.arange(n) // b * b
    inside = lo[:, None] + (rng.random((n, m)) * np.minimum(b, n - lo)[:, None]).astype(np.int64)
    hub = rng.choice(64, 2, replace=False)
    far = np.concatenate([np.stack([np.full(c, h), rng.choice(n, c, replace=False)], 1) for h, c in zip(hub, (3000, 2048))])
    key = np.unique(np.concatenate([(np.arange(n)[:, None] * n + inside).ravel(), far[:, 0] * n + far[:, 1]]))
    row, colidx = key // n, (key % n).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int64)
    vals = rng.uniform(-1, 1, len(key)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=39)
    op = binding.ArrowSpMM(rowptr, colidx, vals, b)
    level = op.levels()[0]
    assert level["window_tiles"] > 200 and 0 < level["chunks"] <= 2048 and level["short_rows"] == 0
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


@pytest.mark.parametrize("blocks", [False, True])
@pytest.mark.parametrize("k", [105, 107, 112])
def test_sampled_product_of_large_factors(torch, k, blocks):
    """Factors beyond the size from which the rows of U are read past the caches: short rows, long ones and rows of
    window tiles, a row length that is no multiple of four columns."""
    n, b = 140003, 512
    assert n * k * 4 >= 56 << 20
    rng = np.random.default_rng(k)
    m = 14 if blocks else 3
    lo = np.arange(n) // b * b
    near = lo[:, None] + (rng.random((n, m)) * np.minimum(b, n - lo)[:, None]).astype(np.int64) if blocks else rng.integers(0, n, (n, m))
    hub = np.repeat([3, 5, 7], [9000, 700, 90])
    key = np.unique(np.concatenate([(np.arange(n)[:, None] * n + near).ravel(), hub * n + rng.integers(0, n, len(hub))]))
    row, colidx = key // n, (key % n).astype(np.int32)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(row, minlength=n))]).astype(np.int64)
    vals = rng.uniform(-1, 1, len(key)).astype(np.float32)
    U, V = synth.normal_matrix(n, k, seed=37), synth.normal_matrix(n, k, seed=38)
    op = binding.ArrowSpMM(rowptr, colidx, vals, b)
    S = torch.full((len(key),), float("nan"), device="cuda")
    op.sddmm(torch.from_numpy(U).cuda(), torch.from_numpy(V).cuda(), S)
    op.close()
    Sref, B = oracle.sddmm(rowptr, colidx, vals, U, V)
    assert_within(S.cpu().numpy(), Sref, B)


@pytest.mark.parametrize("n,k,kc,fuse", [(8192, 256, 0, 1), (17001, 128, 0, 1), (17001, 96, 0, 1), (17001, 160, 0, 0), (17001, 192, 0, 1),
                                         (8192, 260, 0, 1), (17001, 128, 32, 0), (8192, 512, 0, 1), (17001, 150, 0, 1), (135000, 128, 0, 1),
                                         (8192, 320, 32, 1), (8192, 640, 0, 1), (135000, 320, 32, 1)])
def test_column_slices_dealt_to_dies(torch, n, k, kc, fuse):
    """Long, middle and short rows in two, three, four, eight and ten column slices, equal and unequal ones, X on both sides of the
    sizes from which on halves of the dies take halves of the slices; lists in row order and (more than 2^17 rows) in
    window order, whose workgroups fill several runs and a part of one.  Every element is written once per product."""
    rng = np.random.default_rng(n + k)
    length = rng.integers(0, 17, n)
    length[rng.choice(n, n // 40, replace=False)] = rng.integers(17, 300, n // 40)
    length[:4] = (3000, 2500, 700, 49)
    row = np.repeat(np.arange(n), length)
    key = np.unique(row * n + (n * rng.random(len(row)) ** 3).astype(np.int64))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int64)
    colidx = (key % n).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=23)
    op = binding.ArrowSpMM(rowptr, colidx, vals, max(256, n // 16), options=binding.arrow_options_default(kc=kc, fuse_levels=fuse))
    Xd, Y = torch.from_numpy(X).cuda(), torch.full((n, k), float("nan"), device="cuda")
    op.spmm(Xd, Y)
    first = Y.clone()
    op.spmm(Xd, Y.fill_(float("nan")))
    assert torch.equal(first, Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


@pytest.mark.parametrize("b,tiles,k", [(64, 800, 20), (64, 800, 33), (64, 70, 64), (512, 40, 32), (512, 70, 7), (100, 180, 128), (1100, 12, 16),
                                       (1300, 12, 16), (512, 14, 141), (512, 3, 5), (64, 800, 7), (300, 270, 16)])
@pytest.mark.parametrize("fuse", [0, 1])
def test_windows_of_two_workgroups_and_shares_of_tiles(torch, b, tiles, k, fuse):
    """Windows of which a compute unit holds two (up to 1200 positions of 16 columns, 600 of 32 where there are many tiles)
    and one; one, two, three, four, six and eight workgroups to a tile, also more than it has sixteens of rows for."""
    rng = np.random.default_rng(b + tiles)
    n = b * (tiles + 1) - 7
    deg = 12
    inside = rng.integers(0, b, (n, deg)) + (np.arange(n) // b * b)[:, None]
    col = np.concatenate([np.minimum(inside, n - 1), rng.integers(0, 8, (n, 1))], 1)
    key = np.unique((np.repeat(np.arange(n), deg + 1) * n + col.ravel()))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int64)
    colidx = (key % n).astype(np.int32)
    vals = rng.uniform(-1, 1, len(colidx)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=24)
    op = binding.ArrowSpMM(rowptr, colidx, vals, b, options=binding.arrow_options_default(fuse_levels=fuse))
    assert op.levels()[0]["window_tiles"] >= tiles - 1
    Y = torch.full((n, k), float("nan"), device="cuda")
    op.spmm(torch.from_numpy(X).cuda(), Y)
    op.close()
    Yref, B = oracle.spmm(rowptr, colidx, vals, X)
    assert_within(Y.cpu().numpy(), Yref, B)


def test_what_the_python_methods_take_and_refuse(torch):
    """The native calls stand before the general way: results, refusals and allocations are the same on both."""
    w = synth.make_config(0, 2)
    op = binding.ArrowSpMM(*csr_of(w), w.b)
    X = torch.from_numpy(synth.normal_matrix(w.n, 24, seed=25)).cuda()
    Y, S = torch.empty_like(X), torch.empty(op.info["nnz"], device="cuda")
    general, sampled = op.spmm(X), op.sddmm(X, X)
    for x in (X, torch.nn.Parameter(X), X.clone().requires_grad_()):
        with torch.no_grad():
            assert op.spmm(x, Y.fill_(float("nan"))) is Y and torch.equal(Y, general)
            assert op.sddmm(x, X, S.fill_(float("nan"))) is S and torch.equal(S, sampled)
    wide = torch.cat([X, X], 1)                       # more columns than the workspace was bound for
    out = torch.empty_like(wide)
    assert torch.equal(op.spmm(wide, out)[:, 24:], out[:, :24])
    side, late = torch.cuda.Stream(), torch.full_like(X, float("nan"))
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        torch.cuda._sleep(40_000_000)                 # (a call on another stream would find no values in `late`)
        late.copy_(X)
        op.spmm(late, Y.fill_(float("nan")))
        op.sddmm(late, late, S.fill_(float("nan")))
    side.synchronize()
    assert torch.equal(Y, general) and torch.equal(S, sampled)
    for x, y in ((X.double(), Y), (X, Y.double()), (X[:-1], Y[:-1]), (X, Y[:, :8]), (X.t().contiguous().t(), Y), (X.cpu(), Y), (X[0], Y[0])):
        with pytest.raises(AssertionError):
            op.spmm(x, y)
    for u, v, s in ((X, X[:, :8], S), (X, X.double(), S), (X, X, S[:-1]), (X.cpu(), X, S), (X[:, ::2], X, S),
                    (X, wide[:, ::2], S), (X, X, torch.cat([S, S])[::2])):
        with pytest.raises(AssertionError):
            op.sddmm(u, v, s)
    with pytest.raises(binding.ArrowError):
        op.spmm(X, X)                                 # overlap, which the library refuses
    op.close()
    t = [np.array([0, 0, 2], np.int32), np.array([1, 2, 0], np.int32), np.array([3, 0, 1], np.int32)]
    h = binding.Csf3Mttkrp((3, 4, 5), *t, np.array([1, 2, 3], np.float32))
    B, C = torch.rand(4, 6, device="cuda"), torch.rand(5, 6, device="cuda")
    A = torch.empty(3, 6, device="cuda")
    ref = h.mttkrp(B, C)
    assert h.mttkrp(B, C, A) is A and torch.equal(A, ref)
    apart = lambda M: torch.cat([M, M], 1)[:, ::2]
    for b, c, a in ((B[:-1], C, A), (B, C[:, :5], A), (B, C.double(), A), (B, C, A[:-1]), (B.cpu(), C, A), (B.double(), C, A), (B, C, A.double()),
                    (apart(B), C, A), (B, apart(C), A), (B, C, apart(A))):
        with pytest.raises(AssertionError):
            h.mttkrp(b, c, a)
    h.close()


def test_what_the_native_calls_hand_to_the_library(torch):
    """Plain tensors: their addresses, the columns and the current stream.  Anything else in any place: no call."""
    import ctypes
    from paper_2307_05740_amd import tensor_call
    called = []

    def library(tensors):                             # a C function of a handle, so many addresses, the columns and a stream
        return ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_void_p] * (1 + tensors), ctypes.c_int, ctypes.c_void_p)(
            lambda *a: called.append(a) or 0)

    two, three = library(2), library(3)
    at = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    dense = lambda *shape: torch.zeros(shape, device="cuda")
    calls = [   # the call, its tensors
        (lambda *t: tensor_call.spmm(at(two), 77, 0, 6, 8, *t), [dense(6, 8), dense(6, 8)]),
        (lambda *t: tensor_call.sddmm(at(three), 77, 0, 6, 8, 5, *t), [dense(6, 8), dense(6, 8), dense(5)]),
        (lambda *t: tensor_call.mttkrp(at(three), 77, 0, 3, 4, 5, 8, *t), [dense(4, 8), dense(5, 8), dense(3, 8)])]
    side = torch.cuda.Stream()
    for call, good in calls:
        for stream in (torch.cuda.current_stream(), side):
            with torch.cuda.stream(stream):
                assert call(*good) == 1
            assert called.pop() == (77, *[t.data_ptr() for t in good], 8, stream.cuda_stream or None) and not called
        assert call(*[torch.nn.Parameter(t) for t in good]) == 1 and called.pop()
        for place, t in enumerate(good):
            others = [t.double(), t.half(), t.int(), t.cpu(), t.to("meta"), t.to_sparse(), t[:-1], torch.cat([t, t]), t[..., None],
                      torch.cat([t, t], -1)[..., ::2], t.numpy(force=True), None, 1]
            if t.dim() == 2:
                others += [t.t().contiguous().t(), t[:, :4], t[0], torch.cat([t, t], 1)[:, :8], torch.cat([t, t], 1)]
            for bad in others:
                if t.dim() == 1 and bad is not None and getattr(bad, "shape", None) == (5, 1):
                    continue                          # (the entries in any dense shape, as ever)
                assert call(*[bad if q == place else g for q, g in enumerate(good)]) == 0, (place, bad)
        assert call(*[torch.cat([t, t], 1) if t.dim() == 2 else t for t in good]) == 0   # more columns than the workspace has room for
        assert not called


@pytest.mark.parametrize("k", [12, 17, 20, 63, 64, 90, 100, 127, 150])
@pytest.mark.parametrize("kc", [0, 32])
def test_staged_head_in_whole_lines(torch, k, kc):
    """Where there is room the staged head is laid out in whole 128-byte lines (17, 20, 63, 90, 127, 150), else with its
    rows close together: the same results bit for bit, and nothing behind the workspace is written."""
    w = synth.make_config(2, 8)
    op = binding.ArrowSpMM(*csr_of(w), w.b, options=binding.arrow_options_default(stage_short=1, window_rows=1024, kc=kc))
    n, h, st = w.n, op.h, torch.cuda.current_stream().cuda_stream
    X, U = (synth.normal_matrix(n, k, seed=s) for s in (18, 19))
    Xd, Ud = torch.from_numpy(X).cuda(), torch.from_numpy(U).cuda()
    S0 = op.sddmm(Ud, Xd)
    full = binding.arrow_workspace_bytes(h, k)
    xy = -(-n * k * 4 // 256) * 256
    ws = torch.empty(full + xy + 4096, dtype=torch.uint8, device="cuda")

    def all_of(nbytes, l):
        ws.fill_(0xA5)
        binding.arrow_set_workspace(h, ws.data_ptr(), nbytes)
        Y, S, Z = torch.full((n, k), float("nan"), device="cuda"), torch.full_like(S0, float("nan")), Xd.clone()
        binding.arrow_spmm(h, Xd.data_ptr(), Y.data_ptr(), k, st)
        binding.arrow_sddmm(h, Ud.data_ptr(), Xd.data_ptr(), S.data_ptr(), k, st)
        if l:
            binding.arrow_spmm_iter(h, Z.data_ptr(), k, l, st)
        assert bool((ws[nbytes:] == 0xA5).all())
        return [t.cpu().numpy().view(np.uint32) for t in (Y, S, Z)]

    def accepted(nbytes):
        try:
            all_of(nbytes, 0)
        except binding.ArrowError as e:
            assert e.code == binding.ARROW_ETOOSMALL
            return False
        return True

    low, least = 0, full // 256            # the least workspace of a product, in units of 256 bytes
    while least - low > 1:
        m = (low + least) // 2
        low, least = (low, m) if accepted(256 * m) else (m, least)
    close = all_of(256 * least, 0)
    Yref, B = oracle.spmm(*csr_of(w), X)
    assert_within(close[0].view(np.float32), Yref, B)
    Sref, Bs = oracle.sddmm(*csr_of(w), U, X)
    assert_within(close[1].view(np.float32), Sref, Bs)
    for l in (2, 3):
        few = all_of(256 * least + xy, l)
        for nbytes in (full, full + xy):
            for a, b in zip(few, all_of(nbytes, l)):
                assert np.array_equal(a, b)
        assert np.array_equal(few[0], close[0]) and np.array_equal(few[1], close[1])
    binding.arrow_set_workspace(h, ws.data_ptr(), full)            # an operand where only chained products write
    V, S = ws[256 * least:256 * least + n * k * 4].view(torch.float32).view(n, k), torch.full_like(S0, float("nan"))
    V.copy_(Xd)
    binding.arrow_sddmm(h, Ud.data_ptr(), V.data_ptr(), S.data_ptr(), k, st)
    assert np.array_equal(S.cpu().numpy().view(np.uint32), close[1]) and torch.equal(V, Xd)
    Y = torch.full((n, k), float("nan"), device="cuda")
    binding.arrow_spmm_static(h, Xd.data_ptr(), Y.data_ptr(), k, st)
    assert np.array_equal(Y.cpu().numpy().view(np.uint32), close[0])
    op.close()


@pytest.mark.parametrize("k", [33, 48, 64, 96, 200])
@pytest.mark.parametrize("n,pieces,short,long", [(11000, 2000, 8321, 0), (11000, 2000, 8321, 40), (15000, 4001, 8601, 0), (140000, 3000, 60000, 20)])
def test_a_profiled_product_has_the_bits_of_any_other(torch, n, pieces, short, long, k):
    """With a launch of its own for every list it adds up the pieces of long rows as the one launch does; so does arrow_spmm_static."""
    rng = np.random.default_rng(n + k)
    length = np.zeros(n, np.int64)
    length[:pieces] = rng.integers(17, 49, pieces)
    length[pieces:pieces + short] = rng.integers(1, 17, short)
    length[pieces + short:pieces + short + long] = 700
    rng.shuffle(length)
    key = np.unique(np.repeat(np.arange(n), length) * n + (n * rng.random(length.sum())).astype(np.int64))
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=n))]).astype(np.int64)
    colidx, vals = (key % n).astype(np.int32), rng.uniform(-1, 1, len(key)).astype(np.float32)
    X = synth.normal_matrix(n, k, seed=35)
    op = binding.ArrowSpMM(rowptr, colidx, vals, n // 16)
    Xd, st = torch.from_numpy(X).cuda(), torch.cuda.current_stream().cuda_stream
    results = []
    for call in (binding.arrow_spmm, binding.arrow_spmm_static):
        for profiled in (0, 1):
            op._ensure_workspace(k)
            binding.arrow_set_profiling(op.h, profiled)
            Y = torch.full((n, k), float("nan"), device="cuda")
            call(op.h, Xd.data_ptr(), Y.data_ptr(), k, st)
            results.append(Y.cpu().numpy())
    op.close()
    assert_within(results[0], *oracle.spmm(rowptr, colidx, vals, X))
    for Y in results[1:]:
        assert np.array_equal(Y.view(np.uint32), results[0].view(np.uint32))
