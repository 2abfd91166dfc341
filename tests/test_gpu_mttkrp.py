"""GPU parity of the order-3 MTTKRP  A(i,a) = sum_{j,k} T(i,j,k) B(j,a) C(k,a), called through the
C-ABI, against the fp64 CPU oracle on the same seeded inputs.
Bar (elementwise): |A - A_ref| <= 1e-5 * sum |T| |B| |C|, exactly 0 where the bound is 0;
every element of A is written (the output starts as NaN)."""
import os

import numpy as np
import pytest

import oracle
from paper_2307_05740_amd import binding, synth

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible: the parity tests need a real MI355X")
    if not os.path.exists(binding.LIB_PATH):
        pytest.fail("libarrow.so is not built")
    return torch


def assert_within(A, Aref, E):
    A = np.asarray(A, dtype=np.float64)
    assert not np.isnan(A).any(), f"{np.isnan(A).sum()} elements were never written"
    err = np.abs(A - Aref)
    bad = err > TOL * E
    if bad.any():
        i = np.unravel_index(np.argmax(err - TOL * E), err.shape)
        raise AssertionError(f"{bad.sum()} of {bad.size} elements outside the bound; worst at {i}: "
                             f"got {A[i]!r} want {Aref[i]!r} bound {TOL * E[i]!r}")
    assert np.all(A[E == 0] == 0)
    nz = E > 0
    if nz.any():
        assert np.median(err[nz] / E[nz]) < 1e-6


def run(torch, dims, i, j, k, v, B, C):
    op = binding.Csf3Mttkrp(dims, i, j, k, v)
    Bd, Cd = torch.from_numpy(B).cuda(), torch.from_numpy(C).cuda()
    Ad = torch.full((dims[0], B.shape[1]), float("nan"), dtype=torch.float32, device="cuda")
    op.mttkrp(Bd, Cd, Ad)
    torch.cuda.synchronize()
    return op, Bd, Cd, Ad.cpu().numpy()


@pytest.mark.parametrize("idx,shrink", [(0, 3), (1, 4)])
def test_named_workloads_shrunk(torch, idx, shrink):
    w = synth.make_tensor_config(idx, shrink)
    B, C = w.factors()
    op, Bd, Cd, A = run(torch, w.dims, w.i, w.j, w.k, w.vals, B, C)
    if idx == 1:
        assert op.info["split_rows"] > 0                # hub slices cut into several items + reduction
    Aref, E = oracle.mttkrp(w.dims, w.i, w.j, w.k, w.vals, B, C)
    assert_within(A, Aref, E)
    A2 = op.mttkrp(Bd, Cd).cpu().numpy()                # bitwise reproducible run to run
    assert np.array_equal(A.view(np.uint32), A2.view(np.uint32))
    op.close()


@pytest.mark.parametrize("R", [1, 2, 3, 4, 6, 7, 16, 20, 32, 33, 64, 100, 128, 130, 256, 260, 516])
def test_all_ranks(torch, R):
    w = synth.make_tensor_config(1, 6)                  # skewed: hub slices, long fibres, empty slices
    B = synth.normal_matrix(w.dims[1], R, seed=600 + R)
    C = synth.normal_matrix(w.dims[2], R, seed=700 + R)
    op, _, _, A = run(torch, w.dims, w.i, w.j, w.k, w.vals, B, C)
    Aref, E = oracle.mttkrp(w.dims, w.i, w.j, w.k, w.vals, B, C)
    assert_within(A, Aref, E)
    op.close()


@pytest.mark.parametrize("R", [1, 3, 8, 9, 33, 128])
@pytest.mark.parametrize("I,J,K,nnz", [(144, 415, 1945, 116_000), (161, 1645, 160, 66_000), (128, 300, 200, 70_000), (520, 2549, 2550, 300_000)])
def test_few_items_with_factors_in_lds(torch, I, J, K, nnz, R):
    """Fewer items than wavefronts of a column slice, down to the fewest and to the fewest entries, in the form with
    the factors in LDS: workgroups without any at the lowest ranks, none with more than its turn."""
    rng = np.random.default_rng(I + R)
    i, j, k = (rng.integers(0, d, nnz).astype(np.int32) for d in (I, J, K))
    v = rng.uniform(-1, 1, nnz).astype(np.float32)
    B, C = synth.normal_matrix(J, R, seed=31), synth.normal_matrix(K, R, seed=32)
    op, _, _, A = run(torch, (I, J, K), i, j, k, v, B, C)
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_FACTORS_IN_LDS
    Aref, E = oracle.mttkrp((I, J, K), i, j, k, v, B, C)
    assert_within(A, Aref, E)
    op.close()


@pytest.mark.parametrize("I,J,K,nnz,ranks", [
    (600, 3000, 3000, 3_000_000, (1024, 520)),      # items of 16 blocks, shares of a wavefront up to 4725 steps
    (1100, 3000, 3000, 7_950_000, (512, 256)),      # 21 blocks, up to 5708 steps: a third block on its way at R = 512
    (1100, 2000, 2000, 20_000_000, (128, 64))])     # items of 42 blocks; eight columns at a time at R = 128, four at R = 64
def test_columns_do_not_depend_on_their_number(torch, I, J, K, nnz, ranks):
    """With the factors in LDS and no slice in parts, the sums of a column are added in an order that the image alone decides."""
    rng = np.random.default_rng(I)
    i, j, k = (rng.integers(0, d, nnz).astype(np.int32) for d in (I, J, K))
    v = rng.uniform(-1, 1, nnz).astype(np.float32)
    B, C = synth.normal_matrix(J, ranks[0], seed=31), synth.normal_matrix(K, ranks[0], seed=32)
    op, Bd, Cd, A = run(torch, (I, J, K), i, j, k, v, B, C)
    assert binding.csf3_form(op.h) == binding.CSF3_FORM_FACTORS_IN_LDS and op.info["partials"] == 0
    Aref, E = oracle.mttkrp((I, J, K), i, j, k, v, np.ascontiguousarray(B[:, :8]), np.ascontiguousarray(C[:, :8]))
    assert_within(A[:, :8], Aref, E)
    for R in (*ranks[1:], 8, 4, 1):
        fewer = op.mttkrp(Bd[:, :R].contiguous(), Cd[:, :R].contiguous()).cpu().numpy()
        assert np.array_equal(fewer.view(np.uint32), np.ascontiguousarray(A[:, :R]).view(np.uint32)), R
    op.close()


def test_unsorted_input_duplicates_and_long_fibre(torch):
    rng = np.random.default_rng(5)
    I, J, K, R = 40, 30, 700, 24
    # one fibre with every k (cut into 11 segments), a slice with a single long fibre only,
    # scattered entries, and some coordinates twice
    i = np.concatenate([np.full(K, 3), np.full(500, 7), rng.integers(0, I, 3000)])
    j = np.concatenate([np.full(K, 5), np.full(500, 0), rng.integers(0, J, 3000)])
    k = np.concatenate([np.arange(K), rng.integers(0, K, 500), rng.integers(0, K, 3000)])
    i = np.concatenate([i, i[:50]]); j = np.concatenate([j, j[:50]]); k = np.concatenate([k, k[:50]])
    v = rng.uniform(-1, 1, len(i)).astype(np.float32)
    p = rng.permutation(len(i))
    i, j, k, v = i[p].astype(np.int32), j[p].astype(np.int32), k[p].astype(np.int32), v[p]
    B = rng.standard_normal((J, R)).astype(np.float32)
    C = rng.standard_normal((K, R)).astype(np.float32)
    op, _, _, A = run(torch, (I, J, K), i, j, k, v, B, C)
    Aref, E = oracle.mttkrp((I, J, K), i, j, k, v, B, C)
    assert_within(A, Aref, E)
    op.close()


def test_special_operands(torch):
    w = synth.make_tensor_config(0, 5)                  # 128^3
    I, J, K = w.dims
    R = K
    # B = ones, C = identity: A(i,a) = sum_j T(i,j,a), sums of at most J fp32 values
    op, _, _, A = run(torch, w.dims, w.i, w.j, w.k, w.vals, np.ones((J, R), np.float32), np.eye(K, dtype=np.float32))
    T = np.zeros(w.dims); T[w.i, w.j, w.k] = w.vals
    assert np.all(np.abs(A - T.sum(1)) <= 1e-5 * np.abs(T).sum(1)) and np.all(A[np.abs(T).sum(1) == 0] == 0)
    # zero factor -> exactly zero; empty tensor -> exactly zero
    Z = op.mttkrp(torch.zeros((J, 8), device="cuda"), torch.ones((K, 8), device="cuda")).cpu().numpy()
    assert np.all(Z == 0)
    op.close()
    z = np.zeros(0, np.int32)
    op, _, _, A0 = run(torch, (9, 4, 3), z, z, z, np.zeros(0, np.float32), np.ones((4, 5), np.float32), np.ones((3, 5), np.float32))
    assert A0.shape == (9, 5) and np.all(A0 == 0)
    op.close()


def test_k_equal_1_is_the_matrix_product(torch):
    """K = 1, C = ones: the kernel computes A = T_(IxJ) . B -- compared with the matrix-product oracle."""
    g = synth.make_config(0, shrink=2)
    rows = np.repeat(np.arange(g.n), np.diff(g.rowptr)).astype(np.int32)
    B = synth.normal_matrix(g.n, 12, seed=31)
    op, _, _, A = run(torch, (g.n, g.n, 1), rows, g.colidx, np.zeros(g.nnz, np.int32), g.vals, B, np.ones((1, 12), np.float32))
    Y, Bd = oracle.spmm(g.rowptr, g.colidx, g.vals, B)
    assert_within(A, Y, Bd)
    op.close()


def test_errors_on_device(torch):
    w = synth.make_tensor_config(1, 6)                  # has split slices, so the workspace depends on R
    op = binding.Csf3Mttkrp(w.dims, w.i, w.j, w.k, w.vals)
    assert op.info["partials"] > 0
    B = torch.zeros((w.dims[1], 8), device="cuda"); C = torch.zeros((w.dims[2], 8), device="cuda")
    A = op.mttkrp(B, C)
    with pytest.raises(binding.ArrowError):
        binding.csf3_mttkrp(op.h, B.data_ptr(), C.data_ptr(), B.data_ptr(), 8, 0)       # A overlaps B
    with pytest.raises(binding.ArrowError):
        binding.csf3_mttkrp(op.h, B.data_ptr(), C.data_ptr(), A.data_ptr() + 4, 8, 0)   # misaligned
    with pytest.raises(binding.ArrowError):
        binding.csf3_mttkrp(op.h, B.data_ptr(), 0, A.data_ptr(), 8, 0)
    with pytest.raises(binding.ArrowError) as e:                                        # workspace sized for R = 8
        binding.csf3_mttkrp(op.h, B.data_ptr(), C.data_ptr(), A.data_ptr(), 4096, 0)
    assert e.value.code == binding.ARROW_ETOOSMALL
    op.close()
