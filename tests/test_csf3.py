"""Host side of the order-3 MTTKRP: the compressed-sparse-fibre build and its error paths (no GPU)."""
import numpy as np
import pytest

from paper_2307_05740_amd import binding, synth


def build_info(dims, i, j, k, v):
    h = binding.csf3_build(dims, i, j, k, v)
    try:
        return binding.csf3_info(h), binding.csf3_device_bytes(h), binding.csf3_workspace_bytes(h, 8)
    finally:
        binding.csf3_destroy(h)


@pytest.mark.parametrize("idx,shrink", [(0, 4), (0, 6), (1, 5), (1, 7)])
def test_structure_counts(idx, shrink):
    w = synth.make_tensor_config(idx, shrink)
    info, nbytes, ws = build_info(w.dims, w.i, w.j, w.k, w.vals)
    assert (info["I"], info["J"], info["K"]) == tuple(w.dims) and info["nnz"] == w.nnz
    assert info["slices"] == len(np.unique(w.i))
    fib = w.i.astype(np.int64) * w.dims[1] + w.j
    flen = np.unique(fib, return_counts=True)[1]
    assert info["fibers"] == len(flen)
    assert info["segments"] == int(np.sum((flen + 63) // 64))          # fibres cut into runs of <= 64
    sl = np.bincount(w.i, minlength=w.dims[0])
    assert info["items"] >= w.dims[0]                                   # every slice, empty ones too
    assert info["split_rows"] <= np.count_nonzero(sl > 64) and info["partials"] >= 2 * info["split_rows"]
    assert info["items"] == w.dims[0] - info["split_rows"] + info["partials"]
    assert info["distinct_j"] == len(np.unique(w.j)) and info["distinct_k"] == len(np.unique(w.k))
    assert nbytes >= 8 * w.nnz and ws >= 32 * info["partials"]


def test_entry_order_does_not_change_the_structure():
    w = synth.make_tensor_config(1, 6)
    a = build_info(w.dims, w.i, w.j, w.k, w.vals)[0]
    p = np.random.default_rng(3).permutation(w.nnz)
    b = build_info(w.dims, w.i[p], w.j[p], w.k[p], w.vals[p])[0]
    for key in a:
        if key != "build_seconds":
            assert a[key] == b[key], key


def test_empty_tensor_and_duplicates():
    z = np.zeros(0, np.int32)
    info = build_info((5, 4, 3), z, z, z, np.zeros(0, np.float32))[0]
    assert info["nnz"] == 0 and info["items"] == 5 and info["segments"] == 0 and info["partials"] == 0
    i = np.array([1, 1, 1], np.int32); j = np.array([2, 2, 2], np.int32); k = np.array([0, 0, 1], np.int32)
    info = build_info((3, 3, 2), i, j, k, np.ones(3, np.float32))[0]
    assert info["nnz"] == 3 and info["fibers"] == 1 and info["slices"] == 1      # duplicates are kept


def test_error_paths():
    i = np.array([0, 1], np.int32)
    v = np.ones(2, np.float32)
    for dims, (a, b, c) in (((2, 2, 2), (i, i, i + 1)), ((2, 2, 2), (i - 1, i, i)), ((0, 2, 2), (i, i, i)),
                            ((2, 1, 2), (i, i, i))):
        with pytest.raises(binding.ArrowError) as e:
            binding.csf3_build(dims, a, b, c, v)
        assert e.value.code == binding.ARROW_EINVAL and binding.csf3_last_error()
    h = binding.csf3_build((2, 2, 2), i, i, i, v)
    with pytest.raises(binding.ArrowError) as e:            # no image on the device yet
        binding.csf3_mttkrp(h, 16, 32, 48, 4, 0)
    assert e.value.code == binding.ARROW_ENOTREADY
    with pytest.raises(binding.ArrowError):
        binding.csf3_upload(h, 0, 1 << 20, 0)
    with pytest.raises(binding.ArrowError):
        binding.csf3_set_workspace(h, 4, 1 << 20)           # misaligned
    assert binding.csf3_workspace_bytes(h, 0) == 0
    binding.csf3_destroy(h)
    binding.csf3_destroy(0)


def test_items_are_capped_by_segments_as_well_as_entries():
    # slice 0: 300 fibres of one entry -> 300 segments -> items of at most 128 segments;
    # slice 1: one fibre of 1000 entries -> 16 segments of <= 64 -> items of at most 512 entries
    i = np.concatenate([np.zeros(300, np.int32), np.ones(1000, np.int32)])
    j = np.concatenate([np.arange(300, dtype=np.int32), np.zeros(1000, np.int32)])
    k = np.concatenate([np.zeros(300, np.int32), np.arange(1000, dtype=np.int32)])
    info = build_info((3, 300, 1000), i, j, k, np.ones(1300, np.float32))[0]
    assert info["segments"] == 300 + 16 and info["fibers"] == 301
    assert info["split_rows"] == 2
    assert info["partials"] == 3 + 2            # 128 + 128 + 44 segments; 512 + 488 entries
    assert info["items"] == 3 + 2 + 1           # plus the empty slice 2


def uniform(I, J, K, nnz, seed=3):
    """`nnz` entries at uniformly drawn places, as a handle."""
    rng = np.random.default_rng(seed)
    i, j, k = (rng.integers(0, d, nnz, dtype=np.int32) for d in (I, J, K))
    return binding.csf3_build((I, J, K), i, j, k, np.ones(nnz, np.float32))


@pytest.mark.parametrize("I,J,K,nnz,form", [
    (250, 231, 307, 17_730, binding.CSF3_FORM_ITEMS),                   # few entries
    (520, 1000, 1000, 520_000, binding.CSF3_FORM_FACTORS_IN_LDS),       # factors of 2000 rows, read 400 times each
    (520, 8000, 3000, 560_000, binding.CSF3_FORM_ITEMS),                # more rows than the LDS holds
    (520, 9000, 1000, 560_000, binding.CSF3_FORM_ITEMS),                # too few entries for copying the factors to LDS
    (520, 3000, 7000, 560_000, binding.CSF3_FORM_ITEMS),
    (600, 1000, 9100, 500_000, binding.CSF3_FORM_ITEMS),
    (700, 9000, 1000, 1_000_000, binding.CSF3_FORM_ITEMS),              # 192 rows read for every row copied
    (700, 9000, 1000, 1_100_000, binding.CSF3_FORM_FACTORS_IN_LDS),     # 211
    (520, 9000, 1000, 800_000, binding.CSF3_FORM_FACTORS_IN_LDS),       # 154, but an item per wavefront
    (340, 830, 1821, 230_000, binding.CSF3_FORM_FACTORS_IN_LDS),
    (180_000, 30_000, 22_500, 2_200_000, binding.CSF3_FORM_SUMS_IN_LDS),
    (600_000, 1000, 2000, 2_200_000, binding.CSF3_FORM_SUMS_IN_LDS),    # slices of under four entries
    (500, 30_000, 30_000, 2_200_000, binding.CSF3_FORM_ITEMS),          # long slices
    (180_000, 270_000, 270_000, 2_200_000, binding.CSF3_FORM_SUMS_IN_LDS),   # 4.1 entries for every row of the factors
    (180_000, 280_000, 280_000, 2_200_000, binding.CSF3_FORM_ITEMS),         # 3.9
    (190_000, 9000, 3_000_000, 2_200_000, binding.CSF3_FORM_SUMS_IN_LDS)])   # 0.7, but slices of under twelve entries
def test_form_of_the_image(I, J, K, nnz, form):
    h = uniform(I, J, K, nnz)
    try:
        assert binding.csf3_form(h) == form
    finally:
        binding.csf3_destroy(h)


@pytest.mark.parametrize("I,J,K,nnz,form", [
    (144, 415, 1945, 116_000, binding.CSF3_FORM_FACTORS_IN_LDS),        # 144 items, 70 rows read for every row copied
    (282, 223, 1855, 117_000, binding.CSF3_FORM_FACTORS_IN_LDS),        # 1.74 steps for every row
    (161, 1645, 160, 66_000, binding.CSF3_FORM_FACTORS_IN_LDS),         # fibres of one entry
    (161, 1645, 160, 65_000, binding.CSF3_FORM_ITEMS),                  # too few entries
    (127, 1645, 500, 104_000, binding.CSF3_FORM_ITEMS),                 # 127 items
    (4061, 347, 430, 606_000, binding.CSF3_FORM_ITEMS),                 # 2.0 steps for every row
    (520, 2549, 2550, 300_000, binding.CSF3_FORM_FACTORS_IN_LDS),       # the most rows that fit with eight columns
    (700, 2549, 2551, 300_000, binding.CSF3_FORM_ITEMS)])               # 117 rows read for every row copied
def test_form_of_tensors_with_few_entries_or_items(I, J, K, nnz, form):
    rng = np.random.default_rng(7)
    h = binding.csf3_build((I, J, K), *(rng.integers(0, d, nnz).astype(np.int32) for d in (I, J, K)), np.ones(nnz, np.float32))
    assert binding.csf3_form(h) == form
    binding.csf3_destroy(h)


@pytest.mark.parametrize("I,J,live,form", [
    (60_000, 30_000, 700, binding.CSF3_FORM_ITEMS),              # slices of 3143 entries between empty ones
    (60_000, 30_000, 3000, binding.CSF3_FORM_SUMS_IN_LDS),       # of 733
    (150_000, 30_000, 700, binding.CSF3_FORM_SUMS_IN_LDS),       # an empty one for every 15 entries
    (130_000, 30_000, 700, binding.CSF3_FORM_ITEMS)])            # for every 17
def test_empty_slices_do_not_make_the_others_short(I, J, live, form):
    rng = np.random.default_rng(5)
    i = (rng.integers(0, live, 2_200_000) * (I // live)).astype(np.int32)
    j, k = (rng.integers(0, J, len(i), dtype=np.int32) for _ in range(2))
    h = binding.csf3_build((I, J, J), i, j, k, np.ones(len(i), np.float32))
    try:
        assert binding.csf3_info(h)["slices"] == live and binding.csf3_form(h) == form
    finally:
        binding.csf3_destroy(h)


def test_form_of_no_image():
    with pytest.raises(binding.ArrowError) as e:
        binding.csf3_form(0)
    assert e.value.code == binding.ARROW_EINVAL


def test_workspace_holds_laid_out_factors_only_where_they_are():
    """Beyond the partial vectors, room for both factors at ranks whose rows are no whole lines or parts of one."""
    I, J, K = 600_000, 1000, 2000
    rng = np.random.default_rng(4)
    i = rng.integers(0, I, 2_200_000, dtype=np.int32)
    i[:5000] = 3                                                        # a slice of several pieces
    j, k = (rng.integers(0, d, len(i), dtype=np.int32) for d in (J, K))
    h = binding.csf3_build((I, J, K), i, j, k, np.ones(len(i), np.float32))
    try:
        assert binding.csf3_form(h) == binding.CSF3_FORM_SUMS_IN_LDS
        partials = binding.csf3_info(h)["partials"]
        assert partials > 1
        for R in (1, 2, 4, 8, 16, 32, 64, 96, 128, 3, 5, 9, 17, 33, 50, 100):
            width = 8 if R <= 8 else 16 if R <= 16 else 32
            lines = R in (1, 2, 4, 8, 16) or R % 32 == 0
            laid_out = 0 if lines else (J + K) * -(-R // width) * width * 4
            up = lambda nbytes: -(-nbytes // 256) * 256
            assert binding.csf3_workspace_bytes(h, R) == up(partials * R * 4) + up(laid_out) + 256, R
    finally:
        binding.csf3_destroy(h)


def test_workspace_holds_no_factors_that_are_large_for_the_tensor():
    """Laying the factors out anew copies all of their rows; with fewer than three entries for each the product reads them
    where they are, at every rank and with any workspace."""
    for J, K, laid_out in ((400_000, 300_000, True), (400_000, 340_000, False), (3_000_000, 9_000, False)):
        h = uniform(600_000, J, K, 2_200_000)
        try:
            assert binding.csf3_form(h) == binding.CSF3_FORM_SUMS_IN_LDS
            partials = binding.csf3_info(h)["partials"]
            for R in (3, 12, 25, 50):
                width = 8 if R <= 8 else 16 if R <= 16 else 32
                up = lambda nbytes: -(-nbytes // 256) * 256
                more = up((J + K) * -(-R // width) * width * 4) if laid_out else 0
                assert binding.csf3_workspace_bytes(h, R) == up(partials * R * 4) + more + 256, (J, K, R)
        finally:
            binding.csf3_destroy(h)
