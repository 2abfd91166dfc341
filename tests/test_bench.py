"""bench.py quotes a stored counter record only for the image and the kernels that it was taken with, and counts the
bytes of the image that runs."""
import json

import numpy as np
import pytest

import bench
from paper_2307_05740_amd import binding


def test_a_stored_record_of_another_image_or_of_other_kernels_is_ignored(tmp_path):
    path = str(tmp_path / "traffic.json")
    launch = {"nnz": 7, "items": 3}
    assert bench.stored_traffic(path, "spmm", launch) == (None, None)
    rec = {"hbm_bytes_per_launch": 99, "launch": launch, "code": bench.kernel_code("spmm")}
    for change, used in (({}, True), ({"launch": {"nnz": 7, "items": 4}}, False), ({"launch": None}, False),
                         ({"code": bench.kernel_code("sddmm")}, False), ({"code": None}, False)):
        with open(path, "w") as f:
            json.dump(dict(rec, **change), f)
        got, source = bench.stored_traffic(path, "spmm", launch)
        assert (got is not None) == used and ("stale" in source) != used


@pytest.mark.parametrize("dims,nnz,form,least,most", [
    ((300, 300, 400), 50_000, binding.CSF3_FORM_ITEMS, 8, 20),               # {k, value}, and offset and j of a segment
    ((520, 700, 900), 1_500_000, binding.CSF3_FORM_FACTORS_IN_LDS, 6, 14),   # six bytes for an entry and for a fibre
    ((600_000, 1000, 2000), 2_200_000, binding.CSF3_FORM_SUMS_IN_LDS, 12, 16)])
def test_bytes_of_an_order_3_product_follow_the_form_of_its_image(dims, nnz, form, least, most):
    rng = np.random.default_rng(6)
    i, j, k = (rng.integers(0, n, nnz, dtype=np.int32) for n in dims)
    h = binding.csf3_build(dims, i, j, k, np.ones(nnz, np.float32))
    try:
        info, image = binding.csf3_info(h), binding.csf3_device_bytes(h)
        assert binding.csf3_form(h) == form and least * nnz <= image <= most * nnz
        rows = info["distinct_j"] + info["distinct_k"] + info["items"]
        assert bench.algorithmic_bytes_mttkrp(info, image, 64) == image + 256 * rows
    finally:
        binding.csf3_destroy(h)
