"""bench.py quotes a stored counter record only for the image and the kernels that it was taken with."""
import json

import bench


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
