"""What the library's calls hand to their kernels, recorded on the CPU (launch_arguments.cpp) with the library as it was built."""
import os
import subprocess

import pytest

from paper_2307_05740_amd import _build


@pytest.fixture(scope="module")
def launch_arguments(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("launch_arguments") / "launch_arguments")
    rocm = os.path.dirname(os.path.dirname(_build._hipcc()))
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(_build.REPO_DIR, "include"), "-I", os.path.join(_build.PKG_DIR, "csrc"),
                    os.path.join(_build.REPO_DIR, "tests", "launch_arguments.cpp"), _build.ARROW_LIB,
                    f"-Wl,-rpath,{_build.PKG_DIR}", "-L", os.path.join(rocm, "lib"), "-lamdhip64", "-o", out], check=True)

    def run(case):
        proc = subprocess.run([out, case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
        assert proc.returncode == 0, proc.stdout

    return run


def test_a_staged_head_leaves_alone_what_a_caller_keeps_in_the_workspace(launch_arguments):
    """An entry map or an image there is read by the very product, operands by another one."""
    launch_arguments("buffers in the workspace")


@pytest.mark.parametrize("case", ["one launch", "one launch, a wavefront each", "seven workgroups a unit", "slices and chunks", "two launches"])
def test_a_profiled_product_adds_up_pieces_as_any_other(launch_arguments, case):
    """Whether a lane group or four of them add up a piece is not for the launch to say that it happens to be in."""
    launch_arguments("profiled, " + case)


@pytest.mark.parametrize("columns", [48, 100, 200])
def test_items_of_a_sampled_product_go_by_the_rows_with_entries(launch_arguments, columns):
    launch_arguments(f"items of a sampled product, {columns} columns")


@pytest.mark.parametrize("case", ["eight columns, 4000 items of 2.5 blocks, rank 128", "four columns, 1018 items of 12 blocks, rank 16",
                                  "eight columns, 2000 items of 1.2 blocks, rank 64", "four columns, 2000 items of 1.2 blocks, rank 4",
                                  "four columns, 430 items, rank 4742", "eight columns, 229 items, rank 6881"])
def test_four_or_eight_columns_of_the_factors_in_lds(launch_arguments, case):
    """At ordinary ranks (the third is the tensor of test_mttkrp_steps_of_the_last_block), and where eight columns take more than a round of workgroups."""
    launch_arguments(case)


@pytest.mark.parametrize("case", ["127 columns in a workspace for 128", "31 columns in a workspace for 32", "20 columns in a workspace for 25"])
def test_fewer_columns_find_room_for_a_head_in_whole_lines(launch_arguments, case):
    launch_arguments(case)


@pytest.mark.parametrize("case", ["runs of 64, a few workgroups", "runs of 64, the shortest that has one", "runs of 64, the longest", "runs of 128, the shortest",
                                  "runs of 128, two sets of dies", "runs of 256, the shortest", "runs of 256, two sets of dies"])
def test_runs_of_workgroups_take_every_one_of_them_once(launch_arguments, case):
    launch_arguments(case)


@pytest.mark.parametrize("columns", [12, 17, 20, 63, 64, 90, 100, 127, 150])
def test_rows_of_a_staged_head(launch_arguments, columns):
    """In whole 128-byte lines with 17, 20, 63, 90, 127 and 150 columns, where there is room for that."""
    launch_arguments(f"head rows of {columns} columns")


@pytest.mark.parametrize("case", ["four columns, 700 items of 10 blocks, rank 100", "eight columns, 1403 items of 2 blocks, rank 43"])
def test_eight_columns_gain_by_the_item(launch_arguments, case):
    """35.9 us with four columns and 37.0 with eight; 10.3 and 8.9."""
    launch_arguments(case)
