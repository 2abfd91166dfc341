"""Grids of launches that no test has the memory or the time for, recorded on the CPU (launch_grids.cpp) with the library as it was built."""
import os
import subprocess

import pytest

from paper_2307_05740_amd import _build


@pytest.fixture(scope="module")
def launch_grids(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("launch_grids") / "launch_grids")
    rocm = os.path.dirname(os.path.dirname(_build._hipcc()))
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"),
                    "-I", os.path.join(_build.REPO_DIR, "include"), "-I", os.path.join(_build.PKG_DIR, "csrc"),
                    os.path.join(_build.REPO_DIR, "tests", "launch_grids.cpp"), _build.ARROW_LIB,
                    f"-Wl,-rpath,{_build.PKG_DIR}", "-L", os.path.join(rocm, "lib"), "-lamdhip64", "-o", out], check=True)
    return out


@pytest.mark.parametrize("case", ["chunks", "chunks in narrow slices", "chunks, two sets of dies", "short rows", "window rows"])
def test_work_that_fits_a_card_fits_a_grid(launch_grids, case):
    proc = subprocess.run([launch_grids, case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("columns", [4096, 5120, 6144, 9000])
def test_columns_of_a_slice_follow_their_cost_at_every_rank(launch_grids, columns):
    proc = subprocess.run([launch_grids, f"factors in LDS, {columns} columns"], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("case", ["one round", "a row more", "two fifths more", "the widest"])
def test_equal_rows_fill_rounds_of_workgroups(launch_grids, case):
    proc = subprocess.run([launch_grids, "equal rows, " + case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("case", ["chunks of a strip", "chunks of a strip and more", "chunks of a strip, few"])
def test_chunks_of_one_strip_are_not_shared_further(launch_grids, case):
    proc = subprocess.run([launch_grids, case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("case", ["one round", "a row more", "three fifths more", "short"])
def test_rows_of_dense_blocks_fill_rounds_of_workgroups(launch_grids, case):
    proc = subprocess.run([launch_grids, "window rows, " + case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("case", ["long", "many", "short", "alone"])
def test_long_rows_behind_chunks_are_two_to_a_workgroup(launch_grids, case):
    proc = subprocess.run([launch_grids, "unequal rows, " + case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("case", ["fewer", "more", "in window order", "in window order, wide"])
def test_pieces_of_long_rows_have_workgroups_of_their_own(launch_grids, case):
    proc = subprocess.run([launch_grids, "pieces, " + case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("case", ["four workgroups a unit", "a row more", "six and more", "too many"])
def test_pieces_of_a_product_have_a_wavefront_each_where_it_fits_the_chip(launch_grids, case):
    proc = subprocess.run([launch_grids, "pieces of a product, " + case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout


@pytest.mark.parametrize("case", ["many", "most"])
def test_pieces_and_short_rows_that_fit_one_grid_are_not_refused(launch_grids, case):
    proc = subprocess.run([launch_grids, "pieces and short rows, " + case], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert proc.returncode == 0, proc.stdout
