"""The arithmetic that kernels and launches share, compiled for the host: the job-level launch gives every (job, task) one
wavefront, whatever else it is asked to clear; a fit starts from a record its job has."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def launch(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("pxlaunch") / "libpxlaunch.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_host.cpp")], check=True)
    L = ctypes.CDLL(so)
    L.px_host_prep_covers.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    L.px_host_prep_blocks.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    L.px_host_prep_blocks.restype = ctypes.c_uint
    return L


# wavefronts a job: itself alone; with 128 table rows eight, four, two or one at a time
@pytest.mark.parametrize("tasks", [1, 17, 33, 65, 129])
def test_every_job_is_prepared(launch, tasks):
    for jobs in (1, 7, 8, 9, 64, 65, 72, 100, 127, 128, 129, 241, 400, 1000, 4001):
        for counters in (0, 1, 4096, 4096 * 1023, 4096 * 1024 + 1, 4096 * 1025, 16 * 4096, 20000 * 256, 30000 * 256, 1800 * 4096, 32000 * 256, 1 << 34):
            assert launch.px_host_prep_covers(jobs, tasks, counters), (jobs, tasks, counters)


def test_few_jobs_get_workgroups_to_clear_with(launch):
    assert launch.px_host_prep_blocks(1, 17, 1 << 34) == 1024
    assert launch.px_host_prep_blocks(1, 17, 4096 * 100) == 100
    assert launch.px_host_prep_blocks(1000, 17, 0) == launch.px_host_prep_blocks(1000, 17, 4096) == 4256


@pytest.mark.parametrize("jobs,Gm,rows", [
    (1, 1, 2), (16, 64, 2), (16, 65, 2), (17, 64, 4), (17, 65, 4), (17, 256, 4), (17, 257, 2), (32, 64, 4), (33, 64, 8), (33, 65, 4),
    (96, 64, 8), (96, 65, 4), (96, 257, 2), (97, 65, 8), (97, 256, 8), (97, 257, 2), (120, 128, 8), (121, 64, 8), (121, 65, 4),
    (127, 256, 4), (127, 257, 2), (128, 1, 8), (128, 257, 8), (1000, 500, 8)])
def test_table_rows_a_wavefront(launch, jobs, Gm, rows):
    assert launch.px_host_table_rows(jobs, Gm) == rows


@pytest.mark.parametrize("f32", [0, 1])
@pytest.mark.parametrize("inherit", [0, 1])
def test_the_population_pass_takes_every_candidate(launch, f32, inherit):
    """1 to 16 candidates a wavefront, four wavefronts a workgroup, as many workgroups as the candidates need and no more; a sweep
    of four is not asked to find fewer than four candidates when the split is rounded for it."""
    for candidates in (1, 3, 4, 12, 13, 16, 64, 100, 1000, 4096, 22000, 0x7FFFFFFF):
        for jobs in (1, 8, 30, 200, 1000, 100000):
            if candidates * jobs > 0x7FFFFFFF:
                continue
            for Gm, Gs in ((1, 1), (64, 16), (65, 16), (128, 8), (129, 8), (64, 17), (64, 32), (4096, 4)):
                for row4, whole in ((0, 0), (0, 1), (1, 0), (1, 1)):
                    got = launch.px_host_split(candidates, jobs, Gm, Gs, f32, row4, whole, inherit)
                    n, four = (got & 15) + 1, bool(got & 16)
                    groups = launch.px_host_pair_groups(candidates, n)
                    assert (groups - 1) * 4 * n < candidates <= groups * 4 * n
                    assert row4 or not got & 48
                    if four and not inherit and (f32 or not whole) and (f32 or Gs <= 16):
                        assert n % 4 == 0 and candidates > 12
                    if got & 32:
                        assert not four and n < 4


@pytest.mark.parametrize("candidates,jobs,nodes,Gm,Gs,per_wave", [
    # 64 nodes, narrow: as many as 12400 wavefronts leave each, in whole fours where they are swept in fours
    (61, 200, 64, 64, 16, 1), (124, 200, 64, 64, 16, 2), (125, 200, 64, 64, 16, 2), (249, 200, 64, 64, 16, 4), (434, 200, 64, 64, 16, 4),
    (496, 200, 64, 64, 16, 8), (1000, 200, 64, 64, 16, 16), (2000, 200, 64, 64, 16, 16),
    # wide: six, until 25000 wavefronts leave more
    (372, 200, 64, 128, 32, 6), (371, 200, 64, 128, 32, 5), (874, 200, 64, 128, 32, 6), (875, 200, 64, 128, 32, 7), (1000, 200, 64, 128, 32, 8),
    # rows of 65 to 256 nodes: the same at any width
    (373, 200, 65, 64, 16, 6), (500, 200, 130, 64, 16, 6), (200, 1000, 256, 64, 16, 8), (150, 1000, 192, 32, 8, 6), (500, 200, 130, 128, 32, 6),
    # longer, and below four nodes: four
    (249, 200, 257, 64, 16, 4), (500, 200, 257, 64, 16, 4), (500, 200, 3, 64, 16, 4), (625, 200, 500, 128, 32, 5), (150, 1000, 320, 32, 16, 6)])
def test_candidates_a_wavefront(launch, candidates, jobs, nodes, Gm, Gs, per_wave):
    assert launch.px_host_split_nodes(candidates, jobs, nodes, Gm, Gs, 0) == per_wave


def test_a_fit_starts_from_a_record_its_job_has(launch):
    for records in (1, 2, 64, 65, 1000):
        for found in (0, 1, records - 1, records, 1 << 20, 0x7FFFFFFF):        # the last: no record had a time below infinity
            at = launch.px_host_record_or_first(found, records)
            assert at == (found if found < records else 0)
