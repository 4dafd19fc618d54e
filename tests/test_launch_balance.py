"""How a call on rows of 4 to 256 nodes shares its pairs out among wavefronts, compiled for the host."""
import ctypes
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def launch(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("pxbalance") / "libpxlaunch.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-Wall", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "launch_host.cpp")], check=True)
    return ctypes.CDLL(so)


@pytest.mark.parametrize("f32", [0, 1])
@pytest.mark.parametrize("nodes", [3, 4, 33, 64, 65, 256, 257])
def test_every_candidate_is_taken_once(launch, nodes, f32):
    """1 to 16 candidates a wavefront, no workgroup without one; whole fours where four are swept at a time, and never entry by entry
    then; row inheritance, the sampling argmax and rows of other lengths as split_pairs has it."""
    for candidates in (1, 3, 12, 13, 16, 17, 63, 100, 1000, 4096, 22000):
        for jobs in (1, 8, 30, 200, 1000, 90000):
            for Gm, Gs in ((1, 1), (64, 16), (65, 16), (128, 8), (129, 8), (64, 17), (128, 32), (4096, 4)):
                for inherit, sampled in ((0, 0), (1, 0)) if f32 else ((0, 0), (1, 0), (0, 1)):
                    call = candidates, jobs, nodes, Gm, Gs, f32, inherit, sampled
                    got = launch.px_host_balanced(*call)
                    n, four, entries, groups = (got & 15) + 1, bool(got & 16), bool(got & 32), got >> 8
                    assert (groups - 1) * 4 * n < candidates <= groups * 4 * n
                    if inherit or sampled or not 4 <= nodes <= 256:
                        assert got == launch.px_host_unbalanced(*call), call
                        assert not four or 4 <= nodes <= 64
                    elif nodes <= 64 and four and (f32 or Gs <= 16) and candidates > 12:
                        assert n % 4 == 0 and not entries


@pytest.mark.parametrize("candidates,jobs,nodes,Gm,Gs,f32,per_wave,four", [
    (30, 200, 100, 64, 16, 0, 2, 0), (60, 400, 100, 64, 16, 0, 5, 0), (60, 400, 100, 128, 32, 0, 5, 0), (120, 300, 200, 64, 16, 0, 6, 0),
    (1021, 331, 130, 50, 21, 0, 16, 0), (4096, 1000, 256, 128, 32, 0, 16, 0), (20, 30, 100, 64, 16, 0, 1, 0),
    (30, 200, 64, 64, 16, 0, 4, 1), (60, 400, 64, 64, 16, 0, 8, 1), (1000, 200, 64, 64, 16, 0, 16, 1), (12, 30, 64, 64, 16, 0, 3, 1),
    (60, 66, 33, 50, 12, 0, 1, 0), (60, 67, 33, 50, 12, 0, 4, 1), (60, 67, 33, 129, 12, 0, 1, 0), (60, 66, 33, 64, 16, 1, 1, 0), (60, 67, 33, 64, 16, 1, 4, 1),
    (60, 99, 33, 65, 12, 1, 1, 0), (60, 100, 33, 65, 12, 1, 4, 1), (60, 99, 33, 65, 12, 0, 1, 0), (60, 100, 33, 65, 12, 0, 4, 1)])
def test_candidates_a_wavefront(launch, candidates, jobs, nodes, Gm, Gs, f32, per_wave, four):
    got = launch.px_host_balanced(candidates, jobs, nodes, Gm, Gs, f32, 0, 0)
    assert ((got & 15) + 1, (got >> 4) & 1) == (per_wave, four)
