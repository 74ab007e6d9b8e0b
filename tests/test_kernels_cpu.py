"""The batched kernels' own code on the CPU (tests/lanes): a workgroup is a host
thread, its work-items are fibers that meet at cross-lane operations and barriers,
and waves take turns at random.  The state slab has guard words behind every array,
which a write out of range changes, and a barrier that not every lane reaches ends
the run; the centralities are compared with a plain Brandes."""
from __future__ import annotations

import os
import subprocess

import pytest

from paper_1701_05975_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
LANES = os.path.join(HERE, "lanes")


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    exe = tmp_path_factory.mktemp("lanes") / "kernels_check"
    cmd = ["g++", "-std=c++17", "-O1", "-w", "-pthread", "-fno-extern-tls-init",
           "-U_FORTIFY_SOURCE", f"-I{LANES}", f"-I{build.CSRC}",
           os.path.join(LANES, "kernels_check.cpp"), "-o", str(exe)]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(*args):
        r = subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True,
                           timeout=300)
        assert r.stdout.strip().endswith("OK"), (args, r.stdout[-500:], r.stderr[-500:])
        return r.stdout

    return run


@pytest.mark.parametrize("seed", [1, 2])
@pytest.mark.parametrize("n, degree, wmax, delta, wg_deg", [
    (200, 190, 1000, 2000, 64), (300, 298, 255, 1000, 64), (300, 298, 255, 100, 64),
    (640, 1100, 1000, 2000, 512)])
def test_hubs_that_improve_each_other(check, n, degree, wmax, delta, wg_deg, seed):
    """Dense graphs, most of whose vertices are hubs: a queue holds each vertex at
    most once, whatever the band width."""
    check("batched", n, degree, wmax, delta, wg_deg, seed, 0)


@pytest.mark.parametrize("seed", [1, 2, 3])
@pytest.mark.parametrize("delta", [3, 10, 70])
def test_bands_of_a_sparse_graph(check, delta, seed):
    """Many bands of few vertices, with each width of the resident distances: waves
    that reach a band change late take the same way as the first one."""
    check("batched", 120, 8, 20, delta, 512, seed, 0)


@pytest.mark.parametrize("seed", [1, 2, 3])
@pytest.mark.parametrize("group", [-1, 1, 4, 16, 64])
def test_groups_of_lanes(check, group, seed):
    """A group of lanes per queued vertex, also for short queues only: its lanes expand
    the vertex from one distance, and an improvement meanwhile queues it again."""
    check("batched", 206, 4, 20, 5000, 512, seed, group)


@pytest.mark.parametrize("seed", [1, 2, 3])
@pytest.mark.parametrize("n, degree, wmax, delta, wg_deg, teams, members", [
    (200, 12, 30, 15, 16, 2, 2), (120, 110, 255, 100, 64, 1, 3), (150, 4, 1000, 300, 512, 3, 1)])
def test_teams(check, n, degree, wmax, delta, wg_deg, teams, members, seed):
    """Teams in step and with hubs, and one whose members wait for long by the clock (off
    the GPU for ten seconds between two reads of it)."""
    for step in (1, 10**9):
        check("team", n, degree, wmax, delta, wg_deg, seed, teams, members, step, 0)


@pytest.mark.parametrize("looks", [1, 3, 10, 30, 100, 300, 1000, 3000])
def test_failed_team_barrier_is_reported(check, looks):
    """Members that give a barrier up after a few looks, each at another one: every
    workgroup ends, and a result that lacks a share is never taken for one."""
    failed = sum("failed" in check("team", 200, 12, 30, 15, 16, seed, 2, 2, 1, looks)
                 for seed in range(1, 9))
    assert failed > 0 or looks > 1  # at one look, whoever arrives first gives up
