"""The tile relaxation's scheduler (csrc/ff_relax.h) compiled for the host and
run under a simulation of workgroups on a chip (tests/relax_host): whatever the
order of events, every tile ends at the raster-order solution, no tile is
visited twice at once, and the counters, the queue and the count of owed visits
come back to rest."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def relax(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("relax") / "relax_host")
    here = os.path.join(ROOT, "tests", "relax_host")
    subprocess.run(["g++", "-O1", "-std=c++17", "-I", here, "-I", os.path.join(ROOT, "paper_1508_05151_amd", "csrc"),
                    "-I", os.path.join(ROOT, "include"), os.path.join(here, "relax_host.cpp"), "-o", exe], check=True)

    def run(nu, nv, G, slots=10**6, seed=1, stall=0, visit=1500, timeout=2 * 10**6, slow=1, shuffle=0):
        args = [nu, nv, G, slots, seed, stall, visit, timeout, slow, shuffle]
        out = subprocess.run([exe] + [str(int(a)) for a in args], capture_output=True, text=True, timeout=100)
        assert out.returncode == 0, (args, out.stdout, out.stderr)
        w = out.stdout.split()
        return {w[i]: int(w[i + 1]) for i in range(0, len(w), 2)}
    return run


def settled(r):
    return r["status"] == 0 and r["wrong"] == 0 and r["twice"] == 0 and r["left"] == 0


@pytest.mark.parametrize("nu,nv,G", [(1, 1, 1), (2, 1, 2), (12, 10, 120), (12, 10, 17), (40, 1, 40), (1, 30, 7)])
def test_settles_at_the_raster_solution(relax, nu, nv, G):
    """As many workgroups as tiles and fewer, all of them on the chip."""
    for seed in range(3):
        assert settled(relax(nu, nv, G, seed=seed)), seed


def test_queue_entry_taken_once(relax):
    """Few tiles, so that tickets a ring apart share a slot soon, short visits
    and operations held up for much longer than a visit (a workgroup that has
    seen an entry and has not yet taken it)."""
    for nu, nv, seed in [(3, 2, 32), (3, 3, 3), (3, 3, 24), (3, 3, 36), (3, 3, 37), (3, 3, 60), (4, 2, 5)] + \
            [(3, 3, s) for s in range(100, 140)]:
        assert settled(relax(nu, nv, 100, seed=seed, stall=20000, visit=300)), (nu, nv, seed)


@pytest.mark.parametrize("slots", [1, 2, 7, 40, 96, 110])
def test_settles_whatever_places_it_gets(relax, slots):
    """More workgroups than the chip has places for them: those without a tile
    make room for those not yet started, in whichever order these start."""
    for seed in range(2):
        for shuffle in (0, 1):
            assert settled(relax(16, 9, 144, slots=slots, seed=seed, shuffle=shuffle)), (seed, shuffle)
            assert settled(relax(16, 9, 120, slots=slots, seed=seed, stall=300, shuffle=shuffle)), (seed, shuffle)


@pytest.mark.parametrize("nu,visits", [(160, 40), (220, 64)])
def test_watchdog_spares_a_chain_of_visits(relax, nu, visits):
    """One row whose change runs through every tile, one revisit after the
    other in one workgroup while the others wait; a limit shorter than the
    chain and longer than the visits between two signs of progress."""
    r = relax(nu, 1, nu, visit=2000, timeout=visits * 2300, slow=3)
    assert settled(r) and r["visits"] > nu + visits, r


def test_watchdog_fires_on_a_short_limit(relax):
    """The same with a limit of a few visits: the sweep is given up."""
    assert relax(60, 1, 60, visit=2000, timeout=5 * 2300, slow=20)["status"] == -6
