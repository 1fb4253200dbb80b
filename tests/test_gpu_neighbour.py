"""GPU parity of the neighbour-stepped matching kernel where its dispatch and
its tables change: whole schedules and statistics against the CPU oracle
(integers, so equality is exact), and the kernel that ran."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_07019_amd import workloads as W

pytestmark = pytest.mark.gpu


def _generic(name, topo, n_chunks, chunk_bytes, max_dests, seed):
    """Random sources and 1..max_dests destinations over all NPUs."""
    rng = W.SplitMix64(seed)
    n, src, dests = topo.n_npus, [], []
    for _ in range(n_chunks):
        s, k = rng.rand(n), 1 + rng.rand(max_dests)
        src.append(s)
        dests.append(sorted({rng.rand(n) for _ in range(k)} - {s}))
    return W.Workload(name, topo, W.collective_from_lists(n, n_chunks, chunk_bytes, src, dests, [range(n)]), seed)


def _digraph(n, degree, seed):
    rng = W.SplitMix64(seed)
    pairs = W.random_digraph(n, degree, rng)
    return W.make_topology(n, 0, pairs, [300 + rng.rand(900) for _ in pairs], [(20, 35, 90)[rng.rand(3)] for _ in pairs])


def _complete(n):
    return W.make_topology(n, 0, [(i, j) for i in range(n) for j in range(n) if i != j], 500, 50)


def _slow_link(ratio, fast=1000, chunk=100):
    """An 8-ring whose links take `fast` ns but one pair that takes ratio times
    as long: the kernel is chosen up to a factor of 9."""
    pairs = [(i, (i + s) % 8) for i in range(8) for s in (1, 7)]
    alpha = [fast - chunk + (ratio - 1) * fast * ({a, b} == {3, 4}) for a, b in pairs]
    return W.make_topology(8, 0, pairs, alpha, 1)


CASES = {
    # one-way links: readers that are no sources (their progress is polled, not their entries)
    "one-way ring 5": lambda: _generic("ring5", W.ring(5, bidirectional=False), 40, 4096, 3, 1),
    "one-way ring 70": lambda: _generic("ring70", W.ring(70, bidirectional=False), 300, 4096, 4, 2),
    "digraph 60 degree 2": lambda: _generic("digraph60", _digraph(60, 2, 3), 500, 20000, 6, 3),
    "digraph 300 degree 3": lambda: _generic("digraph300", _digraph(300, 3, 4), 3000, 20000, 5, 4),
    # two NPUs that only follow each other's progress (either may be ahead by up to three windows), also over more windows
    # than the 4,096 that a tag counts
    "pair": lambda: _generic("pair", W.make_topology(2, 0, [(0, 1), (1, 0)], [500, 700], 10), 6000, 4096, 1, 16),
    "pair, long": lambda: _generic("pairl", W.make_topology(2, 0, [(0, 1), (1, 0)], [500, 700], 10), 20000, 4096, 1, 31),
    # leaves: an NPU whose only neighbour follows its progress
    "star 3": lambda: W.Workload("star3", W.star(3), W.all_gather(3, range(3), 300, 4096), 17),
    # 56 and 72 polled entries per device: one and several per lane
    "complete 9": lambda: _generic("complete9", _complete(9), 200, 10000, 8, 5),
    "complete 10": lambda: _generic("complete10", _complete(10), 200, 10000, 9, 6),
    # several polled entries per lane in one-way and switched networks
    "digraph 40 degree 9": lambda: _generic("digraph40", _digraph(40, 9, 18), 1200, 20000, 30, 18),
    "digraph 90 degree 9": lambda: _generic("digraph90", _digraph(90, 9, 19), 2500, 20000, 2, 19),
    "rail 12x6 all-gather": lambda: W.Workload("rail12ag", W.switch2level(12, 6), W.all_gather(72, range(72), 5, 9000), 20),
    "rail 12x8 generic": lambda: _generic("rail12g", W.switch2level(12, 8), 3000, 7000, 9, 21),
    "rail 13x8": lambda: W.Workload("rail13x8", W.switch2level(13, 8), W.a2a_bitmaps(104, 8192), 22),
    # more than 128 polled entries and 4,096 chunks, pruned to those a needed chunk can come through: one-way and switched
    # networks, chunks with one and with many destinations, a chunk that several neighbours can offer; both bounds
    "digraph 40 degree 13": lambda: _generic("digraph40p", _digraph(40, 13, 25), 4200, 20000, 30, 25),
    "digraph 90 degree 12": lambda: _generic("digraph90p", _digraph(90, 12, 26), 4100, 20000, 2, 26),
    "rail 20x8 generic": lambda: _generic("rail20g", W.switch2level(20, 8), 4200, 7000, 9, 27),
    "rail 20x8 all-gather": lambda: W.Workload("rail20ag", W.switch2level(20, 8), W.all_gather(160, range(0, 160, 14), 342, 9000), 28),
    "complete 13, 4,096": lambda: _generic("c13a", _complete(13), 4096, 10000, 6, 29),
    "complete 13, 4,097": lambda: _generic("c13b", _complete(13), 4097, 10000, 6, 29),
    "rail 18x8": lambda: W.Workload("rail18", W.switch2level(18, 8), W.a2a_bitmaps(144, 8192), 30),
    # 64 and 65 chunks (one and two row words), 4,096 and 4,160 (one and two summary levels), all needed everywhere
    "ring 4 x 16": lambda: W.Workload("r4", W.ring(4), W.all_gather(4, range(4), 16, 1 << 14), 7),
    "ring 5 x 13": lambda: W.Workload("r5", W.ring(5), W.all_gather(5, range(5), 13, 1 << 14), 8),
    "ring 8 x 512": lambda: W.Workload("r8", W.ring(8), W.all_gather(8, range(8), 512, 1 << 14), 9),
    "ring 8 x 520": lambda: W.Workload("r8b", W.ring(8), W.all_gather(8, range(8), 520, 1 << 14), 10),
    # link times a factor of 9 apart, and of more
    "slow link 9": lambda: _generic("slow9", _slow_link(9), 60, 100, 4, 21),
    "slow link 10": lambda: _generic("slow10", _slow_link(10), 60, 100, 4, 22),
    "slow link 64": lambda: _generic("slow64", _slow_link(64), 60, 100, 4, 11),
    "slow link 65": lambda: _generic("slow65", _slow_link(65), 60, 100, 4, 12),
    # the same bound where the fastest link takes 1 ns
    "slow link 9 of 1 ns": lambda: _generic("fast9", _slow_link(9, 1, 1), 60, 1, 4, 24),
    "slow link 10 of 1 ns": lambda: _generic("fast10", _slow_link(10, 1, 1), 60, 1, 4, 24),
    # four waves per workgroup, and one device too many for them
    "mesh 32x32": lambda: _generic("mesh1024", W.mesh2d(32, 32), 600, 4096, 6, 13),
    "mesh 41x25": lambda: _generic("mesh1025", W.mesh2d(41, 25), 600, 4096, 6, 14),
    # switches with 16,128 columns: their column list stays in device memory
    "rail 64x4": lambda: W.Workload("rail64x4", W.switch2level(64, 4), W.a2a_bitmaps(256, 8192), 15),
    # a switch of 64 in-links and 8,064 columns that shares its LDS: its candidate rows stay in device memory, set by one
    # lane and read by another
    "star 64 x 2": lambda: W.Workload("star64", W.star(64), W.a2a_k_bitmaps(64, 2, 8192), 23),
}


# the kernel expected on each side of its rule, and where polled entries are pruned
WINDOWED = {"slow link 10", "slow link 10 of 1 ns", "slow link 64", "slow link 65", "mesh 41x25"}
PRUNED = {"digraph 40 degree 13", "digraph 90 degree 12", "rail 20x8 generic", "rail 20x8 all-gather", "complete 13, 4,097",
          "rail 64x4"}


@pytest.mark.parametrize("name", list(CASES))
def test_neighbour_stepped_parity(name):
    from paper_2606_07019_amd.pccl import Synthesizer
    print(f"[neighbour] {name}", flush=True)
    wl = CASES[name]()
    ref = O.run_workload(wl)
    assert ref.status == 0, ref.message
    s = Synthesizer(wl.topo, wl.coll, tie_seed=wl.tie_seed)
    try:
        for _ in range(2):   # the second run starts from the first one's tables
            s.synthesize()
            np.testing.assert_array_equal(s.schedule(), ref.sends)
            assert s.collective_time == ref.collective_time
            st = s.stats()
            assert [st[k] for k in ("events", "rounds", "clashes")] == [ref.stats[k] for k in ("events", "rounds", "clashes")]
            assert s.kernel() == ("windowed" if name in WINDOWED else "neighbour", name in PRUNED)
    finally:
        s.close()
