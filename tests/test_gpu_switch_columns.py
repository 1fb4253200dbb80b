"""GPU parity of the switch-group matching kernel over columns where its
dispatch and its tables change: whole schedules and statistics against the
CPU oracle (integers, so equality is exact), and the kernel that ran."""

import pytest

from paper_2606_07019_amd import workloads as W
from tests.test_gpu_neighbour import _generic
from tests.test_gpu_switch import _compare

pytestmark = pytest.mark.gpu


def _meshed_star(n):
    """n NPUs with links between every two of them, and a switch to all."""
    pairs = [(i, j) for i in range(n) for j in range(n) if i != j]
    pairs += [(i, n) for i in range(n)] + [(n, i) for i in range(n)]
    return W.make_topology(n, 1, pairs, [900] * (n * (n - 1)) + [300] * (2 * n), 50)


def _two_switches(n):
    """One-way rings of NPUs and two switches that reach the same NPUs."""
    pairs = [(i, (i + 1) % n) for i in range(n)]
    pairs += [p for s in (n, n + 1) for i in range(n) for p in ((i, s), (s, i))]
    return W.make_topology(n, 2, pairs, [700] * n + [250, 400] * (2 * n), 40)


def _fan(n):
    """4 NPUs that send to n others through one switch."""
    pairs = [(i, 4 + n) for i in range(4)] + [(4 + n, 4 + j) for j in range(n)]
    coll = W.collective_from_lists(4 + n, 80, 4096, [c % 4 for c in range(80)],
                                   [sorted({4 + (c * 7 + k * 5) % n for k in range(9)}) for c in range(80)], [range(4 + n)])
    return W.Workload(f"fan{n}", W.make_topology(4 + n, 1, pairs, 500, 50), coll, 2)


def _limited(wl, buffer, unicast):
    return W.Workload(wl.name, W.with_switch_model(wl.topo, buffer, unicast), wl.coll, wl.tie_seed)


CASES = {
    # 64 out-links of a limited switch (one mask), 65 (the kernel over bitmap rows)
    "fan 64": lambda b, u: _limited(_fan(64), b, u),
    "star 64": lambda b, u: _limited(W.Workload("star64", W.star(64), W.all_gather(64, range(64), 2, 4096), 1), b, u),
    "fan 65": lambda b, u: _limited(_fan(65), b, u),
    # more than 4,096 columns per device: two summary levels
    "star 3 long": lambda b, u: _limited(W.Workload("star3", W.star(3), W.all_gather(3, range(3), 2500, 4096), 3), b, u),
    # a group that polls 1,584 entries (several per thread; pruned over 4,096 chunks) and one of 7,220 (too many: bitmap rows)
    "meshed star 12": lambda b, u: _limited(_generic("mstar12", _meshed_star(12), 400, 9000, 8, 4), b, u),
    "meshed star 12 long": lambda b, u: _limited(_generic("mstar12l", _meshed_star(12), 4100, 9000, 4, 10), b, u),
    "meshed star 20": lambda b, u: _limited(_generic("mstar20", _meshed_star(20), 300, 9000, 8, 5), b, u),
    # two limited switches in one group: chunks come in over both, or past both
    "two switches 9": lambda b, u: _limited(_generic("two9", _two_switches(9), 250, 9000, 6, 6), b, u),
    "two switches 30": lambda b, u: _limited(_generic("two30", _two_switches(30), 900, 9000, 20, 7), b, u),
    # a group per rail
    "rail 9x5": lambda b, u: _limited(W.Workload("rail9", W.switch2level(9, 5), W.all_to_all(45, range(45), 9000), 8), b, u),
    "rail 6x12 a2a": lambda b, u: _limited(W.Workload("rail6a", W.switch2level(6, 12), W.a2a_bitmaps(72, 9000), 11), b, u),
    "rail 6x12": lambda b, u: _limited(W.Workload("rail6", W.switch2level(6, 12), W.all_gather(72, range(72), 3, 9000), 9), b, u),
}


# the kernel expected on each side of its rule, and where polled entries are pruned
ROWS = {"fan 65", "meshed star 20"}
PRUNED = {"meshed star 12 long", "rail 6x12 a2a"}


# buffers of one place, of part of a wave, and of more than 64 places (looked up 64 at a time)
@pytest.mark.parametrize("buffer,unicast", [(1, 1), (7, 0), (70, 1)])
@pytest.mark.parametrize("name", sorted(CASES))
def test_switch_columns_parity(name, buffer, unicast):
    _compare(CASES[name](buffer, unicast), name, ("switch rows" if name in ROWS else "switch columns", name in PRUNED))
