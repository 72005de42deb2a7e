"""A CPU model of the two-group form of hb_sat2d's grid-wide wait (the one-group form has its own), with fewer execution
slots than workgroups, tiny wait limits and random delays.

Workgroups below `first` form a group that waits for itself alone; its `go`, once raised, is one more arrival of the
second group, whose `go` therefore stands for all.  Claims: every thread ends, every region is finished, no region is
finished before all regions that it reads (those of the first group, or all) have published, and the workspace holds
the tables of both region shapes.
"""
import os
import random
import re
import threading
import time

import pytest


class Grid:
    def __init__(self, nwg, first, slots, wait_limit, seed):
        self.nwg, self.first, self.wait_limit = nwg, first, wait_limit
        self.slots = threading.Semaphore(slots)
        self.mu = threading.Lock()
        self.size = (first, nwg - first)
        self.nleaf = [min(n, 8) for n in self.size]
        self.leaf = [[0] * n for n in self.nleaf]
        self.root = [0, 0]
        self.go = [0, 0]
        self.late = 0
        self.todo = [0] * nwg
        self.published = [False] * nwg
        self.finished = [0] * nwg
        self.errors = []
        self.rng = random.Random(seed)

    def pause(self):
        if self.rng.random() < 0.3:
            time.sleep(self.rng.random() * 2e-4)

    def add(self, counters, i):
        with self.mu:
            counters[i] += 1
            return counters[i]

    def finish(self, region):
        with self.mu:
            if not all(self.published[:self.first if region < self.first else self.nwg]):
                self.errors.append(f"region {region} finished too early")
            self.finished[region] += 1

    def workgroup(self, wg):
        with self.slots:
            self.pause()
            with self.mu:
                self.published[wg] = True
            group = 0 if wg < self.first else 1
            idx, n = wg - group * self.first, self.size[group]
            lf = idx % self.nleaf[group]
            every = group == 1
            if self.add(self.leaf[group], lf) == (n - lf + self.nleaf[group] - 1) // self.nleaf[group]:
                if self.add(self.root, group) == self.nleaf[group] + group:
                    with self.mu:
                        self.go[group] = 1
                    if group == 0:
                        self.pause()
                        if self.add(self.root, 1) == self.nleaf[1] + 1:
                            with self.mu:
                                self.go[1] = 1
                            every = True
            passed, polls = True, 0
            while not self.go[group]:
                polls += 1
                if polls > self.wait_limit:
                    passed = False
                    break
                self.pause()
            if not passed:
                with self.mu:
                    self.todo[wg] = 1
                    self.late = 1
                self.pause()
                with self.mu:
                    go = self.go[group]
                    if go and self.todo[wg] == 1:
                        self.todo[wg] = 2
                if not go:
                    return
            with self.mu:
                late = self.late
            self.pause()
            self.finish(wg)
            while late:
                claimed = -1
                with self.mu:
                    for r in range(self.nwg if every else self.first):
                        if self.todo[r] == 1:
                            self.todo[r], claimed = 2, r
                            break
                if claimed < 0:
                    return
                self.pause()
                self.finish(claimed)


@pytest.mark.parametrize("nwg,first,slots,wait_limit", [(2, 1, 1, 0), (3, 2, 3, 50), (40, 20, 7, 3), (40, 24, 7, 0),
                                                        (97, 49, 5, 1), (256, 128, 16, 2), (64, 32, 64, 0)])
def test_two_groups_end_and_finish_every_region(nwg, first, slots, wait_limit):
    for seed in range(3):
        g = Grid(nwg, first, slots, wait_limit, seed)
        threads = [threading.Thread(target=g.workgroup, args=(w,), daemon=True) for w in range(nwg)]
        g.rng.shuffle(threads)
        for t in threads:
            t.start()
        for t in threads:
            t.join(timeout=30)
            assert not t.is_alive(), "a workgroup never ended"
        assert not g.errors, g.errors[0]
        assert all(g.finished), f"unfinished regions: {[r for r, n in enumerate(g.finished) if n == 0]}"
        assert g.go == [1, 1]


def test_workspace_holds_the_tables_of_both_region_shapes():
    """The tables lie at the workspace's start and the words of the wait at its end, in the room that the library asks for."""
    from paper_2512_02371_amd import hb
    text = open(os.path.join(os.path.dirname(__file__), "..", "paper_2512_02371_amd", "csrc", "sat_wait.hpp")).read()
    k = {n: int(v) for n, v in re.findall(r"\b(k\w+) = (\d+)", text)}
    words = (k["kLeaves"] + 1 + k["kGo"] + 1) * k["kLine"] + k["kMaxRegions"]
    assert words == 26 * 32 + 1024

    def up(a, b):
        return -(-a // b)

    rng = random.Random(5)
    sizes = [(H, W) for H in (1, 64, 65, 128, 129, 257, 1000, 2896, 4096, 9000, 40000, 1 << 20)
             for W in (1, 64, 65, 256, 257, 300, 1917, 4096, 33000, 1 << 20)]
    sizes += [tuple(int(2 ** rng.uniform(0, 17)) for _ in range(2)) for _ in range(3000)]
    taken = set()
    for H, W in sizes:
        small, pieces = up(H, 128) * up(W, 128), up(H, 256) * up(W, 256)
        if pieces >= 128 and pieces > k["kMaxRegions"]:
            continue                                       # three launches
        tc = 4 if pieces >= 128 or small > k["kMaxRegions"] else 2
        nsw, nbw = up(H, 128), up(W, 64 * tc)
        if H <= 128 and W <= 256:
            continue                                       # one region publishes nothing
        taken.add(tc)
        room = hb.hb_sat2d_workspace_size(H, W) // 4 - words
        assert nsw * nbw * (128 + 64 * tc + 1) <= room, (H, W, tc)
    assert taken == {2, 4}


class Words:
    """The words of the wait, with anything in them before the first launch."""

    def __init__(self, seed):
        rng = random.Random(seed)
        self.mu = threading.Lock()
        self.claim, self.ready, self.arrived = (rng.choice((0, 5, 77)) for _ in range(3))


def launch(w, call, nwg, slots, patience, rng):
    sem, seen = threading.Semaphore(slots), []

    def take():
        with w.mu:
            mine, w.claim = w.claim != call, call
        if mine:
            time.sleep(rng.random() * 3e-4)
            w.arrived = 0
            w.ready = call

    def workgroup(wg):
        with sem:
            if wg == 0:
                take()
            polls = 0
            while w.ready != call:
                polls += 1
                if polls == patience:
                    take()
                time.sleep(1e-5)
            with w.mu:
                w.arrived += 1
                seen.append(w.arrived)
                if w.arrived == nwg:
                    w.ready = w.claim = 0

    threads = [threading.Thread(target=workgroup, args=(i,), daemon=True) for i in range(nwg)]
    rng.shuffle(threads)
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=30)
        assert not t.is_alive(), "a workgroup never ended"
    return seen


@pytest.mark.parametrize("nwg,slots,patience", [(1, 1, 3), (17, 17, 1000), (17, 4, 3), (40, 1, 2), (40, 40, 1)])
def test_words_are_cleared_once_before_the_first_arrival(nwg, slots, patience):
    """Launches with numbers of their own and replays of one number, workgroup 0 first or last to run."""
    rng = random.Random(nwg + slots)
    w = Words(nwg)
    for call in (1001, 1002, 1002, 1002, 1003, 1002):
        assert launch(w, call, nwg, slots, patience, rng) == list(range(1, nwg + 1))
