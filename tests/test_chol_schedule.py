"""The schedule of the single-launch Cholesky factorisation (chol_chain_kernel in csrc/chol_panel.hip), on the CPU: the chain and every
team of the helpers as a coroutine that runs its tasks in the kernel's order and waits for the kernel's flags, in random interleavings.
Checked: each update finds the tiles of L it reads finished and is applied once and in panel order, flags only ever count up and
only over finished tiles, a team's wait covers every row it reads, nobody waits for ever, and at the end everything is there.
A change of ownership, order or flags in the kernel belongs in here too."""
import random
import shutil
import subprocess

import pytest

from paper_2504_05295_amd import build


def near_order(nb, pr, pc):
    """near_order() of csrc/chol_order.hpp: (shift, far) of the near-diagonal tasks' order over pr * pc helper workgroups"""
    groups, rounds, tasks = pr * pc, 2 * pr, 3 * nb
    beyond = ((nb % rounds) * pc + 1) // 2
    if nb < rounds:
        far = beyond > 0 and tasks + beyond <= groups
    else:
        far = beyond > 0 and groups >= 63 and groups < tasks < 2 * groups and tasks - groups + beyond <= groups
    shift = groups - beyond if nb > rounds and tasks <= groups and 5 * beyond >= 2 * tasks else 0
    return shift, far


class Schedule:
    def __init__(self, nb, pr, pc, inverse, mistake=None):
        self.nb, self.pr, self.pc, self.teams, self.inverse, self.mistake = nb, 2 * pr, pc, 2 * pr * pc, inverse, mistake
        self.shift, self.far = near_order(nb, pr, pc)
        self.w11 = [False] * nb                    # W11(k) is out
        self.lflag = [0] * nb                      # L[i][0 .. lflag[i]) are out
        self.near = {}                             # (i, d): that tile may go to the chain (d = 2: L[i][i-2] is out)
        self.done = set()                          # finished tiles of L
        self.updates = {(i, j): [] for i in range(nb) for j in range(i + 1)}
        self.copies = {}                           # (i, d): panels applied to team d's copy of (i, i-2)
        self.wflag, self.running, self.halves = set(), {}, set()

    # what tasks do
    def update(self, i, j, p):
        assert (i, p) in self.done and (j, p) in self.done, ("operand", i, j, p)
        assert self.updates[i, j] == list(range(p)), ("order", i, j, p, self.updates[i, j])
        self.updates[i, j].append(p)

    def finish(self, i, p, by_copy=None):
        have = self.updates[i, p] if by_copy is None else self.copies.get(by_copy, [])
        assert self.w11[p] and have == list(range(p)), ("tile of L", i, p, have)

    def raise_count(self, i, n):
        assert self.lflag[i] < n and all((i, q) in self.done for q in range(n)), ("count", i, n)
        self.lflag[i] = n

    def chain(self):
        for k in range(self.nb):
            assert self.updates[k, k] == list(range(k))
            yield None
            if 1 <= k < self.nb - 1:
                flags = (0, 1) if self.mistake == "chain ignores the third flag" else (0, 1, 2)
                yield lambda: all((k + 1, d) in self.near for d in flags)
            self.w11[k] = True
            if k + 1 == self.nb:
                return
            yield None
            self.finish(k + 1, k)
            self.done.add((k + 1, k))
            yield None
            self.update(k + 1, k + 1, k)
            yield None
            self.raise_count(k + 1, k + 1)

    def helper(self, group, team):
        nb, pr, pc, teams = self.nb, self.pr, self.pc, self.teams
        h = 2 * group + team
        a, b = h // pc, h % pc
        x = (group + self.shift) % (teams // 2)
        near_h = team * (teams // 2) + (teams // 2 - 1 - x if self.far else x)

        def near_of(i):
            return (near_h - 3 * i) % teams

        def first(start, residue, step):          # the first index from `start` on that is residue mod step
            return start + (residue - start) % step

        def reads(t):
            d = near_of(t)
            near_rows = d < 3 or d == 4 or (6 <= d < 9 and self.mistake != "second row of a task not waited for")
            return t % pr == a or t % pc == b or near_rows

        def near_update(i, d, p):
            if d < 2:
                self.update(i, i - d, p)
            assert (i, p) in self.done and (i - 2, p) in self.done
            copy = self.copies.setdefault((i, d), [])
            assert copy == list(range(p)), (i, d, p, copy)
            copy.append(p)

        def w_ready(p, e):
            return self.w11[p] if e == p else (p, e) in self.wflag

        def w_update(j, e, p):
            assert (j, p) in self.done and w_ready(p, e)
            got = self.running.setdefault((j, e), [])
            assert got == list(range(e, p)), (j, e, p, got)
            got.append(p)

        def w_rest(p):
            j0 = first(p + 2, a, pr)
            if j0 >= nb or b > p:
                return
            yield lambda: all(w_ready(p, t) for t in range(b, p + 1, pc))
            for j in range(j0, nb, pr):
                for e in range(b, p + 1, pc):
                    w_update(j, e, p)
                    yield None

        def w_row(p):
            if p < 1 or p % pr != a or b > p - 1:
                return
            yield lambda: all(w_ready(p - 1, t) for t in range(b, p, pc))
            yield lambda: self.lflag[p] >= p
            for e in range(b, p, pc):
                w_update(p, e, p - 1)
            for e in range(b, p, pc):
                yield lambda: self.w11[p]
                assert self.running[p, e] == list(range(e, p))
                yield None
                self.wflag.add((p, e))
                self.halves.add((p, e))

        def w_diag(p):
            if p % pr == a and p % pc == b:
                yield lambda: self.w11[p]
                self.halves.add((p, p))

        near0 = near_h
        for p in range(nb - 1):
            i, d = p + 2, near_of(p + 2)
            if i < nb and d < 3:                   # the row that feeds the chain
                if d == 1:
                    yield lambda: self.lflag[p + 1] >= p + 1
                else:
                    yield lambda: self.w11[p]
                self.finish(i, p, (i, d))
                yield None
                if d == 2:
                    assert (i, p) not in self.done
                    self.done.add((i, p))
                else:
                    # (the tile's last update, with a private L[i][p])
                    assert self.updates[i, i - d] == list(range(p)) and (d == 0 or (p + 1, p) in self.done)
                    self.updates[i, i - d].append(p)
                yield None
                if d == 2:
                    self.raise_count(i, p + 1)
                    yield None
                self.near[i, d] = True
            if p % pc == b:
                for i in range(first(p + 3, a, pr), nb, pr):
                    yield lambda: self.w11[p]
                    self.finish(i, p)
                    assert (i, p) not in self.done
                    self.done.add((i, p))
                    yield None
                    self.raise_count(i, p + 1)
            i, d = p + 3, near_of(p + 3)
            if i < nb and d < 3:
                yield lambda: all(self.lflag[t] >= p + 1 for t in ((i, i - 2, i - 1) if d == 1 else (i, i - 2)))
                near_update(i, d, p)
                yield None
            if self.inverse:
                if p >= 1:
                    yield from w_rest(p - 1)
                yield from w_row(p)
                yield from w_diag(p)
            yield lambda: all(self.lflag[t] >= p + 1 for t in range(p + 1, nb) if reads(t))
            while near0 < 3 * (p + 4):
                near0 += teams
            for n in range(near0, 3 * nb, teams):
                near_update(n // 3, n % 3, p)
                yield None
            for j in range(first(p + 1, b, pc), nb, pc):
                for i in range(first(j + 3, a, pr), nb, pr):
                    self.update(i, j, p)
                    yield None
        if self.inverse:
            yield from w_row(nb - 1)
            yield from w_diag(nb - 1)

    def run(self, seed):
        rnd = random.Random(seed)
        live = [[self.chain(), None]] + [[self.helper(g, t), None] for g in range(self.teams // 2) for t in range(2)]
        while live:
            progress = False
            rnd.shuffle(live)
            for task in list(live):
                for _ in range(rnd.choice((1, 1, 1, 2, 20))):
                    if task[1] is not None and not task[1]():
                        break
                    progress = True
                    try:
                        task[1] = next(task[0])
                    except StopIteration:
                        live.remove(task)
                        break
            assert progress, "everybody waits"
        nb = self.nb
        assert len(self.done) == nb * (nb - 1) // 2
        assert all(u == list(range(j)) for (i, j), u in self.updates.items() if i - j != 2)
        if self.inverse:
            assert self.wflag == {(p, e) for p in range(nb) for e in range(p)} and self.halves == self.wflag | {(p, p) for p in range(nb)}


# the three grids of plan_chol_grid, sizes around whole rounds of each and around the lines of near_order
@pytest.mark.parametrize("grid,sizes", [((3, 5), [4, 5, 6, 7, 11, 12, 13, 18, 31, 40]), ((7, 9), [4, 8, 9, 14, 15, 19, 20, 22, 25, 26, 28, 33, 40, 64]),
                                        ((15, 17), [16, 22, 24, 30, 31, 35, 36, 46, 59, 60, 64])])
def test_schedule(grid, sizes):
    for nb in sizes:
        for inverse in (False, True):
            for seed in range(3 if nb <= 24 else 1):
                Schedule(nb, *grid, inverse).run(seed)


def test_schedule_without_inverse():
    for nb in (65, 86, 128):
        Schedule(nb, 15, 17, False).run(0)
    Schedule(100, 7, 9, False).run(0)


@pytest.mark.parametrize("grid", [(3, 5), (7, 9), (15, 17)])
def test_order_of_near_diagonal_tasks(grid):
    pr, pc = grid
    for nb in range(4, 129):
        shift, far = near_order(nb, pr, pc)
        groups = pr * pc
        assert 0 <= shift < groups and not (shift and far)
        place = [(x := (g + shift) % groups, groups - 1 - x if far else x)[1] for g in range(groups)]
        assert sorted(place) == list(range(groups))           # one team for every task
        held = {g for g in range(groups) if place[g] < 3 * nb}
        beyond = ((nb % (2 * pr)) * pc + 1) // 2
        if shift or (far and nb < 2 * pr):
            # as many tasks as there are workgroups without rows beyond the last whole round lie on those
            assert len(held - set(range(beyond))) == min(len(held), groups - beyond), (nb, len(held))


def test_rule_is_the_launchers(tmp_path):
    compiler = shutil.which("g++") or shutil.which("c++")
    if compiler is None:
        pytest.skip("no C++ compiler")
    source = tmp_path / "order.cpp"
    source.write_text("""#include <cstdio>
#include "chol_order.hpp"
int main() {
  const int grids[3][2] = {{3, 5}, {7, 9}, {15, 17}};
  for (auto& g : grids)
    for (int nb = 4; nb <= 128; ++nb) {
      const dion::NearOrder o = dion::near_order(nb, g[0], g[1]);
      std::printf("%d %d %d %d %d\\n", nb, g[0], g[1], o.shift, (int)o.far);
    }
}
""")
    subprocess.run([compiler, "-std=c++17", "-I", build.CSRC, str(source), "-o", str(tmp_path / "order")], check=True)
    lines = subprocess.run([str(tmp_path / "order")], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]
    assert len(lines) == 3 * 125
    for line in lines:
        nb, pr, pc, shift, far = map(int, line.split())
        assert near_order(nb, pr, pc) == (shift, bool(far)), line


@pytest.mark.parametrize("mistake", ["chain ignores the third flag", "second row of a task not waited for"])
def test_a_mistake_is_noticed(mistake):
    with pytest.raises(AssertionError):
        for seed in range(20):
            Schedule(24, 7, 9, False, mistake).run(seed)
