"""The enqueued rounds of the pointer-jumping loops suffice: a host model of the two loops on a single path (the deepest
tree a forest can be), every row reading what the round before left, at each row count from 1 on, around every bound and
at the longest lengths that the reach formula covers. The bounds themselves are compiled from the library's header."""
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2311_10337_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include "rounds.h"
int main() {
  long long k;
  while (std::scanf("%lld", &k) == 1)
    std::printf("%d %d %d\n", ce::HOPS, ce::rounds_to_arrive(k), ce::rounds_to_confirm(k));
}
"""


@pytest.fixture(scope="module")
def bounds(tmp_path_factory):
    d = tmp_path_factory.mktemp("rounds")
    (d / "rounds.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "rounds.cpp"), "-o", str(d / "rounds")], check=True)

    def f(links):
        out = subprocess.run([str(d / "rounds")], input="\n".join(str(x) for x in links), capture_output=True,
                             text=True, check=True).stdout
        return [tuple(int(x) for x in line.split()) for line in out.splitlines()]
    return f


def last_round_of_tops(rows, hops):
    """k_dd_top_jump on one path whose last row is the top: rounds until the list is empty."""
    top = np.minimum(np.arange(rows) + 1, rows - 1)
    act = np.arange(rows - 1)
    r = 0
    while len(act):
        t = top[act]
        tt = top[t]
        for _ in range(1, hops):  # (at the top t == tt stays)
            t, tt = tt, top[tt]
        new = top.copy()
        new[act] = tt
        act = act[tt != t]
        top = new
        r += 1
    assert (top == rows - 1).all()
    return r


def last_round_of_arrivals(rows, hops):
    """k_cd_jstep on a path of big rows without births under a virtual root (node `rows`)."""
    J = np.arange(rows) + 1
    act = np.nonzero(J < rows)[0]
    r = 0
    while len(act):
        x = J[act]
        for _ in range(hops):
            x = np.where(x < rows, J[np.minimum(x, rows - 1)], x)
        new = J.copy()
        new[act] = x
        act = act[x < rows]
        J = new
        r += 1
    assert (J == rows).all()
    return r


def test_model_of_both_loops(bounds):
    near = [500, 501, 502, 503, 511, 512, 513, 2500, 2501, 2502, 12501, 12502, 62500, 62501, 62502, 62503, 65535, 65536,
            78125, 78126, 200001]
    sizes = sorted(set(list(range(1, 140)) + near))
    for rows, (hops, _, conf), (_, arr, _) in zip(sizes, bounds([max(s - 1, 0) for s in sizes]), bounds(sizes)):
        assert last_round_of_tops(rows, hops) <= conf, rows
        assert last_round_of_arrivals(rows, hops) <= arr, rows


def test_reach_at_every_length(bounds):
    lengths = sorted({b for k in range(1, 33) for b in ((1 << k) - 2, (1 << k) - 1, 1 << k) if b > 0})
    for links, (hops, arr, conf) in zip(lengths, bounds(lengths)):
        assert (hops + 1) ** arr >= links and hops * (hops + 1) ** (conf - 1) >= links, links
        assert arr <= 14 and conf <= 15, links  # the counter words of a loop
