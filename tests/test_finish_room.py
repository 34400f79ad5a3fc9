"""The (core, phase, degree class) cells of the level peel's finish, on the CPU: for every number of
vertices they stay within the arrays that hold them, and for graphs whose cells come near the room -- a
part of one high core number, a path of many phases, isolated vertices -- so does the cell of every vertex.  The phases are
those of the finish: every bound replaced at once by the largest t such that t neighbours have bounds of
at least t, until none falls."""
import functools
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2106_02762_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "finish_room.h"
using dt::FinishRoom;
int main() {
    std::printf("%u %u %llu %llu %llu %llu %llu %llu\n", dt::kTail, FinishRoom::kClasses, (unsigned long long)FinishRoom::kBase,
                (unsigned long long)FinishRoom::kCur, (unsigned long long)FinishRoom::kWhen,
                (unsigned long long)FinishRoom::kPos, (unsigned long long)FinishRoom::kVal,
                (unsigned long long)FinishRoom::kWords);
    for (uint32_t R = 1; R <= dt::kTail; ++R) std::printf("%u\n", FinishRoom::cells(R));
}
"""


@pytest.fixture(scope="module")
def room(tmp_path_factory):
    d = tmp_path_factory.mktemp("room")
    (d / "room.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-o", str(d / "room"), str(d / "room.cpp")], check=True)
    head, *cells = subprocess.run([str(d / "room")], check=True, capture_output=True, text=True).stdout.split("\n")[:-1]
    return [int(x) for x in head.split()], [0] + [int(x) for x in cells]


def test_arrays_hold_every_count_of_cells(room):
    (tail, _, base, cur, when, pos, val, words), cells = room
    assert len(cells) == tail + 1
    for R in range(1, tail + 1):
        assert R <= cells[R] <= min(cur - base, when - cur), R
    assert pos - when >= tail and val - pos >= tail
    assert words - val >= tail          # two buffers of 16-bit bounds
    assert val % 4 == 0                 # read 16 bytes at a time


@functools.lru_cache(None)
def _path_phases(k):
    """Phase + 1 in which each bound of a path of k >= 2 vertices last fell, and the phases in all."""
    h = np.full(k, 2)
    h[[0, -1]] = 1
    when, ph = np.zeros(k, np.int64), 0
    while True:
        left, right = np.append(0, h[:-1]), np.append(h[1:], 0)
        new = np.where(np.minimum(left, right) >= 2, 2, np.where(np.maximum(left, right) >= 1, 1, 0))
        new = np.minimum(new, h)
        ph += 1
        when[new < h] = ph
        if (new == h).all():
            return when, ph
        h = new


@pytest.mark.parametrize("R", [8160, 8161, 8175, 8190, 8191, 8192, 8193])
@pytest.mark.parametrize("core,path", [(2629, 200), (2621, 200), (1314, 400), (1310, 400), (2032, 258), (130, 4000),
                                       (657, 200), (655, 200), (654, 200), (650, 200), (327, 400), (326, 400), (64, 2000)])
def test_cells_of_a_high_core_beside_a_path(room, R, core, path):
    (_, classes, base, cur, when_at, _, _, _), cells = room
    when, T = _path_phases(path)
    shells = core + 1                                # isolated vertices are the lowest shell
    if shells * T * classes > cells[R]:                        # the finish counts shells only
        assert min(shells, cells[R]) <= min(cur - base, when_at - cur)
        return
    top = max(core * T, T + int(when.max())) * classes + classes - 1
    assert top < min(cur - base, when_at - cur), (top, shells * T * classes, cells[R])
