"""Which form of the bf16 attention kernel a call gets (csrc/attend_plan.h, host code, no GPU): the lists of query tiles are
walked here as the kernel walks them, and the form taken has to be about the one whose longest sequence is shortest.
Head counts that do not fill the XCDs alike, where one XCD has many more tiles than the chip has on average."""
import ctypes
import os
import subprocess

import pytest

from paper_2512_07090_amd import build

PAIRS, SINGLES, HALVES, NARROW = range(4)
N_CU, N_XCD = 256, 8


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(
        '#include "attend_plan.h"\n'
        'extern "C" int plan(int B, int Hq, int m, int ragged, int n_cu, int n_xcd)\n'
        "{ return tf::plan_attend(B, Hq, m, ragged, n_cu, n_xcd); }\n")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", build.CSRC, str(d / "plan.cpp"), "-o",
                    str(d / "plan.so")], check=True)
    f = ctypes.CDLL(str(d / "plan.so")).plan
    return lambda *shape: f(*shape, N_CU, N_XCD)


def longest(form, B, Hq, m, ragged):
    """us of the longest sequence of any compute unit, from the measured cost of a tile in each form."""
    size = 256 if form in (PAIRS, SINGLES) else 128
    n_qt = -(-m // size)
    keys = [-(-min((t + 1) * size, m) // 64) for t in range(n_qt)]       # key tiles of a query tile
    n_groups, worst = B * Hq, 0.0
    for x in range(N_XCD):
        groups = range(x * n_groups // N_XCD, (x + 1) * n_groups // N_XCD)
        resident = (2 if form == NARROW else 1) * N_CU // N_XCD
        workgroups = min(-(-n_groups // N_XCD) * n_qt, resident)
        if form == PAIRS:
            tiles = [(n_qt - 1 - p, p) if p != n_qt - 1 - p else (p,) for _ in groups for p in range((n_qt + 1) // 2)]
        else:
            rows = [[g for g in groups if g // Hq == b] for b in range(B)] if ragged else [groups]
            tiles = [(t,) for row in rows for t in reversed(range(n_qt)) for _ in row]
        sums = [[0, 0] for _ in range(workgroups)]                       # tiles, key tiles
        for e, item in enumerate(tiles):
            r, at = divmod(e, workgroups)
            if form in (SINGLES, HALVES) and r & 1:
                at = workgroups - 1 - at
            if form == NARROW and at >= N_CU // N_XCD:
                at = workgroups - 1 - (at - N_CU // N_XCD)
            for t in item:
                sums[at][0] += 1
                sums[at][1] += keys[t]
        if form == NARROW:
            for j in range(min(workgroups, N_CU // N_XCD)):
                a, b = sums[j][1], sums[j + N_CU // N_XCD][1] if j + N_CU // N_XCD < workgroups else 0
                worst = max(worst, 8.5 + 1.42 * min(a, b) + 1.2 * abs(a - b))
        else:
            item, key = (6.0, 1.1) if form == HALVES else (11.0, 1.47)
            worst = max([worst] + [item * n + key * k for n, k in sums])
    return worst


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("shape", [   # batch, query heads, kept
    (1, 1, 2048), (1, 1, 9117), (1, 1, 11600), (1, 1, 13000), (1, 1, 16384), (1, 9, 1500), (1, 9, 3000), (1, 9, 7000),
    (3, 3, 7000), (9, 1, 7000), (5, 2, 3000), (5, 2, 6000), (1, 12, 5000), (17, 1, 3600), (1, 33, 1024), (1, 32, 1024)])
def test_the_form_with_the_shortest_longest_sequence(plan, shape, ragged):
    us = [longest(form, *shape, ragged) for form in range(4)]
    assert us[plan(*shape, ragged)] <= 1.12 * min(us), us
