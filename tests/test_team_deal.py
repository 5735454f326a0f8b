"""How a batch's rows are dealt out to teams (ad::team_deal): every deal that is accepted has a kernel (row tiles, keys and XCDs a team are
compiled combinations), hands out every packed row once and stays within the XCDs it was given."""
import ctypes
import random

import pytest

from paper_2205_10350_amd import build

I, P, Z = ctypes.c_int, ctypes.c_void_p, ctypes.c_size_t


class TeamRun(ctypes.Structure):   # ad_team.h
    _fields_ = [("n_teams", I), ("stations", I), ("xcd0", I), ("layers", I), ("head_only", I), ("shared", I),
                ("row_lo", (I * 8) * 2), ("row_n", (I * 8) * 2), ("prob_lo", I * 8), ("prob_n", I * 8), ("prob2_off", I), ("form_ticks", ctypes.c_uint),
                ("scale", ctypes.c_float), ("w", P), ("x", P), ("xa", P), ("s", P), ("slots", P), ("hop", P), ("K", P), ("V", P), ("kv_stride", Z),
                ("Km", P), ("Vm", P), ("m_stride", Z), ("self_desc", P), ("cross_desc", P), ("row_dst", P), ("words", P), ("fail", P),
                ("max_rows", I), ("max_keys", I)]


@pytest.fixture(scope="module")
def lib():
    L = ctypes.CDLL(build.LIB_PATH)
    deal = getattr(L, "_ZN2ad9team_dealEPKiS1_iiiiPNS_7TeamRunE")       # ad::team_deal
    deal.restype = ctypes.c_bool
    deal.argtypes = [ctypes.POINTER(I), ctypes.POINTER(I), I, I, I, I, ctypes.POINTER(TeamRun)]
    has = getattr(L, "_ZN2ad15team_has_kernelEbiii")                    # ad::team_has_kernel
    has.restype = ctypes.c_bool
    has.argtypes = [ctypes.c_bool, I, I, I]
    return deal, has


def _check(lib, rows, rows2=None, xcds=8, layers=6, limit=32):
    """The deal, or None where it is refused."""
    deal, has = lib
    n, t = len(rows), TeamRun()
    if not deal((I * n)(*rows), (I * n)(*rows2) if rows2 else None, n, xcds, layers, limit, ctypes.byref(t)):
        return None
    what = (rows, rows2, xcds, t.n_teams, t.stations, t.max_rows)
    assert 1 <= t.n_teams <= 8 and t.stations >= 1, what
    assert t.stations == 1 or t.n_teams * t.stations <= xcds, what
    assert t.max_rows <= limit and t.max_rows == max(t.row_n[0][j] + t.row_n[1][j] for j in range(t.n_teams)), what
    if limit == 32:
        for dec in (False, True):
            for keys in (1, 64, 65, 128):
                assert has(dec, t.max_rows, keys, t.stations), what
    for s, first in ((0, 0), (1, sum(rows))):      # every row of a segment once, in order
        at = first
        for j in range(t.n_teams):
            if t.row_n[s][j]:
                assert t.row_lo[s][j] == at, what
                at += t.row_n[s][j]
        assert at - first == (sum(rows) if s == 0 else sum(rows2 or [0])), what
    for j in range(t.n_teams):                     # a team's problems are those its rows belong to
        lo = sum(rows[:t.prob_lo[j]])
        assert lo <= t.row_lo[0][j] or t.row_n[0][j] == 0, what
        assert t.row_lo[0][j] + t.row_n[0][j] <= sum(rows[:t.prob_lo[j] + t.prob_n[j]]) or t.row_n[0][j] == 0, what
        assert t.prob_n[j] * (2 if rows2 else 1) <= 64, what
    return t


@pytest.mark.parametrize("rows", [[1] * 8 + [17], [17] + [1] * 8, [1] * 4 + [32] + [1] * 4, [1] * 12 + [32], [1] * 31 + [25], [25] + [1] * 31,
                                  [1] * 15 + [32] + [1] * 16, [1] * 8 + [16, 16]])
def test_one_long_sequence_among_many_short_ones(lib, rows):
    """The cut by running row counts leaves two to seven teams there, one of them above a row tile: one XCD each."""
    for xcds in (8, 4):
        t = _check(lib, rows, xcds=xcds)
        assert t is not None and (t.max_rows <= 16 or t.stations == 1)


def test_every_accepted_deal_has_a_kernel(lib):
    rng = random.Random(1)
    accepted, tall, paired = 0, 0, 0
    for _ in range(20000):
        n = rng.choice((1, 2, 3, 4, 6, 8, 9, 12, 16, 32))
        idle, long_ = rng.choice((0, 0.2, 0.5)), rng.choice((0.05, 0.1, 0.5, 1))
        rows = [0 if rng.random() < idle else rng.randint(1, 32) if rng.random() < long_ else rng.randint(1, 3) for _ in range(n)]
        drafts = rng.random() < 0.2
        rows2 = [rng.randint(1, 40) if r else 0 for r in rows] if drafts else None
        t = _check(lib, rows, rows2, xcds=rng.choice((8, 8, 4)), layers=rng.choice((1, 2, 6, 12)), limit=rng.choice((32, 32, 16)))
        if t is not None:
            accepted += 1
            tall += t.max_rows > 16
            paired += t.stations > 1
    assert accepted > 8000 and tall > 500 and paired > 3000
