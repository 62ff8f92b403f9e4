"""Host-side check of the default window shapes (no GPU): the rule by which
the library picks a shape, restated, and the index arithmetic of every
window it yields around the lines of the rule."""

import itertools

import pytest

from test_window_geometry import DIR, NEQ, PER, SPEC, ZG, SMALL_NODES, _axis, _check


def _rounds(nx, ny, wc, wr, h, bx, by):
    ax, ay = _axis(nx, wc, h, bx[0] == NEQ), _axis(ny, wr, h, by[0] == NEQ)
    if ax is None or ay is None:
        return None
    nodes, n = ax["w"] * ay["w"], ax["nwin"] * ay["nwin"]
    threads = (nodes + 63) // 64 * 64
    slots = 256 * (3 if threads <= 256 else 2 if threads <= 384 else 1)
    return n, (n + slots - 1) // slots


def default_window(nx, ny, bx, by):
    if ny <= 16:
        wc = 64 if ny <= 8 else 32
        r12, r = _rounds(nx, ny, wc, ny, 12, bx, by), _rounds(nx, ny, wc, ny, wc // 8, bx, by)
        return wc, ny, 12 if r12 and r12[1] <= r[1] else wc // 8
    for c in [(16, 16, 4), (32, 16, 4), (32, 16, 3)]:
        r = _rounds(nx, ny, *c, bx, by)
        if r and r[0] <= 256:
            return c
    return 16, 16, 3


BCS = [(PER, PER), (ZG, ZG), (SPEC, DIR), (NEQ, NEQ)]


@pytest.mark.parametrize("ny", [1, 2, 4, 5, 8, 9, 16])
def test_narrow(ny):
    n_min = SMALL_NODES // ny + 1
    for nx in sorted({n_min, n_min + 1, 2 * n_min + 5, 2000}):
        for bx in BCS:
            by = (PER, PER) if bx[0] == NEQ or ny < 3 else (SPEC, SPEC)
            _check(nx, ny, *default_window(nx, ny, bx, by), bx, by)


@pytest.mark.parametrize("nx,ny", [(31, 17), (3, 600), (17, 33), (256, 64), (129, 129), (130, 96), (200, 101), (400, 77)])
def test_two_dimensional(nx, ny):
    for bx, by in itertools.product(BCS, BCS):
        if bx[0] == NEQ and by[0] == NEQ:
            continue
        _check(nx, ny, *default_window(nx, ny, bx, by), bx, by)
