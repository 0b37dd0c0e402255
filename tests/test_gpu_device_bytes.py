"""Device memory of list launches, against a layout of two copies of X, the lists and the queue.

A pair (row, estimate) is allowed X by row and by estimate, its count word (8 bytes), a place in the
redo queue (8 bytes) and a share of the 64-row sums; with one Z column X by rank and the radius too.
From 64 estimates on, the groups that X by row is cut into take whole 64-byte lines of a row.
A row of a sample is allowed its lists (8 bytes an entry of the first, 12 of the second, 8 entries past
each), lengths, bounds and copies; without Z the first list holds every row."""

import sys

import pytest

from test_gpu_few_estimates import alone, burst, series_of

pytestmark = pytest.mark.gpu

SLOP = 65536          # tables, counters, the outputs, rounding


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def pair_bytes(dx, dz):
    return 8 * dx + 16.125 + (4 * dx + 4 if dz == 1 else 0)


def line_bytes(dx, E):
    """What whole lines add to a row of X by row."""
    if E < 64:
        return 0
    groups = (E + 63) // 64
    return 4 * dx * (groups * -(-(-(-E // groups)) // 16) * 16 - E)


def row_bytes(n, dx, dz):
    if dz == 0:
        return 8 * (n - 1 + 8) + 96 + 16 + 4 + 4
    m1 = 1024 * 2 ** min(3, max(0, dx + 1 - dz + 1))
    m2 = 8 if dz == 1 else 2 * m1
    return 8 * (min(n - 1, m1) + 8) + 12 * (min(n - 1, m2) + 8) + 16 + 4 * (1 + dz) + (16 if dz == 1 else 0)


# the forms: lists, walk, rank ranges (few estimates; a window; long), wavelet counts, exchanged sides
@pytest.mark.parametrize("n,dx,dz,w,S", [(3000, 1, 3, 0, 7), (3000, 1, 3, 0, 64), (3000, 2, 5, 0, 129),
                                         (3000, 1, 0, 0, 7), (3000, 1, 0, 4, 64), (3000, 1, 1, 0, 20),
                                         (3000, 1, 1, 3, 64), (3000, 2, 1, 3, 64), (21500, 1, 1, 0, 64),
                                         (3000, 1, 1, 0, 64), (3000, 1, 1, 0, 200), (1500, 1, 1, 0, 31),
                                         (3000, 2, 1, 0, 20), (3000, 3, 1, 0, 64)])
def test_bytes_of_one_request(n, dx, dz, w, S):
    got = alone(n, dx, dz, S, w)
    want = n * (row_bytes(n, dx, dz) + (S + 1) * pair_bytes(dx, dz) + line_bytes(dx, S + 1))
    say("bytes", n, dx, dz, w, S, got, want, got / want)
    assert got <= want + SLOP


# many jobs on one sample: what counts is a pair (the sample's lists and ranks are left out: 512 bytes a row)
@pytest.mark.parametrize("n,dz,jobs,S", [(2000, 0, 48, 64), (2000, 0, 24, 200), (2000, 1, 48, 64)])
def test_bytes_of_a_burst(n, dz, jobs, S):
    _, _, got = burst(series_of(60, n, 3), jobs, n, 1, dz, 4, S)
    want = n * (jobs * (S + 1) * pair_bytes(1, dz) + 3 * (512 if dz == 0 else row_bytes(n, 1, dz)))
    say("bytes of a burst", n, dz, jobs, S, got, want, got / want)
    assert got <= want + 3 * SLOP


def test_bytes_of_shared_two_column_jobs():
    """Jobs of 8 estimates and 2 X columns on one sample use its lists: none of 16 KB a row each."""
    n, jobs, S = 3000, 24, 7
    _, _, got = burst(series_of(60, n, 3), jobs, n, 2, 1, 4, S)
    # a job that arrives first may go alone, and then has lists of its own
    want = n * (jobs * (S + 1) * pair_bytes(2, 1) + 3 * (row_bytes(n, 2, 1) + 8 * (2048 + 16)))
    say("two-column jobs", n, jobs, S, got, want, got / want)
    assert got <= want + 3 * SLOP
