"""The dyadic runs of the fold: for every window k (0-based) of a sequence of N windows, the runs that
the fold combines cover exactly the windows before k (filter state) and after k (information), in order,
and every one of them is a node that the tree kernels store. Plain index arithmetic, mirrored from
the kernels; the GPU results at the same sizes are checked in test_gpu_fold.py.
"""
import pytest

TILE, LOG_TILE = 256, 8
SIZES = (1, 2, 3, 15, 16, 17, 100, 240, 241, 255, 256, 257, 271, 272, 273, 511, 512, 513, 768, 1000, 1024, 4096 + 31,
         3 * 4096 + 256)


def top_bit(x):
    return x.bit_length() - 1


def forward_runs(k):
    """(first window, length) of the runs before window k, in the order they are combined."""
    return [(((k >> p) ^ 1) << p, 1 << p) for p in range(top_bit(k) if k else -1, -1, -1) if (k >> p) & 1]


def backward_runs(k, N):
    """The runs after window k, from the last window towards k, as the fold combines them: N's own
    set bits below the top differing bit (low bits first), then k's clear bits below it (high bits first)."""
    b = top_bit(k ^ N)
    tail = [(((N >> p) ^ 1) << p, 1 << p) for p in range(b) if (N >> p) & 1]
    own = [(((k >> p) ^ 1) << p, 1 << p) for p in range(b - 1, -1, -1) if not (k >> p) & 1]
    return tail + own


def stored(run, N):
    """Whether the tree kernels store this run: within a tile any node is (windows past the end count as
    zero measurements, so only whole runs may be asked for); above the tiles the run's tiles are whole."""
    first, n = run
    if first < 0 or first + n > N or first % n:
        return False
    return n < TILE or (first + n) // TILE <= N >> LOG_TILE


@pytest.mark.parametrize("N", SIZES)
def test_runs_cover_the_sequence(N):
    step = 1 if N <= 1024 else 7
    for k in sorted(set(range(0, N, step)) | {N - 1}):
        at = 0
        for run in forward_runs(k):
            assert stored(run, N) and run[0] == at, (k, run)
            at += run[1]
        assert at == k
        at = N
        for run in backward_runs(k, N):
            assert stored(run, N) and run[0] + run[1] == at, (k, run)
            at = run[0]
        assert at == k + 1
    at = 0  # the state after the last window: the place N of the tree
    for run in forward_runs(N):
        assert run[0] == at
        at += run[1]
    assert at == N


@pytest.mark.parametrize("N", [n for n in SIZES if n > TILE])
def test_tile_bits_and_window_bits_split_the_runs(N):
    """A full tile takes the bits of N's tiles above it and all of a window's own bits; a window of the
    partial last tile takes no tile-level backward run."""
    nf, rem = N >> LOG_TILE, N & (TILE - 1)
    for k in range(0, N, 5):
        tile, w = k >> LOG_TILE, k & (TILE - 1)
        runs = backward_runs(k, N)
        if tile == nf:
            b = top_bit(w ^ rem)
            assert b < LOG_TILE and all(n < TILE for _, n in runs)
        else:
            hb = top_bit(tile ^ nf)
            assert top_bit(k ^ N) == LOG_TILE + hb
            small = [r for r in runs if r[1] < TILE and r[0] >= tile * TILE and r[0] < (tile + 1) * TILE]
            assert [r[1] for r in small] == [1 << p for p in range(LOG_TILE - 1, -1, -1) if not (w >> p) & 1]
