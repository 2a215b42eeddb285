"""How the tiles of bytes find the pieces (or sequences) that start in them, restated: merge_cut_tiles_kernel looks at 64
offsets where the average says, merge_byte_runs_kernel goes on from the tile before, both search 64 places at a time
otherwise, and a tile's last part ends at the first offset at or behind its end.  On data without any other start the parts of all
tiles are the pieces, none missing and none twice; with offsets that decrease they can overlap and cover more bytes than there
are, which is why the emit kernels look at the verdict first."""
import numpy as np
import pytest

WAVE = 64


def lower_bound(seq, a, b, x):
    """First k in [a, b) with seq[k] >= x, b if there is none (wave_lower_bound)."""
    while a < b:
        step = -(-(b - a) // WAVE)
        c = WAVE
        for lane in range(WAVE):
            at = a + (lane + 1) * step - 1
            if not (at < b and seq[at] < x):
                c = lane
                break
        after = a + c * step
        a, b = min(after, b), min(after + step - 1, b)
    return a


def leading(flags):
    return next((i for i, f in enumerate(flags) if not f), len(flags))


def window(seq, at):
    n_seqs = len(seq) - 1
    return [(at + lane <= n_seqs, seq[min(at + lane, n_seqs)]) for lane in range(WAVE)]


def parts_of_tile(seq, n, lo, hi, s0, s1, following):
    starts = sorted({v for v in seq[s0:s1] if lo <= v < hi} | ({0} if lo == 0 else set()))
    return [(a, b) for a, b in zip(starts, starts[1:] + [min(following, n)])]


def end_of_starts(seq, n, hi, at, after_window):
    """(index of the first offset >= hi, that offset), looked for among the 64 from `at` on first."""
    inside = leading([ok and v < hi for ok, v in window(seq, at)])
    n_seqs = len(seq) - 1
    s1 = at + inside if inside < WAVE else lower_bound(seq, min(after_window, n_seqs + 1), n_seqs + 1, hi)
    return s1, min(max(seq[s1], hi), n) if s1 <= n_seqs else n


def cut_tiles(seq, n, size, mis):
    n_seqs, parts = len(seq) - 1, []
    for tile in range(-(-(n + 15) // size)):
        lo, hi = min(max(tile * size - mis, 0), n), min((tile + 1) * size - mis, n)
        at = min(max(int(np.float32(lo) * (np.float32(n_seqs) / np.float32(n))) - WAVE // 2, 0), n_seqs)
        below = [ok and v < lo for ok, v in window(seq, at)]
        if (at > 0 and not below[0]) or all(below):
            at = lower_bound(seq, 0, n_seqs + 1, lo)
            below = [False] * WAVE
        s0 = at + leading(below)
        s1, following = end_of_starts(seq, n, hi, at, at + WAVE)
        parts += parts_of_tile(seq, n, lo, hi, s0, max(s0, s1), following)
    return parts


def byte_runs(seq, n, tiles_per_group, mis, size=4096):
    n_seqs, parts, s1 = len(seq) - 1, [], 0
    for tile in range(-(-(n + 15) // size)):
        lo, hi = min(max(tile * size - mis, 0), n), min((tile + 1) * size - mis, n)
        s0 = lower_bound(seq, 0, n_seqs + 1, lo) if tile % tiles_per_group == 0 else s1
        s1, following = end_of_starts(seq, n, hi, s0, s0 + WAVE)
        parts += parts_of_tile(seq, n, lo, hi, s0, s1, following)
    return parts


def random_offsets(rng, n, n_seqs, how):
    if how == "chunks":
        return [min(k * -(-n // n_seqs), n) for k in range(n_seqs)] + [n]
    if how == "crowded":       # most of them in one place, empty ones among them
        inner = np.concatenate([np.full(n_seqs // 2, n // 3), n // 3 + rng.integers(0, 50, n_seqs - 1 - n_seqs // 2)])
    else:
        inner = rng.integers(0, n + 1, n_seqs - 1)
    return [0] + [int(x) for x in np.sort(inner)] + [n]


@pytest.mark.parametrize("how", ["chunks", "random", "crowded"])
@pytest.mark.parametrize("n,n_seqs", [(1, 1), (4097, 1), (30_000, 7), (30_000, 900), (50_000, 65), (200_000, 3000)])
def test_the_parts_of_all_tiles_are_the_pieces(how, n, n_seqs):
    rng = np.random.default_rng(n + n_seqs)
    for trial in range(3):
        seq, mis = random_offsets(rng, n, n_seqs, how), int(rng.integers(0, 16))
        starts = sorted(set(v for v in seq if v < n))
        pieces = list(zip(starts, starts[1:] + [n]))
        for size in (1024, 2048, 3072):
            assert cut_tiles(seq, n, size, mis) == pieces
        for group in (1, 2, 8):
            assert byte_runs(seq, n, group, mis) == pieces


def test_offsets_that_decrease_can_cover_more_bytes_than_there_are():
    covered = lambda parts: sum(b - a for a, b in parts)
    assert covered(cut_tiles([0, 9200, 8200, 8250, 8300, 8400, 10_000], 10_000, 1024, 0)) == 11_000
    seq = list(range(0, 20_001, 100))
    for k in (1, 60, 110, 150):
        seq[k] = 20_000
    assert covered(cut_tiles(seq, 20_000, 1024, 0)) == 53_700
    seq = list(range(0, 1_400_001, 7000))
    for k in (1, 60, 110, 150):
        seq[k] = 1_400_000
    assert covered(byte_runs(seq, 1_400_000, 1, 0)) == 4_676_000
