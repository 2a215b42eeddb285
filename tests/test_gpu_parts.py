"""Pieces of more than 16 bytes that fall into short parts (listed_in_short_parts, merge_pieces_in_parts): parts around the longest
that is taken and around the 64 bytes that a wavefront takes together, at the start of a piece and near its end; pieces around those 64
bytes and over several of them, two of up to 64 bytes together and of more; as many per tile as one, one per wavefront, the most that
are taken and one more, beside pieces that do not fit; merged ids of any kind; given pieces and raw bytes.  Exact against the oracle."""
import numpy as np
import pytest

import oracle
from test_never_joined_rule import joined_pairs

pytestmark = pytest.mark.gpu
PART, LISTED, SHORT = 40, 8, 64          # kPartMax, kPartsPieces; the longest pieces that are listed for columns


def _table(rng, numbered):
    """Rules over the letters 1..6, every pair of them first, so that letters in a row are one part; 7 to 9 and the space
    join nothing, so each is a part of its own."""
    merges, ids = [(a, b) for a in range(1, 7) for b in range(1, 7)], [1, 2, 3, 4, 5, 6]
    new = None if numbered else rng.choice(np.arange(256, 1 << 24), 96, replace=False)
    for k in range(96):
        if k < 36:
            pair = merges[k]
        else:
            pair = merges[0]
            while pair in merges:
                pair = (int(rng.choice(ids)), int(rng.choice(ids)))
            merges.append(pair)
        ids.append(256 + k if numbered else int(new[k]))
    return np.array(merges, dtype=np.int32), None if numbered else np.array(new, dtype=np.int32)


def _piece(rng, n, longest, at_end):
    """A space, then n - 1 bytes with parts of up to `longest`, the first (or the last) exactly that long if there is room."""
    out = []
    while len(out) < n - 1:
        k = longest if not out else int(rng.integers(1, min(longest, PART) + 1))
        out += list(rng.integers(1, 7, k)) + [int(rng.integers(7, 10))] * int(rng.integers(1, 3))
    out = out[:n - 1]
    return bytes(int(x) for x in [32] + (out[::-1] if at_end else out))


def _longest_part(piece, joined):
    best = row = 1
    for x, y in zip(piece, piece[1:]):
        row = row + 1 if (x, y) in joined else 1
        best = max(best, row)
    return best


@pytest.mark.parametrize("numbered", [True, False])
@pytest.mark.parametrize("per_tile", [1, 4, 5, 8, 9])
def test_parts(numbered, per_tile):
    import torch
    import paper_2603_02597_amd as B
    rng = np.random.default_rng(per_tile + 100 * numbered)
    merges, ids = _table(rng, numbered)
    joined = joined_pairs(merges, ids)
    assert all((x, y) in joined for x in range(1, 7) for y in range(1, 7)) and all(max(pair) < 7 for pair in joined)
    table, want_table = B.Table(merges, None, ids), oracle.Table(merges, None, ids)
    sizes = [17, 18, 33, 63, 64, 65, 66, 127, 128, 129, 200, 257, 300, 640, 641]
    small = [17, 18, 31, 32, 33, 46, 47, 63, 64]           # two of them: up to 64 bytes, and beyond
    seen, unfit_tiles, late = set(), 0, 0
    for longest in (3, 16, 17, PART - 1, PART, PART + 1, 64, 65, 100):
        pieces = []
        for i in range(45):
            here = [_piece(rng, int(rng.choice(small)) if i % 2 else sizes[(i + j) % len(sizes)], longest, i % 4 > 1) for j in range(per_tile)]
            parts = [_longest_part(x, joined) for x in here]
            seen.update(parts)
            listed = [k for x, k in zip(here, parts) if len(x) <= SHORT]
            unfit_tiles += 0 < len(listed) <= LISTED and max(listed) > PART
            late += sum(len(x) >= 200 and k > PART and _longest_part(x[:len(x) - k], joined) <= PART for x, k in zip(here, parts))
            short = [b" " + rng.integers(1, 10, int(rng.integers(1, 4))).astype(np.uint8).tobytes() for _ in range(256 - per_tile)]
            both = here + short
            pieces += [both[k] for k in rng.permutation(256)]
        data = np.frombuffer(b"".join(pieces), dtype=np.uint8)
        off = np.concatenate([[0], np.cumsum([len(p) for p in pieces])]).astype(np.int32)
        want = oracle.encode(want_table, data, off)
        d, o = torch.from_numpy(data.copy()).cuda(), torch.from_numpy(off).cuda()
        for kw in ({"pieces_per_wave": 64}, {"fused": -1, "pieces_per_wave": 64}, {"fused": -1, "pieces_per_wave": 64, "long_groups": 1}, {}):
            got = B.encode(table, d, o, B.EncodeOptions(**kw) if kw else None)
            assert np.array_equal(got[1].cpu().numpy(), want[1]) and np.array_equal(got[0].cpu().numpy(), want[0]), (longest, kw)
        # raw bytes: a piece starts at every space; alone, and often enough for the runs of tiles of larger inputs
        for times in (1, 1 + 1_400_000 // data.size):
            raw = d.repeat(times)
            got_ids, at = torch.empty(raw.numel(), dtype=torch.int32, device="cuda"), torch.zeros(2, dtype=torch.int32, device="cuda")
            ws = torch.empty(B.bpe_encode_raw_workspace_bytes(raw.numel()), dtype=torch.uint8, device="cuda")
            B.bpe_encode_raw(table, raw, None, got_ids, at, ws)
            assert B.bpe_encode_status(ws) == 0 and at.tolist() == [0, times * want[0].size], (longest, times)
            assert torch.equal(got_ids[:times * want[0].size], torch.from_numpy(want[0]).cuda().repeat(times)), (longest, times)
    table.free()
    assert {PART - 1, PART, PART + 1, 64} <= seen and unfit_tiles and late
