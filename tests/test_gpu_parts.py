"""Pieces of more than 16 bytes that fall into short parts (merge_pieces_in_parts): parts around the longest that is taken,
pieces around the 64 symbols of a wavefront and over several rounds of them, as many per tile as one, the most that are
taken and one more, beside pieces that do not fit; merged ids of any kind.  Exact against the oracle."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu
PART = 40


def _table(rng, numbered):
    """Rules over the letters 1..6; 7 to 9 join nothing, so they end parts."""
    merges, ids = [], [1, 2, 3, 4, 5, 6]
    new = None if numbered else rng.choice(np.arange(256, 1 << 24), 60, replace=False)
    for k in range(60):
        pair = (int(rng.choice(ids[:6 + k])), int(rng.choice(ids[:6 + k])))
        while pair in merges:
            pair = (int(rng.choice(ids[:6 + k])), int(rng.choice(ids[:6 + k])))
        merges.append(pair)
        ids.append(256 + k if numbered else int(new[k]))
    return np.array(merges, dtype=np.int32), None if numbered else np.array(new, dtype=np.int32)


def _piece(rng, n, longest):
    """n bytes with parts of up to `longest`, one of them exactly that long if there is room."""
    out = []
    while len(out) < n:
        k = longest if not out else int(rng.integers(1, longest + 1))
        out += list(rng.integers(1, 7, k)) + [int(rng.integers(7, 10))] * int(rng.integers(1, 3))
    return bytes(int(x) for x in out[:n])


@pytest.mark.parametrize("numbered", [True, False])
@pytest.mark.parametrize("per_tile", [1, 8, 9])
def test_parts(numbered, per_tile):
    import torch
    import paper_2603_02597_amd as B
    rng = np.random.default_rng(per_tile + 100 * numbered)
    merges, ids = _table(rng, numbered)
    table, want_table = B.Table(merges, None, ids), oracle.Table(merges, None, ids)
    sizes = [17, 18, 33, 63, 64, 65, 66, 127, 128, 129, 300, 640, 641]
    for longest in (3, PART - 1, PART, PART + 1, 64):
        pieces = []
        for i in range(40):
            here = [_piece(rng, sizes[(i + j) % (5 if i % 2 else len(sizes))], longest) for j in range(per_tile)]
            short = [rng.integers(1, 10, int(rng.integers(1, 4))).astype(np.uint8).tobytes() for _ in range(256 - per_tile)]
            both = here + short
            pieces += [both[k] for k in rng.permutation(256)]
        data = np.frombuffer(b"".join(pieces), dtype=np.uint8)
        off = np.concatenate([[0], np.cumsum([len(p) for p in pieces])]).astype(np.int32)
        want = oracle.encode(want_table, data, off)
        d, o = torch.from_numpy(data.copy()).cuda(), torch.from_numpy(off).cuda()
        for kw in ({"pieces_per_wave": 64}, {"fused": -1, "pieces_per_wave": 64}, {"fused": -1, "pieces_per_wave": 64, "long_groups": 1}, {}):
            got = B.encode(table, d, o, B.EncodeOptions(**kw) if kw else None)
            assert np.array_equal(got[1].cpu().numpy(), want[1]) and np.array_equal(got[0].cpu().numpy(), want[0]), (longest, kw)
    table.free()
