"""The whole-piece table and the merging of what it leaves over, at the sizes where they change course: every piece
length around the 12 bytes a table slot holds and the 16 bytes of a row, strings that differ only in trailing zero
bytes, and tiles with every number of left-over pieces around the limits between the row and the lane form.
Exact against the oracle."""
import numpy as np
import pytest

import oracle
from workloads import configs as C

pytestmark = pytest.mark.gpu


def _check(merges, pieces, options=()):
    import torch
    import paper_2603_02597_amd as B
    data = np.frombuffer(b"".join(pieces), dtype=np.uint8)
    off = np.concatenate([[0], np.cumsum([len(p) for p in pieces])]).astype(np.int32)
    want_ids, want_off = oracle.encode(oracle.Table(merges), data, off)
    table = B.Table(merges)
    d, o = torch.from_numpy(data.copy()).cuda(), torch.from_numpy(off).cuda()
    for kw in options or ({},):
        ids, got_off = B.encode(table, d, o, B.EncodeOptions(**kw))
        assert np.array_equal(got_off.cpu().numpy(), want_off), kw
        assert np.array_equal(ids.cpu().numpy(), want_ids), kw


FORMS = ({"fused": 1}, {"fused": -1}, {"fused": -1, "long_groups": 1}, {"fused": -1, "tiny_max_len": 7})


def test_zero_bytes_count():
    """Rules over the bytes 0 and 1: strings of 1..20 bytes that zero-padding alone would not tell apart."""
    merges = [[0, 0], [256, 0], [1, 0], [256, 256], [258, 256], [259, 259], [261, 0], [1, 1], [263, 0], [261, 262]]
    pieces = [bytes([f] * k + [0] * (n - k)) for f in (0, 1) for n in range(1, 21) for k in range(0, min(n, 4))]
    _check(np.array(merges, dtype=np.int32), pieces * 7, FORMS)


def test_two_rules_that_spell_the_same_bytes():
    """(ab)c and a(bc) both spell abc; the loop arrives at one of them."""
    a, b, c = 97, 98, 99
    for first in ([[a, b], [b, c]], [[b, c], [a, b]]):
        ab, bc = (256, 257) if first[0] == [a, b] else (257, 256)
        for last in ([[ab, c], [a, bc]], [[a, bc], [ab, c]]):
            merges = np.array(first + last, dtype=np.int32)
            _check(merges, [b"abc", b"ab", b"bc", b"a", b"abcabc", b"cab", b"abcc", b"aabc"] * 40, FORMS)


def _word_pieces():
    merges = C.load_merges("t50k")
    ev = C.make_eval("seq32k")
    data, off = ev["bytes"], ev["piece_offsets"]
    _, tok_off = oracle.encode(oracle.Table(merges), data, off)
    count = np.diff(tok_off)
    cut = lambda i: data[off[i]:off[i + 1]].tobytes()
    whole = [cut(i) for i in np.nonzero(count == 1)[0][:4000]]
    left = [cut(i) for i in np.nonzero(count > 1)[0][:900]]
    return merges, whole, left


@pytest.mark.parametrize("n_tiles", [1, 5, 300, 1100])
def test_every_number_of_left_over_pieces(n_tiles):
    """Tiles of 256 pieces of which 0, 1 ... 256 are left over, at scattered places (single kernel, several kernels,
    deep grids)."""
    merges, whole, left = _word_pieces()
    rng = np.random.default_rng(n_tiles)
    counts = [0, 1, 4, 5, 16, 17, 31, 32, 33, 64, 65, 127, 128, 129, 255, 256, 3, 8]
    pieces = []
    for t in range(n_tiles):
        n_left = counts[t % len(counts)] if n_tiles > 1 else 129
        kinds = rng.permutation(256) < n_left
        pieces += [left[rng.integers(len(left))] if k else whole[rng.integers(len(whole))] for k in kinds]
    _check(merges, pieces[:-3], ({}, {"fused": -1}))


@pytest.mark.parametrize("n", [1, 2, 11, 12, 13, 15, 16, 17])
def test_piece_lengths(n):
    """Pieces of exactly n bytes: letters, two letters only (many merges), any byte."""
    rng = np.random.default_rng(n)
    merges = C.load_merges("t1k")
    pieces = [bytes(rng.integers(97, 123, n, dtype=np.uint8)) for _ in range(300)]
    pieces += [bytes(rng.choice(np.frombuffer(b"eat ", dtype=np.uint8), n)) for _ in range(300)]
    pieces += [bytes(rng.integers(0, 256, n, dtype=np.uint8)) for _ in range(100)]
    _check(merges, pieces, FORMS)


@pytest.mark.parametrize("n_tiles", [256, 257, 1024])
def test_left_over_pieces_in_the_single_kernel_with_and_without_helpers(n_tiles):
    """The same counts of left-over pieces where the single kernel is asked for: 16 wavefronts a tile up to 256
    tiles, four beyond (few left over: rows; more than 64 or 16: columns), longer pieces in some tiles."""
    merges, whole, left = _word_pieces()
    rng = np.random.default_rng(n_tiles)
    counts = [0, 1, 16, 17, 64, 65, 128, 256, 5]
    pieces = []
    for t in range(n_tiles):
        kinds = rng.permutation(256) < counts[t % len(counts)]
        pieces += [left[rng.integers(len(left))] if k else whole[rng.integers(len(whole))] for k in kinds]
        if t % 4 == 1:
            pieces[-1] = pieces[-1] * 5
    _check(merges, pieces[:-3], ({"fused": 1},))


@pytest.mark.parametrize("name", ["t1k", "t50k"])
def test_table_info_equals_the_images(name):
    import paper_2603_02597_amd as B
    merges = C.load_merges(name)
    assert B.Table(merges).info == B.bpe_table_image_build(merges)[1]
