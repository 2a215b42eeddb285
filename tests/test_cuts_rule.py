"""Where a piece can be cut without changing its tokens: between bytes x, y such that no rule joins a string that ends
with x to one that starts with y.  The rule, kept per byte as bpe_cut_tiles.h keeps it, restated here and checked
against the CPU oracle: a piece's tokens are its parts' tokens one after the other."""
import numpy as np
import pytest

import oracle


def cut_sets(merges):
    """(before, behind, twin): bytes never behind another byte / never before another one in a token / joined to themselves."""
    first, last = list(range(256)), list(range(256))
    before, behind, twin = np.ones(256, bool), np.ones(256, bool), np.zeros(256, bool)
    for a, b in merges:
        x, y = last[a], first[b]
        if x == y:
            twin[x] = True
        else:
            behind[x] = before[y] = False
        first.append(first[a])
        last.append(last[b])
    return before, behind, twin


def cuts(merges, data):
    before, behind, twin = cut_sets(merges)
    x, y = data[:-1], data[1:]
    return np.nonzero((before[y] | behind[x]) & ~((x == y) & twin[y]))[0] + 1


def check(merges, data):
    """Tokens of the whole piece against those of its parts; returns the number of parts."""
    data = np.ascontiguousarray(data, dtype=np.uint8)
    table = oracle.Table(np.asarray(merges, dtype=np.int32).reshape(-1, 2))
    whole, _ = oracle.encode(table, data, np.array([0, data.size], dtype=np.int32))
    off = np.concatenate([[0], cuts(merges, data), [data.size]]).astype(np.int32)
    parts, _ = oracle.encode(table, data, off)
    assert np.array_equal(whole, parts)
    return off.size - 1


def test_hand_worked():
    u8 = lambda b: np.frombuffer(b, np.uint8)
    # " a" and "aa": a space is behind nothing, but "a a" is three parts only where a token may hold "aa"
    assert list(cuts([(32, 97), (97, 97)], u8(b"aa  a a"))) == [2, 3, 5]
    # "  ": spaces may follow each other, nothing else may precede one
    assert list(cuts([(32, 32), (32, 97)], u8(b"a  a b"))) == [1, 4, 5]
    # "ab", "abc" = ab + c: b and c side by side through the merged id
    assert list(cuts([(97, 98), (256, 99)], u8(b"abcab"))) == [3]
    assert list(cuts([], u8(b"abc"))) == [1, 2]


@pytest.mark.parametrize("seed", range(6))
def test_random_tables(seed):
    rng = np.random.default_rng(seed)
    n_parts = []
    for _ in range(60):
        letters = rng.choice(256, size=int(rng.integers(2, 7)), replace=False)
        ids, seen, merges = list(letters), set(), []
        for _ in range(int(rng.integers(0, 25))):
            pair = (int(ids[rng.integers(len(ids))]), int(ids[rng.integers(len(ids))]))
            if pair in seen or (len(merges) < 3 and rng.random() < 0.3):
                continue
            seen.add(pair)
            ids.append(256 + len(merges))
            merges.append(pair)
        for _ in range(5):
            data = rng.choice(letters, size=int(rng.integers(1, 120)))
            data[rng.random(data.size) < 0.2] = letters[0]
            n_parts.append(check(merges, data))
    assert max(n_parts) > 1 and min(n_parts) == 1


@pytest.mark.parametrize("name,workload", [("t1k", "tiny"), ("t50k", "seq32k"), ("t100k", "stress")])
def test_trained_tables(name, workload):
    """Tables trained on words that start with a space: no space stands behind another byte, so a text falls into its words."""
    from workloads import configs as C
    merges = [tuple(map(int, m)) for m in C.load_merges(name)]
    data = C.make_eval(workload)["bytes"]
    for at in (0, 1111):
        piece = data[at:at + 2000]
        assert set(np.nonzero(piece[1:] == 0x20)[0] + 1) <= set(cuts(merges, piece))
        assert check(merges, piece) >= (piece == 0x20).sum()
