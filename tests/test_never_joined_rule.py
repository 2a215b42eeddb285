"""Where no token reaches from one byte to the next: between bytes x, y such that no rule joins a string that ends with x to
one that starts with y (kNeverJoined).  The rule restated and checked against the CPU oracle: a piece's tokens are its
parts' tokens one after the other."""
import numpy as np
import pytest

import oracle


def joined_pairs(merges, ids=None):
    first, last, pairs = {b: b for b in range(256)}, {b: b for b in range(256)}, set()
    for k, (a, b) in enumerate(merges):
        a, b, m = int(a), int(b), 256 + k if ids is None else int(ids[k])
        pairs.add((last[a], first[b]))
        first[m], last[m] = first[a], last[b]
    return pairs


@pytest.mark.parametrize("seed", range(4))
def test_parts_merge_as_if_they_stood_alone(seed):
    rng, n_parts = np.random.default_rng(seed), []
    for _ in range(60):
        letters = [int(x) for x in rng.choice(256, size=int(rng.integers(2, 12)), replace=False)]
        ids, merges = list(letters), []
        for _ in range(int(rng.integers(1, 40))):
            pair = (int(rng.choice(ids)), int(rng.choice(ids)))
            if pair not in merges:
                merges.append(pair)
                ids.append(255 + len(merges))
        data = rng.choice(letters, size=int(rng.integers(2, 400))).astype(np.uint8)
        joined = joined_pairs(merges)
        cut = [i + 1 for i in range(data.size - 1) if (int(data[i]), int(data[i + 1])) not in joined]
        table = oracle.Table(np.array(merges, dtype=np.int32))
        whole, _ = oracle.encode(table, data, np.array([0, data.size], dtype=np.int32))
        parts, _ = oracle.encode(table, data, np.array([0, *cut, data.size], dtype=np.int32))
        assert np.array_equal(whole, parts)
        n_parts.append(len(cut) + 1)
    assert min(n_parts) < 5 < max(n_parts)
