"""Left-over pieces merged one per row of 16 lanes: every length from 2 to 16 bytes beside rows that have none or are done
sooner, byte 0 among the symbols, merged ids in rank order and any others up to the largest.  Exact against the oracle."""
import numpy as np
import pytest

import oracle
from test_oracle_encode import _random_p1_table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("numbered", [True, False])
@pytest.mark.parametrize("form", [{}, {"fused": -1}])
def test_rows(numbered, form):
    import torch
    import paper_2603_02597_amd as B
    rng = np.random.default_rng(11 + numbered)
    for trial in range(12):
        _, merges = _random_p1_table(rng, int(rng.integers(2, 5)), int(rng.integers(3, 60)))
        merges = np.array(merges, dtype=np.int32).reshape(-1, 2)
        to_zero = int(merges[merges < 256].min())                  # one of the letters becomes byte 0
        merges[merges == to_zero] = 0
        letters = np.unique(merges[merges < 256])
        ids = None
        if not numbered:
            ids = rng.choice(np.arange(256, 1 << 24), len(merges), replace=False).astype(np.int32)
            ids[-1] = (1 << 24) - 1
            merges = np.where(merges < 256, merges, ids[np.maximum(merges, 256) - 256]).astype(np.int32)
        pieces = []
        for n in range(2, 17):                                     # a handful per tile of 256, so that rows take them
            pieces += [rng.choice(letters, n).astype(np.uint8).tobytes() for _ in range(trial % 7 + 1)] + [b"x"] * 120
        data = np.frombuffer(b"".join(pieces), dtype=np.uint8)
        off = np.concatenate([[0], np.cumsum([len(p) for p in pieces])]).astype(np.int32)
        want = oracle.encode(oracle.Table(merges, None, ids), data, off)
        got = B.encode(B.Table(merges, None, ids), torch.from_numpy(data.copy()).cuda(), torch.from_numpy(off).cuda(), B.EncodeOptions(**form))
        assert np.array_equal(got[1].cpu().numpy(), want[1]) and np.array_equal(got[0].cpu().numpy(), want[0]), trial


@pytest.mark.parametrize("form", [{}, {"fused": -1}])
def test_as_many_left_over_pieces_as_rows_hold(form):
    """4 wavefronts have 16 rows, 16 have 64, and rows are taken for a quarter more: tiles of 256 with left-over pieces around
    one round of either, that limit, and two rounds."""
    import torch
    import paper_2603_02597_amd as B
    from workloads import configs as C
    rng = np.random.default_rng(8)
    merges = C.load_merges("t1k")
    letters = np.frombuffer(b"etaoinshr", dtype=np.uint8)
    pieces = []
    for n_left in (0, 1, 15, 16, 17, 19, 20, 21, 32, 33, 63, 64, 65, 79, 80, 81, 128, 129, 255, 256):
        tile = [b" " + rng.choice(letters, int(rng.integers(12, 16))).tobytes() for _ in range(n_left)] + [b"e"] * (256 - n_left)
        pieces += [tile[k] for k in rng.permutation(256)]
    data = np.frombuffer(b"".join(pieces), dtype=np.uint8)
    off = np.concatenate([[0], np.cumsum([len(p) for p in pieces])]).astype(np.int32)
    want = oracle.encode(oracle.Table(merges), data, off)
    d, o = torch.from_numpy(data.copy()).cuda(), torch.from_numpy(off).cuda()
    got = B.encode(B.Table(merges), d, o, B.EncodeOptions(pieces_per_wave=64, **form))
    assert np.array_equal(got[1].cpu().numpy(), want[1]) and np.array_equal(got[0].cpu().numpy(), want[0])
