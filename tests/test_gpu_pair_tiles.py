"""merge_kernel's workgroups of two tiles (512 short pieces), every id and offset against the CPU oracle: an
odd and an even number of tiles, a last tile of one piece, and tiles whose pieces are all words, leave a few
pieces over (rows of 16 lanes), more than a wavefront of them (columns) or nearly all (two rounds of columns)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_pieces", [1, 255, 256, 257, 511, 512, 513, 769, 5000])
@pytest.mark.parametrize("unknown", [0.0, 0.05, 0.25, 1.0])
def test_pairs_of_tiles(oracle_mod, n_pieces, unknown):
    import torch
    import paper_2603_02597_amd as B
    from workloads import configs as C
    merges = C.load_merges("t1k")
    ot, table = oracle_mod.Table(merges), B.Table(merges)
    rng = np.random.default_rng(n_pieces + int(1000 * unknown))
    known = [oracle_mod.decode(ot, np.array([i], dtype=np.int32)).tobytes() for i in range(256, 256 + len(merges))]
    known = [k for k in known if len(k) <= 12]
    pieces = []
    for _ in range(n_pieces):
        if rng.random() < unknown:
            pieces.append(rng.integers(97, 123, int(rng.integers(0, 17))).astype(np.uint8).tobytes())
        else:
            pieces.append(known[int(rng.integers(len(known)))])
        if rng.random() < 0.01:
            pieces[-1] = pieces[-1] * 12           # a longer piece: a long-piece workgroup's
    pieces[0] = pieces[0] or b"a"
    off = np.concatenate([[0], np.cumsum([len(x) for x in pieces])]).astype(np.int32)
    data = np.frombuffer(b"".join(pieces), dtype=np.uint8)
    print(f"[case] {n_pieces} pieces, {unknown:.0%} random", flush=True)
    want_ids, want_off = oracle_mod.encode(ot, data, off)
    for mis in (0, 3):
        buf = torch.empty(data.size + 8, dtype=torch.uint8, device="cuda")
        d = buf[mis:mis + data.size]
        d.copy_(torch.from_numpy(data.copy()))
        ids, got_off = B.encode(table, d, torch.from_numpy(off).cuda(), B.EncodeOptions(long_groups=4, fused=-1))
        assert np.array_equal(got_off.cpu().numpy(), want_off)
        assert np.array_equal(ids.cpu().numpy(), want_ids)
    table.free()


@pytest.mark.parametrize("n_left", [15, 16, 17, 255, 256, 257, 512])
def test_left_over_pieces_of_a_pair(oracle_mod, n_left):
    """Pairs of tiles that leave exactly so many pieces over, around what one round of rows (16) and one round of
    columns (256) take, in each half and across both; left-over pieces of 13 to 16 bytes among them."""
    import torch
    import paper_2603_02597_amd as B
    from workloads import configs as C
    merges = C.load_merges("t1k")
    ot, table = oracle_mod.Table(merges), B.Table(merges)
    rng = np.random.default_rng(n_left)
    known = [oracle_mod.decode(ot, np.array([i], dtype=np.int32)).tobytes() for i in range(256, 256 + len(merges))]
    tokens_of = lambda x: oracle_mod.encode(ot, np.frombuffer(x, np.uint8), np.array([0, len(x)], np.int32))[0].size
    known = [k for k in known if len(k) <= 12 and tokens_of(k) == 1]
    left = [bytes(rng.integers(0, 256, int(n)).astype(np.uint8)) for n in rng.integers(5, 17, 200)]
    left += [(known[int(a)] + known[int(b)] + known[int(c)])[:16] for a, b, c in rng.integers(0, len(known), (200, 3))]
    left = [x for x in left if tokens_of(x) > 1]
    pieces = []
    for first in (0, 512 - n_left, -1):            # left-over pieces in front, at the end, scattered
        where = rng.permutation(512)[:n_left] if first < 0 else np.arange(first, first + n_left)
        is_left = np.zeros(512, bool)
        is_left[where] = True
        pieces += [left[rng.integers(len(left))] if k else known[rng.integers(len(known))] for k in is_left]
    off = np.concatenate([[0], np.cumsum([len(x) for x in pieces])]).astype(np.int32)
    data = np.frombuffer(b"".join(pieces), dtype=np.uint8)
    want_ids, want_off = oracle_mod.encode(ot, data, off)
    ids, got_off = B.encode(table, torch.from_numpy(data.copy()).cuda(), torch.from_numpy(off).cuda(),
                            B.EncodeOptions(long_groups=4, fused=-1))
    assert np.array_equal(got_off.cpu().numpy(), want_off)
    assert np.array_equal(ids.cpu().numpy(), want_ids)
    table.free()
