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
