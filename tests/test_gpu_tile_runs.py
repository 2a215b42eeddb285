"""merge_kernel's workgroups of several tiles, every id and offset against the CPU oracle: as many tiles as one, several
and more batches of probes take, a last tile of one piece, and runs of tiles that leave no piece over, a few (rows of
16 lanes), as many as the list holds (it is worked off in between) or all of them."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1025, 3 * 1024 + 1, 5 * 1024 + 1, 17 * 1024 + 3])
@pytest.mark.parametrize("unknown", [0.0, 0.004, 0.3, 1.0])
def test_runs_of_tiles(oracle_mod, tiles, unknown):
    import torch
    import paper_2603_02597_amd as B
    from workloads import configs as C
    merges = C.load_merges("t1k")
    ot, table = oracle_mod.Table(merges), B.Table(merges)
    n_pieces = tiles * 256 - 255
    plan = B.bpe_encode_plan(3 * n_pieces, n_pieces)
    assert plan["launches"][0]["kernel"] == "merge_kernel" and plan["n_tiles"] == tiles
    rng = np.random.default_rng(tiles + int(1000 * unknown))
    decoded = [oracle_mod.decode(ot, np.array([i], dtype=np.int32)).tobytes() for i in range(256, 256 + len(merges))]
    known = [x for x in decoded if len(x) <= 4]
    strange = [rng.integers(97, 123, int(n)).astype(np.uint8).tobytes() for n in rng.choice([2, 3, 3, 4, 5, 16], 400)]
    # a repeating stretch of pieces, not a multiple of a tile; the share of strange ones differs along it
    k = 5000
    share = unknown if unknown in (0.0, 1.0) else np.repeat(rng.random(25) * 2 * unknown, k // 25)
    is_strange = rng.random(k) < share
    stretch = [strange[rng.integers(len(strange))] if x else known[rng.integers(len(known))] for x in is_strange]
    stretch[17] = b"the quick brown fox jumps"                 # a longer piece: a long-piece workgroup's
    stretch[18] = b""
    lens = np.array([len(x) for x in stretch])
    n_rep = -(-n_pieces // k)
    off = np.concatenate([[0], np.cumsum(np.tile(lens, n_rep)[:n_pieces])]).astype(np.int32)
    data = np.resize(np.frombuffer(b"".join(stretch), dtype=np.uint8), int(off[-1]))
    print(f"[case] {tiles} tiles, {unknown:.1%} strange, {data.size} bytes", flush=True)
    want_ids, want_off = oracle_mod.encode(ot, data, off, n_threads=16)
    mis = tiles % 4
    buf = torch.empty(data.size + 8, dtype=torch.uint8, device="cuda")
    d = buf[mis:mis + data.size]
    d.copy_(torch.from_numpy(data.copy()))
    ids, got_off = B.encode(table, d, torch.from_numpy(off).cuda())
    assert np.array_equal(got_off.cpu().numpy(), want_off)
    assert np.array_equal(ids.cpu().numpy(), want_ids)
    table.free()
