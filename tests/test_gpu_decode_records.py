"""The decoder's token records at the edges of their inline form (tokens of up to 12 bytes live in
the record, longer ones in the pool) and of a tile's stage, byte for byte against the CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

TEXT = bytes(range(100, 124))                 # token 256 + k is its first k + 2 bytes
MERGES = [(TEXT[0] if k == 0 else 255 + k, TEXT[k + 1]) for k in range(len(TEXT) - 1)]


# sizes: one thread's tokens and their edges, one round and two rounds per tile; lengths: around the
# words of a record, around the inline limit, and a mean of 20 bytes (a tile of 1024 exceeds the stage)
@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1025, 4099, 512 * 1024 + 3])
@pytest.mark.parametrize("lo,hi", [(1, 5), (7, 9), (11, 13), (1, 24), (18, 22)])
def test_token_lengths(oracle_mod, n, lo, hi):
    import torch
    import paper_2603_02597_amd as B
    rng = np.random.default_rng(n * 100 + lo)
    length = rng.integers(lo, hi + 1, n)
    ids = np.where(length == 1, TEXT[0], 254 + length).astype(np.int32)
    table = oracle_mod.Table(MERGES)
    want, want_off = oracle_mod.decode(table, ids), oracle_mod.token_byte_offsets(table, ids)
    out_ids = (rng.permutation(256 + len(MERGES)) + 50).astype(np.int32)
    vocab = B.Vocab(MERGES, output_ids=out_ids)
    print(f"[case] {n} tokens of {lo}..{hi} bytes", flush=True)
    for renumber in (False, True):
        src = torch.empty(n + 4, dtype=torch.int32, device="cuda")
        shift = n % 4                          # ids, offsets and bytes at every alignment a caller may have
        d_ids = src[shift:shift + n]
        d_ids.copy_(torch.from_numpy(out_ids[ids] if renumber else ids))
        for cap in (want.size, want.size // 2):
            buf = torch.full((want.size + 16,), 0xEE, dtype=torch.uint8, device="cuda")
            tbo = torch.full((n + 8,), -7, dtype=torch.int32, device="cuda")
            nb = torch.zeros(1, dtype=torch.int32, device="cuda")
            ws = torch.empty(B.bpe_decode_workspace_bytes(n), dtype=torch.uint8, device="cuda")
            B.bpe_decode(vocab, d_ids, buf[shift:shift + cap], ws, tbo[shift:shift + n + 1], nb, None, renumber)
            assert B.bpe_encode_status(ws) == (0 if cap == want.size else -2)
            assert int(nb.item()) == cap
            got, off = buf.cpu().numpy(), tbo.cpu().numpy()
            assert np.array_equal(got[shift:shift + cap], want[:cap])
            assert (got[:shift] == 0xEE).all() and (got[shift + cap:] == 0xEE).all()
            assert np.array_equal(off[shift:shift + n + 1], want_off)
            assert (off[:shift] == -7).all() and (off[shift + n + 1:] == -7).all()
    vocab.free()


LONG = MERGES + [(255 + len(MERGES) + k, 255 + len(MERGES) + k) for k in range(3)]     # 48, 96 and 192 bytes


# tiles of 1, 2 and 4 rounds whose rounds do not fit the stage, or only the first ones do: tokens of 9 to 12 bytes,
# which live in their record, between tokens of 192
@pytest.mark.parametrize("n", [5000, 530_001, 4_200_003])
@pytest.mark.parametrize("first_round", [0.0, 0.1, 1.0])
def test_inline_and_long_tokens_in_one_tile(oracle_mod, n, first_round):
    import torch
    import paper_2603_02597_amd as B
    rng = np.random.default_rng(n + int(10 * first_round))
    length = rng.integers(9, 13, n)
    ids = (254 + length).astype(np.int32)
    place = np.arange(n) % 4096                # round 0 of a tile of any kind starts at a multiple of 4096
    share = np.where(place < 1024, first_round, 0.1)
    ids[rng.random(n) < share] = 255 + len(LONG)
    table = oracle_mod.Table(LONG)
    want, want_off = oracle_mod.decode(table, ids), oracle_mod.token_byte_offsets(table, ids)
    vocab = B.Vocab(LONG)
    d_ids = torch.from_numpy(ids).cuda()
    ws = torch.empty(B.bpe_decode_workspace_bytes(n), dtype=torch.uint8, device="cuda")
    for cap in (want.size, want.size - 1, want.size // 3, 700):
        print(f"[case] {n} tokens, {first_round} of the first round long, {cap} of {want.size} bytes", flush=True)
        buf = torch.full((want.size + 16,), 0xEE, dtype=torch.uint8, device="cuda")
        tbo = torch.empty(n + 1, dtype=torch.int32, device="cuda")
        nb = torch.zeros(1, dtype=torch.int32, device="cuda")
        B.bpe_decode(vocab, d_ids, buf[3:3 + cap], ws, tbo, nb)
        assert B.bpe_encode_status(ws) == (0 if cap == want.size else -2) and int(nb.item()) == cap
        got = buf.cpu().numpy()
        assert np.array_equal(got[3:3 + cap], want[:cap]) and (got[:3] == 0xEE).all() and (got[3 + cap:] == 0xEE).all()
        assert np.array_equal(tbo.cpu().numpy(), want_off)
    vocab.free()


# both sides of every line between (rounds, tiles looked at) of vocabularies of more than 2,048 ids; the 100k table's mean token does
# not fit the stage of four rounds
@pytest.mark.parametrize("table_name", ["t50k", "t100k"])
@pytest.mark.parametrize("tiles", [512, 2304, 3072, 4096])
def test_both_sides_of_the_lines_between_tiles(oracle_mod, table_name, tiles):
    import torch
    import paper_2603_02597_amd as B
    from workloads import configs as C
    merges = C.load_merges(table_name)
    rng = np.random.default_rng(tiles)
    n_ids = 256 + len(merges)
    ids = np.where(rng.random(tiles * 1024 + 1) < 0.7, rng.integers(97, 1500, tiles * 1024 + 1), rng.integers(0, n_ids, tiles * 1024 + 1)).astype(np.int32)
    table, vocab = oracle_mod.Table(merges), B.Vocab(merges)
    want, want_off = oracle_mod.decode(table, ids), oracle_mod.token_byte_offsets(table, ids)
    d_ids = torch.from_numpy(ids).cuda()
    for n in (tiles * 1024, tiles * 1024 + 1):
        print(f"[case] {table_name}, {n} tokens", flush=True)
        size = int(want_off[n])
        buf = torch.full((size + 16,), 0xEE, dtype=torch.uint8, device="cuda")
        tbo = torch.empty(n + 1, dtype=torch.int32, device="cuda")
        nb = torch.zeros(1, dtype=torch.int32, device="cuda")
        ws = torch.empty(B.bpe_decode_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        for _ in range(2):
            B.bpe_decode(vocab, d_ids[:n], buf[:size], ws, tbo, nb)
        assert B.bpe_encode_status(ws) == 0 and int(nb.item()) == size
        got = buf.cpu().numpy()
        assert np.array_equal(got[:size], want[:size]) and (got[size:] == 0xEE).all()
        assert np.array_equal(tbo.cpu().numpy(), want_off[:n + 1])
    vocab.free()
