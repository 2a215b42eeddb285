"""bpe_encode on pieces that are longer on average than a lane takes (they are cut where no token can reach across, in
tiles of bytes of three sizes): every id and offset against the CPU oracle.  Pieces of one byte to many tiles, empty
ones, starts at the edges of tiles and of 16-byte groups, unaligned input, data that falls into words, into single bytes
(several passes over a tile), or cannot be cut at all (every path of longer pieces), and tables with rules for runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

u8 = lambda b: np.frombuffer(b, dtype=np.uint8)


def _check(oracle_mod, merges, data, off, misalign, label):
    import torch
    import paper_2603_02597_amd as B
    merges = np.asarray(merges, dtype=np.int32).reshape(-1, 2)
    data, off = np.ascontiguousarray(data, dtype=np.uint8), np.asarray(off, dtype=np.int32)
    plan = B.bpe_encode_plan(data.size, off.size - 1)
    print(f"[case] cut tiles {label} n_bytes={data.size} n_pieces={off.size - 1} misalign={misalign} "
          f"grid={plan['launches'][0]['grid']}", flush=True)
    assert plan["launches"][0]["kernel"] == "merge_cut_tiles_kernel"
    want_ids, want_off = oracle_mod.encode(oracle_mod.Table(merges), data, off, n_threads=16)
    buf = torch.empty(data.size + misalign, dtype=torch.uint8, device="cuda")
    d = buf[misalign:]
    d.copy_(torch.from_numpy(data.copy()))
    table = B.Table(merges)
    o = torch.from_numpy(off.copy()).cuda()
    ids = torch.full((data.size,), -7, dtype=torch.int32, device="cuda")
    got_off = torch.full((off.size + 8,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.bpe_workspace_bytes(data.size, off.size - 1), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        B.bpe_encode(table, d, o, ids, got_off[:off.size], ws)
    assert B.bpe_encode_status(ws) == 0
    got = got_off.cpu().numpy()
    assert np.array_equal(got[:off.size], want_off), f"offsets differ first at {np.nonzero(got[:off.size] != want_off)[0][:5]}"
    assert (got[off.size:] == -7).all()
    got = ids.cpu().numpy()
    assert np.array_equal(got[:want_ids.size], want_ids), f"ids differ first at {np.nonzero(got[:want_ids.size] != want_ids)[0][:5]}"
    assert (got[want_ids.size:] == -7).all()
    table.free()


def _ragged(rng, n, mean, tile):
    """Offsets of about n / mean pieces, some empty, some cuts around the edges of tiles."""
    edges = (np.arange(1, max(n // tile, 1), 9)[:, None] * tile + np.array([-16, -1, 0, 0, 1, 15])).ravel()
    k = max(n // mean - edges.size, 1)
    cut = np.concatenate([rng.integers(0, n + 1, k), edges[(edges > 0) & (edges < n)]])
    cut = np.concatenate([cut, rng.choice(cut, 3)])
    return np.concatenate([[0], np.sort(cut), [n]])


@pytest.mark.parametrize("n,tile", [(1, 1024), (17, 1024), (1025, 1024), (40_000, 1024), (1_048_561, 1024), (1_048_562, 2048),
                                    (2_300_001, 3072)])
@pytest.mark.parametrize("table,misalign", [("t1k", 0), ("t50k", 5), ("t100k", 15)])
def test_text(oracle_mod, n, tile, table, misalign):
    from workloads import configs as C, textgen
    merges = C.load_merges(table)
    data = np.resize(C.make_eval("seq131k" if n % 2 else "stress")["bytes"], n)
    if n < 17:
        return _check_short(oracle_mod, merges, data)
    rng = np.random.default_rng(n)
    for chunk in (19, 64, 1000, 2052) if n < 100_000 else (64, 2052):
        _check(oracle_mod, merges, data, textgen.fixed_chunks(n, chunk), misalign, f"{table} chunks of {chunk}")
    if n > 1000:
        _check(oracle_mod, merges, data, _ragged(rng, n, 120, tile), misalign, f"{table} ragged pieces")


def _check_short(oracle_mod, merges, data):
    import torch  # noqa: F401  (its HIP runtime before the library's)
    import paper_2603_02597_amd as B
    assert B.bpe_encode_plan(17, 1)["launches"][0]["kernel"] == "merge_cut_tiles_kernel"
    assert B.bpe_encode_plan(16, 1)["launches"][0]["kernel"] == "encode_kernel"
    _check(oracle_mod, merges, np.resize(data, 17), [0, 17], 1, "the shortest")


@pytest.mark.parametrize("what", ["no rule", "random bytes", "no space", "runs", "twin rules"])
def test_data_that_is_cut_everywhere_or_nowhere(oracle_mod, what):
    from workloads import configs as C, textgen
    rng = np.random.default_rng(3)
    text = C.make_eval("seq131k")["bytes"]
    merges = C.load_merges("t100k")
    if what == "no rule":
        merges, data = [], text[:30000]
    elif what == "random bytes":
        data = rng.integers(0, 256, 60000).astype(np.uint8)
    elif what == "no space":
        merges, data = C.load_merges("t50k"), text[text != 0x20][:60000]
    elif what == "runs":
        data = np.repeat(rng.integers(0, 256, 300), rng.integers(1, 900, 300)).astype(np.uint8)
    else:      # rules that join a byte to itself and to one other, and one byte that no rule knows
        merges = [(97, 97), (256, 256), (257, 97), (98, 98), (98, 97), (259, 260)]
        data = rng.choice(u8(b"aaaabbc"), 50000)
        data[20000:23000] = 97
    n = data.size
    for chunk in (20, 100, 300, 640, 2052):
        _check(oracle_mod, merges, data, textgen.fixed_chunks(n, chunk), 3, f"{what}, chunks of {chunk}")
    off = _ragged(rng, n, 200, 1024)
    _check(oracle_mod, merges, data, off, 0, f"{what}, ragged")
    _check(oracle_mod, merges, data, off[(off < 3000) | (off > 12000)], 1, f"{what}, one of several tiles")


def test_as_many_tiles_as_need_a_scan(oracle_mod):
    from workloads import configs as C, textgen
    ev = C.make_eval("batch")
    data = np.resize(ev["bytes"], 8193 * 3072 + 5)
    _check(oracle_mod, C.load_merges(ev["table"]), data, textgen.fixed_chunks(data.size, 2048), 0, "scan")
