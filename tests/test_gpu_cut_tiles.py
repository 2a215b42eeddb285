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


def _run_with(B, table, data, off, guard):
    """ids (guard words behind the capacity included), offsets and verdict of a call whose offsets may be bad."""
    import torch
    d, o = torch.from_numpy(data).cuda(), torch.from_numpy(off).cuda()
    ids = torch.full((data.size + guard,), -7, dtype=torch.int32, device="cuda")
    got_off = torch.full((off.size + 64,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.bpe_workspace_bytes(data.size, off.size - 1), dtype=torch.uint8, device="cuda")
    B.bpe_encode(table, d, o, ids[:data.size], got_off[:off.size], ws)
    verdict = B.bpe_encode_status(ws)
    got_off = got_off.cpu().numpy()
    assert (got_off[off.size:] == -7).all()
    return ids.cpu().numpy(), got_off[:off.size], verdict


def _good_pieces(off, n):
    """Which pieces have offsets of their own that are in range, do not decrease, and start and end the input."""
    good = (off[:-1] >= 0) & (off[1:] >= off[:-1]) & (off[1:] <= n)
    good[0] &= off[0] == 0
    good[-1] &= off[-1] == n
    return good


# bytes and pieces: tiles of each size, with and without merge_wide_kernel, and as many as need a scan kernel
@pytest.mark.parametrize("n,n_pieces,kernels", [
    (40_000, 700, 2), (300_000, 4600, 2), (1_500_000, 25_000, 2), (2_500_000, 3000, 2), (8193 * 3072 + 5, 16_000, 3),
    (20_000, 9, 3), (600_000, 200, 3), (1_300_000, 255, 3)])
def test_bad_offsets_yield_no_tokens_for_their_pieces(oracle_mod, n, n_pieces, kernels):
    """Offsets out of range, a first one that is not 0, a last one that is not the end: every other piece has its tokens, every
    offset is written, and nothing behind the capacity."""
    import torch  # noqa: F401  (its HIP runtime before the library's)
    import paper_2603_02597_amd as B
    from workloads import configs as C
    ev = C.make_eval("batch")
    merges = C.load_merges(ev["table"])
    data = np.resize(ev["bytes"], n).copy()
    good_off = (np.arange(n_pieces + 1, dtype=np.int64) * n // n_pieces).astype(np.int32)
    plan = [l["kernel"] for l in B.bpe_encode_plan(n, n_pieces)["launches"]]
    assert "merge_cut_tiles_kernel" in plan and len(plan) == kernels
    table = B.Table(merges)
    all_ids, all_off = oracle_mod.encode(oracle_mod.Table(merges), data, good_off, n_threads=16)
    for name, changes in {"beyond the end": {n_pieces // 2: n + 7}, "negative": {n_pieces // 3: -1},
                          "several": {1: n + 1, n_pieces // 4: -2**31, n_pieces - 1: 2**31 - 1}, "first": {0: 3},
                          "last": {n_pieces: n - 3}, "none": {}}.items():
        off = good_off.copy()
        for k, v in changes.items():
            off[k] = v
        print(f"[case] bad offsets, {name}: n_bytes={n} n_pieces={n_pieces}", flush=True)
        ids, got_off, verdict = _run_with(B, table, data, off, 64)
        assert verdict == (-11 if changes else 0)
        good = _good_pieces(off, n)            # (these have both offsets as they were)
        count = np.where(good, np.diff(all_off), 0)
        want_ids = all_ids[np.repeat(good, np.diff(all_off))]
        assert np.array_equal(got_off, np.concatenate([[0], np.cumsum(count)])), name
        assert np.array_equal(ids[:want_ids.size], want_ids) and (ids[n:] == -7).all(), name
    table.free()


@pytest.mark.parametrize("n,n_pieces", [(10_000, 6), (20_000, 200), (600_000, 200), (2_500_000, 3000)])
def test_offsets_that_decrease_write_nothing_behind_the_output(oracle_mod, n, n_pieces):
    """Pieces that overlap have more tokens than out_ids has room for: bytes that no rule knows, a token each.  out_ids is the
    head of a buffer here that would hold them all."""
    import torch  # noqa: F401  (its HIP runtime before the library's)
    import paper_2603_02597_amd as B
    data = np.random.default_rng(6).integers(0x80, 0x100, n).astype(np.uint8)
    table = B.Table([(97, 97), (97, 98), (98, 97)])
    good_off = (np.arange(n_pieces + 1, dtype=np.int64) * n // n_pieces).astype(np.int32)
    dip, late, back = good_off.copy(), good_off.copy(), good_off.copy()
    dip[n_pieces // 2: 3 * n_pieces // 4] = good_off[1]
    late[[1, n_pieces // 3, n_pieces // 2, -2]] = n
    back[1::2] = n - good_off[1::2]
    cases = {"a dip": dip, "some at the end": late, "back and forth": back}
    if n_pieces == 6:
        cases["overlap in one tile"] = np.array([0, 9200, 8200, 8250, 8300, 8400, n], dtype=np.int32)
    for name, off in cases.items():
        off = off.astype(np.int32)
        assert B.bpe_encode_plan(n, n_pieces)["launches"][-2]["kernel"] == "merge_cut_tiles_kernel"
        good = np.nonzero(_good_pieces(off, n))[0]
        total = int((off[good + 1].astype(np.int64) - off[good]).sum())
        print(f"[case] offsets that decrease, {name}: n_bytes={n} n_pieces={n_pieces}, {total} tokens", flush=True)
        assert total < 2**31
        ids, got_off, verdict = _run_with(B, table, data, off, 2 * n + min(total, 40_000_000))
        assert verdict == -11 and (ids[n:] == -7).all()
        count = np.zeros(n_pieces, dtype=np.int64)
        count[good] = off[good + 1] - off[good]
        assert np.array_equal(got_off, np.concatenate([[0], np.cumsum(count)])), name
        want = np.concatenate([data[off[k]:off[k + 1]] for k in good])[:n] if total < 40_000_000 else None
        assert want is None or np.array_equal(ids[:want.size], want), name
    ids, got_off, verdict = _run_with(B, table, data, good_off, 64)
    assert verdict == 0 and np.array_equal(got_off, good_off) and np.array_equal(ids[:n], data) and (ids[n:] == -7).all()
    table.free()


def test_a_recorded_call_after_one_with_bad_offsets(oracle_mod):
    """The verdict of a replay stays until it is asked for; the next replay's offsets are judged for themselves."""
    import torch
    import paper_2603_02597_amd as B
    from workloads import configs as C
    ev = C.make_eval("seq131k")
    merges = C.load_merges(ev["table"])
    data = ev["bytes"][:50_000].copy()
    good = np.arange(0, 50_001, 500, dtype=np.int32)
    bad = good.copy()
    bad[40] = 50_009
    table, ot = B.Table(merges), oracle_mod.Table(merges)
    want_ids, want_off = oracle_mod.encode(ot, data, good)
    d, off = torch.from_numpy(data).cuda(), torch.from_numpy(good.copy()).cuda()
    ids = torch.full((data.size,), -7, dtype=torch.int32, device="cuda")
    got = torch.full((good.size,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.bpe_workspace_bytes(data.size, good.size - 1), dtype=torch.uint8, device="cuda")
    B.bpe_encode(table, d, off, ids, got, ws)
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        B.bpe_encode(table, d, off, ids, got, ws)
    for o in (bad, good, bad, bad, good):
        off.copy_(torch.from_numpy(o))
        ids.fill_(-7)
        got.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        if o is good:
            assert np.array_equal(got.cpu().numpy(), want_off) and np.array_equal(ids[:want_ids.size].cpu().numpy(), want_ids)
        else:
            left_out = want_off[41] - want_off[39]
            assert int(got[-1]) == want_ids.size - left_out and int(got[39]) == int(got[41])
    assert B.bpe_encode_status(ws) == -11 and B.bpe_encode_status(ws) == 0
    table.free()


@pytest.mark.parametrize("options", [{}, {"fused": -1}, {"fused": -1, "selection_level": 1}, {"fused": -1, "selection_level": 3, "lds_max_len": 700},
                                     {"fused": -1, "selection_level": 2, "lds_max_len": 300, "wave_lds_max_len": 100}])
def test_long_pieces_that_overlap_end_and_stay_in_bounds(options):
    """Pieces that do not fit LDS keep their symbols in the workspace, at their bytes' place: overlapping ones write over each
    other's.  Whatever they then make of it, they end, and write nothing behind the output."""
    import torch
    import paper_2603_02597_amd as B
    n = 60_000
    rng = np.random.default_rng(8)
    data = np.concatenate([np.full(25_000, 97), rng.choice(u8(b"abc"), 15_000), np.full(20_000, 98)]).astype(np.uint8)
    merges = [(97, 97), (256, 256), (257, 257), (98, 98), (259, 259), (97, 98), (98, 97), (98, 99), (99, 97), (256, 98), (261, 262)]
    table = B.Table(merges)
    off = np.array([0, 30_000, 9_000, 40_000, 12_001, 47_003, 26_000, 50_001, 39_000, n, 30_500, n], dtype=np.int32)
    d, o = torch.from_numpy(data).cuda(), torch.from_numpy(off).cuda()
    ids = torch.full((8 * n,), -7, dtype=torch.int32, device="cuda")
    got = torch.full((off.size + 64,), -7, dtype=torch.int32, device="cuda")
    ws = torch.full((B.bpe_workspace_bytes(n, off.size - 1),), 0x7F, dtype=torch.uint8, device="cuda")
    print(f"[case] long pieces that overlap, {options}", flush=True)
    B.bpe_encode(table, d, o, ids[:n], got[:off.size], ws, B.EncodeOptions(**options) if options else None)
    assert B.bpe_encode_status(ws) == -11
    assert (ids[n:] == -7).all() and (got[off.size:] == -7).all()
    tokens = got[:off.size].cpu().numpy()
    assert tokens[0] == 0 and (np.diff(tokens) >= 0).all()
    table.free()
