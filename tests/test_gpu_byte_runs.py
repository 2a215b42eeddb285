"""Token-only raw calls beyond the smallest tiles of bytes (runs of tiles of 4 KiB): every id and sequence offset against
the CPU oracle.  Dense tiles (up to a piece per byte, several passes over a tile), tiles without a start, pieces across
tiles and runs, starts and sequence cuts at the edges of tiles and of 16-byte groups, unaligned input, left-over short
pieces from none to more than the list holds, longer pieces of every path."""
import numpy as np
import pytest

from test_gpu_pretokenize import _check_raw, gpu  # noqa: F401

pytestmark = pytest.mark.gpu

TILE, N_MIN = 4096, 322 * 4096          # from so many bytes on
u8 = lambda b: np.frombuffer(b, dtype=np.uint8)


def _fill(parts, n):
    """The parts, each from a tile's first byte on (text up to there), then text up to n bytes."""
    from workloads import configs as C
    text = C.make_eval("seq131k")["bytes"]
    out = []
    for part in parts:
        part = np.asarray(part, dtype=np.uint8)
        gap = -(len(part)) % TILE + 1500
        out += [part, text[:gap + (-(len(part) + gap)) % TILE]]
    used = sum(map(len, out))
    return np.concatenate(out + [np.resize(text, n - used)])


def _parts():
    from workloads import configs as C
    text = C.make_eval("seq131k")["bytes"]
    letters = text[text != 0x20]
    rng = np.random.default_rng(5)
    stress = C.make_eval("stress")["bytes"]
    edge = lambda at: np.concatenate([letters[:at], u8(b" "), letters[:6000 - at]])
    return {
        "dense": [u8(b" " * 9000), u8(b"a " * 5000), u8(b"ab " * 4000), u8(b"abc  " * 2000),
                  rng.choice(u8(b" \x00\xffe"), size=20000)],
        "pieces across tiles": [letters[:3 * TILE], edge(TILE - 1), edge(TILE), edge(TILE + 1), edge(15), edge(16),
                                u8(b" " + b"e" * 9000 + b" " + b"t" * (TILE - 1) + b" x")],
        "longer pieces": [stress[:300000], rng.integers(0x21, 256, 20000).astype(np.uint8),
                          np.concatenate([np.concatenate([u8(b" "), letters[k:k + n]]) for k, n in
                                          enumerate(rng.integers(1, 40, 1500))])],
    }


@pytest.mark.parametrize("which", ["dense", "pieces across tiles", "longer pieces"])
@pytest.mark.parametrize("table,misalign", [("t1k", 0), ("t50k", 1), ("t100k", 15)])
def test_byte_runs(gpu, oracle_mod, which, table, misalign):
    _, B = gpu
    from workloads import configs as C
    n = N_MIN + 70001 if which != "pieces across tiles" else 2600 * TILE + 77      # one tile per run, and several
    plan = B.kernels_by_interval(B.bpe_encode_raw_plan(n, 0, 1, False, False), B.N_RAW_TIMED_INTERVALS)
    assert plan == ["", "merge_byte_runs_kernel", "", "emit_byte_runs_kernel", ""]
    merges = C.load_merges(table)
    data = _fill(_parts()[which], n)
    rng = np.random.default_rng(misalign)
    near = (np.arange(1, 60, 7)[:, None] * TILE - misalign + np.array([-17, -16, -1, 0, 0, 0, 1, 15, 16])).ravel()
    cuts = np.sort(np.concatenate([near, rng.integers(0, n, 300), np.arange(200000, 203000), [n] * 70]))
    seq = np.concatenate([[0, 0], cuts, [n]]).astype(np.int32)
    _check_raw(gpu, oracle_mod, merges, data, None if misalign == 1 else seq, f"{which}, {table}", own_arrays=False,
               misalign=misalign)


def test_as_many_tiles_as_need_a_scan(gpu, oracle_mod):
    """More than 8,192 tiles: their totals are added up by a kernel of their own."""
    _, B = gpu
    from workloads import configs as C
    ev = C.make_eval("batch")
    n = 8193 * TILE + 5
    data = np.resize(ev["bytes"], n)
    assert B.kernels_by_interval(B.bpe_encode_raw_plan(n, 0, 1, False, False), 5)[2] == "scan_tiles_kernel"
    _check_raw(gpu, oracle_mod, C.load_merges(ev["table"]), data, np.linspace(0, n, 1001).astype(np.int32), "scan", own_arrays=False)


@pytest.mark.parametrize("case", ["entries too large", "too large in the first half", "a dip", "negative", "first", "last", "one sequence"])
def test_bad_sequence_offsets_are_reported_and_nothing_is_written_out_of_bounds(gpu, oracle_mod, case):
    """Each tile searches the offsets for its own part, so with offsets that decrease the pieces of different tiles can
    overlap: text without a space or a rule, 1.4 MB in 200 sequences of which four start at the end, would make 4.7 M tokens.
    out_ids is the head of a larger buffer here that would hold all of them."""
    torch, B = gpu
    n = 1_400_000
    data = np.random.default_rng(2).integers(0x80, 0x100, n).astype(np.uint8)
    good = np.arange(201, dtype=np.int32) * (n // 200)
    bad = good.copy()
    if case == "entries too large":
        bad[[1, 60, 110, 150]] = n
    elif case == "too large in the first half":
        bad[3:100:7] = n
    elif case == "a dip":
        bad[100:150] = bad[20]
    elif case == "negative":
        bad[[5, 77]] = -9
    elif case == "first":
        bad[0] = 5
    elif case == "last":
        bad[-1] = n - 1
    else:
        good, bad = np.array([0, n], dtype=np.int32), np.array([0, n - 3], dtype=np.int32)
    k = bad.size
    merges = np.array([[97, 97]], dtype=np.int32)
    table = B.Table(merges)
    d, seq = torch.from_numpy(data).cuda(), torch.from_numpy(bad).cuda()
    ids = torch.full((8 * n,), -7, dtype=torch.int32, device="cuda")
    seq_tok = torch.full((k + 64,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.bpe_encode_raw_workspace_bytes(n, 0, k - 1), dtype=torch.uint8, device="cuda")
    print(f"[case] byte runs, bad sequence offsets: {case}", flush=True)
    B.bpe_encode_raw(table, d, seq, ids[:n], seq_tok[:k], ws)
    assert B.bpe_encode_status(ws) == -11
    assert (ids == -7).all() and (seq_tok[:k] == 0).all() and (seq_tok[k:] == -7).all()
    # a recorded call that saw bad offsets once encodes the next replay's, with the verdict of the first still there
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        B.bpe_encode_raw(table, d, seq, ids[:n], seq_tok[:k], ws)
    for offsets in (bad, good, bad, good):
        seq.copy_(torch.from_numpy(offsets))
        ids.fill_(-7)
        seq_tok.fill_(-7)
        g.replay()
        torch.cuda.synchronize()
        if offsets is good:
            want = oracle_mod.encode(oracle_mod.Table(merges), data, good)
            assert np.array_equal(ids[:n].cpu().numpy(), want[0]) and (ids[n:] == -7).all()
            assert np.array_equal(seq_tok[:k].cpu().numpy(), want[1]) and (seq_tok[k:] == -7).all()
        else:
            assert (ids == -7).all() and (seq_tok[:k] == 0).all() and (seq_tok[k:] == -7).all()
    assert B.bpe_encode_status(ws) == -11 and B.bpe_encode_status(ws) == 0
    table.free()


def test_a_piece_of_more_tokens_than_its_word_holds(gpu, oracle_mod):
    """2^19 tokens and more: the count is in the word behind the piece's own."""
    _, B = gpu
    rng = np.random.default_rng(4)
    piece = lambda k: np.concatenate([u8(b" "), rng.integers(0x80, 0x100, k - 1).astype(np.uint8)])
    data = np.concatenate([_fill([], 300_000), piece(0x7FFFF), piece(0x7FFFE), u8(b" a b "), piece(0x80000), _fill([], 20_000), piece(600_000)])
    _check_raw(gpu, oracle_mod, np.array([[97, 97], [32, 97]], dtype=np.int32), data, None, "many tokens", own_arrays=False, misalign=2)
