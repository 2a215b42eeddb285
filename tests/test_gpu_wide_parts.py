"""bpe_encode on a few very long pieces: they are cut where no token can reach across, and what is still longer than four
wavefronts keep resident (2,052 symbols) is merged by 16.  Every id and offset against the CPU oracle: parts of 2,052 and
2,053 bytes, at the edges of the spans that a workgroup looks at, one inside a span and one that leaves it, over many
spans, runs, two of them in one tile, none at all, ragged and empty pieces, unaligned input."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(oracle_mod, merges, data, off, misalign, label, want=None):
    import torch
    import paper_2603_02597_amd as B
    data, off = np.ascontiguousarray(data, dtype=np.uint8), np.asarray(off, dtype=np.int32)
    kernels = [l["kernel"] for l in B.bpe_encode_plan(data.size, off.size - 1)["launches"]]
    print(f"[case] wide parts {label} n_bytes={data.size} n_pieces={off.size - 1} misalign={misalign}", flush=True)
    assert kernels == ["merge_wide_kernel", "merge_cut_tiles_kernel", "emit_cut_tiles_kernel"]
    want_ids, want_off = want or oracle_mod.encode(oracle_mod.Table(merges), data, off, n_threads=16)
    buf = torch.empty(data.size + misalign, dtype=torch.uint8, device="cuda")
    buf[misalign:].copy_(torch.from_numpy(data.copy()))
    table = B.Table(merges)
    ids = torch.full((data.size,), -7, dtype=torch.int32, device="cuda")
    got_off = torch.full((off.size,), -7, dtype=torch.int32, device="cuda")
    ws = torch.empty(B.bpe_workspace_bytes(data.size, off.size - 1), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        B.bpe_encode(table, buf[misalign:], torch.from_numpy(off.copy()).cuda(), ids, got_off, ws)
    assert B.bpe_encode_status(ws) == 0
    assert np.array_equal(got_off.cpu().numpy(), want_off)
    got = ids.cpu().numpy()
    assert np.array_equal(got[:want_ids.size], want_ids) and (got[want_ids.size:] == -7).all()
    table.free()


def _word_parts(rng, sizes, letters):
    """Parts of these sizes: a space and bytes that no table lets a cut through."""
    return np.concatenate([np.concatenate([[0x20], rng.choice(letters, n - 1)]) for n in sizes]).astype(np.uint8)


@pytest.mark.parametrize("misalign", [0, 5, 15])
@pytest.mark.parametrize("table", ["t1k", "t50k"])
def test_parts(oracle_mod, table, misalign):
    from workloads import configs as C
    rng = np.random.default_rng(misalign)
    merges = C.load_merges(table)
    text = C.make_eval("seq131k")["bytes"]
    letters = np.unique(text[(text >= 97) & (text <= 122)])
    for sizes in ([2053], [2052, 2053, 2054], [2100, 2100, 5], [4096 - 16, 2053, 40, 2053], [3, 4091, 2060, 7, 9000, 20],
                  [50] * 60 + [2060] + [700, 800] + [2500]):
        data = _word_parts(rng, sizes, letters)
        _check(oracle_mod, merges, data, [0, data.size], misalign, f"{table} parts {sizes[-4:]}")
    data = np.concatenate([text[:20000], _word_parts(rng, [6000], letters), np.full(5000, 97, np.uint8), text[:9000]])
    off = np.concatenate([[0], np.sort(rng.choice(data.size, 9)), [data.size]])
    _check(oracle_mod, merges, data, off, misalign, f"{table} ragged")
    _check(oracle_mod, merges, data, np.sort(np.concatenate([off, off[3:5]])), misalign, f"{table} empty pieces")


@pytest.mark.parametrize("n,n_pieces", [(2_053, 1), (40_000, 1), (840_501, 206), (1_400_000, 255)])
def test_text(oracle_mod, n, n_pieces):
    from workloads import configs as C
    for table, name in (("t100k", "stress"), ("t50k", "seq131k")):
        data = np.resize(C.make_eval(name)["bytes"], n)
        _check(oracle_mod, C.load_merges(table), data, np.arange(n_pieces + 1, dtype=np.int64) * n // n_pieces, 3, name)


@pytest.mark.parametrize("table", ["t50k", "t100k"])
@pytest.mark.parametrize("n_pieces", [4, 60, 230])
def test_pieces_that_little_would_be_gained_by_cutting(oracle_mod, table, n_pieces):
    """Text without spaces and random bytes, in pieces of up to 8,064 bytes, are merged as a whole: among text (which is cut), short
    and empty pieces, runs, and pieces of 2,052, 2,053, 8,064 and 8,065 bytes, with tiles of each size."""
    import torch  # noqa: F401  (its HIP runtime before the library's)
    from workloads import configs as C
    rng = np.random.default_rng(n_pieces)
    merges = C.load_merges(table)
    text = C.make_eval("batch")["bytes"]
    no_space = text[text != 0x20]
    kinds = {"text": text, "no space": no_space, "random": rng.integers(0, 256, 20_000).astype(np.uint8),
             "runs": np.repeat(rng.integers(0, 256, 200), 200).astype(np.uint8), "half": np.concatenate([no_space[:2600], text[:2600]] * 6)}
    names = list(kinds)
    sizes = [2053, 8064, 8065, 2052, 0, 1, 700, 4096, 3072, 9000]
    pieces = []
    for k in range(n_pieces):
        src = kinds[names[int(rng.integers(len(names)))] if k else "no space"]
        size = sizes[k % len(sizes)] if k < 2 * len(sizes) else int(rng.integers(2053, 8100))
        at = int(rng.integers(0, src.size - size)) if src.size > size else 0
        pieces.append(src[at:at + size])
    if n_pieces == 4:
        pieces[2] = no_space[:1024 * 5 - len(pieces[0]) % 1024]
    data = np.concatenate(pieces)
    off = np.concatenate([[0], np.cumsum([len(x) for x in pieces])])
    want = oracle_mod.encode(oracle_mod.Table(merges), data, off.astype(np.int32), n_threads=16)
    for misalign in (0, 7):
        _check(oracle_mod, merges, data, off, misalign, f"{table}, {n_pieces} pieces", want)


@pytest.mark.parametrize("size,n,longest", [(1024, 80_000, 6000), (2048, 500_000, 6200), (3072, 700_000, 9300)])
def test_whole_pieces_that_start_at_the_edges_of_tiles(oracle_mod, size, n, longest):
    import torch  # noqa: F401
    from workloads import configs as C
    import paper_2603_02597_amd as B
    merges = C.load_merges("t50k")
    text = C.make_eval("batch")["bytes"]
    data = np.resize(text[text != 0x20][:40_000], n)
    rng = np.random.default_rng(size)
    off = [0]
    while off[-1] < n - 9300:
        off.append((off[-1] + int(rng.integers(longest - 3000, longest))) // size * size + int(rng.choice([-1, 0, 0, 1, 16])))
    off = np.concatenate([off, [n]]).astype(np.int32)
    assert (np.diff(off) > 0).all() and off.size <= 257
    launches = {l["kernel"]: l["grid"] for l in B.bpe_encode_plan(n, off.size - 1)["launches"]}
    assert launches["merge_cut_tiles_kernel"] == -(-(n + 15) // size)
    want = oracle_mod.encode(oracle_mod.Table(merges), data, off, n_threads=16)
    _check(oracle_mod, merges, data, off, 0, f"tiles of {size}", want)
    _check(oracle_mod, merges, data, off, 5, f"tiles of {size}", want)
