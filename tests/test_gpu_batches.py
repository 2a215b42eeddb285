"""Batches from host to host (Tokenizer on bpe_batch_in, bpe_batch_ids_out, bpe_batch_bytes_out): sizes around the 16 bytes
a lane moves, every kind of text, buffers that grow, outputs beyond the buffers, and arguments that are refused."""
import numpy as np
import pytest

import oracle
from workloads import configs as C

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import paper_2603_02597_amd as B
    merges = C.load_merges("t1k")
    output_ids = (np.random.default_rng(3).permutation(256 + len(merges)) + 5).astype(np.int32)
    return B, merges, output_ids, C.make_eval("seq32k")["bytes"].tobytes()


def _want(merges, output_ids, texts):
    table, out = oracle.Table(merges), []
    for t in texts:
        raw = t.encode("utf-8") if isinstance(t, str) else bytes(t)
        ids = oracle.encode_raw(table, np.frombuffer(raw, dtype=np.uint8))[0]
        out.append(ids if output_ids is None else oracle.map_ids(ids, output_ids))
    return out


@pytest.mark.parametrize("renumber", [False, True])
def test_sizes_and_kinds(setup, renumber):
    B, merges, output_ids, data = setup
    ids_of = output_ids if renumber else None
    tok = B.Tokenizer(merges, output_ids=ids_of)
    ascii_text = data.decode("ascii")
    batches = [[ascii_text[:n]] for n in (0, 1, 3, 7, 8, 9, 15, 16, 17, 31, 33)]
    batches += [[ascii_text[k:k + n] for k in range(n + 1)] for n in (1, 2, 5)]
    batches += [[""] * 70, [ascii_text[:100000], "", ascii_text[:33]], ["café", ascii_text[:20], "中文"], [data[:50], ascii_text[:50]],
                [bytearray(data[:30])], (ascii_text[:10], ascii_text[:11])]
    for texts in batches:
        got, ms = tok.tokenize_batch(texts)
        want = _want(merges, ids_of, texts)
        assert len(got) == len(want) and ms >= 0 and all(np.array_equal(a, b) for a, b in zip(got, want)), texts[:3]
        assert all(a.dtype == np.int32 and a.flags.owndata for a in got)
        assert tok.decode_batch(got) == [t.encode("utf-8") if isinstance(t, str) else bytes(t) for t in texts]
    assert len(tok.tokenize_batch(t for t in ["ab", "c"])[0]) == 2
    ids = np.concatenate(_want(merges, ids_of, [data[:64]]))
    assert b"".join(tok.decode_batch([ids.tolist(), ids[:len(ids) // 2 * 2].reshape(2, -1)])).startswith(data[:64])
    tok.close()


def test_outputs_beyond_the_buffers_and_unknown_ids(setup):
    B, merges, _, _ = setup
    doubling = [(120, 120)] + [(256 + k, 256 + k) for k in range(11)]           # the last id stands for 4,096 bytes
    tok = B.Tokenizer(doubling)
    for n in (255, 256, 257, 3000):                                            # up to and beyond 1 MiB
        assert tok.decode_batch([[267] * n, [120]]) == [b"x" * (4096 * n), b"x"]
    for bad in ([268], [-1]):
        with pytest.raises(B.BpeError) as e:
            tok.decode_batch([bad, [120]])
        assert e.value.code == -11
        assert tok.decode_batch([[256]]) == [b"xx"]
    tok.close()


def test_arguments_that_are_refused(setup):
    import torch
    B, merges, _, _ = setup
    lib = B.load_library()
    host, dev = torch.zeros(64, dtype=torch.uint8, pin_memory=True), torch.zeros(64, dtype=torch.uint8, device="cuda")
    h, d = host.data_ptr(), dev.data_ptr()
    assert lib.bpe_host_visible(h) == 1 and lib.bpe_host_visible(None) == 0
    assert lib.bpe_batch_in(None, d, 16, d, None) == -1 and lib.bpe_batch_in(h + 4, d, 16, d, None) == -2
    assert lib.bpe_batch_in(h, d, -1, d, None) == -2
    assert lib.bpe_batch_ids_out(None, d, 0, 4, h, d, d, h, None) == -2 and lib.bpe_batch_ids_out(None, d, 1, 4, None, d, d, h, None) == -1
    assert lib.bpe_batch_bytes_out(d + 8, 16, d, 1, d, 1, h, h, d, d, h, None) == -2
    tok = B.Tokenizer(merges)
    assert lib.bpe_batch_ids_out(tok.vocab._h, d, 1, 4, h, d, d, h, None) == -10      # no output ids
    tok.close()
