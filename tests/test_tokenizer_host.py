"""The host side of Tokenizer without a GPU: the library's functions restated on host memory, with a check of every
access against the buffers that were allocated (a byte is a token; id k stands for (k >> 8) + 1 times the byte k & 255)."""
import contextlib
import ctypes
import sys
import threading
import time
import tracemalloc
import types

import numpy as np
import pytest
import torch

import paper_2603_02597_amd.tokenizer as tokenizer_module


class Device:
    """Stands in for torch, the binding and the library."""

    def __init__(self):
        self.allocated, self.fail_at, self.pause, self.calls = [], None, 0.0, []
        stream = types.SimpleNamespace(cuda_stream=0, synchronize=lambda: self._call("synchronize"))
        cuda = types.SimpleNamespace(device=lambda d: contextlib.nullcontext(), current_stream=lambda: stream)
        self.torch = types.SimpleNamespace(cuda=cuda, device=lambda d: "cpu", empty=self.empty, zeros=self.empty, uint8=torch.uint8,
                                           int32=torch.int32, int64=torch.int64, from_numpy=torch.from_numpy)
        handle = lambda *a: types.SimpleNamespace(_h=0, info={"max_token_bytes": 4096}, free=lambda: None)
        self.binding = types.SimpleNamespace(
            Table=handle, Vocab=handle, BpeError=RuntimeError, load_library=lambda: self, bpe_decode_workspace_bytes=lambda n: 64,
            bpe_encode_raw_workspace_bytes=lambda *a: 64, bpe_decode=self.decode_tensors, bpe_encode_status=lambda ws: int(self.words(ws.data_ptr(), 1)[0]))

    def _call(self, name):
        self.calls.append(name)
        if self.pause:
            time.sleep(self.pause)

    def empty(self, n, dtype, device=None, pin_memory=False):
        if self.fail_at is not None:
            self.fail_at -= 1
            if self.fail_at < 0:
                raise MemoryError
        t = torch.zeros(max(n, 1), dtype=dtype)
        self.allocated.append(t)
        return t

    def mem(self, at, n):
        assert n == 0 or any(t.data_ptr() <= at and at + n <= t.data_ptr() + t.nbytes for t in self.allocated), "outside every buffer"
        return np.frombuffer((ctypes.c_uint8 * n).from_address(at), dtype=np.uint8) if n else np.zeros(0, np.uint8)

    def words(self, at, n):
        return self.mem(at, 4 * n).view(np.int32)

    # the library
    def bpe_last_error(self):
        return b"error"

    def bpe_host_visible(self, at):
        return 1

    def bpe_status_from_words(self, at):
        return int(self.words(at, 1)[0])

    def bpe_batch_in(self, host, device, n, clock, stream):
        self._call("in")
        self.mem(device, n)[:] = self.mem(host, n)
        return 0

    def bpe_encode_raw(self, table, data, n, starts, n_seqs, ppw, ids, token_starts, a, b, c, ws, ws_bytes, options, stream):
        self._call("encode")
        self.words(ids, n)[:] = self.mem(data, n)
        self.words(token_starts, n_seqs + 1)[:] = self.words(starts, n_seqs + 1)
        self.words(ws, 1)[0] = 0
        return 0

    def bpe_batch_ids_out(self, vocab, words, n_offsets, max_ids, host, ws, clock, head, stream):
        self._call("ids out")
        n = n_offsets + int(self.words(words, n_offsets)[-1])
        self.words(host, n)[:] = self.words(words, n)
        self.words(head, 8)[0] = self.words(ws, 1)[0]
        return 0

    def bpe_decode(self, vocab, ids, n, n_device, output_ids, out, capacity, offsets, n_bytes, ws, ws_bytes, stream):
        self._call("decode")
        ids = self.words(ids, n)
        text = np.repeat((ids & 255).astype(np.uint8), (ids >> 8) + 1)
        self.words(offsets, n + 1)[1:] = np.cumsum((ids >> 8) + 1)
        self.words(offsets, 1)[0] = 0
        fits = min(text.size, capacity)
        self.mem(out, capacity)[:fits] = text[:fits]
        self.words(ws, 1)[0] = 0 if text.size <= capacity else -2
        return 0

    def bpe_batch_bytes_out(self, data, capacity, offsets, n, bounds, n_bounds, host_starts, host, ws, clock, head, stream):
        self._call("bytes out")
        offsets = self.words(offsets, n + 1)
        self.words(host_starts, n_bounds)[:] = offsets[self.words(bounds, n_bounds)]
        fits = min(int(offsets[-1]), capacity)
        self.mem(host, fits)[:] = self.mem(data, fits)
        self.words(head, 8)[0] = self.words(ws, 1)[0]
        return 0

    def decode_tensors(self, vocab, ids, out, ws, token_byte_offsets, ids_are_output_ids):
        self.allocated += [ids, out, ws, token_byte_offsets]
        self.bpe_decode(0, ids.data_ptr(), ids.numel(), None, 0, out.data_ptr(), out.numel(), token_byte_offsets.data_ptr(), None, ws.data_ptr(),
                        ws.numel(), 0)


@pytest.fixture
def device(monkeypatch):
    d = Device()
    monkeypatch.setitem(sys.modules, "torch", d.torch)
    monkeypatch.setattr(tokenizer_module, "B", d.binding)
    return d


def test_threads_that_share_a_tokenizer(device):
    tok, failed = tokenizer_module.Tokenizer([]), []
    device.pause = 0.0005

    def work(k):
        try:
            for i in range(12):
                ids = [np.full(1 + (7 * k + i) % 5, 65 + k, dtype=np.int32), np.full(i, 97 + k, dtype=np.int32)]
                if k == 2:
                    got = [a.tolist() for a in tok.tokenize_batch([a.astype(np.uint8).tobytes() for a in ids])[0]]
                    good = got == [a.tolist() for a in ids]
                else:
                    good = tok.decode_batch(ids) == [a.astype(np.uint8).tobytes() for a in ids]
                if not good:
                    failed.append((k, i))
        except Exception as e:         # (an assertion in a thread would go unseen)
            failed.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed


@pytest.mark.parametrize("fail_at", range(8))
def test_a_batch_whose_buffers_cannot_be_had(device, fail_at):
    """Whichever allocation of a larger batch fails, later batches are right and stay within their buffers."""
    tok = tokenizer_module.Tokenizer([])
    small = [np.arange(65, 90, dtype=np.int32), np.full(300, 0xF00 + 97, dtype=np.int32)]
    text = [b"ABCDEFGHIJKLMNOPQRSTUVWXY", b"a" * 4800]
    between = np.full(70000, 0xF00 + 98, dtype=np.int32)              # 16 bytes per token: more than the first buffers hold
    for grow, batches in ((lambda: tok.decode_batch([np.full(100000, 65, dtype=np.int32)] * 2),
                           (lambda: tok.decode_batch(small) == text, lambda: tok.decode_batch([between]) == [b"b" * 1120000])),
                          (lambda: tok.tokenize_batch([b"c" * 200000] * 100),
                           (lambda: [bytes(a.tolist()) for a in tok.tokenize_batch(text)[0]] == text,))):
        assert all(good() for good in batches[:1])
        device.fail_at = fail_at
        with contextlib.suppress(MemoryError):
            grow()
        device.fail_at = None
        assert all(good() for good in batches)


@pytest.mark.parametrize("refused", ["bpe_encode_raw", "bpe_batch_ids_out", "bpe_decode", "bpe_batch_bytes_out"])
def test_a_batch_that_ends_early_leaves_nothing_under_way(device, refused):
    tok = tokenizer_module.Tokenizer([])
    setattr(device, refused, lambda *a: -1)
    call = tok.tokenize_batch if refused in ("bpe_encode_raw", "bpe_batch_ids_out") else tok.decode_batch
    with pytest.raises(RuntimeError):
        call([b"abc"] if call == tok.tokenize_batch else [[65, 66]])
    assert "in" in device.calls and device.calls[-1] == "synchronize"


def test_texts_that_are_not_ascii_are_joined_once(device):
    """As bytes: each text's bytes and their join, twice the batch, and no join of the strings beside them."""
    tok = tokenizer_module.Tokenizer([])
    texts = ["word " * 4000] * 49 + ["café " * 4000]
    size = sum(len(t.encode()) for t in texts)
    tok.tokenize_batch(texts)                          # (buffers are there)
    device.bpe_batch_in = lambda *a: -1                # what follows the packing is not counted
    tracemalloc.start()
    with pytest.raises(RuntimeError):
        tok.tokenize_batch(texts)
    peak = tracemalloc.get_traced_memory()[1]
    tracemalloc.stop()
    assert peak < 2.5 * size


@pytest.mark.parametrize("n", [1, 5000, 70000])
def test_long_tokens_are_decoded_twice_at_most(device, n):
    """Beyond the buffers (16 bytes per token, 1 MiB at least): once to learn the size, once into memory of that size."""
    tok = tokenizer_module.Tokenizer([])
    per = (1 << 20) // n + 17
    ids = np.full(n, (per - 1) << 8 | 97, dtype=np.int32)
    assert tok.decode_batch([ids, [98]]) == [b"a" * (per * n), b"b"]
    assert device.calls.count("decode") == 2


def test_pinned_memory_for_decoding_is_bounded(device):
    """By the number of texts as well as by that of the tokens, whichever batches came before."""
    tok, empty = tokenizer_module.Tokenizer([]), np.zeros(0, dtype=np.int32)
    for n_tokens, n_texts in ((1, 1 << 18), (1, 1 << 20), (1 << 20, 1), ((1 << 20) + 1, 1), (5, 100)):
        assert tok.decode_batch([np.full(n_tokens, 66, dtype=np.int32)] + [empty] * (n_texts - 1)) == [b"B" * n_tokens] + [b""] * (n_texts - 1)
        assert tok._hd_in.nbytes + tok._hd_out.nbytes <= 24 << 20
