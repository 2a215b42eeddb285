"""The paper's Python-facing call (section 3.7): a list of texts in, token ids
per text and the kernel time out.  Marshalling only: the texts are concatenated
behind their offsets into one pinned host buffer, a kernel brings them to the GPU,
bpe_encode_raw does the rest (piece starts, merges, ids per text), and a kernel puts offsets and ids into
pinned memory; decode_batch goes the other way through bpe_decode.  Buffers grow to
the largest batch seen and are reused, so a steady stream of batches allocates nothing; threads
may share a Tokenizer and use these buffers one after the other."""
from __future__ import annotations

import ctypes
import threading

import numpy as np

from . import binding as B


# decode_batch keeps buffers for batches of up to so many tokens, of up to 16 bytes per token, and of up to so many texts (pinned:
# 4 + 16 bytes per token and 8 per text, 24 MiB at most).  Larger batches have memory of their own.
_DECODE_TOKENS_MAX, _DECODE_TEXTS_MAX = 1 << 20, 1 << 18

_utf8 = ctypes.pythonapi.PyUnicode_AsUTF8AndSize
_utf8.restype = ctypes.c_void_p
_utf8.argtypes = [ctypes.py_object, ctypes.POINTER(ctypes.c_ssize_t)]


def _up16(n: int) -> int:
    return (n + 15) & ~15


class Tokenizer:
    def __init__(self, merges, ranks=None, merged_ids=None, output_ids=None, device="cuda:0"):
        import torch
        self._torch = torch
        self.device = torch.device(device)
        self._lock = threading.Lock()      # held from the packing of a batch until its results are copied out
        with torch.cuda.device(self.device):
            self.table = B.Table(merges, ranks, merged_ids)
            self.vocab = B.Vocab(merges, ranks, merged_ids, output_ids)
            self._clock = torch.zeros(1, dtype=torch.int64, device=self.device)
            self._head = self._pinned(64)
            torch.cuda.current_stream().synchronize()      # (the clock is zero whatever stream the first batch is on)
        self._head_np = self._head.numpy().view(np.int32)
        self._use_output_ids = output_ids is not None
        self._cap_bytes = self._cap_seqs = 0
        self._cap_tokens = self._cap_texts = 0

    def _pinned(self, n_bytes: int):
        t = self._torch.empty(n_bytes, dtype=self._torch.uint8, pin_memory=True)
        if not B.load_library().bpe_host_visible(t.data_ptr()):
            raise RuntimeError("the GPU does not reach pinned host memory at its host address")
        return t

    def _reserve(self, n_bytes: int, n_seqs: int):
        torch = self._torch
        if n_bytes <= self._cap_bytes and n_seqs <= self._cap_seqs:
            return
        nb = max(n_bytes, 2 * self._cap_bytes, 1 << 16)
        ns = max(n_seqs, 2 * self._cap_seqs, 64)
        self._cap_bytes = self._cap_seqs = 0          # until every buffer is there: an allocation may fail
        dev = self.device
        # One buffer each way:
        # in  = [sequence offsets int32 (n_seqs + 1) | bytes], packed per call;
        # out = [first token of every sequence int32 (n_seqs + 1) | token ids].
        n_in, n_out = _up16(4 * (ns + 1) + nb), _up16(4 * (ns + 1 + nb))
        self._h_in, self._h_out = self._pinned(n_in), self._pinned(n_out)
        self._d_in = torch.empty(n_in, dtype=torch.uint8, device=dev)
        self._d_out = torch.empty(n_out, dtype=torch.uint8, device=dev)
        self._h_in_np, self._h_out_np = self._h_in.numpy(), self._h_out.numpy().view(np.int32)
        self._ws = torch.empty(B.bpe_encode_raw_workspace_bytes(nb, 0, ns), dtype=torch.uint8, device=dev)
        self._cap_bytes, self._cap_seqs = nb, ns

    def _finish(self, stream):
        """Waits for the batch and raises if its verdict is an error other than a too small output;
        returns the verdict."""
        stream.synchronize()
        lib = B.load_library()
        st = lib.bpe_status_from_words(self._head.data_ptr())
        if st != 0 and st != -2:
            raise B.BpeError(st, lib.bpe_last_error().decode(errors="replace"))
        return st

    @staticmethod
    def _check(rc: int):
        if rc != 0:
            raise B.BpeError(rc, B.load_library().bpe_last_error().decode(errors="replace"))

    def tokenize_batch(self, texts):
        """texts: list of bytes (or str, encoded as UTF-8).  Returns (list of int32
        arrays, kernel_ms): the ids of every text and the GPU time from the end of the transfer in to the
        start of the transfer out, that is of the encode kernels: neither transfer is in it, nor the
        renumbering to output ids, which the transfer out does on the way.
        The texts are packed into pinned memory; a kernel brings them to the GPU, the encode kernels
        follow, and one more puts the ids, renumbered if need be, and the verdict into pinned memory
        (as many as there are: the number is on the GPU): one synchronisation."""
        torch = self._torch
        if not isinstance(texts, (list, tuple)):
            texts = list(texts)
        n_seqs = len(texts)
        if n_seqs == 0:
            return [], 0.0
        # text that is ASCII is copied from where it lies (every string knows whether it is, so nothing is joined to find out)
        if set(map(type, texts)) == {str} and all(map(str.isascii, texts)):
            joined = texts[0] if n_seqs == 1 else "".join(texts)
            size = ctypes.c_ssize_t()
            source = _utf8(joined, ctypes.byref(size))
            raw = texts
        else:
            source = None
            raw = [t.encode("utf-8") if isinstance(t, str) else t for t in texts]
            joined = raw[0] if n_seqs == 1 else b"".join(raw)
        n_bytes = len(joined)
        if n_bytes >= 2**31 - 1:
            raise ValueError("a batch must stay below 2^31 bytes")
        with torch.cuda.device(self.device), self._lock:
            self._reserve(n_bytes, n_seqs)
            lib = B.load_library()
            n_in = 4 * (n_seqs + 1)
            seq_np = self._h_in_np[:n_in].view(np.int32)
            seq_np[0] = 0
            if n_seqs == 1:
                seq_np[1] = n_bytes
            else:
                seq_np[1:] = np.cumsum(np.fromiter(map(len, raw), dtype=np.int64, count=n_seqs))
            if source is not None:
                ctypes.memmove(self._h_in.data_ptr() + n_in, source, n_bytes)
            elif n_bytes:
                self._h_in_np[n_in:n_in + n_bytes] = np.frombuffer(joined, dtype=np.uint8)
            stream = torch.cuda.current_stream()
            s, clock, ws = stream.cuda_stream, self._clock.data_ptr(), self._ws.data_ptr()
            d_in, d_out = self._d_in.data_ptr(), self._d_out.data_ptr()
            try:
                self._check(lib.bpe_batch_in(self._h_in.data_ptr(), d_in, n_in + n_bytes, clock, s))
                self._check(lib.bpe_encode_raw(self.table._h, d_in + n_in, n_bytes, d_in, n_seqs, 0, d_out + n_in, d_out,
                                               None, None, None, ws, self._ws.numel(), None, s))
                self._check(lib.bpe_batch_ids_out(self.vocab._h if self._use_output_ids else None, d_out, n_seqs + 1, n_bytes,
                                                  self._h_out.data_ptr(), ws, clock, self._head.data_ptr(), s))
                st = self._finish(stream)
            except BaseException:
                stream.synchronize()       # what is under way still writes to the buffers, and the next batch may be on another stream
                raise
            if st != 0:
                raise B.BpeError(st, lib.bpe_last_error().decode(errors="replace"))
            tok = self._h_out_np[:n_seqs + 1].tolist()
            ids = self._h_out_np[n_seqs + 1:n_seqs + 1 + tok[-1]]
            return [ids[a:b].copy() for a, b in zip(tok, tok[1:])], max(int(self._head_np[8]), 0) * 1e-5

    def _reserve_decode(self, n_tokens: int, n_texts: int):
        torch = self._torch
        if n_tokens <= self._cap_tokens and n_texts <= self._cap_texts:
            return
        nt = min(max(n_tokens, 2 * self._cap_tokens, 1 << 14), _DECODE_TOKENS_MAX)
        nx = min(max(n_texts, 2 * self._cap_texts, 64), _DECODE_TEXTS_MAX)
        self._cap_tokens = self._cap_texts = 0        # as in _reserve
        dev = self.device
        # in  = [ids int32 | index of every text's first id, and their number, int32 (n_texts + 1)], packed per call;
        # out = [first byte of every text int32 (n_texts + 1), up to a multiple of 16 bytes | bytes]
        n_in, self._decode_bytes = _up16(4 * (nt + nx + 1)), max(16 * nt, 1 << 20)
        self._hd_in, self._hd_out = self._pinned(n_in), self._pinned(_up16(4 * (nx + 1)) + self._decode_bytes)
        self._dd_in = torch.empty(n_in, dtype=torch.uint8, device=dev)
        self._dd_out = torch.empty(self._decode_bytes, dtype=torch.uint8, device=dev)
        self._dd_tbo = torch.empty(nt + 1, dtype=torch.int32, device=dev)
        self._hd_in_np, self._hd_out_np = self._hd_in.numpy().view(np.int32), self._hd_out.numpy()
        self._dws = torch.empty(B.bpe_decode_workspace_bytes(nt), dtype=torch.uint8, device=dev)
        self._cap_tokens, self._cap_texts = nt, nx

    def _decode_pinned(self, arrs, sizes, n_tokens: int):
        """decode_batch of at most _DECODE_TOKENS_MAX tokens and _DECODE_TEXTS_MAX texts through the pinned buffers.  If the bytes do not fit them, their
        size is known by then: decoded once more, into memory of that size."""
        n_texts = len(arrs)
        self._reserve_decode(n_tokens, n_texts)
        lib = B.load_library()
        h = self._hd_in_np
        np.concatenate(arrs, out=h[:n_tokens])
        h[n_tokens] = 0
        h[n_tokens + 1:n_tokens + 1 + n_texts] = np.cumsum(sizes)
        stream = self._torch.cuda.current_stream()
        s, clock, ws, tbo = stream.cuda_stream, self._clock.data_ptr(), self._dws.data_ptr(), self._dd_tbo.data_ptr()
        d_in, d_out, h_out, n_starts = self._dd_in.data_ptr(), self._dd_out.data_ptr(), self._hd_out.data_ptr(), _up16(4 * (n_texts + 1))
        try:
            self._check(lib.bpe_batch_in(self._hd_in.data_ptr(), d_in, 4 * (n_tokens + n_texts + 1), clock, s))
            self._check(lib.bpe_decode(self.vocab._h, d_in, n_tokens, None, 1 if self._use_output_ids else 0, d_out, self._decode_bytes, tbo,
                                       None, ws, self._dws.numel(), s))
            self._check(lib.bpe_batch_bytes_out(d_out, self._decode_bytes, tbo, n_tokens, d_in + 4 * n_tokens, n_texts + 1, h_out,
                                                h_out + n_starts, ws, clock, self._head.data_ptr(), s))
            st = self._finish(stream)
            starts = self._hd_out_np[:4 * (n_texts + 1)].view(np.int32).tolist()
            text = self._hd_out_np[n_starts:]
            if st != 0:
                if starts[-1] < 0:
                    raise ValueError("the decoded text would exceed 2^31 bytes")
                out = self._torch.empty(starts[-1], dtype=self._torch.uint8, device=self.device)
                self._check(lib.bpe_decode(self.vocab._h, d_in, n_tokens, None, 1 if self._use_output_ids else 0, out.data_ptr(), starts[-1],
                                           tbo, None, ws, self._dws.numel(), s))
                self._check(B.bpe_encode_status(self._dws))
                text = out.cpu().numpy()
        except BaseException:
            stream.synchronize()           # as in tokenize_batch
            raise
        return [text[a:b].tobytes() for a, b in zip(starts, starts[1:])]

    def decode_batch(self, ids_list):
        """ids_list: list of int arrays (output ids if the tokenizer has them).  Returns list of bytes."""
        torch = self._torch
        arrs = [np.ascontiguousarray(a, dtype=np.int32) for a in ids_list]
        if any(a.ndim != 1 for a in arrs):
            arrs = [a.reshape(-1) for a in arrs]
        if not arrs:
            return []
        sizes = [a.size for a in arrs]
        n_tokens = sum(sizes)
        if n_tokens == 0:
            return [b"" for _ in arrs]
        with torch.cuda.device(self.device):
            if n_tokens <= _DECODE_TOKENS_MAX and len(arrs) <= _DECODE_TEXTS_MAX:
                with self._lock:
                    return self._decode_pinned(arrs, sizes, n_tokens)
            dev = self.device
            bounds = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
            ids = torch.from_numpy(np.concatenate(arrs)).to(dev)
            # a first guess of 16 bytes per token; the kernel reports the true size if that is too small
            cap = min(n_tokens * int(self.vocab.info["max_token_bytes"]), max(16 * n_tokens, 1 << 20), 2**31 - 2)
            tbo = torch.empty(n_tokens + 1, dtype=torch.int32, device=dev)
            ws = torch.empty(B.bpe_decode_workspace_bytes(n_tokens), dtype=torch.uint8, device=dev)
            for attempt in range(2):
                out = torch.empty(cap, dtype=torch.uint8, device=dev)
                B.bpe_decode(self.vocab, ids, out, ws, token_byte_offsets=tbo, ids_are_output_ids=self._use_output_ids)
                st = B.bpe_encode_status(ws)
                if st == -2 and attempt == 0:          # BPE_ERR_SIZE: the offsets are the true ones
                    cap = int(tbo[-1].item())
                    if cap < 0:
                        raise ValueError("the decoded text would exceed 2^31 bytes")
                    continue
                if st != 0:
                    raise B.BpeError(st, B.load_library().bpe_last_error().decode(errors="replace"))
                break
            starts = tbo[torch.from_numpy(bounds).to(dev)].cpu().numpy()
            text = out[:int(starts[-1])].cpu().numpy().tobytes()
            return [text[starts[k]:starts[k + 1]] for k in range(len(arrs))]

    def close(self):
        self.table.free()
        self.vocab.free()
