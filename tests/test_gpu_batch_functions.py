"""bpe_batch_in, bpe_batch_ids_out and bpe_batch_bytes_out by themselves, with guard words behind every buffer: lengths around
the 16 bytes a lane moves and beyond one pass of the grid, offsets that end inside a group of four words, lengths that max_ids
and capacity cut off, and output that the decoder had to cut off."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
GUARD = 0x5A
ONE_PASS = 512 * 256 * 16            # bytes that the largest grid moves without a second turn


def _up16(n):
    return (n + 15) & ~15


class Buffers:
    def __init__(self):
        import torch
        import paper_2603_02597_amd as B
        self.torch, self.B, self.lib = torch, B, B.load_library()
        self.clock = torch.zeros(1, dtype=torch.int64, device="cuda")
        self.status = torch.zeros(64, dtype=torch.int32, device="cuda")       # of a workspace that no call has used

    def host(self, n_bytes):
        """A pinned buffer of n_bytes, up to a multiple of 16, with 64 guard bytes behind it."""
        return self.torch.full((_up16(n_bytes) + 64,), GUARD, dtype=self.torch.uint8, pin_memory=True)

    def device(self, a):
        t = self.torch.full((_up16(a.nbytes) + 64,), GUARD, dtype=self.torch.uint8, device="cuda")
        t[:a.nbytes] = self.torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1).copy()).cuda()
        return t


@pytest.fixture(scope="module")
def buffers():
    return Buffers()


def _guarded(t, n_bytes):
    """The first n_bytes of t, behind which only the rest of the last 16 may have changed."""
    a = t.cpu().numpy()
    assert (a[_up16(n_bytes):] == GUARD).all()
    return a[:n_bytes]


@pytest.mark.parametrize("n", [0, 1, 15, 16, 17, 31, 33, 4095, 4097, ONE_PASS - 1, ONE_PASS + 17])
def test_in(buffers, n):
    data = np.random.default_rng(n).integers(0, 256, n).astype(np.uint8)
    h, d = buffers.host(n), buffers.device(np.full(n, 7, dtype=np.uint8))
    h[:n] = buffers.torch.from_numpy(data)
    assert buffers.lib.bpe_batch_in(h.data_ptr(), d.data_ptr(), n, buffers.clock.data_ptr(), None) == 0
    buffers.torch.cuda.synchronize()
    assert np.array_equal(_guarded(d, n), data) and int(buffers.clock.item()) > 0


@pytest.mark.parametrize("renumber", [False, True])
@pytest.mark.parametrize("n_offsets,n_ids,max_ids", [(k, n, m) for k in (1, 2, 3, 4, 5, 8) for n, m in ((0, 9), (1, 9), (3, 3), (7, 9), (9, 9), (9, 2), (9, 0))] +
                         [(3, ONE_PASS // 4 + 5, ONE_PASS // 4 + 5), (6, ONE_PASS // 4 + 9, ONE_PASS // 4 + 1), (ONE_PASS // 4 + 2, 11, 11)])
def test_ids_out(buffers, renumber, n_offsets, n_ids, max_ids):
    rng = np.random.default_rng(n_offsets + n_ids)
    merges = [(97, 98), (256, 99), (257, 257)]
    out_of = (rng.permutation(259) + 1000).astype(np.int32)
    vocab = buffers.B.Vocab(merges, output_ids=out_of)
    ids = rng.integers(-1, 261, n_ids).astype(np.int32)                       # unknown ones among them
    offsets = np.sort(rng.integers(0, n_ids + 1, n_offsets)).astype(np.int32)
    offsets[-1] = n_ids
    n = n_offsets + min(n_ids, max_ids)
    want = np.concatenate([offsets, ids])[:n]
    if renumber:
        known = (want >= 0) & (want < 259)
        want[n_offsets:] = np.where(known, out_of[np.where(known, want, 0)], -1)[n_offsets:]
    words, host, head = buffers.device(np.concatenate([offsets, ids])), buffers.host(4 * n), buffers.host(36)
    assert buffers.lib.bpe_batch_in(host.data_ptr(), buffers.device(np.zeros(4, np.int32)).data_ptr(), 16, buffers.clock.data_ptr(), None) == 0
    assert buffers.lib.bpe_batch_ids_out(vocab._h if renumber else None, words.data_ptr(), n_offsets, max_ids, host.data_ptr(), buffers.status.data_ptr(),
                                         buffers.clock.data_ptr(), head.data_ptr(), None) == 0
    buffers.torch.cuda.synchronize()
    assert np.array_equal(_guarded(host, 4 * n).view(np.int32), want)
    head = _guarded(head, 36).view(np.int32)
    assert not head[:8].any() and 0 <= head[8] < 100_000                       # (1 ms)
    vocab.free()


def _bytes_out(buffers, vocab, ids, bounds, room, capacity):
    """bpe_decode into `room` bytes, bpe_batch_bytes_out of at most `capacity`: (starts, host buffer, head)."""
    torch, lib = buffers.torch, buffers.lib
    d_ids, out = torch.from_numpy(ids).cuda(), torch.zeros(_up16(max(room, 1)) + 16, dtype=torch.uint8, device="cuda")
    at, d_bounds = torch.zeros(ids.size + 1, dtype=torch.int32, device="cuda"), torch.from_numpy(bounds).cuda()
    ws = torch.zeros(buffers.B.bpe_decode_workspace_bytes(ids.size), dtype=torch.uint8, device="cuda")
    starts, host, head = buffers.host(4 * bounds.size), buffers.host(capacity), buffers.host(36)
    assert lib.bpe_batch_in(host.data_ptr(), out.data_ptr(), 0, buffers.clock.data_ptr(), None) == 0
    assert lib.bpe_decode(vocab._h, d_ids.data_ptr(), ids.size, None, 0, out.data_ptr(), room, at.data_ptr(), None, ws.data_ptr(), ws.numel(), None) == 0
    assert lib.bpe_batch_bytes_out(out.data_ptr(), capacity, at.data_ptr(), ids.size, d_bounds.data_ptr(), bounds.size, starts.data_ptr(),
                                   host.data_ptr(), ws.data_ptr(), buffers.clock.data_ptr(), head.data_ptr(), None) == 0
    torch.cuda.synchronize()
    return _guarded(starts, 4 * bounds.size).view(np.int32), host, _guarded(head, 36).view(np.int32)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 4097, ONE_PASS + 17])
def test_bytes_out(buffers, n):
    rng = np.random.default_rng(n)
    vocab = buffers.B.Vocab([(97, 98), (256, 99)])
    ids = rng.integers(97, 100, n).astype(np.int32)
    want = ids.astype(np.uint8)
    bounds = np.concatenate([[0], np.sort(rng.integers(0, n + 1, 5)), [n]]).astype(np.int32)
    for capacity in sorted({n, n + 16, _up16(n), n // 2, max(n - 1, 0), 0}):
        starts, host, head = _bytes_out(buffers, vocab, ids, bounds, n, capacity)
        assert np.array_equal(starts, bounds) and buffers.lib.bpe_status_from_words(head.ctypes.data) == 0 and head[8] > 0
        shown = min(n, capacity)
        assert np.array_equal(_guarded(host, shown), want[:shown])
    vocab.free()


@pytest.mark.parametrize("n", [1, 17, 5000])
def test_bytes_that_the_decoder_cut_off_stay_there(buffers, n):
    vocab = buffers.B.Vocab([(120, 120)] + [(256 + k, 256 + k) for k in range(5)])            # the last id stands for 64 bytes
    ids, bounds = np.full(n, 261, dtype=np.int32), np.array([0, n // 2, n], dtype=np.int32)
    for room in (64 * n - 1, 32 * n, 0):
        starts, host, head = _bytes_out(buffers, vocab, ids, bounds, room, room)
        assert np.array_equal(starts, 64 * bounds) and buffers.lib.bpe_status_from_words(head.ctypes.data) == -2
        assert (host.numpy() == GUARD).all()
    starts, host, head = _bytes_out(buffers, vocab, ids, bounds, 64 * n, 64 * n)
    assert buffers.lib.bpe_status_from_words(head.ctypes.data) == 0 and (_guarded(host, 64 * n) == 120).all()
    vocab.free()
