"""One Tokenizer in several threads, each on a stream of its own: batches that grow while others are under way, encoded and
decoded beside each other, exact against the CPU oracle; and the kernel time that it reports."""
import threading

import numpy as np
import pytest

import oracle
from workloads import configs as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("renumber", [False, True])
def test_threads_that_share_a_tokenizer(renumber):
    import torch
    import paper_2603_02597_amd as B
    merges, data = C.load_merges("t1k"), C.make_eval("seq32k")["bytes"].tobytes()
    output_ids = (np.random.default_rng(3).permutation(256 + len(merges)) + 5).astype(np.int32) if renumber else None
    table, tok, failed = oracle.Table(merges), B.Tokenizer(merges, output_ids=output_ids), []

    def ids_of(t):
        ids = oracle.encode_raw(table, np.frombuffer(t, dtype=np.uint8))[0]
        return oracle.map_ids(ids, output_ids) if renumber else ids

    batches = []               # per thread: other texts, most of them longer than the ones before
    for k in range(4):
        sizes = [100 + 37 * k, 3000, 700, 30000 + 1000 * k, 50, 90000, 2000]
        batches.append([[data[1000 * k:1000 * k + n], b"", data[500 * k:500 * k + n // 3]] for n in sizes])
    wants = [[[ids_of(t) for t in texts] for texts in batch] for batch in batches]

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(20):
                    texts, want = batches[k][i % len(batches[k])], wants[k][i % len(batches[k])]
                    if k % 2:
                        good = tok.decode_batch(want) == texts
                    else:
                        good = all(np.array_equal(a, b) for a, b in zip(tok.tokenize_batch(texts)[0], want))
                    if not good:
                        failed.append((k, i))
        except Exception as e:         # (an assertion in a thread would go unseen)
            failed.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
    tok.close()


@pytest.mark.parametrize("renumber", [False, True])
def test_kernel_time_is_within_the_call(renumber):
    """A clock that is not written, or read before it is, would give none or hours."""
    import time
    import paper_2603_02597_amd as B
    merges, data = C.load_merges("t1k"), C.make_eval("seq32k")["bytes"].tobytes()
    tok = B.Tokenizer(merges, output_ids=np.arange(256 + len(merges), dtype=np.int32) if renumber else None)
    for n in (1, 100, 30000, len(data)):
        for _ in range(3):
            t0 = time.perf_counter()
            _, ms = tok.tokenize_batch([data[:n]])
            assert 0 < ms <= (time.perf_counter() - t0) * 1e3
    tok.close()
