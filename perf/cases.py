"""Cases for timing the framework through its public entry points.

The work is byte-level BPE of word-like text (and of text mixed with random bytes and long
runs) with the three merge tables under workloads/tables, in the forms a program asks for it:

  encode      bpe_encode: bytes and piece offsets are on the GPU, ids and offsets stay there
  chunks      bpe_encode on text cut into chunks of a fixed number of bytes (the paper's own cut)
  raw         bpe_encode_raw: bytes and sequence offsets on the GPU, tokens only
  tokenize    Tokenizer.tokenize_batch: host strings in, host ids out
  decode      bpe_decode: ids on the GPU back to bytes on the GPU
  detokenize  Tokenizer.decode_batch: host ids in, host bytes out

Texts follow the recipe of workloads/textgen.py, drawn on the GPU so that large inputs are
made quickly: a case fixes which pieces each of its documents consists of, and with them the
number of pieces and tokens; the seed puts the pieces of every document in an order of its own.
Tables, vocabularies and tokenizers are kept for the life of the process, as a program keeps
them; inputs, outputs and workspaces are made anew for every state.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2603_02597_amd as B
from workloads import configs, textgen

DEVICE = "cuda:0"
TABLES = ("t1k", "t50k", "t100k")
MIXES = ("text", "stress")

# Pieces and tokens per input byte of each (table, mix), from 400 KB of each with the CPU oracle.
PIECES_PER_BYTE = {"text": 1 / 6.65, "stress": 1 / 7.65}
TOKENS_PER_BYTE = {("t1k", "text"): 0.278, ("t1k", "stress"): 0.397, ("t50k", "text"): 0.156,
                   ("t50k", "stress"): 0.274, ("t100k", "text"): 0.157, ("t100k", "stress"): 0.195}


def listed():
    return [
        # the smallest call: one short document, latency and launches count
        dict(name="encode_4k", op="encode", table="t1k", mix="text", bytes=4096),
        # one long document of about 131,072 tokens
        dict(name="encode_840k", op="encode", table="t50k", mix="text", bytes=840501),
        # a training or serving batch of documents
        dict(name="encode_13m", op="encode", table="t50k", mix="text", bytes=13510208),
        # text with binary data and long runs in it
        dict(name="encode_stress_4m", op="encode", table="t100k", mix="stress", bytes=3999992),
        # fixed chunks instead of word pieces: every piece is long
        dict(name="chunks_840k", op="chunks", table="t50k", mix="text", bytes=840501, chunk=2048),
        # raw bytes: one document, a batch of documents, a shard of a corpus
        dict(name="raw_840k", op="raw", table="t50k", mix="text", bytes=840501, seqs=1),
        dict(name="raw_13m", op="raw", table="t50k", mix="text", bytes=13510208, seqs=256),
        dict(name="raw_134m", op="raw", table="t50k", mix="text", bytes=134217727, seqs=4096),
        # host strings: one prompt with a vocabulary's own numbering, and a batch of prompts
        dict(name="tokenize_prompt", op="tokenize", table="t50k", mix="text", bytes=1537, seqs=1, renumber=True),
        dict(name="tokenize_48", op="tokenize", table="t50k", mix="text", bytes=840501, seqs=48, renumber=False),
        # ids back to bytes: on the GPU, and a batch of answers to host bytes
        dict(name="decode_13m", op="decode", table="t50k", mix="text", bytes=13510208, offsets=False, renumber=False),
        dict(name="detokenize_48", op="detokenize", table="t50k", mix="text", bytes=210001, seqs=48, renumber=False),
    ]


def draw(rng):
    def log_size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(("encode", "encode", "chunks", "raw", "raw", "tokenize", "decode", "detokenize"))
    case = dict(op=op, table=rng.choice(TABLES), mix=rng.choice(MIXES))
    if op == "encode":
        case.update(bytes=log_size(1000, 13_500_000))
    elif op == "chunks":
        case.update(bytes=log_size(20_000, 840_000), chunk=log_size(64, 4096))
    elif op == "raw":
        case.update(bytes=log_size(1000, 64_000_000))
        case.update(seqs=min(log_size(1, 4096), case["bytes"] // 200))
    elif op == "decode":
        case.update(bytes=log_size(1000, 13_500_000), offsets=rng.random() < 0.5, renumber=rng.random() < 0.5)
    else:      # strings, so no random bytes among them
        case.update(mix="text", bytes=log_size(300, 840_000), renumber=rng.random() < 0.5)
        case.update(seqs=min(log_size(1, 48), case["bytes"] // 100))
    return case


def _pieces(case):
    return case["bytes"] / case["chunk"] if case["op"] == "chunks" else case["bytes"] * PIECES_PER_BYTE[case["mix"]]


def work(case):
    """Input bytes and offsets read once, ids and offsets written once; integers only."""
    n, ids = case["bytes"], 4 * case["bytes"] * TOKENS_PER_BYTE[case["table"], case["mix"]]
    total = n + ids
    if case["op"] in ("encode", "chunks"):
        total += 8 * _pieces(case)               # piece offsets in, token offsets out
    elif case["op"] in ("raw", "tokenize", "detokenize"):
        total += 8 * case["seqs"]
    elif case["offsets"]:
        total += ids                             # a byte offset per token
    return {"bytes": total, "flops": 0}


def tolerance(case):
    return "exact"                               # ids, offsets and bytes


# ---------------------------------------------------------------------------
# What a program keeps: tables, vocabularies and tokenizers.

def _output_ids(table):
    """A vocabulary file's own numbering: some permutation of the ids."""
    return np.random.default_rng(7).permutation(256 + len(_merges(table))).astype(np.int32)


@functools.lru_cache(maxsize=None)
def _merges(table):
    return configs.load_merges(table)


@functools.lru_cache(maxsize=None)
def _table(table):
    return B.Table(_merges(table))


@functools.lru_cache(maxsize=None)
def _vocab(table, renumber):
    return B.Vocab(_merges(table), output_ids=_output_ids(table) if renumber else None)


@functools.lru_cache(maxsize=None)
def _tokenizer(table, renumber):
    return B.Tokenizer(_merges(table), output_ids=_output_ids(table) if renumber else None, device=DEVICE)


@functools.lru_cache(maxsize=None)
def _words(table):
    """The word list behind a table's text, on the GPU, and the cumulative Zipf weights of its ranks."""
    t = configs.TABLES[table]
    letters, starts, lens = textgen.make_wordlist(t["n_words"], t["vocab_seed"])
    w = np.arange(1, t["n_words"] + 1, dtype=np.float64) ** -textgen.ZIPF_S
    up = lambda a: torch.from_numpy(np.array(a)).to(DEVICE)
    return up(letters), up(starts), up(lens), up(np.cumsum(w) / w.sum()), up(textgen.PUNCT)


# ---------------------------------------------------------------------------
# Inputs.

def _text(table, mix, n_bytes, seed):
    """n_bytes bytes of units: a space, then a word, some punctuation, random bytes or a run of one byte."""
    letters, starts, lens, cdf, punct = _words(table)
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    m = n_bytes // 5 + 256                       # units are 6.3 bytes and more on average
    uniform = lambda: torch.rand(m, generator=g, device=DEVICE, dtype=torch.float64)
    below = lambda k, size=m: torch.randint(k, (size,), generator=g, device=DEVICE)
    kind, rank = uniform(), torch.searchsorted(cdf, uniform(), right=True).clamp_(max=len(lens) - 1)
    p_run, p_rand = (textgen.STRESS_P_RUN, textgen.STRESS_P_RAND) if mix == "stress" else (0.0, 0.0)
    is_run = kind < p_run
    is_rand = ~is_run & (kind < p_run + p_rand)
    is_text = ~is_run & ~is_rand
    is_punct = is_text & (uniform() < textgen.P_PUNCT)
    newline = (is_text & (uniform() < textgen.P_NEWLINE)).long()
    body = lens[rank]
    body = torch.where(is_punct, below(4) + 1, body)
    body = torch.where(is_rand, below(64) + 1, body)
    body = torch.where(is_run, below(4096 - 64 + 1) + 64, body)
    run_byte = below(255)
    run_byte = run_byte + (run_byte >= 0x20)     # never a space
    size = 1 + body + newline
    end = torch.cumsum(size, 0)
    m = int(torch.searchsorted(end, n_bytes - 1, right=True)) + 1       # the unit that holds the last byte
    assert m <= len(size)
    unit = torch.repeat_interleave(torch.arange(m, device=DEVICE), size[:m])[:n_bytes]
    at = torch.arange(n_bytes, device=DEVICE) - (end - size)[unit] - 1  # -1: the space
    word_at = (starts[rank][unit] + at).clamp_(0, len(letters) - 1)
    out = letters[word_at]
    out = torch.where(is_punct[unit], punct[below(len(punct), n_bytes)], out)
    if mix == "stress":
        out = torch.where(is_rand[unit], below(256, n_bytes).to(torch.uint8), out)
        out = torch.where(is_run[unit], run_byte.to(torch.uint8)[unit], out)
    out = torch.where(at == body[unit], torch.full_like(out, 0x0A), out)
    return torch.where(at < 0, torch.full_like(out, 0x20), out)


def _piece_offsets(data):
    """A piece starts at byte 0 and at every space."""
    start = data == 0x20
    start[0] = True
    return torch.cat([start.nonzero().flatten(), torch.tensor([data.numel()], device=DEVICE)]).to(torch.int32)


def _sequence_offsets(data, n_seqs):
    """n_seqs sequences of ragged lengths (one to sixteen times the shortest), cut at spaces."""
    weight = np.random.default_rng(n_seqs).uniform(1, 16, n_seqs)
    cut = torch.from_numpy(np.cumsum(weight)[:-1] / weight.sum() * data.numel()).to(DEVICE).long()
    pieces = _piece_offsets(data).long()
    cut = pieces[torch.searchsorted(pieces, cut).clamp_(max=len(pieces) - 1)]
    ends = [torch.zeros(1, dtype=torch.long, device=DEVICE), cut, torch.tensor([data.numel()], device=DEVICE)]
    return torch.cat(ends).to(torch.int32)


def _empty(n, dtype):
    return torch.empty(max(int(n), 1), dtype=dtype, device=DEVICE)


def _zeros(n, dtype):
    return torch.zeros(max(int(n), 1), dtype=dtype, device=DEVICE)


def _documents(case, seed):
    """The case's bytes and where its documents start."""
    data = _text(case["table"], case["mix"], case["bytes"], case["bytes"])
    seq = _sequence_offsets(data, case.get("seqs", 1))
    off = _piece_offsets(data).long()
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    document = torch.searchsorted(seq.long(), off[:-1], right=True)
    order = torch.argsort(document + torch.rand(len(off) - 1, generator=g, device=DEVICE, dtype=torch.float64))
    size = (off[1:] - off[:-1])[order]
    piece = torch.repeat_interleave(torch.arange(len(size), device=DEVICE), size)
    at = torch.arange(data.numel(), device=DEVICE) - (torch.cumsum(size, 0) - size)[piece]
    return data[off[:-1][order][piece] + at], seq


def _host_texts(case, seed):
    data, seq = _documents(case, seed)
    cuts = seq.cpu().numpy()
    host = data.cpu().numpy().tobytes()
    return [host[a:b] for a, b in zip(cuts[:-1], cuts[1:])]


def _encoded(case, data):
    """ids of data's pieces under the case's numbering."""
    ids, _ = B.encode(_table(case["table"]), data, _piece_offsets(data))
    if case["renumber"]:
        ids = torch.from_numpy(_output_ids(case["table"])).to(DEVICE)[ids.long()]
    return ids.contiguous()


def prepare(case, seed):
    s = dict(op=case["op"])
    if case["op"] == "tokenize":
        s.update(tokenizer=_tokenizer(case["table"], case["renumber"]),
                 texts=[t.decode("ascii") for t in _host_texts(case, seed)])
        return s
    if case["op"] == "detokenize":
        ids = [_encoded(case, torch.from_numpy(np.frombuffer(t, np.uint8).copy()).to(DEVICE)).cpu().numpy()
               for t in _host_texts(case, seed) if t]
        s.update(tokenizer=_tokenizer(case["table"], case["renumber"]), ids=ids)
        return s

    data, seq = _documents(case, seed)
    n = data.numel()
    if case["op"] == "decode":
        ids = _encoded(case, data)
        s.update(vocab=_vocab(case["table"], case["renumber"]), ids=ids, renumber=case["renumber"],
                 out=_zeros(n, torch.uint8), n_bytes=_zeros(1, torch.int32),
                 offsets=_zeros(ids.numel() + 1, torch.int32) if case["offsets"] else None,
                 workspace=_empty(B.bpe_decode_workspace_bytes(ids.numel()), torch.uint8))
        return s
    # (the ids that are written end where the offsets say; zeros behind them)
    s.update(table=_table(case["table"]), data=data, out_ids=_zeros(n, torch.int32))
    if case["op"] == "raw":
        s.update(seq_offsets=seq, token_offsets=_zeros(seq.numel(), torch.int32),
                 workspace=_empty(B.bpe_encode_raw_workspace_bytes(n, 0, seq.numel() - 1), torch.uint8))
        return s
    if case["op"] == "chunks":
        off = torch.from_numpy(textgen.fixed_chunks(n, case["chunk"])).to(DEVICE)
    else:
        off = _piece_offsets(data)
    s.update(piece_offsets=off, out_offsets=_zeros(off.numel(), torch.int32),
             workspace=_empty(B.bpe_workspace_bytes(n, off.numel() - 1), torch.uint8))
    return s


def run(s):
    """One call of the entry point that the case is about, and what it gives back."""
    if s["op"] == "tokenize":
        return s["tokenizer"].tokenize_batch(s["texts"])[0]
    if s["op"] == "detokenize":
        return [np.frombuffer(t, np.uint8) for t in s["tokenizer"].decode_batch(s["ids"])]
    if s["op"] == "decode":
        B.bpe_decode(s["vocab"], s["ids"], s["out"], s["workspace"], token_byte_offsets=s["offsets"],
                     n_bytes=s["n_bytes"], ids_are_output_ids=s["renumber"])
        return s["out"], s["n_bytes"], s["offsets"]
    if s["op"] == "raw":
        B.bpe_encode_raw(s["table"], s["data"], s["seq_offsets"], s["out_ids"], s["token_offsets"], s["workspace"])
        return s["out_ids"], s["token_offsets"]
    B.bpe_encode(s["table"], s["data"], s["piece_offsets"], s["out_ids"], s["out_offsets"], s["workspace"])
    return s["out_ids"], s["out_offsets"]
