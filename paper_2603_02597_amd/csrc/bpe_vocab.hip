// Vocabulary side of the tokenizer: what every token id stands for.  The paper
// takes GPT-2's vocabulary as given (section 3.2) and decodes on the host; here
// the byte expansion of every id is derived from the merge rules themselves
// (a merged id expands to the expansions of its two parts, section 3.3), kept on
// the device, and used to turn ids back into bytes (bpe_decode).  An optional
// renumbering (internal id <-> output id) lets a caller who has a real
// vocabulary file emit and accept that file's ids (bpe_map_ids).
//
// Decoding is an expansion: length of every token, running sum, copy.  One pass,
// one kernel: tiles of 1024 tokens, the bytes before a tile by decoupled
// look-back, the tile's bytes assembled in LDS and stored as aligned words.
#include <algorithm>
#include <cstring>
#include <new>

#include "bpe_common.h"
#include "bpe_lookback.h"

typedef uint32_t Record __attribute__((ext_vector_type(4)));

struct bpe_vocab {
    bpe_vocab_info_t info;
    void *device_mem;      // one allocation: tok | tok_out | out_of | int_of | pool
    const Record *tok;      // [n_ids] by internal id: see token_record
    const Record *tok_out;  // [n_out] by output id, or nullptr
    const int32_t *out_of, *int_of;
    int64_t token_bytes;    // of all expansions
    const uint8_t *pool;
    int32_t n_out;
    int device;
};

namespace bpe {

constexpr int kTokPerThread = 4;
constexpr int kTileTokens = kGroupThreads * kTokPerThread;
constexpr int kStageBytes = 16384;            // a tile whose bytes fit is assembled in LDS
constexpr int64_t kMaxTokenBytes = 1 << 20;   // longest expansion a vocabulary may hold
constexpr int64_t kMaxPoolBytes = 1ll << 30;

// What a token stands for, as one 16-byte word: x = length in bytes (0 = id not in use); the bytes
// themselves in y, z, w if they are at most kInlineBytes, else y = their offset in the pool (a
// multiple of 4).  Word-like tokens (up to 12 bytes) are one gather instead of an {offset, length}
// and, after it, one of the pool per four bytes: a gather of 64 unrelated lines costs the texture
// path 64 line look-ups whatever its width.  2.1 M tokens (13.5 MB): 24.0 us with the two gathers,
// 22.5 with the records (and the assembly moved in front of the look-back).
constexpr uint32_t kInlineBytes = 12;

struct DecodeParams {
    const Record *tok;               // [n_tok] records of the ids as the caller numbers them
    const uint8_t *pool;
    int32_t n_tok;
    const int32_t *ids;
    int32_t n_tokens;
    const int32_t *n_tokens_dev;    // or nullptr
    uint8_t *out;
    int32_t out_capacity;
    int32_t *token_byte_offsets;    // [n_tokens + 1] or nullptr
    int32_t *n_bytes;               // [1] or nullptr
    unsigned long long *tile_state;
    int32_t *status;
    int32_t call_id;
};

__device__ inline int token_count(const DecodeParams &p) {
    return p.n_tokens_dev ? min(max(__builtin_amdgcn_readfirstlane(*p.n_tokens_dev), 0), p.n_tokens) : p.n_tokens;
}

// Ids come in and the byte offsets of the tokens go out as 16-byte words
// (at 4-byte alignment, which is all the caller promises and all the hardware asks for).
typedef int32_t Int4 __attribute__((ext_vector_type(4), aligned(4)));
static_assert(kTokPerThread == 4, "a thread's tokens are one Int4");

// The records of the thread's four tokens from t0 on; returns whether one of the ids is unknown.
__device__ __forceinline__ bool load_records(const DecodeParams &p, int t0, int n, Record (&rec)[kTokPerThread]) {
    Int4 id;
    if (t0 <= n - kTokPerThread) {             // (t0 + 4 may be 2^31)
        id = *(const Int4 *)(p.ids + t0);
    } else {
#pragma unroll
        for (int j = 0; j < kTokPerThread; ++j) id[j] = t0 + j < n ? p.ids[t0 + j] : -1;
    }
    bool bad = false;
#pragma unroll
    for (int j = 0; j < kTokPerThread; ++j) {
        rec[j] = Record{0, 0, 0, 0};
        if (id[j] >= 0 && id[j] < p.n_tok) rec[j] = p.tok[id[j]];
        bad |= rec[j].x == 0 && t0 + j < n;        // no token is empty: the id is not in the vocabulary
    }
    return bad;
}

// The bytes of a token at sb, which may have any alignment (LDS stores may, too).
__device__ __forceinline__ void put_token(const uint32_t *pool_w, uint8_t *sb, const Record &rec) {
    const uint32_t l = rec.x, w0 = rec.y, w1 = rec.z, w2 = rec.w;
    if (l <= kInlineBytes) {
        uint32_t tail = w0, at = l & ~3u;
        if (l >= 4) { __builtin_memcpy(sb, &w0, 4); tail = w1; }
        if (l >= 8) { __builtin_memcpy(sb + 4, &w1, 4); tail = w2; }
        if (l >= 12) __builtin_memcpy(sb + 8, &w2, 4);
        if (l & 2u) {
            const uint16_t half = (uint16_t)tail;
            __builtin_memcpy(sb + at, &half, 2);
            tail >>= 16;
            at += 2;
        }
        if (l & 1u) sb[at] = (uint8_t)tail;
    } else {
        const uint32_t full = l & ~3u;
        for (uint32_t k = 0; k < full; k += 4) {
            const uint32_t w = pool_w[(w0 + k) >> 2];
            __builtin_memcpy(sb + k, &w, 4);
        }
        if (l & 3u) {
            const uint32_t w = pool_w[(w0 + full) >> 2];
            for (uint32_t q = 0; q < (l & 3u); ++q) sb[full + q] = (uint8_t)(w >> (8 * q));
        }
    }
}

// The n bytes at stage + 1 word to dst: whole aligned words, put together from two words of the
// stage, and the first and the last one byte by byte.  (stage[0] and the word behind the n bytes
// exist and hold anything.)
__device__ __forceinline__ void store_stage(const uint32_t *stage, uint8_t *dst, int n) {
    const int m = (int)((uintptr_t)dst & 3);       // word d of the output starts at byte 4 d - m
    const int n_words = (m + n + 3) >> 2;
    uint32_t *dst_w = (uint32_t *)(dst - m);
    const uint32_t *src = stage + (m ? 0 : 1);
    const uint32_t shift = (4 - m) & 3;
    for (int d = threadIdx.x; d < n_words; d += kGroupThreads) {
        const uint32_t w = __builtin_amdgcn_alignbyte(src[d + 1], src[d], shift);
        const int lo = d == 0 ? m : 0, hi = min(4, m + n - 4 * d);
        if (lo == 0 && hi == 4) {
            dst_w[d] = w;
        } else {
            for (int q = lo; q < hi; ++q) ((uint8_t *)(dst_w + d))[q] = (uint8_t)(w >> (8 * q));
        }
    }
}

// A tile is ROUNDS x 1024 tokens: thread t owns tokens r * 1024 + 4 t .. + 3 of the
// tile for r = 0 .. ROUNDS - 1.  The bytes before the tile are found once per tile
// (every tile polls the state words of WINDOW others, so deep grids want few, large
// tiles).  The tile's bytes are assembled in LDS between the publication of its total
// and the look-back, while the tiles before it finish theirs; only their alignment in
// the output is not known by then, and store_stage makes up for it.
template <int ROUNDS, int WINDOW>
__global__ void __launch_bounds__(kGroupThreads) decode_kernel(DecodeParams p) {
    constexpr int kTile = ROUNDS * kTileTokens;
    // Two rounds: 12 bytes per token, and six workgroups per compute unit.  (With 32 KiB it is four, 1,024 on
    // the chip, and the 1,031 tiles of 2.1 M tokens run a second, nearly empty time: 22.6 against 19.5 us.)
    constexpr int kTileStage = ROUNDS == 1 ? kStageBytes : ROUNDS == 2 ? 24576 : 2 * kStageBytes;
    __shared__ LookbackTmp lb;
    __shared__ int wave_total[ROUNDS][kWavesPerGroup];
    __shared__ uint32_t stage[kTileStage / 4 + 3];
    uint8_t *const staged = (uint8_t *)(stage + 1);
    const uint32_t *pool_w = (const uint32_t *)p.pool;       // every expansion starts at a multiple of 4
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wv = tid / kWave;
    const int tile = blockIdx.x;
    const int n = token_count(p);
    const int n_tiles = max((int)(((uint32_t)n + (kTile - 1)) / kTile), 1);     // (n may be 2^31 - 2)
    if (tile >= n_tiles) return;               // the grid was sized for the host's upper bound
    if (tile == 0 && tid == 0) mark_call(p.status, p.call_id);
    const int32_t epoch = p.status[kStatusEpochDecode];

    const int first = tile * kTile + tid * kTokPerThread;
    uint32_t len[ROUNDS][kTokPerThread];
    int ex[ROUNDS];                            // bytes of the tile before this thread's tokens of a round
    int round_total[ROUNDS], total = 0;
    int n_staged = 0, staged_bytes = 0;
    bool fits;                                 // the whole tile does
    {
        Record rec[ROUNDS][kTokPerThread];
        bool bad = false;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) bad |= load_records(p, first + r * kTileTokens, n, rec[r]);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            int mine = 0;
#pragma unroll
            for (int j = 0; j < kTokPerThread; ++j) mine += (int)(len[r][j] = rec[r][j].x);
            const int inc = wave_scan_inclusive(mine);
            if (lane == kWave - 1) wave_total[r][wv] = inc;
            ex[r] = inc - mine;
        }
        if (__ballot(bad) && lane == 0)
            __hip_atomic_store(&p.status[kStatusBadInput], p.call_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            round_total[r] = 0;
            ex[r] += total;
#pragma unroll
            for (int w = 0; w < kWavesPerGroup; ++w) {
                if (w < wv) ex[r] += wave_total[r][w];
                round_total[r] += wave_total[r][w];
            }
            total += round_total[r];
        }
        if (tid == 0) publish_tile_total(p.tile_state, p.call_id, epoch, tile, total);
        // As many rounds as the stage holds, from the first one on.  (A token has at most 2^20 bytes and a round 2^10
        // tokens: the total of a round cannot wrap, that of four rounds of nothing but such tokens could.)
        fits = total >= 0 && total <= kTileStage;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) fits &= round_total[r] <= kTileStage;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (ROUNDS == 1 ? !fits : (n_staged < r || round_total[r] > kTileStage - staged_bytes)) continue;
            n_staged = r + 1;
            staged_bytes += round_total[r];
            int at = ex[r];
#pragma unroll
            for (int j = 0; j < kTokPerThread; ++j) {
                put_token(pool_w, staged + at, rec[r][j]);
                at += (int)len[r][j];
            }
        }
    }
    const uint32_t base = (uint32_t)__builtin_amdgcn_readfirstlane(
        total_before_tile<1, WINDOW, kWavesPerGroup, true>(p.tile_state, p.status, p.call_id, p.status + kStatusEpochDecode,
                                                           epoch, tile, n_tiles, total, lb));
    const int64_t end = (int64_t)base + (uint32_t)total;
    if ((base > (uint32_t)p.out_capacity || end > p.out_capacity) && tid == 0)
        __hip_atomic_store(&p.status[kStatusOverflow], p.call_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tile == n_tiles - 1 && tid == 0) {
        if (p.token_byte_offsets) p.token_byte_offsets[n] = (int)end;
        if (p.n_bytes) *p.n_bytes = (int)min(end, (int64_t)p.out_capacity);
    }
    if (p.token_byte_offsets) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const int t0 = first + r * kTileTokens;
            Int4 at;
            at[0] = (int)base + ex[r];
#pragma unroll
            for (int j = 1; j < kTokPerThread; ++j) at[j] = at[j - 1] + (int)len[r][j - 1];
            if (t0 <= n - kTokPerThread) {
                *(Int4 *)(p.token_byte_offsets + t0) = at;
            } else {
#pragma unroll
                for (int j = 0; j < kTokPerThread; ++j)
                    if (t0 + j < n) p.token_byte_offsets[t0 + j] = at[j];
            }
        }
    }

    if (fits && end <= p.out_capacity) {
        __syncthreads();                       // (tile 0 has passed no barrier since the stage was written)
        store_stage(stage, p.out + base, total);
        return;
    }
    // Longer tokens than the stage holds, or an output that is too small: the other rounds one by one,
    // through the stage if a round fits both.  Their records are read again: kept, they would cost the
    // common path its registers.  (Tokens of 12 to 16 bytes, 2 M of them: 27.4 us before there was a stage for
    // more than one round, 28.6 when no round of a tile that does not fit was staged ahead, 25.3 now.)
    if (fits || (int64_t)base + staged_bytes > p.out_capacity) n_staged = staged_bytes = 0;
    if (ROUNDS > 1 && n_staged > 0) {
        __syncthreads();
        store_stage(stage, p.out + base, staged_bytes);
    }
    int64_t round_base = (int64_t)base + staged_bytes;
    for (int r = ROUNDS > 1 ? n_staged : 0; r < ROUNDS; ++r) {
        Record rec[kTokPerThread];
        (void)load_records(p, first + r * kTileTokens, n, rec);
        int before = 0, rt = 0;                // as ex[r] and round_total[r], which are indexed by constants only
        {
            int mine = 0;
#pragma unroll
            for (int j = 0; j < kTokPerThread; ++j) mine += (int)rec[j].x;
            before = wave_scan_inclusive(mine) - mine;
            for (int w = 0; w < kWavesPerGroup; ++w) {
                if (w < wv) before += wave_total[r][w];
                rt += wave_total[r][w];
            }
        }
        if (round_base + (uint32_t)rt <= p.out_capacity && (uint32_t)rt <= (uint32_t)kTileStage) {
            __syncthreads();                   // the stage is free
            int at = before;
#pragma unroll
            for (int j = 0; j < kTokPerThread; ++j) {
                put_token(pool_w, staged + at, rec[j]);
                at += (int)rec[j].x;
            }
            __syncthreads();
            store_stage(stage, p.out + round_base, rt);
        } else {
            // bytes straight to the output, a wavefront sharing every token of more than 64 bytes
            int64_t at = round_base + before;
#pragma unroll
            for (int j = 0; j < kTokPerThread; ++j) {
                const uint32_t l = rec[j].x, o = rec[j].y, w1 = rec[j].z, w2 = rec[j].w;
                const bool is_long = l > 64;
                if (!is_long) {
                    for (uint32_t k = 0; k < l; ++k) {
                        const uint32_t w = l > kInlineBytes ? pool_w[(o + k) >> 2] : k < 4 ? o : k < 8 ? w1 : w2;
                        if (at + k < p.out_capacity) p.out[at + k] = (uint8_t)(w >> (8 * (k & 3)));
                    }
                }
                for (uint64_t lm = __ballot(is_long); lm;) {
                    const int src_lane = __builtin_ctzll(lm);
                    lm &= lm - 1;
                    const uint32_t so = (uint32_t)__builtin_amdgcn_readlane((int)o, src_lane);
                    const uint32_t sl = (uint32_t)__builtin_amdgcn_readlane((int)l, src_lane);
                    const int64_t a = ((int64_t)(uint32_t)__builtin_amdgcn_readlane((int)(at >> 32), src_lane) << 32) |
                                      (uint32_t)__builtin_amdgcn_readlane((int)at, src_lane);
                    for (uint32_t k = lane; k < sl; k += kWave)
                        if (a + k < p.out_capacity) p.out[a + k] = p.pool[so + k];
                }
                at += l;
            }
        }
        round_base += (uint32_t)rt;
    }
}

struct MapParams {
    const int32_t *table;   // out_of or int_of
    int32_t n_table;
    const int32_t *in;
    int32_t *out;
    int64_t n;
    const int32_t *n_dev;
};

__global__ void __launch_bounds__(kGroupThreads) map_ids_kernel(MapParams p) {
    int64_t n = p.n;
    if (p.n_dev) n = min<int64_t>(max(*p.n_dev, 0), n);
    const int64_t i = (int64_t)blockIdx.x * kGroupThreads + threadIdx.x;
    if (i >= n) return;
    const int id = p.in[i];
    p.out[i] = id >= 0 && id < p.n_table ? p.table[id] : -1;
}

// ---------------------------------------------------------------------------
// Whole batches between pinned host memory and the device (bpe_batch_in, bpe_batch_ids_out, bpe_batch_bytes_out).  A copy
// command to or from the host takes 10 us and more beside the kernels of the same stream whatever its size (it runs on another
// queue), and one that brings results back has to know how many there are; these kernels take the number from the device, read and write the host's
// memory in place, 16 bytes per lane, and are bound by the bus on large batches.  Through Tokenizer, copy commands / now: one text of 1.5 KB, renumbered
// 62.0 / 35.5 us, 840 KB in 48 texts 170 / 125 (40 of it packing and unpacking on the host), back to 210 KB in 48 texts 155 / 71, to 500
// bytes 100 / 31, 13.5 MB in 200 texts 2,003 / 1,357.
constexpr int64_t kBatchGrid = 512;            // workgroups: 128 k lanes, enough in flight for the bus

// The largest clock value at which a workgroup of bpe_batch_in was done is left in *clock: it only grows, so nothing resets it.
__global__ void __launch_bounds__(kGroupThreads) batch_in_kernel(const uint4 *src, uint4 *dst, int64_t n, unsigned long long *clock) {
    for (int64_t i = (int64_t)blockIdx.x * kGroupThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kGroupThreads) dst[i] = src[i];
    __syncthreads();
    if (threadIdx.x == 0) atomicMax(clock, (unsigned long long)wall_clock64());
}

struct BatchOut {
    const int32_t *status;         // of the workspace
    const unsigned long long *clock;
    int32_t *host;                 // [9] status words, ticks from *clock to the start of this kernel
};
__device__ __forceinline__ void batch_head(const BatchOut &b, unsigned long long start) {
    if (blockIdx.x != 0) return;
    if (threadIdx.x < 8) b.host[threadIdx.x] = b.status[threadIdx.x];
    if (threadIdx.x == 8) b.host[8] = (int32_t)(start - *b.clock);
}

// words: n_offsets offsets, then as many ids as the last of them says; ids go through table unless it is nullptr.
__global__ void __launch_bounds__(kGroupThreads) batch_ids_out_kernel(BatchOut b, const int32_t *words, int64_t n_offsets, int64_t max_ids,
                                                                      const int32_t *table, int32_t n_table, int32_t *host) {
    const unsigned long long start = wall_clock64();
    const int64_t n = n_offsets + min<int64_t>(max(words[n_offsets - 1], 0), max_ids);
    for (int64_t i = 4 * ((int64_t)blockIdx.x * kGroupThreads + threadIdx.x); i < n; i += 4 * (int64_t)gridDim.x * kGroupThreads) {
        const int4 v = *(const int4 *)(words + i);
        int id[4] = {v.x, v.y, v.z, v.w};
        if (table) {
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i + k >= n_offsets && i + k < n) id[k] = id[k] >= 0 && id[k] < n_table ? table[id[k]] : -1;
        }
        *(int4 *)(host + i) = make_int4(id[0], id[1], id[2], id[3]);
    }
    batch_head(b, start);
}

// starts[k] = at[bounds[k]]; then the first at[n_tokens] bytes, at most capacity of them; none that the decoder had to cut off
// (its caller decodes again with more room: 200,000 tokens of 32 bytes through Tokenizer 1,145 us with the cut bytes, 1,110 without).
__global__ void __launch_bounds__(kGroupThreads) batch_bytes_out_kernel(BatchOut b, const uint4 *bytes, int64_t capacity, const int32_t *at,
                                                                        int64_t n_tokens, const int32_t *bounds, int64_t n_bounds,
                                                                        int32_t *starts, uint4 *host) {
    const unsigned long long start = wall_clock64();
    const int64_t first = (int64_t)blockIdx.x * kGroupThreads + threadIdx.x, step = (int64_t)gridDim.x * kGroupThreads;
    for (int64_t k = first; k < n_bounds; k += step) starts[k] = at[bounds[k]];
    const bool cut = b.status[kStatusCallCheck] == (b.status[kStatusCall] ^ kCallCheck) && b.status[kStatusOverflow] == b.status[kStatusCall];
    const int64_t n = cut ? 0 : min<int64_t>(max(at[n_tokens], 0), capacity);
    for (int64_t i = first; 16 * i < n; i += step) host[i] = bytes[i];
    batch_head(b, start);
}

static int64_t batch_grid(int64_t n16) { return std::min(std::max<int64_t>((n16 + kGroupThreads - 1) / kGroupThreads, 1), kBatchGrid); }

static int64_t align256v(int64_t v) { return (v + 255) & ~255ll; }

}  // namespace bpe

using namespace bpe;

extern "C" int bpe_vocab_build(const int32_t *merges, const int32_t *ranks, const int32_t *merged_ids, int64_t n,
                               const int32_t *output_ids, int64_t n_output_ids, bpe_vocab **out_vocab) {
    if (!out_vocab) { set_error("out_vocab is NULL"); return BPE_ERR_NULL; }
    *out_vocab = nullptr;
    RuleOrder ro;
    int rc = order_rules(merges, ranks, merged_ids, n, ro);
    if (rc != BPE_OK) return rc;
    const int64_t n_ids = ro.max_id + 1;
    if (output_ids && n_output_ids != n_ids) {
        set_error("output_ids must have one entry per id up to the largest (%lld), got %lld", (long long)n_ids,
                  (long long)n_output_ids);
        return BPE_ERR_SIZE;
    }
    // expansions in rank order: both parts of a rule are bytes or made by earlier rules
    std::vector<uint32_t> tok_off((size_t)n_ids, 0), tok_len((size_t)n_ids, 0);
    std::vector<uint8_t> pool((size_t)256 * 4, 0);
    for (int b = 0; b < 256; ++b) { tok_off[b] = 4 * b; tok_len[b] = 1; pool[4 * b] = (uint8_t)b; }
    int64_t longest = 1;
    for (int64_t k = 0; k < n; ++k) {
        const int64_t i = ro.by_rank[k].second;
        const int64_t a = merges[2 * i], b = merges[2 * i + 1], m = ro.merged_row[i];
        const int64_t len = (int64_t)tok_len[a] + tok_len[b];
        if (len > kMaxTokenBytes || (int64_t)pool.size() + len + 4 > kMaxPoolBytes) {
            set_error("the expansions of this table are too long to keep (token of %lld bytes, pool of %lld)",
                      (long long)len, (long long)pool.size());
            return BPE_ERR_SIZE;
        }
        const size_t at = pool.size();
        pool.resize(at + (size_t)((len + 3) & ~3ll), 0);
        memcpy(pool.data() + at, pool.data() + tok_off[a], tok_len[a]);
        memcpy(pool.data() + at + tok_len[a], pool.data() + tok_off[b], tok_len[b]);
        tok_off[m] = (uint32_t)at;
        tok_len[m] = (uint32_t)len;
        longest = std::max(longest, len);
    }
    // renumbering: unique output ids in [0, 2^24) for the ids in use
    std::vector<int32_t> out_of, int_of;
    if (output_ids) {
        int64_t max_out = -1;
        for (int64_t id = 0; id < n_ids; ++id) {
            if (tok_len[id] == 0) continue;
            const int64_t o = output_ids[id];
            if (o < 0 || o >= (1ll << kIdBits)) { set_error("output id %lld of id %lld is outside [0, 2^24)", (long long)o, (long long)id); return BPE_ERR_ID_RANGE; }
            max_out = std::max(max_out, o);
        }
        out_of.assign((size_t)n_ids, -1);
        int_of.assign((size_t)(max_out + 1), -1);
        for (int64_t id = 0; id < n_ids; ++id) {
            if (tok_len[id] == 0) continue;
            const int32_t o = output_ids[id];
            if (int_of[o] != -1) { set_error("output id %d is given to ids %d and %lld", o, int_of[o], (long long)id); return BPE_ERR_DUP_MERGED; }
            int_of[o] = (int32_t)id;
            out_of[id] = o;
        }
    }
    auto token_record = [&](int64_t id) {
        Record t = Record{tok_len[id], 0, 0, 0};
        if (t.x > kInlineBytes) t.y = tok_off[id];
        else memcpy((char *)&t + 4, pool.data() + tok_off[id], t.x);
        return t;
    };
    const int64_t b_tok = 0, b_tokout = b_tok + align256v(16 * n_ids),
                  b_outof = b_tokout + align256v(16 * (int64_t)int_of.size()),
                  b_intof = b_outof + align256v(4 * (int64_t)out_of.size()),
                  b_pool = b_intof + align256v(4 * (int64_t)int_of.size()),
                  b_total = b_pool + align256v((int64_t)pool.size());
    std::vector<char> blob((size_t)b_total, 0);
    Record *tok = (Record *)(blob.data() + b_tok), *tok_out = (Record *)(blob.data() + b_tokout);
    for (int64_t id = 0; id < n_ids; ++id) tok[id] = token_record(id);
    for (size_t o = 0; o < int_of.size(); ++o)
        if (int_of[o] >= 0) tok_out[o] = token_record(int_of[o]);
    if (!out_of.empty()) memcpy(blob.data() + b_outof, out_of.data(), out_of.size() * 4);
    if (!int_of.empty()) memcpy(blob.data() + b_intof, int_of.data(), int_of.size() * 4);
    memcpy(blob.data() + b_pool, pool.data(), pool.size());

    bpe_vocab *v = new (std::nothrow) bpe_vocab();
    if (!v) { set_error("out of host memory"); return BPE_ERR_SIZE; }
    hipError_t e = hipGetDevice(&v->device);
    if (e != hipSuccess) { delete v; return hip_fail(e, "hipGetDevice"); }
    e = hipMalloc(&v->device_mem, blob.size());
    if (e != hipSuccess) { delete v; return hip_fail(e, "hipMalloc(vocab)"); }
    e = hipMemcpy(v->device_mem, blob.data(), blob.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) { (void)hipFree(v->device_mem); delete v; return hip_fail(e, "hipMemcpy(vocab)"); }
    char *d = (char *)v->device_mem;
    v->tok = (const Record *)(d + b_tok);
    v->tok_out = int_of.empty() ? nullptr : (const Record *)(d + b_tokout);
    v->out_of = out_of.empty() ? nullptr : (const int32_t *)(d + b_outof);
    v->int_of = int_of.empty() ? nullptr : (const int32_t *)(d + b_intof);
    v->pool = (const uint8_t *)(d + b_pool);
    v->n_out = (int32_t)int_of.size();
    v->info.n_ids = n_ids;
    v->info.n_output_ids = (int64_t)int_of.size();
    v->info.pool_bytes = (int64_t)pool.size();
    v->info.device_bytes = b_total;
    v->info.max_token_bytes = (int32_t)longest;
    for (int64_t id = 0; id < n_ids; ++id) v->token_bytes += tok_len[id];
    v->info.has_output_ids = output_ids ? 1 : 0;
    *out_vocab = v;
    return BPE_OK;
}

extern "C" int bpe_vocab_free(bpe_vocab *v) {
    if (!v) return BPE_OK;
    hipError_t e = hipFree(v->device_mem);
    delete v;
    return e == hipSuccess ? BPE_OK : hip_fail(e, "hipFree(vocab)");
}

extern "C" int bpe_vocab_info(const bpe_vocab *v, bpe_vocab_info_t *info) {
    if (!v || !info) { set_error("null pointer"); return BPE_ERR_NULL; }
    *info = v->info;
    return BPE_OK;
}

extern "C" int bpe_host_visible(const void *host) {
    void *d = nullptr;
    if (host && hipHostGetDevicePointer(&d, const_cast<void *>(host), 0) == hipSuccess && d == host) return 1;
    (void)hipGetLastError();
    return 0;
}

extern "C" int bpe_batch_in(const void *host, void *device, int64_t n_bytes, void *clock, void *stream) {
    if (!host || !device || !clock) { set_error("null pointer"); return BPE_ERR_NULL; }
    if (n_bytes < 0 || ((uintptr_t)host & 15) || ((uintptr_t)device & 15) || ((uintptr_t)clock & 7)) {
        set_error("n_bytes is negative, or a buffer is not 16-byte aligned");
        return BPE_ERR_SIZE;
    }
    const int64_t n16 = (n_bytes + 15) / 16;
    hipLaunchKernelGGL(batch_in_kernel, dim3((unsigned)batch_grid(n16)), dim3(kGroupThreads), 0, (hipStream_t)stream,
                       (const uint4 *)host, (uint4 *)device, n16, (unsigned long long *)clock);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? BPE_OK : hip_fail(e, "bpe_batch_in launch");
}

extern "C" int bpe_batch_ids_out(const bpe_vocab *v, const int32_t *words, int64_t n_offsets, int64_t max_ids, int32_t *host,
                                 const void *workspace, const void *clock, int32_t *host_head, void *stream) {
    if (!words || !host || !workspace || !clock || !host_head) { set_error("null pointer"); return BPE_ERR_NULL; }
    if (n_offsets < 1 || max_ids < 0 || ((uintptr_t)words & 15) || ((uintptr_t)host & 15)) {
        set_error("sizes out of range, or a buffer is not 16-byte aligned");
        return BPE_ERR_SIZE;
    }
    if (v) {
        if (!v->out_of) { set_error("the vocabulary was built without output ids"); return BPE_ERR_OPTION; }
        const int dev_rc = check_device(v->device, "the vocabulary");
        if (dev_rc != BPE_OK) return dev_rc;
    }
    const BatchOut b = {(const int32_t *)workspace, (const unsigned long long *)clock, host_head};
    hipLaunchKernelGGL(batch_ids_out_kernel, dim3((unsigned)batch_grid((n_offsets + max_ids / 4) / 4)), dim3(kGroupThreads), 0, (hipStream_t)stream,
                       b, words, n_offsets, max_ids, v ? v->out_of : nullptr, v ? (int32_t)v->info.n_ids : 0, host);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? BPE_OK : hip_fail(e, "bpe_batch_ids_out launch");
}

extern "C" int bpe_batch_bytes_out(const void *bytes, int64_t capacity, const int32_t *token_byte_offsets, int64_t n_tokens,
                                   const int32_t *bounds, int64_t n_bounds, int32_t *host_starts, void *host,
                                   const void *workspace, const void *clock, int32_t *host_head, void *stream) {
    if (!bytes || !token_byte_offsets || !bounds || !host_starts || !host || !workspace || !clock || !host_head) { set_error("null pointer"); return BPE_ERR_NULL; }
    if (capacity < 0 || n_tokens < 0 || n_bounds < 0 || ((uintptr_t)bytes & 15) || ((uintptr_t)host & 15)) {
        set_error("sizes out of range, or a buffer is not 16-byte aligned");
        return BPE_ERR_SIZE;
    }
    const BatchOut b = {(const int32_t *)workspace, (const unsigned long long *)clock, host_head};
    hipLaunchKernelGGL(batch_bytes_out_kernel, dim3((unsigned)batch_grid(std::max(capacity / 32, n_bounds))), dim3(kGroupThreads), 0,
                       (hipStream_t)stream, b, (const uint4 *)bytes, capacity, token_byte_offsets, n_tokens, bounds, n_bounds, host_starts, (uint4 *)host);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? BPE_OK : hip_fail(e, "bpe_batch_bytes_out launch");
}

extern "C" int bpe_map_ids(const bpe_vocab *v, const int32_t *ids_in, int32_t *ids_out, int64_t n,
                           const int32_t *n_device, int to_output_ids, void *stream) {
    if (!v || (n > 0 && (!ids_in || !ids_out))) { set_error("null pointer"); return BPE_ERR_NULL; }
    if (n < 0 || n >= 0x7FFFFFFFll * kGroupThreads) { set_error("n out of range"); return BPE_ERR_SIZE; }
    if (!v->out_of) { set_error("the vocabulary was built without output ids"); return BPE_ERR_OPTION; }
    if (n == 0) return BPE_OK;
    const int dev_rc = check_device(v->device, "the vocabulary");
    if (dev_rc != BPE_OK) return dev_rc;
    MapParams p = {};
    p.table = to_output_ids ? v->out_of : v->int_of;
    p.n_table = to_output_ids ? (int32_t)v->info.n_ids : v->n_out;
    p.in = ids_in;
    p.out = ids_out;
    p.n = n;
    p.n_dev = n_device;
    hipLaunchKernelGGL(map_ids_kernel, dim3((unsigned)((n + kGroupThreads - 1) / kGroupThreads)), dim3(kGroupThreads),
                       0, (hipStream_t)stream, p);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? BPE_OK : hip_fail(e, "bpe_map_ids launch");
}

extern "C" int64_t bpe_decode_workspace_bytes(int64_t n_tokens) {
    if (n_tokens < 0 || n_tokens >= 0x7FFFFFFFll) { set_error("n_tokens out of range (%lld)", (long long)n_tokens); return BPE_ERR_SIZE; }
    const int64_t n_tiles = std::max<int64_t>((n_tokens + kTileTokens - 1) / kTileTokens, 1);
    return 256 + align256v(8 * n_tiles);
}

extern "C" int bpe_decode(const bpe_vocab *v, const int32_t *ids, int64_t n_tokens, const int32_t *n_tokens_device,
                          int ids_are_output_ids, uint8_t *out_bytes, int64_t out_capacity,
                          int32_t *token_byte_offsets, int32_t *n_bytes, void *workspace, int64_t workspace_bytes,
                          void *stream) {
    if (!v || (n_tokens > 0 && !ids) || (out_capacity > 0 && !out_bytes)) { set_error("null pointer"); return BPE_ERR_NULL; }
    if (out_capacity < 0 || out_capacity >= 0x7FFFFFFFll) { set_error("out_capacity out of range (%lld)", (long long)out_capacity); return BPE_ERR_SIZE; }
    const int64_t need = bpe_decode_workspace_bytes(n_tokens);
    if (need < 0) return (int)need;
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < need) {
        set_error("workspace must be 256-byte aligned and hold %lld bytes (got %lld)", (long long)need,
                  (long long)workspace_bytes);
        return BPE_ERR_WORKSPACE;
    }
    if (ids_are_output_ids && !v->int_of) { set_error("the vocabulary was built without output ids"); return BPE_ERR_OPTION; }
    const int dev_rc = check_device(v->device, "the vocabulary");
    if (dev_rc != BPE_OK) return dev_rc;
    DecodeParams p = {};
    p.tok = ids_are_output_ids ? v->tok_out : v->tok;
    p.n_tok = ids_are_output_ids ? v->n_out : (int32_t)v->info.n_ids;
    p.pool = v->pool;
    p.ids = ids;
    p.n_tokens = (int32_t)n_tokens;
    p.n_tokens_dev = n_tokens_device;
    p.out = out_bytes;
    p.out_capacity = (int32_t)out_capacity;
    p.token_byte_offsets = token_byte_offsets;
    p.n_bytes = n_bytes;
    p.status = (int32_t *)workspace;
    p.tile_state = (unsigned long long *)((char *)workspace + 256);
    p.call_id = next_call_id();
    // Deep grids want fewer, larger tiles and a narrow look-back (every state word of
    // another workgroup is an uncached read), but the registers of a round cost
    // occupancy.  us for 0.5 / 1 / 2.1 / 4.1 / 8 / 40 M tokens of text (rounds, tiles looked at per round):
    //   (1, 256)  9.5  13.1  22.2  39.9  81  431      (1, 32) 11.3  15.5  22.9  41.0  72  340
    //   (2, 64)  10.0  13.6  19.1  33.4  55  269      (2, 256) 8.9  12.5  17.6  31.2  54  293
    //   (4, 32)  13.0  14.7  20.7  30.3  50  238      (4, 256) 11.3 12.4  19.1  28.3  49  264
    // Up to 0.5 M tokens the call's launch hides the difference, but tokens of more than 12 bytes do not fit the stage of two
    // rounds (0.3 to 0.5 M of 13 to 16 bytes: 9.9 to 10.6 us with one round, 13.2 to 13.6 with two).
    // Beyond, it depends on where the records lie: where tiles wait for them, they come to their look-back at different times,
    // and the polls of a full window cost more than they save.  (2, 64), (2, 128) and (2, 256):
    //   2 M tokens    50k table: text 18.3, 18.0, 17.2, with random bytes 14.1, 13.4, 12.9, random ids 19.9, 19.5, 18.9, random ids
    //                 of up to 6 bytes 19.1, 19.4, 21.2; 1k table: text 13.4, 12.6, 11.7, random ids 14.2, 13.6, 12.7
    //   2.5 M         50k table: 20.1, 19.4, 19.1; 15.3, 15.1, 14.7; 24.6, 25.3, 29.4; 23.3, 23.9, 26.9; 1k: 13.6, 13.4, 13.2; 16.5, 15.8, 15.5
    // (2, 64), (4, 32), (4, 64) and (4, 256), text, random bytes, random ids:
    //   3.5 M         50k table: 28.5, 27.0, 25.8, 26.2; 21.8, 19.4, 18.4, 19.3; 32.8, 29.8, 30.3, 31.4; 100k table, whose mean token does not
    //                 fit the 8 bytes that four rounds stage: 28.3, 27.1, 26.1, 25.9; 45.1, 52.9, 52.9, 54.3; 92.5, 113, 113, 113;
    //                 1k table: 19.0, 17.7, 16.5, 15.7; 17.7, 16.2, 15.1, 14.3; 21.7, 20.0, 19.4, 18.7
    //   6 M           50k table: 42.3, 40.6, 40.3, 39.4; 32.8, 31.3, 30.9, 32.1; 50.9, 45.2, 45.5, 46.7; 1k table: 26.9, 26.4, 25.7, 24.9
    // So a full window while a compute unit's cache holds the records (of up to 2,048 ids), and for others up to 2.3 M
    // tokens, 128 tiles up to 3 M, 64 up to 4 M.  With an output numbering records lie anywhere (text with random
    // bytes, 2 and 2.5 M tokens of the 50k table 15.5, 17.8, 18.2 and 17.4, 20.4, 21.1): (2, 64) there up to 4 M tokens, (4, 32) beyond.
    const dim3 block(kGroupThreads);
    auto tiles = [&](int rounds) { return (unsigned)std::max<int64_t>((n_tokens + rounds * kTileTokens - 1) / (rounds * kTileTokens), 1); };
    const hipStream_t st = (hipStream_t)stream;
    const int64_t n_tiles = (n_tokens + kTileTokens - 1) / kTileTokens;
    const bool near = v->info.n_ids <= 2048, long_tokens = v->token_bytes > 8 * v->info.n_ids;
#define LAUNCH_DECODE(ROUNDS, WINDOW) hipLaunchKernelGGL((decode_kernel<ROUNDS, WINDOW>), dim3(tiles(ROUNDS)), block, 0, st, p)
    if (n_tiles <= 512) LAUNCH_DECODE(1, kGroupThreads);
    else if (ids_are_output_ids && n_tiles <= 4096) LAUNCH_DECODE(2, 64);
    else if (ids_are_output_ids) LAUNCH_DECODE(4, 32);
    else if (n_tiles <= (near ? 3072 : 2304)) LAUNCH_DECODE(2, kGroupThreads);
    else if (n_tiles <= 3072) LAUNCH_DECODE(2, 128);
    else if (near && n_tiles <= 8192) LAUNCH_DECODE(4, kGroupThreads);
    else if (n_tiles <= 4096 && long_tokens) LAUNCH_DECODE(2, 64);
    else if (n_tiles <= 4096) LAUNCH_DECODE(4, 64);
    else LAUNCH_DECODE(4, 32);
#undef LAUNCH_DECODE
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? BPE_OK : hip_fail(e, "bpe_decode launch");
}
