// bpe_encode_raw for callers that want tokens only, inputs of more bytes than merge_bytes_kernel's tiles take: no
// pre-tokenizer launch and no piece offsets through memory.  Device code, included by bpe_encode.hip behind the paths
// that merge longer pieces.
//
// A tile is 4 KiB of bytes; a workgroup takes a run of consecutive tiles, one after the other.  It reads a tile's bytes
// once, coalesced, into LDS, finds the pieces that start in it (a piece starts at byte 0, at a space and where a
// sequence starts), and every thread probes the whole-piece table for kBytePieces of them, all in flight together.
// What the probes leave over is listed over the whole run and merged once at its end (or when the list is nearly
// full): that is one chain of round trips for many tiles instead of one for each.  Pieces beyond tiny_max wait on a
// list in the workspace until then.  Between the two kernels a piece is one word in piece_word[first byte of its
// tile's first piece + its number in the tile]: its token, or where it starts and how many tokens lie in scratch.
//
// Per call, through the pre-tokenizer and one tile of 256 pieces per workgroup / now: text of known words 1.9 MB 29.6 /
// 16.0 us, 13.5 MB 95.8 / 40.0, in 256 sequences 99.6 / 42.9 (kernel trace: 16.0 + 60.1 + 4.4 + 4.2 + 16.1 + 4.3 us / 33.1 + 9.2), 64 MB 367 / 131,
// 134 MB 794 / 279; of unknown words 13.5 MB 128 / 120, 64 MB 591 / 530; with runs and random bytes (100k table) 4 MB 110 / 57, 13.5 MB
// 281 / 141; 30 MB of 3-byte pieces 201 / 81; 64 MB of runs in pieces of 1,000 bytes 341 / 289, of 40 1,302 / 1,321 (a tile of few
// pieces takes its round trips all the same).  What bounds it is those round trips: a tile takes about 3 us, a compute unit
// holds four workgroups, 2.2 wavefronts per SIMD are in flight and wait for 62 % of the time (78 % with runs and random bytes).
#pragma once

namespace bpe {

constexpr int kRunTile = 4096;                 // bytes
constexpr int kRunGroups = kRunTile / 16;      // a thread looks at 16 bytes at a time ("group")
constexpr int kRunAhead = 16;                  // groups looked at behind the tile for the end of its last piece
constexpr int kRunStaged = kRunGroups + 2;     // groups kept: the words of a short piece end 19 bytes behind the tile at most
constexpr int kBytePieces = 3;                 // pieces per thread and pass: 616 of word-like text start in a tile
constexpr int kBytePass = kBytePieces * kGroupThreads;
static_assert(kRunGroups == kGroupThreads, "a group per thread");
static_assert(kBytePass <= kRunLeft, "the list holds what a pass leaves over");

// The word of a piece that is not one token: its first byte counted from the tile's first group, and its number of
// tokens (kManyTokens: that is the next word; such a piece is the last one of its tile, and longer, so no other
// piece's word is there).
constexpr uint32_t kSeveral = 0x80000000u, kManyTokens = 0x7FFFFu;
constexpr int kStartShift = 19;

struct LongPiece { int b, n, slot, tile; };    // first byte, length, index of its word, number of its tile in the run

// Bit j set: byte j of the 16-byte group is a space.
__device__ __forceinline__ uint32_t spaces_in_group(const uint4 &x) {
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    uint32_t other[4];                                               // 1 in every byte that is no space
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t y = w[d] ^ 0x20202020u;                       // a space byte becomes 0
        other[d] = ((((y & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | y) >> 7) & 0x01010101u;
    }
    // a dot product with powers of two packs the bits of four bytes
    const uint32_t lo = __builtin_amdgcn_udot4(other[1], 0x80402010u, __builtin_amdgcn_udot4(other[0], 0x08040201u, 0u, false), false);
    const uint32_t hi = __builtin_amdgcn_udot4(other[3], 0x80402010u, __builtin_amdgcn_udot4(other[2], 0x08040201u, 0u, false), false);
    return (lo | hi << 8) ^ 0xFFFFu;
}

// First k in [a, b) with seq[k] >= x, b if there is none, by a wavefront: 64 places a round.  (seq should
// not decrease; if it does, the result is some index in [a, b].)
__device__ __forceinline__ int wave_lower_bound(const int32_t *seq, int a, int b, int x) {
    const int lane = lane_id();
    while (a < b) {
        const int step = (int)(((uint32_t)(b - a) + kWave - 1) / kWave);
        const int64_t at = (int64_t)a + (int64_t)(lane + 1) * step - 1;
        const bool below = at < b && seq[at] < x;
        const uint64_t not_below = ~__ballot(below);
        const int c = not_below ? __builtin_ctzll(not_below) : kWave;          // whole steps below x
        const int64_t next = (int64_t)a + (int64_t)c * step;
        a = (int)min(next, (int64_t)b);
        b = (int)min(next + step - 1, (int64_t)b);
    }
    return __builtin_amdgcn_readfirstlane(a);
}

struct ByteRunShared {
    MergeLds merge;                            // the list of left-over short pieces (MergeLds::run), or what merges them
    union {
        struct {
            uint4 bytes[kRunStaged];           // of the tile
            uint16_t start[kBytePass + 2];     // first byte of every piece of the pass, counted from the first group
            uint32_t group[kRunGroups];        // starts in the tile before the group << 16 | start mask
        } tile;
        struct { uint32_t entry[kGroupThreads]; LongPiece piece[kGroupThreads]; } longer;      // at the end of the run
    };
    GroupTmp tmp;
    int acc[kRunTilesMax];                     // tokens of the run's tiles
    int first[kRunTilesMax];                   // first byte of their first pieces
    int n_left;                                // short pieces on the list
    int wave_n[2][kWavesPerGroup], ahead[2], seek[kWavesPerGroup];
    int n_col, n_long;                         // pieces on the lists in the workspace: from its front, from its back
};

// Words of the workspace that a run's long-piece list may use: the first of `bytes` bytes is number `at` of the input.
// (A list entry is 16 bytes, the area has 8 per byte of the input, and such a piece has 2 bytes at the least.)
__device__ __forceinline__ LongPiece *long_list(const EncodeParams &p, int at) { return (LongPiece *)p.rec + (at >> 1); }

// Merges the n short pieces that sh.merge.run lists ({first byte, length << 16 | number in the tile}) and writes their
// words.  Every thread must call it, behind a barrier.
__device__ __forceinline__ void merge_byte_run_left(const EncodeParams &p, ByteRunShared &sh, int tile0, int n) {
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    auto finish = [&](int2 piece, int c, int first) {
        const uint32_t v = (uint32_t)(piece.x + p.tile_shift);
        const int t = (int)(v / kRunTile) - tile0;
        p.piece_word[sh.first[t] + (piece.y & 0xFFFF)] = c == 1 ? first : (int)(kSeveral | (v % kRunTile) << kStartShift | (uint32_t)c);
        atomicAdd(&sh.acc[t], c);
    };
    if (n <= row_pieces(kWavesPerGroup)) {
        constexpr int kRows = kWave / kTinyMax;
        if (wv * kRows < n) {
            const int j = lane & (kTinyMax - 1), e = wv * kRows + lane / kTinyMax;
            const bool mine = e < n;
            const int2 piece = sh.merge.run.piece[mine ? e : 0];
            uint32_t sym = ((const uint8_t *)&sh.merge.run.bytes[mine ? e : 0])[j] | (3u << 24);
            const int c = row_merge(p, sym, mine ? piece.y >> 16 : 0);
            sym &= 0xFFFFFFu;
            if (j < c) p.scratch[piece.x + j] = (int)sym;
            if (mine && j == 0) finish(piece, c, (int)sym);
        }
        return;
    }
    uint4 b[kRunRounds];
    int2 piece[kRunRounds];
#pragma unroll
    for (int r = 0; r < kRunRounds; ++r) {
        const int e = r * kGroupThreads + tid;
        piece[r] = make_int2(0, 0);
        if (e < n) { b[r] = sh.merge.run.bytes[e]; piece[r] = sh.merge.run.piece[e]; }
    }
    __syncthreads();               // the columns take the place of the list; from here on a wavefront has its own
    TinyState &L = sh.merge.tiny[wv];
#pragma unroll 1
    for (int e0 = wv * kWave; e0 < n; e0 += kGroupThreads) {
        const bool mine = piece[0].y != 0;         // (a listed piece has a length)
        const uint32_t w[4] = {b[0].x, b[0].y, b[0].z, b[0].w};
        const uint32_t alive = tiny_merge(p, L, w, piece[0].y >> 16, mine);
        tiny_store(L, alive, p.scratch + piece[0].x);
        if (mine) finish(piece[0], __builtin_popcount(alive), (int)(L.S[__builtin_ctz(alive)][lane] & 0xFFFFFFu));
#pragma unroll
        for (int r = 0; r + 1 < kRunRounds; ++r) { b[r] = b[r + 1]; piece[r] = piece[r + 1]; }
        piece[kRunRounds - 1] = make_int2(0, 0);
    }
}

__global__ void __launch_bounds__(kGroupThreads, 4) merge_byte_runs_kernel(EncodeParams p, int n_tiles) {
    __shared__ ByteRunShared sh;
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int tile0 = blockIdx.x * p.tiles_per_group, tile1 = min(tile0 + p.tiles_per_group, n_tiles);
    // Positions v are counted from the 16-byte boundary at or below the input: byte i is v = i + mis.
    const uint32_t mis = (uint32_t)p.tile_shift;
    const uint32_t v_end = p.n_bytes ? (uint32_t)p.n_bytes + mis : 0u;
    const uint4 *src = (const uint4 *)(p.bytes - mis);
    if (tid < kRunTilesMax) sh.acc[tid] = 0;
    if (tid == 0) { sh.n_left = 0; sh.n_col = 0; sh.n_long = 0; }
    // the run's bytes; its list of longer pieces lies in the workspace accordingly
    const int run_lo = (int)max((int64_t)tile0 * kRunTile - mis, (int64_t)0);
    const int run_hi = (int)min((int64_t)(tile0 + p.tiles_per_group) * kRunTile - mis, (int64_t)p.n_bytes);

    // A thread's group of a tile, and the 256 bytes behind the tile (by the first wavefront).  (A group that holds a
    // byte of the input lies in that byte's page.)
    auto load_group = [&](int tile, int g) {
        const uint32_t v = (uint32_t)tile * kRunTile + 16u * (uint32_t)g;
        uint4 x = make_uint4(0, 0, 0, 0);
        if (v < v_end) x = src[v >> 4];
        return x;
    };
    uint4 x = load_group(tile0, tid), x_ahead = make_uint4(0, 0, 0, 0);
    if (tid < kRunAhead) x_ahead = load_group(tile0, kRunGroups + tid);

    int s1 = 0;
    for (int tile = tile0; tile < tile1; ++tile) {
        const int par = tile & 1;
        const uint32_t v0 = (uint32_t)tile * kRunTile;
        const int origin = (int)(v0 - mis);                    // input index of the first group's first byte (may be -15)
        const int lo = min(max(origin, 0), p.n_bytes);         // (the last tile may be empty)
        const int hi = (int)min((int64_t)v0 + kRunTile - mis, (int64_t)p.n_bytes);

        // Sequence boundaries: every tile checks a strided share of them and finds the ones among its own bytes,
        // seq_off[s0 .. s1); seq_next: the first one at or behind the tile's end (a piece ends there at the latest).
        // (A single sequence has none inside the text: its two offsets are checked by the first tile.)
        int s0, seq_next = p.n_bytes;
        if (!p.seq_off || p.n_seqs == 1) {
            if (p.seq_off && tile == 0 && tid < 2 && p.seq_off[tid] != (tid ? p.n_bytes : 0))
                __hip_atomic_store(&p.status[kStatusBadInput], p.call_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s1 = p.n_bytes ? 1 : 0;
            s0 = tile ? s1 : 0;
        } else {
            bool bad = false;
            for (int64_t k = (int64_t)tile * kGroupThreads + tid; k <= p.n_seqs; k += (int64_t)n_tiles * kGroupThreads) {
                const int sv = p.seq_off[k];
                bad |= sv < 0 || sv > p.n_bytes || (k == 0 && sv != 0) || (k == p.n_seqs && sv != p.n_bytes);
                if (k < p.n_seqs) bad |= p.seq_off[k + 1] < sv;
            }
            if (__ballot(bad) && lane == 0)
                __hip_atomic_store(&p.status[kStatusBadInput], p.call_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s0 = tile == tile0 ? wave_lower_bound(p.seq_off, 0, p.n_seqs + 1, lo) : s1;
            const int next = p.seq_off[min((int64_t)s0 + lane, (int64_t)p.n_seqs)];        // s1 is nearly always among them
            const uint64_t below = __ballot((int64_t)s0 + lane <= p.n_seqs && next < hi);
            if (~below) {
                const int c = (int)__builtin_ctzll(~below);
                s1 = s0 + c;
                if (s1 <= p.n_seqs) seq_next = min(max(read_lane(next, c), hi), p.n_bytes);
            } else {
                s1 = wave_lower_bound(p.seq_off, s0 + kWave, p.n_seqs + 1, hi);
                if (s1 <= p.n_seqs) seq_next = min(max(__builtin_amdgcn_readfirstlane(p.seq_off[s1]), hi), p.n_bytes);
            }
        }
        const bool any_seq = s1 > s0;                          // the same in every wavefront
        if (any_seq) {
            sh.tile.group[tid] = 0;
            __syncthreads();
            for (int64_t k = (int64_t)s0 + tid; k < s1; k += kGroupThreads) {
                const int sv = p.seq_off ? p.seq_off[k] : 0;
                if (sv < lo || sv >= hi) continue;
                const uint32_t at = (uint32_t)sv + mis - v0;
                atomicOr(&sh.tile.group[at >> 4], 1u << (at & 15));
            }
            __syncthreads();
        }

        // Start masks; starts behind the tile only say where its last piece ends.
        const uint32_t v = v0 + 16u * (uint32_t)tid;           // position of the thread's group
        auto below = [&](uint32_t v, uint32_t limit) { return limit <= v ? 0u : limit - v >= 16u ? 0xFFFFu : (1u << (limit - v)) - 1u; };
        uint32_t mask = spaces_in_group(x);
        if (any_seq) mask |= sh.tile.group[tid];
        if (tile == 0 && tid == 0) mask |= 1u << mis;          // byte 0 starts a piece
        if (tile == 0 || hi == p.n_bytes) mask &= below(v, (uint32_t)hi + mis) & ~below(v, (uint32_t)lo + mis);
        sh.tile.bytes[tid] = x;
        if (tid < kRunStaged - kRunGroups) sh.tile.bytes[kRunGroups + tid] = x_ahead;
        if (wv == 0) {
            const uint32_t va = v + kRunTile;
            const uint32_t m = tid < kRunAhead ? spaces_in_group(x_ahead) & below(va, v_end) : 0u;
            const uint64_t hit = __ballot(m != 0);
            int at = 0x7FFFFFFF;
            if (hit) {
                const int l = __builtin_ctzll(hit);
                at = (int)(v0 + kRunTile + 16u * (uint32_t)l - mis) + __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)m, l));
            }
            if (lane == 0) sh.ahead[par] = at;
        }
        // the next tile's bytes travel while this one is worked on
        if (tile + 1 < tile1) {
            x = load_group(tile + 1, tid);
            if (tid < kRunAhead) x_ahead = load_group(tile + 1, kRunGroups + tid);
        }
        const int c0 = __builtin_popcount(mask);
        const int inc0 = wave_scan_inclusive(c0);
        if (lane == kWave - 1) sh.wave_n[par][wv] = inc0;
        __syncthreads();
        int before = inc0 - c0, n_t = 0;
#pragma unroll
        for (int w = 0; w < kWavesPerGroup; ++w) {
            if (w < wv) before += sh.wave_n[par][w];
            n_t += sh.wave_n[par][w];
        }
        n_t = __builtin_amdgcn_readfirstlane(n_t);
        const int at_ahead = __builtin_amdgcn_readfirstlane(sh.ahead[par]);
        if (tid == 0) {
            p.tile_n[tile] = n_t;
            p.tile_info[tile] = make_int2(0, s0);
            if (tile == n_tiles - 1) p.tile_info[n_tiles] = make_int2(0, s1);
        }
        if (n_t == 0) continue;    // no piece starts here: the bytes are an earlier tile's
        // Where the tile's last piece ends: at the next start behind the tile.
        int end = min(seq_next, p.n_bytes);
        if (at_ahead != 0x7FFFFFFF) {
            end = min(end, at_ahead);
        } else {                   // a long piece: on, 4 KiB at a time
            for (uint32_t vs = v0 + kRunTile + 16u * kRunAhead; vs < (uint32_t)end + mis; vs += 16u * kGroupThreads) {
                const uint32_t mine = vs + 16u * (uint32_t)tid;
                uint32_t m = 0;
                if (mine < v_end) m = spaces_in_group(src[mine >> 4]) & below(mine, v_end);
                const uint32_t found = wave_min_u32(m ? mine + (uint32_t)__builtin_ctz(m) : 0xFFFFFFFFu);
                __syncthreads();
                if (lane == 0) sh.seek[wv] = (int)found;
                __syncthreads();
                uint32_t first = (uint32_t)sh.seek[0];
                for (int w = 1; w < kWavesPerGroup; ++w) first = min(first, (uint32_t)sh.seek[w]);
                if (first != 0xFFFFFFFFu) { end = min(end, (int)(first - mis)); break; }
            }
        }
        end = __builtin_amdgcn_readfirstlane(end);
        if (any_seq) sh.tile.group[tid] = (uint32_t)before << 16 | mask;

        const uint32_t *const words = (const uint32_t *)sh.tile.bytes;
        int r0 = 0;                                            // input index of the tile's first piece
        for (int k0 = 0; k0 < n_t; k0 += kBytePass) {          // nearly always one pass
            if (k0) __syncthreads();                           // the pass before is done
            const int n_left = __builtin_amdgcn_readfirstlane(sh.n_left);
            if (n_left > kRunLeft - kBytePass) {               // there may not be room for what this one leaves over
                merge_byte_run_left(p, sh, tile0, n_left);
                __syncthreads();
                if (tid == 0) sh.n_left = 0;
            }
            // the starts of the pass's pieces, and of the one behind them
            {
                int k = before - k0;
                for (uint32_t m = mask; m; m &= m - 1, ++k)
                    if (k >= 0 && k <= kBytePass) sh.tile.start[k] = (uint16_t)(16 * tid + __builtin_ctz(m));
            }
            __syncthreads();
            const int n_here = min(n_t - k0, kBytePass);
            int s[kBytePieces], len[kBytePieces], tok0[kBytePieces];
            uint32_t w[kBytePieces][4];
            WordKey key[kBytePieces];
            uint4 a[kBytePieces];
            if (k0 == 0) {
                r0 = origin + __builtin_amdgcn_readfirstlane((int)sh.tile.start[0]);
                if (tid == 0) { sh.first[tile - tile0] = r0; p.tile_info[tile].x = r0; }
            }
            // one probe per piece, all of them in flight together, then the second slots where the first says that a
            // word of its own sits there
#pragma unroll
            for (int r = 0; r < kBytePieces; ++r) {
                const int k = r * kGroupThreads + tid;
                s[r] = len[r] = 0;
                w[r][0] = w[r][1] = w[r][2] = w[r][3] = 0;
                a[r] = make_uint4(0, 0, 0, 0);
                if (r * kGroupThreads + wv * kWave >= n_here) continue;        // (the whole wavefront has none)
                if (k < n_here) {
                    s[r] = sh.tile.start[k];
                    len[r] = k0 + k + 1 < n_t ? (int)sh.tile.start[k + 1] - s[r] : end - (origin + s[r]);
                }
                uint32_t raw[5];
#pragma unroll
                for (int j = 0; j < 5; ++j) raw[j] = words[(s[r] >> 2) + j];
#pragma unroll
                for (int j = 0; j < 4; ++j) w[r][j] = __builtin_amdgcn_alignbyte(raw[j + 1], raw[j], (uint32_t)s[r] & 3u);
                key[r] = word_key(w[r], len[r] > 0 && len[r] <= kWordMax ? len[r] : 1);
                a[r] = word_slot(p.table, word_slot1(key[r].hash, p.table.word_shift));
            }
            bool more[kBytePieces];
#pragma unroll
            for (int r = 0; r < kBytePieces; ++r) {
                const bool look = len[r] > 0 && len[r] <= kWordMax;
                tok0[r] = look && word_hit(a[r], key[r], len[r]) ? (int)(a[r].w >> 8) : -1;
                more[r] = look && tok0[r] < 0 && (a[r].w & kWordMore);
            }
#pragma unroll
            for (int r = 0; r < kBytePieces; ++r)
                if (more[r]) a[r] = word_slot(p.table, word_slot2(key[r].hash, p.table.word_shift));
            int whole = 0;
#pragma unroll
            for (int r = 0; r < kBytePieces; ++r) {
                if (more[r] && word_hit(a[r], key[r], len[r])) tok0[r] = (int)(a[r].w >> 8);
                const int k = k0 + r * kGroupThreads + tid;
                if (tok0[r] >= 0) p.piece_word[r0 + k] = tok0[r];
                whole += __builtin_popcountll(__ballot(tok0[r] >= 0));
                const bool left = tok0[r] < 0 && len[r] > 0 && len[r] <= kTinyMax;
                const uint64_t left_mask = __ballot(left);
                if (left_mask) {
                    int e = 0;
                    if (lane == 0) e = atomicAdd(&sh.n_left, __builtin_popcountll(left_mask));
                    e = __builtin_amdgcn_readfirstlane(e) + mbcnt(left_mask);
                    if (left) {
                        sh.merge.run.bytes[e] = make_uint4(w[r][0], w[r][1], w[r][2], w[r][3]);
                        sh.merge.run.piece[e] = make_int2(origin + s[r], len[r] << 16 | k);
                    }
                }
                if (len[r] > kTinyMax) {       // rare in word-like text
                    const bool col = len[r] <= p.col_max;
                    const int e = col ? atomicAdd(&sh.n_col, 1) : atomicAdd(&sh.n_long, 1);
                    LongPiece *list = col ? long_list(p, run_lo + 1) + e : long_list(p, run_hi) - 1 - e;
                    *list = LongPiece{origin + s[r], len[r], r0 + k, tile - tile0};
                }
            }
            if (lane == 0 && whole) atomicAdd(&sh.acc[tile - tile0], whole);
            __syncthreads();       // the starts and the bytes are free
        }
        // Which piece every sequence that starts in the tile starts with (as ~number; the next kernel knows its tokens).
        if (any_seq) {
            for (int64_t q = (int64_t)s0 + tid; q < s1; q += kGroupThreads) {
                const int sv = p.seq_off ? p.seq_off[q] : 0;
                if (sv < lo || sv >= hi) continue;
                const uint32_t at = (uint32_t)sv + mis - v0, g = sh.tile.group[at >> 4];
                p.seq_token_offsets[q] = ~(int)((g >> 16) + __builtin_popcount(g & ((1u << (at & 15)) - 1u)));
            }
            __syncthreads();
        }
    }
    __syncthreads();
    const int n_left = __builtin_amdgcn_readfirstlane(sh.n_left);
    if (n_left) {
        merge_byte_run_left(p, sh, tile0, n_left);
        __syncthreads();
    }
    const int n_col = __builtin_amdgcn_readfirstlane(sh.n_col), n_long = __builtin_amdgcn_readfirstlane(sh.n_long);
    if (n_col + n_long) {
        const EncodeParams &kp = kernel_params();
        constexpr int kAtOnce = kGroupThreads / 2;             // of either list
#pragma unroll 1
        for (int e0 = 0; e0 < max(n_col, n_long); e0 += kAtOnce) {
            const int col_here = max(min(n_col - e0, kAtOnce), 0), long_here = max(min(n_long - e0, kAtOnce), 0);
            if (tid < col_here + long_here) {
                sh.longer.piece[tid] = tid < col_here ? long_list(kp, run_lo + 1)[e0 + tid]
                                                      : *(long_list(kp, run_hi) - 1 - (e0 + tid - col_here));
                sh.longer.entry[tid] = (uint32_t)tid;
            }
            __syncthreads();
            const EncodeParams &lp = kernel_params_here();
            merge_listed_pieces(
                lp, sh.merge, sh.tmp, col_here, long_here, [&](int e) -> uint32_t & { return sh.longer.entry[e]; },
                [&](int k, int &b, int &n) { b = sh.longer.piece[k].b; n = sh.longer.piece[k].n; },
                [&](int, int k, int c) {
                    const LongPiece q = sh.longer.piece[k];
                    const uint32_t v = (uint32_t)(q.b + lp.tile_shift);
                    lp.piece_word[q.slot] = (int)(kSeveral | (v % kRunTile) << kStartShift | min((uint32_t)c, kManyTokens));
                    if ((uint32_t)c >= kManyTokens) lp.piece_word[q.slot + 1] = c;
                    atomicAdd(&sh.acc[q.tile], c);
                });
            __syncthreads();
        }
    }
    if (tid < tile1 - tile0) kernel_params().tile_sum[tile0 + tid] = sh.acc[tid];
}

// Whether the offsets off[0 .. n] are anything but 0, ..., n_bytes without a decrease.  Every thread of the workgroup must
// call it.
__device__ __forceinline__ bool offsets_are_bad(const int32_t *off, int n, int n_bytes) {
    bool bad = false;
    for (int64_t k = threadIdx.x; k <= n; k += kGroupThreads) {
        const int v = off[k];
        bad |= v < 0 || v > n_bytes || (k == 0 && v != 0) || (k == n ? v != n_bytes : off[k + 1] < v);
    }
    return __syncthreads_or(bad);
}

// Assembly: the tokens of every tile to their place in out_ids, and the first token of every sequence.  A workgroup
// takes a tile, a thread three of its pieces (616 of word-like text start in a tile): every 64th of its wavefront's 192
// consecutive ones, so that the loads and, with one token per piece nearly always, the stores of a wavefront are contiguous.
// (Three consecutive ones per thread touched every line with each of three loads and stores: 134 MB 71.0 -> 64.7 us in the kernel
// trace, per call 298 -> 293; 1k table, where many pieces have several tokens, 20 MB 99.5 -> 92.9, 64 MB 308 -> 282.)
// Bound by its round trips.  A wavefront per tile instead, with the totals before it always from scan_tiles_kernel: 134 MB of text
// 282 us per call, but 1k table 64 MB 299.
typedef int32_t int4_any __attribute__((ext_vector_type(4), aligned(4)));       // 16 bytes at any word
constexpr int kEmitPieces = 3;
constexpr int kEmitPass = kEmitPieces * kGroupThreads;
__global__ void __launch_bounds__(kGroupThreads) emit_byte_runs_kernel(EncodeParams p, int n_tiles, int self_scan) {
    __shared__ int before_w[kWavesPerGroup], total_w[2][kWavesPerGroup];
    __shared__ int firsts[kEmitPass];
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int tile = blockIdx.x;
    const int n = p.tile_n[tile], s_end = p.tile_info[tile + 1].y, verdict = p.status[kStatusBadInput];
    const int2 info = p.tile_info[tile];
    // tokens before the tile
    int before = 0;
    if (self_scan) {               // tile_sum is 256-byte aligned
        for (int t = tid * 4; t < tile; t += kGroupThreads * 4) {
            const int4 a = *(const int4 *)(p.tile_sum + t);
            before += a.x + (t + 1 < tile ? a.y : 0) + (t + 2 < tile ? a.z : 0) + (t + 3 < tile ? a.w : 0);
        }
    } else if (tid == 0) {
        before = p.tile_base[tile];
    }
    const int32_t *const words = p.piece_word + info.x;
    const int origin = (int)((uint32_t)tile * kRunTile - (uint32_t)p.tile_shift);
    before = __builtin_amdgcn_readlane(wave_scan_inclusive(before), kWave - 1);
    if (lane == 0) before_w[wv] = before;
    // Sequence offsets that are out of range or decrease: each tile has searched them for its own part, the tiles need not
    // agree on where a piece ends, and pieces that overlap can have more tokens than out_ids has room for.  So no token is
    // stored then, and every sequence is empty.  (The verdict can be that of an earlier replay of a recorded call: the
    // workgroup looks for itself.  Looked at here, behind the loads above: at the head it was 1 % of a call of 13.5 MB.)
    if (p.seq_off && verdict == p.call_id && offsets_are_bad(p.seq_off, p.n_seqs, p.n_bytes)) {
        for (int64_t s = (int64_t)tile * kGroupThreads + tid; s <= p.n_seqs; s += (int64_t)n_tiles * kGroupThreads)
            p.seq_token_offsets[s] = 0;
        if (tile == 0 && tid == 0) mark_call(p.status, p.call_id);
        return;
    }
    int base = 0, par = 0;
    for (int i0 = 0; i0 < n || i0 == 0; i0 += kEmitPass, par ^= 1) {   // nearly always one pass
        const int i = i0 + wv * kEmitPieces * kWave + lane;            // piece j of the thread: i + 64 j
        int word[kEmitPieces], c[kEmitPieces], at[kEmitPieces], inc[kEmitPieces];
#pragma unroll
        for (int j = 0; j < kEmitPieces; ++j) word[j] = i + j * kWave < n ? words[i + j * kWave] : 0;
#pragma unroll
        for (int j = 0; j < kEmitPieces; ++j) {
            const uint32_t u = (uint32_t)word[j];
            at[j] = origin + (int)((u & ~kSeveral) >> kStartShift);
            c[j] = i + j * kWave >= n ? 0 : word[j] < 0 ? (int)(u & kManyTokens) : 1;
            if (word[j] < 0 && c[j] == (int)kManyTokens) c[j] = words[i + j * kWave + 1];
        }
        // the first four tokens of a piece of several, asked for before anything waits (what lies behind them is the workspace's)
        int4_any head[kEmitPieces];
#pragma unroll
        for (int j = 0; j < kEmitPieces; ++j)
            if (word[j] < 0) head[j] = *(const int4_any *)(p.scratch + at[j]);
        int wave_total = 0;
#pragma unroll
        for (int j = 0; j < kEmitPieces; ++j) {
            inc[j] = wave_total + wave_scan_inclusive(c[j]);
            wave_total = __builtin_amdgcn_readlane(inc[j], kWave - 1);
        }
        if (lane == 0) total_w[par][wv] = wave_total;
        __syncthreads();
        if (i0 == 0)
            for (int w = 0; w < kWavesPerGroup; ++w) base += before_w[w];
        int wave_first = base, all = 0;
        for (int w = 0; w < kWavesPerGroup; ++w) {
            if (w < wv) wave_first += total_w[par][w];
            all += total_w[par][w];
        }
        int first[kEmitPieces];
#pragma unroll
        for (int j = 0; j < kEmitPieces; ++j) first[j] = wave_first + inc[j] - c[j];
#pragma unroll
        for (int j = 0; j < kEmitPieces; ++j) {
            if (c[j] && word[j] >= 0) p.out_ids[first[j]] = word[j];
            if (word[j] < 0) {
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if (k < c[j]) p.out_ids[first[j] + k] = head[j][k];
            }
        }
#pragma unroll
        for (int j = 0; j < kEmitPieces; ++j) {                // the fifth to the sixteenth by the thread, the rest by its wavefront
            const int m = word[j] < 0 ? c[j] : 0;
            if (!__ballot(m > 4)) continue;
#pragma unroll
            for (int k = 4; k < 16; k += 4) {
                if (k < m) {
                    const int4_any v = *(const int4_any *)(p.scratch + at[j] + k);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (k + q < m) p.out_ids[first[j] + k + q] = v[q];
                }
            }
            for (uint64_t big = __ballot(m > 16); big;) {
                const int t = __builtin_ctzll(big);
                big &= big - 1;
                copy_words<kWave>(p.scratch + read_lane(at[j], t), p.out_ids + read_lane(first[j], t), 16, read_lane(m, t), lane);
            }
        }
        if (s_end > info.y) {      // sequences start in this tile: with which pieces, the merge kernel has noted
#pragma unroll
            for (int j = 0; j < kEmitPieces; ++j) firsts[i - i0 + j * kWave] = first[j];
            __syncthreads();
            for (int64_t s = (int64_t)info.y + tid; s < s_end; s += kGroupThreads) {
                const int k = ~p.seq_token_offsets[s] - i0;    // (one that has its token is far below)
                if (k >= 0 && k < min(kEmitPass, n - i0)) p.seq_token_offsets[s] = firsts[k];
            }
            __syncthreads();
        }
        base += all;
    }
    if (tile == n_tiles - 1)       // the closing entry, and sequences that start behind the last byte
        for (int64_t s = (int64_t)s_end + tid; s <= p.n_seqs; s += kGroupThreads) p.seq_token_offsets[s] = base;
    if (tile == 0 && tid == 0) mark_call(p.status, p.call_id);
}

}  // namespace bpe
