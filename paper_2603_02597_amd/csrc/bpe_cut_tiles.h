// Encoding pieces that are long on average (fixed chunks of text, whole documents; cut_least_bytes says from where on): a
// piece is cut first, wherever no token can reach across, and its parts are encoded like pieces.  Device code, included by
// bpe_encode.hip behind bpe_byte_runs.h.
//
// A token that reached across the border of two bytes x, y would have them side by side in its expansion, and every
// rule that makes such a token joins a string that ends with x to one that starts with y, or works on one that
// already holds both.  So where no rule joins a string that ends with x to one that starts with y, nothing merges
// across: the parts on either side merge as if they stood alone, whatever the rest does (tests/test_cuts_rule.py).
// Which bytes that concerns is kept per byte (CutSets): tables trained on words never put a space behind another
// byte, and a piece of text then falls into its words, nearly all of them found whole by one probe each.
//
// A workgroup takes TILE consecutive bytes, whatever pieces they belong to, and keeps them in LDS.  The parts that
// start there are a dense list: a thread takes ROUNDS of them, with the probes of the whole-piece table in flight
// together.  What the probes leave over is listed and merged by all wavefronts; then the token counts are scanned
// once and every thread stores its tokens at their place among the tile's: scratch2[first byte of the tile's first
// part ...] (parts have at least as many bytes as tokens, so the tiles do not overlap).  A second kernel copies them to
// their place.  Bound by the chain of a tile: offsets, bytes, cuts, probes, left-over merges, counts.
//
// Per call, every piece by one workgroup, wavefront or lane / cut: 840 KB of text with the 50k table in chunks of 64, 256, 1,024 and
// 2,048 bytes 55, 89, 116 and 157 / 19.6, 16.7, 16.7 and 16.5 us (there wavefronts wait for 71 % of the time, 1.5 per SIMD in flight); with
// runs and random bytes, 100k table, 60, 277, 1,999 and 2,262 / 42, 42, 42 and 42.  Data without a place to cut pays for the look:
// random bytes, 100k table, in pieces of 64, 256, 1,024 and 2,048 39, 376, 532 and 879 / 51, 411, 541 and 1,094; text without spaces 49,
// 196, 300 and 504 / 61, 199, 312 and 532; runs of 200 bytes 53, 38, 18 and 20 / 35, 32, 31 and 33 (there a piece is a handful of runs for one
// wavefront, and cut, each run is one of its own).
#pragma once

namespace bpe {

constexpr int kTileGroup = 16;               // a thread looks at 16 bytes at a time ("group")
constexpr int kAheadGroups = 16;             // groups looked at behind the tile for the end of its last part

// Longest piece that merge_uncut_parts merges as a whole: 16 wavefronts then take as long as the tiles do (text without
// spaces, 50k / 100k table, in pieces of 8,000 bytes 790 / 662 and 778 / 659 us; of 20,000 2,400 / 1,984 and 612 / 2,006).
constexpr int kWideWhole = 2 * kWideBoundMax;

// Bits of byte b in a table of its properties.
constexpr uint32_t kCutBefore = 1, kCutBehind = 2, kTwin = 4;

__device__ __forceinline__ uint32_t cut_code(const CutSets &c, uint32_t b) {
    return ((c.before[b >> 5] >> (b & 31)) & 1u) | ((c.behind[b >> 5] >> (b & 31)) & 1u) << 1 | ((c.twin[b >> 5] >> (b & 31)) & 1u) << 2;
}

// Bit j set: a part starts at byte j of the 16-byte group; prev: the byte before the group.  code: kCutBefore ... of
// every byte.  n_equal: how many of the bytes equal the one before them.
__device__ __forceinline__ uint32_t cuts_in_group(const uint8_t *code, const uint4 &x, uint32_t prev, int &n_equal) {
    const uint32_t w[4] = {x.x, x.y, x.z, x.w};
    uint32_t m = 0, last = prev, last_code = code[prev];
    n_equal = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint32_t b = (w[j / 4] >> (8 * (j % 4))) & 0xFFu, c = code[b];
        const uint32_t cut = ((c & kCutBefore) | (last_code & kCutBehind) >> 1) & ~(b == last ? c >> 2 : 0u);
        n_equal += b == last;
        m |= cut << j;
        last = b;
        last_code = c;
    }
    return m;
}

template <int TILE, int ROUNDS>
struct CutTileShared {
    static constexpr int kPieces = ROUNDS * kGroupThreads;     // pieces merged per pass
    static constexpr int kParts = ROUNDS * kWavesPerGroup;     // a round of a wavefront
    // 16-byte groups that hold bytes of the tile, and that are kept: the words of a short part end 19 bytes behind the
    // tile at most
    static constexpr int kGroups = TILE / kTileGroup;
    static constexpr int kStaged = kGroups + 2;
    union {
        MergeLds merge;
        uint4 bytes[kStaged];      // until the columns, or the paths of longer pieces, take its place
    } lds;
    GroupTmp tmp;
    uint8_t code[256];             // see cuts_in_group
    uint32_t group[kGroups];       // starts in the tile before the group << 16 | start mask
    uint32_t entry[kPieces];       // pieces that the probes leave over, by kind: first the short ones, then those for the
                                   // columns, then the longer ones.  The piece's number in the pass; then its token count;
                                   // then where its tokens go.
    uint32_t part[kParts];         // how many of each kind a round of a wavefront has (10 bits each)
    uint32_t total[kParts];        // tokens
    int long_bytes, run_groups;    // bytes of parts beyond the columns; groups that are mostly one byte
    int2 whole[4];                 // WIDE: pieces that start here and are merged as a whole: first byte, end
    int n_whole;
    uint16_t start[kPieces + 2];   // first byte of every piece of the pass, counted from the first group; later its first token
    int ahead[kWavesPerGroup];
    int wave_n[kWavesPerGroup];
};

// EAGER: both slots of the whole-piece table at once (see find_word).  WIDE: merge_uncut_parts has merged the parts beyond
// kGroupBoundMax bytes, and some pieces as a whole (the tokens in scratch; for their numbers see there).
template <int TILE, int ROUNDS, bool EAGER, bool WIDE>
__global__ void __launch_bounds__(kGroupThreads, 4) merge_cut_tiles_kernel(EncodeParams p, CutSets cuts) {
    using Shared = CutTileShared<TILE, ROUNDS>;
    constexpr int kPieces = Shared::kPieces, kParts = Shared::kParts, kGroups = Shared::kGroups;
    static_assert(kGroups + kAheadGroups <= kGroupThreads, "a group per thread");
    __shared__ Shared sh;
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int tile = blockIdx.x;
    // Positions v are counted from the 16-byte boundary at or below the input: byte i is v = i + mis.
    const uint32_t mis = (uint32_t)((uintptr_t)p.bytes & 15);
    const uint32_t v_end = p.n_bytes ? (uint32_t)p.n_bytes + mis : 0u;
    const int lo = (int)min(max((int64_t)tile * TILE - p.tile_shift, (int64_t)0), (int64_t)p.n_bytes);    // (the last tile may be empty)
    const int hi = (int)min((int64_t)(tile + 1) * TILE - p.tile_shift, (int64_t)p.n_bytes);
    const uint32_t v0 = ((uint32_t)lo + mis) & ~15u;           // the tile's first group
    const uint4 *src = (const uint4 *)(p.bytes - mis);

    // The tile's bytes and the 256 behind them, asked for before anything else.  (A group that holds a byte of
    // the input lies in that byte's page.)
    uint4 x = make_uint4(0, 0, 0, 0);
    const uint32_t group_v = v0 + 16u * (uint32_t)tid;         // position of the thread's group
    if (tid < kGroups + kAheadGroups && group_v < v_end) x = src[group_v >> 4];

    // (the byte before the group, where no lane below holds it)
    const int64_t before_at = (int64_t)group_v - 1 - mis;
    const uint32_t prev = lane == 0 && before_at >= 0 && before_at < p.n_bytes ? p.bytes[before_at] : 0u;
    sh.code[tid] = (uint8_t)cut_code(cuts, (uint32_t)tid);
    if (tid == 0) sh.long_bytes = sh.run_groups = sh.n_whole = 0;
    const bool in_whole = WIDE && p.tile_sum[tile] == 1;       // (looked at only where a piece reaches into the tile)

    // Pieces (seq_off): every tile checks a strided share of their offsets and finds the ones that start among its own
    // bytes, seq_off[s0 .. s1); seq_next: the first one at or behind the tile's end (a part ends there at the latest).
    int s0, s1, seq_next = p.n_bytes, seq_first = p.n_bytes;   // seq_first: the first one of all
    // WIDE: pieces that start here and are merged as a whole, if all offsets needed are among the 64
    auto of_whole_size = [&](int first, int next) {
        return next <= p.n_bytes && next - first > kGroupBoundMax && next - first <= kWideWhole;
    };
    bool at_hand = false;
    int whole_first = -1, whole_end = 0;
    {
        bool bad = false;
        for (int64_t k = (int64_t)tile * kGroupThreads + tid; k <= p.n_seqs; k += (int64_t)gridDim.x * kGroupThreads) {
            const int sv = p.seq_off[k];
            bad |= sv < 0 || sv > p.n_bytes || (k == 0 && sv != 0) || (k == p.n_seqs && sv != p.n_bytes);
            if (k < p.n_seqs) bad |= p.seq_off[k + 1] < sv;
        }
        if (__ballot(bad) && lane == 0)
            __hip_atomic_store(&p.status[kStatusBadInput], p.call_id, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // Pieces of about one length (chunks) are where the average says: 64 offsets around that place, usually the only
        // look.  Otherwise a search, 64 places at a time.
        const float per_byte = (float)p.n_seqs / (float)p.n_bytes;
        const int guess = min(max((int)((float)lo * per_byte) - kWave / 2, 0), p.n_seqs);
        int at = guess, v = p.seq_off[min((int64_t)guess + lane, (int64_t)p.n_seqs)];
        uint64_t below = __ballot((int64_t)guess + lane <= p.n_seqs && v < lo);
        if ((guess > 0 && !(below & 1)) || !~below) {
            at = wave_lower_bound(p.seq_off, 0, p.n_seqs + 1, lo);
            v = p.seq_off[min((int64_t)at + lane, (int64_t)p.n_seqs)];
            below = 0;
        }
        s0 = at + (int)__builtin_ctzll(~below);
        if (WIDE && s0 <= p.n_seqs) seq_first = read_lane(v, s0 - at);
        const uint64_t inside = __ballot((int64_t)at + lane <= p.n_seqs && v < hi);
        if (~inside) {
            const int c = (int)__builtin_ctzll(~inside);
            s1 = at + c;
            if (s1 <= p.n_seqs) seq_next = min(max(read_lane(v, c), hi), p.n_bytes);
        } else {
            s1 = wave_lower_bound(p.seq_off, min(at + kWave, p.n_seqs + 1), p.n_seqs + 1, hi);
            if (s1 <= p.n_seqs) seq_next = min(max(__builtin_amdgcn_readfirstlane(p.seq_off[s1]), hi), p.n_bytes);
        }
        s1 = max(s0, s1);          // (offsets that decrease)
        if (WIDE) {
            const int k = at + lane, next = wave_from_lane_above(v, 0);
            at_hand = s1 - at < kWave;
            if (at_hand && wv == 0 && k >= s0 && k < s1 && k < p.n_seqs && v >= lo && v < hi && of_whole_size(v, next) && p.scratch2[v] >= 0) {
                whole_first = v;
                whole_end = next;
            }
        }
    }
    const bool any_seq = s1 > s0;                              // the same in every wavefront
    if (tid < kGroups) sh.group[tid] = 0;
    __syncthreads();               // (the byte codes, too)
    if (any_seq) {
        auto list_whole = [&](int first, int end) {
            const int i = atomicAdd(&sh.n_whole, 1);
            if (i < 4) sh.whole[i] = make_int2(first, end);                // (more only if the offsets decrease)
        };
        for (int64_t k = (int64_t)s0 + tid; k < s1; k += kGroupThreads) {
            const int sv = p.seq_off[k];
            if (sv < lo || sv >= hi) continue;
            const uint32_t at = (uint32_t)sv + mis - v0;
            atomicOr(&sh.group[at >> 4], 1u << (at & 15));
            if (WIDE && !at_hand && k < p.n_seqs) {
                const int next = p.seq_off[k + 1];
                if (of_whole_size(sv, next) && p.scratch2[sv] >= 0) list_whole(sv, next);
            }
        }
        if (WIDE && whole_first >= 0) list_whole(whole_first, whole_end);
        __syncthreads();
    }
    const int n_whole = WIDE ? __builtin_amdgcn_readfirstlane(min(sh.n_whole, 4)) : 0;
    bool out_of_tile = false;      // the last piece is merged as a whole and reaches out of the tile
    for (int i = 0; i < n_whole; ++i) out_of_tile |= sh.whole[i].y > hi;

    // Start masks of the groups; starts behind the tile only say where its last piece ends.
    uint32_t mask = 0, piece_starts = 0;
    // bits of the group's bytes below position `limit`
    auto below = [&](uint32_t limit) { return limit <= group_v ? 0u : limit - group_v >= 16u ? 0xFFFFu : (1u << (limit - group_v)) - 1u; };
    const uint32_t before_group = (uint32_t)wave_from_lane_below((int)(x.w >> 24), (int)prev);
    int n_equal = 0;
    uint32_t m = tid < kGroups + kAheadGroups ? cuts_in_group(sh.code, x, before_group, n_equal) : 0u;
    const uint32_t ahead = m & below(v_end) & ~below((uint32_t)hi + mis);
    if (tid < kGroups) {
        if (any_seq) piece_starts = sh.group[tid];
        if (lo == 0 && group_v <= mis && mis < group_v + 16u) piece_starts |= 1u << (mis - group_v);     // byte 0 starts a piece
        m |= piece_starts;
        const uint64_t runs = __ballot(n_equal > 12);
        if (lane == 0 && runs) atomicAdd(&sh.run_groups, __builtin_popcountll(runs));
        mask = m & below((uint32_t)hi + mis) & ~below((uint32_t)lo + mis);
        if (in_whole && seq_first > lo) mask &= ~below((uint32_t)min(seq_first, hi) + mis);
        for (int i = 0; i < n_whole; ++i) {
            const int2 w = sh.whole[i];
            mask &= ~(below((uint32_t)min(w.y, hi) + mis) & ~below((uint32_t)w.x + 1u + mis));
        }
    }
    const uint64_t hit = __ballot(ahead != 0);
    int first_ahead = 0x7FFFFFFF;
    if (hit) {
        const int l = __builtin_ctzll(hit);
        first_ahead = (int)(__builtin_amdgcn_readlane((int)group_v, l) - mis) + __builtin_ctz((uint32_t)__builtin_amdgcn_readlane((int)ahead, l));
    }
    if (lane == 0) sh.ahead[wv] = first_ahead;
    if (tid < Shared::kStaged) sh.lds.bytes[tid] = x;
    const int c0 = __builtin_popcount(mask);
    const int inc0 = wave_scan_inclusive(c0);
    if (lane == kWave - 1) sh.wave_n[wv] = inc0;
    __syncthreads();
    int before = inc0 - c0, n_t = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) {
        if (w < wv) before += sh.wave_n[w];
        n_t += sh.wave_n[w];
    }
    if (tid < kGroups) sh.group[tid] = (uint32_t)before << 16 | mask;
    n_t = __builtin_amdgcn_readfirstlane(n_t);
    int2 *const info = p.tile_info + tile;
    if (n_t == 0) {                // no piece starts here: the bytes are an earlier tile's
        if (tid == 0) {
            p.tile_sum[tile] = 0;
            *info = make_int2(0, s0);
            if (tile == (int)gridDim.x - 1) info[1] = make_int2(0, s1);
        }
        return;
    }
    // Where the tile's last piece ends: at the next start behind the tile.
    int end = min(seq_next, p.n_bytes);
    {
        int at = sh.ahead[0];
#pragma unroll
        for (int w = 1; w < kWavesPerGroup; ++w) at = min(at, sh.ahead[w]);
        const uint32_t looked_at = v0 + 16u * (kGroups + kAheadGroups);        // positions below are done with
        if (WIDE && out_of_tile) {                             // up to the next piece
        } else if (at != 0x7FFFFFFF) {
            end = min(end, at);
        } else if ((uint32_t)end + mis > looked_at) {          // a long piece: on, 4 KiB at a time
            for (uint32_t v = looked_at; v < (uint32_t)end + mis; v += 16u * kGroupThreads) {
                const uint32_t mine = v + 16u * (uint32_t)tid;
                uint32_t m = 0;
                int n_equal;
                if (mine < v_end) m = cuts_in_group(sh.code, src[mine >> 4], p.bytes[mine - mis - 1], n_equal);
                if (mine + 16u > v_end) m &= mine < v_end ? (1u << (v_end - mine)) - 1u : 0u;
                const uint32_t found = wave_min_u32(m ? mine + (uint32_t)__builtin_ctz(m) : 0xFFFFFFFFu);
                __syncthreads();
                if (lane == 0) sh.tmp.min_lo[wv] = found;
                __syncthreads();
                uint32_t first = sh.tmp.min_lo[0];
                for (int w = 1; w < kWavesPerGroup; ++w) first = min(first, sh.tmp.min_lo[w]);
                if (first != 0xFFFFFFFFu) { end = min(end, (int)(first - mis)); break; }
            }
        }
    }
    end = __builtin_amdgcn_readfirstlane(end);

    const uint32_t *const words = (const uint32_t *)sh.lds.bytes;
    const uint8_t *const bytes = (const uint8_t *)sh.lds.bytes;
    const int origin = (int)(v0 - mis);                        // input index of the first group's first byte (may be -15)
    int r0 = 0;                                                // input index of the tile's first piece
    int done = 0;                                              // tokens of the passes before
    int whole_tile = 0;                                        // 1: cut at pieces only
    for (int k0 = 0; k0 < n_t; k0 += kPieces) {                // nearly always one pass
        const EncodeParams &p = kernel_params_here();
        const int lane = lane_id_here(), tid = wv * kWave + lane;
        if (k0) {
            __syncthreads();       // the pass before is done with the lists
            if (tid < Shared::kStaged) {                       // the columns may have taken the bytes' place
                const uint32_t at = v0 + 16u * (uint32_t)tid;
                sh.lds.bytes[tid] = at < v_end ? src[at >> 4] : make_uint4(0, 0, 0, 0);
            }
        }
        // the starts of the pass's pieces, and of the one behind them
        const uint32_t starts = tid < kGroups ? sh.group[tid] : 0u;
        int k_next = (int)(starts >> 16) - k0;
        for (uint32_t m = starts & 0xFFFFu; m; m &= m - 1, ++k_next)
            if (k_next >= 0 && k_next <= kPieces) sh.start[k_next] = (uint16_t)(16 * tid + __builtin_ctz(m));
        __syncthreads();
        const int n_here = min(n_t - k0, kPieces);

        int s[ROUNDS], len[ROUNDS], tok0[ROUNDS], n_wide[ROUNDS], kind[ROUNDS];        // kind: 0 none or whole, 1 short, 2 for the columns, 3 longer
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            const int k = r * kGroupThreads + tid;
            s[r] = len[r] = 0;
            tok0[r] = -1;
            if (k < n_here) {
                s[r] = sh.start[k];
                len[r] = k0 + k + 1 < n_t ? (int)sh.start[k + 1] - s[r] : end - (origin + s[r]);
            }
        }
        if (k0 == 0) r0 = origin + __builtin_amdgcn_readfirstlane((int)sh.start[0]);
        // one probe per piece (two with EAGER), all of them in flight together, then the second slots where the first
        // says that a word of its own sits there
        {
            WordKey key[ROUNDS];
            uint4 a[ROUNDS], b[ROUNDS];
            bool look[ROUNDS];
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                look[r] = len[r] > 0 && len[r] <= min(p.tiny_max, kWordMax);
                const int at = s[r] >> 2;
                uint32_t raw[4], w[4] = {0, 0, 0, 0};          // (12 bytes from byte 3 on end in the fourth word)
#pragma unroll
                for (int j = 0; j < 4; ++j) raw[j] = words[at + j];
#pragma unroll
                for (int j = 0; j < 3; ++j) w[j] = __builtin_amdgcn_alignbyte(raw[j + 1], raw[j], (uint32_t)s[r] & 3u);
                key[r] = word_key(w, look[r] ? len[r] : 1);
                a[r] = word_slot(p.table, word_slot1(key[r].hash, p.table.word_shift));
                if (EAGER) b[r] = word_slot(p.table, word_slot2(key[r].hash, p.table.word_shift));
            }
            bool more[ROUNDS];
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                if (look[r] && word_hit(a[r], key[r], len[r])) tok0[r] = (int)(a[r].w >> 8);
                more[r] = look[r] && tok0[r] < 0 && (EAGER || (a[r].w & kWordMore));
            }
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
                if (!EAGER && more[r]) b[r] = word_slot(p.table, word_slot2(key[r].hash, p.table.word_shift));
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
                if (more[r] && word_hit(b[r], key[r], len[r])) tok0[r] = (int)(b[r].w >> 8);
        }

        // What is left over, listed by kind.
        uint64_t of_kind[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            n_wide[r] = 0;
            if (WIDE && !whole_tile && len[r] > kGroupBoundMax) {
                const int n = p.scratch2[origin + s[r]];
                n_wide[r] = min(n < 0 ? ~n : n, len[r]);       // (any number there if the offsets decrease)
                atomicAdd(&sh.run_groups, TILE);               // no cutting at the pieces only: this part is done
            }
            kind[r] = tok0[r] >= 0 || len[r] <= 0 || n_wide[r] ? 0 : len[r] <= p.tiny_max ? 1 : len[r] <= p.col_max ? 2 : 3;
            if (kind[r] == 2) {
                // A run (told by eight equal bytes) is halved by every pass of a wavefront, but merges one pair a time in a
                // column: 64-byte pieces of text with runs and random bytes 59 us with all of them in columns, 34 so, and
                // random bytes 48 and 84 with none there.
                const int at = s[r] + 8;
                const uint32_t w0 = words[at >> 2], w1 = words[(at >> 2) + 1], w2 = words[(at >> 2) + 2];
                const uint32_t a = __builtin_amdgcn_alignbyte(w1, w0, (uint32_t)at & 3u), b = __builtin_amdgcn_alignbyte(w2, w1, (uint32_t)at & 3u);
                if (a == b && a == (a & 0xFFu) * 0x01010101u) kind[r] = 3;
            }
            uint32_t n = 0;
            of_kind[r] = 0;
#pragma unroll
            for (int q = 1; q <= 3; ++q) {
                const uint64_t m = __ballot(kind[r] == q);
                if (kind[r] == q) of_kind[r] = m;
                n |= (uint32_t)__builtin_popcountll(m) << (10 * (q - 1));
            }
            if (lane == 0) sh.part[r * kWavesPerGroup + wv] = n;
            if (kind[r] == 3 && len[r] > p.col_max) atomicAdd(&sh.long_bytes, min(len[r], TILE));
        }
        __syncthreads();
        uint32_t all = 0, mine_from[ROUNDS];
#pragma unroll
        for (int k = 0; k < kParts; ++k) {
            if (k % kWavesPerGroup == wv) mine_from[k / kWavesPerGroup] = all;
            all += sh.part[k];
        }
        all = (uint32_t)__builtin_amdgcn_readfirstlane((int)all);
        const int n_short = all & 1023;
        int n_col = (all >> 10) & 1023, n_long = all >> 20;
        // Little but parts of hundreds of bytes (binary data, text that has no spaces), and no runs: each by itself would take
        // one wavefront most of the time that all four take for the whole tile (1,024-byte pieces of random bytes, which fall
        // into five parts: 1,026 us, and 538 uncut).  So then the tile's bytes are cut at the pieces only.
        if (whole_tile == 0 && n_long >= 2 && n_t <= kPieces &&
            2 * __builtin_amdgcn_readfirstlane(sh.long_bytes) >= hi - r0 && __builtin_amdgcn_readfirstlane(sh.run_groups) <= TILE / 128) {
            whole_tile = 1;
            const int first_at = (int)sh.start[0];
            uint32_t m = tid < kGroups ? piece_starts : 0u;
            if (first_at >> 4 == tid) m |= 1u << (first_at & 15);
            const int c = __builtin_popcount(m), inc = wave_scan_inclusive(c);
            if (lane == kWave - 1) sh.wave_n[wv] = inc;
            __syncthreads();
            int before = inc - c;
            n_t = 0;
#pragma unroll
            for (int w = 0; w < kWavesPerGroup; ++w) {
                if (w < wv) before += sh.wave_n[w];
                n_t += sh.wave_n[w];
            }
            n_t = __builtin_amdgcn_readfirstlane(n_t);
            if (tid < kGroups) sh.group[tid] = (uint32_t)before << 16 | m;
            k0 = -kPieces;
            continue;
        }
        int slot[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            slot[r] = -1;
            if (kind[r]) {
                const int q = kind[r] - 1;
                slot[r] = (q > 0 ? n_short : 0) + (q > 1 ? n_col : 0) + (int)((mine_from[r] >> (10 * q)) & 1023u) + mbcnt(of_kind[r]);
                sh.entry[slot[r]] = (uint32_t)(r * kGroupThreads + tid);
            }
        }
        if (whole_tile && n_col + n_long <= 2 * kWavesPerGroup) {      // (mostly the longer ones: no wavefront for the others alone)
            n_long += n_col;
            n_col = 0;
        }
        // Where the columns leave wavefronts idle, these merge the short parts meanwhile: a chain less.
        const int col_waves = min((n_col + kColumnLanes - 1) / kColumnLanes, kWavesPerGroup);
        const bool beside = n_col && n_short <= kWave * (kWavesPerGroup - col_waves);
        const int first_wave = beside ? col_waves : 0;
        // first byte (counted from the first group) and length of piece k of the pass
        auto bounds = [&](int k, int &at, int &n) {
            at = sh.start[k];
            n = k0 + k + 1 < n_t ? (int)sh.start[k + 1] - at : end - (origin + at);
        };
        // Tokens of left-over short pieces stay with whoever merges them (a row's lanes, a lane's column) until their
        // place is known; if longer pieces need the room, or one round of columns does not do, they go to scratch.
        const bool parked = n_col + n_long > 0 || n_short > kGroupThreads;
        uint32_t row_sym = 0, alive = 0;
        int row_n = 0;
        if (n_short) {
            __syncthreads();
            if (!beside && n_short <= row_pieces(kWavesPerGroup)) {
                constexpr int kRows = kWave / kTinyMax;
                if (wv * kRows < n_short) {
                    const int j = lane & (kTinyMax - 1), e = wv * kRows + lane / kTinyMax;
                    int at = 0, n = 0;
                    if (e < n_short) bounds((int)sh.entry[e], at, n);
                    row_sym = bytes[at + j] | (3u << 24);
                    row_n = row_merge(p, row_sym, n);
                    row_sym &= 0xFFFFFFu;
                    if (parked && j < row_n) p.scratch[origin + at + j] = (int)row_sym;
                    if (e < n_short && j == 0) sh.entry[e] = (uint32_t)row_n;
                }
            } else {
                uint32_t w[ROUNDS][4];
                int at[ROUNDS], n[ROUNDS];
#pragma unroll
                for (int r = 0; r < ROUNDS; ++r) {
                    const int e = r * kGroupThreads + tid - first_wave * kWave;
                    at[r] = n[r] = 0;
                    if (e >= 0 && e < n_short) bounds((int)sh.entry[e], at[r], n[r]);
                    uint32_t raw[5];
#pragma unroll
                    for (int j = 0; j < 5; ++j) raw[j] = words[(at[r] >> 2) + j];
#pragma unroll
                    for (int j = 0; j < 4; ++j) w[r][j] = __builtin_amdgcn_alignbyte(raw[j + 1], raw[j], (uint32_t)at[r] & 3u);
                }
                __syncthreads();   // the columns take the place of the bytes; from here on a wavefront has its own
                TinyState &L = sh.lds.merge.tiny[wv];
#pragma unroll 1
                for (int r = 0; r * kGroupThreads < n_short; ++r) {
                    uint32_t ww[4] = {w[0][0], w[0][1], w[0][2], w[0][3]};
                    int a0 = at[0], nn = n[0];
#pragma unroll
                    for (int q = 1; q < ROUNDS; ++q) {
                        const bool on = r == q;
#pragma unroll
                        for (int j = 0; j < 4; ++j) ww[j] = on ? w[q][j] : ww[j];
                        a0 = on ? at[q] : a0;
                        nn = on ? n[q] : nn;
                    }
                    alive = tiny_merge(p, L, ww, nn, nn > 0);
                    if (parked) tiny_store(L, alive, p.scratch + origin + a0);
                    if (nn > 0) sh.entry[r * kGroupThreads + tid - first_wave * kWave] = (uint32_t)__builtin_popcount(alive);
                }
            }
        }
        if (n_col + n_long) {
            if (!beside || !n_short) __syncthreads();
            merge_listed_pieces(p, sh.lds.merge, sh.tmp, n_col, n_long,
                                [&](int e) -> uint32_t & { return sh.entry[n_short + e]; },
                                [&](int k, int &b, int &n) {
                                    const int at = sh.start[k];
                                    b = origin + at;
                                    n = k0 + k + 1 < n_t ? (int)sh.start[k + 1] - at : end - b;
                                },
                                [&](int e, int, int c) { sh.entry[n_short + e] = (uint32_t)c; });
        }
        if (all) __syncthreads();  // counts
        int c[ROUNDS], inc[ROUNDS];
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            c[r] = slot[r] >= 0 ? (int)sh.entry[slot[r]] : tok0[r] >= 0 ? 1 : n_wide[r];
            inc[r] = wave_scan_inclusive(c[r]);
            if (lane == kWave - 1) sh.total[r * kWavesPerGroup + wv] = (uint32_t)inc[r];
        }
        __syncthreads();
        int32_t *const out = p.scratch2 + r0;
        int first[ROUNDS], sum = done;
#pragma unroll
        for (int k = 0; k < kParts; ++k) {
            if (k % kWavesPerGroup == wv) first[k / kWavesPerGroup] = sum + inc[k / kWavesPerGroup] - c[k / kWavesPerGroup];
            sum += (int)sh.total[k];
        }
        done = __builtin_amdgcn_readfirstlane(sum);
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if (tok0[r] >= 0) out[first[r]] = tok0[r];
        if (WIDE) {
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                for (uint64_t m = __ballot(n_wide[r] > 0); m;) {
                    const int t = __builtin_ctzll(m);
                    m &= m - 1;
                    copy_words<kWave>(p.scratch + origin + read_lane(s[r], t), out + read_lane(first[r], t), 0, read_lane(n_wide[r], t), lane);
                }
            }
        }
        if (all && !parked) {      // whoever merged a left-over piece stores its tokens: the owner says where
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
                if (slot[r] >= 0) sh.entry[slot[r]] = (uint32_t)first[r];
            __syncthreads();
            if (n_short <= row_pieces(kWavesPerGroup)) {
                const int e = wv * (kWave / kTinyMax) + lane / kTinyMax, j = lane & (kTinyMax - 1);
                if (e < n_short && j < row_n) out[sh.entry[e] + j] = (int)row_sym;
            } else {
                tiny_store(sh.lds.merge.tiny[wv], alive, out + (tid < n_short ? (int)sh.entry[tid] : 0));
            }
        } else if (all) {          // from scratch: the first eight tokens by the owner, the rest by its wavefront
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                const int n = slot[r] >= 0 ? c[r] : 0, at = sh.start[r * kGroupThreads + tid];
                const int32_t *from = p.scratch + origin + at;
                for (int i = 0; i < 8; ++i) {
                    if (!__ballot(i < n)) break;
                    if (i < n) out[first[r] + i] = from[i];
                }
                for (uint64_t m = __ballot(n > 8); m;) {
                    const int t = __builtin_ctzll(m);
                    m &= m - 1;
                    copy_words<kWave>(p.scratch + origin + read_lane(at, t), out + read_lane(first[r], t), 8, read_lane(n, t), lane);
                }
            }
        }
        // The first token of every piece that starts in the tile, counted from the tile's first.  (Fewer than
        // 2^16 before any piece: they belong to bytes of the tile.)
        if (any_seq) {
            __syncthreads();
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
                if (r * kGroupThreads + tid < n_here) sh.start[r * kGroupThreads + tid] = (uint16_t)first[r];
            __syncthreads();
            for (int64_t q = (int64_t)s0 + tid; q < s1; q += kGroupThreads) {
                const int sv = p.seq_off[q];
                if (sv < lo || sv >= hi) continue;
                const uint32_t at = (uint32_t)sv + mis - v0, g = sh.group[at >> 4];
                const int k = (int)(g >> 16) + __builtin_popcount(g & ((1u << (at & 15)) - 1u)) - k0;
                if (k >= 0 && k < n_here) p.seq_token_offsets[q] = (int)sh.start[k];
            }
        }
    }
    if (tid == 0) {
        p.tile_sum[tile] = done;
        *info = make_int2(r0, s0);
        if (tile == (int)gridDim.x - 1) info[1] = make_int2(0, s1);
    }
}

// A few very long pieces: what of them has more symbols than four wavefronts keep resident is merged ahead of the tiles
// by 16 (see merge_wide_kernel): parts, or pieces of up to kWideWhole bytes that little would be gained by cutting.  A
// launch more, but four wavefronts take twice the time for a part that long, and in a tile one part waits for the other.  (The
// lines on the number of pieces and on the workspace leave at most 2 MB of input, so positions fit 32 bits.)
// Per call, 16 wavefronts per piece / every piece cut / now, 50k table: text, 24 KB in pieces of 2,358 bytes 107 / 19 / 20 us, 800 KB
// of 4,090 169 / 26 / 25, 40 KB of 20,000 507 / 19 / 20; with runs and random bytes, 100k table, 800 KB of 4,090 4,165 / 80 / 79;
// text without spaces 24 KB of 2,358 298 / 659 / 307, 800 KB of 4,090 457 / 1,073 / 467, 40 KB of 20,000 2,490 / 620 / 620; random bytes, 100k
// table, 800 KB of 4,090 850 / 3,470 / 860; runs of 200 bytes, 100k table, 800 KB of 4,090 530 / 1,001 / 629.
constexpr int kWideSpan = 4 * kWideThreads;
constexpr int kWideParts = kWideWhole / (kGroupBoundMax + 1);
static_assert(kWideSpan < 2 * (kGroupBoundMax + 1), "one part that long lies inside a span, and another one reaches out of it");
static_assert(kWideWhole + 3 <= 8 * kWideThreads, "eight bytes per thread");

// Bit j set: a part may start at byte v + j of the word.  Positions v are counted from the 16-byte boundary at or below the
// input, mis: byte 0.  (A word that holds a byte of the input lies in that byte's page.)  n_equal: see cuts_in_group.
__device__ __forceinline__ uint32_t cuts_in_word(const EncodeParams &p, const uint8_t *code, int mis, int v, int &n_equal) {
    const int v_end = p.n_bytes + mis;
    n_equal = 0;
    if (v >= v_end) return 0u;
    const uint32_t w = *(const uint32_t *)(p.bytes - mis + v);
    uint32_t last = v > mis ? p.bytes[v - 1 - mis] : 0u, last_code = code[last], m = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t b = (w >> (8 * j)) & 0xFFu, c = code[b];
        const uint32_t cut = ((c & kCutBefore) | (last_code & kCutBehind) >> 1) & ~(b == last ? c >> 2 : 0u);
        if (v + j > mis && v + j < v_end) m |= cut << j;
        n_equal += b == last;
        last = b;
        last_code = c;
    }
    return m;
}

struct WideParts {
    uint8_t code[256];
    int2 part[kWideParts + 1 + 2];                 // what the workgroup merges: first byte, length
    int n_parts;
};

// Lists the parts that long of the piece [b, e), if that has no more than kWideWhole bytes.  Where at least half of it are
// parts of more bytes than a column takes, and it is not runs (the rule of the tiles), it is listed as a whole: its parts
// would wait for each other in their tile.  scratch2[first byte] is its number of tokens then, and otherwise ~(number of tokens
// of its first part, if that is one of the long ones).  tile_sum[t] of every tile that starts inside a piece: 1 if that piece is
// merged as a whole.
// at_b: the piece's first byte if its word in scratch2 is of that kind, else -1.  Returns whether it is the whole piece.
__device__ __forceinline__ bool list_piece_parts(const EncodeParams &p, int b, int e, int tile_bytes, WideParts &sh, const WideScope &sc, int &at_b) {
    const int tid = threadIdx.x, mis = p.tile_shift;
    at_b = -1;
    if (b < 0 || e <= b || e > p.n_bytes) return false;
    const int len = e - b;
    bool whole = false;
    if (len > kGroupBoundMax && len <= kWideWhole) {
        const int v = ((b + mis) & ~3) + 8 * tid, at = v - mis - b;        // at: counted from the piece's first byte
        int equal0, equal1;
        uint32_t m = cuts_in_word(p, sh.code, mis, v, equal0);
        m |= cuts_in_word(p, sh.code, mis, v + 4, equal1) << 4;
        auto below = [&](int limit) { return limit <= at ? 0u : limit - at >= 8 ? 0xFFu : (1u << (limit - at)) - 1u; };
        m &= below(len) & ~below(1);
        if (at <= 0 && at > -8) m |= 1u << -at;    // the piece's own start
        const int last = m ? at + 31 - __builtin_clz(m) : -1;
        const int before = sc.scan_max_excl(last), last_of_all = sc.max_all(last);
        const int first = at + __builtin_ctz(m | 256u);
        const int gap = m && before >= 0 ? first - before : 0;             // the part that ends here
        if (gap > kGroupBoundMax) sh.part[atomicAdd(&sh.n_parts, 1)] = make_int2(b + before, gap);
        if (tid == 0 && len - last_of_all > kGroupBoundMax) sh.part[atomicAdd(&sh.n_parts, 1)] = make_int2(b + last_of_all, len - last_of_all);
        const int end_gap = tid == 0 ? len - last_of_all : 0;
        // bytes of long parts | eights of equal bytes << 14 | long parts << 24
        constexpr int kOnePart = 1 << 24, kOneRun = 1 << 14;
        static_assert(kWideWhole < kOneRun && kWideWhole / kColumnMax < 128, "the sums fit");
        int sums;
        (void)sc.scan_sum_excl((gap > kColumnMax ? kOnePart + gap : 0) + (end_gap > kColumnMax ? kOnePart + end_gap : 0) +
                               (at < len && equal0 + equal1 > 6 ? kOneRun : 0), sums);
        sc.sync();
        whole = sums >= 2 * kOnePart && 2 * (sums & (kOneRun - 1)) >= len && 64 * ((sums / kOneRun) & (kOnePart / kOneRun - 1)) <= len;
        if (tid == 0) {
            if (whole) { sh.part[0] = make_int2(b, len); sh.n_parts = 1; }
            else p.scratch2[b] = ~0;
        }
        at_b = b;
    }
    for (int t = (b + mis) / tile_bytes + 1 + tid; t <= (e - 1 + mis) / tile_bytes; t += kWideThreads) p.tile_sum[t] = whole;
    return whole;
}

// Lists the parts that long of pieces beyond kWideWhole that start in span `span` of kWideSpan bytes; text has none.
// [sv, next): the thread's piece (sv < 0: it has none).
__device__ __forceinline__ void list_span_parts(const EncodeParams &p, int span, int sv, int next, WideParts &sh, const WideScope &sc) {
    __shared__ uint32_t bits[kWideSpan / 32];      // bytes of the span that pieces start with
    __shared__ int2 longer[2];                     // the pieces of that many bytes that the span holds bytes of
    __shared__ int n_longer, next_piece;
    const int tid = threadIdx.x, mis = p.tile_shift, v_end = p.n_bytes + mis;
    const int v0 = span * kWideSpan, lo = max(v0, mis), hi = min(v0 + kWideSpan, v_end);
    if (lo >= hi) return;
    if (tid < kWideSpan / 32) bits[tid] = 0;
    if (tid == 0) { n_longer = 0; next_piece = v_end; }
    __syncthreads();
    if (sv >= 0 && sv < p.n_bytes) {
        const int v = sv + mis;
        if (v >= lo && v < hi) atomicOr(&bits[(v - v0) >> 5], 1u << ((v - v0) & 31));
        if (v >= hi) atomicMin(&next_piece, v);
        if (next <= p.n_bytes && next - sv > kWideWhole && v < hi && next + mis > lo) {
            const int at = atomicAdd(&n_longer, 1);
            if (at < 2) longer[at] = make_int2(v, next + mis);             // (more than two only if the offsets decrease)
        }
    }
    __syncthreads();
    const int n_pieces = __builtin_amdgcn_readfirstlane(min(n_longer, 2));
    if (n_pieces == 0) return;
    if (lo == mis && tid == 0) atomicOr(&bits[(mis - v0) >> 5], 1u << ((mis - v0) & 31));      // byte 0 starts a piece
    __syncthreads();
    auto of_longer = [&](int v) { return (v >= longer[0].x && v < longer[0].y) || (n_pieces == 2 && v >= longer[1].x && v < longer[1].y); };
    int n_equal;
    const uint32_t mask = cuts_in_word(p, sh.code, mis, v0 + 4 * tid, n_equal) | ((bits[tid >> 3] >> (4 * (tid & 7))) & 15u);
    const int last = mask ? 4 * tid + 31 - __builtin_clz(mask) : -1;
    const int before = sc.scan_max_excl(last);
    const int last_of_all = sc.max_all(last);
    if (last_of_all < 0) return;                   // (the same in every thread)
    if (mask && before >= 0) {
        const int n = 4 * tid + __builtin_ctz(mask) - before;
        if (n > kGroupBoundMax && of_longer(v0 + before)) sh.part[atomicAdd(&sh.n_parts, 1)] = make_int2(v0 + before - mis, n);
    }
    // the end of the last one: the next start behind the span
    int end = next_piece;
    for (int v = v0 + kWideSpan; v < end; v += kWideSpan) {
        const uint32_t m = cuts_in_word(p, sh.code, mis, v + 4 * tid, n_equal);
        __syncthreads();                           // (between two uses of the scope's words)
        const int at = -sc.max_all(m ? -(v + 4 * tid + __builtin_ctz(m)) : -0x7FFFFFFF);
        end = min(end, at);
        if (at != 0x7FFFFFFF) break;
    }
    __syncthreads();
    const int first = v0 + last_of_all;
    if (tid == 0 && end - first > kGroupBoundMax && of_longer(first)) sh.part[sh.n_parts++] = make_int2(first - mis, end - first);
}

// Workgroup i takes piece i, and if some piece is longer than kWideWhole, span i, too.  Number of tokens in scratch2[first byte].
// (A workgroup for each: 800 KB of text in pieces of 4,090 bytes 28.0 us, the 390 of them are more than the chip holds at once.)
__device__ __forceinline__ void merge_uncut_parts(const EncodeParams &p, const CutSets &cuts, int tile_bytes, uint32_t *X, WideTmp &tmp) {
    __shared__ WideParts sh;
    const int tid = threadIdx.x;
    const WideScope sc{tmp};
    const int i0 = min((int)blockIdx.x, p.n_seqs - 1);
    const int b0 = p.seq_off[i0], e0 = p.seq_off[i0 + 1];      // (asked for ahead of the others)
    static_assert(kWideMaxPieces <= kWideThreads, "a piece per thread");
    int sv = -1, next = -1;
    if (tid < p.n_seqs) { sv = p.seq_off[tid]; next = p.seq_off[tid + 1]; }
    bool longer = (int64_t)next - sv > kWideWhole;
    if (tid < 256) sh.code[tid] = (uint8_t)cut_code(cuts, (uint32_t)tid);
    if (tid == 0) sh.n_parts = 0;
    longer = __syncthreads_or(longer);
    int at_b = -1;
    bool whole = false;
    if ((int)blockIdx.x < p.n_seqs) whole = list_piece_parts(p, b0, e0, tile_bytes, sh, sc, at_b);
    if (longer) {
        __syncthreads();
        list_span_parts(p, blockIdx.x, sv, next, sh, sc);
    }
    __syncthreads();
    const int n = __builtin_amdgcn_readfirstlane(sh.n_parts);
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const int b = __builtin_amdgcn_readfirstlane(sh.part[i].x), len = __builtin_amdgcn_readfirstlane(sh.part[i].y);
        const int c = merge_wide_piece(p, b, len, X, sc);
        __syncthreads();
        if (tid == 0) p.scratch2[b] = b == at_b && !whole ? ~c : c;
    }
}

// Offsets that are out of range or decrease.  Every tile has searched them for its own part, what the tiles found
// need not fit together, and parts that overlap can have more tokens than out_ids has room for.  So all of it is
// dropped and the pieces are encoded as they stand, an equal share by every workgroup, one piece after the other; the last
// workgroup to finish puts the tokens in their place.  A piece whose own offsets are bad yields none, as on the other paths.
// (n_done: 0 at the start of the launch.)
constexpr int kUncutResident = 1020;           // symbols in LDS: 16 KiB, so that the copies keep eight workgroups per compute unit
struct UncutShared {
    uint32_t X[4 * kUncutResident];
    GroupTmp tmp;
    int last;
};
__device__ __forceinline__ void encode_pieces_uncut(const EncodeParams &p, UncutShared &sh, int *n_done) {
    const int tid = threadIdx.x, lane = lane_id();
    const int64_t share = ((int64_t)p.n_seqs + gridDim.x - 1) / gridDim.x;
    const int q0 = (int)min(blockIdx.x * share, (int64_t)p.n_seqs), q1 = (int)min(q0 + share, (int64_t)p.n_seqs);
#pragma unroll 1
    for (int q = q0; q < q1; ++q) {
        const int b = __builtin_amdgcn_readfirstlane(p.seq_off[q]), e = __builtin_amdgcn_readfirstlane(p.seq_off[q + 1]);
        const bool bad = b < 0 || e < b || e > p.n_bytes || (q == 0 && b != 0) || (q == p.n_seqs - 1 && e != p.n_bytes);
        const int len = bad ? 0 : e - b;
        int c = 0;
        if (len > 0) {
            if (p.level >= 3 && !(p.runs_by_best_rank && piece_is_run_like(p, b, len, GroupScope{sh.tmp})))
                c = encode_long_piece_bound(p, b, len, sh.X, kUncutResident, GroupScope{sh.tmp});
            else c = encode_group_piece<int32_t *>(p, b, len, p.scratch + b, p.scratch2 + b, sh.tmp);
        }
        if (tid == 0) p.seq_token_offsets[q] = c;
    }
    __threadfence();
    __syncthreads();
    if (tid == 0) sh.last = atomicAdd(n_done, 1) == (int)gridDim.x - 1;
    __syncthreads();
    if (!sh.last) return;
    __threadfence();
    constexpr int kOwn = 16;       // tokens that a thread copies itself
    int base = 0;
    for (int64_t k = tid; k - tid < p.n_seqs; k += kGroupThreads) {
        const bool has_piece = k < p.n_seqs;
        const int c = has_piece ? p.seq_token_offsets[k] : 0, o = has_piece ? p.seq_off[k] : 0;
        int total;
        const int first = base + group_scan_sum_excl(c, sh.tmp, total);
        if (has_piece) p.seq_token_offsets[k] = first;
        const int n = copy_count(p, c, o, first);
        for (int i = 0; i < min(n, kOwn); ++i) p.out_ids[first + i] = p.scratch[o + i];
        for (uint64_t m = __ballot(n > kOwn); m;) {
            const int t = __builtin_ctzll(m);
            m &= m - 1;
            copy_tokens<kWave>(p, read_lane(o, t), read_lane(first, t), kOwn, read_lane(n, t), lane);
        }
        base += total;
        __syncthreads();           // (the scan's words are free)
    }
    if (tid == 0) {
        p.seq_token_offsets[p.n_seqs] = base;
        mark_call(p.status, p.call_id);
    }
}

// The packed tokens of the tiles to their place in out_ids, and the token offsets of the pieces from
// "in the tile" to "in the output".  A wavefront copies a tile.
constexpr int kCopyTiles = kWavesPerGroup;
__global__ void __launch_bounds__(kGroupThreads) emit_cut_tiles_kernel(EncodeParams p, int n_tiles, int self_scan) {
    __shared__ int before_w[kWavesPerGroup], tile_n[kCopyTiles];
    __shared__ UncutShared uncut;
    const int tid = threadIdx.x, lane = lane_id(), wv = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int tile0 = blockIdx.x * kCopyTiles, tile = tile0 + wv;
    // (the verdict can be that of an earlier replay of a recorded call: the workgroup looks for itself)
    if (p.status[kStatusBadInput] == p.call_id && offsets_are_bad(p.seq_off, p.n_seqs, p.n_bytes)) {
        encode_pieces_uncut(p, uncut, &p.tile_info[n_tiles].x);
        return;
    }
    int n = 0;
    int2 info = make_int2(0, 0);
    int s_end = 0;
    if (tile < n_tiles) {
        n = p.tile_sum[tile];
        info = p.tile_info[tile];
        s_end = p.tile_info[tile + 1].y;
    }
    // tokens before the workgroup's tiles
    int before = 0;
    if (self_scan) {               // tile_sum is 256-byte aligned
        for (int t = tid * 4; t < tile0; t += kGroupThreads * 4) {     // (tile0 is a multiple of 4)
            const int4 a = *(const int4 *)(p.tile_sum + t);
            before += a.x + a.y + a.z + a.w;
        }
        before = __builtin_amdgcn_readlane(wave_scan_inclusive(before), kWave - 1);
    } else {
        before = wv == 0 ? p.tile_base[tile0] : 0;
    }
    n = __builtin_amdgcn_readfirstlane(n);
    if (lane == 0) { before_w[wv] = before; tile_n[wv] = n; }
    __syncthreads();
    int base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) {
        base += before_w[w] + (w < wv ? tile_n[w] : 0);
        total += before_w[w] + tile_n[w];
    }
    const int32_t *src = p.scratch2 + info.x;
    int32_t *dst = p.out_ids + base;
    constexpr int kAtOnce = 4;     // 16-byte loads in flight per thread
    for (int i0 = 4 * lane; i0 < n; i0 += kAtOnce * 4 * kWave) {
        int4_any v[kAtOnce];
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u) {
            const int i = i0 + u * 4 * kWave;
            if (i + 4 <= n) {
                v[u] = *(const int4_any *)(src + i);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[u][j] = i + j < n ? src[i + j] : 0;
            }
        }
#pragma unroll
        for (int u = 0; u < kAtOnce; ++u) {
            const int i = i0 + u * 4 * kWave;
            if (i + 4 <= n) {
                *(int4_any *)(dst + i) = v[u];
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (i + j < n) dst[i + j] = v[u][j];
            }
        }
    }
    for (int64_t s = (int64_t)info.y + lane; s < s_end; s += kWave) p.seq_token_offsets[s] += base;
    if (tile0 + kCopyTiles >= n_tiles) {           // the last tiles: the closing entry, and pieces that start behind the last byte
        for (int64_t s = (int64_t)p.tile_info[n_tiles].y + tid; s <= p.n_seqs; s += kGroupThreads) p.seq_token_offsets[s] = total;
    }
    if (tile0 == 0 && tid == 0) mark_call(p.status, p.call_id);
}

}  // namespace bpe
