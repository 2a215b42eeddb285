// Merge-table validation, host slot image, device upload and the stand-alone
// pair-lookup kernel.  In the host image keys and values are the packed 64-bit
// words of the paper's section 3.3; the placement is two-choice instead of linear
// probing, and the device copy keeps 8 bytes per slot (see TableView).
#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "bpe_common.h"

namespace bpe {

static thread_local char g_error[512] = "";

// Identifier of one call of the library, never 0 in its low 30 bits: the kernels of a call stamp the flags
// they leave in a workspace with it, so that flags of earlier calls read as unset without any clearing.
static std::atomic<int32_t> g_call_id{1};

int32_t next_call_id() {
    int32_t id;
    do {
        const uint32_t n = (uint32_t)g_call_id.fetch_add(1);
        id = (int32_t)((n * 0x9E3779B1u) ^ 0x7F4A7C15u);
    } while ((id & 0x3FFFFFFF) == 0);
    return id;
}

void set_error(const char *fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_error, sizeof(g_error), fmt, ap);
    va_end(ap);
}

int hip_fail(hipError_t e, const char *what) {
    set_error("%s: %s", what, hipGetErrorString(e));
    return BPE_ERR_HIP;
}

__global__ void __launch_bounds__(256) lookup_kernel(TableView t, int32_t max_id, const int32_t *pairs,
                                                    int64_t n, int32_t *out_rank, int32_t *out_merged) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t a = pairs[2 * i], b = pairs[2 * i + 1];
    int32_t rank = -1, merged = -1;
    if (a >= 0 && b >= 0 && a <= max_id && b <= max_id) {
        const uint32_t r = table_find(t, (uint32_t)a, (uint32_t)b);
        if (r != kNoRank) { rank = t.rank_of[r >> kRankShift]; merged = (int32_t)merged_id_of(t, r >> kRankShift); }
    }
    out_rank[i] = rank;
    out_merged[i] = merged;
}

static int log2_exact(int64_t v) {
    int l = 0;
    while ((1ll << l) < v) ++l;
    return l;
}

struct HostImage {
    std::vector<uint64_t> slots;        // 2 words per slot
    std::vector<uint32_t> byte_pairs;   // rank word per pair of bytes
    std::vector<int32_t> merged_of, rank_of;
    std::vector<uint32_t> sym_lr;       // 2 words per id: lowest rank order of a rule with the id as right / left part
    bpe_table_info_t info;
    int32_t merged_delta;
};

// Place every key at one of its two slots; evict and re-place along the way.
static bool place_all(const std::vector<uint64_t> &keys, const std::vector<uint64_t> &vals, int64_t half,
                      int index_bits, const HashSeed &seed, std::vector<uint64_t> &slots) {
    const int low_bits = 24 - index_bits;
    std::fill(slots.begin(), slots.end(), ~0ull);
    for (size_t i = 0; i < keys.size(); ++i) {
        uint64_t key = keys[i], val = vals[i];
        int side = 0;
        bool placed = false;
        for (int kick = 0; kick < 1000; ++kick) {
            const uint32_t a = (uint32_t)(key >> 32), b = (uint32_t)key;
            const uint64_t p1 = slot_of(mix1(seed, a, b), low_bits, index_bits);
            const uint64_t p2 = (uint64_t)half + slot_of(mix2(seed, a, b), low_bits, index_bits);
            if (kick == 0 && slots[2 * p1] == kEmptyKey) { slots[2 * p1] = key; slots[2 * p1 + 1] = val; placed = true; break; }
            if (kick == 0 && slots[2 * p2] == kEmptyKey) { slots[2 * p2] = key; slots[2 * p2 + 1] = val; placed = true; break; }
            const uint64_t p = side == 0 ? p1 : p2;
            std::swap(key, slots[2 * p]);
            std::swap(val, slots[2 * p + 1]);
            if (key == kEmptyKey) { placed = true; break; }
            side ^= 1;     // the evicted key goes to its slot in the other half
        }
        if (!placed) return false;
    }
    return true;
}

int check_device(int device, const char *what) {
    int cur = -1;
    const hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (cur != device) {
        set_error("%s lives on device %d but the current device is %d", what, device, cur);
        return BPE_ERR_HIP;
    }
    return BPE_OK;
}

int order_rules(const int32_t *merges, const int32_t *ranks, const int32_t *merged_ids, int64_t n, RuleOrder &ro) {
    if (n < 0 || n >= (1ll << kMaxRulesLog2)) { set_error("n_merges %lld out of range", (long long)n); return BPE_ERR_SIZE; }
    if (n > 0 && !merges) { set_error("null pointer"); return BPE_ERR_NULL; }
    // rows in rank order; ranks unique and non-negative
    std::vector<std::pair<int64_t, int64_t>> &by_rank = ro.by_rank;
    by_rank.assign((size_t)n, {0, 0});
    for (int64_t i = 0; i < n; ++i) {
        const int64_t r = ranks ? ranks[i] : i;
        if (r < 0) { set_error("rank %lld of rule %lld is negative", (long long)r, (long long)i); return BPE_ERR_DUP_RANK; }
        by_rank[i] = {r, i};
    }
    std::sort(by_rank.begin(), by_rank.end());
    for (int64_t i = 1; i < n; ++i)
        if (by_rank[i].first == by_rank[i - 1].first) { set_error("rank %lld appears twice", (long long)by_rank[i].first); return BPE_ERR_DUP_RANK; }

    // merged ids: >= 256, < 2^24, unique; remember the rank order that makes each id
    int64_t max_id = 255;
    std::vector<int64_t> &merged_row = ro.merged_row;
    merged_row.assign((size_t)n, 0);
    for (int64_t i = 0; i < n; ++i) {
        const int64_t m = merged_ids ? (int64_t)merged_ids[i] : 256 + (ranks ? (int64_t)ranks[i] : i);
        if (m < 256 || m >= (1ll << kIdBits)) { set_error("merged id %lld of rule %lld is outside [256, 2^24)", (long long)m, (long long)i); return BPE_ERR_ID_RANGE; }
        merged_row[i] = m;
        if (m > max_id) max_id = m;
    }
    ro.max_id = max_id;
    std::vector<int32_t> &made_at = ro.made_at;   // -2 unknown id, -1 byte, else rank order
    made_at.assign((size_t)(max_id + 1), -2);
    for (int b = 0; b < 256; ++b) made_at[b] = -1;
    for (int64_t k = 0; k < n; ++k) {
        const int64_t m = merged_row[by_rank[k].second];
        if (made_at[m] != -2) { set_error("merged id %lld is produced twice", (long long)m); return BPE_ERR_DUP_MERGED; }
        made_at[m] = (int32_t)k;
    }
    // parts must exist and be made by strictly earlier ranks
    for (int64_t k = 0; k < n; ++k) {
        const int64_t i = by_rank[k].second;
        for (int s = 0; s < 2; ++s) {
            const int64_t part = merges[2 * i + s];
            if (part < 0 || part > max_id || made_at[part] == -2) { set_error("rule %lld uses unknown id %lld", (long long)i, (long long)part); return BPE_ERR_ID_RANGE; }
            if (made_at[part] >= k) { set_error("rule %lld (rank %lld) uses id %lld that an equal or later rank makes", (long long)i, (long long)by_rank[k].first, (long long)part); return BPE_ERR_ORDER; }
        }
    }
    return BPE_OK;
}

static int build_image(const int32_t *merges, const int32_t *ranks, const int32_t *merged_ids, int64_t n,
                       HostImage &img, RuleOrder &ro) {
    const int rc = order_rules(merges, ranks, merged_ids, n, ro);
    if (rc != BPE_OK) return rc;
    const std::vector<std::pair<int64_t, int64_t>> &by_rank = ro.by_rank;
    const std::vector<int64_t> &merged_row = ro.merged_row;
    const int64_t max_id = ro.max_id;
    const int64_t cap = bpe_table_capacity(n);
    // keys and values in rank order; duplicates show up as equal neighbours after sorting
    std::vector<uint64_t> keys((size_t)n), vals((size_t)n);
    img.merged_of.assign((size_t)std::max<int64_t>(n, 1), 0);
    img.rank_of.assign((size_t)std::max<int64_t>(n, 1), 0);
    img.byte_pairs.assign(65536, kNoRank);
    img.merged_delta = n > 0 ? (int32_t)merged_row[by_rank[0].second] : 256;
    std::vector<uint8_t> is_left((size_t)(max_id + 1), 0), is_right((size_t)(max_id + 1), 0);
    for (int64_t i = 0; i < n; ++i) { is_left[merges[2 * i]] = 1; is_right[merges[2 * i + 1]] = 1; }
    img.sym_lr.assign(2 * (size_t)(max_id + 1), kNoRank);
    for (int64_t k = 0; k < n; ++k) {
        const int64_t i = by_rank[k].second;
        const uint32_t a = (uint32_t)merges[2 * i], b = (uint32_t)merges[2 * i + 1];
        if (img.sym_lr[2 * (size_t)b] == kNoRank) img.sym_lr[2 * (size_t)b] = (uint32_t)k;          // b as right part
        if (img.sym_lr[2 * (size_t)a + 1] == kNoRank) img.sym_lr[2 * (size_t)a + 1] = (uint32_t)k;  // a as left part
        const uint32_t word = (uint32_t)k | (is_left[merged_row[i]] ? kCanLeft : 0u) |
                              (is_right[merged_row[i]] ? kCanRight : 0u);
        keys[k] = ((uint64_t)a << 32) | b;
        vals[k] = ((uint64_t)merged_row[i] << 32) | (uint64_t)word;
        img.merged_of[k] = (int32_t)merged_row[i];
        img.rank_of[k] = (int32_t)by_rank[k].first;
        if (merged_row[i] != (int64_t)img.merged_delta + k) img.merged_delta = -1;
        if (a < 256 && b < 256) img.byte_pairs[(a << 8) | b] = device_rank_word(word);
    }
    {
        std::vector<uint64_t> sorted(keys);
        std::sort(sorted.begin(), sorted.end());
        for (int64_t k = 1; k < n; ++k)
            if (sorted[k] == sorted[k - 1]) { set_error("pair (%u, %u) appears twice", (uint32_t)(sorted[k] >> 32), (uint32_t)sorted[k]); return BPE_ERR_DUP_PAIR; }
    }
    img.slots.assign((size_t)cap * 2, ~0ull);
    const int64_t half = cap / 2;
    const int index_bits = log2_exact(half);
    int attempt = 0;
    for (; attempt < kHashSeeds; ++attempt)
        if (place_all(keys, vals, half, index_bits, hash_seed(attempt), img.slots)) break;
    if (attempt == kHashSeeds) { set_error("could not place the keys with any of the %d hash seeds", kHashSeeds); return BPE_ERR_SIZE; }
    img.info.n_merges = n;
    img.info.capacity = cap;
    img.info.hash_attempt = attempt;
    img.info.max_id = (int32_t)max_id;
    return BPE_OK;
}

// The pair's rank order by the host image, or -1.
static int64_t image_rank(const HostImage &img, const HashSeed &seed, int index_bits, uint32_t a, uint32_t b) {
    if (a < 256 && b < 256) {
        const uint32_t word = img.byte_pairs[(a << 8) | b];
        return word == kNoRank ? -1 : (int64_t)(word >> kRankShift);
    }
    // (most merged ids are no part of any rule; the slots are the largest of these arrays)
    if (img.sym_lr[2 * (size_t)a + 1] == kNoRank || img.sym_lr[2 * (size_t)b] == kNoRank) return -1;
    const int low_bits = 24 - index_bits;
    const uint64_t key = ((uint64_t)a << 32) | b;
    const uint64_t p1 = slot_of(mix1(seed, a, b), low_bits, index_bits);
    if (img.slots[2 * p1] == key) return (int64_t)(img.slots[2 * p1 + 1] & kRankMask);
    const uint64_t p2 = (uint64_t)img.info.capacity / 2 + slot_of(mix2(seed, a, b), low_bits, index_bits);
    return img.slots[2 * p2] == key ? (int64_t)(img.slots[2 * p2 + 1] & kRankMask) : -1;
}

// The whole-piece table of the device (see WordHash): every byte, and every merged id whose
// expansion fits a slot and merges back to that id.  Rank order: what training merged early
// is frequent, and the first to come gets its first slot, the one a kernel reads first.
// (bpe_table_build takes 2.9 / 5.2 ms for 50,000 / 100,000 rules without this table and 6.0 / 12.2 with it; 9.0 / 15.5
// when every string was merged to see whether it becomes its id.)
struct WordImage {
    std::vector<uint32_t> slots;        // 4 words per slot
    int shift;
};

static void build_words(const int32_t *merges, const RuleOrder &ro, const HostImage &img, WordImage &out) {
    struct Word { uint8_t b[kWordMax]; uint8_t len; };
    const int64_t n = (int64_t)ro.by_rank.size();
    std::vector<Word> made((size_t)n);                 // expansion by rank order; len 0: too long, or not one token
    std::vector<std::pair<Word, uint32_t>> words;      // string, id
    words.reserve((size_t)n + 256);
    for (int b = 0; b < 256; ++b) {
        Word w = {};
        w.b[0] = (uint8_t)b;
        w.len = 1;
        words.push_back({w, (uint32_t)b});
    }
    const HashSeed seed = hash_seed(img.info.hash_attempt);
    const int index_bits = log2_exact(img.info.capacity / 2);
    auto part = [&](int32_t id, int s) { return merges[2 * ro.by_rank[ro.made_at[id]].second + s]; };   // of a merged id
    // Rule k joins a and b, whose strings merge to a and to b when they stand alone: whether nothing merges across
    // their border first.  The merge loop works in rank order (a merged symbol's rules rank behind the one that
    // made it), so a symbol stands there from the rank of its own rule to that of the rule that takes it in.  Left
    // of the border that is a's last byte, then the id that takes it in as its right part, up to a; right of it the
    // same with left parts up to b.  A rule that joins two of them merges if it ranks before both are taken in; of
    // equal ranks the left-most goes first, the left symbol's before the border's, the border's before the right's.
    auto border_holds = [&](int64_t k, int32_t a, int32_t b) {
        int32_t left[kWordMax], right[kWordMax];           // from a, b down to their bytes
        int i = 0, j = 0;
        for (left[0] = a; left[i] >= 256; ++i) left[i + 1] = part(left[i], 1);
        for (right[0] = b; right[j] >= 256; ++j) right[j + 1] = part(right[j], 0);
        while (i > 0 || j > 0) {
            const int64_t left_goes = i > 0 ? ro.made_at[left[i - 1]] : k, right_goes = j > 0 ? ro.made_at[right[j - 1]] : k;
            const int64_t r = image_rank(img, seed, index_bits, (uint32_t)left[i], (uint32_t)right[j]);
            if (r >= 0 && r < left_goes && r <= right_goes) return false;
            i -= left_goes <= right_goes;
            j -= right_goes <= left_goes;
        }
        return true;
    };
    for (int64_t k = 0; k < n; ++k) {
        const int64_t row = ro.by_rank[k].second;
        const int32_t a = merges[2 * row], b = merges[2 * row + 1];
        // Every id is made by one rule, so the string merges to this id only if the parts' strings merge to the parts.
        Word w = {};
        bool fits = true;
        for (int s = 0; s < 2 && fits; ++s) {
            const int32_t at = ro.made_at[s ? b : a];
            Word byte = {};
            byte.b[0] = (uint8_t)(s ? b : a);
            byte.len = 1;
            const Word &src = at < 0 ? byte : made[(size_t)at];
            fits = src.len > 0 && w.len + src.len <= kWordMax;
            if (!fits) break;
            memcpy(w.b + w.len, src.b, src.len);
            w.len = (uint8_t)(w.len + src.len);
        }
        if (!fits) continue;
        if (!border_holds(k, a, b)) continue;
        made[(size_t)k] = w;
        words.push_back({w, (uint32_t)ro.merged_row[row]});
    }
    int bits = 10;
    while ((1ll << bits) < 2 * (int64_t)words.size()) ++bits;      // at most half full
    out.shift = 32 - bits;
    out.slots.assign((size_t)4 << bits, 0u);
    std::vector<int32_t> at((size_t)1 << bits, -1);                // which word a slot holds
    auto hash_of = [&](int32_t i) {
        uint32_t d[3];
        memcpy(d, words[(size_t)i].first.b, kWordMax);
        return word_hash(d[0], d[1], d[2]);
    };
    auto second_of = [&](int32_t i, uint32_t slot) {               // the other slot of word i
        const WordHash h = hash_of(i);
        const uint32_t s1 = word_slot1(h, out.shift);
        return slot == s1 ? word_slot2(h, out.shift) : s1;
    };
    for (int32_t i = 0; i < (int32_t)words.size(); ++i) {
        const WordHash h = hash_of(i);
        const uint32_t s1 = word_slot1(h, out.shift), s2 = word_slot2(h, out.shift);
        if (at[s1] < 0) { at[s1] = i; continue; }
        if (at[s2] < 0) { at[s2] = i; continue; }
        // move words along from the second slot on; if none of a bounded number of moves ends at
        // an empty slot, put everything back and leave this word out
        uint32_t path[64];
        int steps = 0;
        bool free_end = false, seen = false;
        for (path[0] = s2; !free_end && !seen && steps < 63;) {
            const uint32_t next = second_of(at[path[steps]], path[steps]);
            for (int k = 0; k <= steps; ++k) seen |= path[k] == next;
            path[++steps] = next;
            free_end = at[next] < 0;
        }
        if (!free_end) continue;
        for (int k = steps; k > 0; --k) at[path[k]] = at[path[k - 1]];
        at[s2] = i;
    }
    for (size_t s = 0; s < at.size(); ++s) {
        if (at[s] < 0) continue;
        const Word &w = words[(size_t)at[s]].first;
        memcpy(&out.slots[4 * s], w.b, kWordMax);
        out.slots[4 * s + 3] |= words[(size_t)at[s]].second << 8 | w.len;
        const uint32_t s1 = word_slot1(hash_of(at[s]), out.shift);
        if (s1 != s) out.slots[4 * (size_t)s1 + 3] |= kWordMore;
    }
}

// Which bytes a piece can be cut at: from the last byte of every rule's left part and the first one of its right part.
static void build_cuts(const int32_t *merges, const RuleOrder &ro, CutSets &cuts) {
    std::vector<uint8_t> first(ro.made_at.size()), last(ro.made_at.size());
    for (int b = 0; b < 256; ++b) first[b] = last[b] = (uint8_t)b;
    bool follows[256] = {}, leads[256] = {}, twin[256] = {};       // behind another byte; before another one; itself
    for (const auto &rule : ro.by_rank) {
        const int64_t row = rule.second;
        const int32_t a = merges[2 * row], b = merges[2 * row + 1];
        first[ro.merged_row[row]] = first[a];
        last[ro.merged_row[row]] = last[b];
        if (last[a] == first[b]) twin[first[b]] = true;
        else leads[last[a]] = follows[first[b]] = true;
    }
    memset(&cuts, 0, sizeof(cuts));
    for (int b = 0; b < 256; ++b) {
        cuts.before[b >> 5] |= (uint32_t)!follows[b] << (b & 31);
        cuts.behind[b >> 5] |= (uint32_t)!leads[b] << (b & 31);
        cuts.twin[b >> 5] |= (uint32_t)twin[b] << (b & 31);
    }
}

// kNeverJoined for the pairs of bytes x, y such that no rule joins a string that ends with x to one that starts with y.
static void mark_never_joined(const int32_t *merges, const RuleOrder &ro, uint32_t *byte_pairs) {
    std::vector<uint8_t> first(ro.made_at.size()), last(ro.made_at.size()), joined(65536);
    for (int b = 0; b < 256; ++b) first[b] = last[b] = (uint8_t)b;
    for (const auto &rule : ro.by_rank) {
        const int64_t row = rule.second;
        const int32_t a = merges[2 * row], b = merges[2 * row + 1];
        first[ro.merged_row[row]] = first[a];
        last[ro.merged_row[row]] = last[b];
        joined[(size_t)last[a] << 8 | first[b]] = 1;
    }
    for (size_t i = 0; i < joined.size(); ++i)
        if (!joined[i]) byte_pairs[i] = kNeverJoined;
}

// The one allocation of a table on the device: where its arrays start, and its size.
struct DeviceLayout { size_t words, byte_pairs, merged_of, rank_of, sym_lr, total; };     // (the slots are first)

static DeviceLayout device_layout(const HostImage &img, const WordImage &words) {
    const size_t rule_bytes = (img.merged_of.size() * 4 + 255) / 256 * 256;
    DeviceLayout l;
    l.words = (size_t)img.info.capacity * 8;
    l.byte_pairs = l.words + words.slots.size() * 4;
    l.merged_of = l.byte_pairs + img.byte_pairs.size() * 4;
    l.rank_of = l.merged_of + rule_bytes;
    l.sym_lr = l.rank_of + rule_bytes;
    l.total = l.sym_lr + img.sym_lr.size() * 4;
    return l;
}

}  // namespace bpe

using namespace bpe;

extern "C" const char *bpe_last_error(void) { return g_error; }

extern "C" int64_t bpe_table_capacity(int64_t n_merges) {
    if (n_merges < 0 || n_merges >= (1ll << kMaxRulesLog2)) return BPE_ERR_SIZE;
    // Two-choice placement needs a load factor safely below 1/2: at most 0.4.  Never
    // fewer than 2^16 slots per half (1 MiB on the device in all): a device slot keeps
    // 32 bits of its key, the right id (24 bits) and the 24 - log2(half) bits of the
    // mix that the slot index does not hold.
    int64_t cap = 131072;
    while (2 * cap < 5 * n_merges) cap <<= 1;
    return cap;
}

extern "C" int bpe_table_image_build(const int32_t *merges, const int32_t *ranks,
                                     const int32_t *merged_ids, int64_t n, uint64_t *slots,
                                     int64_t capacity_slots, bpe_table_info_t *info) {
    if (!slots) { set_error("null pointer"); return BPE_ERR_NULL; }
    const int64_t cap = bpe_table_capacity(n);
    if (cap < 0) { set_error("n_merges %lld out of range", (long long)n); return BPE_ERR_SIZE; }
    if (capacity_slots != cap) { set_error("capacity_slots must be %lld", (long long)cap); return BPE_ERR_SIZE; }
    HostImage img;
    RuleOrder ro;
    int rc = build_image(merges, ranks, merged_ids, n, img, ro);
    if (rc != BPE_OK) return rc;
    memcpy(slots, img.slots.data(), (size_t)cap * 16);
    if (info) {
        WordImage words;
        build_words(merges, ro, img, words);
        img.info.device_bytes = (int64_t)device_layout(img, words).total;
        *info = img.info;
    }
    return BPE_OK;
}

extern "C" int bpe_table_build(const int32_t *merges, const int32_t *ranks, const int32_t *merged_ids,
                               int64_t n, bpe_table **out_table) {
    if (!out_table) { set_error("out_table is NULL"); return BPE_ERR_NULL; }
    *out_table = nullptr;
    HostImage img;
    RuleOrder ro;
    int rc = build_image(merges, ranks, merged_ids, n, img, ro);
    if (rc != BPE_OK) return rc;
    // device slots: 8 bytes each, from the image's {key, value} pairs
    const int64_t half = img.info.capacity / 2;
    const int index_bits = log2_exact(half), low_bits = 24 - index_bits;
    const HashSeed seed = hash_seed(img.info.hash_attempt);
    WordImage words;
    build_words(merges, ro, img, words);
    const DeviceLayout at = device_layout(img, words);
    img.info.device_bytes = (int64_t)at.total;
    std::vector<char> blob(at.total, 0);
    uint32_t *dev_slots = (uint32_t *)blob.data();
    for (int64_t i = 0; i < img.info.capacity; ++i) {
        const uint64_t key = img.slots[2 * (size_t)i], val = img.slots[2 * (size_t)i + 1];
        uint32_t rest = 0, word = kNoRank;
        if (key != kEmptyKey) {
            const uint32_t a = (uint32_t)(key >> 32), b = (uint32_t)key;
            rest = key_rest(i < half ? mix1(seed, a, b) : mix2(seed, a, b), low_bits, b);
            word = device_rank_word((uint32_t)val);
        }
        dev_slots[2 * (size_t)i] = rest;
        dev_slots[2 * (size_t)i + 1] = word;
    }
    memcpy(blob.data() + at.words, words.slots.data(), words.slots.size() * 4);
    memcpy(blob.data() + at.byte_pairs, img.byte_pairs.data(), img.byte_pairs.size() * 4);
    mark_never_joined(merges, ro, (uint32_t *)(blob.data() + at.byte_pairs));
    memcpy(blob.data() + at.merged_of, img.merged_of.data(), img.merged_of.size() * 4);
    memcpy(blob.data() + at.rank_of, img.rank_of.data(), img.rank_of.size() * 4);
    memcpy(blob.data() + at.sym_lr, img.sym_lr.data(), img.sym_lr.size() * 4);

    bpe_table *t = new (std::nothrow) bpe_table();
    if (!t) { set_error("out of host memory"); return BPE_ERR_SIZE; }
    hipError_t e = hipGetDevice(&t->device);
    if (e != hipSuccess) { delete t; return hip_fail(e, "hipGetDevice"); }
    e = hipMalloc(&t->device_mem, blob.size());
    if (e != hipSuccess) { delete t; return hip_fail(e, "hipMalloc(table)"); }
    e = hipMemcpy(t->device_mem, blob.data(), blob.size(), hipMemcpyHostToDevice);
    if (e != hipSuccess) { (void)hipFree(t->device_mem); delete t; return hip_fail(e, "hipMemcpy(table)"); }
    t->info = img.info;
    build_cuts(merges, ro, t->cuts);
    char *d = (char *)t->device_mem;
    t->view.slots = (const uint2 *)d;
    t->view.words = (const uint4 *)(d + at.words);
    t->view.word_shift = words.shift;
    t->view.byte_pairs = (const uint32_t *)(d + at.byte_pairs);
    t->view.merged_of = (const int32_t *)(d + at.merged_of);
    t->view.rank_of = (const int32_t *)(d + at.rank_of);
    t->view.sym_lr = (const uint2 *)(d + at.sym_lr);
    t->view.max_id = (uint32_t)(img.sym_lr.size() / 2 - 1);
    t->view.half = (uint32_t)half;
    t->view.low_bits = low_bits;
    t->view.index_bits = index_bits;
    t->view.merged_delta = img.merged_delta;
    t->view.seed = seed;
    *out_table = t;
    return BPE_OK;
}

extern "C" int bpe_table_free(bpe_table *t) {
    if (!t) return BPE_OK;
    hipError_t e = hipFree(t->device_mem);
    delete t;
    return e == hipSuccess ? BPE_OK : hip_fail(e, "hipFree(table)");
}

extern "C" int bpe_table_info(const bpe_table *t, bpe_table_info_t *info) {
    if (!t || !info) { set_error("null pointer"); return BPE_ERR_NULL; }
    *info = t->info;
    return BPE_OK;
}

extern "C" int bpe_table_lookup(const bpe_table *t, const int32_t *pairs, int64_t n,
                                int32_t *out_rank, int32_t *out_merged, void *stream) {
    if (!t || (n > 0 && (!pairs || !out_rank || !out_merged))) { set_error("null pointer"); return BPE_ERR_NULL; }
    if (n < 0 || n > 0x7FFFFFFFll * 128) { set_error("n out of range"); return BPE_ERR_SIZE; }
    if (n == 0) return BPE_OK;
    const int dev_rc = check_device(t->device, "the table");
    if (dev_rc != BPE_OK) return dev_rc;
    const unsigned grid = (unsigned)((n + 255) / 256);
    hipLaunchKernelGGL(lookup_kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, t->view, t->info.max_id,
                       pairs, n, out_rank, out_merged);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? BPE_OK : hip_fail(e, "lookup_kernel launch");
}
