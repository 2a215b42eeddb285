// The whole-piece table (build_words) against its definition, on the CPU: built by tests/test_sanitizers.py with the
// host sanitizers.  Includes the library's source, whose builders are not exported.  Arguments: files of merge rules
// (int32 pairs).  For every table: each slot that is in use holds a string which the merge loop, written out here as
// the paper's sequential loop, turns into exactly the slot's token, at one of the string's two slots, with the mark in
// its first slot where it sits in its second; no string twice; and every byte and every merged id whose expansion
// fits and merges to one token is there, or both its slots are taken.
#include <cstdio>
#include <map>
#include <string>

#include "bpe_table.hip"

#define CHECK(cond) do { if (!(cond)) { std::fprintf(stderr, "check failed, line %d: %s\n", __LINE__, #cond); return 1; } } while (0)

static uint64_t state = 0x9E3779B97F4A7C15ull;
static uint32_t draw(uint32_t n) {
    state ^= state >> 12; state ^= state << 25; state ^= state >> 27;
    return (uint32_t)((state * 0x2545F4914F6CDD1Dull) >> 33) % n;
}

// rules over `letters` bytes from `first` on: each joins two ids that exist before it, short ones more often
static std::vector<int32_t> random_rules(int64_t n, uint32_t first, uint32_t letters) {
    std::vector<int32_t> m;
    std::map<std::pair<int32_t, int32_t>, bool> seen;
    auto pick = [&](int64_t k) {
        const uint32_t r = draw(3) ? draw((uint32_t)std::min<int64_t>(letters + k, letters + 12)) : draw((uint32_t)(letters + k));
        return r < letters ? (int32_t)(first + r) : (int32_t)(256 + r - letters);
    };
    for (int64_t k = 0, tries = 0; k < n && tries < 1000000; ++tries) {
        const int32_t a = pick(k), b = pick(k);
        if (!seen.insert({{a, b}, true}).second) continue;
        m.push_back(a); m.push_back(b);
        ++k;
    }
    return m;
}

static int check(const std::vector<int32_t> &m, const int32_t *ranks, const int32_t *ids, const char *what) {
    const int64_t n = (int64_t)m.size() / 2;
    HostImage img;
    RuleOrder ro;
    CHECK(build_image(m.data(), ranks, ids, n, img, ro) == BPE_OK);
    WordImage words;
    build_words(m.data(), ro, img, words);
    const int bits = 32 - words.shift;
    CHECK(words.slots.size() == (size_t)4 << bits);
    std::map<std::pair<uint32_t, uint32_t>, std::pair<int64_t, uint32_t>> rule;     // pair -> rank order, merged id
    std::map<uint32_t, std::string> expansion;                                     // up to 13 bytes of it
    for (uint32_t b = 0; b < 256; ++b) expansion[b] = std::string(1, (char)b);
    for (int64_t k = 0; k < n; ++k) {
        const int64_t row = ro.by_rank[k].second;
        const uint32_t a = (uint32_t)m[2 * row], b = (uint32_t)m[2 * row + 1], id = (uint32_t)ro.merged_row[row];
        rule[{a, b}] = {k, id};
        expansion[id] = (expansion[a] + expansion[b]).substr(0, kWordMax + 1);
    }
    auto tokens = [&](const std::string &s) {
        std::vector<uint32_t> sym;
        for (char c : s) sym.push_back((uint8_t)c);
        for (;;) {
            int64_t best = -1;
            size_t at = 0;
            uint32_t id = 0;
            for (size_t i = 0; i + 1 < sym.size(); ++i) {
                const auto f = rule.find({sym[i], sym[i + 1]});
                if (f != rule.end() && (best < 0 || f->second.first < best)) { best = f->second.first; at = i; id = f->second.second; }
            }
            if (best < 0) return sym;
            sym[at] = id;
            sym.erase(sym.begin() + (long)at + 1);
        }
    };
    std::map<std::string, uint32_t> stored;
    for (size_t s = 0; s < words.slots.size() / 4; ++s) {
        const uint32_t *w = &words.slots[4 * s];
        const uint32_t len = w[3] & kWordLenMask;
        if (len == 0) { CHECK(w[0] == 0 && w[1] == 0 && w[2] == 0 && (w[3] & ~kWordMore) == 0); continue; }
        CHECK(len <= (uint32_t)kWordMax);
        std::string str((const char *)w, len);
        for (uint32_t i = len; i < (uint32_t)kWordMax; ++i) CHECK(((const char *)w)[i] == 0);
        const std::vector<uint32_t> t = tokens(str);
        CHECK(t.size() == 1 && t[0] == w[3] >> 8);
        const WordHash h = word_hash(w[0], w[1], w[2]);
        const uint32_t s1 = word_slot1(h, words.shift), s2 = word_slot2(h, words.shift);
        CHECK(s1 < 1u << bits && s2 < 1u << bits && (s == s1 || s == s2));
        if (s != s1) CHECK(words.slots[4 * (size_t)s1 + 3] & kWordMore);
        CHECK(stored.insert({str, t[0]}).second);
    }
    size_t missing = 0;
    for (const auto &e : expansion) {
        if (e.second.size() > (size_t)kWordMax || stored.count(e.second)) continue;
        const std::vector<uint32_t> t = tokens(e.second);
        if (t.size() != 1) continue;
        uint32_t d[3] = {0, 0, 0};
        memcpy(d, e.second.data(), e.second.size());
        const WordHash h = word_hash(d[0], d[1], d[2]);
        CHECK(words.slots[4 * (size_t)word_slot1(h, words.shift) + 3] & kWordLenMask);
        CHECK(words.slots[4 * (size_t)word_slot2(h, words.shift) + 3] & kWordLenMask);
        missing += e.second.back() != 0;       // (strings that differ in trailing zero bytes only share both slots)
    }
    CHECK(missing * 50 <= stored.size());      // the table is at most half full: nearly every string finds room
    std::printf("%s: %lld rules, %zu strings, %zu without room\n", what, (long long)n, stored.size(), missing);
    return 0;
}

int main(int argc, char **argv) {
    for (int round = 0; round < 40; ++round)
        for (uint32_t letters : {1u, 2u, 3u, 26u, 256u})
            if (check(random_rules(1 + draw(400), letters == 256 ? 0 : draw(200), letters), nullptr, nullptr, "random")) return 1;
    if (check({}, nullptr, nullptr, "no rules")) return 1;
    {   // ranks, merged ids and row order of the caller's own: sparse ids up to 2^24
        const std::vector<int32_t> m = random_rules(300, 97, 3);
        const int64_t n = (int64_t)m.size() / 2;
        std::vector<int32_t> rows, ranks((size_t)n), ids((size_t)n);
        auto id_of = [&](int32_t id) { return id < 256 ? id : (1 << 24) - 1 - 7 * (id - 256); };
        for (int64_t i = 0; i < n; ++i) {
            const int64_t k = n - 1 - i;
            rows.push_back(id_of(m[2 * k])); rows.push_back(id_of(m[2 * k + 1]));
            ranks[i] = (int32_t)(5 * k + 3);
            ids[i] = id_of((int32_t)(256 + k));
        }
        if (check(rows, ranks.data(), ids.data(), "own ids")) return 1;
    }
    for (int f = 1; f < argc; ++f) {
        FILE *fp = std::fopen(argv[f], "rb");
        CHECK(fp);
        std::vector<int32_t> m(1 << 20);
        m.resize(std::fread(m.data(), 4, m.size(), fp));
        std::fclose(fp);
        if (check(m, nullptr, nullptr, argv[f])) return 1;
    }
    std::puts("whole-piece table under the sanitizers: ok");
    return 0;
}
