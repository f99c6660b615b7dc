// One wave of the sorted conversion's group kernel on the CPU: row tables, merge
// levels and search steps through csrc/merge_search.hpp, every LDS address checked
// against the wave's slice and the words behind it.  Strips that fit their group,
// empty ones, ones with an unsorted row and ones far past the capacity stand side
// by side; the ones that fit must come out sorted.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "merge_search.hpp"

namespace {

constexpr int kWave = 64, E = 8;
constexpr int kSlice = 2 * kWave * E;  // buffers A and B of a wave, in words
constexpr int kPad = kWave * E;        // words behind the last wave's slice

struct Strip {
    std::vector<int> row_ptr;  // strip-relative, nr + 1 of them
    std::vector<uint32_t> words;
    bool fits = false, sorted = true;
};

[[noreturn]] void fail(const char* what, int hb, int g, long long at) {
    std::printf("%s: height bucket %d, %d lanes per strip, %lld\n", what, hb, g, at);
    std::exit(1);
}

Strip make_strip(std::mt19937& rng, int hb, int g, int kind) {
    const auto pick = [&](int lo, int hi) { return lo + static_cast<int>(rng() % static_cast<unsigned>(hi - lo + 1)); };
    Strip s;
    const int nr = pick(1, hb), cap = g * E;
    const int n = kind == 0 ? 0 : kind == 1 ? pick(0, cap) : kind == 2 ? cap : kind == 3 ? cap + pick(1, 40)
                  : kind == 4 ? pick(10000, 200000) : 600000000 + pick(0, 1000);
    s.row_ptr.assign(1, 0);
    for (int r = 1; r < nr; ++r) s.row_ptr.push_back(pick(0, n));
    s.row_ptr.push_back(n);
    std::sort(s.row_ptr.begin(), s.row_ptr.end());
    s.fits = n <= cap;
    if (!s.fits) return s;
    for (int r = 0; r < nr; ++r) {
        std::vector<uint32_t> c;
        for (int i = s.row_ptr[r]; i < s.row_ptr[r + 1]; ++i) c.push_back(static_cast<uint32_t>(pick(0, 300)));
        std::sort(c.begin(), c.end());
        if (c.size() > 1 && kind == 1 && pick(0, 9) == 0 && c.front() < c.back()) {
            std::swap(c.front(), c.back());
            s.sorted = false;
        }
        for (uint32_t x : c) s.words.push_back((x << 5) | static_cast<uint32_t>(r));
    }
    return s;
}

void run_wave(std::mt19937& rng, int hb, int g) {
    const int ng = kWave / g;
    std::vector<Strip> strips;
    for (int k = 0; k < ng; ++k) strips.push_back(make_strip(rng, hb, g, static_cast<int>(rng() % 6)));
    std::vector<uint32_t> lds(kSlice + kPad, 0x5a5a5a5au);
    const auto word = [&](int address) -> uint32_t& {
        if (address < 0 || address % 4 != 0 || address / 4 >= kSlice + kPad) fail("LDS read outside", hb, g, address);
        return lds[static_cast<size_t>(address / 4)];
    };
    std::vector<std::vector<int>> table;
    int row_max = 0, umax = 0;
    for (const Strip& s : strips) {
        const int nr = static_cast<int>(s.row_ptr.size()) - 1, n = s.row_ptr.back();
        std::vector<int> t;
        for (int q = 0; q < hb; ++q) t.push_back(cmrs::row_place(s.fits, q, nr, q < nr ? s.row_ptr[q] : 0, n));
        t.push_back(cmrs::row_place(s.fits, hb, nr, 0, n));
        table.push_back(t);
        if (!s.fits) continue;
        umax = std::max(umax, (n + g - 1) / g);
        if (s.sorted)
            for (int r = 0; r < nr; ++r) row_max = std::max(row_max, s.row_ptr[r + 1] - s.row_ptr[r]);
    }
    struct Entry {
        int group, place, pos;
        uint32_t wd;
    };
    std::vector<Entry> entries;  // every lane's slots, also those without an entry
    for (int k = 0; k < ng; ++k)
        for (int p = 0; p < g * umax; ++p) {
            const bool in = strips[k].fits && p < strips[k].row_ptr.back();
            const uint32_t wd = in ? strips[k].words[static_cast<size_t>(p)] : rng() % static_cast<unsigned>(hb);
            entries.push_back({k, p, p, wd});
            if (in) word(4 * (k * g * E + p)) = wd;
        }
    int a = 0, b = 4 * kWave * E;
    for (int level = 0; (1 << level) < hb; ++level) {
        const int top = cmrs::merge_first_step(std::min(row_max << level, umax * g));
        for (Entry& e : entries) {
            const std::vector<int>& rt = table[static_cast<size_t>(e.group)];
            const int first = a + 4 * e.group * g * E - 4;
            const int partner = (static_cast<int>(e.wd) & (hb - 1) & -(1 << level)) ^ (1 << level);
            const int start = first + 4 * rt[static_cast<size_t>(partner)];
            const int last = first + 4 * rt[static_cast<size_t>(partner + (1 << level))];
            int cur = start;
            for (int step = top; step > 3; step >>= 1) cur = cmrs::merge_step(cur, step, last, word(cur + step) < e.wd);
            e.pos += (cur - ((e.wd >> level) & 1u ? last : start)) >> 2;
        }
        if ((2 << level) < hb)
            for (const Entry& e : entries) {
                const Strip& s = strips[static_cast<size_t>(e.group)];
                if (s.fits && s.sorted && e.place < s.row_ptr.back()) {
                    if (e.pos < 0 || e.pos >= s.row_ptr.back()) fail("place outside the strip", hb, g, e.pos);
                    word(b + 4 * (e.group * g * E + e.pos)) = e.wd;
                }
            }
        std::swap(a, b);
    }
    for (int k = 0; k < ng; ++k) {
        const Strip& s = strips[static_cast<size_t>(k)];
        if (!s.fits || !s.sorted) continue;
        std::vector<uint32_t> got(s.words.size(), ~0u), want = s.words;
        for (const Entry& e : entries)
            if (e.group == k && e.place < s.row_ptr.back()) got.at(static_cast<size_t>(e.pos)) = e.wd;
        std::sort(want.begin(), want.end());
        if (got != want) fail("strip not sorted", hb, g, k);
    }
}

}  // namespace

int main() {
    std::mt19937 rng(12345);
    for (int hb = 1; hb <= 32; hb *= 2)
        for (int g = std::max(hb, 2); g <= kWave; g *= 2)
            for (int t = 0; t < 60; ++t) run_wave(rng, hb, g);
    std::printf("ok\n");
    return 0;
}
