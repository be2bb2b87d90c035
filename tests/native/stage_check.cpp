// Host-only check of a measurement's way to host memory (compiled with g++ by
// tests/test_stage_host.py; no GPU): a stand-in for the device copies between
// ordinary arrays and refuses what the device's calls refuse.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>
#include <thread>
#include <vector>

#include "sg_layout.h"
#include "sg_stage.h"

#define CHECK(x)                                                   \
    do {                                                           \
        if (!(x)) {                                                \
            std::printf("FAIL line %d: %s\n", __LINE__, #x);       \
            return 1;                                              \
        }                                                          \
    } while (0)

namespace {

struct Log {
    std::vector<sg::PackSeg> seen;   // the segments of the last pack
};

// Does no copy: for lists whose words exist nowhere.
struct Recorder {
    Log* log;
    sg::HostBlock get(size_t bytes) { return sg::HostBlock{log, bytes}; }
    void put(const sg::HostBlock&) {}
    void pack(const sg::PackList& l, uint32_t*, uint64_t, uint64_t) { log->seen.assign(l.seg, l.seg + l.n); }
    void copy(uint32_t*, const uint32_t*, uint64_t) {}
    void copy_rows(uint32_t*, const sg::PackSeg&) {}
    void store(uint32_t*, const uint32_t*, size_t) {}
    void sync() {}
    void sync_quiet() {}
};

// Copies at once between ordinary arrays.
struct Bad {};
struct Copier {
    size_t limit;   // bytes of a block (0: there are none)
    sg::HostBlock get(size_t bytes)
    {
        const size_t n = bytes < limit ? bytes : limit;
        return n ? sg::HostBlock{std::malloc(n), n} : sg::HostBlock{};
    }
    void put(const sg::HostBlock& b) { std::free(b.p); }
    void pack(const sg::PackList& l, uint32_t* block, uint64_t w0, uint64_t w1)
    {
        for (int s = 0; s < l.n; ++s)
            for (uint64_t i = 0; i < sg::pack_words(l.seg[s]); ++i) {
                const uint64_t w = l.seg[s].dst + i;
                if (w < w0 || w >= w1) continue;
                uint32_t* p = l.seg[s].src + sg::pack_from(l.seg[s], i);
                if (block) block[w - w0] = *p;
                if (l.seg[s].clear) *p = 0u;
            }
    }
    void store(uint32_t* dst, const uint32_t* src, size_t words) { std::memcpy(dst, src, words * 4); }
    void copy(uint32_t* dst, const uint32_t* src, uint64_t words) { std::memcpy(dst, src, words * 4); }
    void copy_rows(uint32_t* dst, const sg::PackSeg& g)
    {
        if (g.stride < g.width) throw Bad{};   // an invalid pitch
        for (uint64_t r = 0; r < g.rows; ++r) std::memcpy(dst + r * g.width, g.src + r * g.stride, g.width * 4);
    }
    void sync() {}
    void sync_quiet() {}
};

// The segments of a measurement, as sg_measure adds them: single words and rows
// without a stride, the first columns of rows, none at all, counts that are cleared.
struct Words {
    std::vector<uint32_t> a, b, c, d, e;
};
template <class Dev>
std::vector<uint32_t> bring(Dev dev, Words& w)
{
    sg::Fetch<Dev> F(dev);
    const int i0 = F.add(w.a.data(), 1, 1, 1);
    const int i1 = F.add(w.b.data(), 1, 14, 0);
    const int i2 = F.add(w.c.data(), 7, 6, 10);
    const int i3 = F.add(w.c.data(), 0, 6, 10);
    const int i4 = F.add(w.d.data(), 9, 3, 5, true);
    const int i5 = F.add(w.d.data(), 9, 0, 5, true);
    const int i6 = F.add(w.e.data(), 5, 4, 4, true);
    const int i7 = F.add(w.b.data() + 14, 1, 186, 0);
    F.run();
    std::vector<uint32_t> out;
    auto take = [&](int i, size_t n) {
        const uint32_t* p = F.template at<uint32_t>(i);
        out.insert(out.end(), p, p + n);
    };
    take(i0, 1);
    take(i1, 14);
    take(i2, 42);
    take(i3, 0);
    take(i4, 27);
    take(i5, 0);
    take(i6, 20);
    take(i7, 186);
    return out;
}
Words some_words()
{
    Words w;
    uint32_t x = 1;
    auto fill = [&](std::vector<uint32_t>& v, size_t n) {
        v.resize(n);
        for (uint32_t& e : v) e = x = x * 1664525u + 1013904223u;
    };
    fill(w.a, 1);
    fill(w.b, 200);
    fill(w.c, 70);
    fill(w.d, 45);
    fill(w.e, 20);
    return w;
}

// Without host memory that the device can write to, the copies bring the same words
// and the counts end up clear.
int plain()
{
    Words v = some_words(), w = v;
    const std::vector<uint32_t> want = bring(Copier{SIZE_MAX}, v);
    std::vector<uint32_t> got;
    try {
        got = bring(Copier{0}, w);
    } catch (const Bad&) {
        CHECK(!"a copy by rows whose pitch is below its width");
    }
    CHECK(want.size() == 290 && got == want);
    CHECK(v.d == w.d && v.e == w.e);
    for (size_t i = 0; i < w.d.size(); ++i) CHECK((w.d[i] == 0) == (i % 5 < 3));
    return 0;
}

// Through a block that is too small, the same words come in pieces.
int pieces()
{
    Words v = some_words();
    const std::vector<uint32_t> want = bring(Copier{SIZE_MAX}, v);
    for (size_t limit = 8; limit < 4 * 300; limit += 8) {
        Words w = some_words();
        CHECK(bring(Copier{limit}, w) == want);
        CHECK(v.d == w.d && v.e == w.e);
    }
    return 0;
}

// The pool holds at most its bound, whoever holds its blocks, and gives memory out
// once.
int pool()
{
    typedef sg::BlockPool P;
    std::atomic<size_t> total{0};
    std::atomic<bool> refuse{false};
    auto alloc = [&](size_t n) -> void* {
        if (refuse) return nullptr;
        total += n;
        return std::malloc(64);   // (its address alone counts)
    };
    {
        P p;
        const sg::HostBlock a = p.get(100, alloc), b = p.get(3 << 20, alloc);
        CHECK(a.p && a.bytes == P::kLeast && b.p && b.bytes == (size_t)4 << 20 && total == a.bytes + b.bytes);
        p.put(b);
        CHECK(p.get(200, alloc).p == b.p);                 // (in use again)
        const sg::HostBlock c = p.get(100 << 20, alloc);   // more than a block
        CHECK(c.p && c.bytes == P::kMost);
        const sg::HostBlock d = p.get(60 << 20, alloc);    // the largest that fits
        CHECK(d.p && d.bytes == (size_t)32 << 20);
        p.put(c);
        p.put(d);
        p.put(a);
        const size_t t = total;
        CHECK(p.get(100 << 20, alloc).p == c.p);           // to be used in pieces
        CHECK(p.get(60 << 20, alloc).p == d.p);
        CHECK(p.get(60000, alloc).p == a.p);
        CHECK(total == t);
        // what is left is given out in ever smaller blocks, then nothing
        size_t n = 0;
        while (p.get(60 << 20, alloc).p) ++n;
        CHECK(n >= 3 && n < 100 && total <= P::kBytes && !p.get(60 << 20, alloc).p);
    }
    {
        P p;
        total = 0;
        refuse = true;
        CHECK(!p.get(P::kMost, alloc).p && !p.get(P::kMost, alloc).p);
        refuse = false;                                    // a refusal leaves nothing reserved
        const sg::HostBlock a = p.get(P::kMost, alloc), b = p.get(P::kMost, alloc);
        CHECK(a.p && a.bytes == P::kMost && b.p && b.bytes == P::kMost);
        CHECK(!p.get(1, alloc).p);
        p.put(a);
        CHECK(p.get(1, alloc).p == a.p);
    }
    {
        P p;
        total = 0;
        std::atomic<int> twice{0};
        std::mutex mu;
        std::set<void*> out;
        std::vector<std::thread> th;
        for (int t = 0; t < 16; ++t)
            th.emplace_back([&, t]() {
                uint32_t x = 12345u + (uint32_t)t;
                std::vector<sg::HostBlock> mine;
                for (int i = 0; i < 4000; ++i) {
                    x = x * 1664525u + 1013904223u;
                    if ((x >> 16 & 1) != 0 && !mine.empty()) {
                        {
                            std::lock_guard<std::mutex> lk(mu);
                            out.erase(mine.back().p);
                        }
                        p.put(mine.back());
                        mine.pop_back();
                        continue;
                    }
                    const sg::HostBlock b = p.get((size_t)1 << (x >> 20 & 31) % 28, alloc);
                    if (!b.p) continue;
                    std::lock_guard<std::mutex> lk(mu);
                    if (!out.insert(b.p).second) ++twice;
                    mine.push_back(b);
                }
                for (const sg::HostBlock& b : mine) {
                    {
                        std::lock_guard<std::mutex> lk(mu);
                        out.erase(b.p);
                    }
                    p.put(b);
                }
            });
        for (auto& x : th) x.join();
        CHECK(twice == 0 && total > 0 && total <= P::kBytes);
    }
    return 0;
}

// Segments past 2^32 words keep their length, their neighbours' places and the
// words they are read from.
int large()
{
    const uint64_t big = ((uint64_t)1 << 32) + 6;
    Log log;
    sg::Fetch<Recorder> F(Recorder{&log});
    F.add(nullptr, 1, 3, 3);
    F.add(nullptr, 1, big, big);                              // one long row
    F.add(nullptr, 1000, ((uint64_t)1 << 32) / 500 + 1, (uint64_t)1 << 33, true);   // long together
    F.add(nullptr, big, 1, 2);                                // many rows
    F.add(nullptr, 1, 2, 2);
    F.run();
    CHECK(log.seen.size() == 5);
    CHECK(sg::pack_words(log.seen[1]) == big);
    CHECK(log.seen[1].dst == 4 && log.seen[2].dst == 4 + big);
    const uint64_t w = ((uint64_t)1 << 32) / 500 + 1;
    CHECK(sg::pack_words(log.seen[2]) == 1000 * w);
    CHECK(log.seen[3].dst == log.seen[2].dst + 1000 * w);
    CHECK(log.seen[4].dst == log.seen[3].dst + big);
    CHECK(log.seen[4].dst % 2 == 0);
    CHECK(sg::pack_from(log.seen[1], big - 1) == big - 1);
    CHECK(sg::pack_from(log.seen[2], 999 * w + 5) == ((uint64_t)999 << 33) + 5);
    CHECK(sg::pack_from(log.seen[3], big - 1) == 2 * (big - 1));
    return 0;
}

// The states of multispin units of different sizes are one range with nothing else
// in it, and no array overlaps another.
int states()
{
    sg::Arena A;
    A.take(1000);
    std::vector<sg::VbmArrays> bytes;
    for (size_t u = 0; u < 40; ++u) bytes.push_back(sg::VbmArrays{8 * (100 + 37 * u), 8 * (400 + 99 * u), 32768});
    const std::vector<sg::VbmArrays> off = sg::vbm_layout(A, bytes);
    CHECK(off.size() == bytes.size());
    size_t lo = SIZE_MAX, hi = 0, sum = 0;
    std::vector<std::pair<size_t, size_t>> all;
    for (size_t u = 0; u < off.size(); ++u) {
        lo = std::min(lo, off[u].state);
        hi = std::max(hi, off[u].state + bytes[u].state);
        sum += (bytes[u].state + 255) / 256 * 256;
        all.push_back({off[u].state, bytes[u].state});
        all.push_back({off[u].jw, bytes[u].jw});
        all.push_back({off[u].thr, bytes[u].thr});
    }
    CHECK(hi - lo <= sum);
    std::sort(all.begin(), all.end());
    for (size_t i = 0; i < all.size(); ++i) {
        CHECK(all[i].first % 256 == 0);
        CHECK(all[i].first + all[i].second <= (i + 1 < all.size() ? all[i + 1].first : A.size));
    }
    CHECK(all[0].first >= 1000);
    return 0;
}

}  // namespace

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    int rc = 2;
    if (!std::strcmp(what, "large")) rc = large();
    if (!std::strcmp(what, "states")) rc = states();
    if (!std::strcmp(what, "plain")) rc = plain();
    if (!std::strcmp(what, "pieces")) rc = pieces();
    if (!std::strcmp(what, "pool")) rc = pool();
    if (rc == 0) std::printf("stage ok\n");
    return rc;
}
