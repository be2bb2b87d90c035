// Host-only check of a measurement's way to host memory (compiled with g++ by
// tests/test_stage_host.py; no GPU): a stand-in for the device copies between
// ordinary arrays and refuses what the device's calls refuse.
#include <cstdio>
#include <cstring>
#include <vector>

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
    sg::HostBlock get(size_t) { return sg::HostBlock{log, 1}; }
    void put(const sg::HostBlock&) {}
    void pack(const sg::PackList& l, uint32_t*) { log->seen.assign(l.seg, l.seg + l.n); }
    void copy(uint32_t*, const sg::PackSeg&) {}
    void sync() {}
    void sync_quiet() {}
};

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

}  // namespace

int main(int argc, char** argv)
{
    const char* what = argc > 1 ? argv[1] : "";
    int rc = 2;
    if (!std::strcmp(what, "large")) rc = large();
    if (rc == 0) std::printf("stage ok\n");
    return rc;
}
