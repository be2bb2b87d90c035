// Host-only check of the autotuner's kept sizes (compiled with g++ by
// tests/test_tune_host.py; no GPU).
#include <cstdio>

#include "sg_tune.h"

#define CHECK(x)                                                   \
    do {                                                           \
        if (!(x)) {                                                \
            std::printf("FAIL line %d: %s\n", __LINE__, #x);       \
            return 1;                                              \
        }                                                          \
    } while (0)

int main()
{
    const size_t cap = 159 * 1024;
    const int cu = 256;
    auto key = [&](int units, size_t lds, size_t waves_lds) {
        return sg::tune_key(512, 3000, 2, true, units, cu, lds, lds + waves_lds, cap);
    };
    sg::TuneCache C;
    auto any = [](int) { return true; };
    // 300 units of 80 KB: two of them on some CUs, and twice the size fits
    const sg::TuneKey k = key(300, 80 * 1024, 8192);
    CHECK(C.find(k, any) == -1);
    C.put(k, 1024);
    CHECK(C.find(k, any) == 1024);
    CHECK(C.find(key(300, 80 * 1024, 8192), any) == 1024);
    CHECK(C.find(key(512, 81 * 1024, 8192), any) == (cap / (81 * 1024) == cap / (80 * 1024) ? 1024 : -1));
    // the same number of spins in a graph of larger degree: twice the size does not fit
    CHECK(C.find(key(300, 157 * 1024, 8192), any) == -1);
    // one unit a CU, and units of which a CU holds more: other sizes are best
    CHECK(C.find(key(1, 80 * 1024, 8192), any) == -1);
    CHECK(C.find(key(256, 80 * 1024, 8192), any) == -1);
    CHECK(C.find(key(300, 20 * 1024, 8192), any) == -1);
    // a kept size that does not fit this group is not used, whatever the key says
    CHECK(C.find(k, [](int th) { return th < 1024; }) == -1);
    // no size found: tried again
    const sg::TuneKey one = key(1, 80 * 1024, 8192);
    C.put(one, -1);
    CHECK(C.find(one, any) == -1);
    // sizes of one octave are alike, others not
    auto of_n = [&](int n) { return sg::tune_key(512, n, 2, true, 300, cu, 80 * 1024, 88 * 1024, cap); };
    CHECK(C.find(of_n(2048), any) == 1024 && C.find(of_n(4095), any) == 1024);
    CHECK(C.find(of_n(2047), any) == -1 && C.find(of_n(4096), any) == -1);
    std::printf("tune ok\n");
    return 0;
}
