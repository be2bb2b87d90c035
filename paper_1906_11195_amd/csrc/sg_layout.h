// Where the arrays of a context lie in its one device allocation.
#pragma once
#include <cstddef>
#include <vector>

namespace sg {

// One allocation carved into aligned pieces.
struct Arena {
    size_t size = 0;
    size_t take(size_t bytes)
    {
        const size_t off = size;
        size += (bytes + 255) & ~(size_t)255;
        return off;
    }
};

// The arrays of each multispin unit, in bytes and as offsets.
struct VbmArrays {
    size_t state, jw, thr;
};

// The states of all units first, one after another: a measurement copies the spins of
// a context as one range, and nothing else should lie in it (at degree 4 a unit's
// coupling words are four times its state, at degree 32 32 times).
inline std::vector<VbmArrays> vbm_layout(Arena& A, const std::vector<VbmArrays>& bytes)
{
    std::vector<VbmArrays> off(bytes.size());
    for (size_t u = 0; u < bytes.size(); ++u) off[u].state = A.take(bytes[u].state);
    for (size_t u = 0; u < bytes.size(); ++u) {
        off[u].jw = A.take(bytes[u].jw);
        off[u].thr = A.take(bytes[u].thr);
    }
    return off;
}

}  // namespace sg
