// Workgroup sizes that the autotuner has found, kept for the process by the shape of
// the launch group.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>
#include <tuple>

namespace sg {

// What the best size depends on: the planned size, the units' size and layout, how
// many of them a CU has to run and how many it holds at once, and whether twice the
// planned size fits.  (The last three: two units of 1024 spins a CU are fastest at 512
// threads and one at 1024; and a group of larger degree, whose entries take more LDS,
// may not fit the size that another of the same number of spins was tuned to.)
struct TuneKey {
    int threads, nlog, rpad, resident, per_cu, held, twice;
    bool operator<(const TuneKey& o) const
    {
        return std::tie(threads, nlog, rpad, resident, per_cu, held, twice) <
               std::tie(o.threads, o.nlog, o.rpad, o.resident, o.per_cu, o.held, o.twice);
    }
};

// lds, lds_twice: bytes of a workgroup at the planned size and at twice that; cap: a
// CU's bytes.
inline TuneKey tune_key(int threads, int32_t n_max, int rpad, bool resident, int units, int n_cu, size_t lds,
                        size_t lds_twice, size_t cap)
{
    TuneKey k;
    k.threads = threads;
    k.nlog = 0;
    while (((int64_t)1 << (k.nlog + 1)) <= n_max) ++k.nlog;
    k.rpad = rpad;
    k.resident = resident ? 1 : 0;
    const int cu = std::max(1, n_cu);
    k.per_cu = std::min(16, (units + cu - 1) / cu);   // (more than a CU holds at once: alike)
    k.held = (int)std::min<size_t>(16, cap / std::max<size_t>(1, lds));
    k.twice = lds_twice <= cap ? 1 : 0;
    return k;
}

class TuneCache {
public:
    // The size found for such a group, or -1: there is none, or fits(size) is false.
    template <class Fits>
    int find(const TuneKey& k, Fits&& fits)
    {
        std::lock_guard<std::mutex> lk(mu_);
        auto it = best_.find(k);
        return it != best_.end() && it->second > 0 && fits(it->second) ? it->second : -1;
    }
    void put(const TuneKey& k, int size)
    {
        std::lock_guard<std::mutex> lk(mu_);
        best_[k] = size;
    }

private:
    std::mutex mu_;
    std::map<TuneKey, int> best_;
};

}  // namespace sg
