// The device words of one measurement on their way to host memory.
//
// A measurement lists the segments it needs (Fetch::add) and brings them over
// together (Fetch::run).  What touches the device is in `Dev`, so that the
// arithmetic and the order of the steps can be checked without one.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <vector>

namespace sg {

// Rows of device words that become consecutive words on the host.  (64 bits: the
// spins of one context can be more than 2^32 words.)
struct PackSeg {
    uint32_t* src;
    uint64_t dst;              // word of the destination
    uint64_t stride;           // words from row to row
    uint64_t rows, width;
    uint32_t clear;            // set the words to zero once read
};
struct PackList {
    PackSeg seg[10];
    int n;
};

constexpr uint64_t pack_words(const PackSeg& g) { return g.rows * g.width; }
// Where word i of a segment is read from, in words from src.
constexpr uint64_t pack_from(const PackSeg& g, uint64_t i)
{
    const uint64_t r = pack_words(g) >> 32 ? i / g.width : (uint32_t)i / (uint32_t)g.width;
    return r * g.stride + (i - r * g.width);
}

// Host memory that the device can write to.
struct HostBlock {
    void* p = nullptr;
    size_t bytes = 0;
};

// Dev:
//   HostBlock get(size_t bytes)         such memory, p null if there is none
//   void put(const HostBlock&)          gives it back (does not throw)
//   void pack(const PackList&, uint32_t* block)   enqueues the copy of all segments
//                                       to their places in the block and the clearing
//                                       (block null: only that)
//   void copy(uint32_t* dst, const uint32_t* src, uint64_t words)    enqueues a copy to
//                                       ordinary memory
//   void copy_rows(uint32_t* dst, const PackSeg&)    the same of a segment's rows
//   void sync()                         waits for what was enqueued
//   void sync_quiet()                   the same on the way out of an error
// All but put and sync_quiet may throw.
template <class Dev>
class Fetch {
public:
    explicit Fetch(Dev dev) : dev_(dev) { list_.n = 0; }
    ~Fetch()
    {
        if (pending_) dev_.sync_quiet();
        dev_.put(block_);
    }
    Fetch(const Fetch&) = delete;
    Fetch& operator=(const Fetch&) = delete;
    // `rows` rows of `width` words, `stride` apart; the index to pass to at()
    int add(const void* src, size_t rows, size_t width, size_t stride, bool clear = false)
    {
        PackSeg& g = list_.seg[list_.n];
        g.src = (uint32_t*)src;
        g.dst = words_;
        g.stride = stride;
        g.rows = rows;
        g.width = width;
        g.clear = clear ? 1u : 0u;
        words_ += (rows * width + 1) & ~(size_t)1;
        return list_.n++;
    }
    // enqueues the copies and waits for them
    void run()
    {
        block_ = dev_.get(std::max<size_t>(8, words_ * 4));
        pending_ = true;
        if (block_.p) {
            dev_.pack(list_, (uint32_t*)block_.p);
            base_ = (const uint32_t*)block_.p;
        } else {
            plain_.resize(std::max<size_t>(2, words_));
            for (int i = 0; i < list_.n; ++i) {
                const PackSeg& g = list_.seg[i];
                uint32_t* dst = plain_.data() + g.dst;
                if (pack_words(g) == 0) continue;
                // (a single row's stride means nothing, and a copy by rows takes none
                // below its width)
                if (g.rows == 1 || g.stride == g.width)
                    dev_.copy(dst, g.src, pack_words(g));
                else
                    dev_.copy_rows(dst, g);
            }
            dev_.pack(list_, nullptr);
            base_ = plain_.data();
        }
        dev_.sync();
        pending_ = false;
    }
    template <class T>
    const T* at(int i) const
    {
        return reinterpret_cast<const T*>(base_ + list_.seg[i].dst);
    }

private:
    Dev dev_;
    PackList list_;
    size_t words_ = 0;
    HostBlock block_;
    std::vector<uint32_t> plain_;
    const uint32_t* base_ = nullptr;
    bool pending_ = false;
};

}  // namespace sg
