// The device words of one measurement on their way to host memory.
//
// A measurement lists the segments it needs (Fetch::add) and brings them over
// together (Fetch::run).  What touches the device is in `Dev`, so that the
// arithmetic and the order of the steps can be checked without one.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <memory>
#include <mutex>
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

// Such memory, kept between measurements and shared by all contexts, threads and
// devices of the process: at most kBytes, in use or not, and none of it is freed while
// the process lives.  (An allocation costs 0.05 to 0.4 ms, more than the copy itself in
// small calls; freeing such memory waits for the work of every stream of the device,
// and no context waits for another's.)
class BlockPool {
public:
    static constexpr size_t kBytes = (size_t)128 << 20;
    static constexpr size_t kMost = (size_t)64 << 20;    // largest block (a power of two)
    static constexpr size_t kLeast = (size_t)64 << 10;   // smallest block
    static constexpr size_t kPiece = (size_t)1 << 20;    // smallest block worth working through in pieces
    // A block of `bytes` or more; where that is not to be had, one of kPiece or more
    // to bring the words over in pieces, or else none.  alloc(bytes): new memory, or
    // null.
    template <class Alloc>
    HostBlock get(size_t bytes, Alloc&& alloc)
    {
        size_t size = kLeast;
        {
            std::lock_guard<std::mutex> lk(mu_);
            size_t best = free_.size(), most = free_.size();
            for (size_t i = 0; i < free_.size(); ++i) {
                if (free_[i].bytes >= bytes && (best == free_.size() || free_[i].bytes < free_[best].bytes)) best = i;
                if (most == free_.size() || free_[i].bytes > free_[most].bytes) most = i;
            }
            if (best < free_.size()) return take(best);
            while (size < bytes && size < kMost) size *= 2;
            if (most < free_.size() && free_[most].bytes >= size) return take(most);   // (more than kMost is asked for)
            if (total_ + size > kBytes) {
                if (most < free_.size() && free_[most].bytes >= kPiece) return take(most);
                while (size > kPiece && total_ + size > kBytes) size /= 2;
                if (total_ + size > kBytes) return HostBlock{};
            }
            free_.reserve(blocks_ + 1);   // (put does not allocate)
            total_ += size;
            ++blocks_;
        }
        void* p = alloc(size);
        if (p) return HostBlock{p, size};
        std::lock_guard<std::mutex> lk(mu_);
        total_ -= size;
        --blocks_;
        return HostBlock{};
    }
    void put(const HostBlock& b)
    {
        if (!b.p) return;
        std::lock_guard<std::mutex> lk(mu_);
        free_.push_back(b);
    }

private:
    HostBlock take(size_t i)
    {
        const HostBlock b = free_[i];
        free_[i] = free_.back();
        free_.pop_back();
        return b;
    }
    std::mutex mu_;
    std::vector<HostBlock> free_;
    size_t total_ = 0, blocks_ = 0;
};

// Dev:
//   HostBlock get(size_t bytes)         memory that the device can write to: a block of
//                                       that size, or a smaller one, or p null
//   void put(const HostBlock&)          gives it back (does not throw)
//   void pack(const PackList&, uint32_t* block, uint64_t w0, uint64_t w1)
//                                       enqueues the copy of destination words w0 .. w1
//                                       - 1 to the block and their clearing (block
//                                       null: only that)
//   void copy(uint32_t* dst, const uint32_t* src, uint64_t words)    enqueues a copy to
//                                       ordinary memory
//   void copy_rows(uint32_t* dst, const PackSeg&)    the same of a segment's rows
//   void store(uint32_t* dst, const uint32_t* src, size_t words)     copies on the host
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
        if (block_.p && block_.bytes >= words_ * 4) {
            dev_.pack(list_, (uint32_t*)block_.p, 0, words_);
            base_ = (const uint32_t*)block_.p;
        } else {
            plain_.reset(new uint32_t[std::max<size_t>(2, words_)]);
            base_ = plain_.get();
            if (block_.p) {
                pieces();
            } else {
                copies();
                dev_.pack(list_, nullptr, 0, words_);
            }
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
    // through the halves of a block in turn: one is filled while the host empties the
    // other
    void pieces()
    {
        const size_t half = block_.bytes / 8;   // words
        uint32_t* const b[2] = {(uint32_t*)block_.p, (uint32_t*)block_.p + half};
        auto fill = [&](size_t w0) { dev_.pack(list_, b[w0 / half & 1], w0, std::min(words_, w0 + half)); };
        fill(0);
        for (size_t w0 = 0; w0 < words_; w0 += half) {
            dev_.sync();
            if (w0 + half < words_) fill(w0 + half);
            dev_.store(plain_.get() + w0, b[w0 / half & 1], std::min(half, words_ - w0));
        }
    }
    void copies()
    {
        for (int i = 0; i < list_.n; ++i) {
            const PackSeg& g = list_.seg[i];
            uint32_t* dst = plain_.get() + g.dst;
            if (pack_words(g) == 0) continue;
            // (a single row's stride means nothing, and a copy by rows takes none
            // below its width)
            if (g.rows == 1 || g.stride == g.width)
                dev_.copy(dst, g.src, pack_words(g));
            else
                dev_.copy_rows(dst, g);
        }
    }
    Dev dev_;
    PackList list_;
    size_t words_ = 0;
    HostBlock block_;
    std::unique_ptr<uint32_t[]> plain_;
    const uint32_t* base_ = nullptr;
    bool pending_ = false;
};

}  // namespace sg
