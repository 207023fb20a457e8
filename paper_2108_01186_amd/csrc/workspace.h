// Memory of the entry points that keep no context (fsic_op_*): device and
// pinned blocks kept for the next call instead of allocated and freed in each
// (a Poisson call made about 38 allocations and as many frees, every free
// waiting for the device: 1.1 of 1.6 ms for eight 100^3 densities).
//
// An entry point opens an OpScope for its stream; buffers grown while it is
// open (DBuf, pinned_alloc) come from the cache and belong to the scope.  At
// its end the scope waits for the stream, so no work is pending on a block
// that another thread or stream may take next, and gives the blocks back.
// Nothing in a block survives a call: every kernel writes what it reads.
//
// The cache holds at most kKeepBytes per device (kKeepPinned pinned) and
// kKeepBlocks blocks; the least recently used go first.  Blocks unused for
// kKeepSeconds go at the next call that gives blocks back or trims, and all go
// when an allocation fails, a context is destroyed or the program asks for it.
// (No timer gives them back: hipFree from a thread of its own would end a
// stream capture of the program.)
#pragma once
#include <hip/hip_runtime.h>

#include <chrono>
#include <cstddef>
#include <list>
#include <mutex>

namespace fsic {

class BlockCache {
   public:
    struct Block {
        void *p;
        size_t bytes;
        int dev;  // -1: pinned host memory
        double t;
    };
    static BlockCache &get() {
        static BlockCache *c = new BlockCache;  // not destroyed: the HIP runtime may be gone first
        return *c;
    }
    // a block into the first element of out: the smallest kept one that fits
    // without wasting more than half, or a new one
    hipError_t take(size_t bytes, int dev, std::list<Block> &out) {
        const size_t want = rounded(bytes);
        {
            std::lock_guard<std::mutex> lk(mu_);
            auto best = kept_.end();
            for (auto i = kept_.begin(); i != kept_.end(); ++i)
                if (i->dev == dev && i->bytes >= want && i->bytes / 2 <= want &&
                    (best == kept_.end() || i->bytes < best->bytes))
                    best = i;
            if (best != kept_.end()) {
                out.splice(out.begin(), kept_, best);
                return hipSuccess;
            }
        }
        out.push_front(Block{nullptr, want, dev, 0.0});
        hipError_t e = raw_alloc(&out.front().p, want, dev);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            flush();
            e = raw_alloc(&out.front().p, want, dev);
        }
        if (e != hipSuccess) out.pop_front();
        return e;
    }
    // blocks no work is pending on (list nodes move: nothing is allocated)
    void give(std::list<Block> &blocks) {
        std::list<Block> drop;
        const double now = seconds();
        {
            std::lock_guard<std::mutex> lk(mu_);
            for (Block &b : blocks) b.t = now;
            kept_.splice(kept_.end(), blocks);
            // newest first, so that the oldest of a device are over its limit
            size_t held[kMaxDev + 1] = {}, n = 0;
            for (auto i = kept_.end(); i != kept_.begin();) {
                --i;
                size_t &sum = held[i->dev < 0 ? kMaxDev : i->dev % kMaxDev];
                const size_t lim = i->dev < 0 ? kKeepPinned : kKeepBytes;
                if (sum + i->bytes > lim || n >= kKeepBlocks || now - i->t > kKeepSeconds) {
                    auto d = i++;
                    drop.splice(drop.end(), kept_, d);
                } else {
                    sum += i->bytes;
                    ++n;
                }
            }
        }
        for (const Block &b : drop) raw_free(b);
    }
    // blocks past their time
    void trim() {
        std::list<Block> none;
        give(none);
    }
    void flush() {
        std::list<Block> all;
        {
            std::lock_guard<std::mutex> lk(mu_);
            all.swap(kept_);
        }
        for (const Block &b : all) raw_free(b);
    }
    static void raw_free(const Block &b) {
        if (b.dev < 0) hipHostFree(b.p);
        else hipFree(b.p);  // of any device
    }

   private:
    static constexpr size_t kKeepBytes = (size_t)1 << 30, kKeepPinned = (size_t)16 << 20, kKeepBlocks = 256;
    static constexpr double kKeepSeconds = 30.0;
    static constexpr int kMaxDev = 64;
    static size_t rounded(size_t n) {
        if (n > ((size_t)1 << 20)) return (n + ((size_t)2 << 20) - 1) & ~(((size_t)2 << 20) - 1);
        size_t r = 4096;
        while (r < n) r *= 2;
        return r;
    }
    static hipError_t raw_alloc(void **p, size_t n, int dev) {
        return dev < 0 ? hipHostMalloc(p, n) : hipMalloc(p, n);
    }
    static double seconds() {
        return std::chrono::duration<double>(std::chrono::steady_clock::now().time_since_epoch()).count();
    }
    std::mutex mu_;
    std::list<Block> kept_;
};

class OpScope {
   public:
    explicit OpScope(hipStream_t s) : s_(s), up_(current()) {
        if (hipGetDevice(&dev_) != hipSuccess) dev_ = 0;
        current() = this;
    }
    ~OpScope() {
        current() = up_;
        if (blocks_.empty()) return;
        if (hipStreamSynchronize(s_) == hipSuccess) BlockCache::get().give(blocks_);
        else
            for (const BlockCache::Block &b : blocks_) BlockCache::raw_free(b);
    }
    OpScope(const OpScope &) = delete;
    OpScope &operator=(const OpScope &) = delete;
    hipError_t take(void **p, size_t bytes, bool pinned) {
        const hipError_t e = BlockCache::get().take(bytes, pinned ? -1 : dev_, blocks_);
        *p = e == hipSuccess ? blocks_.front().p : nullptr;
        return e;
    }
    // the scope open on this thread, or null
    static OpScope *&current() {
        static thread_local OpScope *c = nullptr;
        return c;
    }

   private:
    hipStream_t s_;
    OpScope *up_;
    int dev_ = 0;
    std::list<BlockCache::Block> blocks_;
};

// device memory: the open scope's, or (own) the caller's to free
inline hipError_t device_alloc(void **p, size_t bytes, bool &own) {
    OpScope *const sc = OpScope::current();
    own = sc == nullptr;
    if (sc) return sc->take(p, bytes, false);
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        BlockCache::get().flush();
        e = hipMalloc(p, bytes);
    }
    return e;
}
// pinned memory, freed by pinned_free in the same situation (a context lives
// in one scope or in none)
inline hipError_t pinned_alloc(void **p, size_t bytes) {
    OpScope *const sc = OpScope::current();
    return sc ? sc->take(p, bytes, true) : hipHostMalloc(p, bytes);
}
inline void pinned_free(void *p) {
    if (p && !OpScope::current()) hipHostFree(p);
}

}  // namespace fsic
