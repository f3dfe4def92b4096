// Device memory that a ctx keeps between hierarchy builds: one block for the
// temporaries of each of a build's two phases.  Every device allocation of the
// ctx goes through here, so that one that would fail first gets back the
// blocks that no build under way uses.  (Host code over the two functions it is
// given; not thread-safe, like the ctx.)
#pragma once
#include <cstddef>

namespace hgs {

class KeptBlocks {
public:
    using Malloc = int (*)(void **p, size_t bytes);  // 0: success
    using Free = void (*)(void *p);
    static constexpr int kPhases = 2;

    KeptBlocks(Malloc m, Free f) : malloc_(m), free_(f) {}
    KeptBlocks(const KeptBlocks &) = delete;
    KeptBlocks &operator=(const KeptBlocks &) = delete;
    ~KeptBlocks()
    {
        for (Block &b : blocks_) drop(b);
    }

    // The allocator's status; *p is null unless it is 0.
    int alloc(void **p, size_t bytes)
    {
        *p = nullptr;
        int e = malloc_(p, bytes);
        if (e == 0) return 0;
        bool idle = false;
        for (Block &b : blocks_) {
            if (b.in_use || !b.p) continue;
            drop(b);
            idle = true;
        }
        *p = nullptr;
        if (idle) e = malloc_(p, bytes);
        if (e) *p = nullptr;
        return e;
    }

    // The block of phase k, at least `bytes` large and in use until release();
    // null where there is no room for it.
    char *reserve(int k, size_t bytes, size_t &size)
    {
        Block &b = blocks_[k];
        if (b.bytes < bytes) {
            drop(b);
            void *p = nullptr;
            if (alloc(&p, bytes)) {
                size = 0;
                return nullptr;
            }
            b.p = p;
            b.bytes = bytes;
        }
        b.in_use = true;
        size = b.bytes;
        return static_cast<char *>(b.p);
    }

    // The end of a build: blocks of at most `keep` bytes stay for the next.
    void release(size_t keep)
    {
        for (Block &b : blocks_) {
            b.in_use = false;
            if (b.bytes > keep) drop(b);
        }
    }

private:
    struct Block {
        void *p = nullptr;
        size_t bytes = 0;
        bool in_use = false;
    };
    void drop(Block &b)
    {
        if (b.p) free_(b.p);
        b = Block{};
    }
    Malloc malloc_;
    Free free_;
    Block blocks_[kPhases];
};

}  // namespace hgs
