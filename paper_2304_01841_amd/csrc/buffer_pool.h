// Idle device buffers kept for the next allocation of their size.
#pragma once

#include <stddef.h>

#include <algorithm>
#include <mutex>

namespace wcs {

// Buffers of one device that their owners have given back.  At most kSlots of
// them and kMaxBytes in all stay (the oldest go first); one is handed out for a
// request that it holds and is not four times too large for.  Safe with several
// threads.  Api: int alloc(void **, size_t) (0: done), bool out_of_memory(int) and
// void free(void *), which waits for work that still uses the buffer.
template <class Api>
class BufferPool {
public:
    static constexpr size_t kMaxBytes = (size_t)256 << 20;
    static constexpr int kSlots = 4;
    struct Buffer {
        void *ptr = nullptr;
        size_t bytes = 0;
    };

    BufferPool() = default;
    BufferPool(const BufferPool &) = delete;
    BufferPool &operator=(const BufferPool &) = delete;
    ~BufferPool() { release(); }

    // A buffer of at least `bytes`: a kept one, else a new one.
    int take(size_t bytes, Buffer *out)
    {
        *out = Buffer{};
        {
            std::lock_guard<std::mutex> hold(lock_);
            int best = -1;
            for (int i = 0; i < count_; ++i)
                if (kept_[i].bytes >= bytes && kept_[i].bytes / 4 <= bytes &&
                    (best < 0 || kept_[i].bytes < kept_[best].bytes))
                    best = i;
            if (best >= 0) {
                *out = remove(best);
                return 0;
            }
        }
        const int e = alloc(&out->ptr, bytes);
        out->bytes = e ? 0 : bytes;
        return e;
    }

    // A new allocation; without memory, the kept buffers go and it is tried again.
    int alloc(void **ptr, size_t bytes)
    {
        int e = Api::alloc(ptr, bytes);
        if (Api::out_of_memory(e) && release())
            e = Api::alloc(ptr, bytes);
        if (e)
            *ptr = nullptr;
        return e;
    }

    // Takes a buffer back.  `idle`: the device has finished with it, so whoever
    // takes it next may use it on any stream; otherwise it is freed.
    void give(Buffer *b, bool idle)
    {
        Buffer gone[kSlots + 1];
        int n = 0;
        if (b->ptr && (!idle || b->bytes > kMaxBytes)) {
            gone[n++] = *b;
        } else if (b->ptr) {
            std::lock_guard<std::mutex> hold(lock_);
            while (count_ == kSlots || (count_ > 0 && bytes_ + b->bytes > kMaxBytes))
                gone[n++] = remove(0);
            kept_[count_++] = *b;
            bytes_ += b->bytes;
        }
        *b = Buffer{};
        for (int i = 0; i < n; ++i)
            Api::free(gone[i].ptr);
    }

    // Frees the kept buffers; false if there were none.
    bool release()
    {
        Buffer gone[kSlots];
        int n = 0;
        {
            std::lock_guard<std::mutex> hold(lock_);
            while (count_ > 0)
                gone[n++] = remove(0);
        }
        for (int i = 0; i < n; ++i)
            Api::free(gone[i].ptr);
        return n > 0;
    }

private:
    Buffer remove(int i)
    {
        const Buffer b = kept_[i];
        std::copy(kept_ + i + 1, kept_ + count_, kept_ + i);
        --count_;
        bytes_ -= b.bytes;
        return b;
    }

    std::mutex lock_;
    Buffer kept_[kSlots];  // oldest first
    int count_ = 0;
    size_t bytes_ = 0;
};

}  // namespace wcs
