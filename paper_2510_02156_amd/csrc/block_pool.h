// block_pool.h -- device memory taken and given back in whole blocks, a bounded
// number of which stay idle for the next handle.  Host code without a
// dependency on the device runtime; internal to the library.
#pragma once

#include <pthread.h>
#include <stddef.h>

namespace rorbk {

struct Block {
    char *p;
    size_t bytes;
    int dev, misses;
};

// The driver clears freed device memory before it gives it out again and does
// not keep up with programs that set up handles one after another (640 MB taken
// and freed every 4 ms: 0.2 ms a call at first, 28 ms after two seconds;
// 100000-row CSR handles of 128-row blocks made, used for 4 iterations and
// closed: 8 to 41 ms each, 3.75 with idle blocks kept).
// A block is either idle and here or in use and not here, so threads and
// streams never share one.  At most MAX_BYTES in MAX_BLOCKS blocks stay; one
// that MAX_MISSES requests have passed over goes back to the driver, and all
// of them do on trim() and when an allocation made through alloc() or get()
// finds the memory used up.  Nothing here throws.
class BlockPool {
  public:
    typedef int (*AllocFn)(void **p, size_t bytes);   // 0, or an error code
    typedef void (*FreeFn)(void *p);
    static constexpr size_t MAX_BYTES = (size_t)2 << 30;
    static constexpr int MAX_BLOCKS = 8;
    static constexpr int MAX_MISSES = 16;

    constexpr BlockPool(AllocFn a, FreeFn f) : alloc_(a), free_(f) {}

    // Memory of the caller's own (not from the idle blocks); where there is
    // none left the idle blocks are given back and it is tried once more.
    int alloc(void **p, size_t bytes) {
        int e = alloc_(p, bytes);
        if (e != 0 && trim() > 0) e = alloc_(p, bytes);
        return e;
    }

    // A block of at least `bytes` on device `dev`, the current one (contents
    // undefined): the smallest idle one that is not more than twice that, else
    // a new one.
    int get(Block *out, size_t bytes, int dev) {
        if (bytes == 0) bytes = 1;
        Block drop[MAX_BLOCKS];
        int ndrop = 0;
        *out = Block{nullptr, 0, 0, 0};
        pthread_mutex_lock(&mu_);
        int best = -1;
        for (int i = 0; i < count_; ++i)
            if (kept_[i].dev == dev && kept_[i].bytes >= bytes && kept_[i].bytes / 2 <= bytes &&
                (best < 0 || kept_[i].bytes < kept_[best].bytes))
                best = i;
        if (best >= 0) *out = take(best);
        for (int i = count_; i-- > 0;)
            if (++kept_[i].misses >= MAX_MISSES) drop[ndrop++] = take(i);
        pthread_mutex_unlock(&mu_);
        for (int i = 0; i < ndrop; ++i) free_(drop[i].p);
        if (out->p) return 0;
        void *p = nullptr;
        const int e = alloc(&p, bytes);
        if (e == 0) *out = Block{(char *)p, bytes, dev, 0};
        return e;
    }

    // An idle block back (nothing may be using it): kept, or freed where it
    // would pass the bounds.
    void put(Block *b) {
        if (!b->p) return;
        bool keep = false;
        pthread_mutex_lock(&mu_);
        size_t sum = 0;
        for (int i = 0; i < count_; ++i) sum += kept_[i].bytes;
        if (count_ < MAX_BLOCKS && b->bytes <= MAX_BYTES - sum) {
            kept_[count_] = *b;
            kept_[count_++].misses = 0;
            keep = true;
        }
        pthread_mutex_unlock(&mu_);
        if (!keep) free_(b->p);
        *b = Block{nullptr, 0, 0, 0};
    }

    // Every idle block to the driver; how many there were.
    int trim() {
        Block drop[MAX_BLOCKS];
        pthread_mutex_lock(&mu_);
        const int n = count_;
        for (int i = 0; i < n; ++i) drop[i] = kept_[i];
        count_ = 0;
        pthread_mutex_unlock(&mu_);
        for (int i = 0; i < n; ++i) free_(drop[i].p);
        return n;
    }

  private:
    Block take(int i) {
        const Block b = kept_[i];
        kept_[i] = kept_[--count_];
        return b;
    }
    AllocFn alloc_;
    FreeFn free_;
    pthread_mutex_t mu_ = PTHREAD_MUTEX_INITIALIZER;
    Block kept_[MAX_BLOCKS] = {};
    int count_ = 0;
};

}  // namespace rorbk
