// Device memory of freed indexes, kept for the next build of the same size.
//
// A program that publishes builds a new index and frees the one it replaces, over and over; handing hundreds of
// megabytes back to the driver and fetching them again costs 0.3 ms a time, and 10 ms and more once the
// driver has no cleared pages left in stock.  So the block of the most recently freed index stays here, one per
// device and at most kKeepBytes, as long as another index lives on the device (the one that replaced it).  It goes
// back
//   when the last index of the device is freed: a program that has freed its indexes has all their memory back,
//   when an index of another size is built, or another one is freed,
//   when an allocation of the library fails (the allocation is then tried again), and
//   when the program asks for it (release()).
//
// The pool's user passes the allocation and release calls, so that the pool can be tested on the host alone.
// Nothing is called under the lock.
#pragma once
#include <stdint.h>

#include <mutex>

namespace st {

constexpr int64_t kKeepBytes = 1ll << 30;
constexpr int kKeepDevices = 64;

class BlockKeep {
public:
    // alloc(out, bytes), free(ptr) and idle(): 0 or an error code, which the pool passes on.  idle() returns once
    // no work is in flight on the current device (a freed block may still be read by some).
    typedef int (*AllocFn)(void** out, int64_t bytes);
    typedef int (*FreeFn)(void* ptr);
    typedef int (*IdleFn)();

    // Memory of a call, on the current device.
    int get(int device, int64_t bytes, AllocFn alloc, FreeFn free, void** out)
    {
        int rc = alloc(out, bytes);
        if (rc == 0) return 0;
        const Block k = take(device);
        if (!k.ptr) return rc;
        const int rc_free = free(k.ptr);
        return rc_free ? rc_free : alloc(out, bytes);
    }

    // Memory of an index: the kept block if it has the size.
    int get_index(int device, int64_t bytes, AllocFn alloc, FreeFn free, void** out)
    {
        const Block k = take(device);
        int rc = 0;
        if (k.ptr && k.bytes == bytes) {
            *out = k.ptr;
        } else {
            if (k.ptr) rc = free(k.ptr);
            if (rc == 0) rc = get(device, bytes, alloc, free, out);
        }
        if (rc == 0) {
            std::lock_guard<std::mutex> lock(mu_);
            ++live_[device];
        }
        return rc;
    }

    // The index is gone.  An error leaves the caller with the memory (and the index counted).
    int put_index(int device, void* ptr, int64_t bytes, FreeFn free, IdleFn idle)
    {
        bool keep;
        {
            std::lock_guard<std::mutex> lock(mu_);
            keep = live_[device] > 1 && bytes <= kKeepBytes;
        }
        const int rc = keep ? idle() : free(ptr);
        if (rc) return rc;
        Block back[2];  // what goes back to the driver
        {
            std::lock_guard<std::mutex> lock(mu_);
            back[0] = kept_[device];
            kept_[device] = Block{};
            --live_[device];
            if (keep) (live_[device] > 0 ? kept_[device] : back[1]) = Block{ptr, bytes};  // (other threads free as well)
        }
        for (const Block& b : back)
            if (b.ptr) (void)free(b.ptr);  // (the caller's index is gone either way)
        return 0;
    }

    int release(int device, FreeFn free)
    {
        const Block k = take(device);
        return k.ptr ? free(k.ptr) : 0;
    }

private:
    struct Block {
        void* ptr = nullptr;
        int64_t bytes = 0;
    };
    Block take(int device)
    {
        std::lock_guard<std::mutex> lock(mu_);
        const Block k = kept_[device];
        kept_[device] = Block{};
        return k;
    }
    std::mutex mu_;
    Block kept_[kKeepDevices];
    int64_t live_[kKeepDevices] = {};
};

}  // namespace st
