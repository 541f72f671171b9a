// Pinned host buffers for the copies between pageable host memory and the
// device, shared by all calls of the process.  A call takes a buffer of its
// own and gives it back at its end, so calls of several threads never wait for
// one another's copies or streams; what is idle is kept for the next call.
// With one buffer under a lock four threads reading four domains took 2.4 ms a
// round (1375 x 664 cells) where a buffer each takes 0.9, and a read waited
// for the steps queued before another thread's upload.
//
// Kept: at most kStageKept bytes in kStageSlots buffers, one buffer once the
// last domain is gone (trim).  Freeing pinned memory waits for the device, so
// buffers are freed only beyond those bounds.
#pragma once

#include <algorithm>
#include <cstddef>
#include <mutex>

namespace swe {

constexpr size_t kStageCap = (size_t)64 << 20;  // what a call asks for at most (or one row, if that is more)
constexpr size_t kStageKept = 4 * kStageCap;
constexpr int kStageSlots = 16;
constexpr size_t kStageUnit = (size_t)1 << 20;

struct StageBuffer {
    char *p = nullptr;
    size_t bytes = 0;
};

// Memory: static char *get(size_t bytes), nullptr where there is none, and
// static void put(char *)
template <class Memory>
class StagePool {
public:
    // the smallest idle buffer of at least `need` bytes or a new one; p is
    // nullptr where no memory is to be had.  A new buffer has at least twice
    // the bytes of the largest idle one (up to kStageCap) and whole MiB:
    // calls of ever larger sizes pin memory a few times, not each time (135
    // sizes from 0.1 to 67 MB one after another: 7 buffers; pinning 11 MB
    // takes 4 ms)
    StageBuffer take(size_t need)
    {
        size_t want = need;
        {
            std::lock_guard<std::mutex> lk(mu_);
            int k = -1;
            for (int q = 0; q < n_; ++q)
                if (idle_[q].bytes >= need && (k < 0 || idle_[q].bytes < idle_[k].bytes)) k = q;
            if (k >= 0) return remove(k);
            for (int q = 0; q < n_; ++q) want = std::max(want, std::min(2 * idle_[q].bytes, kStageCap));
        }
        want = (want + kStageUnit - 1) / kStageUnit * kStageUnit;
        StageBuffer b;
        b.p = Memory::get(want);
        if (!b.p && want > need) b.p = Memory::get(want = need);
        if (b.p) b.bytes = want;
        return b;
    }

    // no copy may still use it; the smallest idle buffers make room
    void give(const StageBuffer &b)
    {
        if (!b.p) return;
        StageBuffer out[kStageSlots + 1];
        int m = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (b.bytes <= kStageKept) {
                while (n_ == kStageSlots || kept_ + b.bytes > kStageKept) out[m++] = remove(smallest());
                idle_[n_++] = b;
                kept_ += b.bytes;
            } else {
                out[m++] = b;
            }
        }
        while (m > 0) Memory::put(out[--m].p);
    }

    // frees the idle buffers but the largest
    void trim()
    {
        StageBuffer out[kStageSlots];
        int m = 0;
        {
            std::lock_guard<std::mutex> lk(mu_);
            while (n_ > 1) out[m++] = remove(smallest());
        }
        while (m > 0) Memory::put(out[--m].p);
    }

private:
    StageBuffer remove(int k)
    {
        const StageBuffer b = idle_[k];
        idle_[k] = idle_[--n_];
        kept_ -= b.bytes;
        return b;
    }
    int smallest() const
    {
        int k = 0;
        for (int q = 1; q < n_; ++q)
            if (idle_[q].bytes < idle_[k].bytes) k = q;
        return k;
    }

    std::mutex mu_;
    StageBuffer idle_[kStageSlots];
    int n_ = 0;
    size_t kept_ = 0;
};

}  // namespace swe
