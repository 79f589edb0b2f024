// gpr_room.h -- room on a device for launches whose workgroups wait for one another.  Plain C++, so
// that a test can compile it by itself.
//
// A launch with several workgroups per replica ends only if all groups of a replica run at the same
// time.  One launch fits the device by itself; two on different streams, each asking for more
// than half of it, could be placed in part each and then wait until the bounded spin ends.  So every
// such launch of the process takes room here first, one unit for each compute unit, and gives it
// back when the host has waited for it.  Launches on one stream follow each other and share their
// room.  Who takes room holds none while waiting for it and gives it back without taking more, so
// every wait ends; waiting is first come, first served.
#pragma once
#include <condition_variable>
#include <mutex>
#include <thread>

namespace gpr {

class Room {
public:
    // the streams of a per-thread default are told apart by their threads
    struct Key {
        const void *stream;
        std::thread::id thread;
        bool operator==(const Key &o) const { return stream == o.stream && thread == o.thread; }
    };

    // takes `units` of the device's `cap` if they are free and nobody waits for room
    bool try_take(const Key &key, int units, int cap)
    {
        std::lock_guard<std::mutex> lk(mu_);
        return next_ == serving_ && take_now(key, units, cap);
    }

    // the same, waiting for it
    void take(const Key &key, int units, int cap)
    {
        std::unique_lock<std::mutex> lk(mu_);
        const unsigned long long mine = next_++;
        cv_.wait(lk, [&] { return mine == serving_ && take_now(key, units, cap); });
        ++serving_;
        cv_.notify_all();
    }

    void give(const Key &key)
    {
        std::lock_guard<std::mutex> lk(mu_);
        for (int k = 0; k < n_; ++k)
            if (use_[k].key == key) {
                if (--use_[k].refs == 0) use_[k] = use_[--n_];
                break;
            }
        cv_.notify_all();
    }

    // whether a launch of another stream has room or waits for it
    bool others(const Key &key)
    {
        std::lock_guard<std::mutex> lk(mu_);
        if (next_ != serving_) return true;
        for (int k = 0; k < n_; ++k)
            if (!(use_[k].key == key)) return true;
        return false;
    }

private:
    struct Use {
        Key key;
        int units, refs;
    };
    static constexpr int MAX = 64;         // streams with launches under way (more wait)
    std::mutex mu_;
    std::condition_variable cv_;
    Use use_[MAX]{};
    int n_ = 0;
    unsigned long long next_ = 0, serving_ = 0;

    bool take_now(const Key &key, int units, int cap)
    {
        if (units > cap) units = cap;      // the whole device
        int used = 0, at = n_;
        for (int k = 0; k < n_; ++k) {
            if (use_[k].key == key) at = k;
            else used += use_[k].units;
        }
        if (at == MAX || used + units > cap) return false;
        if (at == n_) use_[n_++] = Use{key, 0, 0};
        if (use_[at].units < units) use_[at].units = units;
        use_[at].refs += 1;
        return true;
    }
};

} // namespace gpr
