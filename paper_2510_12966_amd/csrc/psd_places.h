// Places on a device for workgroups that wait for each other inside one launch (host only).
#pragma once
#include <atomic>

namespace psd {

// Launches whose workgroups wait for each other must be resident as a whole.  One alone always is; several in flight (contexts on
// threads of their own, a stream each) can each get a part of the device and wait for the rest until their bound expires.  So
// whoever enqueues one takes places for its workgroups first and gives them back once it is known to be over; who gets none
// goes another way.  Nobody waits for places.
class Places {
    std::atomic<int> used_{0};
    std::atomic<int> total_{0};
public:
    // what a launch of `grid` workgroups takes: consecutive ones go round the eight dies whether a die has room or not, so the
    // fullest die counts
    static int of(int grid) { return (grid + 7) / 8 * 8; }
    void open(int total) { total_.store(total / 8 * 8); }
    int total() const { return total_.load(); }
    bool take(int n) {
        int u = used_.load();
        do {
            if (n > total() - u) return false;
        } while (!used_.compare_exchange_weak(u, u + n));
        return true;
    }
    void give(int n) { used_.fetch_sub(n); }
};

}  // namespace psd
