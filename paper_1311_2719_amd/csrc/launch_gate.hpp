// Admission of kernels whose blocks wait for one another: such a grid ends only
// if all its blocks become resident, so the grids in flight on one device must
// fit it together.  Callers are admitted in the order they came (a large grid
// is not passed by small ones for ever).
#pragma once

#include <condition_variable>
#include <cstdint>
#include <mutex>

namespace stag {

class LaunchGate {
public:
    // Waits until `blocks` more blocks fit `limit` (a grid wider than the limit
    // runs alone) and everyone who came before has been admitted.
    void enter(int blocks, int limit)
    {
        std::unique_lock<std::mutex> lk(mu_);
        const uint64_t me = next_++;
        cv_.wait(lk, [&] { return serving_ == me && (used_ == 0 || used_ + blocks <= limit); });
        ++serving_;
        used_ += blocks;
        cv_.notify_all();
    }
    void leave(int blocks)
    {
        std::lock_guard<std::mutex> lk(mu_);
        used_ -= blocks;
        cv_.notify_all();
    }

private:
    std::mutex mu_;
    std::condition_variable cv_;
    uint64_t next_ = 0, serving_ = 0;
    int used_ = 0;
};

// Admitted for the life of the object.
class LaunchPass {
public:
    LaunchPass(LaunchGate &g, int blocks, int limit) : g_(g), blocks_(blocks) { g_.enter(blocks, limit); }
    ~LaunchPass() { g_.leave(blocks_); }
    LaunchPass(const LaunchPass &) = delete;
    LaunchPass &operator=(const LaunchPass &) = delete;

private:
    LaunchGate &g_;
    int blocks_;
};

}  // namespace stag
