// The CG loop of one right-hand side in one launch (cg_persist.hip).
#pragma once

#include <mutex>

#include "cg_kernels.hpp"

namespace stag {

struct PersistPlan {
    int lps = 0, nblk = 0;
};

// One such kernel at a time per device in this process: held from its launch
// until it has ended, since two could each hold CUs the other waits for.
std::mutex &persist_lock(int device);
// Sums a step exchanges between blocks, and the word that says a wait was given up.
size_t cg_persist_bytes();
inline size_t cg_persist_abort_offset() { return cg_persist_bytes() - 256; }
// Whether a field can be solved this way, and with how many lanes and blocks.
bool cg_persist_plan(int num_cus, const Geom &g, int prec, int rows, PersistPlan &plan);
// Up to max_steps steps of the systems in a.st[0] (M_INIT: from b; else from the
// stored vectors).  slots: cg_persist_bytes() bytes, zeroed before the first
// launch of a solve; uses the sequence numbers seq0 + 1 .. seq0 + 3 max_steps + 1.
hipError_t cg_persist_launch(const PersistPlan &plan, int prec, int rows, const CgArgs &a, void *slots, uint32_t seq0,
                             int max_steps, hipStream_t s);

}  // namespace stag
