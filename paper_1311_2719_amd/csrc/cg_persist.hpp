// The CG loop of one right-hand side in one launch (cg_persist.hip).
#pragma once

#include "cg_kernels.hpp"
#include "launch_gate.hpp"

namespace stag {

struct PersistPlan {
    int lps = 0, nblk = 0;
};

// Passed from the launch of such a kernel until it has ended: two that do not
// fit the CUs together could each hold CUs the other waits for.
LaunchGate &persist_gate(int device);
// What a grid counts there against the number of CUs: blocks are dealt to the
// eight XCDs in turn, and each XCD must hold its share.
inline int persist_share(int nblk) { return (nblk + 7) / 8 * 8; }
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
