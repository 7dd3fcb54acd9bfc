// A batch of CG systems that share one gauge field: workspace, state and the
// launch sequence of one CG iteration.  Used by stag_cg_solve (one right-hand
// side, two parity systems), stag_cg_solve_batch and the serving scheduler.
#pragma once

#include <vector>

#include "cg_launch.hpp"
#include "cg_persist.hpp"
#include "runtime.hpp"

namespace stag {

// Longest epoch (CG steps between two looks at the state) of a solve.
constexpr int kEpochMax = 64;

class Batch {
public:
    Batch(Ctx *ctx, std::shared_ptr<GaugeField> f, int prec, int slots, hipStream_t s);
    ~Batch();
    Batch(const Batch &) = delete;
    Batch &operator=(const Batch &) = delete;

    // Allocate workspace from the arena (single: for blocking solves of one
    // source, which may use the field's own workspace if it is free and large
    // enough, and run in one launch) and pinned host mirrors.  ENOMEM if the
    // arena cannot hold it.
    int create(bool single = false);
    // Use caller-provided memory instead: `dev` (device, dev_bytes >=
    // workspace_bytes) and `host` (ordinary host memory, host_bytes >=
    // host_bytes_for(slots)).  Nothing is allocated: no arena, pinned memory,
    // events, streams or graphs (the stream is synchronised where events
    // would be waited on); the shape is the field's tuned one if a solve of
    // this shape has run, else the default.  EINVAL if either buffer is too small.
    int create_external(void *dev, size_t dev_bytes, void *host, size_t host_bytes);
    static size_t host_bytes_for(int slots);
    // workspace bytes of this batch's field, precision and slots
    size_t needed_bytes() const;
    static size_t workspace_bytes(const Geom &g, int prec, int slots, int pstride);

    int slots() const { return S_; }
    int nsys() const { return 2 * S_; }
    int prec() const { return prec_; }
    const KernelCfg &cfg() const { return cfg_; }
    hipStream_t stream() const { return s_; }
    GaugeField *field() const { return f_.get(); }

    // Stage system j (= parity * slots + slot) for initialisation with source
    // b and solution x (parity halves, device), or mark it idle (b == x == null).
    void stage_system(int j, const stag_cg_params &p, const double *b_half, double *x_half);
    // Copy staged systems [j0, j0 + n) to the device and run the init kernel.
    int upload_and_init(const std::vector<int> &systems);
    // Enqueue `steps` CG steps (rounded up to an even number, so that every
    // epoch starts from state buffer 0), with the tile shape for the number of
    // running systems given to the last set_running.
    int enqueue_epoch(int steps);
    // Record (once) the graph of an epoch of `steps` steps with shape c.
    int record_epoch(int steps, const KernelCfg &c);
    // Enqueue a copy of the device state into the host snapshot and record an
    // event; wait_snapshot blocks until it has arrived.
    int enqueue_snapshot();
    int wait_snapshot();
    bool snapshot_ready();
    // Latest state of system j in the last snapshot (the newer of its two buffers).
    const SysState &state(int j) const
    {
        const SysState &a = snap_[j], &b = snap_[nsys() + j];
        return b.step > a.step ? b : a;
    }
    // Order in which the tiles take the systems: the systems flagged in
    // `running` first (per parity), the rest left out.  Stream-ordered: applies
    // to the kernels enqueued after this call.
    int set_running(const std::vector<char> &running);
    // Whether a solve runs in one launch (cg_persist.hip); solve_in_one_launch
    // runs the staged systems to their end, or gives up (gave_up: a block waited
    // too long for another; the solve must start again with the step kernels).
    bool persistent() const { return persist_; }
    int solve_in_one_launch(bool &gave_up);
    // This workspace's solves take the step kernels from now on (their shape is
    // timed now); systems staged before are to be uploaded again.
    int use_step_kernels();
    // Parities the step kernels cover from now on (bit 0 even, bit 1 odd): a
    // solve of one parity launches no blocks for the other.
    void set_parities(int mask) { parities_ = mask; }
    // Tile shape of the next epoch: the tuned shape, or while fewer systems
    // run per parity than it takes, the smallest tuned tile that holds them.
    const KernelCfg &epoch_cfg() const;

private:
    int launch_step(int ver, hipStream_t st, const KernelCfg &c);
    int finish_create();              // common tail of create / create_external
    void carve(void *base);           // device views into the workspace at base
    int launch_init();
    int choose_shape();  // the step kernels' shape, idle states, recorded epochs
    int one_launch(const CgArgs &a, uint32_t seq);  // launched, and its outcome read back
    int mark_stage();                 // the staged host data are being copied
    void wait_stage();                // ... and may be overwritten after this
    int grid_x(const KernelCfg &c) const;
    int remap_for(const KernelCfg &c, int nblk) const;

    bool uses_reduction(const KernelCfg &c) const;
    hipError_t launch_scalars(hipStream_t st, const CgArgs &a, int ver, int kind, int nblk) const;
    // Tune the tile shape on this workspace; also fills small_.
    KernelCfg tune_cg();
    bool parse_shape(const char *text, const CgLaunchTable &t, KernelCfg &c) const;
    KernelCfg default_cg_cfg() const;
    double time_cg_config(const KernelCfg &c, int nblk, bool reduce, int running, int reps, int runs,
                          bool recompute);
    CgArgs args() const;

    Ctx *ctx_;
    std::shared_ptr<GaugeField> f_;
    int prec_, S_;
    hipStream_t s_;
    KernelCfg cfg_;
    // tuned shapes of tiles smaller than cfg_.rtile, ascending
    std::vector<KernelCfg> small_;
    // blocks per tile row of every kernel of this batch: a prologue reduces
    // one partial sum per block of the kernel before it, so the count never
    // changes between shapes
    int nblk_ = 0;
    // a reduction kernel sums each step kernel's partials before the next
    // kernel reads them (large grids); otherwise every prologue sums them
    bool reduce_ = false;
    int parities_ = 3;  // parities the step kernels cover (set_parities)
    int live_ = 0;  // running systems per parity (the larger count), from set_running
    int pstride_ = 0;
    void *mem_ = nullptr;
    size_t bytes_ = 0;
    // device views into mem_
    void *p_[2] = {nullptr, nullptr}, *ap_ = nullptr, *r_ = nullptr;
    flt2 *xlo_ = nullptr;
    dbl2 *tmp_ = nullptr;
    dbl2 **xhi_d_ = nullptr;
    const dbl2 **b_d_ = nullptr;
    SysState *st_d_[2] = {nullptr, nullptr};
    int *perm_d_ = nullptr;
    double *partials_ = nullptr;
    bool single_ = false;   // blocking solves of one source
    bool persist_ = false;  // solves run in one launch
    PersistPlan persist_plan_;
    void *persist_slots_ = nullptr;
    // pinned host memory
    SysState *stage_ = nullptr;   // [nsys] staged initial states
    SysState *snap_ = nullptr;    // [2][nsys] last snapshot of both state buffers
    dbl2 **xhi_h_ = nullptr;
    const dbl2 **b_h_ = nullptr;
    int *perm_h_ = nullptr;
    int *abort_h_ = nullptr;
    std::vector<int> perm_last_;
    hipEvent_t snap_ev_ = nullptr, stage_ev_ = nullptr;
    std::vector<SysState> tune_st_;  // states a timed shape starts from
    hipEvent_t tune_ev_[2] = {nullptr, nullptr};
    bool stage_busy_ = false;
    bool field_mem_ = false;  // mem_ is the field's own workspace (GaugeField::work)
    bool external_ = false;  // memory from create_external: nothing owned, no events
    // epochs recorded once as HIP graphs (kernel nodes only) and replayed
    bool use_graphs_ = true;
    hipStream_t cap_stream_ = nullptr;
    std::map<int, hipGraphExec_t> graphs_;  // key: graph_key
};

}  // namespace stag
