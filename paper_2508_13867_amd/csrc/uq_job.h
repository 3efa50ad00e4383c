// A UQ job: problem, sample set, device buffers and time-stepping state.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <vector>

#include "uq_internal.h"

namespace uqi {

int64_t storage_bytes(int prec);
int64_t row_pitch(int nx);
void build_mask(const uq_problem &p, int64_t pitch, std::vector<uint32_t> &mask, std::vector<double> &q,
                std::vector<int32_t> &special, int &fluid);
// pipelines = false: without the pipelines that take a second slab on their
// own account
StepShape choose_shape(const uq_problem &p, int64_t S, bool pipelines = true);
// Rows per chunk of a pipelined launch: `items` work items per chunk of rows,
// of which `per_cu` fit a CU, `fill` row steps to fill and drain a pipeline.
// (cost_out: rounds x row steps of that choice.)
double rounds_of(int64_t n, int per_cu, double alone);
int chunk_rows(int ny, int64_t items, int fill, int per_cu, double *cost_out = nullptr);
int group_rows(const int64_t *items, const int *ny, int n, int fill, int per_cu);
int pipeline_per_cu(int prec, int n, int rows, int K, int M);
// steps per launch of resident tiles for a periodic job (0: none), and the time
// of a step in us
double tile_steps(int prec, int nx, int ny, int64_t S, int *n);
// The pipeline of a job that nobody tuned (window, steps per launch, chunk rows;
// AB layout) and about how many us a step takes in it; the same of one step per
// launch. (Channels: those with node-local rules. strips_shape: the strips at the
// most steps per launch, whether or not another pipeline is faster.)
double strips_shape(const uq_problem &p, int64_t S, StepShape *s);
double pipeline_shape(const uq_problem &p, int64_t S, StepShape *s);
double single_step_us(const uq_problem &p, int64_t S);
// the shapes uq_autotune times (at most cap of them to out); returns their number
int64_t tune_candidates(const uq_problem &p, int64_t S, StepShape *out, int64_t cap);
// tuned shape for a problem class, if one was measured in this process
bool tuned_shape(const uq_problem &p, int64_t S, StepShape *out);

// Device buffers of one statistics evaluation (uq_qoi_samples, uq_moments
// and its allocation-free variant): per-sample scalar QoIs qoi[S][4], the
// selected scalar M[S], per-sample fields fields[S][4][ny][nx] (per-sample
// field values only; the moments of a field are formed from the populations
// without them), the outputs out[(K + 3) n_out], one int64 flag and the sums of
// samples cut into chunks, part[QOI_PARTS] (null: in the job's idle slab).
struct StatBufs {
    double *qoi = nullptr, *M = nullptr, *fields = nullptr, *out = nullptr, *part = nullptr;
    int64_t *flag = nullptr;
};

// values per sample of a QoI (1, nx ny or 2 nx ny); 0 for an unknown QoI
int64_t qoi_width(const uq_problem &p, int qoi);

struct Job {
    uq_problem p{};
    uq_device dev{};
    Rule rule;
    int64_t S = 0;
    int K = 0;
    int64_t pitch = 0;
    int scale_exp = 0;
    int fluid = 0;
    int plane_pad = 0;

    hipStream_t user_stream = nullptr;  // caller's stream (ordering only)
    hipStream_t stream = nullptr;       // the job's own work stream
    hipEvent_t ev_in = nullptr, ev_out = nullptr;

    JobDev jd{};
    StepShape shape{};
    int64_t t = 0;            // steps done (host mirror)
    int64_t launches = 0;     // step-kernel launches issued (graph replays counted per launch)
    int64_t graph_launches = 0; // step-kernel launches in the captured graph
    int64_t pending_launches = 0; // counted by enqueue_steps
    int64_t *d_t = nullptr;   // steps done at the last base update (device)

    std::vector<void *> allocs;
    int64_t bytes_held = 0;
    // A second slab that the job took on its own account (nobody asked for the
    // AB layout) is given back when memory runs out: see reclaim_slab. `mu` is
    // held by every call on the job, and by another job's call while it takes
    // the slab.
    bool spare = false;    // holds such a slab (and is in the register)
    bool reclaims = true;  // its own allocations may ask others for theirs
    mutable std::recursive_mutex mu;
    double *d_qoi = nullptr, *d_M = nullptr, *d_out = nullptr, *d_fields = nullptr;
    double *d_wphi = nullptr, *d_a = nullptr, *d_export = nullptr;
    int64_t *d_flag = nullptr;
    int64_t out_cap = 0;

    // hipGraph of `graph_len` steps starting at an even step
    bool use_graph = true;
    int graph_len = 0;
    hipGraph_t graph = nullptr;
    hipGraphExec_t gexec = nullptr;

    ~Job();
    void *dalloc(size_t bytes);
    void *dalloc_now(size_t bytes);  // without asking other jobs for memory
    void dfree(void *p);             // release one block from dalloc
    int64_t slab_bytes() const { return S * 9 * jd.plane * storage_bytes(p.precision); }
    void *to_one_slab();             // AB to AA; the slab that is no longer needed (null: could not)
    void keep_slabs();               // out of the register
    void dfree_all();
    uq_status ensure_stats_buffers(int64_t n_out_max);
    uq_status ensure_fields();
    // the job's own statistics buffers for `qoi` (with the per-sample field
    // buffer if `fields`), allocated on first use
    uq_status own_stat_bufs(int qoi, bool fields, StatBufs *b);
    uq_status check_finite(const StatBufs &b);
    // per-sample values of `qoi` in b (M: value o of sample s at M[s*ld + o])
    uq_status sample_values_in(const StatBufs &b, int qoi, const double **M, int64_t *n_out, int64_t *ld);
    uq_status sample_values(int qoi, const double **M, int64_t *n_out, int64_t *ld);
    // statistics of `qoi` computed in b and copied to out (blocking)
    uq_status moments_in(const StatBufs &b, int qoi, uq_moments_out *out);
    uq_status advance(int64_t steps);
    hipError_t enqueue_steps(int k0, int64_t n);
    int fused_n() const;
    uq_status enter();  // order the job stream after the caller's stream
    uq_status leave();  // order the caller's stream after the job stream
    void release_graph();
};

}  // namespace uqi

struct uq_job : public uqi::Job {};

namespace uqi {
// Build a job; `forced` (may be null) fixes layout and launch shape. reclaim =
// false: its memory is a pool of the library's own, which other jobs' slabs do
// not fill.
uq_status create_job(const uq_problem &p, const uq_device *dev, const StepShape *forced, uq_job **out,
                     bool reclaim = true);
// One job on the device gives back the second slab that it took on its own
// account, for `bytes` that hipMalloc or a caller's allocator (hooked) refused.
// False if there is none to wait for, or none that could help.
bool reclaim_slab(int device, size_t bytes, bool hooked);
// While one is alive such a slab is held by a job outside the register.
struct InTransit {
    const bool on;
    explicit InTransit(bool counts);
    explicit InTransit(std::adopt_lock_t) : on(true) {}  // (counted already)
    ~InTransit();
    InTransit(const InTransit &) = delete;
    InTransit &operator=(const InTransit &) = delete;
};
}  // namespace uqi
