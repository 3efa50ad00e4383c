// Time stepping of one job: eager launches or replays of a captured
// hipGraph of an even number of steps (the AA parity pattern inside the graph
// is then fixed, and the step count lives in device memory so the same graph
// serves every replay).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <string>

#include "fused_shapes.h"
#include "uq_job.h"

namespace uqi {

static int env_int(const char *name, int dflt) {
    const char *v = std::getenv(name);
    if (!v || !*v) return dflt;
    return std::atoi(v);
}

// Rounds that n work items take with `per_cu` of them on a CU at a time. Items
// that have a CU to themselves run faster: a last round that gives each CU at
// most one counts `alone`.
double rounds_of(int64_t n, int per_cu, double alone) {
    const int64_t slots = (int64_t)256 * per_cu, rest = n % slots;
    return (double)(n / slots) + (rest == 0 ? 0.0 : (rest <= 256 && per_cu > 1 ? alone : 1.0));
}

// The chunk count that minimises rounds of work items x row steps per item: a
// last round that leaves most CUs idle costs as much as a full one, and every
// chunk pays the pipeline's fill, so neither short nor tall chunks are best
// by themselves (1024^2 x 16 samples, 9 strips, 8 steps per launch: chunks of
// 32, 64, 128, 256 rows took 50.2, 44.1, 44.7, 52.4 us per step, in the
// ratios of this count).
int chunk_rows(int ny, int64_t items, int fill, int per_cu, double *cost_out) {
    double best = 0.0;
    int rows = ny;
    for (int c = 1; c <= std::max(1, ny / 8); ++c) {
        const int H = (ny + c - 1) / c;
        const double cost = rounds_of(items * ((ny + H - 1) / H), per_cu, 0.6) * (H + fill);
        if (c == 1 || cost < 0.999 * best) {
            best = cost;
            rows = H;
        }
    }
    if (cost_out) *cost_out = best;
    return std::max(8, rows);
}

// The chunk height for several jobs in one launch, by the same count: job q has
// items[q] work items per chunk of its ny[q] rows. Where no CU gets more than one
// item, a round counts 0.78 here: a lone 1024^2 x 2 takes 7.1 us per step in 432
// items of 43 rows, 9.6 in 288 of 64 and 8.9 in 216 of 86.
int group_rows(const int64_t *items, const int *ny, int n, int fill, int per_cu) {
    const int tallest = *std::max_element(ny, ny + n);
    double best = 0.0;
    int rows = tallest;
    for (int c = 1; c <= std::max(1, tallest / 8); ++c) {
        const int H = (tallest + c - 1) / c;
        int64_t work = 0;
        for (int q = 0; q < n; ++q) work += items[q] * ((ny[q] + H - 1) / H);
        const double cost = rounds_of(work, per_cu, work <= 256 ? 0.78 : 0.6) * (H + fill);
        if (c == 1 || cost < 0.999 * best) {
            best = cost;
            rows = H;
        }
    }
    return std::max(8, rows);
}

// Workgroups of a row pipeline that a CU holds: by its LDS rings (160 KB) and
// by its waves' registers. The compiler's counts: single precision 60 VGPRs
// with one column per lane (28 waves per CU) and 101-111 with two (16),
// double precision 110 (16) and 188-197 (8); the channel's 90-98 (20), 135-145
// (12), 147-193 (8) and 235-247 (8).
int pipeline_per_cu(int prec, int n, int rows, int K, int M) {
    const bool ch = rows == RING_ROWS_CH, dbl = prec == UQ_FP64;
    const int waves = M == 1 ? (dbl ? (ch ? 8 : 16) : (ch ? 20 : 28)) : (dbl ? 8 : (ch ? 12 : 16));
    const int64_t lds = (int64_t)(n - 1) * rows * ring_cols(rows, K, M) * (dbl ? 8 : 4);
    return (int)std::max<int64_t>(1, std::min<int64_t>(waves / (n * K), 160 * 1024 / lds));
}

// Steps per launch of resident tiles for a job, and the time of one step in us,
// from a fit to one launch of n steps with one tile per CU (single precision
// 3.45 + 0.54 n us, double 3.6 + 0.81 n) and with more (two share a CU in
// single precision, at 1.6 times the time). Measured, n = 8: FP32 96^2 x 3
// samples 7.8 us a launch, FP64 64^2 x 5 10.1.
double tile_steps(int prec, int nx, int ny, int64_t S, int *n_best) {
    const bool dbl = prec == UQ_FP64;
    double best = 0.0;
    *n_best = 0;
    // many tiles per CU and a ring to compute in each: never
    if (S * nx * ny > ((int64_t)1 << 20) && nx * (int64_t)ny > TILE_NODES) return best;
    for (int n = 3; n <= TILE_MAX_STEPS; ++n) {
        const TileShape g = tile_shape(nx, ny, n);
        if (!g.RW) continue;
        const int64_t rounds = (S * g.tiles_x * g.tiles_y + 255) / 256;
        const double r = dbl || rounds == 1 ? (double)rounds : 0.8 * (double)rounds;
        const double t = (dbl ? 0.3 + r * (3.3 + 0.81 * n) : 1.0 + r * (2.45 + 0.54 * n)) / n;
        if (*n_best && t >= best) continue;
        best = t;
        *n_best = n;
    }
    return best;
}

// Strips of row pipelines at the most steps per launch: window, steps, chunk rows,
// and about how many us a step takes, by fits to 1 to 176 rounds of items on
// lattices of 2 to 1000 rows (9 of 10 of 213 shapes within 20 %). Vortices: row
// steps, whose fill overlaps the item beside it, of 0.86 us (double 0.98, 16-bit
// storage 1.15), 0.78 of it for items with a CU to themselves. Channels: 1.08
// (1.25, where one wave holds both ends 1.45; 1.17); where all items run at once,
// 1.1 (1.5, 1.37) and 2 us for the launch. (A chunk inside a channel also computes
// its halo; the whole height has none.)
double strips_shape(const uq_problem &p, int64_t S, StepShape *s) {
    const bool channel = p.geometry == UQ_GEOM_CHANNEL, dbl = p.precision == UQ_FP64;
    const bool half = storage_bytes(p.precision) == 2;
    int W, strips;
    s->fwin = 3;
    s->fuse = channel ? channel_strips_max_n(p.precision) : 8;
    row_strips(p.precision, p.nx, s->fuse, &W, &strips);
    const int per_cu = channel ? 1 : pipeline_per_cu(p.precision, s->fuse, RING_ROWS_TGV, RowStrips<UQ_FP32>::K,
                                                     RowStrips<UQ_FP32>::M);
    s->fty = chunk_rows(p.ny, S * strips, 3 * (s->fuse - 1), per_cu);
    const int64_t chunks = (p.ny + s->fty - 1) / s->fty;
    const double r = rounds_of(S * strips * chunks, per_cu, 0.78);
    const double rows = std::min(s->fty, p.ny) + (r <= 1.0 && (!channel || chunks > 1) ? 3 : 2) * (s->fuse - 1);
    if (!channel) return r * rows * (dbl ? 0.98 : (half ? 1.15 : 0.86)) / s->fuse;
    return (r <= 1.0 ? rows * (dbl ? 1.5 : (half ? 1.37 : 1.1)) + 2.0
                     : r * rows * (dbl ? (p.nx <= 64 ? 1.45 : 1.25) : (half ? 1.17 : 1.08))) / s->fuse;
}

// A channel's pipeline: strips at the most steps per launch, or 4 steps over
// whole rows where single precision's rings hold them and the count of rounds
// x row steps per step says so (a row step of either takes about 1.1 us). Us
// per step, strips and whole rows: FP32 220 x 41 x 512 samples 31.9, 28.7; 308
// x 57 x 64 10.5, 8.8; 440 x 82 x 64 13.9, 14.3 (3 steps); x 8 5.0, 6.9; 660 x
// 123 x 32 20.0, 21.8 (2 steps); 880 x 164 x 32 25.2, one step per launch 53.9;
// FP64 220 x 41 x 64 8.0, 8.5 (3 steps); 440 x 82 x 64 19.7, 43.9 (2 steps).
// Returns us per step; whole rows by a fit like that of the strips (9 of 10 of 85
// shapes within 15 %): row steps of 1.05 us (16-bit storage 1.15), where all items
// run at once 0.92 (1.0; with two columns per lane 1.3, 1.4 and 2 us for the
// launch).
static double channel_pipeline(const uq_problem &p, int64_t S, StepShape *s) {
    const double us = strips_shape(p, S, s);
    int W, strips, K = 0, M = 0;
    row_strips(p.precision, p.nx, s->fuse, &W, &strips);
    double cost = 0.0, cost4 = 0.0;
    (void)chunk_rows(p.ny, S * strips, 3 * (s->fuse - 1), 1, &cost);
    if (p.precision == UQ_FP64 || !rows_shape(p.precision, 4, RING_ROWS_CH, p.nx, &K, &M)) return us;
    const int per_cu = pipeline_per_cu(p.precision, 4, RING_ROWS_CH, K, M);
    const int rows = chunk_rows(p.ny, S, 9, per_cu, &cost4);
    if (cost4 / 4 > cost / s->fuse) return us;
    s->fwin = 2;
    s->fuse = 4;
    s->fty = rows;
    const bool half = storage_bytes(p.precision) == 2;
    const int64_t chunks = (p.ny + rows - 1) / rows;
    const double steps = std::min(rows, p.ny) + (chunks > 1 ? 9 : 6);
    if (S * chunks <= 256) return (M == 1 ? steps * (half ? 1.0 : 0.92) : steps * (half ? 1.4 : 1.3) + 2.0) / 4;
    return rounds_of(S * chunks, per_cu, 1.0) * steps * (half ? 1.15 : 1.05) / 4;
}

// The pipeline of a periodic lattice: 8 steps per launch over whole rows where
// the LDS rings hold them, else in strips; up to 128 columns 6 steps (one
// column per lane; two workgroups per CU in single precision, and the deepest
// that double precision's rings hold) unless so few samples ask for it that
// every chunk gets a CU of its own; resident tiles where those are faster
// still. Us per step, one step per launch and then: the pipelines, FP64 64^2 x
// 64 samples 6.28 -> 3.39, FP32 128^2 x 135 23.5 -> 8.0, 1024^2 x 16 238 -> 44;
// resident tiles, FP64 64^2 x 5 2.91 -> 1.20 (the pipeline 2.38), 32^2 x 32 2.78
// -> 1.04 (2.37), FP32 96^2 x 3 2.53 -> 0.89 (1.99), FP64 64^2 x 64 3.05.
// Returns us per step: of the tiles' fit, of the strips', or over whole rows as
// theirs with row steps of 0.77 us at one column per lane (double 0.68, 16-bit
// storage 0.98; 9 of 10 of 36 shapes within 9 %).
static double vortex_pipeline(const uq_problem &p, int64_t S, StepShape *s) {
    const bool dbl = p.precision == UQ_FP64, half = storage_bytes(p.precision) == 2;
    int K = 0, M = 0;
    double rows = 0.0, us;
    s->fuse = p.nx > 128 ? 8 : (!dbl && S * p.ny <= 256 * 12 ? 8 : 6);
    if (rows_shape(p.precision, s->fuse, RING_ROWS_TGV, p.nx, &K, &M)) {
        const int per_cu = pipeline_per_cu(p.precision, s->fuse, RING_ROWS_TGV, K, M);
        s->fwin = 2;
        s->fty = chunk_rows(p.ny, S, 3 * (s->fuse - 1), per_cu, &rows);
        const double r = rounds_of(S * ((p.ny + s->fty - 1) / s->fty), per_cu, 0.78);
        us = r * (std::min(s->fty, p.ny) + (r <= 1.0 ? 3 : 2) * (s->fuse - 1)) *
             (M == 1 ? (dbl ? 0.68 : (half ? 0.98 : 0.77)) : (half ? 1.15 : 0.86)) / s->fuse;
    } else {
        int W, strips;
        us = strips_shape(p, S, s);
        row_strips(p.precision, p.nx, s->fuse, &W, &strips);
        M = RowStrips<UQ_FP32>::M;
        (void)chunk_rows(p.ny, S * strips, 3 * (s->fuse - 1),
                         pipeline_per_cu(p.precision, s->fuse, RING_ROWS_TGV, RowStrips<UQ_FP32>::K, M), &rows);
    }
    // Resident tiles instead where they are faster: jobs too small to fill the
    // card with row chunks. A row step of the pipelines takes, in us, 0.7 (FP64,
    // one column per lane), 0.9 (two), 0.55 (single precision, 0.8 where two
    // workgroups share a CU), 0.85 (two columns).
    const double t_row = dbl ? (M == 1 ? 0.7 : 0.9) : (M == 1 ? (rows < 1.0 * (s->fty + 21) ? 0.55 : 0.8) : 0.85);
    int n = 0;
    const double t_tile = tile_steps(p.precision, p.nx, p.ny, S, &n);
    if (!n || t_tile >= 0.95 * rows * t_row / s->fuse) return us;
    s->fwin = 4;
    s->fuse = n;
    s->fty = tile_shape(p.nx, p.ny, n).OH;
    return t_tile;
}

double pipeline_shape(const uq_problem &p, int64_t S, StepShape *s) {
    s->layout = UQ_LAYOUT_AB;
    s->pad = 64;
    s->nt = 0;
    return p.geometry == UQ_GEOM_CHANNEL ? channel_pipeline(p, S, s) : vortex_pipeline(p, S, s);
}

// Us per step of one step per launch in the AA layout: a launch's latency and
// the longer of the memory traffic (7.5 TB/s where the slab stays in the 256 MB
// cache, 5.5 beyond) and the lanes' issue, in ps per lane of a row's whole
// waves (vortices also of whole 4-row tiles): channels 10 and 1.2 us, or 12.5 if
// that is less (double 13), vortices 4.3 (8.3), from memory 6.5 (10.3). 9 of 10 of
// 766 shapes, 2 to 1470 us on lattices 2 to 20000 wide x 2 to 600 samples, within
// 25 %.
double single_step_us(const uq_problem &p, int64_t S) {
    const bool channel = p.geometry == UQ_GEOM_CHANNEL, dbl = p.precision == UQ_FP64;
    const double b = (double)storage_bytes(p.precision), slab = 9.0 * b * (double)S * p.nx * p.ny;
    const double lanes = (double)S * (channel ? p.ny : (p.ny + 3) / 4 * 4) * (double)row_pitch(p.nx);
    const bool far = 9.0 * b * lanes > 512e6;
    const double ps = channel ? (dbl ? 13.0 : 10.0) : (dbl ? (far ? 10.3 : 8.3) : (far ? 6.5 : 4.3));
    const double issue = lanes * ps * 1e-6;
    return (channel ? 2.9 : 2.6) + (dbl ? 0.4 : 0.0) +
           std::max(2.0 * slab / (slab > 256e6 ? 5.5e6 : 7.5e6),
                    channel && !dbl ? std::min(1.25 * issue, 1.2 + issue) : issue);
}

// The pipeline that carries a job whose shape and layout nobody chose (AB
// layout), where it is faster than one step per launch. It is not on lattices
// of few rows, whose pipelines mostly fill and drain, and on channels of few
// nodes, where a row step's latency counts. Us per step, single steps and
// pipeline: FP32 vortices 20000 x 2 x 512 samples 270, 288; 4096 x 4 x 512 93,
// 69; FP16S 32 x 2048 x 32 20.4, 22.8; FP32 channels 400 x 30 x 2 3.4, 4.2 (x 32
// 8.4, 5.0); 1024 x 8 x 512 46, 58; 4096 x 3 x 512 71, 157 (x 16 rows 437,
// 282); FP64 500 x 60 x 2 4.2, 5.8 (x 32 23, 15).
static bool default_pipeline(const uq_problem &p, int64_t S, StepShape *s) {
    if (p.layout != UQ_LAYOUT_AUTO || needs_ab(p)) return false;
    const bool channel = p.geometry == UQ_GEOM_CHANNEL;
    const int64_t plane = (int64_t)p.ny * row_pitch(p.nx) + 64;
    const int64_t b = storage_bytes(p.precision), slab = S * 9 * plane * b;
    if (9 * plane * b >= ((int64_t)1 << 31) || (channel && plane * 4 >= ((int64_t)1 << 31))) return false;
    if (pipeline_shape(p, S, s) >= single_step_us(p, S)) return false;
    // The second slab is given back when the library misses it (reclaim_slab);
    // of what others on the card may miss, a quarter of it stays free beside
    // both slabs. (Memory that a caller's allocator keeps cached counts as taken.)
    if (slab > ((int64_t)256 << 20)) {
        size_t free_b = 0, total_b = 0;
        if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
            (void)hipGetLastError();
            return false;
        }
        if (2 * slab > (int64_t)free_b - (int64_t)(total_b / 4)) return false;
    }
    return true;
}

// Stores of single AB steps that bypass the caches pay where two slabs do not fit
// the 256 MB cache beside HBM; where they do, the next step reads them from it.
// The paper's 440 x 80 cylinder, us per step with and without: FP64 x 11 (57
// MB) 19.8, 14.9; FP32 x 32 (83 MB) 23.8, 20.4; FP64 x 32 (165 MB) 37.2,
// 33.7; FP32 x 100 (258 MB) 63.0, 64.4; FP64 x 100 (516 MB) 105, 121.
static bool stores_bypass(int64_t slab_bytes) { return 2 * slab_bytes > ((int64_t)200 << 20); }

// Launch shape and layout of a job. Order of precedence: a shape measured by
// uq_autotune for this problem class (when the problem leaves the layout to
// AUTO, or fixes the same layout), then the UQ_* environment overrides, then
// the pipeline that suits the problem, then one step per launch (AA, one row
// per thread, 64 elements of plane padding).
StepShape choose_shape(const uq_problem &p, int64_t S, bool pipelines) {
    StepShape s;
    if (tuned_shape(p, S, &s)) {
        if (needs_ab(p)) s.layout = UQ_LAYOUT_AB;
        return s;
    }
    bool asked = false;
    for (const char *name : {"UQ_CPT", "UQ_PERSISTENT", "UQ_NT_STORE", "UQ_PLANE_PAD", "UQ_BX", "UQ_FUSE",
                             "UQ_FUSE_TY", "UQ_FUSE_WINDOW", "UQ_LAYOUT"}) {
        const char *v = std::getenv(name);
        asked = asked || (v && *v);
    }
    if (pipelines && !asked && default_pipeline(p, S, &s)) return s;
    s = StepShape();
    s.cpt = env_int("UQ_CPT", 1);
    s.persistent = env_int("UQ_PERSISTENT", 0);
    s.nt = env_int("UQ_NT_STORE", 1);
    s.pad = env_int("UQ_PLANE_PAD", 64);
    s.bx = env_int("UQ_BX", 64);
    s.fuse = env_int("UQ_FUSE", 0);
    s.fty = env_int("UQ_FUSE_TY", 8);
    s.fwin = env_int("UQ_FUSE_WINDOW", 0);
    if (s.fwin == 2 && p.nx > full_rows_max_nx(p.precision, s.fuse)) s.fwin = 1;  // rows too wide
    s.layout = UQ_LAYOUT_AA;
    if (p.layout == UQ_LAYOUT_AA || p.layout == UQ_LAYOUT_AB) {
        s.layout = p.layout;
    } else {
        const char *v = std::getenv("UQ_LAYOUT");
        if (v && (v[0] == 'a' || v[0] == 'A') && (v[1] == 'b' || v[1] == 'B')) s.layout = UQ_LAYOUT_AB;
    }
    if (needs_ab(p)) s.layout = UQ_LAYOUT_AB;
    const char *nt = std::getenv("UQ_NT_STORE");
    if (s.layout == UQ_LAYOUT_AB && !(nt && *nt))
        s.nt = stores_bypass(S * 9 * (p.ny * row_pitch(p.nx) + s.pad) * storage_bytes(p.precision));
    return s;
}

// The job's own stream is non-blocking, so it is ordered against the
// caller's stream explicitly, also when that is the null stream.
uq_status Job::enter() {
    if (spare && user_stream) {
        // a graph that the caller captures names the slabs of now
        hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(user_stream, &st) != hipSuccess) (void)hipGetLastError();
        if (st != hipStreamCaptureStatusNone) keep_slabs();
    }
    if (user_stream != stream) {
        UQ_HIP_TRY(hipEventRecord(ev_in, user_stream));
        UQ_HIP_TRY(hipStreamWaitEvent(stream, ev_in, 0));
    }
    return UQ_OK;
}

uq_status Job::leave() {
    if (user_stream != stream) {
        UQ_HIP_TRY(hipEventRecord(ev_out, stream));
        UQ_HIP_TRY(hipStreamWaitEvent(user_stream, ev_out, 0));
    }
    return UQ_OK;
}

void Job::release_graph() {
    if (gexec) (void)hipGraphExecDestroy(gexec);
    if (graph) (void)hipGraphDestroy(graph);
    gexec = nullptr;
    graph = nullptr;
    graph_len = 0;
}

// steps per fused launch in effect (0: none)
int Job::fused_n() const {
    if (shape.fuse < 2) return 0;
    if (jd.geom == 1) {  // channel: whole rows, up to 4 steps, where the LDS rows fit; strips, 3 or more
        if (!channel_fusable(jd)) return 0;
        if (shape.fwin == 3) return shape.fuse >= 3 && shape.fuse <= channel_strips_max_n(jd.prec) ? shape.fuse : 0;
        return shape.fwin == 2 && shape.fuse <= 4 && jd.nx <= channel_rows_max_nx(jd.prec, shape.fuse) ? shape.fuse : 0;
    }
    if (shape.fwin == 4)  // resident tiles
        return shape.fuse <= TILE_MAX_STEPS && fused_supported(jd) && tile_shape(jd.nx, jd.ny, shape.fuse).RW
                   ? shape.fuse
                   : 0;
    const int nmax = shape.fwin >= 2 ? 8 : 4;  // whole rows and their strips: up to 8 steps
    if (shape.fwin == 3 && shape.fuse < 3) return 0;
    return (shape.fuse <= nmax && fused_supported(jd)) ? shape.fuse : 0;
}

// Launches for `n` steps starting at step t + k0 of the host mirror. The
// state of step u lives in slab u & 1. A launch of N fused steps reads the
// current slab and writes the other one: for odd N that is the slab of step
// u + N; even N go in pairs (there and back), so that the invariant holds
// after each pair. Steps left over go in single fused launches of an odd
// number (3 or more, at most N) of steps, largest first, then one per launch.
hipError_t Job::enqueue_steps(int k0, int64_t n) {
    hipError_t e = hipSuccess;
    int64_t &enqueued = pending_launches;
    int64_t k = 0;
    const int N = fused_n();
    if (N) {
        const int64_t block = (N & 1) ? N : 2 * N;
        for (; k + block <= n && e == hipSuccess; k += block) {
            const bool odd = ((t + k0 + k) & 1) != 0;
            e = launch_fused(jd, N, odd, shape.fty, shape.fwin, shape.nt != 0, d_t, (int)(k0 + k), stream);
            ++enqueued;
            if (e == hipSuccess && !(N & 1)) {
                e = launch_fused(jd, N, !odd, shape.fty, shape.fwin, shape.nt != 0, d_t, (int)(k0 + k + N), stream);
                ++enqueued;
            }
        }
        // fewer steps than a block: a shape that runs N steps runs fewer
        for (int64_t r = n - k; r >= 3 && e == hipSuccess; r = n - k) {
            int m = (int)std::min<int64_t>(r, N);
            if (!(m & 1)) --m;
            if (m < 3) break;
            const bool odd = ((t + k0 + k) & 1) != 0;
            e = launch_fused(jd, m, odd, shape.fty, shape.fwin, shape.nt != 0, d_t, (int)(k0 + k), stream);
            ++enqueued;
            k += m;
        }
    }
    // (the fused shapes' nt is that of their own stores; FP64 300 x 190 x 100 187
    // -> 175 us for a call of one step, FP32 channel 440 x 82 x 300 186 -> 173)
    StepShape one = shape;
    if (N) one.nt = stores_bypass(slab_bytes());
    for (; k < n && e == hipSuccess; ++k) {
        e = launch_step(jd, d_t, (int)(k0 + k), (int)((t + k0 + k) & 1), one, stream);
        ++enqueued;
    }
    return e;
}

uq_status Job::advance(int64_t steps) {
    int L = env_int("UQ_GRAPH_STEPS", 64) & ~1;
    // whole fused blocks in a graph: multiples of 2N (N even) or 2N (N odd,
    // even length keeps every replay starting at an even step)
    if (const int N = fused_n()) L = L / (2 * N) * (2 * N);
    if (use_graph && L >= 2 && steps >= L + 1) {
        if (t & 1) {
            UQ_HIP_TRY(launch_step(jd, d_t, 0, 1, shape, stream));
            ++launches;
            UQ_HIP_TRY(launch_advance(d_t, 1, stream));
            t += 1;
            steps -= 1;
        }
        if (!gexec || graph_len != L) {
            release_graph();
            UQ_HIP_TRY(hipStreamBeginCapture(stream, hipStreamCaptureModeThreadLocal));
            pending_launches = 0;
            hipError_t e = enqueue_steps(0, L);
            graph_launches = pending_launches;
            pending_launches = 0;
            if (e == hipSuccess) e = launch_advance(d_t, L, stream);
            hipGraph_t g = nullptr;
            hipError_t e2 = hipStreamEndCapture(stream, &g);
            if (e != hipSuccess || e2 != hipSuccess) {
                if (g) (void)hipGraphDestroy(g);
                return fail(UQ_EDEVICE, std::string("graph capture failed: ") +
                                            hipGetErrorString(e != hipSuccess ? e : e2));
            }
            graph = g;
            UQ_HIP_TRY(hipGraphInstantiate(&gexec, graph, nullptr, nullptr, 0));
            graph_len = L;
        }
        while (steps >= L) {
            UQ_HIP_TRY(hipGraphLaunch(gexec, stream));
            t += L;
            steps -= L;
            launches += graph_launches;
        }
    }
    if (steps > 0) {
        pending_launches = 0;
        UQ_HIP_TRY(enqueue_steps(0, steps));
        launches += pending_launches;
        UQ_HIP_TRY(launch_advance(d_t, steps, stream));
        t += steps;
    }
    return UQ_OK;
}

Job::~Job() {
    if (stream) (void)hipStreamSynchronize(stream);
    release_graph();
    dfree_all();
    if (ev_in) (void)hipEventDestroy(ev_in);
    if (ev_out) (void)hipEventDestroy(ev_out);
    if (stream) (void)hipStreamDestroy(stream);
}

}  // namespace uqi
