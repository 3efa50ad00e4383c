// HIP kernels (gfx950) of the batched D2Q9 BGK ensemble and its statistics:
// the single-step kernels, initial state, quantities of interest and
// cross-sample statistics, and the host side of the temporally blocked
// kernels (fused_kernels.hip). The arithmetic they share, the storage layouts
// and the references are in lbm_device.h.
#include "lbm_device.h"

#include "fused_shapes.h"

// as in lbm_device.h: no implicit contraction in any kernel
#pragma clang fp contract(off)

namespace uqi {

// One tile of one sample: blockDim.x nodes along x by blockDim.y*CPT rows;
// each thread takes CPT rows blockDim.y apart. All CPT nodes of a thread are gathered before any is
// written back: in the AA pattern a node reads and writes only its own nine
// locations (and in AB reads and writes different slabs), so the nodes are
// independent and the loads of all CPT rows can be in flight together.
template <int P, bool CHANNEL, int PARITY, int CPT, int LAYOUT, bool NT>
__device__ inline void tile_update(const JobDev &j, int64_t t, int64_t smp, int tx, int ty) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    constexpr int MODE = ModeOf<LAYOUT, PARITY>::value;
    const int x = tx * (int)blockDim.x + threadIdx.x;
    if (x >= j.nx) return;
    T *src_all = (T *)(LAYOUT == UQ_LAYOUT_AB && PARITY ? j.f2 : j.f);
    T *dst_all = (T *)(LAYOUT == UQ_LAYOUT_AB && !PARITY ? j.f2 : j.f);
    const double omega_d = j.smp[smp].omega;
    const C omega = (C)omega_d;
    const double u_peak = CHANNEL ? j.smp[smp].u_peak : 0.0;
    const T *src = src_all + smp * 9 * j.plane;
    T *dst = dst_all + smp * 9 * j.plane;
    const int by = (int)blockDim.y;
    const int y0 = ty * by * CPT + threadIdx.y;
    C f[CPT][9];
    uint32_t m[CPT];
    bool live[CPT];
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        const int y = y0 + r * by;
        live[r] = y < j.ny;
        m[r] = 0;
        if (CHANNEL && live[r]) {
            m[r] = j.mask[(int64_t)y * j.pitch + x];
            // solid nodes, and the boundary nodes that k_step_interp updates
            // apart (interpolated links, finite-difference open columns),
            // are not stepped here
            live[r] = !(m[r] & (M_SOLID | M_SPECIAL));
        }
        if (live[r]) gather<P, CHANNEL, MODE, false, false>(j, src, site(j, x, y), m[r], t, u_peak, omega_d, f[r]);
    }
#pragma unroll
    for (int r = 0; r < CPT; ++r) {
        if (!live[r]) continue;
        C drho, ux, uy;
        bgk(f[r], omega, drho, ux, uy);
        scatter<P, CHANNEL, MODE, NT>(j, dst, site(j, x, y0 + r * by), m[r], f[r]);
    }
}

// One step for every live node of every sample of one job.
template <int P, bool CHANNEL, int PARITY, int CPT, int LAYOUT, bool NT>
__global__ __launch_bounds__(256) void k_step(JobDev j, const int64_t *d_t, int k, int tiles_x, int tiles_y,
                                              int64_t ntiles) {
    const int64_t t = *d_t + k;
    const int64_t G = gridDim.x;
    const int64_t per_sample = (int64_t)tiles_x * tiles_y;
    for (int64_t tile = xcd_logical(blockIdx.x, G); tile < ntiles; tile += G) {
        const int64_t smp = tile / per_sample;
        const int64_t rem = tile - smp * per_sample;
        const int ty = (int)(rem / tiles_x), tx = (int)(rem - (int64_t)ty * tiles_x);
        tile_update<P, CHANNEL, PARITY, CPT, LAYOUT, NT>(j, t, smp, tx, ty);
    }
}

// Boundary nodes of jobs with interpolated boundaries (AB layout). Both items
// below read only the source slab and write only their own nodes of the
// destination slab, so they and the bulk tiles of the same step are
// independent.
//
// A node with interpolated cylinder links (listed in j.special) of one
// sample. Every value that any of its links may want (its streamed and own
// populations, those of the nodes behind, the link fractions) is loaded before
// the first is used: with the loads under each link's branch a step of the
// list was a chain of some ten memory latencies (12.7 us for 80 nodes).
template <int P>
__device__ inline void qlink_node(const JobDev &j, const void *src_all, void *dst_all, int64_t t, int64_t smp, int e) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    const int node = j.special[e];
    const int y = node / (int)j.pitch, x = node - y * (int)j.pitch;
    const uint32_t m = j.mask[node];
    const Site s = site(j, x, y);
    const T *base = (const T *)src_all + smp * 9 * j.plane;
    const SampleDev &sd = j.smp[smp];
    const float inv = j.inv_scale;
    C f[9], own[9], behind[9];
    double q[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        f[i] = PR::ld(base + i * j.plane + (int64_t)sy_of(s, -CYd[i]) * j.pitch + sx_of(s, -CXd[i]), inv);
        own[i] = PR::ld(base + i * j.plane + node, inv);
        behind[i] = PR::ld(base + OPPd[i] * j.plane + (int64_t)sy_of(s, CYd[i]) * j.pitch + sx_of(s, CXd[i]), inv);
        q[i] = j.q[(int64_t)i * j.ny * j.pitch + node];
    }
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        const bool bb = (m >> (M_BB + i)) & 1u;
        const C fk = own[OPPd[i]];
        C v = fk;  // a half-way link (channel wall)
        if (q[i] > 0.0) {
            if (q[i] >= 0.5) {
                const double a = 1.0 / (2.0 * q[i]);
                v = (C)a * fk + (C)(1.0 - a) * own[i];
            } else {
                v = (C)(2.0 * q[i]) * fk + (C)(1.0 - 2.0 * q[i]) * behind[i];
            }
        }
        f[i] = bb ? v : f[i];
    }
    // beyond an open column, as in the gather
    if (m & (0x1FFu << M_OPEN)) {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = ((m >> (M_OPEN + i)) & 1u) ? C(0) : f[i];
        if (t > 0 && j.xbc != UQ_XBC_INTERP) zou_he(f, j, x, y, t, sd.u_peak);
    }
    C drho, ux, uy;
    bgk(f, (C)sd.omega, drho, ux, uy);
    scatter<P, true, AB_PULL, false>(j, (T *)dst_all + smp * 9 * j.plane, s, m, f);
}

// A chunk of FD_ROWS rows of an open column (inlet chunks first) of a
// finite-difference inlet/outlet, of one sample. A workgroup's threads
// gather, one node each, the column node and the two nodes next to it into the
// fluid, for the chunk's rows plus two halo rows on each side, and share the
// velocities through LDS; the column threads then rebuild, collide and store.
constexpr int FD_RB = 85, FD_HALO = 2, FD_ROWS = FD_RB - 2 * FD_HALO, FD_BLOCK = 256;
struct FdLds {
    double ub[FD_RB], u1x[FD_RB], u1y[FD_RB], u2x[FD_RB], u2y[FD_RB];
};

template <int P>
__device__ inline void fd_column_chunk(const JobDev &j, const void *src_all, void *dst_all, int64_t t, int64_t smp,
                                       int item, FdLds &l) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    const int chunks = (j.ny + FD_ROWS - 1) / FD_ROWS;
    const bool inlet = item < chunks;
    const int chunk = inlet ? item : item - chunks;
    const int tid = (int)(threadIdx.y * blockDim.x + threadIdx.x);
    const int c = tid / FD_RB, r = tid - c * FD_RB;  // c: 0 the column, 1 and 2 into the fluid
    const int x = inlet ? c : j.nx - 1 - c;
    const int y = chunk * FD_ROWS - FD_HALO + r;
    const bool valid = c < 3 && y >= 0 && y < j.ny;
    const bool own = valid && c == 0 && r >= FD_HALO && r < FD_RB - FD_HALO;
    const uint32_t m = valid ? j.mask[(int64_t)y * j.pitch + x] : 0u;
    const SampleDev &sd = j.smp[smp];
    const T *src = (const T *)src_all + smp * 9 * j.plane;
    C f[9];
    double rho = 1.0, ux = 0.0;
    if (valid) {
        const Site st = site(j, x, y);
        if (c == 0) {
            gather<P, true, AB_PULL, false, false>(j, src, st, m, t, sd.u_peak, sd.omega, f);
            fd_state(j, f, inlet, y, t, sd.u_peak, rho, ux);
            l.ub[r] = ux;
        } else {
            C drho, gx, gy;
            gather<P, true, AB_PULL, false, true>(j, src, st, m, t, sd.u_peak, sd.omega, f);
            moments(f, drho, gx, gy);
            if (c == 1) {
                l.u1x[r] = (double)gx;
                l.u1y[r] = (double)gy;
            } else {
                l.u2x[r] = (double)gx;
                l.u2y[r] = (double)gy;
            }
        }
    }
    __syncthreads();
    if (own) {
        if (t > 0) {  // the state at t = 0 is the rest state as gathered
            const double sdx = inlet ? 1.0 : -1.0;
            const double dyux = fd_dy(y, j.ny, l.ub[r - 2], l.ub[r - 1], ux, l.ub[r + 1], l.ub[r + 2]);
            const double dxux = sdx * (-3.0 * ux + 4.0 * l.u1x[r] - l.u2x[r]) * 0.5;
            const double dxuy = sdx * (-3.0 * 0.0 + 4.0 * l.u1y[r] - l.u2y[r]) * 0.5;
            fd_rebuild(f, rho, ux, dxux, dxuy, dyux, sd.omega);
        }
        C drho, gx, gy;
        bgk(f, (C)sd.omega, drho, gx, gy);
        scatter<P, true, AB_PULL, false>(j, (T *)dst_all + smp * 9 * j.plane, site(j, x, y), m, f);
    }
}

// One step of a job with interpolated boundaries in one launch: workgroups
// [0, nfd) take the open-column chunks, [nfd, nb) the cylinder's nodes (one
// per thread, samples side by side), the rest the bulk tiles of k_step. The
// boundary work, the longest chain of loads, starts first; handed out among
// the tiles, or sample by sample with them, it took longer (11 samples of 440 x
// 80: 11.7 us per step first, 15.1 and 14.5 so). As three kernels, two of them
// on a side stream, the step took 28.5 us, half of it the host's: a graph node
// per kernel and a fork and a join per step. 1000 samples: 618 us, as before
// (held to 8 waves per SIMD; 636 at the 7 the compiler takes otherwise).
template <int P, int PARITY, bool NT>
__global__ __launch_bounds__(FD_BLOCK, P == UQ_FP64 ? 4 : 8) void k_step_interp(JobDev j, const int64_t *d_t, int k,
                                                                               int fd_items, int nfd, int nb,
                                                                               int tiles_x, int tiles_y,
                                                                               int64_t ntiles) {
    __shared__ FdLds lds;
    const int64_t t = *d_t + k;
    const void *src = PARITY ? j.f2 : j.f;
    void *dst = PARITY ? j.f : j.f2;
    const int g = blockIdx.x;
    if (g < nb) {
        if (g < nfd) {
            fd_column_chunk<P>(j, src, dst, t, g / fd_items, g % fd_items, lds);
        } else {
            const int64_t w = (int64_t)(g - nfd) * FD_BLOCK + threadIdx.y * blockDim.x + threadIdx.x;
            const int64_t smp = w / j.n_special;
            if (smp < j.S) qlink_node<P>(j, src, dst, t, smp, (int)(w - smp * j.n_special));
        }
        return;
    }
    const int64_t per_sample = (int64_t)tiles_x * tiles_y, G = (int64_t)gridDim.x - nb;
    for (int64_t tile = xcd_logical(g - nb, G); tile < ntiles; tile += G) {
        const int64_t smp = tile / per_sample;
        const int64_t rem = tile - smp * per_sample;
        const int ty = (int)(rem / tiles_x), tx = (int)(rem - (int64_t)ty * tiles_x);
        tile_update<P, true, PARITY, 1, UQ_LAYOUT_AB, NT>(j, t, smp, tx, ty);
    }
}
// The same address as a pointer into global memory. A pointer loaded from a
// table in device memory is generic to the compiler, and the accesses through
// it compile to flat instructions (64-bit addresses in vector registers, and
// waits on the LDS counter as well); rebuilt from its integer value in the
// global address space, they compile to global loads and stores, as those of
// a kernel argument do.
template <typename T>
__device__ inline T *global_ptr(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)(uintptr_t)p;
}

// One step for every live node of every sample of every job in a table
// (continuous batching). Jobs may differ in geometry, lattice, sample count
// and step parity; all use the AA layout, one row per thread. Tiles of job q
// are the global tiles [tile0_q, tile0_{q+1}); a job whose step count has
// reached its target is skipped, so the same launch (or captured graph) stays
// valid while jobs finish.
template <int P>
__global__ __launch_bounds__(256) void k_step_multi(const MultiJob *jobs, int njobs, int64_t ntiles, int k) {
    const int64_t G = gridDim.x;
    for (int64_t tile = xcd_logical(blockIdx.x, G); tile < ntiles; tile += G) {
        int lo = 0, hi = njobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].tile0 <= tile) lo = mid;
            else hi = mid - 1;
        }
        const MultiJob &q = jobs[lo];
        const int64_t t = q.t + k;
        if (t >= q.n_steps || k >= q.adv) continue;
        JobDev jd = q.j;
        jd.f = global_ptr(jd.f);
        jd.smp = global_ptr(jd.smp);
        jd.mask = global_ptr(jd.mask);
        const int64_t per_sample = (int64_t)q.tiles_x * q.tiles_y;
        const int64_t local = tile - q.tile0;
        const int64_t smp = local / per_sample;
        const int64_t rem = local - smp * per_sample;
        const int ty = (int)(rem / q.tiles_x), tx = (int)(rem - (int64_t)ty * q.tiles_x);
        if (jd.geom == 1) {
            if (t & 1) tile_update<P, true, 1, 1, UQ_LAYOUT_AA, false>(jd, t, smp, tx, ty);
            else tile_update<P, true, 0, 1, UQ_LAYOUT_AA, false>(jd, t, smp, tx, ty);
        } else {
            if (t & 1) tile_update<P, false, 1, 1, UQ_LAYOUT_AA, false>(jd, t, smp, tx, ty);
            else tile_update<P, false, 0, 1, UQ_LAYOUT_AA, false>(jd, t, smp, tx, ty);
        }
    }
}

__global__ void k_advance_multi(MultiJob *jobs, int njobs) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < njobs) jobs[q].t += jobs[q].adv;
}

// ------------------------------------------------------------------ init
// Equilibrium start. AA stores f~_eq(x) in slot i of node x. AB stores
// g_i(x - c_i) = f~_eq,i(x) (the value the first pull of node x reads), so
// every node computes its own equilibrium once and writes it to the nine
// nodes x - c_i (periodic wrap; the channel starts at rest, f~ = 0).
template <int P, int LAYOUT>
__global__ __launch_bounds__(256) void k_init(JobDev j) {
    using PR = Prec<P>;
    using T = typename PR::T;
    const int64_t cells = (int64_t)j.ny * j.pitch;
    for (int64_t smp = blockIdx.y; smp < j.S; smp += gridDim.y) {
        T *base = (T *)j.f + smp * 9 * j.plane;
        const SampleDev sd = j.smp[smp];
        for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cells;
             c += (int64_t)gridDim.x * blockDim.x) {
            const int y = (int)(c / j.pitch), x = (int)(c - (int64_t)y * j.pitch);
            double f[9];
            for (int i = 0; i < 9; ++i) f[i] = 0.0;
            if (x < j.nx && j.geom == 0) {
                double ux, uy, p;
                if (j.init == UQ_INIT_TGV_HARMONIC) {
                    // perturbed vortex (Eq. taylorGreen), two periods per side,
                    // amplitude u0 (1 + eps) with first-order harmonics of 2 kappa
                    const double kx = 4.0 * M_PI / j.nx, ky = 4.0 * M_PI / j.ny;
                    const double ax = kx * x, ay = ky * y;
                    const double sx = sin(2.0 * ax), cx = cos(2.0 * ax), sy = sin(2.0 * ay), cy = cos(2.0 * ay);
                    const double eps = 0.25 * (sd.zeta[0] * sx * sy + sd.zeta[1] * sx * cy + sd.zeta[2] * cx * sy +
                                               sd.zeta[3] * cx * cy);
                    const double uR = sd.u0 * (1.0 + eps);
                    ux = -uR * cos(ax) * sin(ay);
                    uy = uR * sin(ax) * cos(ay);
                    p = -0.25 * uR * uR * (cos(2.0 * ax) + cos(2.0 * ay));
                } else {
                    // Taylor-Green vortex (Eqs. TGV_vel, TGV_press at t = 0)
                    const double kx = 2.0 * M_PI / j.nx, ky = 2.0 * M_PI / j.ny;
                    const double ax = kx * x + sd.phase_x, ay = ky * y + sd.phase_y;
                    ux = -sd.u0 * cos(ax) * sin(ay);
                    uy = sd.u0 * sin(ax) * cos(ay);
                    p = -0.25 * sd.u0 * sd.u0 * (cos(2.0 * ax) + (kx / ky) * (kx / ky) * cos(2.0 * ay));
                }
                const double drho = 3.0 * p, rho = 1.0 + drho;  // rho = 1 + p/cs2
                const double uu = 1.5 * (ux * ux + uy * uy);
                for (int i = 0; i < 9; ++i) {
                    const double cu = CXd[i] * ux + CYd[i] * uy;
                    f[i] = wgt<double>(i) * (drho + rho * (3.0 * cu + 4.5 * cu * cu - uu));
                }
            }
            if (LAYOUT == UQ_LAYOUT_AB && x < j.nx) {
                const Site s = site(j, x, y);
                for (int i = 0; i < 9; ++i) {
                    const int xd = sx_of(s, -CXd[i]), yd = sy_of(s, -CYd[i]);
                    PR::st(base + i * j.plane + (int64_t)yd * j.pitch + xd, (typename PR::C)f[i], j.scale);
                }
            } else if (LAYOUT != UQ_LAYOUT_AB) {
                for (int i = 0; i < 9; ++i) PR::st(base + i * j.plane + c, (typename PR::C)f[i], j.scale);
            }
        }
    }
}

// The state at step t of an AB job, in the AA layout of that step, in the other
// slab: bit copies of the stored values. Even t: every node its pulls (a pull
// beyond an open column brings whatever lies there, as in the gather: its rule
// overwrites it); odd t: f*_i(x, t-1) in slot opp(i). Once per job at most, for
// memory that something else needs more; one pass over both slabs.
template <typename T>
__global__ __launch_bounds__(256) void k_to_aa(JobDev j, const T *src_all, T *dst_all, int odd) {
    const int64_t cells = (int64_t)j.ny * j.nx;
    for (int64_t smp = blockIdx.y; smp < j.S; smp += gridDim.y) {
        const T *src = src_all + smp * 9 * j.plane;
        T *dst = dst_all + smp * 9 * j.plane;
        for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cells;
             c += (int64_t)gridDim.x * blockDim.x) {
            const int y = (int)(c / j.nx), x = (int)(c - (int64_t)y * j.nx);
            const Site s = site(j, x, y);
            const int64_t own = (int64_t)y * j.pitch + x;
            const uint32_t m = j.geom == 1 ? j.mask[own] : 0u;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                if (odd) {
                    dst[OPPd[i] * j.plane + own] = src[i * j.plane + own];
                } else {
                    const bool bb = (m >> (M_BB + i)) & 1u;
                    const int64_t from = (int64_t)sy_of(s, -CYd[i]) * j.pitch + sx_of(s, -CXd[i]);
                    dst[i * j.plane + own] = src[bb ? OPPd[i] * j.plane + own : i * j.plane + from];
                }
            }
        }
    }
}

// ------------------------------------------------------------------ QoIs
// Neumaier's compensated sum
struct NSum {
    double s = 0.0, c = 0.0;
    __device__ inline void add(double x) {
        const double t = s + x;
        c += (fabs(s) >= fabs(x)) ? ((s - t) + x) : ((x - t) + s);
        s = t;
    }
    // another sum's terms
    __device__ inline void join(double os, double oc) {
        add(os);
        c += oc;
    }
    __device__ inline double val() const { return s + c; }
};

// The sums of a wave's 64 lanes, joined in a fixed tree: whole in lane 0.
__device__ inline void wave_join(NSum &a) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) a.join(__shfl_down(a.s, d), __shfl_down(a.c, d));
}

// KE, momentum-exchange force and non-finite count of a sample, or of one of
// its chunks of `per` nodes: workgroup (chunk, sample). A job with fewer
// samples than the card takes workgroups is cut into chunks, whose sums go to
// part[sample][chunk] = {KE, Fx, Fy as sum and compensation, count} and are
// joined by k_qoi_join (one workgroup per sample read 1024^2 nodes x 16
// samples in 3.2 ms, 0.2 TB/s; latency bound).
template <int P, bool CHANNEL, int MODE>
__global__ __launch_bounds__(256) void k_qoi(JobDev j, int64_t t, int per, double *part, double *out) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    const int64_t smp = (int64_t)blockIdx.y * gridDim.z + blockIdx.z;
    if (smp >= j.S) return;
    const T *base = (const T *)(MODE == AB_PULL && (t & 1) ? j.f2 : j.f) + smp * 9 * j.plane;
    const SampleDev sd = j.smp[smp];
    NSum ke, fx, fy;
    double bad = 0.0;
    const uint32_t nx = (uint32_t)j.nx, first = blockIdx.x * (uint32_t)per;
    const uint32_t end = min(nx * (uint32_t)j.ny, first + (uint32_t)per);
    for (uint32_t c = first + threadIdx.x; c < end; c += blockDim.x) {
        const int y = (int)(c / nx), x = (int)(c - (uint32_t)y * nx);
        uint32_t m = 0;
        if (CHANNEL) {
            m = j.mask[(int64_t)y * j.pitch + x];
            if (m & M_SOLID) continue;
        }
        const Site s = site(j, x, y);
        C f[9], drho, ux, uy;
        gather<P, CHANNEL, MODE>(j, base, s, m, t, sd.u_peak, sd.omega, f);
        if (CHANNEL && (m & (0x1FFu << M_CYL))) {
            bgk(f, (C)sd.omega, drho, ux, uy);
            for (int k = 1; k < 9; ++k)
                if (m & (1u << (M_CYL + k))) {
                    // exchange on link k: c_k (f*_k(x) + what the wall returns
                    // at t+1), both unshifted; half-way: 2 c_k f*_k(x)
                    const double fk = (double)f[k] + wgt<double>(k);
                    double back = fk;
                    if (MODE == AB_PULL && (m & M_QLINK)) {
                        const int i = OPPd[k];
                        const double q = j.q[(int64_t)i * j.ny * j.pitch + (int64_t)y * j.pitch + x];
                        if (q >= 0.5) {
                            const double a = 1.0 / (2.0 * q);
                            back = a * fk + (1.0 - a) * ((double)f[i] + wgt<double>(i));
                        } else if (q > 0.0) {
                            // f*_k of the node behind, x - c_k = x + c_i
                            const int xb = sx_of(s, CXd[i]), yb = sy_of(s, CYd[i]);
                            C g[9], gr, gx, gy;
                            gather<P, CHANNEL, MODE>(j, base, site(j, xb, yb), j.mask[(int64_t)yb * j.pitch + xb], t,
                                                     sd.u_peak, sd.omega, g);
                            bgk(g, (C)sd.omega, gr, gx, gy);
                            back = 2.0 * q * fk + (1.0 - 2.0 * q) * ((double)g[k] + wgt<double>(k));
                        }
                    }
                    fx.add(CXd[k] * (fk + back));
                    fy.add(CYd[k] * (fk + back));
                }
        } else {
            moments(f, drho, ux, uy);
        }
        const double dux = (double)ux, duy = (double)uy;
        if (!isfinite(dux) || !isfinite(duy) || !isfinite((double)drho)) bad += 1.0;
        ke.add(dux * dux + duy * duy);
    }
    // a fixed tree over the lanes, then the waves in order (deterministic)
    __shared__ double red[4][QOI_PART];
    wave_join(ke);
    if (CHANNEL) {
        wave_join(fx);
        wave_join(fy);
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) bad += __shfl_down(bad, d);
    if ((threadIdx.x & 63) == 0) {
        double *r = red[threadIdx.x >> 6];
        r[0] = ke.s, r[1] = ke.c, r[2] = fx.s, r[3] = fx.c, r[4] = fy.s, r[5] = fy.c, r[6] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) {
            ke.join(red[w][0], red[w][1]);
            fx.join(red[w][2], red[w][3]);
            fy.join(red[w][4], red[w][5]);
            bad += red[w][6];
        }
        if (gridDim.x > 1) {
            double *q = part + (smp * gridDim.x + blockIdx.x) * QOI_PART;
            q[0] = ke.s, q[1] = ke.c, q[2] = fx.s, q[3] = fx.c, q[4] = fy.s, q[5] = fy.c, q[6] = bad;
        } else {
            out[smp * 4] = ke.val() * j.ke_norm;
            out[smp * 4 + 1] = fx.val();
            out[smp * 4 + 2] = fy.val();
            out[smp * 4 + 3] = bad;
        }
    }
}

// Per-sample fields: out[s][4][ny][nx] = ux, uy, rho, |u| (0 at solid nodes).
template <int P, bool CHANNEL, int MODE>
__global__ __launch_bounds__(256) void k_fields(JobDev j, int64_t t, double *out) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    const int64_t cells = (int64_t)j.nx * j.ny;
    for (int64_t smp = blockIdx.y; smp < j.S; smp += gridDim.y) {
    const T *base = (const T *)(MODE == AB_PULL && (t & 1) ? j.f2 : j.f) + smp * 9 * j.plane;
    const double u_peak = j.smp[smp].u_peak, omega = j.smp[smp].omega;
    double *o = out + smp * 4 * cells;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cells; c += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(c / j.nx), x = (int)(c - (int64_t)y * j.nx);
        uint32_t m = 0;
        if (CHANNEL) {
            m = j.mask[(int64_t)y * j.pitch + x];
            if (m & M_SOLID) {
                o[c] = 0.0;
                o[cells + c] = 0.0;
                o[2 * cells + c] = 0.0;
                o[3 * cells + c] = 0.0;
                continue;
            }
        }
        const Site s = site(j, x, y);
        C f[9], drho, ux, uy;
        gather<P, CHANNEL, MODE>(j, base, s, m, t, u_peak, omega, f);
        moments(f, drho, ux, uy);
        o[c] = (double)ux;
        o[cells + c] = (double)uy;
        o[2 * cells + c] = 1.0 + (double)drho;
        o[3 * cells + c] = sqrt((double)ux * (double)ux + (double)uy * (double)uy);
    }
    }
}

// One sample's unshifted populations, natural order [9][ny][nx] in double.
template <int P, bool CHANNEL, int MODE>
__global__ __launch_bounds__(256) void k_export(JobDev j, int64_t t, int64_t smp, double *out) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    const int64_t cells = (int64_t)j.nx * j.ny;
    const T *base = (const T *)(MODE == AB_PULL && (t & 1) ? j.f2 : j.f) + smp * 9 * j.plane;
    const double u_peak = j.smp[smp].u_peak, omega = j.smp[smp].omega;
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < cells; c += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(c / j.nx), x = (int)(c - (int64_t)y * j.nx);
        uint32_t m = 0;
        if (CHANNEL) {
            m = j.mask[(int64_t)y * j.pitch + x];
            if (m & M_SOLID) {
                for (int i = 0; i < 9; ++i) out[i * cells + c] = 0.0;
                continue;
            }
        }
        const Site s = site(j, x, y);
        C f[9];
        gather<P, CHANNEL, MODE>(j, base, s, m, t, u_peak, omega, f);
        for (int i = 0; i < 9; ++i) out[i * cells + c] = (double)f[i] + wgt<double>(i);
    }
}

// ------------------------------------------------------------------ field statistics from the slab
// Statistics of a field QoI read straight from the populations, without a
// per-sample field buffer: the value of a (sample, node) is formed from its
// pulled populations exactly as k_fields forms it (velocity u_x, u_y; density
// 1 + drho; speed |u|; 0 at solid nodes), and every sum over the samples is
// Neumaier-compensated (FP64) in an order fixed by the lattice and the sample
// count.
// Field QoIs: which = 0 velocity (two components), 1 density, 2 speed.
constexpr int FP_JB = 16;  // samples per LDS block of values
constexpr int FP_KA = 12;  // (component, coefficient) pairs per thread

template <int P, bool CHANNEL, int MODE>
__device__ inline void field_value(const JobDev &j, const typename Prec<P>::T *base, int64_t t, int64_t smp,
                                   int64_t c, int which, double &v0, double &v1) {
    using C = typename Prec<P>::C;
    const int y = (int)((uint32_t)c / (uint32_t)j.nx), x = (int)c - y * j.nx;
    uint32_t m = 0;
    v0 = v1 = 0.0;
    if (CHANNEL) {
        m = j.mask[(int64_t)y * j.pitch + x];
        if (m & M_SOLID) return;
    }
    C f[9], drho, ux, uy;
    gather<P, CHANNEL, MODE>(j, base, site(j, x, y), m, t, j.smp[smp].u_peak, j.smp[smp].omega, f);
    moments(f, drho, ux, uy);
    if (which == 0) {
        v0 = (double)ux;
        v1 = (double)uy;
    } else if (which == 1) {
        v0 = 1.0 + (double)drho;
    } else {
        v0 = sqrt((double)ux * (double)ux + (double)uy * (double)uy);
    }
}

// SC-gPC coefficients c_k(o) = sum_j a_j Phi_k(xi_j) M_j(o) (Eq.
// coef_discrete) of a field: a workgroup takes 64 nodes (one per lane) and
// 4 FP_KA (component, k) pairs (FP_KA per wave); per block of FP_JB samples
// the four waves form the values of the 64 nodes into LDS, then every
// thread adds its pairs' terms. coeffs[k][n_out], o = component * cells + node.
template <int P, bool CHANNEL, int MODE>
__global__ __launch_bounds__(256) void k_field_coeffs(JobDev j, int64_t t, int which,
                                                      const double *__restrict__ wphi, int K, double *coeffs) {
    using T = typename Prec<P>::T;
    __shared__ double val[FP_JB][2][64];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t cells = (int64_t)j.nx * j.ny;
    const int comps = which == 0 ? 2 : 1;
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const bool on = c < cells;
    const int npair = comps * K;
    const int p0 = (int)blockIdx.y * 4 * FP_KA + w * FP_KA;
    int kq[FP_KA], cq[FP_KA];
#pragma unroll
    for (int q = 0; q < FP_KA; ++q) {
        const int p = min(p0 + q, npair - 1);
        cq[q] = p / K;
        kq[q] = p - cq[q] * K;
    }
    const T *slab = (const T *)(MODE == AB_PULL && (t & 1) ? j.f2 : j.f);
    NSum acc[FP_KA];
    for (int64_t j0 = 0; j0 < j.S; j0 += FP_JB) {
        const int nj = (int)min((int64_t)FP_JB, j.S - j0);
#pragma unroll
        for (int i = 0; i < FP_JB / 4; ++i) {
            const int jj = w + 4 * i;
            double v0 = 0.0, v1 = 0.0;
            if (jj < nj && on)
                field_value<P, CHANNEL, MODE>(j, slab + (j0 + jj) * 9 * j.plane, t, j0 + jj, c, which, v0, v1);
            val[jj][0][lane] = v0;
            val[jj][1][lane] = v1;
        }
        __syncthreads();
        for (int jj = 0; jj < nj; ++jj) {
            const double *wr = wphi + (j0 + jj) * K;
#pragma unroll
            for (int q = 0; q < FP_KA; ++q) acc[q].add(wr[kq[q]] * val[jj][cq[q]][lane]);
        }
        __syncthreads();
    }
    if (on) {
#pragma unroll
        for (int q = 0; q < FP_KA; ++q)
            if (p0 + q < npair) coeffs[(int64_t)kq[q] * comps * cells + cq[q] * cells + c] = acc[q].val();
    }
}

// The rest of a field's statistics (both velocity components of a node at
// once): SC (wphi != null): mean = c_0, var = sum_{k>=1} c_k^2 (Eq. gpc_std)
// and the quadrature variance sum_j a_j (M_j - mean)^2; MC: mean (Eq.
// meanMCS), var with 1/(N-1) (Eq. varMCS) and 1/N, two passes.
// A workgroup takes 64 nodes, one per lane; its G = blockDim / 64 waves take
// every G-th sample and their sums are joined in order, so the result depends
// on G (the lattice and the sample count) only within the compensation. With
// one thread per node over all samples a 128^2 lattice gave 64 workgroups, each
// a serial chain of 2 x 4096 gathers: 5.5 ms for 2 x 0.6 GB.
constexpr int FF_MAX_G = 16;
template <int P, bool CHANNEL, int MODE>
__global__ __launch_bounds__(64 * FF_MAX_G) void k_field_finish(JobDev j, int64_t t, int which,
                                                                const double *__restrict__ a, int K,
                                                                const double *coeffs, double *mean, double *var,
                                                                double *var_alt) {
    using T = typename Prec<P>::T;
    __shared__ double red[FF_MAX_G][4][64];
    const int64_t cells = (int64_t)j.nx * j.ny;
    const int comps = which == 0 ? 2 : 1;
    const int64_t n_out = comps * cells;
    const int lane = threadIdx.x & 63, G = blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t c = (int64_t)blockIdx.x * 64 + lane;
    const bool on = c < cells;
    const T *slab = (const T *)(MODE == AB_PULL && (t & 1) ? j.f2 : j.f);
    // the waves' sums of two quantities, joined: the same in every wave
    auto join = [&](const NSum *s, double *v) {
        red[w][0][lane] = s[0].s;
        red[w][1][lane] = s[0].c;
        red[w][2][lane] = s[1].s;
        red[w][3][lane] = s[1].c;
        __syncthreads();
        NSum a0, a1;
        for (int g = 0; g < G; ++g) {
            a0.join(red[g][0][lane], red[g][1][lane]);
            a1.join(red[g][2][lane], red[g][3][lane]);
        }
        v[0] = a0.val();
        v[1] = a1.val();
        __syncthreads();
    };
    double mu[2] = {0.0, 0.0};
    if (K > 0) {
        if (on)
            for (int q = 0; q < comps; ++q) {
                const int64_t o = q * cells + c;
                mu[q] = coeffs[o];
                if (w != 0) continue;
                NSum v;
                for (int k = 1; k < K; ++k) {
                    const double ck = coeffs[(int64_t)k * n_out + o];
                    v.add(ck * ck);
                }
                mean[o] = mu[q];
                var[o] = v.val();
            }
    } else {
        NSum s[2];
        if (on)
#pragma unroll 2
            for (int64_t smp = w; smp < j.S; smp += G) {
                double v0, v1;
                field_value<P, CHANNEL, MODE>(j, slab + smp * 9 * j.plane, t, smp, c, which, v0, v1);
                s[0].add(v0);
                s[1].add(v1);
            }
        join(s, mu);
        mu[0] /= (double)j.S;
        mu[1] /= (double)j.S;
    }
    NSum q[2];
    if (on)
#pragma unroll 2
        for (int64_t smp = w; smp < j.S; smp += G) {
            double v0, v1;
            field_value<P, CHANNEL, MODE>(j, slab + smp * 9 * j.plane, t, smp, c, which, v0, v1);
            const double e0 = v0 - mu[0], e1 = v1 - mu[1];
            if (K > 0) {
                q[0].add(a[smp] * e0 * e0);
                q[1].add(a[smp] * e1 * e1);
            } else {
                q[0].add(e0 * e0);
                q[1].add(e1 * e1);
            }
        }
    double qs[2];
    join(q, qs);
    if (!on || w != 0) return;
    for (int k = 0; k < comps; ++k) {
        const int64_t o = k * cells + c;
        if (K > 0) {
            var_alt[o] = qs[k];
        } else {
            mean[o] = mu[k];
            var[o] = j.S > 1 ? qs[k] / (double)(j.S - 1) : 0.0;
            var_alt[o] = qs[k] / (double)j.S;
        }
    }
}

// ------------------------------------------------------------------ scalar statistics
// A scalar QoI (one value per sample): every sum over the samples is split
// across a workgroup's 256 threads (thread r takes samples r, r + 256, ...
// in order, a compensated partial each) and the partials are joined in a fixed
// tree of compensated sums, so the result does not depend on timing (one
// thread adding up 256 partials took most of these kernels' 8 us). SC: workgroup k forms c_k (Eq. coef_discrete); then one workgroup
// forms mean = c_0, var = sum_{k>=1} c_k^2 and the quadrature variance. MC:
// one workgroup forms mean, var (1/(N-1)) and var_alt (1/N).
__device__ inline double block_nsum(NSum part, double *red) {
    wave_join(part);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        red[2 * w] = part.s;
        red[2 * w + 1] = part.c;
    }
    __syncthreads();
    NSum acc;
    for (int i = 0; i < 4; ++i) acc.join(red[2 * i], red[2 * i + 1]);
    __syncthreads();
    return acc.val();
}

__global__ __launch_bounds__(256) void k_scalar_coeffs(const double *M, int64_t S, const double *wphi, int K,
                                                       double *coeffs) {
    __shared__ double red[8];
    const int k = blockIdx.x;
    NSum acc;
    for (int64_t jx = threadIdx.x; jx < S; jx += blockDim.x) acc.add(wphi[jx * K + k] * M[jx]);
    const double v = block_nsum(acc, red);
    if (threadIdx.x == 0) coeffs[k] = v;
}

__global__ __launch_bounds__(256) void k_scalar_finish(const double *M, int64_t S, const double *a, int K,
                                                       const double *coeffs, double *mean, double *var,
                                                       double *var_alt) {
    __shared__ double red[8];
    double mu;
    if (K > 0) {
        mu = coeffs[0];
    } else {
        NSum s;
        for (int64_t jx = threadIdx.x; jx < S; jx += blockDim.x) s.add(M[jx]);
        mu = block_nsum(s, red) / (double)S;
    }
    NSum q;
    for (int64_t jx = threadIdx.x; jx < S; jx += blockDim.x) {
        const double e = M[jx] - mu;
        q.add(K > 0 ? a[jx] * e * e : e * e);
    }
    const double qs = block_nsum(q, red);
    if (threadIdx.x == 0) {
        mean[0] = mu;
        if (K > 0) {
            NSum v;
            for (int k = 1; k < K; ++k) v.add(coeffs[k] * coeffs[k]);
            var[0] = v.val();
            var_alt[0] = qs;
        } else {
            var[0] = S > 1 ? qs / (double)(S - 1) : 0.0;
            var_alt[0] = qs / (double)S;
        }
    }
}

// ------------------------------------------------------------------ small kernels
__global__ void k_advance(int64_t *d_t, int64_t n) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *d_t += n;
}

// The chunks of a sample in order (chunks > 1), and flag[0] = smallest s < S
// with qoi[4s + 3] != 0 (non-finite values in sample s), else S. One workgroup.
__global__ __launch_bounds__(256) void k_qoi_join(double ke_norm, int64_t S, int chunks, const double *part,
                                                  double *qoi, int64_t *flag) {
    __shared__ int64_t red[256];
    int64_t first = S;
    for (int64_t s = threadIdx.x; s < S; s += blockDim.x) {
        double bad;
        if (chunks > 1) {
            NSum ke, fx, fy;
            bad = 0.0;
            for (int k = 0; k < chunks; ++k) {
                const double *q = part + (s * chunks + k) * QOI_PART;
                ke.join(q[0], q[1]);
                fx.join(q[2], q[3]);
                fy.join(q[4], q[5]);
                bad += q[6];
            }
            qoi[4 * s] = ke.val() * ke_norm;
            qoi[4 * s + 1] = fx.val();
            qoi[4 * s + 2] = fy.val();
            qoi[4 * s + 3] = bad;
        } else {
            bad = qoi[4 * s + 3];
        }
        if (bad != 0.0 && s < first) first = s;
    }
    red[threadIdx.x] = first;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = min(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) flag[0] = red[0];
}

// which: UQ_QOI_KE -> KE; UQ_QOI_CD / UQ_QOI_CL -> 2 F/(u_peak^2 D) with the
// sample's peak inflow velocity and rho0 = 1
__global__ void k_select(const double *qoi, const SampleDev *smp, int64_t S, int which, double dia, double u_fac,
                         double *M) {
    const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= S) return;
    if (which == UQ_QOI_KE) {
        M[s] = qoi[4 * s];
    } else {
        const double u = u_fac * smp[s].u_peak;
        const double F = which == UQ_QOI_CD ? qoi[4 * s + 1] : qoi[4 * s + 2];
        M[s] = 2.0 * F / (u * u * dia);
    }
}

// ------------------------------------------------------------------ launchers
// Launch a read-only state kernel (QoIs, fields, export) in the access mode
// of the job's layout and the parity of t.
#define UQ_DISPATCH_P(KERNEL, PP, MODE_, CH_, GRID, BLOCK, STREAM, ...)                               \
    do {                                                                                           \
        if (CH_) {                                                                                 \
            if (MODE_ == AA_EVEN) KERNEL<PP, true, AA_EVEN><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);  \
            else if (MODE_ == AA_ODD) KERNEL<PP, true, AA_ODD><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__); \
            else KERNEL<PP, true, AB_PULL><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);               \
        } else {                                                                                   \
            if (MODE_ == AA_EVEN) KERNEL<PP, false, AA_EVEN><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__); \
            else if (MODE_ == AA_ODD) KERNEL<PP, false, AA_ODD><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__); \
            else KERNEL<PP, false, AB_PULL><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);              \
        }                                                                                          \
    } while (0)

#define UQ_DISPATCH(KERNEL, PARITY, GRID, BLOCK, STREAM, ...)                                      \
    do {                                                                                           \
        const int md_ = j.layout == UQ_LAYOUT_AB ? AB_PULL : ((PARITY) ? AA_ODD : AA_EVEN);        \
        const bool ch_ = j.geom == 1;                                                              \
        switch (j.prec) {                                                                          \
            case UQ_FP64: UQ_DISPATCH_P(KERNEL, UQ_FP64, md_, ch_, GRID, BLOCK, STREAM, __VA_ARGS__); break;   \
            case UQ_FP32: UQ_DISPATCH_P(KERNEL, UQ_FP32, md_, ch_, GRID, BLOCK, STREAM, __VA_ARGS__); break;   \
            case UQ_FP16S: UQ_DISPATCH_P(KERNEL, UQ_FP16S, md_, ch_, GRID, BLOCK, STREAM, __VA_ARGS__); break; \
            default: UQ_DISPATCH_P(KERNEL, UQ_BF16S, md_, ch_, GRID, BLOCK, STREAM, __VA_ARGS__); break;       \
        }                                                                                          \
    } while (0)

hipError_t launch_init(const JobDev &j, hipStream_t s) {
    const int64_t cells = (int64_t)j.ny * j.pitch;
    dim3 grid((unsigned)std::min<int64_t>((cells + 255) / 256, 1024), (unsigned)std::min<int64_t>(j.S, 65535));
    const bool ab = j.layout == UQ_LAYOUT_AB;
    switch (j.prec) {
        case UQ_FP64:
            if (ab) k_init<UQ_FP64, UQ_LAYOUT_AB><<<grid, 256, 0, s>>>(j);
            else k_init<UQ_FP64, UQ_LAYOUT_AA><<<grid, 256, 0, s>>>(j);
            break;
        case UQ_FP32:
            if (ab) k_init<UQ_FP32, UQ_LAYOUT_AB><<<grid, 256, 0, s>>>(j);
            else k_init<UQ_FP32, UQ_LAYOUT_AA><<<grid, 256, 0, s>>>(j);
            break;
        case UQ_FP16S:
            if (ab) k_init<UQ_FP16S, UQ_LAYOUT_AB><<<grid, 256, 0, s>>>(j);
            else k_init<UQ_FP16S, UQ_LAYOUT_AA><<<grid, 256, 0, s>>>(j);
            break;
        default:
            if (ab) k_init<UQ_BF16S, UQ_LAYOUT_AB><<<grid, 256, 0, s>>>(j);
            else k_init<UQ_BF16S, UQ_LAYOUT_AA><<<grid, 256, 0, s>>>(j);
            break;
    }
    return hipGetLastError();
}

hipError_t launch_to_aa(const JobDev &j, int64_t t, hipStream_t s) {
    const int64_t cells = (int64_t)j.ny * j.nx;
    dim3 grid((unsigned)std::min<int64_t>((cells + 255) / 256, 1024), (unsigned)std::min<int64_t>(j.S, 65535));
    const int odd = (int)(t & 1);
    const void *src = odd ? j.f2 : j.f;
    void *dst = odd ? j.f : j.f2;
    if (j.prec == UQ_FP64) k_to_aa<<<grid, 256, 0, s>>>(j, (const uint64_t *)src, (uint64_t *)dst, odd);
    else if (j.prec == UQ_FP32) k_to_aa<<<grid, 256, 0, s>>>(j, (const uint32_t *)src, (uint32_t *)dst, odd);
    else k_to_aa<<<grid, 256, 0, s>>>(j, (const uint16_t *)src, (uint16_t *)dst, odd);
    return hipGetLastError();
}

template <int P, bool CH, int CPT>
static void step_p(const JobDev &j, const int64_t *d_t, int k, int parity, bool nt, dim3 grid, dim3 block,
                   hipStream_t s, int tiles_x, int tiles_y, int64_t ntiles) {
#define UQ_STEP(PAR, LAY, NT_) k_step<P, CH, PAR, CPT, LAY, NT_><<<grid, block, 0, s>>>(j, d_t, k, tiles_x, tiles_y, ntiles)
    if (j.layout == UQ_LAYOUT_AB) {
        if (nt) { if (parity) UQ_STEP(1, UQ_LAYOUT_AB, true); else UQ_STEP(0, UQ_LAYOUT_AB, true); }
        else { if (parity) UQ_STEP(1, UQ_LAYOUT_AB, false); else UQ_STEP(0, UQ_LAYOUT_AB, false); }
    } else {
        if (parity) UQ_STEP(1, UQ_LAYOUT_AA, false); else UQ_STEP(0, UQ_LAYOUT_AA, false);
    }
#undef UQ_STEP
}

template <int CPT>
static void step_cpt(const JobDev &j, const int64_t *d_t, int k, int parity, bool nt, dim3 grid, dim3 block,
                     hipStream_t s, int tiles_x, int tiles_y, int64_t ntiles) {
    const bool ch = j.geom == 1;
    switch (j.prec) {
        case UQ_FP64:
            if (ch) step_p<UQ_FP64, true, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            else step_p<UQ_FP64, false, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            break;
        case UQ_FP32:
            if (ch) step_p<UQ_FP32, true, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            else step_p<UQ_FP32, false, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            break;
        case UQ_FP16S:
            if (ch) step_p<UQ_FP16S, true, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            else step_p<UQ_FP16S, false, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            break;
        default:
            if (ch) step_p<UQ_BF16S, true, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            else step_p<UQ_BF16S, false, CPT>(j, d_t, k, parity, nt, grid, block, s, tiles_x, tiles_y, ntiles);
            break;
    }
}

template <int P>
static void step_interp_p(const JobDev &j, const int64_t *d_t, int k, bool odd, bool nt, int64_t tile_groups,
                          dim3 block, hipStream_t s, int tiles_x, int tiles_y) {
    const int64_t ntiles = (int64_t)j.S * tiles_x * tiles_y;
    const int fd_items = j.xbc == UQ_XBC_INTERP ? 2 * ((j.ny + FD_ROWS - 1) / FD_ROWS) : 0;
    const int nfd = fd_items * j.S;
    const int nb = nfd + (int)(((int64_t)j.n_special * j.S + FD_BLOCK - 1) / FD_BLOCK);
    const int64_t G = nb + std::min<int64_t>(tile_groups, 0x3fffffff);
#define UQ_STEP(PAR, NT_)                                                                                             \
    k_step_interp<P, PAR, NT_><<<(unsigned)G, block, 0, s>>>(j, d_t, k, fd_items, nfd, nb, tiles_x, tiles_y, ntiles)
    if (nt) { if (odd) UQ_STEP(1, true); else UQ_STEP(0, true); }
    else { if (odd) UQ_STEP(1, false); else UQ_STEP(0, false); }
#undef UQ_STEP
}

hipError_t launch_step(const JobDev &j, const int64_t *d_t, int k, int parity, const StepShape &shape,
                       hipStream_t s) {
    const bool interp = j.geom == 1 && j.layout == UQ_LAYOUT_AB && (j.xbc == UQ_XBC_INTERP || j.n_special > 0);
    const int cpt = shape.cpt <= 1 || interp ? 1 : 2;
    const int bx = shape.bx == 128 || shape.bx == 256 ? shape.bx : BX;
    const int by = 256 / bx;
    const int tiles_x = (j.nx + bx - 1) / bx;
    const int tiles_y = (j.ny + by * cpt - 1) / (by * cpt);
    const int64_t ntiles = (int64_t)j.S * tiles_x * tiles_y;
    int64_t G = ntiles;
    if (shape.persistent > 0) G = std::min<int64_t>(ntiles, (int64_t)256 * shape.persistent);
    if (G > 0x7fffffff) G = 0x7fffffff;
    dim3 block(bx, by);
    const bool nt = shape.nt != 0;
    if (interp) {
        const bool odd = parity & 1;
        switch (j.prec) {
            case UQ_FP64: step_interp_p<UQ_FP64>(j, d_t, k, odd, nt, G, block, s, tiles_x, tiles_y); break;
            case UQ_FP32: step_interp_p<UQ_FP32>(j, d_t, k, odd, nt, G, block, s, tiles_x, tiles_y); break;
            case UQ_FP16S: step_interp_p<UQ_FP16S>(j, d_t, k, odd, nt, G, block, s, tiles_x, tiles_y); break;
            default: step_interp_p<UQ_BF16S>(j, d_t, k, odd, nt, G, block, s, tiles_x, tiles_y); break;
        }
        return hipGetLastError();
    }
    dim3 grid((unsigned)G);
    if (cpt == 1) step_cpt<1>(j, d_t, k, parity & 1, nt, grid, block, s, tiles_x, tiles_y, ntiles);
    else step_cpt<2>(j, d_t, k, parity & 1, nt, grid, block, s, tiles_x, tiles_y, ntiles);
    return hipGetLastError();
}

hipError_t launch_step_multi(const MultiJob *jobs, int njobs, int64_t ntiles, int k, int prec, hipStream_t s) {
    if (ntiles <= 0 || njobs <= 0) return hipSuccess;
    const int64_t G = std::min<int64_t>(ntiles, 0x7fffffff);
    dim3 block(BX, BY);
    switch (prec) {
        case UQ_FP64: k_step_multi<UQ_FP64><<<(unsigned)G, block, 0, s>>>(jobs, njobs, ntiles, k); break;
        case UQ_FP32: k_step_multi<UQ_FP32><<<(unsigned)G, block, 0, s>>>(jobs, njobs, ntiles, k); break;
        case UQ_FP16S: k_step_multi<UQ_FP16S><<<(unsigned)G, block, 0, s>>>(jobs, njobs, ntiles, k); break;
        default: k_step_multi<UQ_BF16S><<<(unsigned)G, block, 0, s>>>(jobs, njobs, ntiles, k); break;
    }
    return hipGetLastError();
}

hipError_t launch_advance_multi(MultiJob *jobs, int njobs, hipStream_t s) {
    if (njobs <= 0) return hipSuccess;
    k_advance_multi<<<(unsigned)((njobs + 63) / 64), 64, 0, s>>>(jobs, njobs);
    return hipGetLastError();
}
bool fused_supported(const JobDev &j) {
    // periodic AB jobs whose per-sample slab fits one buffer descriptor's range
    const int64_t b = j.prec == UQ_FP64 ? 8 : (j.prec == UQ_FP32 ? 4 : 2);
    return j.geom == 0 && j.layout == UQ_LAYOUT_AB && 9 * j.plane * b < ((int64_t)1 << 31);
}
// strips of at most 64 - 2(N - 1) columns (a wave's 64 lanes less the ring
// of N - 1 columns per side), balanced
void window_strips(int nx, int n, int *W, int *strips) {
    const int wmax = 64 - 2 * (n - 1);
    *strips = (nx + wmax - 1) / wmax;
    *W = (nx + *strips - 1) / *strips;
}
int rows_shape(int prec, int n, int rows, int nx, int *K, int *M) {
    for (int m = 1; m <= 2; ++m) {
        const int k = std::max(2, (nx + 64 * m - 1) / (64 * m));
        if (rows_fit(prec, n, rows, k, m)) {
            *K = k;
            *M = m;
            return 1;
        }
    }
    return 0;
}

static int rows_max_nx(int prec, int n, int rows) {
    int best = 0;
    for (int nx = 64; nx <= 768; nx += 64) {
        int K, M;
        if (rows_shape(prec, n, rows, nx, &K, &M)) best = nx;
    }
    return best;
}

int full_rows_max_nx(int prec, int n) { return rows_max_nx(prec, n, RING_ROWS_TGV); }
int channel_rows_max_nx(int prec, int n) { return rows_max_nx(prec, n, RING_ROWS_CH); }
TileShape tile_shape(int nx, int ny, int n) {
    const int ring = 2 * (n - 1);
    TileShape best{};
    for (int tx = 1; tx <= nx; ++tx) {
        TileShape g;
        g.OW = (nx + tx - 1) / tx;
        if (best.RW && g.OW < 8) break;  // (all ring)
        g.RW = tx == 1 ? nx : g.OW + ring;
        const int rows = TILE_NODES / std::max(1, g.RW);
        if (tx > 1 && g.RW >= nx) continue;  // (a ring that meets itself: fewer tiles or narrower ones)
        g.OH = rows >= ny ? ny : rows - ring;
        if (g.OH < 1) continue;
        g.tiles_x = (nx + g.OW - 1) / g.OW;
        g.tiles_y = (ny + g.OH - 1) / g.OH;
        g.OH = (ny + g.tiles_y - 1) / g.tiles_y;  // of equal height
        g.RH = g.tiles_y == 1 && rows >= ny ? ny : g.OH + ring;
        if (!best.RW || g.tiles_x * g.tiles_y < best.tiles_x * best.tiles_y) best = g;
    }
    return best;
}
int channel_strips_max_n(int prec) { return prec == UQ_FP64 ? 7 : 8; }
void row_strips(int prec, int nx, int n, int *W, int *strips) {
    const int lanes = prec == UQ_FP64 ? 64 * RowStrips<UQ_FP64>::K * RowStrips<UQ_FP64>::M
                                      : 64 * RowStrips<UQ_FP32>::K * RowStrips<UQ_FP32>::M;
    const int wmax = lanes - 2 * (n - 1);
    *strips = (nx + wmax - 1) / wmax;
    *W = (nx + *strips - 1) / *strips;
}

bool channel_fusable(const JobDev &j) {
    const int64_t b = j.prec == UQ_FP64 ? 8 : (j.prec == UQ_FP32 ? 4 : 2);
    return j.geom == 1 && j.layout == UQ_LAYOUT_AB && j.n_special == 0 && j.q == nullptr &&
           j.xbc != UQ_XBC_INTERP && 9 * j.plane * b < ((int64_t)1 << 31) && j.plane * 4 < ((int64_t)1 << 31);
}
// ------------------------------------------------------------------ batched fused launches
// One launch of a batched fused instance (kind 0: periodic rows,
// k_stepR_multi; kind 1: channel rows, k_stepRC_multi; kind 2: strips of
// periodic rows, k_stepRS_multi; kind 3: of channel rows, k_stepRCS_multi):
// every work item of the table's jobs. The server keeps to N in {4, 6, 8}
// (periodic rows), {2, 3, 4} (channel) and 8 (strips) and to single precision
// storage (FP32, FP16S, BF16S), so that a tick of 48 steps holds a whole number
// of launch pairs of every instance.
int rows_instance(int kind, int prec, int n, int nx, int *K, int *M) {
    if (kind >= 2) {  // strips: any width
        *K = *M = 0;
        return 1;
    }
    return rows_shape(prec, n, kind == 0 ? RING_ROWS_TGV : RING_ROWS_CH, nx, K, M);
}
bool fused_multi_supported(int kind, int prec, int n, int K, int M) {
    if (prec == UQ_FP64) return false;
    if (kind >= 2) return n == 8;
    if (kind == 0 ? (n != 4 && n != 6 && n != 8) : (n < 2 || n > 4)) return false;
    return rows_fit(prec, n, kind == 0 ? RING_ROWS_TGV : RING_ROWS_CH, K, M);
}

hipError_t launch_fused_multi(int kind, int prec, int n, int K, int M, const FusedJob *jobs, int njobs,
                              int64_t nwork, int launch, hipStream_t s) {
    if (njobs <= 0 || nwork <= 0) return hipSuccess;
    if (!fused_multi_supported(kind, prec, n, K, M)) return hipErrorInvalidValue;
    bool ok = false;
    switch (prec) {
        case UQ_FP32: ok = fused_launch_multi<UQ_FP32>(kind, n, K, M, jobs, njobs, nwork, launch, s); break;
        case UQ_FP16S: ok = fused_launch_multi<UQ_FP16S>(kind, n, K, M, jobs, njobs, nwork, launch, s); break;
        default: ok = fused_launch_multi<UQ_BF16S>(kind, n, K, M, jobs, njobs, nwork, launch, s); break;
    }
    if (!ok) return hipErrorInvalidValue;
    return hipGetLastError();
}
// *d_t[q] += n for every job of a table (one thread per job)
__global__ void k_advance_ptrs(int64_t *const *d_t, int njobs, int64_t n) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < njobs) *d_t[q] += n;
}

hipError_t launch_advance_ptrs(int64_t *const *d_t, int njobs, int64_t n, hipStream_t s) {
    if (njobs <= 0) return hipSuccess;
    k_advance_ptrs<<<(unsigned)((njobs + 63) / 64), 64, 0, s>>>(d_t, njobs, n);
    return hipGetLastError();
}
hipError_t launch_fused(const JobDev &j, int n, bool src2, int fty, int window, bool nt, const int64_t *d_t, int k,
                        hipStream_t s) {
    if (j.geom == 1) {
        if (!channel_fusable(j) || (window != 2 && window != 3)) return hipErrorInvalidValue;
        if (window == 2 && (n < 2 || n > 4 || j.nx > channel_rows_max_nx(j.prec, n))) return hipErrorInvalidValue;
        if (window == 3 && (n < 3 || n > channel_strips_max_n(j.prec))) return hipErrorInvalidValue;
        switch (j.prec) {
            case UQ_FP64: fused_launch_channel<UQ_FP64>(j, n, d_t, k, src2, fty, window, s); break;
            case UQ_FP32: fused_launch_channel<UQ_FP32>(j, n, d_t, k, src2, fty, window, s); break;
            case UQ_FP16S: fused_launch_channel<UQ_FP16S>(j, n, d_t, k, src2, fty, window, s); break;
            default: fused_launch_channel<UQ_BF16S>(j, n, d_t, k, src2, fty, window, s); break;
        }
        return hipGetLastError();
    }
    if (!fused_supported(j) || n < 2 || n > (window == 4 ? TILE_MAX_STEPS : (window >= 2 ? 8 : 4)) ||
        (window == 3 && n < 3))
        return hipErrorInvalidValue;
    if (window == 4 && !tile_shape(j.nx, j.ny, n).RW) return hipErrorInvalidValue;
    if (window == 2 && j.nx > full_rows_max_nx(j.prec, n)) return hipErrorInvalidValue;
    switch (j.prec) {
        case UQ_FP64: fused_launch_tgv<UQ_FP64>(j, n, src2, fty, window, nt, s); break;
        case UQ_FP32: fused_launch_tgv<UQ_FP32>(j, n, src2, fty, window, nt, s); break;
        case UQ_FP16S: fused_launch_tgv<UQ_FP16S>(j, n, src2, fty, window, nt, s); break;
        default: fused_launch_tgv<UQ_BF16S>(j, n, src2, fty, window, nt, s); break;
    }
    return hipGetLastError();
}

void tile_counts(const JobDev &j, int cpt, int *tiles_x, int *tiles_y) {
    *tiles_x = (j.nx + BX - 1) / BX;
    *tiles_y = (j.ny + BY * cpt - 1) / (BY * cpt);
}

hipError_t launch_advance(int64_t *d_t, int64_t n, hipStream_t s) {
    k_advance<<<1, 64, 0, s>>>(d_t, n);
    return hipGetLastError();
}

hipError_t launch_select_scalar(const JobDev &j, const double *qoi, int which, double *M, hipStream_t s) {
    k_select<<<(unsigned)((j.S + 255) / 256), 256, 0, s>>>(qoi, j.smp, j.S, which, j.dia, j.u_fac, M);
    return hipGetLastError();
}

// Chunks per sample of k_qoi: about 8 workgroups per CU in all, 4 nodes or
// more per thread. Their sums go to part (QOI_PARTS values), or if that is null
// to the slab that does not hold the state (AB: the next step overwrites all of
// it that is ever read).
hipError_t launch_qoi_scalars(const JobDev &j, int64_t t, double *out, int64_t *flag, double *part, hipStream_t s) {
    const int64_t cells = (int64_t)j.nx * j.ny;
    const int64_t slab2 = j.plane * (j.prec == UQ_FP64 ? 72 : (j.prec == UQ_FP32 ? 36 : 18));  // bytes a sample
    int64_t chunks = 1;
    if (j.layout == UQ_LAYOUT_AB) {
        if (!part) part = (double *)((t & 1) ? j.f : j.f2);
        chunks = std::min<int64_t>(std::min<int64_t>(QOI_CHUNKS / j.S, (cells + 1023) / 1024), slab2 / (QOI_PART * 8));
        chunks = std::max<int64_t>(1, chunks);
    }
    const int per = (int)((cells + chunks - 1) / chunks);
    const unsigned gy = (unsigned)std::min<int64_t>(j.S, 32768);
    dim3 grid((unsigned)chunks, gy, (unsigned)((j.S + gy - 1) / gy));
    UQ_DISPATCH(k_qoi, t & 1, grid, 256, s, j, t, per, part, out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_qoi_join<<<1, 256, 0, s>>>(j.ke_norm, j.S, (int)chunks, part, out, flag);
    return hipGetLastError();
}

hipError_t launch_fields(const JobDev &j, int64_t t, double *out, hipStream_t s) {
    const int64_t cells = (int64_t)j.nx * j.ny;
    dim3 grid((unsigned)std::min<int64_t>((cells + 255) / 256, 4096), (unsigned)std::min<int64_t>(j.S, 65535));
    UQ_DISPATCH(k_fields, t & 1, grid, 256, s, j, t, out);
    return hipGetLastError();
}

hipError_t launch_field_moments(const JobDev &j, int64_t t, int qoi, const double *wphi, const double *a, int K,
                                double *coeffs, double *mean, double *var, double *var_alt, hipStream_t s) {
    const int which = qoi == UQ_QOI_VEL ? 0 : (qoi == UQ_QOI_RHO ? 1 : 2);
    const int64_t cells = (int64_t)j.nx * j.ny;
    if (K > 0) {
        const int npair = (which == 0 ? 2 : 1) * K;
        dim3 grid((unsigned)((cells + 63) / 64), (unsigned)((npair + 4 * FP_KA - 1) / (4 * FP_KA)));
        UQ_DISPATCH(k_field_coeffs, t & 1, grid, 256, s, j, t, which, wphi, K, coeffs);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // waves per 64 nodes: 8 samples or more each, and no more than give every
    // CU 32 waves (large lattices have enough nodes)
    const int64_t blocks = (cells + 63) / 64;
    const int64_t G = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(FF_MAX_G, (j.S + 7) / 8), (256 * 32 + blocks - 1) / blocks));
    UQ_DISPATCH(k_field_finish, t & 1, dim3((unsigned)blocks), 64 * (unsigned)G, s, j, t, which, a, K, coeffs, mean, var, var_alt);
    return hipGetLastError();
}

hipError_t launch_scalar_moments(const double *M, int64_t S, const double *wphi, const double *a, int K,
                                 double *coeffs, double *mean, double *var, double *var_alt, hipStream_t s) {
    if (K > 0) {
        k_scalar_coeffs<<<(unsigned)K, 256, 0, s>>>(M, S, wphi, K, coeffs);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    k_scalar_finish<<<1, 256, 0, s>>>(M, S, a, K, coeffs, mean, var, var_alt);
    return hipGetLastError();
}

hipError_t launch_export(const JobDev &j, int64_t t, int64_t sample, double *out, hipStream_t s) {
    const int64_t cells = (int64_t)j.nx * j.ny;
    dim3 grid((unsigned)std::min<int64_t>((cells + 255) / 256, 4096));
    UQ_DISPATCH(k_export, t & 1, grid, 256, s, j, t, sample, out);
    return hipGetLastError();
}

}  // namespace uqi
