// The temporally blocked step kernels (several LBM steps per launch), of one
// storage precision: compiled once per precision (UQ_PREC), so that the
// builds run side by side.
#include "fused_shapes.h"
#include "lbm_device.h"

// as in lbm_device.h: no implicit contraction in any kernel
#pragma clang fp contract(off)

namespace uqi {

// ------------------------------------------------------------------ fused steps
// Periodic lattices (no boundary rules), AB layout: N = 2..4 steps per launch
// (temporal blocking). A workgroup takes a tile of 64 x TY output nodes of
// one sample and keeps a ring of N - 1 nodes around it in LDS. Phase 1 pulls
// the state at t for tile and ring from the source slab and collides it
// (step t); each later phase pulls from LDS, collides the next step on a
// region one node narrower (held in registers across a barrier, then written
// back to LDS); the last phase covers the tile itself and stores f*(t+N-1)
// to the other slab. Each population crosses HBM once per N steps (the
// ring's re-reads are served by L2: neighbouring tiles run together). Same
// per-node arithmetic as k_step, including the storage rounding of every
// intermediate state.
constexpr int FUSE_TX = 64;
template <int P, int TY, int N>
__global__ __launch_bounds__(256) void k_stepN(JobDev j, bool src2, int tiles_x, int tiles_y, int64_t ntiles) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    constexpr int RG = N - 1;                 // ring width
    constexpr int LW = FUSE_TX + 2 * RG;      // LDS row length
    constexpr int LH = TY + 2 * RG;           // LDS rows
    constexpr int PER = (LW * LH + 255) / 256; // region nodes per thread (bound)
    __shared__ C lds[9][LH][LW];
    const T *src_all = (const T *)(src2 ? j.f2 : j.f);
    T *dst_all = (T *)(src2 ? j.f : j.f2);
    const int nx = j.nx, ny = j.ny;
    // offsets inside one sample fit in 32 bits (9 planes < 2^31 elements)
    const int pitch = (int)j.pitch, plane = (int)j.plane;
    const float inv = j.inv_scale, sc = j.scale;
    const int tid = threadIdx.x;
    const int64_t G = gridDim.x;
    const int64_t per_sample = (int64_t)tiles_x * tiles_y;
    for (int64_t tile = xcd_logical(blockIdx.x, G); tile < ntiles; tile += G) {
        const int64_t smp = tile / per_sample;
        const int64_t rem = tile - smp * per_sample;
        const int ty = (int)(rem / tiles_x), tx = (int)(rem - (int64_t)ty * tiles_x);
        const int x0 = tx * FUSE_TX, y0 = ty * TY;
        const int w = min(FUSE_TX, nx - x0), h = min(TY, ny - y0);
        const T *src = src_all + smp * 9 * (int64_t)plane;
        T *dst = dst_all + smp * 9 * (int64_t)plane;
        const C omega = (C)j.smp[smp].omega;
        const int plane_b = plane * (int)sizeof(T);
        const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(src, 9 * plane_b);
        // phase 1: step t on tile and ring, from the source slab. A thread's
        // elements e = tid + 256 k (their (r, c) advance by (256 / RW,
        // 256 % RW) per k) issue all their loads before any is used.
        {
            const int RW = w + 2 * RG, RH = h + 2 * RG, n_el = RW * RH;
            const int dq = 256 / RW, dr = 256 - dq * RW;
            int rr[PER], cc[PER];
            {
                int r = tid / RW, c = tid - r * RW;
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    rr[k] = r;
                    cc[k] = c;
                    r += dq;
                    c += dr;
                    if (c >= RW) {
                        c -= RW;
                        ++r;
                    }
                }
            }
            // B elements at a time issue their loads together: all of them in
            // FP64 (long load latency per byte, registers to spare), one at a
            // time in the 4- and 2-byte formats (more waves in flight instead)
            constexpr int B = P == UQ_FP64 ? PER : 1;
#pragma unroll
            for (int kb = 0; kb < PER; kb += B) {
                C f[B][9];
#pragma unroll
                for (int q2 = 0; q2 < B; ++q2) {
                    const int k = kb + q2;
                    if (k < PER && tid + 256 * k < n_el) {
                        int gx = x0 - RG + cc[k], gy = y0 - RG + rr[k];
                        if (gx < 0 || gx >= nx) gx = wrap_coord(gx, nx);
                        if (gy < 0 || gy >= ny) gy = wrap_coord(gy, ny);
                        // the pull sources: columns x-1, x, x+1 and rows y-1,
                        // y, y+1 (wrapped), one byte offset per direction
                        const int xm = gx == 0 ? nx - 1 : gx - 1, xp = gx == nx - 1 ? 0 : gx + 1;
                        const int ym = gy == 0 ? ny - 1 : gy - 1, yp = gy == ny - 1 ? 0 : gy + 1;
                        const int r0 = gy * pitch, rm = ym * pitch, rp = yp * pitch;
#pragma unroll
                        for (int i = 0; i < 9; ++i) {
                            const int col = CXd[i] > 0 ? xm : (CXd[i] < 0 ? xp : gx);
                            const int row = CYd[i] > 0 ? rm : (CYd[i] < 0 ? rp : r0);
                            f[q2][i] = BufLd<P>::ld(rsrc, (row + col) * (int)sizeof(T), i * plane_b, inv);
                        }
                    }
                }
#pragma unroll
                for (int q2 = 0; q2 < B; ++q2) {
                    const int k = kb + q2;
                    if (k < PER && tid + 256 * k < n_el) {
                        C drho, ux, uy;
                        bgk(f[q2], omega, drho, ux, uy);
#pragma unroll
                        for (int i = 0; i < 9; ++i) lds[i][rr[k]][cc[k]] = PR::rt(f[q2][i], sc, inv);
                    }
                }
            }
        }
        __syncthreads();
        // middle phases: steps t+1 .. t+N-2 on shrinking regions, in LDS;
        // each thread keeps its new values in registers across the barrier
        auto middle = [&](auto ph_c) {
            constexpr int PH = decltype(ph_c)::value;
            constexpr int PERM = ((LW - 2 * PH) * (LH - 2 * PH) + 255) / 256;
            const int RW = w + 2 * (RG - PH), RH = h + 2 * (RG - PH), n_el = RW * RH;
            const int dq = 256 / RW, dr = 256 - dq * RW;
            C g[PERM][9];
            int rr[PERM], cc[PERM];
            {
                int r = tid / RW, c = tid - r * RW;
#pragma unroll
                for (int k = 0; k < PERM; ++k) {
                    rr[k] = r + PH;
                    cc[k] = c + PH;
                    r += dq;
                    c += dr;
                    if (c >= RW) {
                        c -= RW;
                        ++r;
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < PERM; ++k) {
                if (tid + 256 * k < n_el) {
#pragma unroll
                    for (int i = 0; i < 9; ++i) g[k][i] = lds[i][rr[k] - CYd[i]][cc[k] - CXd[i]];
                    C drho, ux, uy;
                    bgk(g[k], omega, drho, ux, uy);
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PERM; ++k) {
                if (tid + 256 * k < n_el) {
#pragma unroll
                    for (int i = 0; i < 9; ++i) lds[i][rr[k]][cc[k]] = PR::rt(g[k][i], sc, inv);
                }
            }
            __syncthreads();
        };
        if constexpr (N >= 3) middle(std::integral_constant<int, 1>());
        if constexpr (N >= 4) middle(std::integral_constant<int, 2>());
        // last phase: step t+N-1 on the tile, to the destination slab
        const int cx = tid & 63;
        for (int r = tid >> 6; r < h; r += 4) {
            if (cx < w) {
                C f[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) f[i] = lds[i][r + RG - CYd[i]][cx + RG - CXd[i]];
                C drho, ux, uy;
                bgk(f, omega, drho, ux, uy);
                const int own = (y0 + r) * pitch + x0 + cx;
#pragma unroll
                for (int i = 0; i < 9; ++i) PR::st_nt(dst + (i * plane + own), f[i], sc);
            }
        }
        __syncthreads();  // LDS is reused by the next tile
    }
}

// ------------------------------------------------------------------ fused steps, sliding window
// The same N-step fusion organised as a pipeline down a strip of W columns
// of one sample (W <= 64 - 2(N-1)): each wave of the workgroup computes one
// time level, one lattice row per iteration, two rows behind the level it
// reads. Level 1 pulls from the source slab (D rows ahead, in registers);
// levels 2..N pull from LDS rows of the level below; level N stores to the
// other slab. Only the strip's x-ring (N-1 columns per side) and a chunk's
// y-halo are computed twice (11 % at N = 4 with 52-column strips and 64-row
// chunks, against 45 % for the 8-row tiles above), and every address that
// depends on the row is wave-uniform (scalar registers): a lane keeps one
// column for the whole strip.
// Between two levels each direction is read once, by the row that pulls it:
// c_y = -1 directions one iteration after they are written (rows kept: 2),
// c_y = 0 two iterations after (3), c_y = +1 three after (4). Rows are
// offset by 12 (a multiple of 2, 3 and 4) to keep slots positive.
template <int P, int N>
struct WindowRings {
    static constexpr int NR = N > 1 ? N - 1 : 1;
    using C = typename Prec<P>::C;
    C ra[NR][2][3][64], rb[NR][3][3][64], rc[NR][4][3][64];
};

// One work item of the strip window: strip `strip` (columns [strip W,
// strip W + W)) of rows [chunk H, chunk H + H) of sample smp, N steps, from
// the slab src2 names to the other one; the wave's level is lvl. Ends with
// a barrier, so the rings may be reused by the next item at once.
template <int P, int N, int D>
__device__ __forceinline__ void stepW_item(const JobDev &j, bool src2, int W, int H, int64_t smp, int chunk,
                                           int strip, bool nt, int lvl, WindowRings<P, N> &rings) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    constexpr int RG = N - 1;
    auto &ra = rings.ra;
    auto &rb = rings.rb;
    auto &rc = rings.rc;
    const T *src_all = (const T *)(src2 ? j.f2 : j.f);
    T *dst_all = (T *)(src2 ? j.f : j.f2);
    const int nx = j.nx, ny = j.ny;
    const int pitch = (int)j.pitch, plane = (int)j.plane;
    const int plane_b = plane * (int)sizeof(T), pitch_b = pitch * (int)sizeof(T);
    const float inv = j.inv_scale, sc = j.scale;
    const int lane = threadIdx.x & 63;
    {
        const int x0 = strip * W, w = min(W, nx - x0);
        const int yb = chunk * H, ye = min(ny, yb + H);
        const T *src = src_all + smp * 9 * (int64_t)plane;
        T *dst = dst_all + smp * 9 * (int64_t)plane;
        const C omega = (C)j.smp[smp].omega;
        const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(src, 9 * plane_b), wrsrc = make_rsrc(dst, 9 * plane_b);
        const int wvo = (x0 + lane) * (int)sizeof(T);  // level N's store column
        // this lane's column at this level, and its LDS column (0 = x0 - RG)
        const int span = RG - (lvl - 1);  // columns beyond the strip on each side
        const bool lane_on = lane < w + 2 * span;
        const int lc = lane + (lvl - 1);
        int gc = x0 - span + lane;
        while (gc < 0) gc += nx;
        while (gc >= nx) gc -= nx;
        const int vo0 = gc * (int)sizeof(T), vom = (gc == 0 ? nx - 1 : gc - 1) * (int)sizeof(T),
                  vop = (gc == nx - 1 ? 0 : gc + 1) * (int)sizeof(T);
        // level 1 pulls row y + D while it collides row y: D rows of loads in
        // flight per strip. D + 1 register buffers in rotation: each step
        // collides one in place and refills the one the step before used, so
        // a load never targets a live register (that would leave a copy that
        // waits for the load).
        constexpr int B = D + 1;
        using R = typename BufLd<P>::R;
        R buf[B][9];
        auto pull = [&](R *f, int y) {
            int gy = y;
            while (gy < 0) gy += ny;
            while (gy >= ny) gy -= ny;
            const int r0 = gy * pitch_b, rm = (gy == 0 ? ny - 1 : gy - 1) * pitch_b,
                      rp = (gy == ny - 1 ? 0 : gy + 1) * pitch_b;
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int vo = CXd[i] > 0 ? vom : (CXd[i] < 0 ? vop : vo0);
                const int ro = CYd[i] > 0 ? rm : (CYd[i] < 0 ? rp : r0);
                f[i] = BufLd<P>::raw(rsrc, vo, i * plane_b + ro);
            }
        };
        const int y1_end = ye + RG;  // level 1 rows: [yb - RG, ye + RG)
        // collide a pulled row and hand it to the next level (or store it)
        auto finish = [&](C *f, int y) {
            C drho, ux, uy;
            bgk(f, omega, drho, ux, uy);
            if (lvl < N) {
                const int sa = (y + 12) & 1, sb = (y + 12) % 3, sc3 = (y + 12) & 3, L = lvl - 1;
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const C v = PR::rt(f[i], sc, inv);
                    const int g = GJd[i];
                    if (CYd[i] < 0) ra[L][sa][g][lc] = v;
                    else if (CYd[i] == 0) rb[L][sb][g][lc] = v;
                    else rc[L][sc3][g][lc] = v;
                }
            } else if (nt) {
                const int own = y * pitch + x0 + lane;
#pragma unroll
                for (int i = 0; i < 9; ++i) PR::st_nt(dst + (i * plane + own), f[i], sc);
            } else {
#pragma unroll
                for (int i = 0; i < 9; ++i) BufSt<P>::st(wrsrc, f[i], wvo, i * plane_b + y * pitch_b, sc);
            }
        };
        // Level 1's loads are issued by every lane of the wave and for every
        // row (rows past the chunk's end reload its last row), so that no
        // register holds a mix of new and old values.
        if (lvl == 1) {
#pragma unroll
            for (int k = 0; k < D; ++k) pull(buf[k], min(yb - RG + k, y1_end - 1));
        }
        const int n_it = (ye - yb) + 3 * RG;
        for (int it0 = 0; it0 < n_it; it0 += B) {
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const int it = it0 + k;
                if (it >= n_it) break;
                const int y = yb - RG + it - 2 * (lvl - 1);  // this level's row (wave-uniform)
                const bool row_on = y >= yb - span && y < ye + span;
                if (lvl == 1) {
                    if (row_on) {
                        pull(buf[(k + D) % B], min(y + D, y1_end - 1));
                        if (lane_on) {
                            C f[9];  // (buffers are written only by loads)
#pragma unroll
                            for (int i = 0; i < 9; ++i) f[i] = BufLd<P>::cvt(buf[k][i], inv);
                            finish(f, y);
                        }
                    }
                } else if (row_on && lane_on) {
                    C f[9];
                    const int L = lvl - 2;
                    const int sa = (y + 13) & 1, sb = (y + 12) % 3, sc3 = (y + 11) & 3;
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        const int g = GJd[i], c = lc - CXd[i];
                        f[i] = CYd[i] < 0 ? ra[L][sa][g][c] : (CYd[i] == 0 ? rb[L][sb][g][c] : rc[L][sc3][g][c]);
                    }
                    finish(f, y);
                }
                __syncthreads();
            }
        }
    }
}

// level of a wave of the strip window, rotated with the workgroup index so
// that the levels' different instruction mixes spread evenly over a CU's
// SIMDs
template <int N>
__device__ inline int window_level() {
    return __builtin_amdgcn_readfirstlane((int)((threadIdx.x >> 6) + blockIdx.x) % N) + 1;  // 1..N
}

template <int P, int N, int D>
__global__ __launch_bounds__(64 * N) void k_stepW(JobDev j, bool src2, int W, int strips, int H, int chunks,
                                                  int64_t nwork, bool nt) {
    __shared__ WindowRings<P, N> rings;
    const int lvl = window_level<N>();
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const int64_t smp = wk / ((int64_t)chunks * strips);
        const int rem = (int)(wk - smp * chunks * strips);
        const int chunk = rem / strips;
        stepW_item<P, N, D>(j, src2, W, H, smp, chunk, rem - chunk * strips, nt, lvl, rings);
    }
}

// ------------------------------------------------------------------ fused steps, full rows
// The sliding window over whole rows: K waves per time level, M columns per
// lane, cover the nx <= 64 K M columns of a row, so on a periodic lattice no
// column is computed twice (only a chunk's row halo is). Each LDS row holds
// one direction of the nx columns at 0..nx-1, already shifted by the
// direction's c_x (periodic wrap included), so that every pull from the row
// below reads the lane's own column. N K waves in one workgroup, one barrier
// per row.
// LDS rings of the level below, by the row a direction group pulls from:
// c_y = -1 (row y + 1, slots 0-1) and c_y = 0 (row y, slots 2-3): 2 rows;
// c_y = +1 (row y - 1, slots 4-6): 3 rows. A row sits in slot s mod 2 or
// s mod 3 of its group, s the row step it is written in. A row holds 64 K M
// values (no padding:
// the shifted writes wrap inside the row), so the three rows of a slot, and
// the same slot of the first two groups, lie a multiple of 64 words apart:
// the compiler pairs those accesses into ds_read2st64 / ds_write2st64.
template <int P, int N, int K, int M>
struct RowsRing {
    static constexpr int NR = N > 1 ? N - 1 : 1;
    static constexpr int CW = 64 * K * M;
    using Array = typename Prec<P>::C[NR][7][3][CW];
};

// One work item of the full-row pipeline: rows [chunk H, chunk H + H) of
// sample smp (with the halo rows the levels need), N steps, from the slab
// src2 names to the other one. Every wave of the workgroup passes the same
// number of barriers, the last one after the item's final row step, so the
// rings may be reused by the next item at once.
// STRIP: the item is a strip of W columns [x0, x0 + W) of those rows instead
// of whole rows. The 64 K M lanes take the columns x0 - (N - 1) .. (periodic,
// so W <= 64 K M - 2 (N - 1)); what a pull brings in from beyond the outermost
// lane is wrong, and the wrong columns move one further in per level, so the
// W in the middle are right at level N, which stores only those.
template <int P, int N, int K, int M, int D, bool STRIP = false>
__device__ __forceinline__ void stepR_item(const JobDev &j, bool src2, int H, int64_t smp, int chunk, bool nt,
                                           typename RowsRing<P, N, K, M>::Array &rg, int x0 = 0, int W = 0) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    constexpr int RG = N - 1;
    const T *src_all = (const T *)(src2 ? j.f2 : j.f);
    T *dst_all = (T *)(src2 ? j.f : j.f2);
    const int nx = j.nx, ny = j.ny;
    const int plane = (int)j.plane;
    const int plane_b = plane * (int)sizeof(T), pitch_b = (int)j.pitch * (int)sizeof(T);
    const float inv = j.inv_scale, sc = j.scale;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lvl = wave / K + 1;  // 1..N
    // Lanes past the lattice take the last column: they read what its own
    // lane reads, compute the same values and write them to the same places
    // (the same bits), so no lane needs a guard and the compiler keeps the
    // collisions and the LDS reads that feed them unconditional.
    int c[M], gx[M], vo0[M], vom[M], vop[M], wp[M], wm[M];
    bool st[M];  // the column is stored
#pragma unroll
    for (int m = 0; m < M; ++m) {
        c[m] = ((wave - (lvl - 1) * K) * M + m) * 64 + lane;
        if constexpr (STRIP) {
            gx[m] = wrap_coord(x0 - RG + c[m], nx);
            st[m] = c[m] >= RG && c[m] < RG + W;
        } else {
            gx[m] = c[m] = min(c[m], nx - 1);
            st[m] = true;
        }
        const int cw = STRIP ? 64 * K * M : nx;  // LDS columns
        vo0[m] = gx[m] * (int)sizeof(T);
        vom[m] = (gx[m] == 0 ? nx - 1 : gx[m] - 1) * (int)sizeof(T);
        vop[m] = (gx[m] == nx - 1 ? 0 : gx[m] + 1) * (int)sizeof(T);
        wp[m] = c[m] == cw - 1 ? 0 : c[m] + 1;  // LDS columns of the c_x = +1 and -1 pushes
        wm[m] = c[m] == 0 ? cw - 1 : c[m] - 1;
    }
    // LDS byte offsets of the lane's columns: x, wm, wp in the ring this
    // level writes (ring lvl - 1), x in the ring it reads (ring lvl - 2).
    // Every ring access is one of these plus a constant (slot and
    // direction-row), which the DS instructions take as their immediate
    // offset; the offsets pass through an empty asm once per turn of the row
    // loops so that the compiler keeps them as the bases instead of hoisting
    // one address register per access out of the loop.
    constexpr int GB = RowsRing<P, N, K, M>::CW * (int)sizeof(C), SB = 3 * GB, RB = 7 * SB;
    char *const ring = reinterpret_cast<char *>(&rg);
    int ox[M], om[M], op[M], orx[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        ox[m] = (lvl - 1) * RB + c[m] * (int)sizeof(C);
        om[m] = (lvl - 1) * RB + wm[m] * (int)sizeof(C);
        op[m] = (lvl - 1) * RB + wp[m] * (int)sizeof(C);
        orx[m] = (lvl - 2) * RB + c[m] * (int)sizeof(C);
    }
    auto at = [&](int base, int slot, int g) -> C & { return *reinterpret_cast<C *>(ring + base + slot * SB + g * GB); };
    auto fresh = [&]() {
#pragma unroll
        for (int m = 0; m < M; ++m) asm("" : "+v"(ox[m]), "+v"(om[m]), "+v"(op[m]), "+v"(orx[m]));
    };
    const int span = RG - (lvl - 1);  // rows beyond the chunk on each side
    constexpr int B = D + 1;
    using R = typename BufLd<P>::R;
    R buf[B][M][9];
    {
        const int yb = chunk * H, ye = min(ny, yb + H);
        const T *src = src_all + smp * 9 * (int64_t)plane;
        T *dst = dst_all + smp * 9 * (int64_t)plane;
        const C omega = (C)j.smp[smp].omega;
        const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(src, 9 * plane_b), wrsrc = make_rsrc(dst, 9 * plane_b);
        auto pull = [&](R (*f)[9], int y) {
            int gy = y;
            while (gy < 0) gy += ny;
            while (gy >= ny) gy -= ny;
            const int r0 = gy * pitch_b, rm = (gy == 0 ? ny - 1 : gy - 1) * pitch_b,
                      rp = (gy == ny - 1 ? 0 : gy + 1) * pitch_b;
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const int vo = CXd[i] > 0 ? vom[m] : (CXd[i] < 0 ? vop[m] : vo0[m]);
                    const int ro = CYd[i] > 0 ? rm : (CYd[i] < 0 ? rp : r0);
                    f[m][i] = BufLd<P>::raw(rsrc, vo, i * plane_b + ro);
                }
        };
        // a level hands direction i of its column c on to LDS column
        // (c + c_ix) mod nx, where the level above pulls it: every pull
        // then reads the puller's own column, and the periodic wrap costs no
        // extra copies
        // (the c_y = -1 and c_y = 0 groups use slots of the same index, two
        // apart: their writes of equal c_x go in pairs, ds_write2st64).
        // Slots are named by the row step a row is written in, the same
        // count for every level: a row written in step it goes to slot
        // it mod 2 of the first two groups and it mod 3 of the c_y = +1
        // group, and is read in step it + 1 (c_y <= 0 groups) or it + 2
        // (c_y = +1). The row loops advance six steps at a time, so for
        // the unrolled step u (it = 6 n + u) every slot is a constant and
        // each LDS address is the lane's column base plus an immediate.
        auto put = [&](int u, int m, const C *v) {
            const int sa = u & 1, sc3 = u % 3;
            at(ox[m], sa, 0) = v[4];
            at(ox[m], 2 + sa, 0) = v[0];
            at(om[m], sa, 1) = v[7];
            at(om[m], 2 + sa, 2) = v[3];
            at(op[m], sa, 2) = v[8];
            at(op[m], 2 + sa, 1) = v[1];
            at(ox[m], 4 + sc3, 0) = v[2];
            at(op[m], 4 + sc3, 1) = v[5];
            at(om[m], 4 + sc3, 2) = v[6];
        };
        // collide the lane's M nodes of row y and hand each on to the next
        // level
        auto finish = [&](C (*f)[9], int y, int u) {
#pragma unroll
            for (int m = 0; m < M; ++m) {
                C drho, ux, uy;
                bgk(f[m], omega, drho, ux, uy);
            }
            // one uniform branch for all the lane's columns, so that both
            // collisions stay in one block
            if (lvl < N) {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    C v[9];
#pragma unroll
                    for (int i = 0; i < 9; ++i) v[i] = PR::rt(f[m][i], sc, inv);
                    put(u, m, v);
                }
            } else if (nt) {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    if (STRIP && !st[m]) continue;
                    const int own = y * (int)j.pitch + gx[m];
#pragma unroll
                    for (int i = 0; i < 9; ++i) PR::st_nt(dst + (i * plane + own), f[m][i], sc);
                }
            } else {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    if (STRIP && !st[m]) continue;
#pragma unroll
                    for (int i = 0; i < 9; ++i)
                        BufSt<P>::st(wrsrc, f[m][i], vo0[m], i * plane_b + y * pitch_b, sc);
                }
            }
        };
        const int y1_end = ye + RG;  // level 1 rows: [yb - RG, ye + RG)
        const int n_it = (ye - yb) + 3 * RG;
        // Both loops below pass n_it barriers, one per row step, six steps
        // per turn (the slot period; also a multiple of the B load buffers).
        static_assert(6 % B == 0, "the row loops turn over six steps");
        if (lvl == 1) {
#pragma unroll
            for (int k = 0; k < D; ++k) pull(buf[k], min(yb - RG + k, y1_end - 1));
            for (int it0 = 0; it0 < n_it; it0 += 6) {
#pragma unroll
                for (int u = 0; u < 6; ++u) {
                    const int it = it0 + u;
                    if (it >= n_it) break;
                    const int y = yb - RG + it;
                    if (u == 0) fresh();
                    if (y < ye + span) {
                        pull(buf[(u + D) % B], min(y + D, y1_end - 1));
                        C f[M][9];
#pragma unroll
                        for (int m = 0; m < M; ++m)
#pragma unroll
                            for (int i = 0; i < 9; ++i) f[m][i] = BufLd<P>::cvt(buf[u % B][m][i], inv);
                        finish(f, y, u);
                    }
                    __syncthreads();
                }
            }
        } else {
            // Levels above the first read the level below from the LDS rows.
            // The c_y = 0 and c_y = +1 pulls of the next row (rows y + 1 and
            // y of the level below) are complete before this row step begins
            // and their slots are not rewritten in it, so they are read one
            // step ahead into registers (two sets, alternating; for the first
            // row in the step before it), and only the c_y = -1 pulls (row
            // y + 1, written in the previous step) wait at the start of the
            // step. What is read ahead never sits in LDS for more than one
            // step, hence the short rings.
            C pre[2][M][6];
            // step u reads the rows the level below wrote in steps u - 1
            // (slot (u + 1) mod 2) and u - 2 (slot (u + 1) mod 3)
            auto ahead = [&](C (*q)[6], int u) {  // c_y >= 0 pulls of the next row
                const int sb = (u + 1) & 1, sc3 = (u + 1) % 3;
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    int n = 0;
#pragma unroll
                    for (int i = 0; i < 9; ++i) {
                        if (CYd[i] < 0) continue;
                        q[m][n++] = at(orx[m], CYd[i] == 0 ? 2 + sb : 4 + sc3, GJd[i]);
                    }
                }
            };
            const int y_lo = yb - span, y_hi = ye + span;  // this level's rows
            for (int it0 = 0; it0 < n_it; it0 += 6) {
#pragma unroll
                for (int u = 0; u < 6; ++u) {
                    const int it = it0 + u, k = u & 1;
                    if (it >= n_it) break;
                    const int y = yb - RG + it - 2 * (lvl - 1);  // this level's row (wave-uniform)
                    if (u == 0) fresh();
                    if (y == y_lo - 1) {
                        ahead(pre[k ^ 1], u);  // the first row's
                    } else if (y >= y_lo && y < y_hi) {
                        // row y + 1 of the level below: this row's c_y = -1
                        // pulls and the next row's c_y = 0 pulls (slots of the
                        // same index, two apart); row y: the next row's c_y = +1
                        // pulls. All at the lane's own column, 64-word multiples
                        // apart (ds_read2st64 pairs). Past the last row the
                        // values read ahead are not used.
                        const int sa = (u + 1) & 1, sc3 = (u + 1) % 3;
                        C f[M][9];
                        C (*q)[6] = pre[k ^ 1];
#pragma unroll
                        for (int m = 0; m < M; ++m) {
                            // at the lane's own LDS column
                            f[m][4] = at(orx[m], sa, 0);       // (0, -1)
                            f[m][7] = at(orx[m], sa, 1);       // (-1, -1)
                            f[m][8] = at(orx[m], sa, 2);       // (1, -1)
                            q[m][0] = at(orx[m], 2 + sa, 0);   // (0, 0)
                            q[m][1] = at(orx[m], 2 + sa, 1);   // (1, 0)
                            q[m][3] = at(orx[m], 2 + sa, 2);   // (-1, 0)
                            q[m][2] = at(orx[m], 4 + sc3, 0);  // (0, 1)
                            q[m][4] = at(orx[m], 4 + sc3, 1);  // (1, 1)
                            q[m][5] = at(orx[m], 4 + sc3, 2);  // (-1, 1)
                            // this row's c_y >= 0 pulls, read a step ago
                            f[m][0] = pre[k][m][0];
                            f[m][1] = pre[k][m][1];
                            f[m][2] = pre[k][m][2];
                            f[m][3] = pre[k][m][3];
                            f[m][5] = pre[k][m][4];
                            f[m][6] = pre[k][m][5];
                        }
                        // every LDS read of the step (both columns, and the
                        // next row's read-ahead) is issued before the first
                        // collision, which then waits only for its own three
                        __builtin_amdgcn_sched_barrier(0);
                        finish(f, y, u);
                    }
                    __syncthreads();
                }
            }
        }
    }
}

template <int P, int N, int K, int M, int D>
__global__ __launch_bounds__(64 * N * K) void k_stepR(JobDev j, bool src2, int H, int chunks, int64_t nwork,
                                                      bool nt) {
    __shared__ typename RowsRing<P, N, K, M>::Array rg;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const int64_t smp = wk / chunks;
        stepR_item<P, N, K, M, D>(j, src2, H, smp, (int)(wk - smp * chunks), nt, rg);
    }
}

// The same pipeline down strips of any periodic lattice, wider than the LDS
// rows of a whole-row instance hold: K waves per level of M columns per lane
// (RowStrips in fused_shapes.h). strip runs fastest, so that neighbouring
// strips, which share their halo columns' cache lines, run together.
template <int P, int N, int D>
__global__ __launch_bounds__(64 * N * RowStrips<P>::K, RowStrips<P>::WAVES) void k_stepRS(JobDev j, bool src2, int W,
                                                                                    int strips, int H, int chunks,
                                                                                    int64_t nwork) {
    constexpr int K = RowStrips<P>::K, M = RowStrips<P>::M;
    __shared__ typename RowsRing<P, N, K, M>::Array rg;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const int64_t smp = wk / ((int64_t)chunks * strips);
        const int rem = (int)(wk - smp * chunks * strips);
        const int chunk = rem / strips;
        const int x0 = min((rem - chunk * strips) * W, j.nx - W);
        stepR_item<P, N, K, M, D, true>(j, src2, H, smp, chunk, false, rg, x0, W);
    }
}

// Batched form: every chunk of every sample of every job in the table, N
// steps per launch; launch number `launch` of a tick reads the slab of
// parity par ^ (launch & 1) of its job (the state of step t + launch N;
// even N go in pairs, as in the single-job schedule).
template <int P, int N, int K, int M, int D>
__global__ __launch_bounds__(64 * N * K) void k_stepR_multi(const FusedJob *jobs, int njobs, int64_t nwork,
                                                            int launch, bool nt) {
    __shared__ typename RowsRing<P, N, K, M>::Array rg;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const FusedJob q = fused_entry(jobs, njobs, wk);
        const JobDev j = q.j;
        const int64_t local = wk - q.work0;
        const int64_t smp = local / q.chunks;
        stepR_item<P, N, K, M, D>(j, ((q.par ^ launch) & 1) != 0, q.H, smp, (int)(local - smp * q.chunks), nt, rg);
    }
}

// Batched strips of rows (see k_stepR_multi): every strip of every row chunk
// of every sample of every job in the table, N steps per launch.
template <int P, int N, int D>
__global__ __launch_bounds__(64 * N * RowStrips<P>::K, RowStrips<P>::WAVES) void k_stepRS_multi(const FusedJob *jobs,
                                                                                          int njobs, int64_t nwork,
                                                                                          int launch) {
    constexpr int K = RowStrips<P>::K, M = RowStrips<P>::M;
    __shared__ typename RowsRing<P, N, K, M>::Array rg;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const FusedJob q = fused_entry(jobs, njobs, wk);
        const JobDev j = q.j;
        const int64_t local = wk - q.work0;
        const int64_t smp = local / ((int64_t)q.chunks * q.strips);
        const int rem = (int)(local - smp * q.chunks * q.strips);
        const int chunk = rem / q.strips;
        const int x0 = min((rem - chunk * q.strips) * q.W, j.nx - q.W);
        stepR_item<P, N, K, M, D, true>(j, ((q.par ^ launch) & 1) != 0, q.H, smp, chunk, false, rg, x0, q.W);
    }
}

// ------------------------------------------------------------------ fused channel steps, full rows
// The full-row pipeline on the channel with half-way bounce-back walls and
// cylinder and Zou-He inlet / outlet (no interpolated rules): the same wall
// and open-column rules as the single-step gather, applied at every level.
// A bounce-back pull takes the node's own opposite population of the level
// below, so the LDS also keeps the row being computed: 3 rows of the
// c_y = -1 directions (their opposites), 3 of c_y = 0, 4 of c_y = +1. Rows
// outside the channel are not computed (their pulls are bounce-backs);
// along x the end columns are open, walls or periodic, as the node masks
// say. Solid nodes are skipped.
// Level L of a launch computes step t0 + L - 1 (the inflow ramp).
// one LDS array for the three rings (c_y = -1: slots 0-2, c_y = 0: 3-5,
// c_y = +1: 6-9), rows padded to a multiple of 64 values: the rows of a
// slot, and the slots of equal index of the first two groups, lie 64-word
// multiples apart, and the compiler pairs those accesses (ds_read2st64 /
// ds_write2st64)
template <int P, int N, int K, int M>
struct RowsRingCh {
    static constexpr int NR = N > 1 ? N - 1 : 1;
    static constexpr int CW = 64 * K * M + 64;
    using Array = typename Prec<P>::C[NR][10][3][CW];
};

// One work item of the channel pipeline: rows [chunk H, chunk H + H) of
// sample smp, steps t0 .. t0 + N - 1 (t0 = *d_t + k0), from the slab src2
// names to the other one; ends with a barrier, like stepR_item.
template <int P, int N, int K, int M, int D>
__device__ __forceinline__ void stepRC_item(const JobDev &j, const int64_t *d_t, int k0, bool src2, int H,
                                            int64_t smp, int chunk, typename RowsRingCh<P, N, K, M>::Array &rq) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    constexpr int RG = N - 1;
    constexpr uint32_t BB_BITS = 0x1FFu << M_BB, OPEN_BITS = 0x1FFu << M_OPEN;
    const int64_t t0 = *d_t + k0;
    const T *src_all = (const T *)(src2 ? j.f2 : j.f);
    T *dst_all = (T *)(src2 ? j.f : j.f2);
    const int nx = j.nx, ny = j.ny;
    const int plane = (int)j.plane;
    const int plane_b = plane * (int)sizeof(T), pitch_b = (int)j.pitch * (int)sizeof(T);
    const float inv = j.inv_scale, sc = j.scale;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lvl = wave / K + 1;  // 1..N
    const int64_t t_lvl = t0 + (lvl - 1);
    // the level's K column blocks rotate with the level, so that the blocks
    // with the open end columns (and the cylinder) fall on different SIMDs
    // at different levels (wave w runs on SIMD w mod 4)
    const int kb = (wave - (lvl - 1) * K + (lvl - 1)) % K;
    int c[M], vo0[M], vom[M], vop[M], mvo[M];
    bool on[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        c[m] = (kb * M + m) * 64 + lane;
        on[m] = c[m] < nx;
        const int cc = on[m] ? c[m] : nx - 1;
        mvo[m] = cc * 4;
        vo0[m] = cc * (int)sizeof(T);
        vom[m] = (cc == 0 ? nx - 1 : cc - 1) * (int)sizeof(T);
        vop[m] = (cc == nx - 1 ? 0 : cc + 1) * (int)sizeof(T);
    }
    const __amdgpu_buffer_rsrc_t mrsrc = make_rsrc(j.mask, ny * (int)j.pitch * 4);
    const int span = RG - (lvl - 1);
    constexpr int B = D + 1;
    using R = typename BufLd<P>::R;
    R buf[B][M][9];
    uint32_t mb[B][M];
    {
        const int yb = chunk * H, ye = min(ny, yb + H);
        const int lo = max(0, yb - span), hi = min(ny, ye + span);  // this level's rows
        const T *src = src_all + smp * 9 * (int64_t)plane;
        T *dst = dst_all + smp * 9 * (int64_t)plane;
        const C omega = (C)j.smp[smp].omega;
        // s(t) 4 u_peak of this level's step (uniform)
        const double a_in = ramp_factor(t_lvl, j.ramp) * 4.0 * j.smp[smp].u_peak;
        const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(src, 9 * plane_b), wrsrc = make_rsrc(dst, 9 * plane_b);
        auto clampy = [&](int y) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };
        auto pull = [&](R (*f)[9], int y) {
            const int gy = clampy(y);
            const int r0 = gy * pitch_b, rm = (gy == 0 ? ny - 1 : gy - 1) * pitch_b,
                      rp = (gy == ny - 1 ? 0 : gy + 1) * pitch_b;
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    const int vo = CXd[i] > 0 ? vom[m] : (CXd[i] < 0 ? vop[m] : vo0[m]);
                    const int ro = CYd[i] > 0 ? rm : (CYd[i] < 0 ? rp : r0);
                    f[m][i] = BufLd<P>::raw(rsrc, vo, i * plane_b + ro);
                }
        };
        auto pullm = [&](uint32_t *mm, int y) {
            const int mo = clampy(y) * (int)j.pitch * 4;
#pragma unroll
            for (int m = 0; m < M; ++m) mm[m] = __builtin_amdgcn_raw_buffer_load_b32(mrsrc, mvo[m], mo, 0);
        };
        auto put = [&](int L, int y, int col, const C *v) {  // by direction-row, c_y = -1 and 0 in pairs
            const int s3 = (y + 12) % 3, s4 = (y + 12) & 3;
            rq[L][s3][0][col] = v[4];
            rq[L][3 + s3][0][col] = v[0];
            rq[L][s3][1][col] = v[7];
            rq[L][3 + s3][1][col] = v[1];
            rq[L][s3][2][col] = v[8];
            rq[L][3 + s3][2][col] = v[3];
            rq[L][6 + s4][0][col] = v[2];
            rq[L][6 + s4][1][col] = v[5];
            rq[L][6 + s4][2][col] = v[6];
        };
        // the open-column rule, then collide, then hand on or store
        auto finish = [&](C (*f)[9], const uint32_t *mm, int y) {
#pragma unroll
            for (int m = 0; m < M; ++m) {
                if (mm[m] & OPEN_BITS) {
                    // Zou-He overwrites every pull from beyond the column
                    // (inlet 1, 5, 8; outlet 3, 6, 7) without reading it, so
                    // where it runs (t > 0) and the inlet is not also the
                    // outlet (nx > 1) those pulls need not be zeroed first:
                    // the same values as the single-step gather, which
                    // zeroes them at every step (both conditions uniform)
                    if (t_lvl == 0 || nx == 1) {
#pragma unroll
                        for (int i = 0; i < 9; ++i) f[m][i] = ((mm[m] >> (M_OPEN + i)) & 1u) ? C(0) : f[m][i];
                    }
                    if (t_lvl > 0)
                        zou_he_u(f[m], c[m] == 0, c[m] == 0 ? (C)inflow_u_a(a_in, ny, y) : C(0));
                }
            }
#pragma unroll
            for (int m = 0; m < M; ++m) {
                C drho, ux, uy;
                bgk(f[m], omega, drho, ux, uy);
            }
            // one uniform branch for all the lane's columns (see stepR_item)
            if (lvl < N) {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    if (!on[m] || (mm[m] & M_SOLID)) continue;
                    C v[9];
#pragma unroll
                    for (int i = 0; i < 9; ++i) v[i] = PR::rt(f[m][i], sc, inv);
                    put(lvl - 1, y, c[m] + 1, v);
                    // end-column copies (read only when x is periodic)
                    if (c[m] == nx - 1) put(lvl - 1, y, 0, v);
                    if (c[m] == 0) put(lvl - 1, y, nx + 1, v);
                }
            } else {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    if (!on[m] || (mm[m] & M_SOLID)) continue;
#pragma unroll
                    for (int i = 0; i < 9; ++i)
                        BufSt<P>::st(wrsrc, f[m][i], vo0[m], i * plane_b + y * pitch_b, sc);
                }
            }
        };
        const int y_first = yb - RG - 2 * (lvl - 1);  // this level's row at iteration 0
        if (lvl == 1) {
#pragma unroll
            for (int k = 0; k < D; ++k) pull(buf[k], yb - RG + k);
        }
#pragma unroll
        for (int k = 0; k < D; ++k) pullm(mb[k], y_first + k);
        const int n_it = (ye - yb) + 3 * RG;
        for (int it0 = 0; it0 < n_it; it0 += B) {
#pragma unroll
            for (int k = 0; k < B; ++k) {
                const int it = it0 + k;
                if (it >= n_it) break;
                const int y = y_first + it;  // this level's row (wave-uniform)
                const bool row_on = y >= lo && y < hi;
                pullm(mb[(k + D) % B], y + D);
                if (lvl == 1) {
                    pull(buf[(k + D) % B], y + D);
                    if (row_on) {
                        C f[M][9];
#pragma unroll
                        for (int m = 0; m < M; ++m) {
#pragma unroll
                            for (int i = 0; i < 9; ++i) f[m][i] = BufLd<P>::cvt(buf[k][m][i], inv);
                            if (mb[k][m] & BB_BITS) {
                                // bounce-back: the node's own opposite population
#pragma unroll
                                for (int i = 0; i < 9; ++i) {
                                    const C o = BufLd<P>::ld(rsrc, vo0[m], OPPd[i] * plane_b + y * pitch_b, inv);
                                    f[m][i] = ((mb[k][m] >> (M_BB + i)) & 1u) ? o : f[m][i];
                                }
                            }
                        }
                        finish(f, mb[k], y);
                    }
                } else if (row_on) {
                    const int L = lvl - 2;
                    const int pa = (y + 13) % 3, pb = (y + 12) % 3, pc = (y + 11) & 3;  // pull rows
                    const int oa = (y + 12) % 3, oc = (y + 12) & 3;                     // own row
                    C f[M][9];
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        const int lc = c[m] + 1;
#pragma unroll
                        for (int i = 0; i < 9; ++i) {
                            const int g = GJd[i], cl = lc - CXd[i];
                            f[m][i] = CYd[i] < 0 ? rq[L][pa][g][cl]
                                                 : (CYd[i] == 0 ? rq[L][3 + pb][g][cl] : rq[L][6 + pc][g][cl]);
                        }
                        if (mb[k][m] & BB_BITS) {
                            // this node's populations of the level below, by direction
                            C own[9];
                            own[0] = rq[L][3 + pb][0][lc];
                            own[1] = rq[L][3 + pb][1][lc];
                            own[3] = rq[L][3 + pb][2][lc];
                            own[2] = rq[L][6 + oc][0][lc];
                            own[5] = rq[L][6 + oc][1][lc];
                            own[6] = rq[L][6 + oc][2][lc];
                            own[4] = rq[L][oa][0][lc];
                            own[7] = rq[L][oa][1][lc];
                            own[8] = rq[L][oa][2][lc];
#pragma unroll
                            for (int i = 0; i < 9; ++i)
                                f[m][i] = ((mb[k][m] >> (M_BB + i)) & 1u) ? own[OPPd[i]] : f[m][i];
                        }
                    }
                    finish(f, mb[k], y);
                }
                __syncthreads();
            }
        }
    }
}

template <int P, int N, int K, int M, int D>
__global__ __launch_bounds__(64 * N * K) void k_stepRC(JobDev j, const int64_t *d_t, int k0, bool src2, int H,
                                                       int chunks, int64_t nwork) {
    __shared__ typename RowsRingCh<P, N, K, M>::Array rq;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const int64_t smp = wk / chunks;
        stepRC_item<P, N, K, M, D>(j, d_t, k0, src2, H, smp, (int)(wk - smp * chunks), rq);
    }
}

// Batched form (see k_stepR_multi); launch number `launch` of a tick runs
// steps t + launch N .. of each job, t its step count at the tick's start.
template <int P, int N, int K, int M, int D>
__global__ __launch_bounds__(64 * N * K) void k_stepRC_multi(const FusedJob *jobs, int njobs, int64_t nwork,
                                                             int launch) {
    __shared__ typename RowsRingCh<P, N, K, M>::Array rq;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const FusedJob q = fused_entry(jobs, njobs, wk);
        const JobDev j = q.j;
        const int64_t local = wk - q.work0;
        const int64_t smp = local / q.chunks;
        stepRC_item<P, N, K, M, D>(j, q.d_t, launch * N, ((q.par ^ launch) & 1) != 0, q.H, smp,
                                   (int)(local - smp * q.chunks), rq);
    }
}

// ------------------------------------------------------------------ fused channel steps, strips
// The row pipeline down strips (STRIP in stepR_item) on the channels that
// stepRC_item takes, with the bounce-back on the writing side: a node hands
// f*_opp(i) on as its own f_i where its pull from x - c_i would meet a wall,
// writing it into the place in the rings where its solid neighbour would have
// put that pull. The reading side is then the periodic one (unconditional
// reads at the lane's own column, c_y >= 0 a row ahead), and only waves that
// hold a wall node pay, per such direction. The places lie in the row the node
// is in (c_iy = 0), the one before (c_iy = 1, written a step ago and not yet
// read) or the next (c_iy = -1: one more slot than the periodic rings keep, so
// that the row being read is left alone). No other lane may write them: solid
// nodes hand nothing on, and rows beyond the walls are not computed.
// A strip wraps around the lattice in x as the periodic one does; what comes
// in through an open end is then overwritten by its rule, and where the ends
// are walls (WALLS) nothing may cross the seam: the columns beside it push
// towards it into the rows' outermost place (column 0 of c_x = +1, the last of
// c_x = -1), which no neighbour in the strip fills and whose value never gets
// to a stored column. (An instance of its own: two selects before the row loop
// move the registers inside it, BF16S 3 to 4 % slower, FP64 2 %, FP32 2.5 %
// faster or 3.5 % slower as they were written.)
// 24 direction-rows of 128 columns per level, where the whole rows of
// stepRC_item keep 30 of up to 512: 6 to 8 steps per launch on any width
// instead of 2 to 4, and few samples make more work items.
template <int P, int N>
struct RowsRingCS {
    static constexpr int NR = N > 1 ? N - 1 : 1;
    static constexpr int CW = 64 * RowStrips<P>::M, MR = 2 * N;
    typename Prec<P>::C f[NR][8][3][CW];
    // the node masks of the last 2N rows of level 1, for the levels above: a
    // load of their own each row would wait, on the last level, for the stores
    // of the row before as well (one counter serves both: 1.9 us per row step,
    // whatever N)
    uint32_t mask[MR][CW];
};

template <int P, int N, int D, bool WALLS>
__device__ __forceinline__ void stepRCS_item(const JobDev &j, const int64_t *d_t, int k0, bool src2, int H,
                                             int64_t smp, int chunk, RowsRingCS<P, N> &rg, int x0, int W) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    constexpr int M = RowStrips<P>::M, RG = N - 1, CW = RowsRingCS<P, N>::CW, MR = RowsRingCS<P, N>::MR;
    constexpr uint32_t BB_BITS = 0x1FFu << M_BB, OPEN_BITS = 0x1FFu << M_OPEN;
    const T *src_all = (const T *)(src2 ? j.f2 : j.f);
    T *dst_all = (T *)(src2 ? j.f : j.f2);
    const int nx = j.nx, ny = j.ny;
    const int plane = (int)j.plane;
    const int plane_b = plane * (int)sizeof(T), pitch_b = (int)j.pitch * (int)sizeof(T);
    const float inv = j.inv_scale, sc = j.scale;
    const int lane = threadIdx.x & 63;
    const int lvl = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) + 1;  // 1..N
    const int64_t t_lvl = *d_t + k0 + (lvl - 1);
    int gx[M], vo0[M], vom[M], vop[M];
    bool st[M];  // the column is stored
    // LDS byte offsets of the lane's columns (see stepR_item)
    constexpr int GB = CW * (int)sizeof(C), SB = 3 * GB, RB = 8 * SB;
    char *const ring = reinterpret_cast<char *>(&rg.f);
    int ox[M], om[M], op[M], orx[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        const int c = m * 64 + lane;
        gx[m] = wrap_coord(x0 - RG + c, nx);
        st[m] = c >= RG && c < RG + W;
        vo0[m] = gx[m] * (int)sizeof(T);
        vom[m] = (gx[m] == 0 ? nx - 1 : gx[m] - 1) * (int)sizeof(T);
        vop[m] = (gx[m] == nx - 1 ? 0 : gx[m] + 1) * (int)sizeof(T);
        ox[m] = (lvl - 1) * RB + c * (int)sizeof(C);
        om[m] = (lvl - 1) * RB + (c == 0 ? CW - 1 : c - 1) * (int)sizeof(C);
        op[m] = (lvl - 1) * RB + (c == CW - 1 ? 0 : c + 1) * (int)sizeof(C);
        orx[m] = (lvl - 2) * RB + c * (int)sizeof(C);
    }
    if constexpr (WALLS) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            if (gx[m] == 0) om[m] = (lvl - 1) * RB + (CW - 1) * (int)sizeof(C);
            if (gx[m] == nx - 1) op[m] = (lvl - 1) * RB;
        }
    }
    auto at = [&](int base, int slot, int g) -> C & { return *reinterpret_cast<C *>(ring + base + slot * SB + g * GB); };
    auto fresh = [&]() {
#pragma unroll
        for (int m = 0; m < M; ++m) asm("" : "+v"(ox[m]), "+v"(om[m]), "+v"(op[m]), "+v"(orx[m]));
    };
    const __amdgpu_buffer_rsrc_t mrsrc = make_rsrc(j.mask, ny * (int)j.pitch * 4);
    const int span = RG - (lvl - 1);  // rows beyond the chunk on each side
    constexpr int B = D + 1;
    using R = typename BufLd<P>::R;
    R buf[B][M][9];
    const int yb = chunk * H, ye = min(ny, yb + H);
    const int y_lo = max(0, yb - span), y_hi = min(ny, ye + span);  // this level's rows
    const T *src = src_all + smp * 9 * (int64_t)plane;
    T *dst = dst_all + smp * 9 * (int64_t)plane;
    const C omega = (C)j.smp[smp].omega;
    // s(t) 4 u_peak of this level's step (uniform)
    const double a_in = ramp_factor(t_lvl, j.ramp) * 4.0 * j.smp[smp].u_peak;
    const __amdgpu_buffer_rsrc_t rsrc = make_rsrc(src, 9 * plane_b), wrsrc = make_rsrc(dst, 9 * plane_b);
    auto clampy = [&](int y) { return y < 0 ? 0 : (y >= ny ? ny - 1 : y); };
    auto pullm = [&](uint32_t *mm, int y) {
        const int mo = clampy(y) * (int)j.pitch * 4;
#pragma unroll
        for (int m = 0; m < M; ++m) mm[m] = __builtin_amdgcn_raw_buffer_load_b32(mrsrc, gx[m] * 4, mo, 0);
    };
    // Level 1's pulls of a row whose masks mm are known: the wall rule selects
    // each lane's address (the node's own opposite population), for every row
    // (a branch for the waves that hold a wall node leaves copies of the load
    // buffers, which wait for them).
    auto pull = [&](R (*f)[9], int y, const uint32_t *mm) {
        const int gy = clampy(y);
        const int r0 = gy * pitch_b, rm = (gy == 0 ? ny - 1 : gy - 1) * pitch_b,
                  rp = (gy == ny - 1 ? 0 : gy + 1) * pitch_b;
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const int vo = CXd[i] > 0 ? vom[m] : (CXd[i] < 0 ? vop[m] : vo0[m]);
                const int ro = CYd[i] > 0 ? rm : (CYd[i] < 0 ? rp : r0);
                const int from = vo + i * plane_b + ro, own = vo0[m] + OPPd[i] * plane_b + r0;
                f[m][i] = BufLd<P>::raw(rsrc, ((mm[m] >> (M_BB + i)) & 1u) ? own : from, 0);
            }
    };
    // Slots by the row step a row is written in (see stepR_item): c_y = -1 in
    // 0-2 and c_y = +1 in 5-7, each step mod 3, c_y = 0 in 3-4, step mod 2;
    // read one step later, the c_y = +1 ones two.
    auto put = [&](int u, int m, const C *v) {
        const int s3 = u % 3, sb = 3 + (u & 1);
        at(ox[m], s3, 0) = v[4];
        at(ox[m], sb, 0) = v[0];
        at(om[m], s3, 1) = v[7];
        at(om[m], sb, 2) = v[3];
        at(op[m], s3, 2) = v[8];
        at(op[m], sb, 1) = v[1];
        at(ox[m], 5 + s3, 0) = v[2];
        at(op[m], 5 + s3, 1) = v[5];
        at(om[m], 5 + s3, 2) = v[6];
    };
    auto bounce = [&](int u, int m, uint32_t mm, const C *v) {
        const int next = (u + 1) % 3, prev = (u + 2) % 3, sb = 3 + (u & 1);
#pragma unroll
        for (int i = 1; i < 9; ++i)
            if ((mm >> (M_BB + i)) & 1u)
                at(ox[m], CYd[i] < 0 ? next : (CYd[i] == 0 ? sb : 5 + prev), GJd[i]) = v[OPPd[i]];
    };
    // the open-column rule, then collide, then hand on or store
    auto finish = [&](C (*f)[9], const uint32_t *mm, int y, int u) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            if (mm[m] & OPEN_BITS) {
                // (which pulls need zeroing: see stepRC_item)
                if (t_lvl == 0 || nx == 1) {
#pragma unroll
                    for (int i = 0; i < 9; ++i) f[m][i] = ((mm[m] >> (M_OPEN + i)) & 1u) ? C(0) : f[m][i];
                }
                if (t_lvl > 0) zou_he_u(f[m], gx[m] == 0, gx[m] == 0 ? (C)inflow_u_a(a_in, ny, y) : C(0));
            }
        }
#pragma unroll
        for (int m = 0; m < M; ++m) {
            C drho, ux, uy;
            bgk(f[m], omega, drho, ux, uy);
        }
        if (lvl < N) {
#pragma unroll
            for (int m = 0; m < M; ++m)
#pragma unroll
                for (int i = 0; i < 9; ++i) f[m][i] = PR::rt(f[m][i], sc, inv);
            uint32_t any = 0;
#pragma unroll
            for (int m = 0; m < M; ++m) any |= mm[m];
            // (uniform: most waves hold neither solid nodes nor their neighbours)
            if (!__any((any & (BB_BITS | M_SOLID)) != 0)) {
#pragma unroll
                for (int m = 0; m < M; ++m) put(u, m, f[m]);
            } else {
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    if (!(mm[m] & M_SOLID)) put(u, m, f[m]);
                    if (mm[m] & BB_BITS) bounce(u, m, mm[m], f[m]);
                }
            }
        } else {
#pragma unroll
            for (int m = 0; m < M; ++m) {
                if (!st[m] || (mm[m] & M_SOLID)) continue;
#pragma unroll
                for (int i = 0; i < 9; ++i) BufSt<P>::st(wrsrc, f[m][i], vo0[m], i * plane_b + y * pitch_b, sc);
            }
        }
    };
    const int y_first = yb - RG - 2 * (lvl - 1);  // this level's row at step 0
    const int n_it = (ye - yb) + 3 * RG;
    static_assert(6 % B == 0, "the row loops turn over six steps");
    if (lvl == 1) {
        // masks four rows ahead (the pulls, D rows ahead, need them)
        uint32_t mb[6][M];
        int ms = 0;  // this step's row of the mask ring
#pragma unroll
        for (int k = 0; k < 4; ++k) pullm(mb[k], y_first + k);
#pragma unroll
        for (int k = 0; k < D; ++k) pull(buf[k], y_first + k, mb[k]);
        for (int it0 = 0; it0 < n_it; it0 += 6) {
#pragma unroll
            for (int u = 0; u < 6; ++u) {
                const int it = it0 + u;
                if (it >= n_it) break;
                const int y = y_first + it;
                if (u == 0) fresh();
                if (y < y_hi) {
                    pullm(mb[(u + 4) % 6], y + 4);
                    pull(buf[(u + D) % B], y + D, mb[(u + D) % 6]);
                    if (y >= y_lo) {
                        C f[M][9];
#pragma unroll
                        for (int m = 0; m < M; ++m) rg.mask[ms][m * 64 + lane] = mb[u][m];
#pragma unroll
                        for (int m = 0; m < M; ++m)
#pragma unroll
                            for (int i = 0; i < 9; ++i) f[m][i] = BufLd<P>::cvt(buf[u % B][m][i], inv);
                        finish(f, mb[u], y, u);
                    }
                }
                if (++ms == MR) ms = 0;
                __syncthreads();
            }
        }
    } else {
        C pre[2][M][6];
        int ms = MR - 2 * (lvl - 1);  // the mask ring's row of this level's row: 2 (lvl - 1) steps old
        for (int it0 = 0; it0 < n_it; it0 += 6) {
#pragma unroll
            for (int u = 0; u < 6; ++u) {
                const int it = it0 + u, k = u & 1;
                if (it >= n_it) break;
                const int y = y_first + it;  // this level's row (wave-uniform)
                if (u == 0) fresh();
                if (y >= y_lo - 1 && y < y_hi) {
                    // row y's c_y = -1 pulls and the next row's others
                    const int s3 = (u + 2) % 3, sb = 3 + ((u + 1) & 1), sc3 = 5 + (u + 1) % 3;
                    C f[M][9];
                    C (*q)[6] = pre[k ^ 1];
                    uint32_t mm[M];
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        mm[m] = rg.mask[ms][m * 64 + lane];
                        f[m][4] = at(orx[m], s3, 0);
                        f[m][7] = at(orx[m], s3, 1);
                        f[m][8] = at(orx[m], s3, 2);
                        q[m][0] = at(orx[m], sb, 0);   // (0, 0)
                        q[m][1] = at(orx[m], sb, 1);   // (1, 0)
                        q[m][3] = at(orx[m], sb, 2);   // (-1, 0)
                        q[m][2] = at(orx[m], sc3, 0);  // (0, 1)
                        q[m][4] = at(orx[m], sc3, 1);  // (1, 1)
                        q[m][5] = at(orx[m], sc3, 2);  // (-1, 1)
                        f[m][0] = pre[k][m][0];
                        f[m][1] = pre[k][m][1];
                        f[m][2] = pre[k][m][2];
                        f[m][3] = pre[k][m][3];
                        f[m][5] = pre[k][m][4];
                        f[m][6] = pre[k][m][5];
                    }
                    __builtin_amdgcn_sched_barrier(0);
                    if (y >= y_lo) finish(f, mm, y, u);
                }
                if (++ms == MR) ms = 0;
                __syncthreads();
            }
        }
    }
}

// strip runs fastest, as in k_stepRS
template <int P, int N, int D, bool WALLS>
__global__ __launch_bounds__(64 * N, 2) void k_stepRCS(
    JobDev j, const int64_t *d_t, int k0, bool src2, int W, int strips, int H, int chunks, int64_t nwork) {
    __shared__ RowsRingCS<P, N> rg;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const int64_t smp = wk / ((int64_t)chunks * strips);
        const int rem = (int)(wk - smp * chunks * strips);
        const int chunk = rem / strips;
        const int x0 = min((rem - chunk * strips) * W, j.nx - W);
        stepRCS_item<P, N, D, WALLS>(j, d_t, k0, src2, H, smp, chunk, rg, x0, W);
    }
}

// Batched form (see k_stepRC_multi), for channels whose ends are not walls
template <int P, int N, int D>
__global__ __launch_bounds__(64 * N, 2) void k_stepRCS_multi(const FusedJob *jobs, int njobs, int64_t nwork,
                                                             int launch) {
    __shared__ RowsRingCS<P, N> rg;
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const FusedJob q = fused_entry(jobs, njobs, wk);
        const JobDev j = q.j;
        const int64_t local = wk - q.work0;
        const int64_t smp = local / ((int64_t)q.chunks * q.strips);
        const int rem = (int)(local - smp * q.chunks * q.strips);
        const int chunk = rem / q.strips;
        const int x0 = min((rem - chunk * q.strips) * q.W, j.nx - q.W);
        stepRCS_item<P, N, D, false>(j, q.d_t, launch * N, ((q.par ^ launch) & 1) != 0, q.H, smp, chunk, rg, x0, q.W);
    }
}

// ------------------------------------------------------------------ fused steps, resident tiles
// Small periodic jobs, which leave most of the card idle and take the latency
// of a launch and of its steps: one node per lane, its populations in registers
// for all n steps of the launch, the eight moving ones exchanged through LDS
// once per step (two buffers in turn, one barrier). A workgroup takes a region
// of up to 1024 nodes; in x and in y it is either the whole period, whose ends
// meet, or an output range with a ring of n - 1 nodes around it, which turns
// wrong by one node per step and is not stored. The row pipelines take n + (rows
// of a chunk) + 2 n row steps of 0.5 us for n steps whatever the job's size;
// here a step takes about as long as one of theirs.
template <int P>
__global__ __launch_bounds__(TILE_NODES) void k_stepT(JobDev j, bool src2, int n, TileShape g, int64_t nwork) {
    using PR = Prec<P>;
    using C = typename PR::C;
    using T = typename PR::T;
    __shared__ C lds[2][8][TILE_NODES];
    const T *src_all = (const T *)(src2 ? j.f2 : j.f);
    T *dst_all = (T *)(src2 ? j.f : j.f2);
    const int nx = j.nx, ny = j.ny, e = threadIdx.x;
    const int pitch = (int)j.pitch, plane = (int)j.plane;
    const float inv = j.inv_scale, sc = j.scale;
    const int rx = g.RW == nx ? 0 : n - 1, ry = g.RH == ny ? 0 : n - 1;  // ring
    // lanes past the region repeat its last row's nodes and store nothing
    const int row = e / g.RW, c = e - row * g.RW, r = min(row, g.RH - 1);
    const bool in = row < g.RH && c >= rx && c < rx + g.OW && r >= ry && r < ry + g.OH;
    // where each direction is pulled from: across the ends of a whole period,
    // else (on the region's edge) from the node itself, whatever that gives
    int from[9];
#pragma unroll
    for (int i = 1; i < 9; ++i) {
        int fr = r - CYd[i], fc = c - CXd[i];
        fr = fr < 0 ? (ry ? 0 : g.RH - 1) : (fr >= g.RH ? (ry ? g.RH - 1 : 0) : fr);
        fc = fc < 0 ? (rx ? 0 : g.RW - 1) : (fc >= g.RW ? (rx ? g.RW - 1 : 0) : fc);
        from[i] = fr * g.RW + fc;
    }
    const int64_t G = gridDim.x;
    for (int64_t wk = xcd_logical(blockIdx.x, G); wk < nwork; wk += G) {
        const int64_t smp = wk / (g.tiles_x * g.tiles_y);
        const int rem = (int)(wk - smp * (g.tiles_x * g.tiles_y));
        const int ty = rem / g.tiles_x, tx = rem - ty * g.tiles_x;
        // the last tile of a row or column moves back to end at the lattice's
        const int x0 = min(tx * g.OW, nx - g.OW), y0 = min(ty * g.OH, ny - g.OH);
        const int gx = wrap_coord(x0 - rx + c, nx), gy = wrap_coord(y0 - ry + r, ny);
        const T *src = src_all + smp * 9 * (int64_t)plane;
        T *dst = dst_all + smp * 9 * (int64_t)plane;
        const C omega = (C)j.smp[smp].omega;
        const int xm = gx == 0 ? nx - 1 : gx - 1, xp = gx == nx - 1 ? 0 : gx + 1;
        const int ym = gy == 0 ? ny - 1 : gy - 1, yp = gy == ny - 1 ? 0 : gy + 1;
        C f[9], drho, ux, uy;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int x = CXd[i] > 0 ? xm : (CXd[i] < 0 ? xp : gx), y = CYd[i] > 0 ? ym : (CYd[i] < 0 ? yp : gy);
            f[i] = PR::ld(src + (i * plane + y * pitch + x), inv);
        }
        bgk(f, omega, drho, ux, uy);
        for (int s = 1; s < n; ++s) {
            C(*b)[TILE_NODES] = lds[s & 1];
            f[0] = PR::rt(f[0], sc, inv);
#pragma unroll
            for (int i = 1; i < 9; ++i) b[i - 1][e] = PR::rt(f[i], sc, inv);
            __syncthreads();
#pragma unroll
            for (int i = 1; i < 9; ++i) f[i] = b[i - 1][from[i]];
            bgk(f, omega, drho, ux, uy);
        }
        if (in) {
            const int own = gy * pitch + gx;
#pragma unroll
            for (int i = 0; i < 9; ++i) PR::st(dst + (i * plane + own), f[i], sc);
        }
        __syncthreads();  // both buffers are free for the next tile
    }
}

// ------------------------------------------------------------------ launchers
template <int P, int N>
static void stepN_p(const JobDev &j, bool src2, int fty, hipStream_t s) {
    const int tiles_x = (j.nx + FUSE_TX - 1) / FUSE_TX;
    auto go = [&](auto ty_c) {
        constexpr int TY = decltype(ty_c)::value;
        const int tiles_y = (j.ny + TY - 1) / TY;
        const int64_t ntiles = (int64_t)j.S * tiles_x * tiles_y;
        const int64_t G = std::min<int64_t>(ntiles, 0x7fffffff);
        k_stepN<P, TY, N><<<(unsigned)G, 256, 0, s>>>(j, src2, tiles_x, tiles_y, ntiles);
    };
    // FP64 tiles are half as tall (the LDS tile holds doubles)
    if constexpr (P == UQ_FP64) {
        if (fty <= 4) go(std::integral_constant<int, 4>());
        else go(std::integral_constant<int, 8>());
    } else {
        if (fty <= 8) go(std::integral_constant<int, 8>());
        else go(std::integral_constant<int, 16>());
    }
}
template <int P, int N>
static void stepW_p(const JobDev &j, bool src2, int rows, bool nt, hipStream_t s) {
    int W, strips;
    window_strips(j.nx, N, &W, &strips);
    const int H = std::max(8, std::min(rows, j.ny));
    const int chunks = (j.ny + H - 1) / H;
    const int64_t nwork = (int64_t)j.S * strips * chunks;
    const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
    // rows of loads in flight: 3 (2 at FP64, whose registers are scarcer)
    constexpr int D = P == UQ_FP64 ? 2 : 3;
    k_stepW<P, N, D><<<(unsigned)G, 64 * N, 0, s>>>(j, src2, W, strips, H, chunks, nwork, nt);
}

template <int P>
static void stepT_p(const JobDev &j, bool src2, int n, hipStream_t s) {
    const TileShape g = tile_shape(j.nx, j.ny, n);
    const int64_t nwork = (int64_t)j.S * g.tiles_x * g.tiles_y;
    const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
    const int threads = (g.RW * g.RH + 63) / 64 * 64;
    k_stepT<P><<<(unsigned)G, threads, 0, s>>>(j, src2, n, g, nwork);
}

template <int P, int N>
static void stepRS_p(const JobDev &j, bool src2, int rows, hipStream_t s) {
    int W, strips;
    row_strips(P, j.nx, N, &W, &strips);
    const int H = std::max(8, std::min(rows, j.ny));
    const int chunks = (j.ny + H - 1) / H;
    const int64_t nwork = (int64_t)j.S * strips * chunks;
    const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
    k_stepRS<P, N, 2><<<(unsigned)G, 64 * N * RowStrips<P>::K, 0, s>>>(j, src2, W, strips, H, chunks, nwork);
}

// full-row kernel: K waves per level of M columns per lane cover nx, with
// N K <= 16 waves and (N - 1) 21 LDS rows of 64 K M values within 160 KB
template <int P, int N, int K, int M>
static void stepR_k(const JobDev &j, bool src2, int rows, bool nt, hipStream_t s) {
    const int H = std::max(8, std::min(rows, j.ny));
    const int chunks = (j.ny + H - 1) / H;
    const int64_t nwork = (int64_t)j.S * chunks;
    const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
    k_stepR<P, N, K, M, 2><<<(unsigned)G, 64 * N * K, 0, s>>>(j, src2, H, chunks, nwork, nt);
}
template <int P, int N>
static void stepR_p(const JobDev &j, bool src2, int rows, bool nt, hipStream_t s) {
    int K = 0, M = 0;
    if (!rows_shape(P, N, RING_ROWS_TGV, j.nx, &K, &M)) return;
#define UQ_ROWS_CASE(kk, mm)                                                      \
    if constexpr (rows_fit(P, N, RING_ROWS_TGV, kk, mm)) {                        \
        if (K == kk && M == mm) return stepR_k<P, N, kk, mm>(j, src2, rows, nt, s); \
    }
    UQ_ROWS_CASES(UQ_ROWS_CASE)
#undef UQ_ROWS_CASE
}
template <int P, int N, int K, int M>
static void stepRC_k(const JobDev &j, const int64_t *d_t, int k, bool src2, int rows, hipStream_t s) {
    const int H = std::max(8, std::min(rows, j.ny));
    const int chunks = (j.ny + H - 1) / H;
    const int64_t nwork = (int64_t)j.S * chunks;
    const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
    k_stepRC<P, N, K, M, 2><<<(unsigned)G, 64 * N * K, 0, s>>>(j, d_t, k, src2, H, chunks, nwork);
}

template <int P, int N>
static void stepRC_p(const JobDev &j, const int64_t *d_t, int k, bool src2, int rows, hipStream_t s) {
    int K = 0, M = 0;
    if (!rows_shape(P, N, RING_ROWS_CH, j.nx, &K, &M)) return;
#define UQ_ROWS_CASE(kk, mm)                                                              \
    if constexpr (rows_fit(P, N, RING_ROWS_CH, kk, mm)) {                                 \
        if (K == kk && M == mm) return stepRC_k<P, N, kk, mm>(j, d_t, k, src2, rows, s);  \
    }
    UQ_ROWS_CASES(UQ_ROWS_CASE)
#undef UQ_ROWS_CASE
}
template <int P, int N>
static void stepRCS_p(const JobDev &j, const int64_t *d_t, int k, bool src2, int rows, hipStream_t s) {
    int W, strips;
    row_strips(P, j.nx, N, &W, &strips);
    const int H = std::max(8, std::min(rows, j.ny));
    const int chunks = (j.ny + H - 1) / H;
    const int64_t nwork = (int64_t)j.S * strips * chunks;
    const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
    if (j.xbc == UQ_XBC_WALLS)
        k_stepRCS<P, N, 2, true><<<(unsigned)G, 64 * N, 0, s>>>(j, d_t, k, src2, W, strips, H, chunks, nwork);
    else
        k_stepRCS<P, N, 2, false><<<(unsigned)G, 64 * N, 0, s>>>(j, d_t, k, src2, W, strips, H, chunks, nwork);
}
template <int P, int N, int K, int M>
static void multi_k(int kind, const FusedJob *jobs, int njobs, int64_t nwork, int launch, hipStream_t s) {
    const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
    if (kind == 0) {
        if constexpr (rows_fit(P, N, RING_ROWS_TGV, K, M))
            k_stepR_multi<P, N, K, M, 2><<<(unsigned)G, 64 * N * K, 0, s>>>(jobs, njobs, nwork, launch, false);
    } else {
        if constexpr (N <= 4 && rows_fit(P, N, RING_ROWS_CH, K, M))
            k_stepRC_multi<P, N, K, M, 2><<<(unsigned)G, 64 * N * K, 0, s>>>(jobs, njobs, nwork, launch);
    }
}

template <int P, int N>
static bool multi_n(int kind, int K, int M, const FusedJob *jobs, int njobs, int64_t nwork, int launch,
                    hipStream_t s) {
#define UQ_MULTI_CASE(kk, mm)                                         \
    if (K == kk && M == mm) {                                         \
        multi_k<P, N, kk, mm>(kind, jobs, njobs, nwork, launch, s);   \
        return true;                                                  \
    }
    UQ_ROWS_CASES(UQ_MULTI_CASE)
#undef UQ_MULTI_CASE
    return false;
}

template <int P>
bool fused_launch_multi(int kind, int n, int K, int M, const FusedJob *jobs, int njobs, int64_t nwork, int launch,
                    hipStream_t s) {
    if (kind == 2) {
        if (n != 8) return false;
        const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
        k_stepRS_multi<P, 8, 2><<<(unsigned)G, 512 * RowStrips<P>::K, 0, s>>>(jobs, njobs, nwork, launch);
        return true;
    }
    if (kind == 3) {
        if (n != 8) return false;
        const int64_t G = std::min<int64_t>(nwork, 0x7fffffff);
        k_stepRCS_multi<P, 8, 2><<<(unsigned)G, 512, 0, s>>>(jobs, njobs, nwork, launch);
        return true;
    }
    if (kind == 0) {
        if (n == 4) return multi_n<P, 4>(0, K, M, jobs, njobs, nwork, launch, s);
        if (n == 6) return multi_n<P, 6>(0, K, M, jobs, njobs, nwork, launch, s);
        if (n == 8) return multi_n<P, 8>(0, K, M, jobs, njobs, nwork, launch, s);
        return false;
    }
    if (n == 2) return multi_n<P, 2>(1, K, M, jobs, njobs, nwork, launch, s);
    if (n == 3) return multi_n<P, 3>(1, K, M, jobs, njobs, nwork, launch, s);
    if (n == 4) return multi_n<P, 4>(1, K, M, jobs, njobs, nwork, launch, s);
    return false;
}
template <int P>
void fused_launch_channel(const JobDev &j, int n, const int64_t *d_t, int k, bool src2, int fty, int window,
                          hipStream_t s) {
    if (window == 3) {
        if (n == 3) stepRCS_p<P, 3>(j, d_t, k, src2, fty, s);
        else if (n == 4) stepRCS_p<P, 4>(j, d_t, k, src2, fty, s);
        else if (n == 5) stepRCS_p<P, 5>(j, d_t, k, src2, fty, s);
        else if (n == 6) stepRCS_p<P, 6>(j, d_t, k, src2, fty, s);
        else if (n == 7 || P == UQ_FP64) stepRCS_p<P, 7>(j, d_t, k, src2, fty, s);
        else if constexpr (P != UQ_FP64) stepRCS_p<P, 8>(j, d_t, k, src2, fty, s);
    } else if (n == 2) stepRC_p<P, 2>(j, d_t, k, src2, fty, s);
    else if (n == 3) stepRC_p<P, 3>(j, d_t, k, src2, fty, s);
    else stepRC_p<P, 4>(j, d_t, k, src2, fty, s);
}

template <int P>
void fused_launch_tgv(const JobDev &j, int n, bool src2, int fty, int window, bool nt, hipStream_t s) {
    if (window == 4) {
        stepT_p<P>(j, src2, n, s);
    } else if (window == 3) {
        if (n == 3) stepRS_p<P, 3>(j, src2, fty, s);
        else if (n == 4) stepRS_p<P, 4>(j, src2, fty, s);
        else if (n == 5) stepRS_p<P, 5>(j, src2, fty, s);
        else if (n == 6) stepRS_p<P, 6>(j, src2, fty, s);
        else if (n == 7) stepRS_p<P, 7>(j, src2, fty, s);
        else stepRS_p<P, 8>(j, src2, fty, s);
    } else if (window == 2) {
        if (n == 2) stepR_p<P, 2>(j, src2, fty, nt, s);
        else if (n == 3) stepR_p<P, 3>(j, src2, fty, nt, s);
        else if (n == 4) stepR_p<P, 4>(j, src2, fty, nt, s);
        else if (n == 5) stepR_p<P, 5>(j, src2, fty, nt, s);
        else if (n == 6) stepR_p<P, 6>(j, src2, fty, nt, s);
        else if (n == 7) stepR_p<P, 7>(j, src2, fty, nt, s);
        else stepR_p<P, 8>(j, src2, fty, nt, s);
    } else if (window) {
        if (n == 2) stepW_p<P, 2>(j, src2, fty, nt, s);
        else if (n == 3) stepW_p<P, 3>(j, src2, fty, nt, s);
        else stepW_p<P, 4>(j, src2, fty, nt, s);
    } else {
        if (n == 2) stepN_p<P, 2>(j, src2, fty, s);
        else if (n == 3) stepN_p<P, 3>(j, src2, fty, s);
        else stepN_p<P, 4>(j, src2, fty, s);
    }
}

template void fused_launch_tgv<UQ_PREC>(const JobDev &, int, bool, int, int, bool, hipStream_t);
template void fused_launch_channel<UQ_PREC>(const JobDev &, int, const int64_t *, int, bool, int, int, hipStream_t);
#if UQ_PREC != 0  // the server runs double precision (UQ_FP64) in single steps
template bool fused_launch_multi<UQ_PREC>(int, int, int, int, const FusedJob *, int, int64_t, int, hipStream_t);
#endif

}  // namespace uqi
