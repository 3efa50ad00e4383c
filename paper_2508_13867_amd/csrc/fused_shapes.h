// Launch shapes of the temporally blocked kernels: what the launchers (one
// translation unit per storage precision) and the host-side rules share.
#pragma once

#include "uq_internal.h"

namespace uqi {

// Shapes of the full-row kernels: K waves per level of M columns per lane
// (K <= 4 with one column, <= 6 with two: rows up to 768 columns), N K <= 16
// waves, and (N - 1) LDS rings of ROWS direction-rows (21 on the periodic
// lattice, 30 on the channel) of about 64 K M compute values within 160 KB.
// The shape used for a lattice nx wide: the fewest columns per lane (M = 1,
// else 2) whose K = ceil(nx / 64 M) fits; 0 if none.
constexpr int RING_ROWS_TGV = 21, RING_ROWS_CH = 30;

// Registers: in single precision a lane of the periodic kernel colliding two
// columns fits 128 VGPRs (4 waves per SIMD: up to 16 waves), the channel
// kernel's about 165 (12 waves, 3 per SIMD); in double precision two columns
// keep to 8 waves (256 VGPRs) and one column to 12 (168). One column per
// lane fits 128 in single precision. (__launch_bounds__ holds the compiler to
// the budget of the workgroup size, so these limits only keep out shapes
// that would spill.)
constexpr bool rows_regs_fit(int prec, int waves, int M, bool channel) {
    return prec == UQ_FP64 ? waves <= (M == 2 ? 8 : 12) : (M == 2 && channel ? waves <= 12 : true);
}

// values per LDS row: the periodic kernel's rows hold its 64 K M columns
// (shifted writes wrap inside the row); the channel's also two end columns,
// padded to a multiple of 64
constexpr int ring_cols(int rows, int K, int M) { return 64 * K * M + (rows == RING_ROWS_CH ? 64 : 0); }

constexpr bool rows_fit(int prec, int n, int rows, int K, int M) {
    return n * K <= 16 && K <= (M == 2 ? 6 : 4) && rows_regs_fit(prec, n * K, M, rows == RING_ROWS_CH) &&
           (int64_t)(n - 1) * rows * ring_cols(rows, K, M) * (prec == UQ_FP64 ? 8 : 4) <= 160 * 1024;
}

// waves per level and columns per lane for rows nx wide (0 if none fits)
int rows_shape(int prec, int n, int rows, int nx, int *K, int *M);

// the instances (K, M) a launcher may take
#define UQ_ROWS_CASES(CASE) \
    CASE(2, 1) CASE(3, 1) CASE(4, 1) CASE(2, 2) CASE(3, 2) CASE(4, 2) CASE(5, 2) CASE(6, 2)

// The strip form of the row pipelines (window 3, any width): K waves per level
// of M columns per lane, WAVES per SIMD at least (the channel's: 2).
template <int P>
struct RowStrips {
    static constexpr int K = 1, M = 2, WAVES = P == UQ_FP64 ? 2 : 4;
};
// Regions of the resident-tile kernel (window 4): OW x OH output nodes and the
// RW x RH <= TILE_NODES nodes computed for them.
constexpr int TILE_NODES = 1024, TILE_MAX_STEPS = 16;
struct TileShape {
    int RW, RH, OW, OH, tiles_x, tiles_y;
};
// the fewest tiles for n steps per launch
TileShape tile_shape(int nx, int ny, int n);

// One fused launch of precision P (see launch_fused, launch_fused_multi):
// defined in fused_kernels.hip, which is compiled once per precision.
template <int P>
void fused_launch_tgv(const JobDev &j, int n, bool src2, int fty, int window, bool nt, hipStream_t s);
template <int P>
void fused_launch_channel(const JobDev &j, int n, const int64_t *d_t, int k, bool src2, int fty, int window,
                          hipStream_t s);
template <int P>
bool fused_launch_multi(int kind, int n, int K, int M, const FusedJob *jobs, int njobs, int64_t nwork, int launch,
                        hipStream_t s);

}  // namespace uqi
