// Internal interface between the HIP kernels (scf_kernels.hip) and the host runtime
// (scf_runtime.hip) of libscf.  Not installed; the public ABI is include/scf.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace scf {

// Per-channel constants, one table entry per channel, read by every kernel.
// Device region of a channel, in floats from the workspace base:
//   off + b*18*plane     population buffer b in {0,1}: [k][i][y][pitch], k = A,B; i = 0..8
//   off + 36*plane       density field [k][y][pitch]
//   off + 38*plane       (masked channels) solid-neighbourhood codes, uint16 [y][pitch]
struct Chan {
    int32_t nx, ny, pitch, x0, x1, xs;   // xs = x0/2: liquid-reservoir centre (scan start)
    int32_t row_base;                    // first entry of this channel in the packed row list
    int32_t masked;                      // 1: solid nodes from the mask codes, 0: wall rows
    int64_t off;                         // float offset of population buffer 0
    int64_t plane;                       // ny * pitch
    int64_t moff;                        // float offset of the code field (masked channels)
    float G;                             // bulk coupling (D2Q9 weights)
    float gw[2];                         // wall couplings
    float omega[2];                      // 1/tau_k
    float tm[2];                         // tau_k / m_k
    float wm[2];                         // m_k / tau_k
    float c1[2];                         // (1 - alpha_k) / 5: axis rest coefficient
    float c0[2];                         // alpha_k: rest-direction coefficient (used at init)
    float inv_m[2];                      // 1 / m_k
    float pad1;
};

// One row of one channel, for the per-row kernels (two-kernel step, observe, init, copies).
struct RowRef {
    int32_t chan, y;
};

// Per-row partial sums written by the observe pass.
struct RowPartial {
    double mass[2];
    int32_t bad;
    int32_t pad[3];
};

// Observation record (layout of scf_obs in include/scf.h).
struct ObsRec {
    int64_t t;
    double mass[2];
    double z, precursor, precursor_lo, precursor_hi;
    int32_t flags;
    int32_t reserved;
};

struct TileDesc {
    int32_t chan, xb, yb, ye;   // strip [xb, xb+bx) x rows [yb, ye)
    int32_t down;               // 0: rows walked upward from yb, 1: downward from ye-1
    int32_t w;                  // output columns of the strip (two-step tiles)
    int32_t pad[2];
};

// Kernel launchers (all asynchronous on `stream`; return hipSuccess or the launch error).
// launch_init builds the masked channels' codes, then the initial populations.
hipError_t launch_init(const Chan* chans, const RowRef* rows, int nrows, float* ws, hipStream_t s);
// Fused steps: with `first` non-NULL (persistent schedules) the launch has exactly `grid` blocks
// and block b runs tiles [first[b], first[b+1]); otherwise blocks stride over the whole list.
hipError_t launch_step_fused(int bx, bool masked, const Chan* chans, const TileDesc* tiles,
                             int ntiles, const int32_t* first, int grid, float* ws, int src,
                             hipStream_t s);
// Two time steps in one pass; each tile carries its output width w <= bx - 6 (see k_step_fused2).
hipError_t launch_step_fused2(int bx, bool masked, const Chan* chans, const TileDesc* tiles,
                              int ntiles, const int32_t* first, int grid, float* ws, int src,
                              hipStream_t s);
// k = 2..4 time steps of a large box per pass, k wavefront groups of kPipeCols columns (see
// k_step_pipe): `grid` blocks, block b runs tiles [first[b], first[b+1]), each at most
// pipe_out_x(kPipeSteps) columns wide.
constexpr int kPipeCols = 256, kPipeSteps = 4;
// Rows of a tile's stream: its own, 2k - 1 before and after, and one more for an even number.
__host__ __device__ inline int pipe_rows(int rows, int k) { return (rows + 2 * (2 * k - 1) + 1) & ~1; }
constexpr int pipe_out_x(int k) { return kPipeCols - 2 * (2 * k - 1); }
hipError_t launch_step_pipe(int k, bool masked, const Chan* chans, const TileDesc* tiles, const int32_t* first, int grid,
                            float* ws, int src, hipStream_t s);
// k = 1..4 time steps of a small tile per launch, one thread per node (see k_step_region).  The
// block's region of nodes is 22 x 23 or 32 x 32; its output tile is 2 (2k - 1) nodes smaller each
// way.  `one` holds a single channel's constants, its tiles following from the block index; with
// `tiles` (several channels) both come from the tables.
enum { kRegionSmall = 0, kRegionLarge = 1, kRegionMaxSteps = 4 };
inline int region_out_x(int region, int k) { return (region == kRegionSmall ? 22 : 32) - 2 * (2 * k - 1); }
inline int region_out_y(int region, int k) { return (region == kRegionSmall ? 23 : 32) - 2 * (2 * k - 1); }
hipError_t launch_step_region(int region, int k, bool masked, const Chan& one, const Chan* chans, const TileDesc* tiles,
                              int ntiles, float* ws, int src, hipStream_t s);
// Blocks of the fused step (fuse 1 or 2) that one CU holds at once; 0 if the query fails.
int resident_blocks_per_cu(int bx, bool masked, int fuse);
hipError_t launch_step_two_kernel(const Chan* chans, const RowRef* rows, int nrows, float* ws,
                                  int src, hipStream_t s);
hipError_t launch_observe(const Chan* chans, const RowRef* rows, int nrows, int nchan, float* ws,
                          int src, RowPartial* partials, ObsRec* now, ObsRec* ring,
                          int32_t* counter, int max_samples, int record, hipStream_t s);
// Densities of channel ch (n_A, n_B, ny x nx each, unpadded) into `out`.
hipError_t launch_density_out(const Chan* chans, int ch, int ny, const float* ws, int src, double* out, hipStream_t s);
hipError_t launch_density_out(const Chan* chans, int ch, int ny, const float* ws, int src, float* out, hipStream_t s);
// The first `have` (>= 1) records of every channel's ring, packed into `out`.
hipError_t launch_pack_ring(const ObsRec* ring, int nchan, int max_samples, int have, ObsRec* out, hipStream_t s);
hipError_t launch_pull_out(const Chan* chans, const RowRef* rows, int nrows, float* ws, int src,
                           hipStream_t s);

}  // namespace scf
