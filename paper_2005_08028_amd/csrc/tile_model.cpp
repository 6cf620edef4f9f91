// Untuned choice of the fused 2D denoiser's shape and pass count: an estimate
// of the time of one pass for every shape, from what bounds the kernels on
// this GPU (256 CUs of 4 SIMDs, one vector instruction per SIMD and 4 cycles).
//
// A tiled workgroup spends max(j W, W + L) cycles per iteration when j of them
// share a CU: W = vector instructions of its waves at full rate (17 per pixel
// for ITV2D, 14 for ATV, halo included), L = the latency of the two barriers
// and row exchanges, which other workgroups hide. A row-pipelined wavefront
// spends max(j V, V + LR) cycles per row step when j share a SIMD, V = M levels
// of 2 columns; the register file admits 512 / (20 M + 14) of them. Rounds that
// fill the chip run at full rate, the last one at its own occupancy, and a pass
// takes no less than its bytes at 7.5 TB/s (beyond the 256 MB Infinity Cache
// 5, and 3.2 with duals in and out: ten streams a tile apart).
//
// Measured against every shape and up to three passes on 13 sizes from
// 64x64x8 to 1024x1024x24 and 3 to 14 iterations, cold and with warm duals
// (GAP iterations in a graph, 104 cases): the estimate's choice is within 6 %
// of the best pair in all but 6 (21 % at worst) and 18 % faster on average
// than the rule before it (shape 1 with passes of about 5 iterations, a
// row-pipelined shape for large cold calls).
#include <algorithm>

#include "k_fgp_tile_shapes.h"
#include "sci_internal.h"

namespace sci {
namespace {

constexpr double kClockPerUs = 2400.0;
constexpr double kLaunchUs = 1.8;
constexpr double kTileLatency = 450.0, kTileStart = 2400.0, kTileStartShared = 550.0;
constexpr double kRowLatency = 450.0, kRowStart = 3500.0;
constexpr double kBytesPerCycle = 10.0; // one CU's share of the memory rate

// Workgroups of a tiled shape that fit one CU (threads and registers).
int tile_groups_per_cu(int rows, int waves, int cols)
{
    const int per_lane = rows * cols; // pixels of a lane; about 10 registers each
    if (cols > 1 || per_lane > 5) return waves <= 8 && cols == 1 ? 2 : 1;
    return 32 / waves;
}

} // namespace

// Tiles (or row segments) of one frame for shape and pass length m; 0 when the
// pass does not fit the shape.
long tile_units(int shape, int m, int nx, int ny)
{
    int r = 0, w = 0, c = 0;
    if (!tile_shape_info(shape, &r, &w, &c)) return 0;
    const long tx = 64L * c - 2 * m - 1;
    const long ty = tile_shape_pipelined(shape) ? r : (long)w * r - 2 * m - 1;
    if (tx <= 0 || ty <= 0) return 0;
    return ((ny + tx - 1) / tx) * ((nx + ty - 1) / ty);
}

// Estimated microseconds of one pass of m iterations over `units` tiles (row
// segments) holding `voxels`, moving `io` float32 fields per voxel.
double tile_pass_us(int num_cus, int tv, int shape, int m, long units, double voxels, int io)
{
    int r = 0, w = 0, c = 0;
    if (units <= 0 || !tile_shape_info(shape, &r, &w, &c)) return 1e30;
    const double ops = tv == SCI_TV_ATV ? 14.0 : 17.0;
    const long cus = num_cus > 0 ? num_cus : 256;
    double cyc = 0.0;
    if (!tile_shape_pipelined(shape)) {
        const int k = tile_groups_per_cu(r, w, c);
        // five rows per lane leave no registers to spare at two groups per CU
        const double W = (double)r * c * w * ops, shared = k == 2 && r == 5 ? 1.2 : 1.0;
        // x and theta; the dual fields' loads overlap better (measured: +6 us of
        // 52 at 512x512x16 with four in and four out on shape 1, +20 of 44 on
        // shape 7, whose groups have a CU each)
        const double field = (double)r * c * w * 64 * 4 / kBytesPerCycle;
        auto move = [&](double two, double more) { return field * (2 * two + (io - 2) * more); };
        auto iteration = [&](long j) { return std::max(j * W * (j > 1 ? shared : 1.0), W + kTileLatency); };
        const long full = units / (k * cus), rem = units % (k * cus);
        cyc += full * (m * iteration(k) + (k > 1 ? k * kTileStartShared : kTileStart) + k * (k > 1 ? move(0.35, 0.15) : move(1.0, 0.85)));
        if (rem) {
            const long j = (rem + cus - 1) / cus;
            cyc += m * iteration(j) + kTileStart + 300 * (j - 1) + j * (j > 1 ? move(0.6, 0.3) : move(1.0, 0.85));
        }
    } else {
        const long simds = 4 * cus, k = std::min(8, 512 / (20 * m + 14));
        const double V = 8.0 * m * ops + 60 + 30 * io, steps = r + m + 2;
        const long full = units / (k * simds), rem = units % (k * simds);
        cyc += full * steps * k * V * (k > 2 ? 0.85 : 1.0) + kRowStart;
        if (rem) {
            const long j = (rem + simds - 1) / simds;
            cyc += steps * std::max(j * V * (j > 2 ? 0.85 : 1.0), V + kRowLatency + (j > 1 && j < k ? 0.2 * j * V : 0.0));
        }
    }
    const double bytes = 4.0 * io * voxels;
    return std::max(cyc / kClockPerUs + kLaunchUs, bytes / (bytes < 2.2e8 ? 7.5e6 : io > 4 ? 3.2e6 : 5.0e6) + 2.0);
}

// The shape, or the two shapes of which every launch takes the cheaper, with the
// smallest total of launches[c] * cost[shape * nc + c]. Returns their number: 2
// only where the second one lowers the total of the best single shape.
int pick_shape_pair(int ns, int nc, const double *cost, const double *launches, int shape[2])
{
    double best = -1.0;
    int found = 0;
    for (int gap = 0; gap < ns; ++gap) // single shapes first
        for (int a = 0; a + gap < ns; ++a) {
            const double *ca = cost + (size_t)a * nc, *cb = cost + (size_t)(a + gap) * nc;
            double t = 0.0;
            for (int c = 0; c < nc; ++c) t += launches[c] * std::min(ca[c], cb[c]);
            if (best >= 0.0 && t >= best) continue;
            best = t;
            shape[0] = a;
            shape[1] = a + gap;
            found = gap ? 2 : 1;
        }
    return found;
}

} // namespace sci
