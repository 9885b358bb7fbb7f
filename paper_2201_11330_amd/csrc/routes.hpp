// Which boxes take launches of several time steps, and how their work is
// split: rules on sizes, types and boundaries, decided by measurement.  Plain
// host code without HIP.
#pragma once

#include <cstddef>

namespace imexlbm {

// ---------------------------------------------------------------------------
// Two steps per launch through the planes of a 3D box (march3d.hpp).

constexpr int kMarchCols = 64;  // stored columns per workgroup, one per lane

// Wavefronts per workgroup: one per row of level 1 and one for the two edge
// columns; 16, or as many as LDS holds rows for.
constexpr int march_waves(int lattice) { return lattice == 2 ? 12 : 16; }
constexpr int march_rows(int lattice) { return march_waves(lattice) - 3; }  // stored rows of a tile at most

// Workgroups per CU that the registers are shared out for: LDS holds one
// with FP64 and two with FP32.
constexpr int march_per_cu(size_t storage_bytes) { return storage_bytes == 8 ? 1 : 2; }

// Largest plane: the byte offset of a population in a plane fits 32 bits and
// the tile number in a plane 24.
constexpr unsigned kMarchMaxPlane = 1u << 24;

// Planes per segment when `cols` columns of tiles cover a plane and the GPU
// runs `slots` workgroups at once: a launch takes about ceil(workgroups /
// slots) rounds of planes + 2 iterations and the start of the pipeline, so
// the planes that minimise the product (the fewest among equals).
// 256^3 FP64 (80 columns, 256 slots): 86 planes, 240 workgroups, 467 us.
inline int march_planes(int nz, long long cols, long long slots)
{
    int best = 1;
    long long best_cost = -1;
    for (int planes = 1; planes <= nz; ++planes) {
        const long long wg = cols * ((nz + planes - 1) / planes);
        const long long cost = (wg + slots - 1) / slots * (planes + 3);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = planes;
        }
    }
    return best;
}

// A box as the rule sees it.  bc: 0 periodic, 1 solid end planes, 2 walls
// outside, 3 nodal walls.
struct MarchBox {
    int lattice;           // 1 D3Q19, 2 D3Q27
    size_t storage_bytes;  // 8 FP64, 4 FP32
    int n[3];              // nx, ny, nz
    int bc[3];
    bool mask;             // solid mask
    bool comp;             // compressible equilibrium
};

struct MarchPlan {
    int tiles_x, tiles_y;  // tiles of kMarchCols columns and `rows` rows
    int rows;              // stored rows per tile
    int planes;            // stored planes per segment
};

// The tiles of a plane, with segments of `planes`.
inline MarchPlan march_plan(const MarchBox& b, int planes)
{
    const int most = march_rows(b.lattice);
    MarchPlan p;
    p.tiles_x = (b.n[0] + kMarchCols - 1) / kMarchCols;
    p.tiles_y = (b.n[1] + most - 1) / most;
    p.rows = (b.n[1] + p.tiles_y - 1) / p.tiles_y;
    p.planes = planes;
    return p;
}

// What bounds the launches by walls: nothing; walls on y or z; walls on x,
// next to which every wavefront lies; a solid mask.
enum MarchWallKind { kMarchNoWalls, kMarchWallsYZ, kMarchWallsX, kMarchSolids };

inline MarchWallKind march_wall_kind(const MarchBox& b)
{
    if (b.mask) return kMarchSolids;
    if (b.bc[0] != 0) return kMarchWallsX;
    return b.bc[1] != 0 || b.bc[2] != 0 ? kMarchWallsYZ : kMarchNoWalls;
}

// Estimated time of two one-step launches over that of a two-step launch with
// `slots` workgroups at once, each in units of a row of 64 nodes.
//   * One step: the fluid nodes (solid end planes are skipped) and about 4 us
//     of launch at the 6.3 TB/s of those kernels.  Rows that are not whole
//     cache lines cost 1.2-1.9 x as much there, the more the longer the
//     padding of their lanes (FP64, ps per node: 128 x 128 x 128 49,
//     100^3 58, 193 x 127 x 101 67, 257 x 100 x 100 83).
//   * Two steps: every workgroup slot makes planes + 3 iterations per round,
//     an iteration costs its stored rows and what does not depend on their
//     number (level 1 next to the tile, barriers, link bits between walls).
//     FP64 D3Q19, us per iteration at 2, 4, 8 and 13 rows: periodic 2.8, 3.9,
//     6.8, 10.4; between solid end planes 4.2, 5.4, 8.1, 11.6.
inline double march_gain(const MarchBox& b, const MarchPlan& p, long long slots)
{
    const double bytes = 2.0 * (b.lattice == 1 ? 19 : 27) * double(b.storage_bytes);
    double nodes = double(b.n[0]) * b.n[1] * b.n[2];
    for (int d = 0; d < 3; ++d)
        if (b.bc[d] == 1) nodes *= double(b.n[d] - 2) / b.n[d];
    int lanes = 1;
    while (lanes < b.n[0] && lanes < 256) lanes *= 2;
    const double padded = double((b.n[0] + lanes - 1) / lanes) * lanes / b.n[0];
    if (size_t(b.n[0]) * b.storage_bytes % 128 != 0) nodes *= 1.1 + 0.25 * (padded - 1.0);
    const double one = nodes / 64 + 4e-6 * 6.3e12 / (64 * bytes);
    const MarchWallKind kind = march_wall_kind(b);
    const int fixed = kind == kMarchNoWalls ? 6 : kind == kMarchSolids ? 4 : 11;
    const long long groups = (long long)p.tiles_x * p.tiles_y * ((b.n[2] + p.planes - 1) / p.planes);
    const double rounds = double((groups + slots - 1) / slots);
    return 2.0 * one / (double(slots) * rounds * (p.planes + 3) * (p.rows + fixed));
}

// The least march_gain with which two-step launches are taken: per kind of
// walls and model the smallest value above which at most a handful of about
// 5,500 boxes (edges of 24-700 nodes, a few rows or planes among them) ran
// below x0.96 of one-step launches.  On 3,200 other random boxes of edges
// 16-512 none is slower than one-step launches by more than 5 % and the rule
// gains x1.16 in the mean, with two steps for all x1.17 and 128 of them slower
// than that, the faster launch of each box x1.18.  Where it refuses, two-step
// launches took up to 2.7 times as long (us per step: 512 x 3 x 512
// compressible between solid end planes 19.2 -> 52.0, 512 x 512 x 4 between
// solid end planes 29.7 -> 70.3, D3Q27 112^3 around a sphere 98.6 -> 121.8,
// D3Q19 FP32 160^3 around a sphere 104.9 -> 126.0).  Columns: D3Q19 FP64,
// D3Q27 FP64, FP32.  Second rows: the compressible model, for which 64
// registers (FP32) or 128 between walls do not hold what a node keeps.
inline double march_least_gain(const MarchBox& b)
{
    static const double least[4][2][3] = {{{0.44, 0.44, 0.62}, {0.50, 0.50, 0.70}},
                                          {{0.52, 0.60, 0.80}, {0.57, 0.64, 0.84}},
                                          {{0.65, 0.65, 0.85}, {0.65, 0.65, 0.90}},
                                          {{0.97, 1.08, 1.15}, {1.00, 1.15, 1.30}}};
    return least[march_wall_kind(b)][b.comp][b.storage_bytes == 4 ? 2 : b.lattice - 1];
}

// Planes per segment of the two-step launches of a box on a GPU of `cus` CUs,
// or -1 where it takes one-step launches.  Besides march_least_gain: rows
// padded to more lanes than in the one-step kernels (nx <= 32), boxes of
// fewer than 4 planes and small boxes (FP64 below 2^18 nodes; between walls
// 2^19, D3Q27 2^20; FP32 5 * 2^17 and 2^21, D3Q27 between walls not at all)
// lost.
inline int march_route(const MarchBox& b, int cus)
{
    const unsigned long long plane = (unsigned long long)b.n[0] * b.n[1], nodes = plane * b.n[2];
    if (b.n[0] <= 32 || b.n[2] < 4 || plane > kMarchMaxPlane) return -1;
    const bool walls = march_wall_kind(b) != kMarchNoWalls;
    if (b.storage_bytes == 8) {
        if (nodes < (!walls ? 1u << 18 : b.lattice == 1 ? 1u << 19 : 1u << 20)) return -1;
    } else {
        if (walls ? b.lattice == 2 || nodes < 1u << 21 : nodes < 5u << 17) return -1;
    }
    const long long slots = (long long)march_per_cu(b.storage_bytes) * cus;
    MarchPlan p = march_plan(b, 0);
    p.planes = march_planes(b.n[2], (long long)p.tiles_x * p.tiles_y, slots);
    return march_gain(b, p, slots) >= march_least_gain(b) ? p.planes : -1;
}

}  // namespace imexlbm
