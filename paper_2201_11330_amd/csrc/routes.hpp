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

// What a node costs the one-step kernels, in units of its bytes at 6.3 TB/s
// (medians over 2,500 boxes).  Rows of whole cache lines: 1.0, and above 256
// nodes, where a row takes several workgroups, more the longer the padding of
// the last one (272 nodes, 512 lanes: FP64 1.27, FP32 1.6).  Other rows: FP64
// 1.4-1.5 up to 256 nodes and 1.4-1.8 above, FP32 1.6-1.9 and 1.85-2.05; rows of
// half lines FP64 1.04, FP32 1.1 and up to 1.5.
inline double one_step_cost(int nx, size_t storage_bytes)
{
    int lanes = 1;
    while (lanes < nx && lanes < 256) lanes *= 2;
    const double pad = double((nx + lanes - 1) / lanes) * lanes / nx - 1.0;
    const bool wide = nx > 256;
    if (storage_bytes == 8) {
        if (nx % 8 == 0) return (nx % 16 == 0 ? 1.0 : 1.06) + (wide ? 0.3 * pad : 0.0);
        return 1.38 + (wide ? 0.4 : 0.12) * pad;
    }
    if (nx % 32 == 0) return 1.0 + (wide ? 0.65 : 0.05) * pad;
    if (nx % 16 == 0) return 1.1 + (wide ? 0.5 : 0.05) * pad;
    return 1.6 + (wide ? 0.25 + 0.15 * pad : 0.0);
}

// Estimated time of two one-step launches over that of a two-step launch with
// `slots` workgroups at once, each in units of a row of 64 nodes.
//   * One step: the fluid nodes (solid end planes are skipped) and about 4 us
//     of launch.
//   * Two steps: every workgroup slot makes planes + 3 iterations per round,
//     an iteration costs its stored rows and what does not depend on their
//     number (level 1 next to the tile, barriers, link bits between walls).
//     FP64 D3Q19, us per iteration at 2, 4, 8 and 13 rows: periodic 2.8, 3.9,
//     6.8, 10.4; between solid end planes 4.2, 5.4, 8.1, 11.6.
inline double march_gain(const MarchBox& b, const MarchPlan& p, long long slots)
{
    const double bytes = 2.0 * (b.lattice == 1 ? 19 : 27) * double(b.storage_bytes);
    double nodes = double(b.n[0]) * b.n[1] * b.n[2] * one_step_cost(b.n[0], b.storage_bytes);
    for (int d = 0; d < 3; ++d)
        if (b.bc[d] == 1) nodes *= double(b.n[d] - 2) / b.n[d];
    const double one = nodes / 64 + 4e-6 * 6.3e12 / (64 * bytes);
    const MarchWallKind kind = march_wall_kind(b);
    const int fixed = kind == kMarchNoWalls ? 4 : kind == kMarchSolids ? 2 : b.comp ? 14 : 10;
    const long long groups = (long long)p.tiles_x * p.tiles_y * ((b.n[2] + p.planes - 1) / p.planes);
    const double rounds = double((groups + slots - 1) / slots);
    return 2.0 * one / (double(slots) * rounds * (p.planes + 3) * (p.rows + fixed));
}

// The least march_gain with which two-step launches are taken: per kind of
// walls and model the smallest value above which few of 9,800 boxes (edges of
// 24-700 nodes, a few rows or planes among them) ran below x0.95 of one-step
// launches (30 of them, 619 with two steps for all).  On 3,000 other boxes of
// random edges the rule gains x1.328 in the mean, two steps for all x1.322, the
// faster launch of each box x1.331.  Where it refuses, two-step launches took
// up to 2.7 times as long (us per step: 512 x 3 x 512 compressible between solid
// end planes 19.2 -> 52.0, 512 x 512 x 4 between solid end planes 29.7 -> 70.3,
// D3Q27 112^3 around a sphere 98.6 -> 121.8, D3Q19 FP32 160^3 around a sphere
// 104.9 -> 126.0).  Columns: D3Q19 FP64, D3Q27 FP64, FP32.  Second rows: the
// compressible model, for which 64 registers (FP32) or 128 between walls do
// not hold what a node keeps.
inline double march_least_gain(const MarchBox& b)
{
    static const double least[4][2][3] = {{{0.46, 0.46, 0.62}, {0.52, 0.58, 0.78}},
                                          {{0.52, 0.60, 0.80}, {0.50, 0.60, 0.74}},
                                          {{0.76, 0.70, 0.84}, {0.70, 0.72, 0.85}},
                                          {{1.04, 1.16, 1.26}, {1.06, 1.26, 1.30}}};
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

// ---------------------------------------------------------------------------
// Several steps per launch of a D2Q9 box: regions in LDS (fused2d.hpp), and
// strips streamed up the rows of large boxes (stream2d.hpp).

constexpr int kFuseSteps = 4;  // steps that every region can take in a launch

inline long long fuse_blocks(int nx, int ny, int inner)
{
    return (long long)((nx + inner - 1) / inner) * ((ny + inner - 1) / inner);
}

// Regions of a box, E x E nodes with a ring of H.
enum FuseRegions { kRegions24x8, kRegions32x8, kRegions32x6, kRegions32x4 };

// Choice of region and placement, measured on MI355X on boxes from 64^2 to
// 3000 x 2000 (us per step; before: four steps per launch on 16 x 16 regions,
// from 256 blocks up on 32 x 32 regions of four nodes per work-item):
//  * 24 x 24 regions with eight steps where their 8 x 8 blocks are at most one
//    per CU: FP64 128^2 1.47 -> 1.20, FP32 1.33 -> 1.00, FP16 1.27 -> 0.96.
//  * 32 x 32 regions have 1024 work-items and, in FP64, 72 KB of LDS: two fit a
//    CU, 32 wavefronts.  With eight steps the launches of boxes of up to 288
//    blocks pay their latency half as often: FP64 170^2 1.92 -> 1.43, 256^2
//    2.05 -> 1.52, 512 x 128 around a cylinder 2.37 -> 1.74; FP32 256^2 1.78 ->
//    1.24.  On larger boxes the ring of eight is too much arithmetic (300^2,
//    361 blocks, 2.10, 384^2 2.76, between walls 2.63 and 3.56) and six steps
//    are better: 2.49 -> 1.77, 3.19 -> 2.50, 3.29 -> 2.10, 3.77 -> 3.10; 1000 x
//    777 10.5 -> 8.3; then four: 1024^2 13.4 -> 11.3 (FP16 10.8 -> 6.8), 900 x
//    800 between walls 9.6 (six steps: 9.8).
// XCD-aware tiles of 4 x 4 blocks (fewer where the box has fewer) for rings of
// eight and six up to 512 blocks: 256^2 2.04 -> 1.78, 300^2 2.43 -> 2.03; but
// 512^2, 676 blocks, 4.1 -> 4.7: the padding to whole tiles.  Padding a column
// of blocks to tiles of four left three quarters of the workgroups empty and
// the others on a quarter of the CUs: 1 x 4096 FP64 24.6 us for eight steps,
// now 10.0; 4096 x 16 between walls 18.3, now 12.7.
constexpr int kFuseTile = 4;
constexpr int kFuseXcdMaxBlocks = 512;

inline FuseRegions fuse_regions(int nx, int ny, bool walls)
{
    if (fuse_blocks(nx, ny, 8) <= 256) return kRegions24x8;
    if (fuse_blocks(nx, ny, 16) <= 288) return kRegions32x8;
    return fuse_blocks(nx, ny, 20) <= (walls ? 1280 : 2000) ? kRegions32x6 : kRegions32x4;
}

// Steps per launch.
inline int fuse_levels(FuseRegions r)
{
    return r == kRegions24x8 || r == kRegions32x8 ? 8 : r == kRegions32x6 ? 6 : 4;
}

constexpr int kStreamCols = 256;  // columns per workgroup, one per work-item
constexpr int kStreamHalo = 16;   // loaded columns on each side of the stored ones
constexpr int kStreamStore = kStreamCols - 2 * kStreamHalo;  // 224 stored columns
// Smaller boxes take the regions of fused2d.hpp.  us per step, strips against
// regions: FP64 1024^2 14.7 / 11.4, 1500 x 1100 17.4 / 17.3, 2048 x 1024 20.5 /
// 21.7, 2048^2 32.8 / 42.7; FP32 1024^2 8.4 / 7.6, 2048 x 1024 12.6 / 13.3;
// FP16 1500^2 16.0 / 12.8, 2048^2 23.5 / 23.8.  Between walls (FP64: 218
// registers instead of 138, two wavefronts per SIMD instead of three) FP64
// 1500^2 26.3 / 25.5, 2048^2 45.0 / 46.2, FP32 2048^2 27.5 / 31.3.
constexpr unsigned kStreamMinNodes = 1u << 21;
constexpr unsigned kStreamMinNodes16 = 1u << 22;     // 16-bit storage
constexpr unsigned kStreamMinNodesWalls = 3u << 20;  // between walls

// Steps per launch of a box (0: it does not take strips).  Eight steps read
// and write the state half as often as four, but hold twice the registers
// (FP64: 234 instead of 138, two wavefronts per SIMD instead of three) and
// repeat 16 rows per segment instead of 8.  us per step, four against eight:
// FP64 1500 x 1100 17.7 / 18.0, 2048^2 35.2 / 32.9, 4096^2 120.9 / 101.9;
// FP32 2048^2 20.0 / 19.8, 4096^2 67.0 / 53.6; FP16 (bound by instructions)
// 4096^2 72.8 / 74.8.  Between walls 256 registers would not hold eight.
inline int stream_levels(unsigned nodes, size_t storage_bytes, bool walls)
{
    if (nodes < (walls ? kStreamMinNodesWalls : storage_bytes == 2 ? kStreamMinNodes16 : kStreamMinNodes)) return 0;
    if (walls || storage_bytes == 2) return 4;
    return nodes >= (storage_bytes == 8 ? 1u << 22 : 1u << 23) ? 8 : 4;
}

// A box as the rule sees it; storage as in lbm_storage.
struct Box2D {
    int nx, ny;
    int storage;       // 0 FP64, 1 FP32, 2 FP16, 3 BF16, 4 e4m11
    bool walls, mask;  // walls: on an axis or of a mask
    bool comp;         // compressible equilibrium
};

struct Route2D {
    int strips;           // steps per launch of strips (0: regions only)
    FuseRegions regions;  // for the other launches
    int most, fewest;     // steps per launch (most 0: one-step launches only)
    bool fours;           // six-step regions: up to four steps on regions of four
};

// Measured on boxes from 16^2 to 2900^2, 4096 x 1 .. 1024, 1 .. 32 x 4096, 65000 x
// 3 and x 16, in five storages, periodic, between walls and with masks,
// against one-step launches (us per step, one-step / several).
//  * At most one block per CU (regions of eight steps, and of six in long
//    boxes): two steps and more in one launch are never slower, mostly 1.3-3.5
//    times faster.
//  * Larger boxes of which the blocks store less than half (65000 x 3 between
//    walls: 576-node blocks with 72 stored nodes): FP64 7.8 / 11.5, FP16 4.1 /
//    14.5: one step.
//  * 16-bit storage: the conversions of each step weigh more, and short
//    launches do not pay (FP16 two steps: 512^2 between walls 5.3 / 6.0, 2048^2
//    27.0 / 39.4): six-step regions from three steps up (1.05-1.5), other
//    launches from four, or three where rows of partial cache lines slow the
//    one-step kernels.  Between walls on the axes strips lost (2048^2 30.4 /
//    34.8), and with the compressible model regions of four where rows are
//    whole lines (1024^2 10.6 / 11.4; 42 boxes of other rows gained 1.15 in the
//    mean).
//  * e4m11: a conversion costs as much as a third of a collision.  Only whole
//    launches pay: six-step regions of the incompressible model (512^2 5.4 /
//    4.5, 700^2 8.4 / 6.9; between walls up to 512 blocks, 384^2 4.5 / 3.6,
//    512^2 4.9 / 4.9), around obstacles also of the compressible one and regions
//    of four where rows are partial lines (1.1-1.4); and strips of rows that the
//    row-addressed one-step kernel does not take (2900^2 88.8 / 76.5, but
//    2048^2 26.8 / 47.2), or from 2^23 nodes up around obstacles (2900^2 102.8 /
//    86.0, 2048^2 43.4 / 50.8).  Other regions of four: 1024^2 9.0 / 12.1, 1448^2
//    22.2 / 21.9, between walls 22.7 / 24.8.
//  * Regions of four that store less than three quarters (16 x 65000, 65000 x
//    16): compressible between walls FP16 11.3 / 15.1 and FP32 two steps alone
//    17.1 / 20.1; e4m11 around obstacles 14.5 / 17.4; the others 1.0-2.6 times
//    faster.
//  * FP32 rows of whole cache lines with the compressible model between walls or
//    in strips: two steps alone lost (512^2 6.8 / 7.1, 4096 x 1024 49.6 / 52.5).
inline Route2D route_2d(const Box2D& b)
{
    const unsigned nodes = unsigned(b.nx) * unsigned(b.ny);
    const size_t bytes = b.storage == 0 ? 8 : b.storage == 1 ? 4 : 2;
    Route2D r;
    r.regions = fuse_regions(b.nx, b.ny, b.walls);
    r.strips = stream_levels(nodes, bytes, b.walls);
    r.most = r.strips ? r.strips : fuse_levels(r.regions);
    r.fewest = 2;
    r.fours = false;
    if (r.regions == kRegions24x8 || r.regions == kRegions32x8) return r;
    const Route2D one_step = {0, r.regions, 0, 0, false};
    const bool six = r.regions == kRegions32x6 && !r.strips, axes_only = b.walls && !b.mask;
    const int inner = r.regions == kRegions32x6 ? 20 : 24;
    const long long blocks = fuse_blocks(b.nx, b.ny, inner);
    r.fours = six && !b.walls;
    if (six && blocks <= 256) return r;
    if (!r.strips && 2ll * nodes < blocks * inner * inner) return one_step;
    const bool thin = !r.strips && !six && 4ll * nodes < 3ll * blocks * inner * inner;
    if (b.storage == 4) {
        const bool row_addressed = !b.walls && b.nx >= 64 && b.nx <= 4096 && (b.nx & (b.nx - 1)) == 0;
        bool take;
        if (r.strips) take = !b.walls ? !row_addressed && !b.comp : b.mask && !b.comp && nodes >= 1u << 23;
        else if (six) take = b.mask ? !b.comp || b.nx % 32 != 0 : !b.comp && (!b.walls || blocks <= 512);
        else take = b.mask && !b.comp && b.nx % 64 != 0 && !thin;
        if (!take) return one_step;
        r.fewest = r.most;
    } else if (bytes == 2) {
        if (axes_only && (r.strips || (b.comp && !six && (thin || b.nx % 64 == 0)))) return one_step;
        r.fewest = (six || b.nx % 64 != 0) && !(axes_only && b.comp) ? 3 : 4;
    } else if (b.storage == 1 && ((b.nx % 32 == 0 && ((b.walls && b.comp) || r.strips)) ||
                                  (thin && axes_only && b.comp))) {
        r.fewest = 3;
    }
    return r;
}

// Steps of the next launch when `left` are to be made (0: one-step launches
// from here on).  Of eight steps a periodic six-step box makes four and four
// instead of six and two (FP64 512^2 40.0 -> 32.0 us, FP32 700^2 45.9 -> 40.4),
// and where the rest after a whole launch would be several one-step launches,
// two equal ones (eight steps in 16-bit storage on 28 six-step boxes, in the mean
// over one-step launches: 6 + 1 + 1 x1.37, 4 + 4 x1.46).
inline int next_launch(const Route2D& r, int left)
{
    if (!r.most || left < r.fewest) return 0;
    if (left < r.most) return r.strips && left > kFuseSteps ? kFuseSteps : left;
    const int rest = left - r.most;
    if (!r.strips && r.regions == kRegions32x6 && r.fewest <= kFuseSteps) {
        if (r.fours && rest == 2) return kFuseSteps;
        if (rest > 1 && rest < r.fewest && left >= 2 * r.fewest) return (left + 1) / 2;
    }
    return r.most;
}

// The regions of a launch of `steps` steps that does not run as strips.  In a
// periodic six-step box up to four steps take the smaller ring (700^2, four
// steps: FP64 28.6 -> 25.4 us, FP32 22.3 -> 18.7, FP16 19.9 -> 19.4).
inline FuseRegions launch_regions(const Route2D& r, int steps)
{
    return r.fours && steps <= kFuseSteps ? kRegions32x4 : r.regions;
}

// Rows per segment for an nx x ny box when the GPU runs `slots` workgroups
// of the kernel at once.  Every workgroup runs rows + 2 H iterations, so a
// launch takes about ceil(workgroups / slots) rounds of that many: the rows
// from 8 to 256 that minimise the product (the fewest among equals).  Long
// segments re-read fewer rows (8 per segment) but leave part of the last
// round idle unless the workgroups fill it.  Measured with four levels at 4096^2 FP64 (19
// strips, 768 slots): 103 rows (760 workgroups, the rule's choice) 135,500-
// 136,700 MLUPS; 64 rows (1216) 130,400-132,300; 52 (1501) 131,900; 86
// (912) 121,400; 120 (665) 128,500.
inline int stream_rows(int nx, int ny, long long slots, int levels)
{
    const long long strips = (nx + kStreamStore - 1) / kStreamStore;
    int best = 8;
    long long best_cost = -1;
    for (int rows = 8; rows <= 256; ++rows) {
        const long long wg = strips * ((ny + rows - 1) / rows);
        const long long cost = (wg + slots - 1) / slots * (rows + 2 * levels);
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost;
            best = rows;
        }
    }
    return best;
}

}  // namespace imexlbm
