// Several time steps of a D2Q9 box in one launch (two-lattice pattern,
// temporal blocking in LDS).
//
// A workgroup holds an E x E region of nodes, one per work-item, loads the
// stored state of that region once and runs up to H steps on it: each step
// puts the post-collision values into LDS, pulls f_a(x) from x - e_a in LDS
// (Eq. (propagation)) and collides (Eq. (collision), the collide() of the
// one-step kernels).  A node's value after H steps depends only on nodes
// within H links (Chebyshev distance), so the inner (E - 2 H) x (E - 2 H)
// nodes are exact and are the ones stored; the ring around them is
// recomputed by the neighbouring workgroups, which replaces a grid-wide
// barrier by redundant arithmetic.  Region nodes take their coordinates
// modulo the box, so boxes smaller than a region wrap the same way; across
// walls nothing pulls from such an image.  Where a pull source is a wall
// (Eq. (bb)) a node takes its own opposite population, by link bits formed or
// read once per launch.  With a reduced-precision storage every step rounds
// its result through the storage type, as a store and reload would, so the
// state after H steps is bit for bit that of H one-step launches.
//
// Why: a small box is latency-bound with one launch per step (128 x 128
// nodes: 64 workgroups, ~3-4 us per step, most of it one dependent
// load-collide-store chain), and on large boxes a launch reads and writes
// the state once per H steps at the price of the ring's arithmetic, (E / (E -
// 2 H))^2 of the useful collisions, less what the outer nodes leave out: each
// step they skip as soon as nothing stored depends on them, whole wavefronts
// at a time (128^2 FP64 1.38 -> 1.20 us per step, 256^2 1.79 -> 1.53, 512^2
// around an obstacle 4.43 -> 4.37).  Which E and H: see route_2d().
#pragma once

#include "kernels.hpp"
#include "routes.hpp"

namespace imexlbm {

// Inner (stored) nodes per region edge.
template <int E, int H>
inline constexpr int kFuseInnerOf = E - 2 * H;

// Placement of the workgroups (one per inner block; gx x gy blocks).  With
// tw = 0 the launch is a gx x gy grid.  Otherwise it is one-dimensional and
// XCD-aware: the hardware hands workgroup i to XCD i % 8, and the k-th
// workgroup of an XCD takes block k % (tw*th) of that XCD's (k / (tw*th))-th
// tile of tw x th blocks, so the neighbouring regions whose rings overlap
// are read through the same L2.  Padding workgroups (past the last tile or
// the box) exit at once.
struct FuseMap {
    int gx, gy;        // inner blocks along x and y
    int tw, th;        // blocks per tile (0: plain 2D grid)
    int tiles_x, tiles;
};

__device__ __forceinline__ bool fuse_block(const FuseMap& m, int& bx, int& by)
{
    if (m.tw == 0) {
        bx = int(blockIdx.x);
        by = int(blockIdx.y);
        return true;
    }
    const int id = int(blockIdx.x), per_tile = m.tw * m.th;
    const int k = id >> 3, t = (k / per_tile) * 8 + (id & 7), w = k % per_tile;
    if (t >= m.tiles) return false;
    bx = (t % m.tiles_x) * m.tw + w % m.tw;
    by = (t / m.tiles_x) * m.th + w / m.tw;
    return bx < m.gx && by < m.gy;
}

// The placement of an nx x ny box in blocks of `inner` x `inner` stored
// nodes: tiles of tile x tile blocks (0: plain grid), and the launch grid
// that goes with it.
inline FuseMap fuse_plan(int nx, int ny, int inner, int tile, dim3* grid)
{
    FuseMap m{};
    m.gx = (nx + inner - 1) / inner;
    m.gy = (ny + inner - 1) / inner;
    if (tile <= 0) {
        *grid = dim3(unsigned(m.gx), unsigned(m.gy), 1);
        return m;
    }
    m.tw = tile < m.gx ? tile : m.gx;
    m.th = tile < m.gy ? tile : m.gy;
    m.tiles_x = (m.gx + m.tw - 1) / m.tw;
    m.tiles = m.tiles_x * ((m.gy + m.th - 1) / m.th);
    *grid = dim3(unsigned((m.tiles + 7) / 8) * 8u * unsigned(m.tw * m.th), 1, 1);
    return m;
}

// Link bits of a node: bit a where the pull source x - e_a is a wall, bit 31
// where the node is solid; from the mask where there is one, else what the
// walls across x and those across y give.  Directions are a = 3 (e_x + 1) +
// (e_y + 1).
__device__ __forceinline__ unsigned axis_bits_2d(const Dims& g, int axis, int c)
{
    const int n = axis == 0 ? g.nx : g.ny;
    const Axis3 w = axis3<true>(c, n, g.bc[axis]);
    const unsigned minus = axis == 0 ? 0x007u : 0x049u;  // directions with e = -1, 0, +1
    const unsigned zero = axis == 0 ? 0x038u : 0x092u, plus = axis == 0 ? 0x1C0u : 0x124u;
    return (w.wall[0] ? plus : 0u) | (w.wall[1] ? zero : 0u) | (w.wall[2] ? minus : 0u) |
           (g.bc[axis] == kSolidEnds && (c == 0 || c == n - 1) ? 1u << 31 : 0u);
}

__device__ __forceinline__ unsigned link_bits_2d(const Dims& g, int x, int y)
{
    if (g.links) return g.links[node_index(g, x, y, 0)];
    return axis_bits_2d(g, 0, x) | axis_bits_2d(g, 1, y);
}

// An E x E region with a ring of H nodes, one work-item per node; `steps`
// (1 .. H) is the number of steps of this launch.  After step s of it only
// nodes within steps - s links of the stored block are needed, so the others
// (whole rows, and with them whole wavefronts) skip that step.
template <int E, int H, class S, bool WALLS, bool FORCE, bool COMP, bool NT>
__global__ __launch_bounds__((E * E)) void k_step_ab_fused2d(const S* __restrict__ src, S* __restrict__ dst,
                                                             StepArgs<typename Store<S>::C> p, FuseMap m, int steps)
{
    using C = typename Store<S>::C;
    constexpr int L = 0, Q = Lattice<L>::Q, I = kFuseInnerOf<E, H>;
    static_assert(I >= 1, "region edge must exceed the ring");
    int bx, by;
    if (!fuse_block(m, bx, by)) return;  // uniform over the workgroup
    __shared__ C sh[Q][E][E];
    const Dims& g = p.g;
    const int lx = int(threadIdx.x) % E, ly = int(threadIdx.x) / E;
    const int TS = g.S;
    // Links to the stored block (none inside it).
    const int out_x = max(H - lx, lx - (E - 1 - H)), out_y = max(H - ly, ly - (E - 1 - H));
    const int out = max(out_x, out_y);
    C f[Q];
    unsigned bits = 0;
    if (out <= steps) {
        int gx = (bx * I - H + lx) % g.nx;
        int gy = (by * I - H + ly) % g.ny;
        gx += gx < 0 ? g.nx : 0;
        gy += gy < 0 ? g.ny : 0;
        const unsigned node = unsigned(gx) + unsigned(g.nx) * unsigned(gy);
        static_for<Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            f[a] = Store<S>::load(src[slot<Q>(a, node, TS)]);
        });
        if constexpr (WALLS) bits = link_bits_2d(g, gx, gy);
    }
    for (int left = steps; left > 0; --left) {
        if (out <= left) {
            static_for<Q>([&](auto ac) {
                constexpr int a = decltype(ac)::value;
                sh[a][ly][lx] = f[a];
            });
        }
        __syncthreads();
        const bool needed = out < left;  // then out < H: no pull leaves the region
        if (needed) {
            static_for<Q>([&](auto ac) {
                constexpr int a = decltype(ac)::value;
                constexpr int ex = kLattice<L>.e[a][0], ey = kLattice<L>.e[a][1];
                f[a] = sh[a][ly - ey][lx - ex];
                if constexpr (WALLS) {  // from a wall: the node's own opposite population
                    if ((bits >> a) & 1u) f[a] = sh[Lattice<L>::opp(a)][ly][lx];
                }
            });
        }
        __syncthreads();
        if (needed) {
            if constexpr (WALLS) {
                if (g.nodal >= 0)
                    nodal_fill<L>(g, wrap_into(bx * I - H + lx, g.nx), wrap_into(by * I - H + ly, g.ny), 0, f);
            }
            collide<L, C, FORCE, COMP, Store<S>::kDeviation>(f, p.c);
            if constexpr (!std::is_same_v<S, C>) {
                static_for<Q>([&](auto ac) {
                    constexpr int a = decltype(ac)::value;
                    f[a] = Store<S>::load(Store<S>::save(f[a]));
                });
            }
        }
    }
    const int ix = lx - H, iy = ly - H;
    if (out > 0) return;
    const int ox = bx * I + ix, oy = by * I + iy;
    if (ox >= g.nx || oy >= g.ny) return;
    if (WALLS && (bits >> 31)) return;
    const unsigned own = unsigned(ox) + unsigned(g.nx) * unsigned(oy);
    // Non-temporal global stores: the nt | sc1 buffer stores of the
    // one-step kernels measured slower here (four steps per launch on 16 x 16
    // regions, 128^2: 11,950 vs 12,500-13,300 MLUPS; on 32 x 32, 4096^2: 83,900
    // vs 89,600-91,000), the written state being read again, largely from
    // cache, by the next launch.
    static_for<Q>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        put<NT>(dst + slot<Q>(a, own, TS), Store<S>::save(f[a]));
    });
}

}  // namespace imexlbm
