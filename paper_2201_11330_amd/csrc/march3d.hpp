// Two time steps of a D3Q19 or D3Q27 box in one pass over the state
// (two-lattice pattern, FP64 and FP32 storage), marching up the planes of a
// column of tiles.
//
// A workgroup owns a tile of 64 columns x up to R - 2 rows of stored nodes
// and a segment of planes.  It walks up the planes once.  In iteration q it
// pulls the stored state (the post-collision state of the previous launch)
// of plane q and collides it ("level 1", the first step) on the tile and one
// node around it, and then pulls and collides level 1 in plane q - 1 ("level
// 2", the second step) on the tile and stores it.  The work-items:
//   * one wavefront per row of level 1 (rows 0 .. R - 1, stored rows
//     1 .. R - 2), one lane per column, so a wavefront's loads and stores are
//     64 consecutive nodes (which start on a cache line where nx is a multiple
//     of 16 in FP64 or of 32 in FP32, and touch one line more elsewhere);
//   * one wavefront for the two columns next to the tile (level 1 only).
// Level 2 needs level 1 of plane q - 1 from three planes: e_z = -1 from
// plane q, e_z = 0 from plane q - 1, e_z = +1 from plane q - 2.  Only the
// plane just made is in LDS (all Q directions of the tile and its ring:
// 150,480 bytes for D3Q19 FP64); as soon as it is there a work-item takes
// from it, moved along x and y (Eq. (propagation)), the e_z = 0 and e_z = +1
// populations that its own node pulls in the next two iterations, and keeps
// them in registers.  The loads of plane q + 1 are issued before level 2 of
// plane q - 1 and arrive while it runs.
//
// Which boxes take it: march_route().  What bounds it: HBM.  A launch must
// read and write the state once for two steps, half the bytes of the one-step
// kernels.  D3Q19 FP64 256^3 (rocprofv3 FETCH_SIZE and WRITE_SIZE, GB per
// launch): 2.83 read (2.55 stored, the rest are the rings, mostly served by
// the L2 of the XCD), 2.55 written.  512 x 128 x 128 with a force between
// walls moves 5.0 TB/s against these 5.8, with 1.6 times the vector
// instructions per node.
// Measured on one MI355X, us per step against the one-step kernels, periodic:
// D3Q19 FP64 256^3 806 -> 467 (36,000 MLUPS), 512 x 128 x 128 405 -> 241,
// 193 x 127 x 101 170 -> 117; FP32 256^3 407 -> 275; D3Q27 FP64 192^3
// 498 -> 320.  512 x 128 x 128 with a force: D3Q19 FP64 between solid end
// planes 405 -> 272, D3Q27 around a sphere 580 -> 415.
//
// Why this split: level 1 is made twice where tiles meet, (R / (R - 2)) x
// (66 / 64) of the work, and the stored state is read (R + 2) / (R - 2)
// times in y; 16 wavefronts are the most a workgroup can have, and 64 x 13
// stored nodes per workgroup (64 x 9 for D3Q27 FP64, 12 wavefronts) the most
// that LDS holds.  Without walls everything a work-item keeps stays in its
// 128 (D3Q27: 168, FP32: 64, 80) registers, but for two or three of the D3Q27
// FP32 forms with a force.  With walls what walls above return waits in memory
// (below), and up to 20 registers are spilled all the same (D3Q27 FP64
// compressible with nodal walls; D3Q19 FP64 at most 6, FP32 at most 9).  Two
// rows per work-item (FP32: 64 x 28 tiles, one workgroup per CU instead of
// two) ran 285 instead of 273 us per step at 256^3, and issuing a quarter of
// the loads before level 1 was 10 % slower.
// 16-bit storage does not take this path: FP16 256^3 went from 197 to 243 us.
// That form, held to the 64 registers of two workgroups per CU, issued 17.1 M
// vector memory instructions per launch where the FP32 form issues 11.6 M
// (LDS instructions: 11.59 M in both), for the same loads and stores of the
// state; the rest is most likely registers spilled to memory.
//
// The arithmetic per node and step is that of the one-step kernels, in the
// same order, so the state after two steps is bit for bit that of two
// one-step launches.
#pragma once

#include "kernels.hpp"
#include "routes.hpp"

namespace imexlbm {

// What stops a population on its way: nothing (periodic box), walls on the
// axes, walls of a solid mask (link bits), or walls on the axes or of a mask
// with a nodal-wall axis among them.
enum MarchWalls : int { kMarchOpen = 0, kMarchAxes = 1, kMarchMask = 2, kMarchNodal = 3 };

template <int L>
inline constexpr int kMarchWaves = march_waves(L);
template <int L>
inline constexpr int kMarchThreads = kMarchWaves<L> * 64;
template <int L, class S>
inline constexpr int kMarchWavesPerSimd = kMarchWaves<L> * march_per_cu(sizeof(S)) / 4;

struct MarchMap {
    MarchPlan p;
    int total, chunk;      // workgroups, and how many of them each XCD gets
};

template <int L>
struct MarchDirs {
    static constexpr int Q = Lattice<L>::Q;
    // Place of direction a among those with its e_z, and their number.
    static constexpr int rank(int a)
    {
        int n = 0;
        for (int b = 0; b < a; ++b) n += kLattice<L>.e[b][2] == kLattice<L>.e[a][2];
        return n;
    }
    static constexpr int count(int ez)
    {
        int n = 0;
        for (int b = 0; b < Q; ++b) n += kLattice<L>.e[b][2] == ez;
        return n;
    }
};

// Buffer resource over `bytes` bytes from p (accesses past them read 0 and
// write nothing), and loads and stores through it at byte offset voff (per
// lane) + soff (wave-uniform).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_at(const char* p, size_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(p), 0,
                                             bytes > 0xFFFFFFFFull ? 0xFFFFFFFFu : unsigned(bytes), 0x00020000);
}

template <class S>
__device__ __forceinline__ S buffer_get(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff)
{
    if constexpr (sizeof(S) == 8) return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b64(rs, voff, soff, 0));
    else return __builtin_bit_cast(S, __builtin_amdgcn_raw_buffer_load_b32(rs, voff, soff, 0));
}

template <int AUX, class S>
__device__ __forceinline__ void buffer_put(__amdgpu_buffer_rsrc_t rs, unsigned voff, unsigned soff, S v)
{
    typedef unsigned U32x2 __attribute__((ext_vector_type(2)));
    if constexpr (sizeof(S) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U32x2, v), rs, voff, soff, AUX);
    else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rs, voff, soff, AUX);
}

// The collision arguments with the force hidden from the optimiser, so that
// what is the same in every plane (sums e_a.F) is formed where it is used
// and not kept in registers through the march.
template <bool FORCE, class C>
__device__ __forceinline__ CollideArgs<C> plane_args(const CollideArgs<C>& c)
{
    CollideArgs<C> r = c;
    if constexpr (FORCE) asm volatile("" : "+s"(r.F[0]), "+s"(r.F[1]), "+s"(r.F[2]));
    return r;
}

template <int L, class S, int WK, bool FORCE, bool COMP>
__global__ __launch_bounds__((kMarchThreads<L>)) __attribute__((amdgpu_waves_per_eu((kMarchWavesPerSimd<L, S>)))) void
k_step_ab_march(const S* __restrict__ src, S* __restrict__ dst, StepArgs<S> p, MarchMap m)
{
    static_assert(std::is_same_v<S, typename Store<S>::C>, "storage types that are computed in");
    using D = MarchDirs<L>;
    constexpr int Q = Lattice<L>::Q, R = kMarchWaves<L> - 1;  // rows of level 1
    constexpr int W = kMarchCols + 2;
    constexpr int N0 = D::count(0), N1 = D::count(1);
    constexpr unsigned B = sizeof(S);
    constexpr bool WALLS = WK != kMarchOpen;
    // Link bits read from memory are kept for the next planes; those of the
    // axes cost a few scalar operations per plane.
    constexpr bool kCarryBits = WK == kMarchMask || WK == kMarchNodal;
    constexpr unsigned kSolid = 1u << 31;
    __shared__ S sh[Q][R][W];
    const Dims& g = p.g;
    // Workgroup i runs on XCD i mod 8: each XCD gets `chunk` consecutive
    // tiles, whose rings overlap.
    const int k = int(blockIdx.x & 7) * m.chunk + int(blockIdx.x >> 3);
    if (k >= m.total) return;
    const int x0 = (k % m.p.tiles_x) * kMarchCols;
    const int y0 = (k / m.p.tiles_x % m.p.tiles_y) * m.p.rows;
    const int z0 = (k / (m.p.tiles_x * m.p.tiles_y)) * m.p.planes;
    const int z1 = min(z0 + m.p.planes, g.nz);
    const int rows = min(m.p.rows, g.ny - y0);
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), lane = int(threadIdx.x) & 63;
    const bool edge = wave == R;  // lanes 0-31: rows of the column on the left, 32-63: on the right
    const int row = edge ? min(lane & 31, R - 1) : wave;
    const int col = edge ? (lane < 32 ? 0 : W - 1) : lane + 1;
    // Nodes past the end of the box are images of those at its other end: on
    // a periodic axis the ones that are pulled from, else never used.
    const int gx = wrap_into(x0 + col - 1, g.nx), gy = wrap_into(y0 + row - 1, g.ny);
    const bool level1 = edge || row <= rows + 1;
    const bool to_lds = edge ? (lane & 31) < R : level1;
    const bool level2 = !edge && row >= 1 && row <= rows;
    const bool store_x = x0 + col - 1 < g.nx;
    const int TS = g.S;
    const int tile_shift = TS + (B == 8 ? 3 : 2);
    const unsigned run_bytes = B << TS, tile_bytes = unsigned(Q) * run_bytes;
    const unsigned plane = unsigned(g.nx) * unsigned(g.ny), row_bytes = B * unsigned(g.nx);
    const size_t total = size_t((g.N + (1u << TS) - 1) >> TS) * tile_bytes;
    const bool whole_tiles = (plane & ((1u << TS) - 1u)) == 0;

    // Plane z of the state: a resource based at the tile its first node lies
    // in, and the byte position of that node in the tile's runs.
    struct Plane {
        size_t base;
        unsigned at;
    };
    const auto plane_at = [&](int z) -> Plane {
        const unsigned n = plane * unsigned(z);
        return {size_t(n >> TS) * tile_bytes, (n & ((1u << TS) - 1u)) * B};
    };
    // Offset in that resource of byte position i among the nodes of the
    // plane (as if each node took one element).
    const auto offset = [&](unsigned i) -> unsigned {
        return __umul24(i >> tile_shift, tile_bytes) + (i & (run_bytes - 1u));
    };
    const auto up = [&](int z) { return z == g.nz - 1 ? 0 : z + 1; };

    // Link bits of this work-item's node in plane z: bit a where the pull
    // source x - e_a is a wall, bit 31 where the node is solid.
    unsigned bits_xy = 0;
    if constexpr (WALLS) {
        const Axis3 ax = axis3<true>(gx, g.nx, g.bc[0]), ay = axis3<true>(gy, g.ny, g.bc[1]);
        static_for<Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            if (ax.wall[1 - kLattice<L>.e[a][0]] || ay.wall[1 - kLattice<L>.e[a][1]]) bits_xy |= 1u << a;
        });
        if ((g.bc[0] == kSolidEnds && (gx == 0 || gx == g.nx - 1)) ||
            (g.bc[1] == kSolidEnds && (gy == 0 || gy == g.ny - 1)))
            bits_xy |= kSolid;
    }
    const auto link_bits = [&](int z) -> unsigned {
        if constexpr (!WALLS) return 0u;
        if (WK == kMarchMask || (WK == kMarchNodal && g.links)) return g.links[node_index(g, gx, gy, z)];
        const Axis3 az = axis3<true>(z, g.nz, g.bc[2]);
        unsigned b = (g.bc[2] == kSolidEnds && (z == 0 || z == g.nz - 1)) ? kSolid : 0u;
        static_for<Q>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            if (az.wall[1 - kLattice<L>.e[a][2]]) b |= 1u << a;
        });
        return b | bits_xy;
    };
    // Whether any node of the wavefront has a wall next to it.
    const auto near_walls = [&](unsigned b) { return WALLS && __any((b & ~kSolid) != 0); };

    // The pulls of level 1 in plane z.  With on = false (past the last plane)
    // the loads return 0 without an access.
    const auto load_plane = [&](int z, unsigned bits, S (&out)[Q], bool on) {
        const Plane pl[3] = {plane_at(z == 0 ? g.nz - 1 : z - 1), plane_at(z), plane_at(up(z))};
        const char* base = reinterpret_cast<const char*>(src);
        const __amdgpu_buffer_rsrc_t rs[3] = {rsrc_at(base + pl[0].base, on ? total - pl[0].base : 0),
                                              rsrc_at(base + pl[1].base, on ? total - pl[1].base : 0),
                                              rsrc_at(base + pl[2].base, on ? total - pl[2].base : 0)};
        // Byte positions of x - 1, x, x + 1 and of rows y - 1, y, y + 1,
        // formed anew for each plane (the empty asm keeps the compiler from
        // holding them, and the offsets below, in registers all the time).
        int cx = gx, cy = gy;
        asm volatile("" : "+v"(cx), "+v"(cy));
        unsigned xs[3], ys[3];
        xs[1] = B * unsigned(cx);
        xs[0] = cx == 0 ? B * unsigned(g.nx - 1) : xs[1] - B;
        xs[2] = cx == g.nx - 1 ? 0u : xs[1] + B;
        ys[1] = row_bytes * unsigned(cy);
        ys[0] = cy == 0 ? row_bytes * unsigned(g.ny - 1) : ys[1] - row_bytes;
        ys[2] = cy == g.ny - 1 ? 0u : ys[1] + row_bytes;
        // One source column and row after the other, so that few offsets are
        // held at a time.
        const auto fetch = [&](auto&& off) {
            static_for<9>([&](auto kc) {
                constexpr int kx = decltype(kc)::value / 3, ky = decltype(kc)::value % 3;
                const auto o = off(xs[kx] + ys[ky]);
                static_for<Q>([&](auto ac) {
                    constexpr int a = decltype(ac)::value;
                    constexpr int kz = 1 - kLattice<L>.e[a][2];
                    if constexpr (1 - kLattice<L>.e[a][0] == kx && 1 - kLattice<L>.e[a][1] == ky)
                        out[a] = buffer_get<S>(rs[kz], o(kz), unsigned(a) * run_bytes);
                });
            });
        };
        if (!level1) return;
        // In a plane of whole tiles (256^3, 512 x 128 x 128) a node has the
        // same offset in every plane.  FP64 (not bound by instructions) keeps
        // one form and has the registers instead.
        if (B < 8 && whole_tiles) {
            fetch([&](unsigned spot) {
                const unsigned o = offset(spot);
                return [o](int) { return o; };
            });
        } else {
            fetch([&](unsigned spot) { return [&, spot](int kz) { return offset(spot + pl[kz].at); }; });
        }
        if (near_walls(bits)) {  // a population from a wall is the node's own opposite one
            const unsigned own = offset(xs[1] + ys[1] + pl[1].at);
            static_for<Q>([&](auto ac) {
                constexpr int a = decltype(ac)::value;
                if ((bits >> a) & 1u) out[a] = buffer_get<S>(rs[1], own, unsigned(Lattice<L>::opp(a)) * run_bytes);
            });
        }
    };

    // Carried from plane to plane for the pulls of level 2: e_z = 0 of one
    // plane and e_z = +1 of two.
    S d0[N0], dp1[N1], dp2[N1], f1[Q];
#pragma unroll
    for (int j = 0; j < N0; ++j) d0[j] = S(0);
#pragma unroll
    for (int j = 0; j < N1; ++j) dp1[j] = dp2[j] = S(0);
    int z = z0 == 0 ? g.nz - 1 : z0 - 1;  // q, wrapped
    unsigned bits = link_bits(z), bits_next = link_bits(up(z)), bits_prev = 0;
    load_plane(z, bits, f1, true);
    for (int q = z0 - 1; q <= z1; ++q) {
        if constexpr (WALLS && !kCarryBits) {
            bits = link_bits(z);
            bits_prev = q > z0 ? link_bits(q - 1) : 0u;
        }
        // Level 1 of plane q.
        if (level1) {
            if constexpr (WK == kMarchNodal) nodal_fill<L>(g, gx, gy, z, f1);
            collide<L, S, FORCE, COMP, Store<S>::kDeviation>(f1, plane_args<FORCE>(p.c));
        }
        __syncthreads();  // level 2 has taken the previous plane from LDS
        if (to_lds) {
#pragma unroll
            for (int a = 0; a < Q; ++a) sh[a][row][col] = f1[a];
        }
        const int zn = up(z);
        unsigned bits_far = 0;
        if constexpr (kCarryBits) bits_far = link_bits(up(zn));  // read a plane ahead of their use
        else bits_next = link_bits(zn);
        // What walls above plane q - 1 return to it (kept by the end of the
        // previous iteration).
        S back[N1];
        if constexpr (WALLS) {
#pragma unroll
            for (int j = 0; j < N1; ++j) back[j] = S(0);
            if (level2 && q > z0 && store_x && near_walls(bits_prev)) {
                const S* at = dst + slot<Q>(0, node_index(g, gx, gy, q - 1), TS);
                static_for<Q>([&](auto ac) {
                    constexpr int a = decltype(ac)::value;
                    if constexpr (kLattice<L>.e[a][2] == -1) {
                        if ((bits_prev >> a) & 1u) back[D::rank(a)] = at[size_t(a) << TS];
                    }
                });
            }
        }
        load_plane(zn, bits_next, f1, q < z1);
        __syncthreads();
        if (level2) {
            if (q > z0) {  // level 2 of plane q - 1
                S f[Q];
                static_for<Q>([&](auto ac) {
                    constexpr int a = decltype(ac)::value;
                    constexpr int ex = kLattice<L>.e[a][0], ey = kLattice<L>.e[a][1], ez = kLattice<L>.e[a][2];
                    constexpr int j = D::rank(a);
                    if constexpr (ez == 0) {
                        f[a] = d0[j];
                    } else if constexpr (ez == 1) {
                        f[a] = dp2[j];
                    } else {
                        f[a] = sh[a][row - ey][col - ex];
                        if constexpr (WALLS) {
                            if ((bits_prev >> a) & 1u) f[a] = back[j];
                        }
                    }
                });
                if constexpr (WK == kMarchNodal) nodal_fill<L>(g, gx, gy, q - 1, f);
                collide<L, S, FORCE, COMP, Store<S>::kDeviation>(f, plane_args<FORCE>(p.c));
                if (store_x && !(WALLS && (bits_prev & kSolid))) {
                    const Plane pl = plane_at(q - 1);
                    const auto rs = rsrc_at(reinterpret_cast<const char*>(dst) + pl.base, total - pl.base);
                    const unsigned voff = offset(B * unsigned(gx) + row_bytes * unsigned(gy) + pl.at);
                    static_for<Q>([&](auto ac) {
                        constexpr int a = decltype(ac)::value;
                        buffer_put<WaveStores<S>::kAux>(rs, voff, unsigned(a) * run_bytes, f[a]);
                    });
                }
            }
            static_for<Q>([&](auto ac) {
                constexpr int a = decltype(ac)::value;
                constexpr int ex = kLattice<L>.e[a][0], ey = kLattice<L>.e[a][1], ez = kLattice<L>.e[a][2];
                constexpr int j = D::rank(a);
                if constexpr (ez == 0) {
                    d0[j] = sh[a][row - ey][col - ex];
                } else if constexpr (ez == 1) {
                    dp2[j] = dp1[j];
                    dp1[j] = sh[a][row - ey][col - ex];
                }
            });
            if (near_walls(bits)) {
                // Walls next to plane q: its e_z = 0 and (from plane q - 1)
                // e_z = +1 pulls that come from a wall are its own opposite
                // populations.  Its e_z = -1 pulls that come from a wall
                // above are its own e_z = +1 populations, which LDS loses
                // before level 2 needs them; they wait in the places of dst
                // that this work-item stores to then (in registers they
                // would make every wavefront spill: D3Q27 sphere box 500
                // instead of 410 us per step).
                S* own = dst + slot<Q>(0, node_index(g, gx, gy, z), TS);
                static_for<Q>([&](auto ac) {
                    constexpr int a = decltype(ac)::value;
                    constexpr int abar = Lattice<L>::opp(a), ez = kLattice<L>.e[a][2];
                    constexpr int j = D::rank(a);
                    if constexpr (ez == 0) {
                        if ((bits >> a) & 1u) d0[j] = sh[abar][row][col];
                    } else if constexpr (ez == 1) {
                        if ((bits >> a) & 1u) dp2[j] = sh[abar][row][col];
                    } else if (store_x && q >= z0 && q < z1) {
                        if ((bits >> a) & 1u) own[size_t(a) << TS] = sh[abar][row][col];
                    }
                });
            }
        }
        z = zn;
        if constexpr (kCarryBits) {
            bits_prev = bits;
            bits = bits_next;
            bits_next = bits_far;
        }
    }
}

}  // namespace imexlbm
