// Kernels of the coupled phase-field + P-u lattice Boltzmann step
// (Otomo et al., arXiv 2512.01027, Sec. II) for gfx950.
//
// One time step is up to four launches over every resident case:
//   k_moments  per node, no halo: gathers h and g (AA pattern) and writes
//              phi = sum h, u* = sum g c, P* = rho_ref T sum g (the pressure
//              the populations carry; the stored rest population lacks the
//              previous P, which is added back) and M2 = sum g c c (in
//              2-byte storage as 2-byte codes, two to a 32-bit word).
//   k_pressure 1-halo LDS tile: the pressure formula of Sec. II with K_i of
//              P* and, in the omega term, u* at x - c_i.  Link terms are
//              summed per shell in the auxiliary type (FP64 in FP64 storage,
//              FP32 otherwise); the shell-weighted sum and the final
//              combination are FP64.
//   k_velocity 1-halo LDS tile: u = sum_i (g_i + K_i) c_i with K_i of the new
//              pressure, i.e. u = u* - D P / rho.
//   k_collide  1-halo LDS tile of phi and u: the isotropic central
//              differences of phi, rho and u, the BGK phase-field collision
//              and the filter collision of the hydrodynamic LBE, written back
//              in place (AA pattern).  Cases without walls, open end or block
//              on D3Q19 hydro (with 4- or 8-byte storage) rebuild u here from
//              u* and a 2-node halo of the new P, and a step skips k_velocity;
//              2D cases rebuild P as well (from a 3-node halo of P* and u*),
//              and a step is k_moments and k_collide alone.
// Large single 3D cases take pressure and velocity on wide tiles
// (k_pressure_wide, k_velocity_wide).
//
// Memory layout (per case): structure of arrays, x fastest; population i of
// node n at f[i*N + n].  AA pattern: on even steps node x reads slot i of x
// and writes its post-collision f*_i to slot opp(i) of x; on odd steps it reads
// slot opp(i) of x - c_i and writes slot i of x + c_i.  Each node reads and
// writes the same set of slots within a step, so the update is in place with
// no race.  Halfway bounce-back: a population that would leave through a
// wall is written to the slot the node itself reads as the reflected
// direction next step.
//
// The rest population of g is stored as g_0 - P/(rho_ref T): the pressure
// (kept separately as state) never passes through the distribution storage,
// and k_moments needs no pressure at all.
//
// Addressing: case descriptors and tile tables are read through the
// constant address space (scalar loads, values in SGPRs); arrays are used
// through global-address-space pointers with 32-bit node indices.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "codec.hpp"
#include "lattice.hpp"

namespace pulbm {

// The tiles of one shape that cover a case's grid, and their order.
struct TileMap {
    int32_t ntx, nty, ntz;  // tiles per axis
    int32_t tband;          // tile rows per y band of the tile order (>= 1)
    // The tile order's divisors -- ntx, tband ntz, tband and the last band's
    // rows -- as multipliers M = floor(2^40 / d) + 1 split into high and low
    // words, so that a block takes its tile apart with scalar multiplies:
    // n / d = (n Mh + mulhi(n, Ml)) >> 8, exact while n d < 2^40 (fastdiv
    // = 1, checked for every divisor against its largest dividend when the
    // case is created; otherwise the kernels divide).
    int32_t fastdiv;
    uint32_t dvh[4], dvl[4];
};

// Per-case descriptor, resident in device memory (one per case of a launch).
struct CaseDev {
    int32_t nx, ny, nz, dim;
    int32_t wall[3];
    TileMap map;   // the lattice set's tiles (Model)
    TileMap wide;  // the tiles of k_pressure_wide and k_velocity_wide (3D)
    int32_t near_lo[3], near_n[3];  // the box of wide tiles whose halo reaches the block
    int32_t near_subs;  // their tiles of the lattice set's shape, rounded up to 8 (0: no block)
    int32_t delta_theta;
    int32_t sx;        // row pitch in nodes: nx rounded up to 32, so that every row of a
                       // tile starts on a 128-byte line (node n = x + sx (y + ny z))
    int64_t N;         // nodes per field including the row padding (sx ny nz)
    int64_t step;      // steps done
    int64_t step_end;  // the case is advanced while step < step_end
    void* h;           // Q_h * N populations (storage type)
    void* g;           // Q_g * N populations (storage type)
    void* P[2];        // pressure ping-pong: P[step & 1] is the previous-step pressure
    void* phi[2];      // N each: phi of this step's moments at phi[step & 1]; phi[(step + 1) & 1]
                       // keeps the previous step's, the reference of the 2-byte h codec
    void* J;           // dim*N  scratch: u* = sum g c
    void* Ps;          // N      scratch: P* = previous P + rho_ref T sum g, the pressure the
                       //        streamed populations carry (the rest population holds
                       //        g_0 - P/(rho_ref T), so the previous P is added back)
    void* M2;          // 3 (2D) or 6 (3D) * N scratch: sum g c c
    void* U[2];        // dim*N each: velocity of this step at U[step & 1]; U[(step + 1) & 1]
                       // keeps the previous step's, the second reference of the 2-byte codecs
    double rho_a, rho_w, tau_a, tau_w, tau_phi, M, W, sigma, lambda_b;
    double grav[3];
    double h_scale, h_inv_scale, g_scale, g_inv_scale;
    double p_top;           // pressure of an open high end (wall = 2 on the last axis)
    int32_t blk_lo[3], blk_hi[3];  // solid block, nodes lo <= x < hi (has_block)
    int32_t has_block;
    int32_t fuse_u; // 1: the collide kernel rebuilds u itself and a step skips k_velocity
                    // (no wall, open end or block, 4- or 8-byte storage, every axis >= 3,
                    // D3Q19 hydro)
                    // 2: it rebuilds P and u, and a step skips k_pressure and k_velocity
                    // (2D, no block, both axes >= 3)
    int32_t tile_rev;  // 1: the case's tiles are taken in reverse order (a race check, pulbm_set_tile_order)
    int32_t ntiles;
    int32_t nt_odd_moments;  // 1: k_moments streams its 4- and 8-byte loads on odd steps too
    // Constants of the collision derived once on the host (so no thread
    // divides in FP64): 1 / tau_phi, M / (T W), 48 sigma / W, 1.5 sigma W;
    // and every constant the FP32 kernels use, rounded once to FP32.
    double inv_tau_phi, theta0, sig48W, sigW15;
    struct {
        float rho_a, drho, tau_a, dtau, inv_tau_phi, theta0, sig48W, sigW15, lambda_b, grav[3];
        float h_scale, h_inv_scale, g_scale, g_inv_scale;
    } f32;
};

using CDesc = const PULBM_CST CaseDev;

template <class T> __device__ __forceinline__ PULBM_GLB T* glb(void* p) { return (PULBM_GLB T*)p; }

// A launch covers the tiles of every case in a table of case pointers.  The
// table's header lives in device memory next to it -- hdr[0] cases,
// hdr[1] tiles in all, hdr[2 + c] the first tile of case c -- so a captured
// graph stays valid while cases join and leave, as long as the grid has a
// block for every tile.
//
// A launch for one case alone has no table: hdr is NULL and the table argument is
// the case's descriptor itself.  The descriptor's fields are then one scalar
// load away from the kernel's arguments; through the table they were three
// (header, table, descriptor), each waiting for the one before (24^3 FP64 22.5
// -> 21.3 us a step, 200 x 400 15.6 -> 14.9, 128^3 FP32 242 -> 239, with the
// arguments preloaded into registers).
using CaseTab = CaseDev* const*;

// --------------------------------------------------------------- launch map

// Blocks are dealt to the 8 XCDs round-robin; remapping gives each XCD one
// contiguous run of tiles, so tiles that share halo planes share an L2.
// The grid is a multiple of 8.
__device__ __forceinline__ int xcd_tile(int bid, int nblocks)
{
    const int per = nblocks >> 3;
    return (bid & 7) * per + (bid >> 3);
}

// n / d for the multiplier (mh, ml) of d (TileMap::dvh, dvl): the high word
// of n times the 40-bit multiplier, shifted down by 8.  n mh stays below 2^32
// for n < 2^23 (mh <= 256).
__device__ __forceinline__ uint32_t udiv_m(uint32_t n, uint32_t mh, uint32_t ml)
{
    return (n * mh + __umulhi(n, ml)) >> 8;
}

__device__ __forceinline__ int find_case(const PULBM_CST int* tstart, int ncases, int tile)
{
    int lo = 0, hi = ncases - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (tstart[mid] <= tile) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

struct TileCtx {
    CDesc* cs;
    int ox, oy, oz;  // tile origin
    int64_t step;
    bool active;
};

// Tile lt of a case, in the tile order: x fastest, then z within a band of
// tband tile rows, then the bands along y.  Tiles that share z-halo rows then
// run close together (a band's width of tiles apart), while each plane is
// still read in runs of whole rows.
__device__ __forceinline__ void tile_xyz(const PULBM_CST TileMap& m, int lt, int* tx, int* ty, int* tz)
{
    if (m.fastdiv) {
        const uint32_t l = (uint32_t)lt;
        const uint32_t r = udiv_m(l, m.dvh[0], m.dvl[0]);
        *tx = (int)(l - r * (uint32_t)m.ntx);
        const uint32_t yb = udiv_m(r, m.dvh[1], m.dvl[1]);
        const uint32_t rem = r - yb * (uint32_t)(m.tband * m.ntz);
        const int rows = m.nty - (int)yb * m.tband;  // rows of this band: tband, or fewer in the last
        const int k = rows < m.tband ? 3 : 2;
        const uint32_t tq = udiv_m(rem, m.dvh[k], m.dvl[k]);
        *tz = (int)tq;
        *ty = (int)yb * m.tband + (int)(rem - tq * (uint32_t)min(m.tband, rows));
    } else {
        *tx = lt % m.ntx;
        lt /= m.ntx;
        const int yb = lt / (m.tband * m.ntz);
        const int rem = lt - yb * m.tband * m.ntz;
        const int by = min(m.tband, m.nty - yb * m.tband);
        *tz = rem / by;
        *ty = yb * m.tband + rem % by;
    }
}

template <class Mo>
__device__ __forceinline__ TileCtx tile_ctx(CaseTab cases, const int* hdr_, int step_off)
{
    TileCtx t;
    const PULBM_CST int* hdr = (const PULBM_CST int*)hdr_;
    int lt, ntiles;
    if (!hdr) {
        t.cs = (CDesc*)(uintptr_t)cases;
        ntiles = t.cs->ntiles;
        const int used = (ntiles + 7) & ~7;
        t.active = (int)blockIdx.x < used;
        if (!t.active) return t;
        lt = xcd_tile(blockIdx.x, used);
        t.active = lt < ntiles;
        if (!t.active) return t;
    } else {
        const int ncases = hdr[0], total_tiles = hdr[1];
        // the first blocks (a multiple of 8) take the tiles; the XCD remap runs
        // over them only, so every XCD gets its share however large the grid
        const int used = (total_tiles + 7) & ~7;
        t.active = (int)blockIdx.x < used;
        if (!t.active) return t;
        const int tile = xcd_tile(blockIdx.x, used);
        t.active = tile < total_tiles;
        if (!t.active) return t;
        const PULBM_CST int* tstart = hdr + 2;
        const int ci = find_case(tstart, ncases, tile);
        const PULBM_CST uint64_t* tab = (const PULBM_CST uint64_t*)(const void*)cases;
        t.cs = (CDesc*)(uintptr_t)tab[ci];
        lt = tile - tstart[ci];
        ntiles = tstart[ci + 1] - tstart[ci];
    }
    CDesc& cs = *t.cs;
    // step_off < 0: read mode (the moment stage of the current state, run
    // whatever the case's step limit)
    t.step = cs.step + (step_off > 0 ? step_off : 0);
    t.active = step_off < 0 || t.step < cs.step_end;
    if (cs.tile_rev) lt = ntiles - 1 - lt;
    int tx, ty, tz;
    tile_xyz(cs.map, lt, &tx, &ty, &tz);
    t.ox = tx * Mo::TX;
    t.oy = ty * Mo::TY;
    t.oz = tz * Mo::TZ;
    return t;
}

// Tile shape of k_pressure_wide and k_velocity_wide: four nodes to a thread,
// one above the other in z.
struct WideTile {
    static constexpr int TX = 64, TY = 4, TZ = 4;
};

// The wide tile of a block of a single case's launch.
// Wide tiles near the solid block, whose ghosts mirror cell by cell, are taken
// as tiles of the lattice set's shape, a block each (*sub; the first near_subs
// blocks): one after another in the wide tile's own block they held up the XCD
// whose run holds them (293 x 91 x 91 with a block: pressure 41 us).
template <class Mo> __device__ __forceinline__ TileCtx wide_ctx(CaseTab cases, int step_off, bool* sub)
{
    TileCtx t;
    t.cs = (CDesc*)(uintptr_t)cases;
    CDesc& cs = *t.cs;
    t.step = cs.step + (step_off > 0 ? step_off : 0);
    *sub = (int)blockIdx.x < cs.near_subs;
    if (*sub) {
        constexpr int SY = WideTile::TY / Mo::TY, SUBS = SY * (WideTile::TZ / Mo::TZ);
        const int k = (int)blockIdx.x % SUBS, w = (int)blockIdx.x / SUBS;
        const int wx = w % cs.near_n[0], wy = w / cs.near_n[0] % cs.near_n[1], wz = w / (cs.near_n[0] * cs.near_n[1]);
        t.ox = (cs.near_lo[0] + wx) * WideTile::TX;
        t.oy = (cs.near_lo[1] + wy) * WideTile::TY + k % SY * Mo::TY;
        t.oz = (cs.near_lo[2] + wz) * WideTile::TZ + k / SY * Mo::TZ;
        t.active = wz < cs.near_n[2] && t.oy < cs.ny && t.oz < cs.nz && (step_off < 0 || t.step < cs.step_end);
        return t;
    }
    const int bid = (int)blockIdx.x - cs.near_subs;
    const int total = cs.wide.ntx * cs.wide.nty * cs.wide.ntz, used = (total + 7) & ~7;
    t.active = bid < used;
    if (!t.active) return t;
    int lt = xcd_tile(bid, used);
    t.active = lt < total && (step_off < 0 || t.step < cs.step_end);
    if (!t.active) return t;
    if (cs.tile_rev) lt = total - 1 - lt;
    int tx, ty, tz;
    tile_xyz(cs.wide, lt, &tx, &ty, &tz);
    t.ox = tx * WideTile::TX;
    t.oy = ty * WideTile::TY;
    t.oz = tz * WideTile::TZ;
    return t;
}

// Q slots of N elements of T (structure of arrays).  Addresses are formed as
// a uniform slot base (SGPRs) plus a 32-bit per-node byte offset, which maps
// onto the saddr + voffset form of the global memory instructions.
// Buffer load / store of populations: the slot's base and length sit in a
// buffer resource (SGPRs) and each lane supplies only its 32-bit byte offset.
// Through plain pointers the compiler forms every population address as a
// per-lane 64-bit sum; through buffer resources the collision kernel issues
// about 12% fewer vector instructions and keeps fewer registers live.  No
// offset past the slot is formed: every target node lies in the grid.  aux 2
// marks the access non-temporal.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(PULBM_GLB char* base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000);
}
template <bool NT, class T> __device__ __forceinline__ T buf_ld(__amdgpu_buffer_rsrc_t r, uint32_t boff, uint32_t soff)
{
    constexpr int aux = NT ? 2 : 0;
    if constexpr (sizeof(T) == 2) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, (int)boff, (int)soff, aux));
    else if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, (int)boff, (int)soff, aux));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, (int)boff, (int)soff, aux));
}
template <bool NT, class T> __device__ __forceinline__ void buf_st(__amdgpu_buffer_rsrc_t r, uint32_t boff, uint32_t soff, T v)
{
    constexpr int aux = NT ? 2 : 0;
    if constexpr (sizeof(T) == 2) {
        __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, v), r, (int)boff, (int)soff, aux);
    } else if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, (int)boff, (int)soff, aux);
    } else {
        typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, (int)boff, (int)soff, aux);
    }
}

// PAIRED: one resource serves the two slots of an opposite pair (2 slot_bytes
// stay below 2^32), the second at a scalar offset; otherwise a slot has its
// own.  A resource takes four SGPRs, and the collide, which loads and stores
// every slot, spills twice as many with one per slot (160^3 walls, FP32 odd
// collide 281 paired / 298 us).  The moments only load: one per slot in 4-byte 3D
// storage (128^3 odd 101.9 paired / 100.1 us), paired in the others (512 x 256 x
// 256 BF16 odd 864 / 941 us, 2000 x 1200 FP64 step 297 / 310; FP16 the same within
// 0.5% of the step; 2D FP32, where forming them is not hidden on small grids, a
// batch of 12 of 128^2 13.0 / 13.4, though 1024^2 54.4 / 52.8).
template <class T, bool PAIRED = true>
struct Slots {
    PULBM_GLB char* base;
    uint64_t slot_bytes;  // N * sizeof(T), below 2^31
    __device__ __forceinline__ PULBM_GLB T* at(int slot, uint32_t boff) const
    {
        return (PULBM_GLB T*)(base + (uint64_t)slot * slot_bytes + boff);
    }
    __device__ static __forceinline__ int first(int slot) { return !PAIRED || slot == 0 ? slot : ((slot - 1) | 1); }
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(int slot) const
    {
        return buf_rsrc(base + (uint64_t)first(slot) * slot_bytes, (PAIRED ? 2u : 1u) * (uint32_t)slot_bytes);
    }
    __device__ __forceinline__ uint32_t soff(int slot) const { return slot == first(slot) ? 0u : (uint32_t)slot_bytes; }
};

template <class T, bool PAIRED = true> __device__ __forceinline__ Slots<T, PAIRED> slots(void* p, int64_t N)
{
    Slots<T, PAIRED> s;
    s.base = (PULBM_GLB char*)p;
    s.slot_bytes = (uint64_t)N * sizeof(T);
    return s;
}

// M2, the second moment of g that the moment stage writes and the collision
// reads once, is kept in the compute type, except in 2-byte storage: there
// each component is encoded with g's codec and scale (no shift) and two of
// them share a 32-bit word (word j holds components 2j and 2j + 1, the first
// in the low half), so a node's six values take three loads and three
// registers.  The collide keeps 2-byte h in registers the same way.
template <class S> __device__ __forceinline__ uint32_t pair_pack(S lo, S hi)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, lo) | ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
}
template <class S> __device__ __forceinline__ S pair_half(uint32_t w, int k)
{
    return __builtin_bit_cast(S, (uint16_t)(k ? w >> 16 : w & 0xffffu));
}

template <class T> __device__ __forceinline__ PULBM_GLB T* at_node(void* p, uint32_t n)
{
    return (PULBM_GLB T*)((PULBM_GLB char*)p + n * (uint32_t)sizeof(T));
}

// Neighbour navigation of one node: byte offsets (elements of ESZ bytes) of a
// -1/0/+1 step along each axis (periodic wrap included) and which steps
// leave through a wall.
struct Nav {
    int o[3][3];
    uint32_t solid;  // bit 2a: the -1 step on axis a is outside a wall; bit 2a+1: the +1 step
    uint32_t open;   // the same bits for a step out through an open end
    uint32_t blk[3]; // bit k: coordinate + k - 1 on axis a lies in the block's range
};

// Is node (x, y, z) inside the solid block?
__device__ __forceinline__ bool in_block(CDesc& cs, int x, int y, int z)
{
    return cs.has_block && x >= cs.blk_lo[0] && x < cs.blk_hi[0] && y >= cs.blk_lo[1] && y < cs.blk_hi[1] &&
           z >= cs.blk_lo[2] && z < cs.blk_hi[2];
}

__device__ __forceinline__ Nav make_nav(CDesc& cs, int x, int y, int z, int esz)
{
    Nav v;
    const int p[3] = {x, y, z};
    const int n[3] = {cs.nx, cs.ny, cs.nz};
    const int st[3] = {esz, esz * cs.sx, esz * cs.sx * cs.ny};
    v.solid = 0;
    v.open = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        v.o[a][1] = 0;
        v.o[a][0] = (p[a] == 0) ? (n[a] - 1) * st[a] : -st[a];
        v.o[a][2] = (p[a] == n[a] - 1) ? -(n[a] - 1) * st[a] : st[a];
        if (cs.wall[a]) {
            if (p[a] == 0) v.solid |= 1u << (2 * a);
            if (p[a] == n[a] - 1) {
                if (cs.wall[a] == 2) v.open |= 1u << (2 * a + 1);
                else v.solid |= 1u << (2 * a + 1);
            }
        }
        // a block spanning a whole periodic axis holds every coordinate
        const bool full = cs.blk_lo[a] == 0 && cs.blk_hi[a] == n[a];
        v.blk[a] = 0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int q = p[a] + k - 1;
            if (cs.has_block && (full || (q >= cs.blk_lo[a] && q < cs.blk_hi[a]))) v.blk[a] |= 1u << k;
        }
    }
    return v;
}

// Nav of a node whose neighbours all lie inside the grid (no wall, block or
// wrap within one node): the offsets are the strides, the same for every
// node of the workgroup.
__device__ __forceinline__ Nav make_nav_inner(CDesc& cs, int esz)
{
    Nav v;
    const int st[3] = {esz, esz * cs.sx, esz * cs.sx * cs.ny};
    v.solid = 0;
    v.open = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        v.o[a][0] = -st[a];
        v.o[a][1] = 0;
        v.o[a][2] = st[a];
        v.blk[a] = 0;
    }
    return v;
}

template <class L>
__device__ __forceinline__ int nav_off(const Nav& v, int i, int sgn)
{
    return v.o[0][sgn * L::c(i, 0) + 1] + v.o[1][sgn * L::c(i, 1) + 1] + v.o[2][sgn * L::c(i, 2) + 1];
}

template <class L> __device__ __forceinline__ uint32_t nav_mask(int i, int sgn)
{
    uint32_t m = 0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const int ca = sgn * L::c(i, a);
        if (ca == -1) m |= 1u << (2 * a);
        if (ca == 1) m |= 1u << (2 * a + 1);
    }
    return m;
}

// Does the step along sgn c_i leave through the open end?
template <class L>
__device__ __forceinline__ bool nav_open(const Nav& v, int i, int sgn)
{
    return (v.open & nav_mask<L>(i, sgn)) != 0;
}

// Does the step along sgn c_i leave the fluid (through a wall or the open
// end, or into the block)?  Its population then stays at the node, in the
// slot of the opposite direction.
template <class L>
__device__ __forceinline__ bool nav_solid(const Nav& v, int i, int sgn)
{
    const bool blk = ((v.blk[0] >> (sgn * L::c(i, 0) + 1)) & (v.blk[1] >> (sgn * L::c(i, 1) + 1)) &
                      (v.blk[2] >> (sgn * L::c(i, 2) + 1)) & 1u) != 0;
    return ((v.solid | v.open) & nav_mask<L>(i, sgn)) != 0 || blk;
}

// Does the tile (or its ghost layer) touch a wall, the open end or the
// block?  Uniform per block; tiles that do not skip every boundary test.
template <class Mo>
__device__ __forceinline__ bool tile_at_wall(CDesc& cs, int ox, int oy, int oz)
{
    const bool blk = cs.has_block && ox - 1 < cs.blk_hi[0] && ox + Mo::TX >= cs.blk_lo[0] && oy - 1 < cs.blk_hi[1] &&
                     oy + Mo::TY >= cs.blk_lo[1] && oz - 1 < cs.blk_hi[2] && oz + Mo::TZ >= cs.blk_lo[2];
    return (cs.wall[0] && (ox == 0 || ox + Mo::TX >= cs.nx)) || (cs.wall[1] && (oy == 0 || oy + Mo::TY >= cs.ny)) ||
           (cs.wall[2] && (oz == 0 || oz + Mo::TZ >= cs.nz)) || blk;
}

// Population loads and stores.  The populations of a step are read once and
// written once, and at the sizes that matter the state is far larger than the
// caches, so accesses can be marked non-temporal.  Which accesses gain from it
// was measured per storage width (bit 0: loads in k_moments, bit 1: loads in
// k_collide, bit 2: stores in k_collide, bit 3: loads in k_moments on even
// steps only): populations of every width stream the collide's loads, the
// collide's stores on even steps (odd-step stores stay in L2, see
// collide_tile) and k_moments' loads on even steps: on odd steps, shifted by
// one node in x, a line is read partly by one tile and partly by its x
// neighbour, and streamed past L2 it is fetched twice.  Wide populations of
// a small grid stream on odd steps too (CaseDev::nt_odd_moments): the
// second fetch then hits the last-level cache.
// The per-node fields a kernel reads only at its own nodes (the codecs'
// previous-step phi and u, the previous P, u*, phi and M2 where no halo of
// them is taken) are loaded non-temporal too (FP16 step 3.03 -> 2.99 ms).
enum PopAccess { kLoadMoments = 1, kLoadCollide = 2, kStoreCollide = 4, kLoadMomentsEven = 8 };
constexpr int kNtWide = kLoadMomentsEven | kLoadCollide | kStoreCollide, kNtHalf = kNtWide;
template <class S, int A> constexpr bool nt_access() { return ((sizeof(S) >= 4 ? kNtWide : kNtHalf) & A) != 0; }

// Population arriving at the node (byte offset nb) along direction i.
template <class L, bool WALL, bool NT, class S, bool PAIRED>
__device__ __forceinline__ S aa_load(const Slots<S, PAIRED>& f, uint32_t nb, const Nav& v, int i, bool odd)
{
    if (!odd) return buf_ld<NT, S>(f.rsrc(i), nb, f.soff(i));
    if (WALL && nav_solid<L>(v, i, -1)) return buf_ld<NT, S>(f.rsrc(i), nb, f.soff(i));  // reflected at a wall last step
    return buf_ld<NT, S>(f.rsrc(opp(i)), nb + (uint32_t)nav_off<L>(v, i, -1), f.soff(opp(i)));
}

// Store the node's post-collision population i where it streams to; a
// population leaving through a wall goes to the slot the node reads back as
// the reflected direction.
template <class L, bool WALL, bool NT, class S>
__device__ __forceinline__ void aa_store(const Slots<S>& f, uint32_t nb, const Nav& v, int i, bool odd, S val,
                                         bool bb)
{
    if (!odd || (WALL && bb)) buf_st<NT, S>(f.rsrc(opp(i)), nb, f.soff(opp(i)), val);
    else buf_st<NT, S>(f.rsrc(i), nb + (uint32_t)nav_off<L>(v, i, +1), f.soff(i), val);
}

// ---------------------------------------------------------- tile regions

// Resolve global coordinate t on an axis of n nodes: periodic wrap, or the
// mirror node of a ghost outside a wall (off = t - mirror).  A ghost beyond
// an open end (wall = 2, high side) takes the nearest node too, marked by
// kOpenGhost in *crossed instead of counting as a wall crossing.
// Branch-free, without division: a 1-node halo reaches at most one node past
// either end, where one +-n wraps exactly.  Cells further out belong only to
// the halo of nodes outside the grid (a ragged last tile); they are kept
// inside the grid by the clamp and their values are never used.
constexpr int kOpenGhost = 256;
__device__ __forceinline__ int resolve_axis(int t, int n, int wall, int* off, int* crossed)
{
    const bool lo = t < 0, hi = t >= n;
    const int near = lo ? 0 : (hi ? n - 1 : t);
    const int wrapped = min(lo ? t + n : (hi ? t - n : t), n - 1);
    *off = wall ? t - near : 0;
    *crossed += (wall && (lo || hi)) ? ((wall == 2 && hi) ? kOpenGhost : 1) : 0;
    return wall ? near : wrapped;
}

template <int RX, int RY, int RZ>
struct Region {
    static constexpr int N = RX * RY * RZ;
    __device__ static __forceinline__ int idx(int ix, int iy, int iz) { return ix + RX * (iy + RY * iz); }
    // The 3x3(x3) neighbourhood of cell (cx, cy, cz): its lowest corner
    // (cx - 1, cy - 1, cz - ZL) as a base index, and each cell of it at a
    // constant offset from there that is never negative, which LDS reads
    // take as their immediate (DS offsets are unsigned).
    template <int ZL>
    __device__ static __forceinline__ int nb_base(int cx, int cy, int cz) { return idx(cx - 1, cy - 1, cz - ZL); }
    template <int ZL>
    static constexpr int nb(int dx, int dy, int dz) { return (1 + dx) + RX * ((1 + dy) + RY * (ZL + dz)); }
};

// The stencil fields of a tile's cells in LDS: NF values to a cell, in 16-byte
// words (one ds_read_b128 brings four FP32 or two FP64 values of a neighbour)
// and, where NF is odd, one value apart.  Each word array has a 16-byte pitch,
// so a wavefront's row is read without bank conflicts.
template <class CT, int NF, int NC> struct Cells {
    static constexpr int PW = 16 / (int)sizeof(CT), NW = NF / PW, REM = NF % PW;
    static_assert(REM <= 1, "at most one value apart");
    typedef CT V __attribute__((ext_vector_type(PW)));
    V w[NW][NC];
    CT r[REM ? NC : 1];
    // A cell that neighbours are read from at constant offsets: its byte
    // offset in each array, hidden from the compiler's bit tracking so that
    // every read takes its offset as an immediate from one register per pitch.
    // (Left visible, each row of the 3x3x3 block gets an address of its own,
    // formed from the bits of the thread index and kept live.)
    struct At {
        int bw, br;
        __device__ __forceinline__ void hide()
        {
            asm volatile("" : "+v"(bw));
            asm volatile("" : "+v"(br));
        }
    };
    __device__ static __forceinline__ At at(int k)
    {
        At a = {k * 16, k * (int)sizeof(CT)};
        a.hide();
        return a;
    }
    __device__ __forceinline__ void get(At at, int off, CT* f) const
    {
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            const V v = *(const V*)((const char*)&w[j][off] + at.bw);
#pragma unroll
            for (int c = 0; c < PW; ++c) f[j * PW + c] = v[c];
        }
        if constexpr (REM != 0) f[NF - 1] = *(const CT*)((const char*)&r[off] + at.br);
    }
    __device__ __forceinline__ void put(int k, const CT* f)
    {
#pragma unroll
        for (int j = 0; j < NW; ++j) {
            V v;
#pragma unroll
            for (int c = 0; c < PW; ++c) v[c] = f[j * PW + c];
            w[j][k] = v;
        }
        if constexpr (REM != 0) r[k] = f[NF - 1];
    }
};

// Halo region of a tile, DH nodes deep: cell k -> mirror node index, wall
// offsets, crossings.  (Cells two and more beyond a wall or the open end, and
// inside the block behind its faces, hold values that no node uses.)
template <class Mo, int DIMV, int DH>
struct HaloN {
    static constexpr int D = DH;  // halo depth
    static constexpr int ZH = DIMV == 3 ? DH : 0;
    static constexpr int RX = Mo::TX + 2 * DH, RY = Mo::TY + 2 * DH, RZ = Mo::TZ + 2 * ZH;
    using R = Region<RX, RY, RZ>;
    static constexpr bool VEC = false;  // LDS cells are written one by one
    __device__ static __forceinline__ int slot(int k) { return k; }
    // BND: the tile touches a wall, the open end or the block (tiles that do
    // not never meet the block, and skip its test)
    template <bool BND = true>
    __device__ static __forceinline__ uint32_t cell(CDesc& cs, const TileCtx& t, int k, int off[3], int* cr)
    {
        const int ix = k % RX, iy = (k / RX) % RY, iz = k / (RX * RY);
        *cr = 0;
        int m[3];
        m[0] = resolve_axis(t.ox - DH + ix, cs.nx, cs.wall[0], &off[0], cr);
        m[1] = resolve_axis(t.oy - DH + iy, cs.ny, cs.wall[1], &off[1], cr);
        m[2] = resolve_axis(t.oz - ZH + iz, cs.nz, cs.wall[2], &off[2], cr);
        if (BND && in_block(cs, m[0], m[1], m[2])) {
            // a block node mirrors across each exposed face it lies on
            const int n[3] = {cs.nx, cs.ny, cs.nz};
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (m[a] == cs.blk_lo[a] && cs.blk_lo[a] >= 1) {
                    m[a] -= 1;
                    off[a] += 1;
                    *cr += 1;
                } else if (m[a] == cs.blk_hi[a] - 1 && cs.blk_hi[a] <= n[a] - 1) {
                    m[a] += 1;
                    off[a] -= 1;
                    *cr += 1;
                }
            }
        }
        return (uint32_t)m[0] + (uint32_t)cs.sx * ((uint32_t)m[1] + (uint32_t)cs.ny * (uint32_t)m[2]);
    }
};

template <class Mo, int DIMV> using Halo1 = HaloN<Mo, DIMV, 1>;

// 2-halo region of a tile on a grid without walls, open end or block and
// with every axis of at least 3 nodes, so that one +-n wraps a coordinate
// two nodes past either end.
template <class Mo, int DIMV>
struct Halo2 {
    static constexpr int D = 2;
    static constexpr int ZH = DIMV == 3 ? 2 : 0;
    static constexpr int RX = Mo::TX + 4, RY = Mo::TY + 4, RZ = Mo::TZ + 2 * ZH;
    using R = Region<RX, RY, RZ>;
    static constexpr bool VEC = false;
    __device__ static __forceinline__ int slot(int k) { return k; }
    template <bool BND = false>
    __device__ static __forceinline__ uint32_t cell(CDesc& cs, const TileCtx& t, int k, int off[3], int* cr)
    {
        static_assert(!BND, "periodic grids only");
        const int ix = k % RX, iy = (k / RX) % RY, iz = k / (RX * RY);
        *cr = 0;
        const int x = resolve_axis(t.ox - 2 + ix, cs.nx, 0, &off[0], cr);
        const int y = resolve_axis(t.oy - 2 + iy, cs.ny, 0, &off[1], cr);
        const int z = resolve_axis(t.oz - ZH + iz, cs.nz, 0, &off[2], cr);
        return (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)z);
    }
};

// The 1-halo region of a wide tile.  Its rows start at cell 3 of a pitch of 68
// in LDS (the last of a row's 66 cells takes the next row's unused first), so
// that a row's interior starts on 16 bytes (in 4-byte fields) and is written as
// the 4-element vectors it is read in.
struct HaloW : Halo1<WideTile, 3> {
    using B = Halo1<WideTile, 3>;
    struct R {
        static constexpr int PITCH = 68, N = PITCH * B::RY * B::RZ + 4;
        __device__ static __forceinline__ int idx(int ix, int iy, int iz) { return 3 + ix + PITCH * (iy + B::RY * iz); }
    };
    static constexpr bool VEC = true;
    __device__ static __forceinline__ int slot(int k)
    {
        return R::idx(k % B::RX, (k / B::RX) % B::RY, k / (B::RX * B::RY));
    }
};

// Fills a tile's halo region in LDS (HR: Halo1, or Halo2 two nodes deep)
// from NV arrays (src[j]: node-indexed array of CT).  store(k, cr, off, v)
// writes cell k from the NV values v of its node, with the crossing flags and
// wall offsets of HR::cell.
//
// A tile clear of walls, the open end and the block whose x range lies in the
// grid takes the row path: each halo row's TX interior cells are read as
// aligned 4-element vectors (tile origins and row pitches are multiples of 32
// nodes), its D end cells on either side one by one.  Only y and z wrap, once
// per row.
//
// Other tiles take the cell path: each thread takes the cells
// k = threadIdx.x + 256 it, resolves all of them and issues all their loads
// before the first LDS write, so they are in flight together.  Cells past the
// region repeat its last cell, and write it too, with the same values as its
// owner: control flow stays uniform, so no load is sunk into a conditional
// store.
//
// Tiles at a wall or the open end (WALL) take the row path too, as long as
// their halo region keeps clear of the block: a halo row beyond a wall or the
// open end is the mirror row (resolve_axis, with the row's offsets and
// crossings), and so is an end cell beyond a wall in x; the cells within a
// row share the row's y and z resolution.
template <class HR, bool WALL, int NV, class CT, bool FENCE, class StoreF>
__device__ __forceinline__ void halo_rows(CDesc& cs, const TileCtx& t, void* const* src, StoreF store)
{
    using R = typename HR::R;
    constexpr int DH = HR::D, TX = HR::RX - 2 * DH, ROWS = HR::RY * HR::RZ, LPR = TX / 4;
    constexpr int NVEC = ROWS * LPR, NEDGE = 2 * DH * ROWS;
    constexpr int PV = (NVEC + 255) / 256, PE = (NEDGE + 255) / 256;
    static_assert(TX % 4 == 0, "rows of 4-element vectors");
    typedef CT V4 __attribute__((ext_vector_type(4)));
    const int tid = (int)threadIdx.x;
    // node index of the start of halo row r, its first LDS cell, and (at
    // walls) the row's wall offsets and crossings
    auto row_of = [&](int r, int* kr, int* off, int* cr) {
        const int iy = r % HR::RY, iz = r / HR::RY;
        int y = t.oy - DH + iy, z = t.oz - HR::ZH + iz;
        off[0] = off[1] = off[2] = 0;
        *cr = 0;
        if constexpr (WALL) {
            y = resolve_axis(y, cs.ny, cs.wall[1], &off[1], cr);
            z = resolve_axis(z, cs.nz, cs.wall[2], &off[2], cr);
        } else {
            y += y < 0 ? cs.ny : (y >= cs.ny ? -cs.ny : 0);
            y = min(y, cs.ny - 1);
            z += z < 0 ? cs.nz : (z >= cs.nz ? -cs.nz : 0);
            z = min(z, cs.nz - 1);
        }
        *kr = R::idx(0, iy, iz);
        return (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)z);
    };
    // items past the last one repeat it (same loads, same LDS cells, same
    // values), so every load is unconditional and issued before any store
    V4 v[PV][NV];
    int kv[PV], crv[PV], offv[PV][3];
#pragma unroll
    for (int p = 0; p < PV; ++p) {
        const int it = min(tid + 256 * p, NVEC - 1);
        const int q = it % LPR;
        int kr;
        const uint32_t m = row_of(it / LPR, &kr, offv[p], &crv[p]) + (uint32_t)(t.ox + 4 * q);
        kv[p] = kr + DH + 4 * q;
#pragma unroll
        for (int j = 0; j < NV; ++j) v[p][j] = *(const PULBM_GLB V4*)at_node<CT>(src[j], m);
    }
    CT e[PE][NV];
    int ke[PE], cre[PE], offe[PE][3];
#pragma unroll
    for (int p = 0; p < PE; ++p) {
        const int it = min(tid + 256 * p, NEDGE - 1);
        const int side = it % (2 * DH);  // 0 .. DH-1 before the row, DH .. 2DH-1 after it
        int kr;
        const uint32_t row = row_of(it / (2 * DH), &kr, offe[p], &cre[p]);
        int x = side < DH ? t.ox - DH + side : t.ox + TX + side - DH;
        if constexpr (WALL) {
            x = resolve_axis(x, cs.nx, cs.wall[0], &offe[p][0], &cre[p]);
        } else {
            x += x < 0 ? cs.nx : (x >= cs.nx ? -cs.nx : 0);
            x = min(x, cs.nx - 1);
        }
        ke[p] = kr + (side < DH ? side : TX + side);
#pragma unroll
        for (int j = 0; j < NV; ++j) e[p][j] = *at_node<CT>(src[j], row + (uint32_t)x);
    }
    if constexpr (FENCE) __builtin_amdgcn_sched_barrier(0);  // every load issued, then the LDS writes
#pragma unroll
    for (int p = 0; p < PV; ++p) {
        if constexpr (HR::VEC) {
            store(kv[p], crv[p], offv[p], v[p]);
            continue;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            CT w[NV];
#pragma unroll
            for (int j = 0; j < NV; ++j) w[j] = v[p][j][c];
            store(kv[p] + c, crv[p], offv[p], w);
        }
    }
#pragma unroll
    for (int p = 0; p < PE; ++p) store(ke[p], cre[p], offe[p], e[p]);
}

// Does the halo region of a tile reach a node of the block?
template <class HR>
__device__ __forceinline__ bool halo_near_block(CDesc& cs, const TileCtx& t)
{
    constexpr int DH = HR::D, TX = HR::RX - 2 * DH, TY = HR::RY - 2 * DH, TZ = HR::RZ - 2 * HR::ZH;
    return cs.has_block && t.ox - DH < cs.blk_hi[0] && t.ox + TX + DH > cs.blk_lo[0] &&
           t.oy - DH < cs.blk_hi[1] && t.oy + TY + DH > cs.blk_lo[1] && t.oz - HR::ZH < cs.blk_hi[2] &&
           t.oz + TZ + HR::ZH > cs.blk_lo[2];
}

template <class HR, bool WALL, int NV, class CT, bool FENCE = false, class StoreF>
__device__ __forceinline__ void halo_stage(CDesc& cs, const TileCtx& t, void* const* src, StoreF store)
{
    if (t.ox + HR::RX - 2 * HR::D <= cs.nx) {
        if constexpr (!WALL) {
            halo_rows<HR, false, NV, CT, FENCE>(cs, t, src, store);
            return;
        } else {
            if (!halo_near_block<HR>(cs, t)) {
                halo_rows<HR, true, NV, CT, FENCE>(cs, t, src, store);
                return;
            }
        }
    }
    constexpr int RN = HR::RX * HR::RY * HR::RZ;
    // all loads of up to 5 cells a thread before their LDS writes
    constexpr int NIT = (RN + 255) / 256, STEP = NIT < 5 ? NIT : 5;
#pragma unroll 1
    for (int i0 = 0; i0 < NIT; i0 += STEP) {
        CT v[STEP][NV];
        int cr[STEP], off[STEP][3];
#pragma unroll
        for (int it = 0; it < STEP; ++it) {
            const int k = min((int)threadIdx.x + 256 * (i0 + it), RN - 1);
            const uint32_t m = HR::template cell<WALL>(cs, t, k, off[it], &cr[it]);
#pragma unroll
            for (int j = 0; j < NV; ++j) v[it][j] = *at_node<CT>(src[j], m);
        }
#pragma unroll
        for (int it = 0; it < STEP; ++it)
            store(HR::slot(min((int)threadIdx.x + 256 * (i0 + it), RN - 1)), cr[it], off[it], v[it]);
    }
}

// ------------------------------------------------------------ physics

template <class CT> __device__ __forceinline__ CT rcp(CT x) { return (CT)1 / x; }
template <> __device__ __forceinline__ float rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <class CT> __device__ __forceinline__ CT sqrt_(CT x) { return sqrt(x); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
template <> __device__ __forceinline__ float sqrt_<float>(float x) { return __builtin_amdgcn_sqrtf(x); }

template <class CT>
struct Phys {
    CT rho_a, drho, tau_a, dtau, inv_tau_phi;
    CT theta0;   // M / (T W)
    CT sig48W;   // 48 sigma / W
    CT sigW15;   // 3 sigma W / 2
    CT lambda_b;
    CT grav[3];
    int delta_theta;
};

// A case constant in the compute type: the host's FP32 copy for FP32
// arithmetic, the FP64 value otherwise.
template <class CT> __device__ __forceinline__ CT cconst(double d, float f)
{
    if constexpr (std::is_same_v<CT, float>) return f;
    else return (CT)d;
}

template <class CT>
__device__ __forceinline__ Phys<CT> make_phys(CDesc& cs)
{
    Phys<CT> p;
    p.rho_a = cconst<CT>(cs.rho_a, cs.f32.rho_a);
    p.drho = cconst<CT>(cs.rho_w - cs.rho_a, cs.f32.drho);
    p.tau_a = cconst<CT>(cs.tau_a, cs.f32.tau_a);
    p.dtau = cconst<CT>(cs.tau_w - cs.tau_a, cs.f32.dtau);
    p.inv_tau_phi = cconst<CT>(cs.inv_tau_phi, cs.f32.inv_tau_phi);
    p.theta0 = cconst<CT>(cs.theta0, cs.f32.theta0);
    p.sig48W = cconst<CT>(cs.sig48W, cs.f32.sig48W);
    p.sigW15 = cconst<CT>(cs.sigW15, cs.f32.sigW15);
    p.lambda_b = cconst<CT>(cs.lambda_b, cs.f32.lambda_b);
#pragma unroll
    for (int a = 0; a < 3; ++a) p.grav[a] = cconst<CT>(cs.grav[a], cs.f32.grav[a]);
    p.delta_theta = cs.delta_theta;
    return p;
}

template <class CT> __device__ __forceinline__ CT clamp01(CT v) { return v < (CT)0 ? (CT)0 : (v > (CT)1 ? (CT)1 : v); }

// Local macroscopic values and gradients of one node.
template <class CT>
struct NodeVals {
    CT phi, u[3], gphi[3], lphi, grho[3];
    // of the velocity gradients G_ab = d u_a / d x_b: div u, 2 G_aa, and
    // G_01 + G_10, G_02 + G_20, G_12 + G_21
    CT div, G2[3], Gs[3];
};

// Macroscopic part of the collision of one node (everything but the
// per-direction loops): phase-field theta and normal, hydrodynamic force,
// first moment of g^eq, B div u and the non-equilibrium momentum flux Pi.
template <int DIMV, class CT>
struct NodeCoef {
    CT theta, nv[3];     // phase field
    CT base_h;           // 1 - u^2 / (2T)
    CT rho, F[3];        // for the wall correction
    CT av[3];            // u + F / rho + sigma . grad rho / rho^2
    CT gbase;            // B div / T - u^2 / (2T)
    CT Bdiv;
    // (1 - 1/tau) / (2 T^2) * Pi: its diagonal, twice its off-diagonal
    // entries (xy, xz, yz), and * T tr(Pi)
    CT kPi[3], kPi2[3], kTr;
};

template <int DIMV, bool INIT, class CT>
__device__ __forceinline__ NodeCoef<DIMV, CT> node_coef(const Phys<CT>& p, const NodeVals<CT>& v,
                                                        const CT* __restrict__ M2)
{
    constexpr int D = DIMV;
    const CT T = (CT)kT, i2T2 = (CT)4.5, i2T = (CT)1.5, iT = (CT)3.0;
    const CT eps = (CT)1.0e-10;
    NodeCoef<DIMV, CT> k;
    const CT phi = v.phi;
    // phase field: normal, theta (+ delta theta)
    CT gn2 = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) gn2 += v.gphi[a] * v.gphi[a];
    const CT gn = sqrt_(gn2);
    const CT inv_n = rcp(gn + eps);
#pragma unroll
    for (int a = 0; a < 3; ++a) k.nv[a] = a < D ? v.gphi[a] * inv_n : (CT)0;
    const CT dphi = phi - (CT)0.5;
    CT theta = p.theta0 * ((CT)1 - (CT)4 * dphi * dphi);
    if (p.delta_theta) {
        const CT s = v.lphi * rcp(fabs(v.lphi) + eps);
        const CT iD = (CT)1.0e4;
        const CT Y1 = fmin(clamp01((phi - (CT)0.8) * iD), clamp01(-(phi - (CT)1) * iD));
        const CT Y2 = fmin(clamp01(phi * iD), clamp01(-(phi - (CT)0.2) * iD));
        theta += (CT)(-22.5) * p.theta0 * gn * (((CT)1 + s) * Y1 + ((CT)1 - s) * Y2);
    }
    k.theta = theta;
    CT u2 = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) u2 += v.u[a] * v.u[a];
    k.base_h = (CT)1 - u2 * i2T;
    // hydrodynamics
    const CT pc = clamp01(phi);
    const CT rho = p.rho_a + pc * p.drho;
    const CT tau = p.tau_a + pc * p.dtau;
    const CT nu = T * (tau - (CT)0.5);
    const CT mu = p.sig48W * phi * (phi - (CT)1) * dphi - p.sigW15 * v.lphi;
    const CT irho = rcp(rho);
    k.rho = rho;
#pragma unroll
    for (int a = 0; a < 3; ++a) k.F[a] = a < D ? rho * p.grav[a] + mu * v.gphi[a] : (CT)0;
    const CT div = v.div;
    const CT bulk = rho * (CT)(2.0 / 3.0) * (p.lambda_b - nu) * div;
    const CT rnu = rho * nu;
#pragma unroll
    for (int l = 0; l < 3; ++l) {
        if (l >= D) { k.av[l] = 0; continue; }
        CT sg = 0;
#pragma unroll
        for (int m = 0; m < D; ++m) {
            CT s_lm = rnu * (l == m ? v.G2[l] : v.Gs[l + m - 1]);
            if (l == m) s_lm += bulk;
            sg += s_lm * v.grho[m];
        }
        k.av[l] = v.u[l] + (k.F[l] + sg * irho) * irho;
    }
    const CT B = (CT)(2.0 / 3.0) * (nu - p.lambda_b) + T * (CT)0.5;
    k.Bdiv = B * div;
    k.gbase = k.Bdiv * iT - u2 * i2T;
#pragma unroll
    for (int a = 0; a < 3; ++a) k.kPi[a] = k.kPi2[a] = 0;
    k.kTr = 0;
    if (!INIT) {
        // Pi = sum c c (g - g^eq) = M2 - (u u + B div I) on these lattices;
        // diagonal entries, then xy, xz, yz (M2 holds xx, yy, [zz,] xy[, xz, yz])
        CT Pd[3] = {0, 0, 0}, Po[3] = {0, 0, 0};
#pragma unroll
        for (int a = 0; a < D; ++a) Pd[a] = M2[a] - v.u[a] * v.u[a] - k.Bdiv;
        Po[0] = M2[D] - v.u[0] * v.u[1];
        if (D == 3) {
            Po[1] = M2[4] - v.u[0] * v.u[2];
            Po[2] = M2[5] - v.u[1] * v.u[2];
        }
        const CT kf = ((CT)1 - rcp(tau)) * i2T2;
        CT tr = Pd[0];
#pragma unroll
        for (int a = 1; a < D; ++a) tr += Pd[a];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            k.kPi[a] = kf * Pd[a];
            k.kPi2[a] = (kf + kf) * Po[a];
        }
        k.kTr = kf * T * tr;
    }
    return k;
}

// c_i . x over the axes where direction j of lattice L is nonzero, started
// from the first such term: an accumulator started at zero costs one more
// add per sum (0 + x is not x when x is -0, so the compiler keeps the add).
template <class L, int D, class CT>
__device__ __forceinline__ CT c_dot(int j, const CT* x)
{
    CT s = 0;
    bool first = true;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const int c = L::c(j, a);
        if (c == 0) continue;
        s = first ? (c == 1 ? x[a] : -x[a]) : (c == 1 ? s + x[a] : s - x[a]);
        first = false;
    }
    return s;
}

// h^eq_j (INIT) or the BGK post-collision h*_j from the incoming h_j.
template <class H, int D, bool INIT, class CT>
__device__ __forceinline__ CT h_out(const Phys<CT>& p, const NodeVals<CT>& v, const NodeCoef<D, CT>& k, int j,
                                    CT hj)
{
    const CT cu = c_dot<H, D>(j, v.u), cn = c_dot<H, D>(j, k.nv);
    const CT wj = (CT)H::w(j);
    const CT heq = wj * (v.phi * (k.base_h + cu * (CT)3.0 + cu * cu * (CT)4.5) + k.theta * cn);
    return INIT ? heq : hj + (heq - hj) * p.inv_tau_phi;
}

// The part of g^eq_i (INIT) or of the filtered g*_i that is even in c_i,
// before the weight: 4.5 (c_i.u)^2 + B div u / T - u^2 / (2T), and when
// filtered c_i.kPi.c_i - T tr(kPi).  c_i.kPi.c_i is summed as the diagonal
// entries of the axes c_i spans, then the off-diagonal ones (kPi2 = 2 kPi),
// so that directions spanning the same axes share one diagonal sum.
template <class G, int D, bool INIT, class CT>
__device__ __forceinline__ CT g_even(const NodeCoef<D, CT>& k, int i, CT cu)
{
    CT e = k.gbase;
    if (!INIT) {
        e = e - k.kTr;
#pragma unroll
        for (int a = 0; a < D; ++a)
            if (G::c(i, a) != 0) e = e + k.kPi[a];
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int b = a + 1; b < D; ++b) {
                const int cc = G::c(i, a) * G::c(i, b);
                const CT p2 = k.kPi2[a + b - 1];  // (0,1) -> 0, (0,2) -> 1, (1,2) -> 2
                if (cc == 1) e = e + p2;
                if (cc == -1) e = e - p2;
            }
    }
    return cu * cu * (CT)4.5 + e;
}

// g^eq_i (INIT) or the filtered post-collision g*_i; the rest entry excludes
// the P / (rho_ref T) part.
template <class G, int D, bool INIT, class CT>
__device__ __forceinline__ CT g_out(const NodeVals<CT>& v, const NodeCoef<D, CT>& k, int i)
{
    const CT wi = (CT)G::w(i);
    const CT ca = c_dot<G, D>(i, k.av), cu = c_dot<G, D>(i, v.u);
    CT geq = wi * (g_even<G, D, INIT>(k, i, cu) + ca * (CT)3.0);
    if (i == 0) geq -= k.Bdiv * (CT)3.0;
    return geq;
}

// Opposite directions i and i+1 (i odd) have c_{i+1} = -c_i: the terms odd in
// c change sign and the even ones do not, so each pair shares one evaluation.
// The products of the weight with per-node values (w phi, w theta, ...) are
// written alike in every pair, so directions of one weight share them.
// h^eq (INIT) or the BGK post-collision h* for the pair (j, j+1).
template <class H, int D, bool INIT, class CT>
__device__ __forceinline__ void h_pair(const Phys<CT>& p, const NodeVals<CT>& v, const NodeCoef<D, CT>& k,
                                       int j, CT hj, CT hk, CT* oj, CT* ok)
{
    const CT cu = c_dot<H, D>(j, v.u), cn = c_dot<H, D>(j, k.nv);
    const CT pw = (CT)H::w(j) * v.phi;
    const CT even = cu * cu * (pw * (CT)4.5) + pw * k.base_h;
    const CT odd = cu * (pw * (CT)3.0) + ((CT)H::w(j) * k.theta) * cn;
    const CT ej = even + odd, ek = even - odd;
    *oj = INIT ? ej : hj + (ej - hj) * p.inv_tau_phi;
    *ok = INIT ? ek : hk + (ek - hk) * p.inv_tau_phi;
}

// g^eq (INIT) or the filtered post-collision g* for the pair (i, i+1).
template <class G, int D, bool INIT, class CT>
__device__ __forceinline__ void g_pair(const NodeVals<CT>& v, const NodeCoef<D, CT>& k, int i, CT* oi, CT* ok)
{
    const CT wi = (CT)G::w(i);
    const CT ca = c_dot<G, D>(i, k.av), cu = c_dot<G, D>(i, v.u);
    const CT we = wi * g_even<G, D, INIT>(k, i, cu);
    const CT w3 = wi * (CT)3.0;
    *oi = ca * w3 + we;
    *ok = we - ca * w3;
}

template <class Mo>
__device__ __forceinline__ void local_xyz(int* lx, int* ly, int* lz)
{
    *lx = threadIdx.x % Mo::TX;
    *ly = (threadIdx.x / Mo::TX) % Mo::TY;
    *lz = threadIdx.x / (Mo::TX * Mo::TY);
}

// ================================================================ kernels

// phi of this node one step earlier: the reference of the incoming h in
// 2-byte storage (wider storage keeps h as it is and reads nothing).
template <class S, class CT = typename Codec<S>::CT>
__device__ __forceinline__ CT h_reference(void* phi_prev, uint32_t n)
{
    if constexpr (sizeof(S) == 2) return __builtin_nontemporal_load(at_node<CT>(phi_prev, n));
    else return (CT)0;
}

// Shifts of the 2-byte codecs: a population is stored less the part of its
// equilibrium that the node reading it rebuilds from its own values of the
// step before: w_j phi for h, w_i c_i.u / T for g (T = 1/3).  Writer and
// reader evaluate one expression on the same FP32 values, so the reader's
// decode of a value equals the writer's own decode of it.
template <class CT> __device__ __forceinline__ CT g_shift(CT w, CT cu) { return (w * (CT)3) * cu; }
// shift of an incoming g_i read by a node whose previous-step velocity is u
template <class G, int D, class CT>
__device__ __forceinline__ CT g_ref(int i, const CT* u)
{
    return g_shift((CT)G::w(i), c_dot<G, D>(i, u));
}

// previous-step velocity of node n in 2-byte storage (wider storage: zero, unread)
template <class S, int D, class CT = typename Codec<S>::CT>
__device__ __forceinline__ void u_reference(void* u_prev, int64_t N, uint32_t n, CT* ur)
{
#pragma unroll
    for (int a = 0; a < 3; ++a) ur[a] = 0;
    if constexpr (sizeof(S) == 2) {
        const Slots<CT> Up = slots<CT>(u_prev, N);
#pragma unroll
        for (int a = 0; a < D; ++a) ur[a] = __builtin_nontemporal_load(Up.at(a, n * (uint32_t)sizeof(CT)));
    }
}

// --- moments: phi, u* = sum g c, P*, M2 (per node; no halo).  NTL: the
// population loads stream past L2 (non-temporal); odd is the step parity,
// a constant in every instantiation the kernel calls.
template <int LS, class S, bool WALL, bool NTL>
__device__ __forceinline__ void moments_node(CDesc& cs, int x, int y, int z, bool odd)
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using G = typename Mo::G;
    using H = typename Mo::H;
    using CT = typename Codec<S>::CT;
    const uint32_t n = (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)z);
    const uint32_t nb = n * (uint32_t)sizeof(S);
    const Nav nv = make_nav(cs, x, y, z, (int)sizeof(S));
    constexpr bool PAIRED = sizeof(S) != 4 || DIMV == 2;
    const Slots<S, PAIRED> hs = slots<S, PAIRED>(cs.h, cs.N), gs = slots<S, PAIRED>(cs.g, cs.N);
    const CT hsc = cconst<CT>(cs.h_inv_scale, cs.f32.h_inv_scale), gsc = cconst<CT>(cs.g_inv_scale, cs.f32.g_inv_scale);
    // 2-byte storage holds the populations less shifts made of phi (h) and
    // u (g) of this node one step earlier
    const CT php = h_reference<S>(cs.phi[odd ? 0 : 1], n);
    CT ur[3];
    u_reference<S, DIMV>(cs.U[odd ? 0 : 1], cs.N, n, ur);
    CT phi = 0;
#pragma unroll
    for (int j = 0; j < H::Q; ++j)
        phi += Codec<S>::dec(aa_load<H, WALL, NTL>(hs, nb, nv, j, odd), hsc,
                             php * (CT)H::w(j));
    CT sum = 0, J[3] = {0, 0, 0}, m2[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < G::Q; ++i) {
        const CT f = Codec<S>::dec(aa_load<G, WALL, NTL>(gs, nb, nv, i, odd), gsc,
                                   g_ref<G, DIMV>(i, ur));
        sum += f;
#pragma unroll
        for (int a = 0; a < DIMV; ++a) {
            if (G::c(i, a) == 1) J[a] += f;
            if (G::c(i, a) == -1) J[a] -= f;
        }
        if (i != 0) {
#pragma unroll
            for (int a = 0; a < DIMV; ++a)
                if (G::c(i, a) != 0) m2[a] += f;  // c_a^2 = 1
            if (DIMV == 2) {
                const int xy = G::c(i, 0) * G::c(i, 1);
                if (xy) m2[2] += xy > 0 ? f : -f;
            } else {
                const int xy = G::c(i, 0) * G::c(i, 1), xz = G::c(i, 0) * G::c(i, 2),
                          yz = G::c(i, 1) * G::c(i, 2);
                if (xy) m2[3] += xy > 0 ? f : -f;
                if (xz) m2[4] += xz > 0 ? f : -f;
                if (yz) m2[5] += yz > 0 ? f : -f;
            }
        }
    }
    const uint32_t na = n * (uint32_t)sizeof(CT);
    // the moment fields are written once and read by the next kernels after
    // the whole grid has been written: stored non-temporal (FP16 moments 3%
    // faster, the kernels reading them unchanged)
    __builtin_nontemporal_store(phi, at_node<CT>(cs.phi[odd ? 1 : 0], n));
    const Slots<CT> Js = slots<CT>(cs.J, cs.N);
#pragma unroll
    for (int a = 0; a < DIMV; ++a) __builtin_nontemporal_store(J[a], Js.at(a, na));
    using AT = CT;
    const double Pprev = (double)__builtin_nontemporal_load(at_node<AT>(cs.P[odd ? 1 : 0], n));
    __builtin_nontemporal_store((AT)(Pprev + cs.rho_a * kT * (double)sum), at_node<AT>(cs.Ps, n));
    constexpr int NM = DIMV == 2 ? 3 : 6;
    if constexpr (sizeof(S) == 2) {
        const Slots<uint32_t> Ms = slots<uint32_t>(cs.M2, cs.N);
        const CT gsc_out = cconst<CT>(cs.g_scale, cs.f32.g_scale);
#pragma unroll
        for (int j = 0; j < (NM + 1) / 2; ++j) {
            const S lo = Codec<S>::enc(m2[2 * j], gsc_out, (CT)0);
            const S hi = 2 * j + 1 < NM ? Codec<S>::enc(m2[2 * j + 1], gsc_out, (CT)0) : (S)0;
            __builtin_nontemporal_store(pair_pack<S>(lo, hi), Ms.at(j, n * 4u));
        }
    } else {
        const Slots<CT> Ms = slots<CT>(cs.M2, cs.N);
#pragma unroll
        for (int k = 0; k < NM; ++k) __builtin_nontemporal_store(m2[k], Ms.at(k, na));
    }
}

template <int LS, class S>
__global__ __launch_bounds__(256) void k_moments(CaseTab cases, const int* hdr, int step_off)
{
    using Mo = Model<LS>;
    const TileCtx t = tile_ctx<Mo>(cases, hdr, step_off);
    if (!t.active) return;
    CDesc& cs = *t.cs;
    int lx, ly, lz;
    local_xyz<Mo>(&lx, &ly, &lz);
    const int x = t.ox + lx, y = t.oy + ly, z = t.oz + lz;
    if (x >= cs.nx || y >= cs.ny || z >= cs.nz) return;
    const bool odd = t.step & 1;
    constexpr bool nt_odd = nt_access<S, kLoadMoments>();
    constexpr bool nt_even = nt_odd || nt_access<S, kLoadMomentsEven>();
    constexpr bool nt_odd_wide = !nt_odd && sizeof(S) >= 4;
    if (tile_at_wall<Mo>(cs, t.ox, t.oy, t.oz)) {
        if (in_block(cs, x, y, z)) {
            // block nodes carry no fluid: phi, u*, P*, M2 = 0
            using CT = typename Codec<S>::CT;
            constexpr int DIMV = Model<LS>::DIM;
            const uint32_t n = (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)z);
            const uint32_t na = n * (uint32_t)sizeof(CT);
            *at_node<CT>(cs.phi[odd ? 1 : 0], n) = 0;
            *at_node<CT>(cs.Ps, n) = 0;
            const Slots<CT> Js = slots<CT>(cs.J, cs.N);
#pragma unroll
            for (int a = 0; a < DIMV; ++a) *Js.at(a, na) = 0;
            constexpr int NM = DIMV == 2 ? 3 : 6;
            if constexpr (sizeof(S) == 2) {
                const Slots<uint32_t> Ms = slots<uint32_t>(cs.M2, cs.N);
#pragma unroll
                for (int j = 0; j < (NM + 1) / 2; ++j) *Ms.at(j, n * 4u) = 0u;  // +0 in both halves
            } else {
                const Slots<CT> Ms = slots<CT>(cs.M2, cs.N);
#pragma unroll
                for (int k = 0; k < NM; ++k) *Ms.at(k, na) = 0;
            }
            return;
        }
        if (!odd) moments_node<LS, S, true, nt_even>(cs, x, y, z, false);
        else if (nt_odd_wide && cs.nt_odd_moments) moments_node<LS, S, true, true>(cs, x, y, z, true);
        else moments_node<LS, S, true, nt_odd>(cs, x, y, z, true);
    } else {
        if (!odd) moments_node<LS, S, false, nt_even>(cs, x, y, z, false);
        else if (nt_odd_wide && cs.nt_odd_moments) moments_node<LS, S, false, true>(cs, x, y, z, true);
        else moments_node<LS, S, false, nt_odd>(cs, x, y, z, true);
    }
}

// --- pressure (Sec. II): P = rho_ref T sum_i (g_i + (1 + omega) K_i)
//     + omega rho_ref sum_i w_i c_i . u*(x - c_i), one evaluation of this
//     equation (which holds P on both sides, through K_i) started from the
//     pressure the streamed populations carry, P* = rho_ref T sum g: K_i from
//     P*.  Difference form: opposite links enter as
//     (P(x - c) - P0) + (P(x + c) - P0) and as u*(x - c) - u*(x + c), each
//     formed in the auxiliary type and so rounded relative to itself (the
//     single differences exact for P within a factor 2); the sums within a
//     shell are in the auxiliary type, the sum over shells and the final
//     combination FP64.
template <int LS, class AT, bool WALL, class R>
__device__ __forceinline__ void pressure_tile(CDesc& cs, const TileCtx& t, AT* sP, AT* sGD, AT (*sJ)[R::N])
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using G = typename Mo::G;
    using HR = Halo1<Mo, DIMV>;
    const Slots<AT> Js = slots<AT>(cs.J, cs.N);
    int lx, ly, lz;
    local_xyz<Mo>(&lx, &ly, &lz);
    const int x = t.ox + lx, y = t.oy + ly, z = t.oz + lz;
    const bool live = x < cs.nx && y < cs.ny && z < cs.nz;
    const uint32_t n = (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)z);
    // the node's own phi is loaded first, so its latency overlaps the halo's
    const AT phi = live ? __builtin_nontemporal_load(at_node<AT>(cs.phi[t.step & 1], n)) : (AT)0;
    void* src[1 + DIMV];
    src[0] = cs.Ps;
#pragma unroll
    for (int a = 0; a < DIMV; ++a) src[1 + a] = (void*)Js.at(a, 0);
    halo_stage<HR, WALL, 1 + DIMV, AT>(
        cs, t, src,
        [&](int k, int cr, const int* off, const AT* v) {
            AT p = v[0], gd = 0;
            // ghost pressure = P(mirror) + rho(x) g.(ghost - mirror): keep g.off;
            // beyond the open end 2 p_top - P(mirror), p_top half a link out
            if (WALL) gd = (AT)(cs.grav[0] * off[0] + cs.grav[1] * off[1] + cs.grav[2] * off[2]);
            if (WALL && (cr & kOpenGhost)) {
                p = (AT)(2.0 * cs.p_top - (double)p);
                gd = 0;
            }
            sP[k] = p;
            if (WALL) sGD[k] = gd;
#pragma unroll
            for (int a = 0; a < DIMV; ++a) {
                AT j = v[1 + a];
                // u* at a ghost: flow part odd, body-force part even
                if (WALL && (cr & 1)) j = (AT)(-(double)j + 2.0 * cs.grav[a]);
                sJ[a][k] = j;
            }
        });
    __syncthreads();
    if (!live) return;
    if (WALL && in_block(cs, x, y, z)) {
        *at_node<AT>(cs.P[(t.step + 1) & 1], n) = 0;
        return;
    }
    // omega = (rho - rho_ref) / rho_ref with omega_max = rho_w / rho_ref, so
    // (1 + omega) rho_ref / rho = 1 and omega rho_ref = rho - rho_ref, which
    // weights the u* term by up to the density ratio: the shell-weighted sums
    // and this combination are taken in FP64 (the per-shell sums below are in
    // the auxiliary type)
    const double drho = (double)clamp01(phi) * (cs.rho_w - cs.rho_a);
    const double rho = cs.rho_a + drho;
    const int kb = R::template nb_base<HR::ZH>(lx + 1, ly + 1, lz + HR::ZH);
    const AT P0 = sP[kb + R::template nb<HR::ZH>(0, 0, 0)];
    // The weight of a link depends on its shell alone, so the link terms are
    // summed per shell, unweighted, in the auxiliary type (a handful of terms
    // of one magnitude class, each a difference rounded relative to itself);
    // the weighted sum over shells and the combination are FP64.
    constexpr int NS = shell<G>(G::Q - 1) + 1;
    AT sks[NS], sgs[NS], dus[3][NS];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        sks[s] = sgs[s] = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) dus[a][s] = 0;
    }
#pragma unroll
    for (int i = 1; i < G::Q; i += 2) {  // pairs (i, i+1) are opposite
        const int s = shell<G>(i);
        const int km = kb + R::template nb<HR::ZH>(-G::c(i, 0), -G::c(i, 1), -G::c(i, 2));
        const int kp = kb + R::template nb<HR::ZH>(G::c(i, 0), G::c(i, 1), G::c(i, 2));
        // the pair's second difference of P
        sks[s] += (sP[km] - P0) + (sP[kp] - P0);
        if (WALL) sgs[s] += sGD[km] + sGD[kp];
#pragma unroll
        for (int a = 0; a < DIMV; ++a) {
            if (G::c(i, a) == 0) continue;
            const AT d = sJ[a][km] - sJ[a][kp];
            if (G::c(i, a) == 1) dus[a][s] += d;
            else dus[a][s] -= d;
        }
    }
    double sk = 0, sg = 0, su = 0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const double w = shell_w<G>(s);
        sk += w * (double)sks[s];
        if (WALL) sg += w * (double)sgs[s];
#pragma unroll
        for (int a = 0; a < DIMV; ++a) su += w * (double)dus[a][s];
    }
    if (WALL) sk += rho * sg;
    // rho_ref T (1 + omega) sum K = (1 + omega) rho_ref / rho * sum w dP = sk
    *at_node<AT>(cs.P[(t.step + 1) & 1], n) = (AT)((double)P0 + (sk + drho * su));
}

template <int LS, class AT>
__global__ __launch_bounds__(256) void k_pressure(CaseTab cases, const int* hdr, int step_off)
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using R = typename Halo1<Mo, DIMV>::R;
    __shared__ AT sP[R::N], sGD[R::N], sJ[DIMV][R::N];
    const TileCtx t = tile_ctx<Mo>(cases, hdr, step_off);
    if (!t.active) return;
    CDesc& cs = *t.cs;
    // a fused case's collide rebuilds P itself; the read pass (step_off < 0) still needs it here
    if (cs.fuse_u == 2 && step_off >= 0) return;
    if (tile_at_wall<Mo>(cs, t.ox, t.oy, t.oz)) pressure_tile<LS, AT, true, R>(cs, t, sP, sGD, sJ);
    else pressure_tile<LS, AT, false, R>(cs, t, sP, sGD, sJ);
}

// --- velocity: u = u* + sum_i K_i c_i with K_i of the new pressure.
template <int LS, class CT, bool WALL, class R>
__device__ __forceinline__ void velocity_tile(CDesc& cs, const TileCtx& t, CT* sP, CT* sGD)
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using G = typename Mo::G;
    using HR = Halo1<Mo, DIMV>;
    void* Pn = cs.P[(t.step + 1) & 1];
    int lx, ly, lz;
    local_xyz<Mo>(&lx, &ly, &lz);
    const int x = t.ox + lx, y = t.oy + ly, z = t.oz + lz;
    const bool live = x < cs.nx && y < cs.ny && z < cs.nz;
    const uint32_t n = (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)z);
    const uint32_t na = n * (uint32_t)sizeof(CT);
    // the node's own operands are loaded first, so their latency overlaps the halo's
    const Slots<CT> Js = slots<CT>(cs.J, cs.N), Us = slots<CT>(cs.U[t.step & 1], cs.N);
    CT phi = 0, J[3] = {0, 0, 0};
    if (live) {
        phi = __builtin_nontemporal_load(at_node<CT>(cs.phi[t.step & 1], n));
#pragma unroll
        for (int a = 0; a < DIMV; ++a) J[a] = __builtin_nontemporal_load(Js.at(a, na));
    }
    void* src[1] = {Pn};
    halo_stage<HR, WALL, 1, CT>(
        cs, t, src,
        [&](int k, int cr, const int* off, const CT* v) {
            CT p = v[0], gd = 0;
            if (WALL) gd = (CT)(cs.grav[0] * off[0] + cs.grav[1] * off[1] + cs.grav[2] * off[2]);
            if (WALL && (cr & kOpenGhost)) {
                p = (CT)(2.0 * cs.p_top - (double)p);
                gd = 0;
            }
            sP[k] = p;
            if (WALL) sGD[k] = gd;
        });
    __syncthreads();
    if (!live) return;
    if (WALL && in_block(cs, x, y, z)) {
#pragma unroll
        for (int a = 0; a < DIMV; ++a) *Us.at(a, na) = 0;
        return;
    }
    const CT ra = cconst<CT>(cs.rho_a, cs.f32.rho_a), dr = cconst<CT>(cs.rho_w - cs.rho_a, cs.f32.drho);
    const CT rho = ra + clamp01(phi) * dr;
    const CT irho = rcp(rho);
    const int kb = R::template nb_base<HR::ZH>(lx + 1, ly + 1, lz + HR::ZH);
    CT gr[3] = {0, 0, 0};
#pragma unroll
    for (int i = 1; i < G::Q; i += 2) {
        const int kp = kb + R::template nb<HR::ZH>(G::c(i, 0), G::c(i, 1), G::c(i, 2));
        const int km = kb + R::template nb<HR::ZH>(-G::c(i, 0), -G::c(i, 1), -G::c(i, 2));
        const CT d = (WALL ? (sP[kp] + rho * sGD[kp]) - (sP[km] + rho * sGD[km]) : sP[kp] - sP[km]) * (CT)G::w(i);
#pragma unroll
        for (int a = 0; a < DIMV; ++a) {
            if (G::c(i, a) == 1) gr[a] += d;
            if (G::c(i, a) == -1) gr[a] -= d;
        }
    }
#pragma unroll
    for (int a = 0; a < DIMV; ++a) *Us.at(a, na) = J[a] - gr[a] * (CT)3.0 * irho;
}

template <int LS, class CT>
__global__ __launch_bounds__(256) void k_velocity(CaseTab cases, const int* hdr, int step_off)
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using R = typename Halo1<Mo, DIMV>::R;
    __shared__ CT sP[R::N], sGD[R::N];
    const TileCtx t = tile_ctx<Mo>(cases, hdr, step_off);
    if (!t.active) return;
    CDesc& cs = *t.cs;
    // a fused case's collide rebuilds u itself; the read pass (step_off < 0) still needs it here
    if (cs.fuse_u && step_off >= 0) return;
    if (tile_at_wall<Mo>(cs, t.ox, t.oy, t.oz)) velocity_tile<LS, CT, true, R>(cs, t, sP, sGD);
    else velocity_tile<LS, CT, false, R>(cs, t, sP, sGD);
}

// --- pressure and velocity of large 3D cases in 4-byte fields: wide tiles, four
// nodes to a thread, one above the other in z (64 x 4 x 4 nodes).  k_pressure
// and k_velocity are bound by the issue of vector instructions (280 and 171 per
// wave and node, half of it addressing and halo work).  Here the halo is 2.3
// cells a node instead of 4.1, its rows go to LDS as vectors, and a thread
// slides a 3x3x3 window up its column, which reads 13.5 cells a node from LDS
// instead of 27 (186 and 104 instructions).  The arithmetic of a node is
// k_pressure's and k_velocity's, term by term.  512x256x256 dam break:
// pressure 313 -> 241 us (3.8 TB/s; its FP64 sums and 12 LDS words a cell keep
// it from the copy's 6.3), velocity 227 -> 179 us (6.0 TB/s).  LDS and registers
// hold 4 workgroups per CU in pressure (at 3: 264 us) and registers 6 in velocity.
// Pressure on D3Q27 hydro takes all 128 registers of its 4 waves and spills one
// on the wall path: 4.2 instead of 4.0 bytes written a node there.

// f of a value, or of each element of a vector of them.
template <class T, class F> __device__ __forceinline__ T each(T v, F f)
{
    if constexpr (std::is_arithmetic_v<T>) {
        return f(v);
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = f(v[c]);
        return v;
    }
}
template <class T, class CT> __device__ __forceinline__ void lds_put(CT* s, int k, T v) { *(T*)(s + k) = v; }

// Three planes of 3x3 cells of an LDS field around a column of a wide tile,
// plane p of the column (its first node at p = 1) in slot p % 3.  The planes are
// read in order through one LDS address, hidden from the compiler: it would
// read them all at once (200 registers), and pair reads through addresses of
// their own.
template <class CT> struct Window {
    const __attribute__((address_space(3))) CT* next;
    CT v[3][9];
    __device__ __forceinline__ void start(const CT* s, int lx, int ly)
    {
        next = (const __attribute__((address_space(3))) CT*)(s + HaloW::R::idx(lx, ly, 0));
    }
    __device__ __forceinline__ void load(int p)
    {
        asm volatile("" : "+v"(next));
#pragma unroll
        for (int n = 0; n < 9; ++n) v[p % 3][n] = next[n % 3 + HaloW::R::PITCH * (n / 3)];
        next += HaloW::R::PITCH * HaloW::RY;
    }
    // the cell at (dx, dy, dz) from node q of the column
    __device__ __forceinline__ CT at(int q, int dx, int dy, int dz) const
    {
        return v[(q + 1 + dz) % 3][1 + dx + 3 * (1 + dy)];
    }
};

// The hydrostatic part of P at the cells around a column's nodes, in a tile at
// a wall and clear of the block: g . (ghost - mirror), 0 inside the grid and
// beyond an open end.  Formed where it is used: kept in LDS it would cost the
// fourth workgroup per CU, kept in registers the fourth wave.
template <class CT> struct Ghosts {
    double gx[2], gy[2], gz[2];
    bool open;
    __device__ __forceinline__ void column(CDesc& cs, int x, int y)
    {
        gx[0] = cs.wall[0] && x == 0 ? -cs.grav[0] : 0.0;
        gx[1] = cs.wall[0] && x == cs.nx - 1 ? cs.grav[0] : 0.0;
        gy[0] = cs.wall[1] && y == 0 ? -cs.grav[1] : 0.0;
        gy[1] = cs.wall[1] && y == cs.ny - 1 ? cs.grav[1] : 0.0;
    }
    __device__ __forceinline__ void node(CDesc& cs, int z)
    {
        gz[0] = cs.wall[2] && z == 0 ? -cs.grav[2] : 0.0;
        gz[1] = cs.wall[2] && z == cs.nz - 1 ? cs.grav[2] : 0.0;
        open = cs.wall[2] == 2 && z == cs.nz - 1;
    }
    __device__ __forceinline__ CT at(int dx, int dy, int dz) const
    {
        double g = dx < 0 ? gx[0] : (dx > 0 ? gx[1] : 0.0);
        if (dy != 0) g = g + (dy < 0 ? gy[0] : gy[1]);
        if (dz != 0) g = g + (dz < 0 ? gz[0] : gz[1]);
        return dz > 0 && open ? (CT)0 : (CT)g;
    }
};

template <int LS, class AT, bool WALL>
__device__ __forceinline__ void pressure_wide(CDesc& cs, const TileCtx& t, AT* sP, AT (*sJ)[HaloW::R::N])
{
    using G = typename Model<LS>::G;
    using W = WideTile;
    const Slots<AT> Js = slots<AT>(cs.J, cs.N);
    const int lx = threadIdx.x % W::TX, ly = threadIdx.x / W::TX;
    const int x = t.ox + lx, y = t.oy + ly;
    const uint32_t n0 = (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)t.oz);
    const uint32_t pl = (uint32_t)cs.sx * (uint32_t)cs.ny;
    const bool col = x < cs.nx && y < cs.ny;
    // the nodes' own phi is loaded first, so its latency overlaps the halo's
    AT phi[W::TZ];
#pragma unroll
    for (int q = 0; q < W::TZ; ++q)
        phi[q] = col && t.oz + q < cs.nz ? __builtin_nontemporal_load(at_node<AT>(cs.phi[t.step & 1], n0 + q * pl)) : (AT)0;
    void* src[4] = {cs.Ps, (void*)Js.at(0, 0), (void*)Js.at(1, 0), (void*)Js.at(2, 0)};
    halo_stage<HaloW, WALL, 4, AT>(cs, t, src, [&](int k, int cr, const int*, const auto* v) {
        auto p = v[0];
        if (WALL && (cr & kOpenGhost)) p = each(p, [&](AT q) { return (AT)(2.0 * cs.p_top - (double)q); });
        lds_put(sP, k, p);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            auto j = v[1 + a];
            if (WALL && (cr & 1)) j = each(j, [&](AT q) { return (AT)(-(double)q + 2.0 * cs.grav[a]); });
            lds_put(sJ[a], k, j);
        }
    });
    __syncthreads();
    if (!col) return;
    Window<AT> wP, wJ[3];
    Ghosts<AT> gd;
    wP.start(sP, lx, ly);
#pragma unroll
    for (int a = 0; a < 3; ++a) wJ[a].start(sJ[a], lx, ly);
    if (WALL) gd.column(cs, x, y);
    auto plane = [&](int p) {
        wP.load(p);
#pragma unroll
        for (int a = 0; a < 3; ++a) wJ[a].load(p);
    };
    plane(0);
    plane(1);
    constexpr int NS = shell<G>(G::Q - 1) + 1;
#pragma unroll
    for (int q = 0; q < W::TZ; ++q) {
        plane(q + 2);
        const int z = t.oz + q;
        if (WALL) gd.node(cs, z);
        const double drho = (double)clamp01(phi[q]) * (cs.rho_w - cs.rho_a);
        const double rho = cs.rho_a + drho;
        const AT P0 = wP.at(q, 0, 0, 0);
        AT sks[NS], sgs[NS], dus[3][NS];
#pragma unroll
        for (int s = 0; s < NS; ++s) sks[s] = sgs[s] = dus[0][s] = dus[1][s] = dus[2][s] = 0;
#pragma unroll
        for (int i = 1; i < G::Q; i += 2) {  // pairs (i, i+1) are opposite
            const int s = shell<G>(i), cx = G::c(i, 0), cy = G::c(i, 1), cz = G::c(i, 2);
            sks[s] += (wP.at(q, -cx, -cy, -cz) - P0) + (wP.at(q, cx, cy, cz) - P0);
            if (WALL) sgs[s] += gd.at(-cx, -cy, -cz) + gd.at(cx, cy, cz);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (G::c(i, a) == 0) continue;
                const AT d = wJ[a].at(q, -cx, -cy, -cz) - wJ[a].at(q, cx, cy, cz);
                if (G::c(i, a) == 1) dus[a][s] += d;
                else dus[a][s] -= d;
            }
        }
        double sk = 0, sg = 0, su = 0;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const double w = shell_w<G>(s);
            sk += w * (double)sks[s];
            if (WALL) sg += w * (double)sgs[s];
#pragma unroll
            for (int a = 0; a < 3; ++a) su += w * (double)dus[a][s];
        }
        if (WALL) sk += rho * sg;
        AT P = (AT)((double)P0 + (sk + drho * su));
        asm volatile("" : "+v"(P));
        if (z < cs.nz) *at_node<AT>(cs.P[(t.step + 1) & 1], n0 + q * pl) = P;
    }
}

template <int LS, class AT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_pressure_wide(CaseTab cases, int step_off)
{
    using R = HaloW::R;
    using S = typename Halo1<Model<LS>, 3>::R;
    __shared__ __align__(16) AT sP[R::N], sJ[3][R::N];
    static_assert(2 * S::N <= R::N, "a sub-tile's fields fit");
    bool sub;
    const TileCtx t = wide_ctx<Model<LS>>(cases, step_off, &sub);
    if (!t.active) return;
    CDesc& cs = *t.cs;
    if (sub) pressure_tile<LS, AT, true, S>(cs, t, sP, sP + S::N, (AT(*)[S::N])sJ);
    else if (halo_near_block<HaloW>(cs, t)) return;
    else if (tile_at_wall<WideTile>(cs, t.ox, t.oy, t.oz)) pressure_wide<LS, AT, true>(cs, t, sP, sJ);
    else pressure_wide<LS, AT, false>(cs, t, sP, sJ);
}

template <int LS, class CT, bool WALL>
__device__ __forceinline__ void velocity_wide(CDesc& cs, const TileCtx& t, CT* sP)
{
    using G = typename Model<LS>::G;
    using W = WideTile;
    const Slots<CT> Js = slots<CT>(cs.J, cs.N), Us = slots<CT>(cs.U[t.step & 1], cs.N);
    const int lx = threadIdx.x % W::TX, ly = threadIdx.x / W::TX;
    const int x = t.ox + lx, y = t.oy + ly;
    const uint32_t n0 = (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)t.oz);
    const uint32_t pl = (uint32_t)cs.sx * (uint32_t)cs.ny;
    const bool col = x < cs.nx && y < cs.ny;
    // the nodes' own operands are loaded first, so their latency overlaps the halo's
    CT phi[W::TZ], J[W::TZ][3];
#pragma unroll
    for (int q = 0; q < W::TZ; ++q) {
        phi[q] = J[q][0] = J[q][1] = J[q][2] = 0;
        if (col && t.oz + q < cs.nz) {
            phi[q] = __builtin_nontemporal_load(at_node<CT>(cs.phi[t.step & 1], n0 + q * pl));
#pragma unroll
            for (int a = 0; a < 3; ++a) J[q][a] = __builtin_nontemporal_load(Js.at(a, (n0 + q * pl) * (uint32_t)sizeof(CT)));
        }
    }
    void* src[1] = {cs.P[(t.step + 1) & 1]};
    halo_stage<HaloW, WALL, 1, CT>(cs, t, src, [&](int k, int cr, const int*, const auto* v) {
        auto p = v[0];
        if (WALL && (cr & kOpenGhost)) p = each(p, [&](CT q) { return (CT)(2.0 * cs.p_top - (double)q); });
        lds_put(sP, k, p);
    });
    __syncthreads();
    if (!col) return;
    const CT ra = cconst<CT>(cs.rho_a, cs.f32.rho_a), dr = cconst<CT>(cs.rho_w - cs.rho_a, cs.f32.drho);
    Window<CT> wP;
    Ghosts<CT> gd;
    wP.start(sP, lx, ly);
    if (WALL) gd.column(cs, x, y);
    wP.load(0);
    wP.load(1);
#pragma unroll
    for (int q = 0; q < W::TZ; ++q) {
        wP.load(q + 2);
        const int z = t.oz + q;
        if (WALL) gd.node(cs, z);
        const uint32_t na = (n0 + q * pl) * (uint32_t)sizeof(CT);
        const CT rho = ra + clamp01(phi[q]) * dr;
        const CT irho = rcp(rho);
        CT gr[3] = {0, 0, 0};
#pragma unroll
        for (int i = 1; i < G::Q; i += 2) {
            const int cx = G::c(i, 0), cy = G::c(i, 1), cz = G::c(i, 2);
            const CT p = wP.at(q, cx, cy, cz), m = wP.at(q, -cx, -cy, -cz);
            const CT d = (WALL ? (p + rho * gd.at(cx, cy, cz)) - (m + rho * gd.at(-cx, -cy, -cz)) : p - m) * (CT)G::w(i);
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                if (G::c(i, a) == 1) gr[a] += d;
                if (G::c(i, a) == -1) gr[a] -= d;
            }
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) asm volatile("" : "+v"(gr[a]));
        if (z < cs.nz) {
#pragma unroll
            for (int a = 0; a < 3; ++a) *Us.at(a, na) = J[q][a] - gr[a] * (CT)3.0 * irho;
        }
    }
}

template <int LS, class CT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void k_velocity_wide(CaseTab cases, int step_off)
{
    using R = HaloW::R;
    using S = typename Halo1<Model<LS>, 3>::R;
    __shared__ __align__(16) CT sP[R::N];
    bool sub;
    const TileCtx t = wide_ctx<Model<LS>>(cases, step_off, &sub);
    if (!t.active) return;
    CDesc& cs = *t.cs;
    if (cs.fuse_u && step_off >= 0) return;
    if (sub) velocity_tile<LS, CT, true, S>(cs, t, sP, sP + S::N);
    else if (halo_near_block<HaloW>(cs, t)) return;
    else if (tile_at_wall<WideTile>(cs, t.ox, t.oy, t.oz)) velocity_wide<LS, CT, true>(cs, t, sP);
    else velocity_wide<LS, CT, false>(cs, t, sP);
}

// Fields of a cell of the collide and init tiles, in LDS order: phi, u, rho.
template <int DIMV> struct CellF {
    static constexpr int NF = DIMV + 2, PHI = 0, U = 1, RHO = DIMV + 1;
};

// Rounding of the gradient sums, written out so that a kernel's results do
// not depend on where the compiler places a product: it contracts a product
// into the sum only within one basic block, and the run-time parity and the
// BF16 codec split the collide into several.
// Which velocity-gradient terms add a product rounded on its own instead of
// contracting it (SPLIT 0: none, 1: d u_y / dz and d u_z / dy, 2: every
// off-diagonal component): terms of d u_a / d x_b along a direction i whose
// product another component takes first.
template <class G, int SPLIT> __host__ __device__ constexpr bool grad_split(int i, int a, int b)
{
    if (SPLIT == 0 || a < 0 || a >= G::DIM || a == b || G::c(i, b) == 0) return false;
    if (a > 0 && b > 0) return G::c(i, a) != 0 || G::c(i, 0) != 0;
    return SPLIT == 2 && G::c(i, a) != 0;
}
template <class S, bool WALL, bool BGK, int PAR> constexpr int grad_split_of()
{
    if (std::is_same_v<S, uint16_t>) return 2;
    return PAR == 1 && WALL ? (BGK ? 2 : 1) : 0;
}

// Isotropic central differences (Sec. II) of phi, rho and u at the cell whose
// 3x3(x3) neighbourhood starts at cell kb (R::nb_base):
// grad_a q = sum_i w_i c_ia (q(+c_i) - q(-c_i)) / (2T), lap q = 2 sum_i w_i (q(+c_i) - q0) / T.
template <int LS, class R, int ZH, int SPLIT, class C, class CT>
__device__ __forceinline__ void tile_gradients(const C& cells, typename C::At kb, NodeVals<CT>& v)
{
    constexpr int DIMV = Model<LS>::DIM;
    using G = typename Model<LS>::G;
    using F = CellF<DIMV>;
    CT q0[F::NF];
    cells.get(kb, R::template nb<ZH>(0, 0, 0), q0);
    v.phi = q0[F::PHI];
#pragma unroll
    for (int a = 0; a < 3; ++a) v.u[a] = a < DIMV ? q0[F::U + a] : (CT)0;
    CT gr[F::NF][3], l = 0;
#pragma unroll
    for (int f = 0; f < F::NF; ++f) gr[f][0] = gr[f][1] = gr[f][2] = 0;
    // The reads of a pair are issued AHEAD pairs before its sums, and no
    // sooner: the sums are pinned in order and the reads' address depends on
    // the last pin.  Left to itself the compiler issues all 26 neighbours'
    // reads first, which alone takes 130 registers (the FP16 D3Q27 collide then
    // needs 153-168; with 2 pairs ahead 75 on even and 106 on odd steps; 1 pair
    // ahead is 1-5% slower, 3 and more no faster).
    constexpr int AHEAD = 2, NP = G::Q / 2;
    CT qp[AHEAD][F::NF], qm[AHEAD][F::NF];
    auto read = [&](int n) {
        const int i = 2 * n + 1;
        cells.get(kb, R::template nb<ZH>(G::c(i, 0), G::c(i, 1), G::c(i, 2)), qp[n % AHEAD]);
        cells.get(kb, R::template nb<ZH>(-G::c(i, 0), -G::c(i, 1), -G::c(i, 2)), qm[n % AHEAD]);
    };
#pragma unroll
    for (int n = 0; n < AHEAD; ++n) read(n);
#pragma unroll
    for (int n = 0; n < NP; ++n) {
        const int i = 2 * n + 1;  // the opposite directions i and i + 1
        const CT* p = qp[n % AHEAD];
        const CT* m = qm[n % AHEAD];
#pragma unroll
        for (int f = 0; f < F::NF; ++f) {
            const CT s = p[f] - m[f], d = s * (CT)G::w(i);
#pragma unroll
            for (int a = 0; a < DIMV; ++a) {
                if (grad_split<G, SPLIT>(i, f - F::U, a)) {
                    CT r = s * (CT)G::w(i);
                    asm("" : "+v"(r));
                    if (G::c(i, a) == 1) gr[f][a] += r;
                    if (G::c(i, a) == -1) gr[f][a] -= r;
                } else {
                    if (G::c(i, a) == 1) gr[f][a] += d;
                    if (G::c(i, a) == -1) gr[f][a] -= d;
                }
            }
        }
        l += (p[F::PHI] + m[F::PHI] - (CT)2 * q0[F::PHI]) * (CT)G::w(i);
#pragma unroll
        for (int f = 0; f < F::NF; ++f)
#pragma unroll
            for (int a = 0; a < DIMV; ++a)
                if (G::c(i, a) != 0) asm volatile("" : "+v"(gr[f][a]));
        asm volatile("" : "+v"(l));
        kb.hide();
        if (n + AHEAD < NP) read(n + AHEAD);
    }
    // 2 * (1/(2T)): each pair counted once
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        v.gphi[a] = gr[F::PHI][a] * (CT)3.0;
        v.grho[a] = gr[F::RHO][a] * (CT)3.0;
        v.G2[a] = a < DIMV ? gr[F::U + (a < DIMV ? a : 0)][a] * (CT)6.0 : (CT)0;
        v.Gs[a] = 0;
    }
    // the sums the collision takes of the velocity gradients, each rounding
    // its second term alone (written out, so that every kernel rounds alike)
    const CT(*gu)[3] = gr + F::U;
    v.div = SPLIT == 1 ? fma_((CT)3.0, gu[1][1], gu[0][0] * (CT)3.0) : fma_((CT)3.0, gu[0][0], gu[1][1] * (CT)3.0);
    v.Gs[0] = fma_((CT)3.0, gu[0][1], gu[1][0] * (CT)3.0);
    if constexpr (DIMV == 3) {
        v.div = fma_((CT)3.0, gu[2][2], v.div);
        v.Gs[1] = fma_((CT)3.0, gu[0][2], gu[2][0] * (CT)3.0);
        v.Gs[2] = fma_((CT)3.0, gu[1][2], gu[2][1] * (CT)3.0);
    }
    v.lphi = l * (CT)6.0;  // 2/T
}

// --- collide + stream.  A tile first issues the loads of its own nodes'
// incoming h and M2 together with the halo loads of phi and u, so that their
// latencies overlap (h then waits in registers, two to each, in 2-byte storage
// and in LDS otherwise); then it takes the gradients from LDS and collides one
// direction at a time.
// The tile's step read again from the descriptor (a volatile load, so the
// compiler cannot take it for the value a branch already tested).
__device__ __forceinline__ int64_t step_parity(CDesc& cs, const TileCtx& t)
{
    return *(const volatile PULBM_CST int64_t*)&cs.step + (t.step - cs.step);
}

template <int LS, class S>
using TileCells = Cells<typename Codec<S>::CT, CellF<Model<LS>::DIM>::NF, Halo1<Model<LS>, Model<LS>::DIM>::R::N>;

// Does a lattice set's collide kernel rebuild u for some cases (CaseDev::fuse_u)?
template <int LS, class S> constexpr bool can_fuse_u() { return LS == 4 && sizeof(S) >= 4; }

// --- pressure and velocity of a 2D tile inside its collide kernel (CaseDev::fuse_u
// 2).  A 2D step on the grids it is run on is bound by the latency of its
// launches, about 4.7 us each (200 x 400: 19.4 us a step for four kernels), not
// by their work, so a tile takes P* and u* three nodes deep and forms P two and
// u one node deep itself (2.1 and 1.5 times its 256 nodes), each value by
// k_pressure's and k_velocity's expressions, term by term.  A ghost beyond a wall
// or the open end is formed at its mirror node, inward in the same region.  (A
// block's ghosts mirror outward, past the region: cases with a block keep the
// separate kernels.)
template <class S> struct Flow2D {
    using CT = typename Codec<S>::CT;
    using H3 = HaloN<Model<2>, 2, 3>;
    Cells<CT, 4, H3::R::N> f;  // P*, u*, phi
    CT gd[H3::R::N];           // g . (ghost - mirror)
    CT P[Halo2<Model<2>, 2>::R::N];
};

// LDS bytes that a 2D collide's launch asks for: h (parked there but in 2-byte
// storage), in the same place as the fields of the rebuild if some case of the
// launch is FUSED, which are read for the last time before h is parked.  In FP64
// a CU's LDS then holds 3 workgroups with a fused case and 5 without; with room
// for both in every launch it held 2 (step, before / after: 1024^2 104 / 96 us,
// with walls 109 / 99, with a block 118 / 111; serving 12 of 200 x 400 with walls
// 137 / 120, with a block each 143 / 127; a batch that mixes both kinds 153 /
// 137).  The other storage widths held 5 and more: the same within 2%.
template <class S> constexpr int collide_lds_2d(bool fused)
{
    const int h = sizeof(S) == 2 ? 0 : (int)sizeof(S) * D2Q9::Q * 256;
    return fused && (int)sizeof(Flow2D<S>) > h ? (int)sizeof(Flow2D<S>) : h;
}

// The node that a 2D cell beyond a wall or the open end mirrors: (x - dx, y - dy).
struct Mirror {
    int dx, dy;
    bool odd, open;
};
template <bool WALL> __device__ __forceinline__ Mirror mirror(CDesc& cs, int x, int y)
{
    Mirror m = {0, 0, false, false};
    if constexpr (WALL) {
        int cr = 0;
        (void)resolve_axis(x, cs.nx, cs.wall[0], &m.dx, &cr);
        (void)resolve_axis(y, cs.ny, cs.wall[1], &m.dy, &cr);
        m.odd = cr & 1;
        m.open = cr & kOpenGhost;
    }
    return m;
}

template <class S, bool WALL>
__device__ __forceinline__ void rebuild_2d(CDesc& cs, const TileCtx& t, TileCells<2, S>& sC, Flow2D<S>& s, int lx,
                                           int ly, typename Codec<S>::CT* Pown)
{
    using CT = typename Codec<S>::CT;
    using G = D2Q9;
    using F = CellF<2>;
    using Mo = Model<2>;
    using H3 = HaloN<Mo, 2, 3>;
    using H2 = Halo2<Mo, 2>;
    using H1 = Halo1<Mo, 2>;
    const Slots<CT> Js = slots<CT>(cs.J, cs.N);
    void* src[4] = {cs.Ps, (void*)Js.at(0, 0), (void*)Js.at(1, 0), cs.phi[t.step & 1]};
    halo_stage<H3, WALL, 4, CT, true>(cs, t, src, [&](int k, int cr, const int* off, const CT* v) {
        CT c[4] = {v[0], v[1], v[2], v[3]}, gd = 0;
        if (WALL) gd = (CT)(cs.grav[0] * off[0] + cs.grav[1] * off[1] + cs.grav[2] * off[2]);
        if (WALL && (cr & kOpenGhost)) {
            c[0] = (CT)(2.0 * cs.p_top - (double)c[0]);
            gd = 0;
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
            if (WALL && (cr & 1)) c[1 + a] = (CT)(-(double)c[1 + a] + 2.0 * cs.grav[a]);
        s.f.put(k, c);
        if (WALL) s.gd[k] = gd;
    });
    __syncthreads();
    // (cells past a region repeat its last one: every pass's cells are in flight
    // together)
    // P two nodes deep
    constexpr int N2 = H2::R::N, N1 = H1::R::N;
#pragma unroll
    for (int it = 0; it < (N2 + 255) / 256; ++it) {
        const int k = min((int)threadIdx.x + 256 * it, N2 - 1), ix = k % H2::RX, iy = k / H2::RX;
        const Mirror m2 = mirror<WALL>(cs, t.ox - 2 + ix, t.oy - 2 + iy);
        const int k3 = H3::R::idx(ix + 1 - m2.dx, iy + 1 - m2.dy, 0);
        auto cell = [&](int i, int sgn, CT* v) {
            const int m = k3 + sgn * (G::c(i, 0) + H3::RX * G::c(i, 1));
            s.f.get({m * 16, m * (int)sizeof(CT)}, 0, v);
        };
        CT c0[4];
        cell(0, 1, c0);
        const double drho = (double)clamp01(c0[3]) * (cs.rho_w - cs.rho_a);
        const double rho = cs.rho_a + drho;
        constexpr int NS = shell<G>(G::Q - 1) + 1;
        CT sks[NS], sgs[NS], dus[2][NS];
#pragma unroll
        for (int h = 0; h < NS; ++h) sks[h] = sgs[h] = dus[0][h] = dus[1][h] = 0;
#pragma unroll
        for (int i = 1; i < G::Q; i += 2) {
            const int h = shell<G>(i);
            CT m[4], p[4];
            cell(i, -1, m);
            cell(i, 1, p);
            sks[h] += (m[0] - c0[0]) + (p[0] - c0[0]);
            if (WALL) {
                const int o = G::c(i, 0) + H3::RX * G::c(i, 1);
                sgs[h] += s.gd[k3 - o] + s.gd[k3 + o];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (G::c(i, a) == 0) continue;
                const CT d = m[1 + a] - p[1 + a];
                if (G::c(i, a) == 1) dus[a][h] += d;
                else dus[a][h] -= d;
            }
        }
        double sk = 0, sg = 0, su = 0;
#pragma unroll
        for (int h = 0; h < NS; ++h) {
            const double w = shell_w<G>(h);
            sk += w * (double)sks[h];
            if (WALL) sg += w * (double)sgs[h];
#pragma unroll
            for (int a = 0; a < 2; ++a) su += w * (double)dus[a][h];
        }
        if (WALL) sk += rho * sg;
        CT P = (CT)((double)c0[0] + (sk + drho * su));
        if (WALL && m2.open) P = (CT)(2.0 * cs.p_top - (double)P);
        s.P[k] = P;
    }
    __syncthreads();
    *Pown = s.P[H2::R::idx(lx + 2, ly + 2, 0)];
    // u one node deep
    const CT ra = cconst<CT>(cs.rho_a, cs.f32.rho_a), dr = cconst<CT>(cs.rho_w - cs.rho_a, cs.f32.drho);
#pragma unroll
    for (int it = 0; it < (N1 + 255) / 256; ++it) {
        const int k = min((int)threadIdx.x + 256 * it, N1 - 1), ix = k % H1::RX, iy = k / H1::RX;
        const Mirror m1 = mirror<WALL>(cs, t.ox - 1 + ix, t.oy - 1 + iy);
        const int k2 = H2::R::idx(ix + 1 - m1.dx, iy + 1 - m1.dy, 0), k3 = H3::R::idx(ix + 2 - m1.dx, iy + 2 - m1.dy, 0);
        CT c[4], f[F::NF];
        s.f.get({k3 * 16, k3 * (int)sizeof(CT)}, 0, c);
        const CT rho = ra + clamp01(c[3]) * dr;
        const CT irho = rcp(rho);
        CT gr[2] = {0, 0};
#pragma unroll
        for (int i = 1; i < G::Q; i += 2) {
            const int o2 = G::c(i, 0) + H2::RX * G::c(i, 1), o3 = G::c(i, 0) + H3::RX * G::c(i, 1);
            const CT p = s.P[k2 + o2], m = s.P[k2 - o2];
            const CT d = (WALL ? (p + rho * s.gd[k3 + o3]) - (m + rho * s.gd[k3 - o3]) : p - m) * (CT)G::w(i);
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                if (G::c(i, a) == 1) gr[a] += d;
                if (G::c(i, a) == -1) gr[a] -= d;
            }
        }
        f[F::PHI] = c[3];
        f[F::RHO] = rho;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            const CT u = c[1 + a] - gr[a] * (CT)3.0 * irho;
            f[F::U + a] = m1.odd ? -u : u;  // no slip
        }
        sC.put(k, f);
    }
    __syncthreads();
}

template <int LS, class S, bool WALL, bool BGK, class R, int PAR>
__device__ __forceinline__ void collide_tile(CDesc& cs, const TileCtx& t, TileCells<LS, S>& sC, S (*sH)[256],
                                             typename Codec<S>::CT* sP2, Flow2D<S>* s2)
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using G = typename Mo::G;
    using H = typename Mo::H;
    using CT = typename Codec<S>::CT;
    using HR = Halo1<Mo, DIMV>;
    using F = CellF<DIMV>;
    constexpr int NM = DIMV == 2 ? 3 : 6;
    const Phys<CT> ph = make_phys<CT>(cs);
    int lx, ly, lz;
    local_xyz<Mo>(&lx, &ly, &lz);
    const int x = t.ox + lx, y = t.oy + ly, z = t.oz + lz;
    // block nodes carry no fluid and are skipped like nodes past the grid
    const bool inside = x < cs.nx && y < cs.ny && z < cs.nz && !(WALL && in_block(cs, x, y, z));
    // What a lane outside the grid loads is never used.  It loads the nearest
    // node, in a line that a lane inside loads (all of them node 0 made its lines
    // a hot spot of the whole chip, 100 x 90 x 80, FP32 odd collide 72 / 58 us,
    // FP16 48 / 41), or nothing in a tile at a wall, where the nearest node's
    // registers cost more than the branch (512 x 256 x 256 dam break, FP16 odd
    // collide 1.55 / 1.48 ms).
    const int xc = WALL ? (inside ? x : 0) : min(x, cs.nx - 1), yc = WALL ? (inside ? y : 0) : min(y, cs.ny - 1),
              zc = WALL ? (inside ? z : 0) : min(z, cs.nz - 1);
    const uint32_t n = (uint32_t)xc + (uint32_t)cs.sx * ((uint32_t)yc + (uint32_t)cs.ny * (uint32_t)zc);
    const uint32_t nb = n * (uint32_t)sizeof(S), na = n * (uint32_t)(sizeof(S) == 2 ? 4 : sizeof(CT));
    // the step's parity, which decides the slots the AA pattern reads and
    // writes.  PAR 0: even, fixed at compile time.  PAR 1: odd, read again at
    // run time (step_parity), so that each load and store decides its slot
    // as it runs: a copy with the odd slots fixed keeps a node's neighbour
    // offsets in registers and spills past the 3-waves budget.  PAR 2: odd,
    // fixed, for a tile whose nodes have every neighbour inside the grid,
    // whose offsets are then the strides (scalars).
    const bool odd = PAR == 0 ? false : (PAR == 2 ? true : (bool)(step_parity(cs, t) & 1));
    const Nav nv = PAR == 2 ? make_nav_inner(cs, (int)sizeof(S))
                            : make_nav(cs, xc, yc, zc, (int)sizeof(S));
    // stores stream past L2 on even steps (FP32 even collide 3% faster); on
    // odd steps, shifted by one node in x, each line is written partly by
    // this tile and partly by its x neighbour, and kept in L2 the parts merge
    // (512 x 256 x 256, FP16: the odd steps' writes 123 streamed, 97 B/node kept)
    constexpr bool nts = PAR == 0 && nt_access<S, kStoreCollide>();
    const Slots<S> hs = slots<S>(cs.h, cs.N), gs = slots<S>(cs.g, cs.N);
    // own-node loads first
    S hraw[H::Q];
    // M2 as loaded: compute-type values, or words of two 2-byte codes
    using M2L = std::conditional_t<sizeof(S) == 2, uint32_t, CT>;
    constexpr int NL = sizeof(S) == 2 ? (NM + 1) / 2 : NM;
    M2L m2l[NL];
    CT php = 0;  // reference of the incoming h (2-byte storage)
    CT dP = 0;   // BGK: (previous P - new P) / (rho_ref T), restores the stored rest population
    CT ur[3] = {0, 0, 0};  // BGK, 2-byte storage: reference of the incoming g
    if (!WALL || inside) {
        php = h_reference<S>(cs.phi[(t.step + 1) & 1], n);
        if constexpr (BGK) u_reference<S, DIMV>(cs.U[(t.step + 1) & 1], cs.N, n, ur);
#pragma unroll
        for (int j = 0; j < H::Q; ++j) hraw[j] = aa_load<H, WALL, nt_access<S, kLoadCollide>()>(hs, nb, nv, j, odd);
        if constexpr (BGK) {
            dP = *at_node<CT>(cs.P[t.step & 1], n);  // the previous P; the new one below
        } else {
            const Slots<M2L> Ms = slots<M2L>(cs.M2, cs.N);
#pragma unroll
            for (int k = 0; k < NL; ++k) m2l[k] = __builtin_nontemporal_load(Ms.at(k, na));
        }
    }
    __builtin_amdgcn_sched_barrier(0);  // the own-node loads are issued first
    // halo of phi, rho and u; a fused case (no wall, open end or block)
    // loads u* instead of u and the new P two nodes deep, and rebuilds u
    // itself below
    bool fused = false;
    if constexpr (!WALL && can_fuse_u<LS, S>()) fused = cs.fuse_u;
    const bool fused2d = LS == 2 && cs.fuse_u == 2;
    CT Pnew = 0;
    if constexpr (LS == 2) {
        if (fused2d) {
            // ghosts show in the 3-node halo of a tile up to two nodes clear of a wall
            if (WALL || (cs.wall[0] && t.ox + Mo::TX + 2 >= cs.nx) || (cs.wall[1] && t.oy + Mo::TY + 2 >= cs.ny))
                rebuild_2d<S, true>(cs, t, sC, *s2, lx, ly, &Pnew);
            else
                rebuild_2d<S, false>(cs, t, sC, *s2, lx, ly, &Pnew);
        }
    }
    if (!fused2d) {
        const Slots<CT> Us = slots<CT>(fused ? cs.J : cs.U[t.step & 1], cs.N);
        void* src[1 + DIMV];
        src[0] = cs.phi[t.step & 1];
#pragma unroll
        for (int a = 0; a < DIMV; ++a) src[1 + a] = (void*)Us.at(a, 0);
        halo_stage<HR, WALL, 1 + DIMV, CT, true>(
            cs, t, src,
            [&](int k, int cr, const int*, const CT* v) {
                CT f[F::NF];
                f[F::PHI] = v[0];
                f[F::RHO] = ph.rho_a + clamp01(v[0]) * ph.drho;
#pragma unroll
                for (int a = 0; a < DIMV; ++a) f[F::U + a] = (WALL && (cr & 1)) ? -v[1 + a] : v[1 + a];  // no slip
                sC.put(k, f);
            });
    }
    if constexpr (!WALL && can_fuse_u<LS, S>()) {
        if (fused) {
            void* psrc[1] = {cs.P[(t.step + 1) & 1]};
            halo_stage<Halo2<Mo, DIMV>, false, 1, CT>(cs, t, psrc,
                                                      [&](int k, int, const int*, const CT* v) { sP2[k] = v[0]; });
        }
    }
    // 4- and 8-byte storage parks h in LDS until the direction loop; 2-byte
    // storage keeps it in registers, two values to each
    uint32_t h2[(H::Q + 1) / 2];
    if constexpr (sizeof(S) == 2) {
#pragma unroll
        for (int j = 0; j < H::Q; j += 2) h2[j / 2] = pair_pack<S>(hraw[j], j + 1 < H::Q ? hraw[j + 1] : (S)0);
    } else {
#pragma unroll
        for (int j = 0; j < H::Q; ++j) sH[j][threadIdx.x] = hraw[j];
    }
    auto h_in = [&](int j) -> S {
        if constexpr (sizeof(S) == 2) return pair_half<S>(h2[j / 2], j & 1);
        else return sH[j][threadIdx.x];
    };
    __syncthreads();
    if constexpr (!WALL && can_fuse_u<LS, S>()) {
        if (fused) {
            // u = u* - D P / rho at every cell of the 1-halo region, the
            // expression of k_velocity term by term
            using R2 = typename Halo2<Mo, DIMV>::R;
            constexpr int DZ = Halo2<Mo, DIMV>::ZH - HR::ZH;
#pragma unroll
            for (int it = 0; it < (R::N + 255) / 256; ++it) {
                const int k = (int)threadIdx.x + 256 * it;
                if (k < R::N) {
                    const int ix = k % HR::RX, iy = (k / HR::RX) % HR::RY, iz = k / (HR::RX * HR::RY);
                    const int cx2 = ix + 1, cy2 = iy + 1, cz2 = iz + DZ;
                    CT gr[3] = {0, 0, 0};
#pragma unroll
                    for (int i = 1; i < G::Q; i += 2) {
                        const int kp = R2::idx(cx2 + G::c(i, 0), cy2 + G::c(i, 1), cz2 + G::c(i, 2));
                        const int km = R2::idx(cx2 - G::c(i, 0), cy2 - G::c(i, 1), cz2 - G::c(i, 2));
                        const CT d = (sP2[kp] - sP2[km]) * (CT)G::w(i);
#pragma unroll
                        for (int a = 0; a < DIMV; ++a) {
                            if (G::c(i, a) == 1) gr[a] += d;
                            if (G::c(i, a) == -1) gr[a] -= d;
                        }
                    }
                    CT f[F::NF];
                    sC.get({k * 16, k * (int)sizeof(CT)}, 0, f);
                    const CT irho = rcp(f[F::RHO]);
#pragma unroll
                    for (int a = 0; a < DIMV; ++a) f[F::U + a] = f[F::U + a] - gr[a] * (CT)3.0 * irho;
                    sC.put(k, f);
                }
            }
            __syncthreads();
        }
    }
    if constexpr (LS == 2) {
        // the new P of the tile's own nodes, and in 2-byte storage their u, the
        // codec's reference of the next step (no kernel reads u otherwise)
        if (fused2d && inside) {
            *at_node<CT>(cs.P[(t.step + 1) & 1], n) = Pnew;
            if constexpr (sizeof(S) == 2) {
                CT f[F::NF];
                const int c = R::idx(lx + 1, ly + 1, 0);
                sC.get({c * 16, c * (int)sizeof(CT)}, 0, f);
                const Slots<CT> Un = slots<CT>(cs.U[t.step & 1], cs.N);
#pragma unroll
                for (int a = 0; a < DIMV; ++a) *Un.at(a, n * (uint32_t)sizeof(CT)) = f[F::U + a];
            }
        }
    }
    if (!inside) return;
    if constexpr (BGK) {
        if (!fused2d) Pnew = *at_node<CT>(cs.P[(t.step + 1) & 1], n);
        dP = (CT)(((double)dP - (double)Pnew) * (3.0 / cs.rho_a));
        asm("" : "+v"(dP));
    }

    CT m2[NM];
    if constexpr (!BGK) {
        if constexpr (sizeof(S) == 2) {
            const CT gsc_m = cconst<CT>(cs.g_inv_scale, cs.f32.g_inv_scale);
#pragma unroll
            for (int k = 0; k < NM; ++k) m2[k] = Codec<S>::dec(pair_half<S>(m2l[k / 2], k & 1), gsc_m, (CT)0);
        } else {
#pragma unroll
            for (int k = 0; k < NM; ++k) m2[k] = m2l[k];
        }
    }
    NodeVals<CT> v;
    const int k0 = R::template nb_base<HR::ZH>(lx + 1, ly + 1, lz + HR::ZH);
    auto kb = sC.at(k0);
    tile_gradients<LS, R, HR::ZH, grad_split_of<S, WALL, BGK, PAR>()>(sC, kb, v);
    // the BGK collision needs the equilibria alone (no Pi: the INIT form)
    const NodeCoef<DIMV, CT> kc = node_coef<DIMV, BGK, CT>(ph, v, m2);
    const CT omf = BGK ? (CT)1 - rcp(ph.tau_a + clamp01(v.phi) * ph.dtau) : (CT)0;  // 1 - 1/tau_mix
    const CT hisc = cconst<CT>(cs.h_inv_scale, cs.f32.h_inv_scale), hsc = cconst<CT>(cs.h_scale, cs.f32.h_scale);
    const CT gsc = cconst<CT>(cs.g_scale, cs.f32.g_scale), gsc_in = cconst<CT>(cs.g_inv_scale, cs.f32.g_inv_scale);
    const CT corr = (CT)6.0 * rcp(kc.rho);  // 2 / (rho T)
    // shifts of an outgoing g_i and h_i in 2-byte storage, from phi and u
    // (this step) of the node that reads it next step: x + c_i, or x itself
    // for a population reflected at a wall, which that node reads as moving
    // along -c_i
    // (each read again where it is used, which keeps the register budget:
    // merged with the gradients' reads they would stay live to the end)
    __builtin_amdgcn_sched_barrier(0);
    const auto kd = sC.at(k0);
    constexpr int c0 = R::template nb<HR::ZH>(0, 0, 0);
    auto gref_out = [&](int i, bool reflected) -> CT {
        if constexpr (sizeof(S) != 2) {
            return (CT)0;
        } else {
            const int k = reflected ? c0 : R::template nb<HR::ZH>(G::c(i, 0), G::c(i, 1), G::c(i, 2));
            CT f[F::NF], ud[3] = {0, 0, 0};
            sC.get(kd, k, f);
#pragma unroll
            for (int a = 0; a < DIMV; ++a)
                if (G::c(i, a) != 0) ud[a] = f[F::U + a];
            CT cu = c_dot<G, DIMV>(i, ud);
            if (reflected) cu = -cu;
            return g_shift((CT)G::w(i), cu);
        }
    };
    auto href_out = [&](int i, bool reflected) -> CT {
        if constexpr (sizeof(S) != 2) {
            return (CT)0;
        } else {
            const int k = reflected ? c0 : R::template nb<HR::ZH>(H::c(i, 0), H::c(i, 1), H::c(i, 2));
            CT f[F::NF];
            sC.get(kd, k, f);
            return (CT)H::w(i) * f[F::PHI];
        }
    };
    // rest direction of g, the opposite pairs, then the rest direction of h;
    // both lattices share the direction order, so h_i and g_i stream to the
    // same node
    {
        CT g0 = g_out<G, DIMV, BGK>(v, kc, 0);
        if constexpr (BGK) {
            // BGK (Eq. BGK_LBeq_hydroeq) on the full rest population; both the
            // stored incoming value and the equilibrium lack their P / (rho_ref T)
            const CT gin = Codec<S>::dec(aa_load<G, WALL, false>(gs, nb, nv, 0, odd), gsc_in,
                                         g_ref<G, DIMV>(0, ur)) + dP;
            g0 += omf * (gin - g0);
        }
        aa_store<G, WALL, nts>(gs, nb, nv, 0, odd, Codec<S>::enc(g0, gsc, (CT)0), false);
    }
    // sum over j != 0 of the incoming h_j less the outgoing h*_j as its reader
    // will decode it (the rest population balances it below)
    CT hmoved = 0;
#pragma unroll
    for (int i = 1; i < G::Q; i += 2) {
        // keep the scheduler from interleaving pairs (4-byte storage: more than
        // two of them): the fewer registers buy another wave per SIMD
        if (sizeof(S) != 4 || i / 2 % 2 == 0) __builtin_amdgcn_sched_barrier(0);
        const bool bi = WALL && nav_solid<G>(nv, i, +1);
        const bool bk = WALL && nav_solid<G>(nv, i + 1, +1);
        CT gi, gk;
        g_pair<G, DIMV, BGK>(v, kc, i, &gi, &gk);
        if constexpr (BGK) {
            // incoming g_i, g_i+1: within a step a node reads and writes one set
            // of slots (AA), and the slots of this pair are written just below
            const CT ai = Codec<S>::dec(aa_load<G, WALL, false>(gs, nb, nv, i, odd), gsc_in,
                                        g_ref<G, DIMV>(i, ur));
            const CT ak = Codec<S>::dec(aa_load<G, WALL, false>(gs, nb, nv, i + 1, odd), gsc_in,
                                        g_ref<G, DIMV>(i + 1, ur));
            gi += omf * (ai - gi);
            gk += omf * (ak - gk);
        }
        if (WALL) {
            const bool oi = nav_open<G>(nv, i, +1), ok = nav_open<G>(nv, i + 1, +1);
            CT cF = 0;
#pragma unroll
            for (int a = 0; a < DIMV; ++a) {
                if (G::c(i, a) == 1) cF += kc.F[a];
                if (G::c(i, a) == -1) cF -= kc.F[a];
            }
            // a reflected population keeps the force part of its equilibrium
            const CT fc = (CT)G::w(i) * cF * corr;
            gi -= (bi && !oi) ? fc : (CT)0;
            gk += (bk && !ok) ? fc : (CT)0;
            // through the open end: the population leaves, and the opposite
            // one entering this node is the node's own equilibrium
            if (oi || ok) {
                CT ei, ek;
                g_pair<G, DIMV, true>(v, kc, i, &ei, &ek);
                if (oi) gi = ek;
                if (ok) gk = ei;
            }
        }
        aa_store<G, WALL, nts>(gs, nb, nv, i, odd, Codec<S>::enc(gi, gsc, gref_out(i, bi)),
                                                         bi);
        aa_store<G, WALL, nts>(gs, nb, nv, i + 1, odd,
                                                         Codec<S>::enc(gk, gsc, gref_out(i + 1, bk)), bk);
        if (i < H::Q) {
            const CT hi = Codec<S>::dec(h_in(i), hisc, php * (CT)H::w(i));
            const CT hk = Codec<S>::dec(h_in(i + 1), hisc, php * (CT)H::w(i + 1));
            CT oi, ok;
            h_pair<H, DIMV, false>(ph, v, kc, i, hi, hk, &oi, &ok);
            const CT ri = href_out(i, bi), rk = href_out(i + 1, bk);
            const S ei = Codec<S>::enc(oi, hsc, ri), ek = Codec<S>::enc(ok, hsc, rk);
            hmoved += (hi - Codec<S>::dec(ei, hisc, ri)) + (hk - Codec<S>::dec(ek, hisc, rk));
            aa_store<H, WALL, nts>(hs, nb, nv, i, odd, ei, bi);
            aa_store<H, WALL, nts>(hs, nb, nv, i + 1, odd, ek, bk);
        }
    }
    // rest population of h: BGK conserves phi (sum_j h^eq_j = phi), so
    // h*_0 = h_0 + sum_{j != 0} (h_j - h*_j).  Taking it in that form, with the
    // outgoing values as stored, keeps the weights' rounding (their FP32
    // values sum to 1 + 1.5e-8 on D3Q19) and the rounding of identical bulk
    // nodes from drifting phi's mass step after step.
    {
        const CT h0 = Codec<S>::dec(h_in(0), hisc, php * (CT)H::w(0));
        aa_store<H, WALL, nts>(hs, nb, nv, 0, odd,
                                                         Codec<S>::enc(h0 + hmoved, hsc, href_out(0, true)), false);
    }
}

// Occupancy of the collision kernel: what bounds it in 2-byte storage is the
// issue of vector instructions (about 1100 per wave) and the latency of its
// loads, so it wants waves.  The least number of waves per SIMD is set here;
// registers (tile_gradients) and LDS (h kept in registers, no u-rebuild halo
// on lattice sets that never use it) allow on D3Q27 6 on even and 4 on odd steps
// in FP16, 4 in BF16 and in 4-byte storage (by LDS; 3 where collide_lds_3d says
// so) and 2 in 8-byte storage (by LDS).  Against 3, 3 and 1 before (512x256x256
// dam break, FP16, even / odd step: 1.46 / 1.75 -> 1.11 / 1.49 ms; 101x53x45
// FP64: 58 -> 45 us).  Held to 3 waves by LDS the FP16 collide takes 1.50 ms on
// average; asked for 5 waves on odd steps it spills (1.57 ms).
// (D3Q19 hydro in 4- and 8-byte storage: 3 and 1, by the LDS of the u rebuild.)
template <int LS, class S> constexpr int collide_waves()
{
    return LS == 4 ? (sizeof(S) == 8 ? 1 : (sizeof(S) == 4 ? 3 : 4)) : (sizeof(S) == 8 ? 2 : 4);
}
#define PULBM_COLLIDE_ATTR __attribute__((amdgpu_waves_per_eu(collide_waves<LS, S>())))
// One kernel per step parity: PAR 0 takes the tiles of cases at an even
// step, with every load and store on its fixed slot (no branch: the FP16
// collide's even steps run 17% faster than with the parity read at run
// time); PAR 1 takes the tiles of cases at an odd step, with fixed slots
// on tiles clear of the grid's edges (PAR 2 of collide_tile, 6% faster)
// and slots decided at run time on the others.  A single case
// launches the kernel of its step's parity, a serving batch (whose cases may
// differ in parity) both, each skipping the other's tiles, so a case runs the
// same code alone and in a batch, bitwise.
template <int LS, class S, bool BGK, int PAR>
__global__ __launch_bounds__(256) PULBM_COLLIDE_ATTR void k_collide(CaseTab cases, const int* hdr, int step_off)
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using H = typename Mo::H;
    using CT = typename Codec<S>::CT;
    using R = typename Halo1<Mo, DIMV>::R;
    __shared__ TileCells<LS, S> sC;
    // the new P two nodes deep, for cases whose collide rebuilds u
    __shared__ CT sP2[can_fuse_u<LS, S>() ? Halo2<Mo, DIMV>::R::N : 1];
    S(*sH)[256];
    Flow2D<S>* s2 = nullptr;
    if constexpr (LS == 2) {
        // h, and before it P*, u* and the new P for cases whose collide rebuilds
        // both, in the LDS of the launch (collide_lds_2d)
        extern __shared__ __align__(16) char collide_dyn[];
        sH = (S(*)[256])collide_dyn;
        s2 = (Flow2D<S>*)collide_dyn;
    } else {
        __shared__ S sHs[sizeof(S) == 2 ? 1 : H::Q][256];
        sH = sHs;
    }
    const TileCtx t = tile_ctx<Mo>(cases, hdr, step_off);
    if (!t.active || (int)(t.step & 1) != PAR) return;
    CDesc& cs = *t.cs;
    if (tile_at_wall<Mo>(cs, t.ox, t.oy, t.oz)) {
        collide_tile<LS, S, true, BGK, R, PAR>(cs, t, sC, sH, sP2, s2);
    } else if (PAR == 1 && t.ox >= 1 && t.ox + Mo::TX < cs.nx && t.oy >= 1 && t.oy + Mo::TY < cs.ny &&
               (DIMV == 2 || (t.oz >= 1 && t.oz + Mo::TZ < cs.nz))) {
        // every node of the tile has its neighbours inside the grid
        collide_tile<LS, S, false, BGK, R, 2>(cs, t, sC, sH, sP2, s2);
    } else {
        collide_tile<LS, S, false, BGK, R, PAR>(cs, t, sC, sH, sP2, s2);
    }
}

// --- initial state: equilibria of (phi0, P0, u0) in the even AA layout,
//     previous-step pressure P[0] = P0.  Inputs are FP64 device arrays.
template <int LS, class S>
__global__ __launch_bounds__(256) void k_init(CaseTab cases, const int* hdr,
                                              const double* __restrict__ phi0, const double* __restrict__ P0,
                                              const double* __restrict__ u0)
{
    constexpr int DIMV = Model<LS>::DIM;
    using Mo = Model<LS>;
    using G = typename Mo::G;
    using H = typename Mo::H;
    using CT = typename Codec<S>::CT;
    using HR = Halo1<Mo, DIMV>;
    using R = typename HR::R;
    using F = CellF<DIMV>;
    __shared__ TileCells<LS, S> sC;
    const TileCtx t = tile_ctx<Mo>(cases, hdr, 0);
    if (!t.active) return;
    CDesc& cs = *t.cs;
    const uint32_t N = (uint32_t)cs.N;
    const Phys<CT> ph = make_phys<CT>(cs);
    // the halo cell by cell (initialisation runs once; the step kernels use
    // halo_stage)
#pragma unroll
    for (int it = 0; it < (R::N + 255) / 256; ++it) {
        const int k = threadIdx.x + 256 * it;
        if (k >= R::N) break;
        int off[3], cr;
        const uint32_t m = HR::cell(cs, t, k, off, &cr);
        CT f[F::NF];
        f[F::PHI] = (CT)phi0[m];
        f[F::RHO] = ph.rho_a + clamp01(f[F::PHI]) * ph.drho;
#pragma unroll
        for (int a = 0; a < DIMV; ++a) {
            const CT ua = (CT)u0[(size_t)a * N + m];
            f[F::U + a] = (cr & 1) ? -ua : ua;
        }
        sC.put(k, f);
    }
    __syncthreads();
    int lx, ly, lz;
    local_xyz<Mo>(&lx, &ly, &lz);
    const int x = t.ox + lx, y = t.oy + ly, z = t.oz + lz;
    if (x >= cs.nx || y >= cs.ny || z >= cs.nz) return;
    const uint32_t n = (uint32_t)x + (uint32_t)cs.sx * ((uint32_t)y + (uint32_t)cs.ny * (uint32_t)z);
    const Slots<S> hs = slots<S>(cs.h, cs.N), gs = slots<S>(cs.g, cs.N);
    const uint32_t nb = n * (uint32_t)sizeof(S);
    const Slots<CT> U1 = slots<CT>(cs.U[1], cs.N);
    if (in_block(cs, x, y, z)) {
        // block nodes hold no populations and no fluid
#pragma unroll
        for (int j = 0; j < H::Q; ++j) *hs.at(j, nb) = Codec<S>::enc((CT)0, (CT)1, (CT)0);
#pragma unroll
        for (int i = 0; i < G::Q; ++i) *gs.at(i, nb) = Codec<S>::enc((CT)0, (CT)1, (CT)0);
        *at_node<CT>(cs.P[0], n) = 0;
        *at_node<CT>(cs.P[1], n) = 0;
        *at_node<CT>(cs.phi[1], n) = 0;
#pragma unroll
        for (int a = 0; a < DIMV; ++a) *U1.at(a, n * (uint32_t)sizeof(CT)) = 0;
        return;
    }
    NodeVals<CT> v;
    tile_gradients<LS, R, HR::ZH, grad_split_of<S, false, false, 0>()>(sC, sC.at(R::template nb_base<HR::ZH>(lx + 1, ly + 1, lz + HR::ZH)), v);
    const NodeCoef<DIMV, CT> kc = node_coef<DIMV, true, CT>(ph, v, (const CT*)nullptr);
    const CT hsc = cconst<CT>(cs.h_scale, cs.f32.h_scale), gsc = cconst<CT>(cs.g_scale, cs.f32.g_scale);
    // 2-byte storage: h_j - w_j phi0 (the previous-step phi of step 0 is phi0)
    const CT phr = sizeof(S) == 2 ? v.phi : (CT)0;
    CT hmoved = 0;
#pragma unroll
    for (int j = 1; j < H::Q; ++j) {
        const CT hj = h_out<H, DIMV, true>(ph, v, kc, j, (CT)0);
        hmoved += hj;
        *hs.at(j, nb) = Codec<S>::enc(hj, hsc, phr * (CT)H::w(j));
    }
    // rest population as the remainder, so that sum_j h_j = phi0 exactly
    *hs.at(0, nb) = Codec<S>::enc(v.phi - hmoved, hsc, phr * (CT)H::w(0));
    // 2-byte storage: g_i - w_i c_i.u0 / T (the previous-step u of step 0 is u0)
#pragma unroll
    for (int i = 0; i < G::Q; ++i)
        *gs.at(i, nb) = Codec<S>::enc(g_out<G, DIMV, true>(v, kc, i), gsc,
                                      sizeof(S) == 2 ? g_ref<G, DIMV>(i, v.u) : (CT)0);
    *at_node<CT>(cs.P[0], n) = (CT)P0[n];
    *at_node<CT>(cs.phi[1], n) = v.phi;
#pragma unroll
    for (int a = 0; a < DIMV; ++a) *U1.at(a, n * (uint32_t)sizeof(CT)) = v.u[a];
}

// --- step counters: every case of a table advances by k (up to its end).
__global__ void k_advance(CaseTab cases, const int* hdr, int k)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= hdr[0]) return;
    CaseDev* cs = cases[c];
    const int64_t s = cs->step + k;
    cs->step = s < cs->step_end ? s : cs->step_end;
}

// --- conservation diagnostics of a read pass: per-block FP64 partials
//     (wave64 shuffles, then across the block), reduced in a fixed order.
constexpr int kDiagBlocks = 1024;
constexpr int kDiagVals = 10;  // phi, u[3], rho u[3], umax, nonfinite, spare

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}

template <class AT>
__global__ __launch_bounds__(256) void k_diag(const CaseDev* __restrict__ csp, double* __restrict__ partial)
{
    const CaseDev& cs = *csp;
    const int64_t N = cs.N;
    const AT* phi = (const AT*)cs.phi[cs.step & 1];
    const AT* P = (const AT*)cs.P[(cs.step + 1) & 1];
    const AT* U = (const AT*)cs.U[cs.step & 1];
    double acc[kDiagVals] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t n = (int64_t)blockIdx.x * 256 + threadIdx.x; n < N; n += (int64_t)gridDim.x * 256) {
        if (n % cs.sx >= cs.nx) continue;  // row padding
        const double f = (double)phi[n];
        const double pc = f < 0.0 ? 0.0 : (f > 1.0 ? 1.0 : f);
        const double rho = cs.rho_a + pc * (cs.rho_w - cs.rho_a);
        bool bad = !isfinite(f) || !isfinite((double)P[n]);
        double um2 = 0.0;
        acc[0] += f;
        for (int a = 0; a < cs.dim; ++a) {
            const double ua = (double)U[a * N + n];
            bad |= !isfinite(ua);
            acc[1 + a] += ua;
            acc[4 + a] += rho * ua;
            um2 += ua * ua;
        }
        acc[7] = fmax(acc[7], sqrt(um2));
        acc[8] += bad ? 1.0 : 0.0;
    }
    __shared__ double red[4][kDiagVals];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kDiagVals; ++k) {
        const double r = k == 7 ? wave_max(acc[k]) : wave_sum(acc[k]);
        if (lane == 0) red[wv][k] = r;
    }
    __syncthreads();
    if (threadIdx.x < kDiagVals) {
        const int k = threadIdx.x;
        double r = red[0][k];
        for (int w = 1; w < 4; ++w) r = k == 7 ? fmax(r, red[w][k]) : r + red[w][k];
        partial[blockIdx.x * kDiagVals + k] = r;
    }
}

// one wave per value: lane l takes blocks l, l + 64, ... in order, then a
// fixed shuffle tree (the result does not depend on scheduling)
__global__ __launch_bounds__(64) void k_diag_final(const double* __restrict__ partial, int nblocks,
                                                   double* __restrict__ out)
{
    const int k = blockIdx.x, lane = threadIdx.x;
    double r = 0.0;
    for (int b = lane; b < nblocks; b += 64) r = k == 7 ? fmax(r, partial[b * kDiagVals + k]) : r + partial[b * kDiagVals + k];
    r = k == 7 ? wave_max(r) : wave_sum(r);
    if (lane == 0) out[k] = r;
}

}  // namespace pulbm
