// Building blocks shared by the z-sweep kernels of the 55-point and the
// 19-point methods: raw buffer access, tile geometry, plane addressing.
#pragma once

#include <cstdlib>
#include <type_traits>

#include "exp_fp64.hpp"
#include "fd6_internal.hpp"

namespace fd6 {
namespace {

constexpr int sl8(int x) { return ((x % 8) + 8) % 8; }

// Raw buffer access: an SGPR descriptor for one plane of one field plus a
// 32-bit per-lane byte offset.  Loads beyond the descriptor's range return 0
// and stores beyond it are dropped, which replaces bounds branches.
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr int kBufFlags = 0x00020000;        // raw, untyped access (word 3)
constexpr unsigned kDropOffset = 0x80000000u;  // beyond every plane's range

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const T* p, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, (int)bytes, kBufFlags);
}
// Cache policy of an access (the instruction's cache-policy field): 0 keeps
// the default, kNonTemporal marks a stream whose lines are not reused before
// eviction (the new state and the RK register: each is touched once per
// substep).
constexpr int kNonTemporal = 2;

template <int CP = 0>
__device__ __forceinline__ float bload(float*, __amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, CP));
}
template <int CP = 0>
__device__ __forceinline__ double bload(double*, __amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, CP));
}
template <int CP = 0>
__device__ __forceinline__ void bstore(float v, __amdgpu_buffer_rsrc_t r, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), r, off, 0, CP);
}
template <int CP = 0>
__device__ __forceinline__ void bstore(double v, __amdgpu_buffer_rsrc_t r, unsigned off) {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, CP);
}

// One grid point of the array-of-structures layout: the four fields in 16
// (FP32) or 32 (FP64) consecutive bytes, moved with 16-byte accesses.
// (Whole vectors are bit-cast: with this compiler a bit cast of a single
// element of the loaded vector shrank the access to one dword and gave wrong
// values for the other elements.)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int CP = 0>
__device__ __forceinline__ void bload_point(float (&v)[4], __amdgpu_buffer_rsrc_t r,
                                            unsigned off) {
    const f32x4 a = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, CP));
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = a[i];
}
template <int CP = 0>
__device__ __forceinline__ void bload_point(double (&v)[4], __amdgpu_buffer_rsrc_t r,
                                            unsigned off) {
    // a dropped point (off = kDropOffset) stays beyond the range at off + 16
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, CP);
    const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16u, 0, CP);
    v[0] = __builtin_bit_cast(double, u32x2{a[0], a[1]});
    v[1] = __builtin_bit_cast(double, u32x2{a[2], a[3]});
    v[2] = __builtin_bit_cast(double, u32x2{b[0], b[1]});
    v[3] = __builtin_bit_cast(double, u32x2{b[2], b[3]});
}
template <int CP = 0>
__device__ __forceinline__ void bstore_point(const float (&v)[4], __amdgpu_buffer_rsrc_t r,
                                             unsigned off) {
    const f32x4 a{v[0], v[1], v[2], v[3]};
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, a), r, off, 0, CP);
}
template <int CP = 0>
__device__ __forceinline__ void bstore_point(const double (&v)[4], __amdgpu_buffer_rsrc_t r,
                                             unsigned off) {
    const u32x2 p0 = __builtin_bit_cast(u32x2, v[0]), p1 = __builtin_bit_cast(u32x2, v[1]);
    const u32x2 p2 = __builtin_bit_cast(u32x2, v[2]), p3 = __builtin_bit_cast(u32x2, v[3]);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{p0[0], p0[1], p1[0], p1[1]}, r, off, 0, CP);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{p2[0], p2[1], p3[0], p3[1]}, r, off + 16u, 0, CP);
}

// A w point of doubles in the array of structures lies as two pairs in two arrays, 2
// wfelems apart, so that the 64 lanes of a store fill whole lines.  As one 32-byte cell,
// stored in 16-byte halves past the caches, the register cost 7-16% more bytes than it
// has (512^3: 6.91 and 7.46 GB written in substeps 1 and 2 for 6.44; the step with
// diagnostics 6.29 -> 5.85 ms, 256^3 0.793 -> 0.738).
template <typename TW, int VS>
constexpr bool kWPairs = VS == 4 && sizeof(TW) == 8;
template <int CP = 0>
__device__ __forceinline__ void bload_pairs(double (&v)[4], __amdgpu_buffer_rsrc_t r0,
                                            __amdgpu_buffer_rsrc_t r1, unsigned off) {
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(r0, off, 0, CP);
    const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(r1, off, 0, CP);
    v[0] = __builtin_bit_cast(double, u32x2{a[0], a[1]});
    v[1] = __builtin_bit_cast(double, u32x2{a[2], a[3]});
    v[2] = __builtin_bit_cast(double, u32x2{b[0], b[1]});
    v[3] = __builtin_bit_cast(double, u32x2{b[2], b[3]});
}
template <int CP = 0>
__device__ __forceinline__ void bstore_pairs(const double (&v)[4], __amdgpu_buffer_rsrc_t r0,
                                             __amdgpu_buffer_rsrc_t r1, unsigned off) {
    const u32x2 p0 = __builtin_bit_cast(u32x2, v[0]), p1 = __builtin_bit_cast(u32x2, v[1]);
    const u32x2 p2 = __builtin_bit_cast(u32x2, v[2]), p3 = __builtin_bit_cast(u32x2, v[3]);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{p0[0], p0[1], p1[0], p1[1]}, r0, off, 0, CP);
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{p2[0], p2[1], p3[0], p3[1]}, r1, off, 0, CP);
}

// A TX x TY column tile, its halo and its LDS planes.
template <typename T, int TX, int TY>
struct SweepShape {
    static constexpr int NT = TX * TY;
    static constexpr int NW = NT / 64;              // wavefronts per workgroup
    static constexpr int W = TX + 2 * kR;           // LDS row length
    static constexpr int H = TY + 2 * kR;           // LDS rows
    static constexpr int PLANE = W * H;             // cells per plane
    static constexpr int HALO = 2 * kR * W + 2 * kR * TY;  // halo cells per plane
    static constexpr int NH = (HALO + NT - 1) / NT; // halo loads per thread
    // cell stride of a field in LDS: cell PLANE is a dummy target for unused
    // halo slots; even, so that pairs stay aligned beside an odd number of planes
    static constexpr int FS = (PLANE + 2) / 2 * 2;
};

// Element index of the ghost corner (-3, -3) of interior plane p mod nz.
__device__ __forceinline__ long long plane_corner(const Geom& g, int p) {
    const int pz = p < 0 ? p + g.nz : (p >= g.nz ? p - g.nz : p);
    return g.origin + (long long)pz * g.plane - kR * g.px - kR;
}

// Workgroup-to-XCD remapping of tiles (FD6_XCD_REMAP=0 disables it).
inline int xcd_remap() {
    static const int v = [] {
        const char* e = getenv("FD6_XCD_REMAP");
        return (e && e[0] == '0') ? 0 : 1;
    }();
    return v;
}

// Per-thread addressing of one tile: byte offsets, relative to the ghost
// corner (-3, -3) of a plane, of the cells this thread loads (beyond the
// plane's range the load returns 0; such cells are only read by threads whose
// outputs are dropped), LDS slots of its halo loads, and its output offsets.
template <typename T, int TX, int TY>
struct SweepCtx {
    using Sh = SweepShape<T, TX, TY>;
    unsigned goff_int;
    unsigned goff_h[Sh::NH];
    int loff_h[Sh::NH];   // LDS slot of each halo load (dummy cell if unused)
    unsigned lane_o;      // byte offset of the output point in a state plane
    unsigned lane_w;      // byte offset of the output point in a w plane
    unsigned plane_bytes, wplane_bytes;
};

// Addressing of the tile with corner (x0, y0).  The periodic boundary
// condition (Sec. 4) is resolved here: a halo cell outside the interior reads
// its periodic image, so the sweep kernels neither read nor need the ghost
// zone.  Cells beyond x < nx + 3, y < ny + 3 never feed a stored point and are
// dropped.
// VS: values per point in memory (1, or 4 for the array-of-structures
// layout); all byte offsets and plane sizes scale with it.  WRAP_ALL: every
// cell at any offset takes its periodic image and none is dropped (the
// extended tile of the substep-1+2 fusion, whose cells may lie a whole tile
// beyond the box).
template <typename T, typename TW, int TX, int TY, int VS = 1, bool WRAP_ALL = false>
__device__ __forceinline__ void sweep_ctx_init(SweepCtx<T, TX, TY>& X, const Geom& g, int x0,
                                               int y0) {
    using Sh = SweepShape<T, TX, TY>;
    // bytes per point, of w in one of the arrays that hold it
    constexpr int PT = VS * (int)sizeof(T), PW = (kWPairs<TW, VS> ? 2 : VS) * (int)sizeof(TW);
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    X.plane_bytes = (unsigned)(g.plane * (long long)PT);
    X.wplane_bytes = (unsigned)(g.wplane * (long long)PW);
    auto wrapped_off = [&](int gx, int gy) -> unsigned {  // gx, gy in [-3, ...)
        if constexpr (WRAP_ALL) {
            const int ix = ((gx % g.nx) + g.nx) % g.nx, iy = ((gy % g.ny) + g.ny) % g.ny;
            return (unsigned)(((iy + kR) * g.px + (ix + kR)) * PT);
        }
        if (gx >= g.nx + kR || gy >= g.ny + kR) return kDropOffset;
        const int ix = gx < 0 ? gx + g.nx : (gx >= g.nx ? gx - g.nx : gx);
        const int iy = gy < 0 ? gy + g.ny : (gy >= g.ny ? gy - g.ny : gy);
        return (unsigned)(((iy + kR) * g.px + (ix + kR)) * PT);
    };
    X.goff_int = wrapped_off(x0 + tx, y0 + ty);
#pragma unroll
    for (int h = 0; h < Sh::NH; ++h) {
        const int e = threadIdx.x + h * Sh::NT;
        int r = 0, c = 0;
        if (e < 2 * kR * Sh::W) {
            const int row = e / Sh::W;
            r = row < kR ? row : row + TY;
            c = e - row * Sh::W;
        } else {
            const int e2 = e - 2 * kR * Sh::W;
            r = kR + e2 / (2 * kR);
            const int cc = e2 % (2 * kR);
            c = cc < kR ? cc : cc + TX;
        }
        const bool in_range = e < Sh::HALO;
        X.goff_h[h] = in_range ? wrapped_off(x0 - kR + c, y0 - kR + r) : kDropOffset;
        X.loff_h[h] = in_range ? r * Sh::W + c : Sh::PLANE;
    }
    const int xo = x0 + tx, yo = y0 + ty;
    const bool store = xo < g.nx && yo < g.ny;
    X.lane_o = store ? (unsigned)(((yo + kR) * g.px + (xo + kR)) * PT) : kDropOffset;
    X.lane_w = store ? (unsigned)((yo * g.wpx + xo) * PW) : kDropOffset;
}

// Workgroup index -> (tile x, tile y, z chunk).  Each XCD receives every 8th
// workgroup; with remap the grid is renumbered so that one XCD takes a
// contiguous range of tiles instead.  Within a z chunk the tiles are ordered
// in column blocks gx tiles wide (x fastest inside a block, then y, then the
// next block), so the tiles an XCD holds at once cover a near-square region
// and the halo rows and columns they read from outside it (from HBM rather
// than from that XCD's L2) are few.  gx >= ntx is plain row order.
struct SweepGrid {
    int ntx, nty, zlen, blocks;
    int gx;     // column-block width in tiles
    int remap;  // 1: contiguous tile ranges per XCD
};

// Column-block width that minimises the halo fraction of the region one XCD
// holds at once (per_xcd tiles of tx x ty; a region spanning a whole
// periodic axis reads no halo along it).  FD6_SWEEP_GX > 0 overrides it.
inline int sweep_block_width(int ntx, int nty, int tx, int ty, int per_xcd) {
    static const int forced = [] {
        const char* e = getenv("FD6_SWEEP_GX");
        return e ? atoi(e) : 0;
    }();
    if (forced > 0) return forced < ntx ? forced : ntx;
    int best = ntx;
    double best_cost = 1e30;
    for (int gx = ntx; gx >= 1; --gx) {
        const int rows = (per_xcd + gx - 1) / gx;
        const double xh = gx >= ntx ? 0.0 : 2.0 * kR / (gx * tx);
        const double yh = rows >= nty ? 0.0 : 2.0 * kR / ((double)rows * ty);
        if (xh + yh < best_cost - 1e-12) best_cost = xh + yh, best = gx;
    }
    return best;
}

// zchunk > 0 fixes the chunk length (planes); 0 chooses it.  resident: how
// many workgroups of the kernel the device holds at once.  The automatic
// choice minimises (rounds of resident workgroups) x (planes swept per chunk,
// including the 6 re-read planes), i.e. it prefers long chunks unless they
// leave compute units idle.  Chunks under 8 planes serve small boxes, where one
// round of workgroups does not fill the device (a plane of such a chunk costs
// 1.0 us in FP32, the refill and the launch 7 us: 32^3, ms per step with
// diagnostics, 32 x 8 tiles: 0.049 with 8 planes, 0.037 with 4, 0.031 with 2).
// most > 0: the automatic choice stays within so many workgroups where it can (the
// fused diagnostics have a slot each; 704^3 FP32 with 32 x 8 tiles in 5 chunks is past
// them, and the separate pass costs 1.48 of the step's 11.4 ms).
inline SweepGrid sweep_grid(const Geom& g, int tx, int ty, int zchunk, int resident,
                            int most = 0) {
    SweepGrid s;
    s.ntx = (g.nx + tx - 1) / tx;
    s.nty = (g.ny + ty - 1) / ty;
    const long long tiles = (long long)s.ntx * s.nty;
    int nch = 1;
    if (zchunk > 0) {
        nch = (g.nz + zchunk - 1) / zchunk;
    } else {
        const long long res = resident > 0 ? resident : 1;
        long long best = -1;
        for (int c = 1; c <= g.nz && (c <= (g.nz + 7) / 8 || tiles * c <= res); ++c) {
            if (most > 0 && c > 1 && tiles * c > most) break;
            const long long len = (g.nz + c - 1) / c;
            const long long cost = ((tiles * c + res - 1) / res) * (len + 2 * kR);
            if (best < 0 || cost < best) best = cost, nch = c;
        }
    }
    s.zlen = (g.nz + nch - 1) / nch;
    nch = (g.nz + s.zlen - 1) / s.zlen;
    s.blocks = (int)(tiles * nch);
    s.remap = xcd_remap();
    s.gx = s.remap ? sweep_block_width(s.ntx, s.nty, tx, ty, resident > 8 ? resident / 8 : 1)
                   : s.ntx;
    return s;
}

inline int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus <= 0)
        cus = 256;
    return cus;
}

// Workgroups of Kernel (block threads) the current device holds at once
// (the per-CU occupancy is queried once per kernel).
template <auto Kernel>
int resident_blocks(int block) {
    static const int per_cu = [&] {
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, Kernel, block, 0) != hipSuccess)
            n = 1;
        return n > 0 ? n : 1;
    }();
    return per_cu * device_cus();
}

struct TileXY {
    int tx, ty, zb, ze;
};

__device__ __forceinline__ TileXY sweep_tile_of(const Geom& g, int TX, int TY,
                                                const SweepGrid& m) {
    int b = blockIdx.x;
    const int nb = gridDim.x;
    if (m.remap && (nb & 7) == 0) b = (b & 7) * (nb >> 3) + (b >> 3);
    const int per = m.ntx * m.nty;
    const int ch = b / per;
    int l = b - ch * per;                     // tile within the chunk
    const int blk = l / (m.gx * m.nty);       // column block
    const int bx0 = blk * m.gx;
    const int bw = min(m.gx, m.ntx - bx0);    // the last block may be narrower
    l -= blk * m.gx * m.nty;
    const int tiy = l / bw;
    const int tix = bx0 + (l - tiy * bw);
    const int zb = ch * m.zlen;
    return TileXY{tix * TX, tiy * TY, zb, min(zb + m.zlen, g.nz)};
}

// FP64 diagnostics of one point of the new state (the quantities of the
// standalone reduction): per thread, red = {sum rho, sum rho |u|^2, sum
// lnrho, max |u|^2} and bad = points holding a non-finite value.  The caller
// leaves out points that are not outputs.  The kinetic energy's factor
// 1/2 is applied once per workgroup (exact).  Non-finite values are found by
// class checks of the stored values; the mass and kinetic-energy terms of
// such a point are meaningless and the final combination reports them as
// NaN whenever bad > 0.
template <typename T>
__device__ __forceinline__ void red_point(double red[4], int& bad, T lr, T ux, T uy, T uz) {
    const bool finite = __builtin_isfinite(lr) && __builtin_isfinite(ux) &&
                        __builtin_isfinite(uy) && __builtin_isfinite(uz);
    bad += finite ? 0 : 1;
    const double l = (double)lr, a = (double)ux, b = (double)uy, c = (double)uz;
    const double rho = exp_fp64<sizeof(T) == 8>(l);  // FP64 sweeps: no vector registers to spare
    const double u2 = a * a + b * b + c * c;
    red[0] += rho;
    red[1] += rho * u2;
    red[2] += l;
    red[3] = __builtin_fmax(red[3], u2);
}

// Combines the per-thread diagnostics of a workgroup in a fixed order (xor
// tree within each wave, then waves in order) and stores the partial:
// sums for slots 0-2 and 4, the maximum for slot 3.
template <int NW>
__device__ __forceinline__ void red_store_n(const double red[4], int bad, double* part) {
    double v[5] = {red[0], 0.5 * red[1], red[2], red[3], (double)bad};
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const double o = __shfl_xor(v[i], off, 64);
            v[i] = i == 3 ? (o > v[i] ? o : v[i]) : v[i] + o;
        }
    }
    __shared__ double sw[NW][5];
    const int wv = threadIdx.x / 64;
    if ((threadIdx.x & 63) == 0) {
#pragma unroll
        for (int i = 0; i < 5; ++i) sw[wv][i] = v[i];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        for (int k = 0; k < NW; ++k)
#pragma unroll
            for (int i = 0; i < 5; ++i)
                a[i] = i == 3 ? (sw[k][i] > a[i] ? sw[k][i] : a[i]) : a[i] + sw[k][i];
        double* p = part + (size_t)blockIdx.x * kReduceSlots;
        p[0] = a[0];
        p[1] = a[1];
        p[2] = a[2];
        p[3] = sqrt(a[3]);  // max |u| = sqrt(max |u|^2): sqrt is monotonic
        p[4] = a[4];
    }
}

// Kernel shapes of the z-sweep substeps.  Index 0 is the direct kernel (one
// thread per point, taps from the ghost zone); the others are (TX, TY) column
// tiles.  pd: how many planes ahead the loader fetches (1, 2 or 4; 2 and 4 also
// load the update's other operand one step early).  FP64 states always fetch one:
// a second set of planes fills the registers (512^3, ms per step: 7.33 with one
// plane, 7.30 with two; with diagnostics 7.50 and 7.96, which spills).  Shape 9 is
// shape 2 for boxes with one array per field.
struct TileCfg {
    int tx, ty, pd;
    bool soa;  // one array per field only
    bool nt;   // new state and RK register streamed past the caches
};
constexpr TileCfg kTiles[] = {
    {0, 0, 1, false, false},  {64, 4, 1, false, true},  {64, 8, 1, false, true},
    {128, 4, 1, false, true}, {32, 8, 1, false, true},  {64, 4, 2, false, true},
    {64, 8, 2, false, true},  {128, 4, 2, false, true}, {32, 8, 2, false, true},
    {64, 8, 1, true, true},   {64, 8, 4, false, true},  {64, 8, 1, false, false},
    {64, 8, 2, false, false}, {32, 8, 2, false, false}};
template <typename T, int PD>
constexpr int kPd = sizeof(T) == 8 ? 1 : PD;
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// Shape and z-chunk of a box that has neither set nor tuned: a wide (64 x 8) or a
// narrow (32 x 8) tile.  Both run two waves per SIMD, so the sweeps of a round cost
// the same; ms per step with diagnostics, wide against narrow:
//  * FP32 state and register, array of structures: narrow, 3-6% faster at every
//    size (its two workgroups per compute unit wait at separate barriers): 64^3
//    0.035 / 0.036, 96^3 0.062 / 0.052, 128^3 0.085 / 0.083, 256^3 0.520 / 0.508,
//    384^3 1.86 / 1.78, 640^3 8.40 / 7.98.  Whole columns in more than one round
//    are the exception (512^3: 4.11 / 4.21); in two chunks they are not (4.03).
//    There substeps 2 and 3, which read two state sets and are bound by HBM, take wide
//    columns if those need no more plane steps, one plane ahead with the diagnostics
//    (the step in ms, all narrow in two chunks / substep 1 only: 512^3 4.04 / 3.93, 300
//    x 512 x 512 2.41 / 2.33; in boxes that are swept in chunks anyway a change of shape
//    between the substeps costs more than it gives: 576^3 5.78 / 5.80, 640^3 7.85 /
//    7.90).
//  * Otherwise wide, whose halo costs less where a cell's fields lie apart or the
//    state is twice as large (FP32 one array per field 256^3 0.569 / 0.619, FP64
//    512^3 7.55 / 8.11, 19-point FP32 256^3 0.759 / 0.840), unless the box is no
//    wider than the narrow tile (32^3: FP32 0.032 / 0.028, FP64 0.038 / 0.034) or
//    the wide tile needs over 6/5 of the narrow one's plane steps (FP64 96^3: 16
//    against 13 per workgroup, 0.093 / 0.086), 3/2 with an FP32 state in one array per
//    field, whose narrow tiles spend more on their halo (150 x 75 x 101: 19 against 17,
//    0.116 / 0.139; 19-point 78 x 84 x 150: 20 against 16, 0.138 / 0.167).  Plane steps
//    alone do not decide: over 33 random boxes of 0.3 to 8 million points whose wide
//    tiles need 1.05-1.55 times the steps, wide / narrow was 0.89-1.19 in FP64 with one
//    array per field (1.02-1.27 with the array of structures), 0.79-1.22 in FP32 and
//    0.77-1.25 with the 19-point method in FP32.
struct AutoShape {
    int tile, zchunk;
};
template <typename T, typename TW, int VS, bool P19>
AutoShape auto_shape(const Geom& g, int zchunk, int s, bool red, bool forced) {
    // one plane ahead where two do not pay (1-3% in 19-point FP32, 0.7% with the FP64
    // register)
    constexpr bool pd1 = sizeof(T) == 8 || P19 || sizeof(TW) == 8;
    // cached stores for FP64 points, whose 32 bytes go out in two halves that the cache
    // merges (ms per step with diagnostics, cached / past the caches: 512^3 7.33 / 7.47,
    // 256^3 0.920 / 0.942, 400 x 300 x 500 3.50 / 3.58; 192^3 0.446 / 0.438 loses 2%, and
    // no line is drawn for it)
    constexpr bool halves = sizeof(T) == 8 && VS == 4;
    // ... and two planes ahead in the diagnostics sweep beside the FP64 register (the
    // step at 256^3 0.705 / 0.720 with one, 500 x 300 x 400 2.74 / 2.82; without
    // diagnostics 512^3 5.81 / 5.70)
    const int wide = halves ? 11 : !pd1 || (red && VS == 4 && !P19) ? 6 : 2;
    constexpr int narrow = halves ? 13 : pd1 ? 4 : 8;
    const int cus = device_cus();
    auto grid = [&](int tile) {
        const int tx = kTiles[tile].tx, ty = kTiles[tile].ty;
        return sweep_grid(g, tx, ty, zchunk, cus * (512 / (tx * ty)));
    };
    const SweepGrid n = grid(narrow);
    const int rn = (n.blocks + 2 * cus - 1) / (2 * cus);
    if (VS == 4 && std::is_same_v<T, float> && std::is_same_v<TW, float>) {
        const bool columns = zchunk == 0 && rn > 1 && n.zlen >= g.nz;
        if (columns && s > 1) {
            const int tile = red ? 2 : forced ? wide : 10;
            const SweepGrid w = grid(tile);
            if (((w.blocks + cus - 1) / cus) * (long long)(w.zlen + 2 * kR) <=
                rn * (long long)(n.zlen + 2 * kR))
                return AutoShape{tile, zchunk};
        }
        return AutoShape{narrow, columns ? (g.nz + 1) / 2 : zchunk};
    }
    if (g.nx <= kTiles[narrow].tx) return AutoShape{narrow, zchunk};
    const SweepGrid w = grid(wide);
    const int rw = (w.blocks + cus - 1) / cus;
    const long long cn = (long long)rn * (n.zlen + 2 * kR), cw = (long long)rw * (w.zlen + 2 * kR);
    const bool fewer = sizeof(T) == 4 && VS == 1 ? 3 * cn < 2 * cw : 6 * cn < 5 * cw;
    return AutoShape{fewer ? narrow : wide, zchunk};
}

// Calls f(std::integral_constant<int, tile>) so that f can use kTiles[tile]
// as template arguments; returns `bad` for an out-of-range tile.
template <int I = 0, typename R, typename F>
R with_tile(int tile, R bad, F&& f) {
    if constexpr (I < kNumTiles) {
        if (tile == I) return f(std::integral_constant<int, I>{});
        return with_tile<I + 1>(tile, bad, f);
    } else {
        return bad;
    }
}

}  // namespace
}  // namespace fd6
