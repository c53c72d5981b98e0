// 55-point fused substep (Sec. 4.1, Algorithm 2): the right-hand side of the
// continuity and momentum equations (Sec. 2.1) from sixth-order first, second
// and bidiagonal mixed differences (Sec. 2.3), followed by the 2N-RK3 update
// (Sec. 2.4) of the RK3 register w and of the output state, in one pass.
//
// Kernel design for gfx950 (the paper's K40 shared-memory cube and rolling
// cache are not reused):
//
//  * One workgroup owns a TX x TY column tile of the xy-plane and sweeps a
//    chunk of z.  Each step loads one new xy-plane (tile + 3-cell halo) of the
//    four fields from HBM into LDS (coalesced x-rows, double buffered, one
//    barrier per plane), prefetching the next plane into registers.  LDS holds
//    the fields in pairs (PlaneBuf).
//  * From that plane every thread forms, for its own column, the x and y first
//    derivatives of all fields and all of the right-hand side that needs no z
//    derivative, into the pending sum of that plane's output.
//  * z derivatives come from a register queue holding the thread's column
//    over 7 planes.
//  * The xz and yz mixed derivatives are built by scatter: the bidiagonal
//    stencil at output plane z is sum_k c_k [A_k(z+k) - A_k(z-k)], where
//    A_k(p) = f(x+k, p) - f(x-k, p) is the same x (or y) difference the plane
//    step already forms, so each plane adds +-c_k A_k into pending sums of the
//    output planes p -+ k (a register ring of 8 planes).
//  * Output plane z is finished 3 planes behind the load front: the terms with z
//    derivatives join, and the RK3 update is written out.
//  * The z loop is unrolled by 8 so every ring index is a compile-time
//    register; the workgroup-to-tile map gives each XCD a near-square block
//    of neighbouring tiles, so most halo cells are served from its L2.
//  * What bounds it, at 512^3 in the array-of-structures layout with diagnostics: FP32
//    3.91 ms per step, HBM in substeps 2 and 3 (4.8 and 4.3 TB/s of their actual
//    traffic in the mean of a trace, 5.1 and 4.6 at best, where a 1 GiB copy runs at
//    5.1) and instruction issue in substep 1 (VALU busy 90% of the cycles; 223-273
//    vector instructions per point, 254-312 before).  FP64 HBM
//    since two waves fit a SIMD: 7.35 ms per step against 10.2 with one wave.
//  * Template switches: VS = 4 reads and writes the array-of-structures
//    layout (one 16-byte access per cell and field set); NT streams the new
//    state and the RK3 register past the caches; FRC adds the external
//    force; RED accumulates the FP64 diagnostics; P19 turns the sweep into
//    that of the 19-point method, over the state and its divergence.
#pragma once

#include "sweep_common.hpp"

namespace fd6 {
namespace {

// ---------------------------------------------------------------------------
// Shared per-point pieces
// ---------------------------------------------------------------------------

// Right-hand side from the derivatives at one point (eqs. continuity,
// navierstokes with f = 0, tensor):
//   u: centre velocity, g = grad lnrho, J[i][a] = d_a u_i,
//   L[i] = nu (lap u_i + (1/3) d_i div u) (already scaled by nu).
template <typename T>
__device__ __forceinline__ void assemble_rhs(const T u[3], const T g[3], const T J[3][3],
                                             const T L[3], T nu, T cs2, T r[4]) {
    const T div = J[0][0] + J[1][1] + J[2][2];
    r[0] = -(u[0] * g[0] + u[1] * g[1] + u[2] * g[2]) - div;
    // 2 S = J + J^T - (2/3) div I, and 2 nu S . grad lnrho = nu (2S) g
    const T d23 = div * T(2.0 / 3.0);
    const T s01 = J[0][1] + J[1][0], s02 = J[0][2] + J[2][0], s12 = J[1][2] + J[2][1];
    const T s00 = T(2) * J[0][0] - d23, s11 = T(2) * J[1][1] - d23, s22 = T(2) * J[2][2] - d23;
    const T sg[3] = {s00 * g[0] + s01 * g[1] + s02 * g[2], s01 * g[0] + s11 * g[1] + s12 * g[2],
                     s02 * g[0] + s12 * g[1] + s22 * g[2]};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const T adv = u[0] * J[i][0] + u[1] * J[i][1] + u[2] * J[i][2];
        r[1 + i] = (L[i] + nu * sg[i]) - cs2 * g[i] - adv;
    }
}

// 2N-RK3 update of one value (eq. 2N-RK_scheme, Algorithm 2) with the register
// formed from the states: w(s - 1) = (in - prev) / beta(s - 1), where prev is
// the previous substep's input at this point.  Substeps 2 and 3 read prev from
// the place they then write, so no register is stored or read: 128 instead of
// 160 bytes per point and step in FP32 (512^3 array of structures, 10 steps
// with diagnostics and a snapshot: 49.0 -> 45.5 ms; FP64, 4 steps: 50.7 -> 42.8
// ms).  It also follows the rounding of the
// stored states: of the errors e1, e2, e3 made when the three substeps round
// their new states, on a mode whose time step times eigenvalue is z,
//   (1/2 + z^2/2) e1 + (0.32 + (8/15) z) e2 + e3
// remains after the step, with the register kept apart
//   (1 + (5/6) z + z^2/2) e1 + (1 + (8/15) z) e2 + e3.
// That is less on waves and on modes that decay slowly, more on those near the
// scheme's diffusive limit z = -2.51: the error of one FP32 step of grid-scale noise
// is 0.69 of the direct kernel's (which keeps it) where viscosity takes z to -0.1,
// 0.85 at -0.6, 1.06 at -1 and 1.4 from -2 on.
template <int S, typename T>
__device__ __forceinline__ T rk_update(T in, T r, T prev, const RKCoef<T>& rk) {
    T q = r;
    if constexpr (S != 1) q = rk.c * (in - prev) + q;
    return rk.b * q + in;
}

// The same with a register wider than the state (FP64 beside an FP32 state),
// which stays in memory: w <- alpha w + dt r, out <- in + beta w.  The rounding
// error e of the stored state is known here, and w takes up the multiple of it
// (rk.c) whose later contributions to the state cancel most of it.  With z the
// time step times the linear operator's eigenvalue and k e taken up, what is
// left of e at the end of the step is
//   substep 1:  (1 - k / 6) + (5/6) (1 - k / 3) z + z^2 / 2
//   substep 2:  (1 - 51/80 k) + (8/15) z
// times e.  Rounding errors are white in space, so z = i y with y^2 = 0.2 (a
// velocity) to 0.6 (lnrho) in the mean at Courant number 0.4: k = 4 leaves 0.07
// and 0.05 of e's variance in substep 1 (forming w from the states is k = 3:
// 0.16 and 0.05), k = 80/51 the least in substep 2.  (On decaying modes it leaves less
// of e down to z = -0.6, more beyond.)
template <int S, typename T, typename TW>
__device__ __forceinline__ T rk_update_reg(T in, T r, TW& w, const RKCoef<TW>& rk) {
    TW wn = rk.dt * TW(r);
    if constexpr (S != 1) wn = rk.alpha * w + rk.dt * TW(r);
    const TW v = rk.beta * wn + TW(in);
    const T out = T(v);
    if constexpr (S != 3) w = rk.c * (TW(out) - v) + wn;
    return out;
}

// Whether the RK3 register is kept in memory (wider than the state) or formed
// from the states.
template <typename T, typename TW>
constexpr bool kRegInMemory = !std::is_same_v<T, TW>;

// ---------------------------------------------------------------------------
// Direct kernel: one thread per point, every tap read from global memory.
// Kept as the simplest statement of the per-point arithmetic.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T d1_at(const T* f, long long c, long long s, const T* w) {
    return w[0] * (f[c + s] - f[c - s]) + w[1] * (f[c + 2 * s] - f[c - 2 * s]) +
           w[2] * (f[c + 3 * s] - f[c - 3 * s]);
}

template <typename T>
__device__ __forceinline__ T d2w_at(const T* f, long long c, long long s, const T* w) {
    return w[0] * f[c] + w[1] * (f[c + s] + f[c - s]) + w[2] * (f[c + 2 * s] + f[c - 2 * s]) +
           w[3] * (f[c + 3 * s] + f[c - 3 * s]);
}

template <typename T>
__device__ __forceinline__ T mix_at(const T* f, long long c, long long sa, long long sb,
                                    const T* w) {
    T acc = T(0);
#pragma unroll
    for (int k = 1; k <= 3; ++k) {
        const T t = (f[c + k * sa + k * sb] - f[c - k * sa + k * sb]) +
                    (f[c - k * sa - k * sb] - f[c + k * sa - k * sb]);
        acc += w[k - 1] * t;
    }
    return acc;
}

template <typename T, typename TW, int S, bool FRC>
__global__ __launch_bounds__(256) void substep55_direct(Geom g, Fields4<T> in, Fields4<T> out,
                                                        Fields4<TW> w, Coef<T> cf, RKCoef<TW> rk,
                                                        ForceArgs<T> fa) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    const long long c = g.origin + (long long)k * g.plane + (long long)j * g.px + i;
    const long long s[3] = {1, g.px, g.plane};
    T gr[3], J[3][3], L[3], u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) gr[a] = d1_at(in.f[0], c, s[a], cf.d1[a]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        u[q] = in.f[1 + q][c];
#pragma unroll
        for (int a = 0; a < 3; ++a) J[q][a] = d1_at(in.f[1 + q], c, s[a], cf.d1[a]);
    }
    // L_i = sum_a lw[i][a] . D2_a u_i + (1/3) sum_{j != i} D_ij u_j (nu folded)
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        T acc = T(0);
#pragma unroll
        for (int a = 0; a < 3; ++a) acc += d2w_at(in.f[1 + q], c, s[a], cf.lw[q][a]);
        L[q] = acc;
    }
    L[0] += mix_at(in.f[2], c, s[0], s[1], cf.mw[0]) + mix_at(in.f[3], c, s[0], s[2], cf.mw[1]);
    L[1] += mix_at(in.f[1], c, s[0], s[1], cf.mw[0]) + mix_at(in.f[3], c, s[1], s[2], cf.mw[2]);
    L[2] += mix_at(in.f[1], c, s[0], s[2], cf.mw[1]) + mix_at(in.f[2], c, s[1], s[2], cf.mw[2]);
    T r[4];
    assemble_rhs(u, gr, J, L, cf.nu, cf.cs2, r);
    if constexpr (FRC) {  // f = a cos(k.x + phase), eq. (forcing)
        const ForceDev<T>* fd = fa.dev;
        const T ph = T(cos(fd->kx * (i * fd->dx) + fd->ky * (j * fd->dy) + fd->kz * (k * fd->dz) +
                           fd->phase));
#pragma unroll
        for (int q = 0; q < 3; ++q) r[1 + q] += fd->a[q] * ph;
    }
    const long long cw = (long long)k * g.wplane + (long long)j * g.wpx + i;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        TW wv = rk.dt * TW(r[q]);
        if constexpr (S != 1) wv = rk.alpha * w.f[q][cw] + rk.dt * TW(r[q]);
        out.f[q][c] = T(TW(in.f[q][c]) + rk.beta * wv);
        if constexpr (S != 3) w.f[q][cw] = wv;
    }
}

// ---------------------------------------------------------------------------
// z-sweep kernel
// ---------------------------------------------------------------------------

// Values of a plane that wait for its output, 3 planes later: of the right-hand
// side everything that holds no z derivative is formed with the plane itself and
// added to the pending L; the terms with one need nu d_x lnrho, nu d_y lnrho,
// d_x uz, d_y uz, d_x ux + d_y uy, and lnrho's in-plane advection.
constexpr int kInPlane = 6;
// They wait in per-thread LDS slots (a ring of 3 planes) in FP64, where that
// keeps a thread within 256 registers and so two waves on a SIMD; in registers
// in FP32, and where the slots do not fit beside NF field planes.
constexpr int kLdsBytes = 160 * 1024;
template <typename T, int TX, int TY, int NF>
constexpr bool kInPlaneLds =
    sizeof(T) == 8 && sizeof(T) * (2 * NF * SweepShape<T, TX, TY>::FS + 3 * kInPlane * TX * TY) <=
                          kLdsBytes - 1024;
// LDS elements of a workgroup's in-plane values
template <typename T, int TX, int TY, int NF>
constexpr int kInPlaneElems = kInPlaneLds<T, TX, TY, NF> ? 3 * kInPlane * TX * TY : 2;
// LDS elements of the diagnostics' per-thread accumulators, which join the
// in-plane values there where that costs no workgroup: a compute unit holds 512 threads
// at two waves per SIMD.  Only the FP64 32 x 8 tile of the 19-point method is too full;
// its accumulators stay in registers (3-9 spilled), and the diagnostics in the sweep,
// instead of a pass of their own (ms per step with diagnostics, LDS and a pass /
// registers: 2048 x 6 x 6 0.120 / 0.111, 1024 x 16 x 16 0.123 / 0.112, 96^3 0.141 / 0.136).
template <typename T, int TX, int TY, int NF>
constexpr int kRedElems = [] {
    constexpr int most = 512 / (TX * TY);
    constexpr int base = (int)sizeof(T) *
                         (2 * NF * SweepShape<T, TX, TY>::FS + 3 * kInPlane * TX * TY);
    auto held = [](int bytes) {
        const int n = kLdsBytes / (bytes + 1024);
        return n < most ? n : most;
    };
    const int with = held(base + 4 * TX * TY * (int)sizeof(T));
    return kInPlaneLds<T, TX, TY, NF> && with > 0 && with == held(base) ? 4 * TX * TY : 0;
}();
// Waves per SIMD the register budget is set for.
constexpr int kMinWaves = 2;

// Terms w[k-1] s of a stencil whose weights w are 270, -27 and 2 times w[3]
// (second and mixed derivatives), k = 1, 2, 3 in turn, added to acc.  FP32 takes
// the three weights from scalar registers.  In FP64 all weights of the sweep
// would fill 88 of the 102 (and spilled 80 into vector lanes: 51 lane moves per
// point and plane), so the integers are factored out there: the terms gather in
// part, and end() adds it with the factor, for one instruction more.
template <typename T>
struct Weighted {
    T part;
    template <int K>
    __device__ __forceinline__ void add(const T* w, T s, T& acc) {
        if constexpr (sizeof(T) == 8) {
            constexpr T c = K == 1 ? T(270) : (K == 2 ? T(-27) : T(2));
            part = K == 1 ? c * s : c * s + part;
        } else {
            acc = w[K - 1] * s + acc;
        }
    }
    __device__ __forceinline__ void end(const T* w, T& acc) {
        if constexpr (sizeof(T) == 8) acc = w[3] * part + acc;
    }
};

template <typename T, typename TW, int NH>
struct SweepRegs {
    using Reg = std::conditional_t<kRegInMemory<T, TW>, TW, T>;
    // fields in the order ux, uy, uz, lnrho, that of a point's values in the array
    // of structures
    T q[4][8];       // raw column values of the 4 fields, ring over planes
    T L[3][8];       // pending momentum right-hand sides, ring over output planes
    T dd[4][kInPlane];  // what an output still needs from its own plane, ring of 4 planes
    T pf[4][4];      // prefetched interior values of the next plane(s)
    T ph[4][NH][4];  // prefetched halo values of the next plane(s)
    // 19-point method: the same of the divergence field
    T qd[8], pfd[4], phd[4][NH];
    int slot;        // in-plane values in LDS: the plane's slot
    Reg wq[2][4];    // previous substep's input, or the RK3 register in memory, at the
                     // output point (PD >= 2: loaded a step early)
    double red[4];   // fused diagnostics of the thread's column (RED): sum rho,
                     // sum rho u^2, sum lnrho, max u^2
    int bad;         // RED: points of the column with a non-finite value
    T fc, fs;        // FRC: cos / sin(kx x + ky y) of the thread's column
    T fa[3];         // FRC: force amplitude vector
};

// Memory operations of a plane step are never skipped by a branch: a step
// that has nothing to load or store gives its descriptors a zero range (loads
// return 0, stores are dropped).  Branch-free memory code lets the compiler
// count outstanding loads exactly across steps instead of draining the memory
// pipeline (stores share the load counter on this architecture).

// Loads plane `corner` of the four fields (this thread's cells) into
// register set RS; bytes = 0 loads nothing.  One array per field: the arrays of a
// state set follow one another, felems apart, so one pointer serves all (four
// would cost scalar registers the weights need).
template <int RS, int VS, bool P19, typename T, typename TW, int TX, int TY, int NH>
__device__ __forceinline__ void sweep_prefetch(SweepRegs<T, TW, NH>& R,
                                               const SweepCtx<T, TX, TY>& X,
                                               const Fields4<T>& in, long long felems,
                                               const T* dv, long long corner,
                                               unsigned bytes) {
    if constexpr (P19) {
        const __amdgpu_buffer_rsrc_t rs = plane_rsrc(dv + corner, bytes);
        R.pfd[RS] = bload((T*)nullptr, rs, X.goff_int);
#pragma unroll
        for (int h = 0; h < NH; ++h) R.phd[RS][h] = bload((T*)nullptr, rs, X.goff_h[h]);
    }
    if constexpr (VS == 4) {
        const __amdgpu_buffer_rsrc_t rs = plane_rsrc(in.f[1] + 4 * corner, bytes);
        bload_point(R.pf[RS], rs, X.goff_int);
#pragma unroll
        for (int h = 0; h < NH; ++h) bload_point(R.ph[RS][h], rs, X.goff_h[h]);
    } else {
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const __amdgpu_buffer_rsrc_t rs = plane_rsrc(in.f[0] + (corner + ((f + 1) & 3) * felems), bytes);
            R.pf[RS][f] = bload((T*)nullptr, rs, X.goff_int);
#pragma unroll
            for (int h = 0; h < NH; ++h) R.ph[RS][h][f] = bload((T*)nullptr, rs, X.goff_h[h]);
        }
    }
}

// What the update of output plane o needs beside the plane's input: the
// previous substep's input, which the state set being written still holds
// there, or the RK3 register.  on: the plane is an output plane of the chunk.
template <int RS, bool NT, int VS, typename T, typename TW, typename Ctx, int NH>
__device__ __forceinline__ void load_prev(SweepRegs<T, TW, NH>& R, const Ctx& X,
                                          const Fields4<T>& out, const Fields4<TW>& w,
                                          const Geom& g, int o, bool on) {
    constexpr int CP = NT ? kNonTemporal : 0;
    constexpr bool REG = kRegInMemory<T, TW>;
    using P = typename SweepRegs<T, TW, NH>::Reg;
    const long long at = REG ? (long long)o * g.wplane
                             : g.origin + (long long)o * g.plane - kR * g.px - kR;
    const unsigned bytes = on ? (REG ? X.wplane_bytes : X.plane_bytes) : 0u;
    const unsigned lane = REG ? X.lane_w : X.lane_o;
    auto base = [&](int f) -> const P* {
        if constexpr (REG)
            return VS == 4 ? w.f[1] : w.f[0] + ((f + 1) & 3) * g.wfelems;
        else
            return VS == 4 ? out.f[1] : out.f[0] + ((f + 1) & 3) * g.felems;
    };
    if constexpr (REG && kWPairs<TW, VS>) {
        const P* const p = base(0) + 2 * at;
        bload_pairs<CP>(R.wq[RS], plane_rsrc(p, bytes), plane_rsrc(p + 2 * g.wfelems, bytes),
                        lane);
    } else if constexpr (VS == 4) {
        bload_point<CP>(R.wq[RS], plane_rsrc(base(0) + 4 * at, bytes), lane);
    } else {
#pragma unroll
        for (int f = 0; f < 4; ++f)
            R.wq[RS][f] = bload<CP>((P*)nullptr, plane_rsrc(base(f) + at, bytes), lane);
    }
}

// Makes the compiler form a value where it stands (no instruction).
template <typename T>
__device__ __forceinline__ void keep_here(T& x) {
    asm volatile("" : "+v"(x));
}

// A plane buffer in LDS holds the cells of the tile and its halo as pairs, first
// (ux, uy), then (uz, lnrho), then, for the 19-point method, the divergence.  A
// tap brings both fields of a pair in one access, and every tap of a thread is
// at a constant offset from one address.  (One plane per field needed a register
// for nearly every row and field: two-address reads reach only 255 elements.)
template <typename T, int FS>
struct PlaneBuf {
    using T2 = T __attribute__((ext_vector_type(2)));
    T* b;
    __device__ __forceinline__ T2* u() const { return reinterpret_cast<T2*>(b); }
    __device__ __forceinline__ T2* v() const { return reinterpret_cast<T2*>(b) + FS; }
    __device__ __forceinline__ T* d() const { return b + 4 * FS; }
    __device__ __forceinline__ void put(int cell, const T (&x)[4]) const {
        u()[cell] = T2{x[0], x[1]};
        v()[cell] = T2{x[2], x[3]};
    }
};

// One step of the sweep: plane p = zb - 3 + t comes in, output plane p - 3 is
// finished.  PH = t mod 8 (ring positions), ST: the step's number where it is one
// of the first 6 of a chunk, which fill the rings and have no output; 6 later.
// A plane below the chunk (ST < 3) only fills the z queues and contributes the
// xz / yz terms of the outputs it reaches, and planes 0 .. 2 (ST 3 .. 5) lack
// the output: of the 6 steps' arithmetic 2.3 are left, which matters where
// chunks are short (small boxes, ensembles).
//
// TB selects the two stages of the substep-1+2 fusion (fused12_tile): 0 is
// the plain sweep; 1 is substep 1 over the extended region, whose new state
// goes to the LDS plane buffer tb_u (layout of the inner tile's sweep) and
// whose input, for the inner columns, to the LDS ring tb_w; 2 is substep 2 of
// the inner tile, which takes its plane from tb_u (passed as lds, loaded by
// stage 1) and the substep-1 input from tb_w, leaves the substep-1 state in w,
// and starts output planes 2 * kR steps later.  Both run every step in full.
template <int PH, int ST, int S, int PD, bool NT, int VS, bool P19, bool RED, bool FRC,
          int TB = 0, typename T, typename TW, int TX, int TY, int NH>
__device__ __forceinline__ void sweep_step(int t, int nplanes, int zb, SweepRegs<T, TW, NH>& R,
                                           const SweepCtx<T, TX, TY>& X, T* lds, const Geom& g,
                                           const Fields4<T>& in, const Fields4<T>& out,
                                           const Fields4<TW>& w, const T* dv, const Coef<T>& cf,
                                           const RKCoef<TW>& rk, const T* ftab, T* ipl,
                                           T* tb_u = nullptr, TW* tb_w = nullptr) {
    using Sh = SweepShape<T, TX, TY>;
    constexpr int W = Sh::W, NF = P19 ? 5 : 4;
    constexpr bool IPL = TB == 0 && kInPlaneLds<T, TX, TY, NF>;
    static_assert(TB == 0 || (!P19 && !RED && !FRC && ST == 6), "fusion: plain sweep only");
    if (t >= nplanes) return;
    const int p = zb - kR + t;  // plane loaded in this step
    const int o = p - kR;       // output plane finished in this step
    const bool outstep = TB == 0 || t >= (TB == 2 ? 4 : 2) * kR;

    const PlaneBuf<T, Sh::FS> buf{lds + (PH & 1) * NF * Sh::FS};
    const int ci = (threadIdx.x / TX + kR) * W + (threadIdx.x % TX + kR);
    // register sets: plane p sits in set RS (PD sets, PD divides the unroll
    // of 8); the previous input of output o in set WS
    static_assert(PD == 1 || PD == 2 || PD == 4, "prefetch depth");
    constexpr int RS = PH % PD;
    constexpr int WS = PD >= 2 ? (PH & 1) : 0;
    if constexpr (TB != 2) {  // (stage 2: plane p was written to LDS by stage 1)
        // previous input of an output point, issued early: PD = 1 loads the one
        // finished in this step, PD >= 2 the one finished in the next step
        if constexpr (S >= 2) {
            if constexpr (PD >= 2 && ST >= 5)
                load_prev<(PH + 1) & 1, NT, VS>(R, X, out, w, g, o + 1, t + 1 < nplanes);
            else if constexpr (PD < 2 && ST == 6)
                load_prev<0, NT, VS>(R, X, out, w, g, o, outstep);
        }
        // prefetched plane p -> LDS buffer (PH & 1), and the top of the z queues
        buf.put(ci, R.pf[RS]);
#pragma unroll
        for (int h = 0; h < NH; ++h) buf.put(X.loff_h[h], R.ph[RS][h]);
        if constexpr (P19) {
            buf.d()[ci] = R.pfd[RS];
#pragma unroll
            for (int h = 0; h < NH; ++h) buf.d()[X.loff_h[h]] = R.phd[RS][h];
            R.qd[sl8(PH)] = R.pfd[RS];
        }
        // plane p + PD -> the register set just emptied
        sweep_prefetch<RS, VS, P19>(R, X, in, g.felems, dv, plane_corner(g, p + PD),
                                    t + PD < nplanes ? X.plane_bytes : 0u);
        __syncthreads();
    }
    using T2 = typename PlaneBuf<T, Sh::FS>::T2;
    const T2* const U = buf.u() + ci;
    const T2* const V = buf.v() + ci;
    {
        R.q[0][sl8(PH)] = U[0].x;
        R.q[1][sl8(PH)] = U[0].y;
        R.q[2][sl8(PH)] = V[0].x;
        R.q[3][sl8(PH)] = V[0].y;
    }
    constexpr int P = sl8(PH);
    constexpr int DS = PH & 3;  // in-plane slot of plane p
    T ip[kInPlane];             // in-plane values of plane p
    // in-plane values in LDS: this thread's pairs of slot t mod 3
    [[maybe_unused]] T2* const ip2 =
        reinterpret_cast<T2*>(ipl) + R.slot * (kInPlane / 2 * Sh::NT) + threadIdx.x;

    // (C) what plane p contributes: the x / y first derivatives of the four
    // fields, the in-plane part of the right-hand side of output p, and the xz /
    // yz terms of outputs p -+ k.  The bidiagonal xz / yz stencil at output z is
    // sum_k c_k [A_k(z + k) - A_k(z - k)], with A_k the x or y difference at
    // distance k, so plane p adds +c_k A_k to the pending output p - k and
    // -c_k A_k to p + k; the first contribution to output p + 3 assigns.  (The
    // 19-point form has no mixed terms.)
    auto scatter = [&](auto k, int i, const T* m, T a, bool first) {
        constexpr int K = decltype(k)::value;
        constexpr int N = sl8(PH + K), Q = sl8(PH - K);
        if constexpr (ST + K >= 3) {
            if (K == 3 && first)
                R.L[i][N] = -m[K - 1] * a;
            else
                R.L[i][N] = -m[K - 1] * a + R.L[i][N];
        }
        if constexpr (ST - K >= 3) R.L[i][Q] = m[K - 1] * a + R.L[i][Q];
    };
    if constexpr (ST >= 3) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
            R.L[i][P] = P19 ? cf.kc19 * R.q[i][P] : cf.kc[i] * R.q[i][P] + R.L[i][P];
        const T u0 = R.q[0][P], u1 = R.q[1][P];
        T g0, g1, J20, J21;
        {  // lnrho and uz
            Weighted<T> zx, zy;
            auto tap = [&](auto k) {
                constexpr int K = decltype(k)::value;
                const T2 xp = V[K], xm = V[-K], yp = V[K * W], ym = V[-K * W];
                const T ax = xp.x - xm.x, ay = yp.x - ym.x;
                const T bx = xp.y - xm.y, by = yp.y - ym.y;
                g0 = K == 1 ? cf.d1[0][0] * bx : cf.d1[0][K - 1] * bx + g0;
                g1 = K == 1 ? cf.d1[1][0] * by : cf.d1[1][K - 1] * by + g1;
                J20 = K == 1 ? cf.d1[0][0] * ax : cf.d1[0][K - 1] * ax + J20;
                J21 = K == 1 ? cf.d1[1][0] * ay : cf.d1[1][K - 1] * ay + J21;
                zx.template add<K>(cf.s[0], xp.x + xm.x, R.L[2][P]);
                zy.template add<K>(cf.s[1], yp.x + ym.x, R.L[2][P]);
                if constexpr (!P19) {
                    scatter(k, 0, cf.m[1], ax, true);  // (1/3) Dxz uz
                    scatter(k, 1, cf.m[2], ay, true);  // (1/3) Dyz uz
                }
            };
            tap(std::integral_constant<int, 1>{});
            tap(std::integral_constant<int, 2>{});
            tap(std::integral_constant<int, 3>{});
            zx.end(cf.s[0], R.L[2][P]);
            zy.end(cf.s[1], R.L[2][P]);
        }
        const T h0 = cf.nu * g0, h1 = cf.nu * g1;
        const T v0 = cf.nu * g0 - u0, v1 = cf.nu * g1 - u1;
        R.L[2][P] = J20 * v0 + R.L[2][P];
        R.L[2][P] = J21 * v1 + R.L[2][P];
        T J00, J01, J10, J11;
        {  // ux and uy
            Weighted<T> x0, y0, x1, y1, m0, m1;
            constexpr bool F = !P19;
            const T* sx0 = F ? cf.s4[0] : cf.s[0];
            const T* sy1 = F ? cf.s4[1] : cf.s[1];
            auto tap = [&](auto k) {
                constexpr int K = decltype(k)::value;
                const T2 xp = U[K], xm = U[-K], yp = U[K * W], ym = U[-K * W];
                const T ax = xp.x - xm.x, ay = yp.x - ym.x;
                const T bx = xp.y - xm.y, by = yp.y - ym.y;
                J00 = K == 1 ? cf.d1[0][0] * ax : cf.d1[0][K - 1] * ax + J00;
                J01 = K == 1 ? cf.d1[1][0] * ay : cf.d1[1][K - 1] * ay + J01;
                J10 = K == 1 ? cf.d1[0][0] * bx : cf.d1[0][K - 1] * bx + J10;
                J11 = K == 1 ? cf.d1[1][0] * by : cf.d1[1][K - 1] * by + J11;
                x0.template add<K>(sx0, xp.x + xm.x, R.L[0][P]);
                y0.template add<K>(cf.s[1], yp.x + ym.x, R.L[0][P]);
                x1.template add<K>(cf.s[0], xp.y + xm.y, R.L[1][P]);
                y1.template add<K>(sy1, yp.y + ym.y, R.L[1][P]);
                if constexpr (!P19) {
                    const T2 pp = U[K * W + K], pm = U[K * W - K];
                    const T2 mp = U[-K * W + K], mm = U[-K * W - K];
                    // (1/3) Dxy ux into uy's equation and the other way round
                    m1.template add<K>(cf.m[0], (pp.x - pm.x) + (mm.x - mp.x), R.L[1][P]);
                    m0.template add<K>(cf.m[0], (pp.y - pm.y) + (mm.y - mp.y), R.L[0][P]);
                    scatter(k, 2, cf.m[1], ax, true);   // (1/3) Dxz ux
                    scatter(k, 2, cf.m[2], by, false);  // (1/3) Dyz uy
                }
            };
            tap(std::integral_constant<int, 1>{});
            tap(std::integral_constant<int, 2>{});
            tap(std::integral_constant<int, 3>{});
            x0.end(sx0, R.L[0][P]);
            y0.end(cf.s[1], R.L[0][P]);
            x1.end(cf.s[0], R.L[1][P]);
            y1.end(sy1, R.L[1][P]);
            if constexpr (!P19) {
                m1.end(cf.m[0], R.L[1][P]);
                m0.end(cf.m[0], R.L[0][P]);
            }
        }
        // the in-plane terms of the x and y momentum and of lnrho
        const T D = J00 + J11;
        const T e = -cf.tn * D - cf.cs2;
        T l = R.L[0][P];
        l = J00 * (v0 + h0) + l;
        l = J01 * v1 + l;
        l = J10 * h1 + l;
        l = e * g0 + l;
        R.L[0][P] = l;
        l = R.L[1][P];
        l = J11 * (v1 + h1) + l;
        l = J10 * v0 + l;
        l = J01 * h0 + l;
        l = e * g1 + l;
        R.L[1][P] = l;
        ip[0] = h0, ip[1] = h1, ip[2] = J20, ip[3] = J21, ip[4] = D;
        ip[5] = u0 * g0 + u1 * g1;
        if constexpr (P19) {  // (nu/3) d_x and d_y of div u
            const T* const F = buf.d() + ci;
            const T dx = cf.d1[0][0] * (F[1] - F[-1]) + cf.d1[0][1] * (F[2] - F[-2]) +
                         cf.d1[0][2] * (F[3] - F[-3]);
            const T dy = cf.d1[1][0] * (F[W] - F[-W]) + cf.d1[1][1] * (F[2 * W] - F[-2 * W]) +
                         cf.d1[1][2] * (F[3 * W] - F[-3 * W]);
            R.L[0][P] = cf.n3 * dx + R.L[0][P];
            R.L[1][P] = cf.n3 * dy + R.L[1][P];
        }
    } else if constexpr (!P19) {
        auto tap = [&](auto k) {
                constexpr int K = decltype(k)::value;
            if constexpr (ST + K >= 3) {
                scatter(k, 0, cf.m[1], V[K].x - V[-K].x, true);
                scatter(k, 1, cf.m[2], V[K * W].x - V[-K * W].x, true);
                scatter(k, 2, cf.m[1], U[K].x - U[-K].x, true);
                scatter(k, 2, cf.m[2], U[K * W].y - U[-K * W].y, false);
            }
        };
        tap(std::integral_constant<int, 1>{});
        tap(std::integral_constant<int, 2>{});
        tap(std::integral_constant<int, 3>{});
    }

    // (B) finish output plane o = p - 3: the terms with z derivatives, from the
    // queues (plane p is their top) and the in-plane values of plane o, which
    // plane p's then replace.
    if constexpr (ST == 6) {
        const unsigned ob = outstep ? X.plane_bytes : 0u;
        const unsigned wb = outstep ? X.wplane_bytes : 0u;
        constexpr int Q = sl8(PH - 3);
        T io[kInPlane];  // of plane o
#pragma unroll
        for (int i = 0; i < kInPlane; i += 2) {
            T2 v;
            if constexpr (IPL)
                v = ip2[(i / 2) * Sh::NT];
            else
                v = T2{R.dd[(PH + 1) & 3][i], R.dd[(PH + 1) & 3][i + 1]};
            io[i] = v.x;
            io[i + 1] = v.y;
        }
        T dz[4];
#pragma unroll
        for (int f = 0; f < 4; ++f)
            dz[f] = cf.d1[2][0] * (R.q[f][sl8(PH - 2)] - R.q[f][sl8(PH - 4)]) +
                    cf.d1[2][1] * (R.q[f][sl8(PH - 1)] - R.q[f][sl8(PH - 5)]) +
                    cf.d1[2][2] * (R.q[f][sl8(PH)] - R.q[f][sl8(PH - 6)]);
        T Lf[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const T* sz = (i == 2 && !P19) ? cf.s4[2] : cf.s[2];
            const T* c = R.q[i];
            Weighted<T> z;
            Lf[i] = R.L[i][Q];
            z.template add<1>(sz, c[sl8(PH - 2)] + c[sl8(PH - 4)], Lf[i]);
            z.template add<2>(sz, c[sl8(PH - 1)] + c[sl8(PH - 5)], Lf[i]);
            z.template add<3>(sz, c[sl8(PH)] + c[sl8(PH - 6)], Lf[i]);
            z.end(sz, Lf[i]);
        }
        if constexpr (P19) {  // (nu/3) d_z div u
            const T dd = cf.d1[2][0] * (R.qd[sl8(PH - 2)] - R.qd[sl8(PH - 4)]) +
                         cf.d1[2][1] * (R.qd[sl8(PH - 1)] - R.qd[sl8(PH - 5)]) +
                         cf.d1[2][2] * (R.qd[sl8(PH)] - R.qd[sl8(PH - 6)]);
            Lf[2] = cf.n3 * dd + Lf[2];
        }
        // dz: d_z of ux, uy, uz (J22) and lnrho (g2)
        const T u2 = R.q[2][Q], g2 = dz[3], J22 = dz[2];
        const T h2 = cf.nu * g2, v2 = cf.nu * g2 - u2;
        const T x = T(-2.0 / 3.0) * J22;
        const T div = io[4] + J22;
        const T e2 = -cf.tn * div - cf.cs2;
        T r[4];
        r[0] = x * io[0] + Lf[0];
        r[0] = dz[0] * v2 + r[0];
        r[0] = io[2] * h2 + r[0];
        r[1] = x * io[1] + Lf[1];
        r[1] = dz[1] * v2 + r[1];
        r[1] = io[3] * h2 + r[1];
        r[2] = dz[0] * io[0] + Lf[2];
        r[2] = dz[1] * io[1] + r[2];
        r[2] = J22 * (v2 + h2) + r[2];
        r[2] = e2 * g2 + r[2];
        // the small advection terms are summed before the divergence joins them:
        // rounded together with it they bias the mean of lnrho
        r[3] = -(u2 * g2 + io[5]) - div;
        if constexpr (FRC) {
            // f = a cos(k.x + phase) at the output point (eq. forcing).  The
            // table is read-only during the kernel: reading it through the
            // constant address space makes these scalar loads, which keep out
            // of the vector-memory counter the sweep's pipeline depends on
            const __attribute__((address_space(4))) T* ct =
                (const __attribute__((address_space(4))) T*)ftab;
            const T cz = ct[2 * o], sz = ct[2 * o + 1];
            const T ph = R.fc * cz - R.fs * sz;
#pragma unroll
            for (int i = 0; i < 3; ++i) r[i] += R.fa[i] * ph;
        }
        // ghost corner (-3, -3) of output plane o
        const long long ocorner = g.origin + (long long)o * g.plane - kR * g.px - kR;
        constexpr int CP = NT ? kNonTemporal : 0;
        // w receives the right-hand side (S = 0), the RK3 register where that is
        // kept in memory or, in stage 2 of the fusion, the substep-1 state
        constexpr bool REG = kRegInMemory<T, TW>;
        constexpr bool WOUT = S == 0 || TB == 2 || (REG && S != 3);
        T vout[4];
        TW wout[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const T uc = R.q[f][sl8(PH - 3)];
            T v = T(0);
            if constexpr (S == 0) {
                wout[f] = TW(r[f]);
            } else if constexpr (REG) {
                wout[f] = S >= 2 ? R.wq[WS][f] : TW(0);
                v = rk_update_reg<S>(uc, r[f], wout[f], rk);
            } else {
                // stage 2 of the fusion: the input stage 1 kept 3 steps earlier
                T prev = T(0);
                if constexpr (TB == 2)
                    prev = tb_w[((PH + 1) & 3) * 4 * (TX * TY) + f * (TX * TY) + threadIdx.x];
                else if constexpr (S >= 2)
                    prev = R.wq[WS][f];
                v = rk_update<S>(uc, r[f], prev, rk);
                wout[f] = uc;
            }
            vout[f] = v;
            if constexpr (TB == 1) {
                // the input of the inner columns into ring slot (step & 3)
                constexpr int NI = (TX - 2 * kR) * (TY - 2 * kR);
                const int ix = (int)(threadIdx.x % TX) - kR, iy = (int)(threadIdx.x / TX) - kR;
                if (ix >= 0 && ix < TX - 2 * kR && iy >= 0 && iy < TY - 2 * kR)
                    tb_w[(PH & 3) * 4 * NI + f * NI + iy * (TX - 2 * kR) + ix] = uc;
            } else if constexpr (VS == 1) {
                if constexpr (S >= 1)
                    bstore<CP>(v, plane_rsrc(out.f[0] + (ocorner + ((f + 1) & 3) * g.felems), ob),
                               X.lane_o);
                if constexpr (WOUT)
                    bstore<CP>(wout[f],
                               plane_rsrc(w.f[0] + ((long long)o * g.wplane +
                                                    ((f + 1) & 3) * g.wfelems), wb),
                               X.lane_w);
            }
        }
        if constexpr (TB == 1) {
            // new state of every extended column into the inner sweep's plane
            // buffer (its cell is this thread's index)
            constexpr int FS2 = SweepShape<T, TX - 2 * kR, TY - 2 * kR>::FS;
            PlaneBuf<T, FS2>{tb_u + (PH & 1) * 4 * FS2}.put(threadIdx.x, vout);
        }
        if constexpr (VS == 4 && TB != 1) {
            if constexpr (S >= 1)
                bstore_point<CP>(vout, plane_rsrc(out.f[1] + 4 * ocorner, ob), X.lane_o);
            if constexpr (WOUT && kWPairs<TW, VS>) {
                TW* const p = w.f[1] + 2 * (long long)o * g.wplane;
                bstore_pairs<CP>(wout, plane_rsrc(p, wb), plane_rsrc(p + 2 * g.wfelems, wb),
                                 X.lane_w);
            } else if constexpr (WOUT) {
                bstore_point<CP>(wout, plane_rsrc(w.f[1] + 4 * (long long)o * g.wplane, wb),
                                 X.lane_w);
            }
        }
        // FP64 diagnostics of the new state, from the values just stored (the
        // same per-point quantities as the standalone reduction); without a
        // branch: sweep_tile drops the sums of columns outside the box
        if constexpr (RED) {
            if constexpr (kRedElems<T, TX, TY, NF> > 0) {
                double2* const a =
                    reinterpret_cast<double2*>(ipl + kInPlaneElems<T, TX, TY, NF>) + threadIdx.x;
                const double2 p0 = a[0], p1 = a[Sh::NT];
                double s[4] = {p0.x, p0.y, p1.x, p1.y};
                red_point(s, R.bad, vout[3], vout[0], vout[1], vout[2]);
                a[0] = make_double2(s[0], s[1]);
                a[Sh::NT] = make_double2(s[2], s[3]);
            } else {
                red_point(R.red, R.bad, vout[3], vout[0], vout[1], vout[2]);
            }
        }
    }
    // Pin what this step formed: left alone, the compiler moves the arithmetic of
    // a value to the step that uses it, and keeps its many operands alive instead
    // (19-point FP64: 122 registers spilled).
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        if constexpr (ST >= 3) keep_here(R.L[i][P]);
        if constexpr (!P19) {
            if constexpr (ST + 1 >= 3) keep_here(R.L[i][sl8(PH + 1)]);
            if constexpr (ST + 2 >= 3) keep_here(R.L[i][sl8(PH + 2)]);
            keep_here(R.L[i][sl8(PH + 3)]);
            if constexpr (ST >= 4) keep_here(R.L[i][sl8(PH - 1)]);
            if constexpr (ST >= 5) keep_here(R.L[i][sl8(PH - 2)]);
        }
    }
    // the in-plane values of plane p
    if constexpr (ST >= 3) {
#pragma unroll
        for (int i = 0; i < kInPlane; i += 2) {
            if constexpr (IPL) {
                ip2[(i / 2) * Sh::NT] = T2{ip[i], ip[i + 1]};
            } else {
                keep_here(ip[i]);
                keep_here(ip[i + 1]);
                R.dd[DS][i] = ip[i];
                R.dd[DS][i + 1] = ip[i + 1];
            }
        }
    }
    if constexpr (IPL) R.slot = R.slot == 2 ? 0 : R.slot + 1;
}

// One tile-chunk: columns [x0, x0 + TX) x [y0, y0 + TY) of the box, output
// planes [zb, ze).  Every thread of the workgroup calls it with the same
// arguments.  P19: the 19-point method (dv holds the divergence of in).
// RED: also reduce the FP64 diagnostics of the output and store this
// workgroup's partial at part[blockIdx.x * kReduceSlots ...].
template <typename T, typename TW, int TX, int TY, int S, int PD, bool NT, int VS,
          bool P19 = false, bool RED = false, bool FRC = false>
__device__ __forceinline__ void sweep_tile(const Geom& g, const Fields4<T>& in,
                                           const Fields4<T>& out, const Fields4<TW>& w,
                                           const T* dv, const Coef<T>& cf,
                                           const RKCoef<TW>& rk, int x0, int y0, int zb, int ze,
                                           T* lds, double* part, ForceArgs<T> fa, T* ipl) {
    using Sh = SweepShape<T, TX, TY>;
    constexpr int NH = Sh::NH;
    SweepCtx<T, TX, TY> X;
    static_assert(VS == 1 || !P19, "the 19-point sweep uses one array per field");
    sweep_ctx_init<T, TW, TX, TY, VS>(X, g, x0, y0);

    SweepRegs<T, TW, NH> R;
#pragma unroll
    for (int i = 0; i < 4; ++i) R.red[i] = 0.0;
    R.bad = 0;
    R.slot = 0;
    if constexpr (FRC) {
        const ForceDev<T>* fd = fa.dev;
        const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
        const double ang = fd->kx * ((x0 + tx) * fd->dx) + fd->ky * ((y0 + ty) * fd->dy);
        double sn, cs;
        sincos(ang, &sn, &cs);
        R.fc = T(cs);
        R.fs = T(sn);
#pragma unroll
        for (int i = 0; i < 3; ++i) R.fa[i] = fd->a[i];
    }

    constexpr int NF = P19 ? 5 : 4;
    constexpr bool RL = RED && kRedElems<T, TX, TY, NF> > 0;
    T* const redl = ipl + kInPlaneElems<T, TX, TY, NF>;
    if constexpr (RL) {
#pragma unroll
        for (int s = 0; s < 4; ++s) redl[s * Sh::NT + threadIdx.x] = T(0);
    }
    const int nplanes = (ze - zb) + 2 * kR;  // at least 7
    sweep_prefetch<0, VS, P19>(R, X, in, g.felems, dv, plane_corner(g, zb - kR), X.plane_bytes);
    if constexpr (PD >= 2)
        sweep_prefetch<1, VS, P19>(R, X, in, g.felems, dv, plane_corner(g, zb - kR + 1),
                                   X.plane_bytes);
    if constexpr (PD == 4) {
        sweep_prefetch<2, VS, P19>(R, X, in, g.felems, dv, plane_corner(g, zb - kR + 2),
                                   X.plane_bytes);
        sweep_prefetch<3, VS, P19>(R, X, in, g.felems, dv, plane_corner(g, zb - kR + 3),
                                   X.plane_bytes);
    }
    auto step = [&](auto ph, auto st, int t) {
        sweep_step<decltype(ph)::value, decltype(st)::value, S, PD, NT, VS, P19, RED, FRC>(
            t, nplanes, zb, R, X, lds, g, in, out, w, dv, cf, rk, fa.tab, ipl);
    };
    using I0 = std::integral_constant<int, 0>;
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    using I3 = std::integral_constant<int, 3>;
    using I4 = std::integral_constant<int, 4>;
    using I5 = std::integral_constant<int, 5>;
    using I6 = std::integral_constant<int, 6>;
    using I7 = std::integral_constant<int, 7>;
    step(I0{}, I0{}, 0);
    step(I1{}, I1{}, 1);
    step(I2{}, I2{}, 2);
    step(I3{}, I3{}, 3);
    step(I4{}, I4{}, 4);
    step(I5{}, I5{}, 5);
    for (int t = 2 * kR; t < nplanes; t += 8) {
        step(I6{}, I6{}, t);
        step(I7{}, I6{}, t + 1);
        step(I0{}, I6{}, t + 2);
        step(I1{}, I6{}, t + 3);
        step(I2{}, I6{}, t + 4);
        step(I3{}, I6{}, t + 5);
        step(I4{}, I6{}, t + 6);
        step(I5{}, I6{}, t + 7);
    }
    if constexpr (RED) {
        if constexpr (RL) {
            const double* a = reinterpret_cast<const double*>(redl) + 2 * threadIdx.x;
            R.red[0] = a[0], R.red[1] = a[1];
            R.red[2] = a[2 * Sh::NT], R.red[3] = a[2 * Sh::NT + 1];
        }
        if (X.lane_o == kDropOffset) {  // not a point of the box
            R.red[0] = R.red[1] = R.red[2] = R.red[3] = 0.0;
            R.bad = 0;
        }
        red_store_n<Sh::NW>(R.red, R.bad, part);
    }
}

template <typename T, typename TW, int TX, int TY, int S, int PD, bool NT, int VS,
          bool FRC>
__global__ __launch_bounds__(TX* TY, kMinWaves)
void substep55_sweep(Geom g, Fields4<T> in, Fields4<T> out, Fields4<TW> w, Coef<T> cf,
                     RKCoef<TW> rk, SweepGrid m, ForceArgs<T> fa) {
    using Sh = SweepShape<T, TX, TY>;
    __shared__ __attribute__((aligned(16))) T lds[2 * 4 * Sh::FS];
    __shared__ __attribute__((aligned(16))) T ipl[kInPlaneElems<T, TX, TY, 4>];
    const TileXY t = sweep_tile_of(g, TX, TY, m);
    if (t.zb >= t.ze) return;
    sweep_tile<T, TW, TX, TY, S, PD, NT, VS, false, false, FRC>(
        g, in, out, w, nullptr, cf, rk, t.tx, t.ty, t.zb, t.ze, lds, nullptr, fa, ipl);
}

// Substeps 1 and 2 of one step in one launch: the temporal blocking the
// paper's discussion of Sec. 7 proposes, in the z-sweep.  A workgroup of
// (TX + 6) x (TY + 6) threads owns a TX x TY output tile.
//  * Stage 1: the substep-1 sweep over the extended tile (the output tile
//    and a 3-column ring), one column per thread, loading the input state as
//    the plain sweep does.  Its new state does not go to memory: plane o1
//    goes into an LDS plane buffer laid out as the inner tile's sweep reads
//    its planes, and the input of the inner columns into an LDS ring of 4
//    planes.
//  * Stage 2 (threads 0 .. TX TY - 1, whole waves): the substep-2 sweep of
//    the output tile with that buffer as its plane source, 3 planes behind
//    stage 1, storing the substep-2 state and, into w, the substep-1 state
//    that substep 3 needs.
// Substeps 1 and 2 move 16 + 32 bytes per point (FP32), and 32 more to put
// the substep-1 state where substep 3 reads it, instead of 32 + 48, at the
// price of substep 1 on (TX + 6)(TY + 6) / (TX TY) times the columns.  Per point the
// arithmetic is the plain sweep's, so the result is bit for bit that of two
// plain launches.  The loaded planes start 2 * kR further back (nplanes =
// chunk + 4 kR).
template <typename T, typename TW, int TX, int TY, int PD, bool NT, int VS>
__device__ __forceinline__ void fused12_tile(const Geom& g, const Fields4<T>& in,
                                             const Fields4<T>& out, const Fields4<TW>& w,
                                             const Coef<T>& cf, const RKCoef<TW>& rk1,
                                             const RKCoef<TW>& rk2, int x0, int y0, int zb,
                                             int ze, T* lds1, T* lds2, TW* ring) {
    constexpr int EX = TX + 2 * kR, EY = TY + 2 * kR;
    using Sh1 = SweepShape<T, EX, EY>;
    using Sh2 = SweepShape<T, TX, TY>;
    static_assert(Sh2::W == EX && Sh2::H == EY, "stage-2 planes are the stage-1 tile");
    static_assert((TX * TY) % 64 == 0, "stage 2 runs on whole waves");
    SweepCtx<T, EX, EY> X1;
    sweep_ctx_init<T, TW, EX, EY, VS, true>(X1, g, x0 - kR, y0 - kR);
    SweepCtx<T, TX, TY> X2;
    const bool inner = threadIdx.x < TX * TY;
    if (inner) sweep_ctx_init<T, TW, TX, TY, VS>(X2, g, x0, y0);
    SweepRegs<T, TW, Sh1::NH> R1;
    SweepRegs<T, TW, Sh2::NH> R2;
#pragma unroll
    for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int s = 0; s < 8; ++s) R1.q[f][s] = R2.q[f][s] = T(0);
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < kInPlane; ++i) R1.dd[s][i] = R2.dd[s][i] = T(0);
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int s = 0; s < 8; ++s) R1.L[i][s] = R2.L[i][s] = T(0);
    const int nplanes = (ze - zb) + 4 * kR;
    const int zb1 = zb - kR, zb2 = zb - 2 * kR;  // stage 1 outputs from zb - 3
    const T* const nodiv = nullptr;
    sweep_prefetch<0, VS, false>(R1, X1, in, g.felems, nodiv, plane_corner(g, zb1 - kR), X1.plane_bytes);
    if constexpr (PD >= 2)
        sweep_prefetch<1, VS, false>(R1, X1, in, g.felems, nodiv, plane_corner(g, zb1 - kR + 1),
                                     X1.plane_bytes);
    static_assert(PD == 1 || PD == 2, "prefetch depth of the fused sweep");
    const Fields4<T> none{{nullptr, nullptr, nullptr, nullptr}};
    for (int t0 = 0; t0 < nplanes; t0 += 8) {
#define FD6_FUSED_STEP(PH)                                                                      \
        sweep_step<PH, 6, 1, PD, NT, VS, false, false, false, 1>(                                \
            t0 + PH, nplanes, zb1, R1, X1, lds1, g, in, none, w, nodiv, cf,            \
            rk1, (const T*)nullptr, (T*)nullptr, lds2, ring);                                                 \
        __syncthreads();                                                                         \
        if (inner)                                                                               \
            sweep_step<PH, 6, 2, PD, NT, VS, false, false, false, 2>(                            \
                t0 + PH, nplanes, zb2, R2, X2, lds2, g, in, out, w, nodiv, cf,         \
                rk2, (const T*)nullptr, (T*)nullptr, (T*)nullptr, ring);
        FD6_FUSED_STEP(0)
        FD6_FUSED_STEP(1)
        FD6_FUSED_STEP(2)
        FD6_FUSED_STEP(3)
        FD6_FUSED_STEP(4)
        FD6_FUSED_STEP(5)
        FD6_FUSED_STEP(6)
        FD6_FUSED_STEP(7)
#undef FD6_FUSED_STEP
    }
}

template <typename T, typename TW, int TX, int TY, int PD, bool NT, int VS>
__global__ __launch_bounds__((TX + 2 * kR) * (TY + 2 * kR))
void substep55_fused12(Geom g, Fields4<T> in, Fields4<T> out, Fields4<TW> w, Coef<T> cf,
                       RKCoef<TW> rk1, RKCoef<TW> rk2, SweepGrid m) {
    using Sh1 = SweepShape<T, TX + 2 * kR, TY + 2 * kR>;
    using Sh2 = SweepShape<T, TX, TY>;
    __shared__ __attribute__((aligned(16))) T lds1[2 * 4 * Sh1::FS];
    __shared__ __attribute__((aligned(16))) T lds2[2 * 4 * Sh2::FS];
    __shared__ TW ring[4 * 4 * TX * TY];
    const TileXY t = sweep_tile_of(g, TX, TY, m);
    if (t.zb >= t.ze) return;
    fused12_tile<T, TW, TX, TY, PD, NT, VS>(g, in, out, w, cf, rk1, rk2, t.tx, t.ty, t.zb, t.ze,
                                            lds1, lds2, ring);
}

// Substep 3 with the FP64 diagnostics of the new state fused in: one partial
// per workgroup (every workgroup of the grid has a non-empty chunk).
template <typename T, typename TW, int TX, int TY, int PD, bool NT, int VS, bool FRC>
__global__ __launch_bounds__(TX* TY, kMinWaves)
void substep55_sweep_red(Geom g, Fields4<T> in, Fields4<T> out, Fields4<TW> w, Coef<T> cf,
                         RKCoef<TW> rk, SweepGrid m, double* part,
                         ForceArgs<T> fa) {
    using Sh = SweepShape<T, TX, TY>;
    __shared__ __attribute__((aligned(16))) T lds[2 * 4 * Sh::FS];
    __shared__ __attribute__((aligned(16))) T ipl[kInPlaneElems<T, TX, TY, 4> +
                                                  kRedElems<T, TX, TY, 4>];
    const TileXY t = sweep_tile_of(g, TX, TY, m);
    sweep_tile<T, TW, TX, TY, 3, PD, NT, VS, false, true, FRC>(
        g, in, out, w, nullptr, cf, rk, t.tx, t.ty, t.zb, t.ze, lds, part, fa, ipl);
}

// The 19-point method (Sec. 4.2, Algorithm 3): the same sweep over the state
// and the divergence field of its input (substep19_div), with nu lap u and
// (nu/3) grad d in place of the viscous operator.  Algorithm 3 adds the second
// term to the stored velocity and register in a pass of its own: 304 bytes per
// point and step in FP32.  With the divergence computed first, every value is
// written once: 188 bytes (256^3 FP32 with a new force every step, 10 steps and
// a snapshot: 10.96 -> 8.18 ms; 300 x 240 x 192 FP64, 5 steps: 11.46 -> 9.57 ms).
template <typename T, typename TW, int TX, int TY, int S, int PD, bool NT, bool FRC,
          bool RED = false>
__global__ __launch_bounds__(TX* TY, kMinWaves)
void substep19_sweep(Geom g, Fields4<T> in, Fields4<T> out, Fields4<TW> w, const T* dv,
                     Coef<T> cf, RKCoef<TW> rk, SweepGrid m, double* part, ForceArgs<T> fa) {
    using Sh = SweepShape<T, TX, TY>;
    static_assert(!RED || S == 3, "diagnostics of the final substep only");
    __shared__ __attribute__((aligned(16))) T lds[2 * 5 * Sh::FS];
    __shared__ __attribute__((aligned(16))) T ipl[kInPlaneElems<T, TX, TY, 5> +
                                                  (RED ? kRedElems<T, TX, TY, 5> : 0)];
    const TileXY t = sweep_tile_of(g, TX, TY, m);
    if (!RED && t.zb >= t.ze) return;
    sweep_tile<T, TW, TX, TY, S, PD, NT, 1, true, RED, FRC>(
        g, in, out, w, dv, cf, rk, t.tx, t.ty, t.zb, t.ze, lds, part, fa, ipl);
}

// Batched form: one persistent launch advances every box of an ensemble by
// one substep.  The host gives every workgroup its own list of tile-chunks
// (items wg_first[L] .. wg_first[L + 1] - 1), where L = remap(blockIdx) numbers
// the workgroups of one XCD contiguously, so that the host can hand one XCD
// neighbouring tiles of the same boxes and they share its L2.  Per-box
// geometry, pointers, coefficients and time step come from device memory, so
// a captured graph never needs re-capture when they change.  Per point the
// arithmetic is the single-box kernel's.
template <typename T, typename TW, int TX, int TY, int S, int PD, bool NT, int VS>
__global__ __launch_bounds__(TX* TY, kMinWaves)
void substep55_batch(const BatchBox<T, TW>* __restrict__ boxes,
                     const BatchItem* __restrict__ items, const int* __restrict__ wg_first,
                     int parity) {
    using Sh = SweepShape<T, TX, TY>;
    __shared__ __attribute__((aligned(16))) T lds[2 * 4 * Sh::FS];
    __shared__ __attribute__((aligned(16))) T ipl[kInPlaneElems<T, TX, TY, 4>];
    const int G = gridDim.x;
    int b = blockIdx.x;
    if ((G & 7) == 0) b = (b & 7) * (G >> 3) + (b >> 3);
    const int last = wg_first[b + 1];
    for (int it = wg_first[b]; it < last; ++it) {
        const BatchItem wi = items[it];
        const BatchBox<T, TW>* bx = boxes + wi.box;
        const Geom g = bx->g;
        const Coef<T> cf = bx->cf;
        const Fields4<T> in = bx->st[parity], out = bx->st[parity ^ 1];
        const Fields4<TW> w = bx->w;
        const RKCoef<TW> rk = bx->rk[S - 1];
        sweep_tile<T, TW, TX, TY, S, PD, NT, VS>(g, in, out, w, nullptr, cf, rk, wi.x0, wi.y0,
                                                   wi.zb, wi.ze, lds, nullptr,
                                                   ForceArgs<T>{nullptr, nullptr}, ipl);
        __syncthreads();  // the next item's first LDS write must follow every read
    }
}

// Launch helpers: the substep index S is a template argument of every kernel.
template <template <int> class K, typename... A>
hipError_t launch_s(int s, dim3 grid, dim3 block, hipStream_t st, A... args) {
    switch (s) {
    case 0: return hipErrorInvalidValue;
    case 1: hipLaunchKernelGGL(K<1>::fn, grid, block, 0, st, args...); break;
    case 2: hipLaunchKernelGGL(K<2>::fn, grid, block, 0, st, args...); break;
    default: hipLaunchKernelGGL(K<3>::fn, grid, block, 0, st, args...); break;
    }
    return hipGetLastError();
}

template <typename T, typename TW, int TX, int TY, int PD, bool NT, int VS, bool FRC>
struct K55 {
    template <int S>
    struct at {
        static constexpr auto fn = substep55_sweep<T, TW, TX, TY, S, PD, NT, VS, FRC>;
    };
};
template <typename T, typename TW, int TX, int TY, int PD, bool NT, int VS, bool FRC>
struct KRed {
    static constexpr auto fn = substep55_sweep_red<T, TW, TX, TY, PD, NT, VS, FRC>;
};
template <typename T, typename TW, int TX, int TY, int PD, bool NT, bool FRC>
struct K19 {
    template <int S>
    struct at {
        static constexpr auto fn = substep19_sweep<T, TW, TX, TY, S, PD, NT, FRC>;
    };
};
template <typename T, typename TW, int TX, int TY, int PD, bool NT, bool FRC>
struct K19Red {
    static constexpr auto fn = substep19_sweep<T, TW, TX, TY, 3, PD, NT, FRC, true>;
};
template <typename T, typename TW, int TX, int TY, int PD, bool NT, int VS>
struct KBatch {
    template <int S>
    struct at {
        static constexpr auto fn = substep55_batch<T, TW, TX, TY, S, PD, NT, VS>;
    };
};
// Shape that evaluates the bare right-hand side (S = 0).
template <typename T>
constexpr int kRhsTile = sizeof(T) == 8 ? 8 : 6;
template <typename T, typename TW, bool FRC>
struct KDirect {
    template <int S>
    struct at {
        static constexpr auto fn = substep55_direct<T, TW, S, FRC>;
    };
};

// VS = 1: one array per field; VS = 4: array of structures (register-loader
// z-sweep shapes only).
template <typename T, typename TW, int VS>
hipError_t launch_substep55_vs(const Geom& g, Fields4<T> in, Fields4<T> out, Fields4<TW> w,
                               const Coef<T>& c, const RKCoef<TW>& rk, int s, int tile,
                               int zchunk, double* partials, int part_cap, int* nparts,
                               const ForceArgs<T>* frc, hipStream_t st) {
    if (nparts) *nparts = 0;
    if (g.vs != VS) return hipErrorInvalidValue;
    const ForceArgs<T> fa = frc ? *frc : ForceArgs<T>{nullptr, nullptr};
    if (s == 0) {  // every z-sweep shape gives the same bits: one serves them all
        if (tile == 0) return hipErrorInvalidValue;
        auto rhs = [&](auto force) -> hipError_t {
            constexpr TileCfg k = kTiles[kRhsTile<T>];
            constexpr auto fn = substep55_sweep<T, TW, k.tx, k.ty, 0, kPd<T, k.pd>, k.nt, VS,
                                                decltype(force)::value>;
            const SweepGrid sg =
                sweep_grid(g, k.tx, k.ty, 0, resident_blocks<fn>(k.tx * k.ty));
            hipLaunchKernelGGL(fn, dim3(sg.blocks), dim3(k.tx * k.ty), 0, st, g, in, out, w, c,
                               rk, sg, fa);
            return hipGetLastError();
        };
        return frc ? rhs(std::true_type{}) : rhs(std::false_type{});
    }
    if (tile == kAutoTile) {
        const AutoShape a =
            auto_shape<T, TW, VS, false>(g, zchunk, s, s == 3 && partials, frc != nullptr);
        tile = a.tile;
        zchunk = a.zchunk;
    }
    auto go = [&](auto force) -> hipError_t {
        constexpr bool FRC = decltype(force)::value;
        return with_tile(tile, hipErrorInvalidValue, [&](auto I) -> hipError_t {
            constexpr TileCfg k = kTiles[decltype(I)::value];
            if constexpr (VS != 1 && (k.tx == 0 || k.soa)) {
                return hipErrorInvalidValue;
            } else if constexpr (k.tx == 0) {
                const dim3 grid((unsigned)((g.nx + 63) / 64), (unsigned)((g.ny + 3) / 4),
                                (unsigned)g.nz);
                return launch_s<KDirect<T, TW, FRC>::template at>(s, grid, dim3(256), st, g, in,
                                                                  out, w, c, rk, fa);
            } else {
                using K = K55<T, TW, k.tx, k.ty, kPd<T, k.pd>, k.nt, VS, FRC>;
                using KR = KRed<T, TW, k.tx, k.ty, kPd<T, k.pd>, k.nt, VS, FRC>;
                const int res = resident_blocks<K::template at<2>::fn>(k.tx * k.ty);
                const SweepGrid sg = sweep_grid(g, k.tx, k.ty, zchunk, res,
                                                s == 3 && partials ? part_cap : 0);
                // fuse only where the extra accumulators cost no occupancy
                static const bool fuse_ok = [] {
                    int a = 0, b = 0;
                    const int blk = k.tx * k.ty;
                    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&a, KR::fn, blk, 0) !=
                            hipSuccess ||
                        hipOccupancyMaxActiveBlocksPerMultiprocessor(
                            &b, K::template at<3>::fn, blk, 0) != hipSuccess)
                        return false;
                    return a >= b && a > 0;
                }();
                if (s == 3 && partials && nparts && fuse_ok && sg.blocks <= part_cap) {
                    hipLaunchKernelGGL(KR::fn, dim3(sg.blocks), dim3(k.tx * k.ty), 0, st, g, in,
                                       out, w, c, rk, sg, partials, fa);
                    *nparts = sg.blocks;
                    return hipGetLastError();
                }
                return launch_s<K::template at>(s, dim3(sg.blocks), dim3(k.tx * k.ty), st, g, in,
                                                out, w, c, rk, sg, fa);
            }
        });
    };
    return frc ? go(std::true_type{}) : go(std::false_type{});
}

}  // namespace

template <typename T, typename TW>
hipError_t launch_substep55(const Geom& g, Fields4<T> in, Fields4<T> out, Fields4<TW> w,
                            const Coef<T>& c, const RKCoef<TW>& rk, int s, int tile, int zchunk,
                            double* partials, int part_cap, int* nparts,
                            const ForceArgs<T>* frc, hipStream_t st) {
    return launch_substep55_vs<T, TW, 1>(g, in, out, w, c, rk, s, tile, zchunk, partials,
                                         part_cap, nparts, frc, st);
}

template <typename T, typename TW>
hipError_t launch_substep55_aos(const Geom& g, Fields4<T> in, Fields4<T> out, Fields4<TW> w,
                                const Coef<T>& c, const RKCoef<TW>& rk, int s, int tile,
                                int zchunk, double* partials, int part_cap, int* nparts,
                                const ForceArgs<T>* frc, hipStream_t st) {
    return launch_substep55_vs<T, TW, 4>(g, in, out, w, c, rk, s, tile, zchunk, partials,
                                         part_cap, nparts, frc, st);
}

// The 19-point method in a z-sweep shape (tile >= 1), after launch_div19.
template <typename T, typename TW>
hipError_t launch_substep19(const Geom& g, Fields4<T> in, Fields4<T> out, Fields4<TW> w,
                            const T* dv, const Coef<T>& c, const RKCoef<TW>& rk, int s, int tile,
                            int zchunk, double* partials, int part_cap, int* nparts,
                            const ForceArgs<T>* frc, hipStream_t st) {
    if (nparts) *nparts = 0;
    const ForceArgs<T> fa = frc ? *frc : ForceArgs<T>{nullptr, nullptr};
    double* const none = nullptr;
    if (s == 0) {
        auto rhs = [&](auto force) -> hipError_t {
            constexpr TileCfg k = kTiles[kRhsTile<T>];
            constexpr auto fn = substep19_sweep<T, TW, k.tx, k.ty, 0, kPd<T, k.pd>, k.nt,
                                                decltype(force)::value>;
            const SweepGrid sg =
                sweep_grid(g, k.tx, k.ty, 0, resident_blocks<fn>(k.tx * k.ty));
            hipLaunchKernelGGL(fn, dim3(sg.blocks), dim3(k.tx * k.ty), 0, st, g, in, out, w, dv,
                               c, rk, sg, none, fa);
            return hipGetLastError();
        };
        return frc ? rhs(std::true_type{}) : rhs(std::false_type{});
    }
    if (tile == kAutoTile) {
        const AutoShape a =
            auto_shape<T, TW, 1, true>(g, zchunk, s, s == 3 && partials, frc != nullptr);
        tile = a.tile;
        zchunk = a.zchunk;
    }
    auto go = [&](auto force) -> hipError_t {
        constexpr bool FRC = decltype(force)::value;
        return with_tile(tile, hipErrorInvalidValue, [&](auto I) -> hipError_t {
            constexpr TileCfg k = kTiles[decltype(I)::value];
            if constexpr (k.tx == 0) {
                return hipErrorInvalidValue;
            } else {
                using K = K19<T, TW, k.tx, k.ty, kPd<T, k.pd>, k.nt, FRC>;
                using KR = K19Red<T, TW, k.tx, k.ty, kPd<T, k.pd>, k.nt, FRC>;
                const int blk = k.tx * k.ty;
                const int res = resident_blocks<K::template at<2>::fn>(blk);
                const SweepGrid sg = sweep_grid(g, k.tx, k.ty, zchunk, res,
                                                s == 3 && partials ? part_cap : 0);
                // fuse only where the extra accumulators cost no occupancy
                if (s == 3 && partials && nparts && sg.blocks <= part_cap &&
                    resident_blocks<KR::fn>(blk) >= resident_blocks<K::template at<3>::fn>(blk)) {
                    hipLaunchKernelGGL(KR::fn, dim3(sg.blocks), dim3(blk), 0, st, g, in, out, w,
                                       dv, c, rk, sg, partials, fa);
                    *nparts = sg.blocks;
                    return hipGetLastError();
                }
                return launch_s<K::template at>(s, dim3(sg.blocks), dim3(blk), st, g, in, out, w,
                                                dv, c, rk, sg, none, fa);
            }
        });
    };
    return frc ? go(std::true_type{}) : go(std::false_type{});
}

namespace {

template <typename T, typename TW, int VS>
hipError_t launch_batch55_vs(const BatchBox<T, TW>* boxes, const BatchItem* items,
                             const int* wg_first, int grid, int parity, int s, int tile,
                             hipStream_t st) {
    return with_tile(tile, hipErrorInvalidValue, [&](auto I) -> hipError_t {
        constexpr TileCfg k = kTiles[decltype(I)::value];
        if constexpr (k.tx == 0 || (VS != 1 && k.soa)) {
            return hipErrorInvalidValue;
        } else {
            return launch_s<KBatch<T, TW, k.tx, k.ty, kPd<T, k.pd>, k.nt, VS>::template at>(
                s, dim3(grid), dim3(k.tx * k.ty), st, boxes, items, wg_first, parity);
        }
    });
}

template <typename T, typename TW, int VS>
int batch55_blocks_per_cu_vs(int tile) {
    return with_tile(tile, 1, [&](auto I) -> int {
        constexpr TileCfg k = kTiles[decltype(I)::value];
        if constexpr (k.tx == 0 || (VS != 1 && k.soa)) {
            return 1;
        } else {
            int n = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(
                    &n, substep55_batch<T, TW, k.tx, k.ty, 2, kPd<T, k.pd>, k.nt, VS>, k.tx * k.ty,
                    0) != hipSuccess)
                return 1;
            return n > 0 ? n : 1;
        }
    });
}

}  // namespace

template <typename T, typename TW>
hipError_t launch_batch55(const BatchBox<T, TW>* boxes, const BatchItem* items,
                          const int* wg_first, int grid, int parity, int s, int tile,
                          hipStream_t st) {
    return launch_batch55_vs<T, TW, 1>(boxes, items, wg_first, grid, parity, s, tile, st);
}

template <typename T, typename TW>
hipError_t launch_batch55_aos(const BatchBox<T, TW>* boxes, const BatchItem* items,
                              const int* wg_first, int grid, int parity, int s, int tile,
                              hipStream_t st) {
    return launch_batch55_vs<T, TW, 4>(boxes, items, wg_first, grid, parity, s, tile, st);
}

template <typename T, typename TW>
int batch55_blocks_per_cu(int tile) {
    return batch55_blocks_per_cu_vs<T, TW, 1>(tile);
}

template <typename T, typename TW>
int batch55_blocks_per_cu_aos(int tile) {
    return batch55_blocks_per_cu_vs<T, TW, 4>(tile);
}

}  // namespace fd6
