// 19-point two-pass substep (Sec. 4.2, Algorithm 3, Appendix A).
//
// The direct kernels (one thread per point, taps through the caches from the
// ghost zones) are Algorithm 3 as printed.  Pass 1 computes the divergence
// field d = D1x ux + D1y uy + D1z uz, the right-hand side without the
// (nu/3) grad(div u) term, and the partial RK3 register and output.  Pass 2
// adds dt (nu/3) D1_i d to w_i and beta dt (nu/3) D1_i d to the output velocity.
// Both passes read only axis-aligned taps (19 points).
//
// The z-sweep shapes compute d first (substep19_div, here) and then the whole
// update in one sweep, which shares the 55-point sweep's code.
#include "sweep_common.hpp"

namespace fd6 {
namespace {

template <typename T>
__device__ __forceinline__ T d1_taps(const T* f, long long c, long long s, const T* w) {
    return w[0] * (f[c + s] - f[c - s]) + w[1] * (f[c + 2 * s] - f[c - 2 * s]) +
           w[2] * (f[c + 3 * s] - f[c - 3 * s]);
}

template <typename T>
__device__ __forceinline__ T d2_taps(const T* f, long long c, long long s, const T* w) {
    return w[0] * f[c] + w[1] * (f[c + s] + f[c - s]) + w[2] * (f[c + 2 * s] + f[c - 2 * s]) +
           w[3] * (f[c + 3 * s] + f[c - 3 * s]);
}

template <typename T, typename TW, int S, bool FRC>
__global__ __launch_bounds__(256) void pass19a_kernel(Geom g, Fields4<T> in, Fields4<T> out,
                                                      Fields4<TW> w, T* __restrict__ dv,
                                                      Coef<T> cf, RKCoef<TW> rk,
                                                      ForceArgs<T> fa) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    const long long c = g.origin + (long long)k * g.plane + (long long)j * g.px + i;
    const long long s[3] = {1, g.px, g.plane};
    T gr[3], J[3][3], u[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) gr[a] = d1_taps(in.f[0], c, s[a], cf.d1[a]);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        u[q] = in.f[1 + q][c];
#pragma unroll
        for (int a = 0; a < 3; ++a) J[q][a] = d1_taps(in.f[1 + q], c, s[a], cf.d1[a]);
    }
    const T div = J[0][0] + J[1][1] + J[2][2];
    dv[c] = div;
    // nu lap u_i with plain (not 4/3-weighted) second-derivative weights
    T L[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        T acc = T(0);
#pragma unroll
        for (int a = 0; a < 3; ++a) acc += d2_taps(in.f[1 + q], c, s[a], cf.lp[a]);
        L[q] = acc;
    }
    T r[4];
    r[0] = -(u[0] * gr[0] + u[1] * gr[1] + u[2] * gr[2]) - div;
    const T third = T(1) / T(3);
    const T dv3 = div * third;
    const T sxy = T(0.5) * (J[0][1] + J[1][0]);
    const T sxz = T(0.5) * (J[0][2] + J[2][0]);
    const T syz = T(0.5) * (J[1][2] + J[2][1]);
    const T sxx = J[0][0] - dv3, syy = J[1][1] - dv3, szz = J[2][2] - dv3;
    const T sg[3] = {sxx * gr[0] + sxy * gr[1] + sxz * gr[2],
                     sxy * gr[0] + syy * gr[1] + syz * gr[2],
                     sxz * gr[0] + syz * gr[1] + szz * gr[2]};
    const T two_nu = cf.nu + cf.nu;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const T adv = u[0] * J[q][0] + u[1] * J[q][1] + u[2] * J[q][2];
        r[1 + q] = (L[q] + two_nu * sg[q]) - cf.cs2 * gr[q] - adv;
    }
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
        TW wn;
        if constexpr (S == 1)
            wn = rk.dt * TW(r[q]);
        else
            wn = rk.alpha * w.f[q][cw] + rk.dt * TW(r[q]);
        // pass 2 completes w_u, so every substep stores it here
        w.f[q][cw] = wn;
        out.f[q][c] = T(TW(in.f[q][c]) + rk.beta * wn);
    }
}

template <typename T, typename TW>
__global__ __launch_bounds__(256) void pass19b_kernel(Geom g, const T* __restrict__ dv,
                                                      Fields4<T> out, Fields4<TW> w, Coef<T> cf,
                                                      RKCoef<TW> rk, TW cgd) {
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
    const int k = blockIdx.z;
    if (i >= g.nx || j >= g.ny) return;
    const long long c = g.origin + (long long)k * g.plane + (long long)j * g.px + i;
    const long long s[3] = {1, g.px, g.plane};
    const long long cw = (long long)k * g.wplane + (long long)j * g.wpx + i;
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const TW t = cgd * TW(d1_taps(dv, c, s[q], cf.d1[q]));
        w.f[1 + q][cw] = w.f[1 + q][cw] + t;
        out.f[1 + q][c] = T(TW(out.f[1 + q][c]) + rk.beta * t);
    }
}

// The divergence of the velocity, d = D1x ux + D1y uy + D1z uz.  A workgroup
// sweeps a z chunk of a kDivTX x kDivTY column tile.  Only ux needs its x
// neighbours and only uy its y neighbours: one LDS plane each (rows of ux with
// 3 cells more at both ends; uy with 3 rows more above and below), both of the
// output plane o, while uz runs 3 planes ahead through a register queue.  A
// thread loads one point of each field and at most one halo cell, one plane
// ahead.  Bound by HBM: 12 bytes read and 4 written per point in FP32.
constexpr int kDivTX = 64, kDivTY = 8;

template <typename T>
struct DivRegs {
    T q[8];        // uz of the thread's column, ring over planes
    T px, py, pz;  // prefetched ux, uy of the next output plane, uz 3 planes beyond
    T ph;          // prefetched halo cell (ux or uy)
};

struct DivAddr {
    unsigned in, halo, out;    // byte offsets from the ghost corner of a plane
    int lx, ly, lh;            // LDS elements of this thread's ux, uy and halo cell
    bool hx;                   // the halo cell belongs to ux
    unsigned bytes;            // of a plane
};

template <typename T>
__device__ __forceinline__ void div_load(DivRegs<T>& R, const DivAddr& A, const Geom& g,
                                         const Fields4<T>& in, int o, bool xy, bool z) {
    const long long oc = plane_corner(g, o);
    const unsigned b = xy ? A.bytes : 0u;
    const __amdgpu_buffer_rsrc_t rx = plane_rsrc(in.f[1] + oc, b);
    const __amdgpu_buffer_rsrc_t ry = plane_rsrc(in.f[2] + oc, b);
    R.px = bload((T*)nullptr, rx, A.in);
    R.py = bload((T*)nullptr, ry, A.in);
    // one of the two loads is out of range for every thread
    const T hx = bload((T*)nullptr, rx, A.hx ? A.halo : kDropOffset);
    const T hy = bload((T*)nullptr, ry, A.hx ? kDropOffset : A.halo);
    R.ph = A.hx ? hx : hy;
    R.pz = bload((T*)nullptr,
                 plane_rsrc(in.f[3] + plane_corner(g, o + kR), z ? A.bytes : 0u), A.in);
}

template <int PH, typename T>
__device__ __forceinline__ void div_step(int t0, int nsteps, int zb, DivRegs<T>& R,
                                         const DivAddr& A, T* lds, const Geom& g,
                                         const Fields4<T>& in, T* dv, const Coef<T>& cf) {
    constexpr int WX = kDivTX + 2 * kR;
    constexpr int NX = kDivTY * WX, NB = NX + (kDivTY + 2 * kR) * kDivTX + 1;
    const int t = t0 + PH;
    if (t >= nsteps) return;
    const int o = zb - 2 * kR + t;  // output plane of this step, from t = 6
    T* buf = lds + (PH & 1) * NB;
    buf[A.lx] = R.px;
    buf[A.ly] = R.py;
    buf[A.lh] = R.ph;
    R.q[sl8(PH)] = R.pz;
    div_load(R, A, g, in, o + 1, t + 1 >= 2 * kR && t + 1 < nsteps, t + 1 < nsteps);
    __syncthreads();
    const T* X = buf + A.lx;
    const T* Y = buf + A.ly;
    const T dx = cf.d1[0][0] * (X[1] - X[-1]) + cf.d1[0][1] * (X[2] - X[-2]) +
                 cf.d1[0][2] * (X[3] - X[-3]);
    const T dy = cf.d1[1][0] * (Y[kDivTX] - Y[-kDivTX]) +
                 cf.d1[1][1] * (Y[2 * kDivTX] - Y[-2 * kDivTX]) +
                 cf.d1[1][2] * (Y[3 * kDivTX] - Y[-3 * kDivTX]);
    const T dz = cf.d1[2][0] * (R.q[sl8(PH - 2)] - R.q[sl8(PH - 4)]) +
                 cf.d1[2][1] * (R.q[sl8(PH - 1)] - R.q[sl8(PH - 5)]) +
                 cf.d1[2][2] * (R.q[sl8(PH)] - R.q[sl8(PH - 6)]);
    const long long oc = g.origin + (long long)o * g.plane - kR * g.px - kR;
    bstore(dx + dy + dz, plane_rsrc(dv + oc, t >= 2 * kR ? A.bytes : 0u), A.out);
}

template <typename T>
__global__ __launch_bounds__(kDivTX* kDivTY) void substep19_div(Geom g, Fields4<T> in, T* dv,
                                                                Coef<T> cf, SweepGrid m) {
    constexpr int TX = kDivTX, TY = kDivTY, WX = TX + 2 * kR;
    constexpr int NX = TY * WX, NB = NX + (TY + 2 * kR) * TX + 1;
    static_assert(2 * kR * (TX + TY) <= TX * TY, "one halo cell per thread");
    __shared__ T lds[2 * NB];
    const TileXY tl = sweep_tile_of(g, TX, TY, m);
    if (tl.zb >= tl.ze) return;
    const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
    DivAddr A;
    A.bytes = (unsigned)(g.plane * (long long)sizeof(T));
    // byte offset of the periodic image of cell (x, y), x < nx + 3, y < ny + 3
    auto image = [&](int x, int y) -> unsigned {
        if (x >= g.nx + kR || y >= g.ny + kR) return kDropOffset;
        const int i = x < 0 ? x + g.nx : (x >= g.nx ? x - g.nx : x);
        const int j = y < 0 ? y + g.ny : (y >= g.ny ? y - g.ny : y);
        return (unsigned)(((j + kR) * g.px + (i + kR)) * (int)sizeof(T));
    };
    A.in = image(tl.tx + tx, tl.ty + ty);
    A.out = tl.tx + tx < g.nx && tl.ty + ty < g.ny ? A.in : kDropOffset;
    A.lx = ty * WX + tx + kR;
    A.ly = NX + (ty + kR) * TX + tx;
    // threads 0 .. 6 TX - 1: the rows of uy above and below the tile; the next
    // 6 TY: the cells of ux left and right of it; the rest fill the spare cell
    const int e = threadIdx.x - 2 * kR * TX;
    A.hx = e >= 0;
    if (e < 0) {
        const int r = threadIdx.x / TX, row = r < kR ? r : r + TY;
        A.halo = image(tl.tx + tx, tl.ty - kR + row);
        A.lh = NX + row * TX + tx;
    } else if (e < 2 * kR * TY) {
        const int r = e / (2 * kR), c = e - r * 2 * kR, col = c < kR ? c : c + TX;
        A.halo = image(tl.tx - kR + col, tl.ty + r);
        A.lh = r * WX + col;
    } else {
        A.halo = kDropOffset;
        A.lh = NB - 1;
    }
    DivRegs<T> R;
#pragma unroll
    for (int s = 0; s < 8; ++s) R.q[s] = T(0);
    const int zb = tl.zb, nsteps = (tl.ze - tl.zb) + 2 * kR;
    div_load(R, A, g, in, zb - 2 * kR, false, true);
    for (int t0 = 0; t0 < nsteps; t0 += 8) {
        div_step<0>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
        div_step<1>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
        div_step<2>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
        div_step<3>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
        div_step<4>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
        div_step<5>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
        div_step<6>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
        div_step<7>(t0, nsteps, zb, R, A, lds, g, in, dv, cf);
    }
}

}  // namespace

template <typename T>
hipError_t launch_div19(const Geom& g, Fields4<T> in, T* div, const Coef<T>& c, hipStream_t st) {
    constexpr int blk = kDivTX * kDivTY;
    const SweepGrid sg =
        sweep_grid(g, kDivTX, kDivTY, 0, resident_blocks<substep19_div<T>>(blk));
    hipLaunchKernelGGL(substep19_div<T>, dim3(sg.blocks), dim3(blk), 0, st, g, in, div, c, sg);
    return hipGetLastError();
}

template <typename T, typename TW>
hipError_t launch_pass19a(const Geom& g, Fields4<T> in, Fields4<T> out, Fields4<TW> w, T* div,
                          const Coef<T>& c, const RKCoef<TW>& rk, int s,
                          const ForceArgs<T>* frc, hipStream_t st) {
    const dim3 grid((unsigned)((g.nx + 63) / 64), (unsigned)((g.ny + 3) / 4), (unsigned)g.nz);
    const ForceArgs<T> fa = frc ? *frc : ForceArgs<T>{nullptr, nullptr};
    auto go = [&](auto force) {
        constexpr bool FRC = decltype(force)::value;
        if (s == 1)
            hipLaunchKernelGGL((pass19a_kernel<T, TW, 1, FRC>), grid, dim3(256), 0, st, g, in, out,
                               w, div, c, rk, fa);
        else
            hipLaunchKernelGGL((pass19a_kernel<T, TW, 2, FRC>), grid, dim3(256), 0, st, g, in, out,
                               w, div, c, rk, fa);
    };
    if (frc)
        go(std::true_type{});
    else
        go(std::false_type{});
    return hipGetLastError();
}

template <typename T, typename TW>
hipError_t launch_pass19b(const Geom& g, const T* div, Fields4<T> out, Fields4<TW> w,
                          const Coef<T>& c, const RKCoef<TW>& rk, hipStream_t st) {
    const dim3 grid((unsigned)((g.nx + 63) / 64), (unsigned)((g.ny + 3) / 4), (unsigned)g.nz);
    hipLaunchKernelGGL((pass19b_kernel<T, TW>), grid, dim3(256), 0, st, g, div, out, w, c, rk,
                       TW((double)rk.dt * c.nu3));
    return hipGetLastError();
}

#define FD6_INST19(T, TW)                                                                       \
    template hipError_t launch_pass19a<T, TW>(const Geom&, Fields4<T>, Fields4<T>, Fields4<TW>, \
                                              T*, const Coef<T>&, const RKCoef<TW>&, int,      \
                                              const ForceArgs<T>*, hipStream_t);               \
    template hipError_t launch_pass19b<T, TW>(const Geom&, const T*, Fields4<T>, Fields4<TW>,   \
                                              const Coef<T>&, const RKCoef<TW>&, hipStream_t);
FD6_INST19(double, double)
FD6_INST19(float, float)
FD6_INST19(float, double)
template hipError_t launch_div19<double>(const Geom&, Fields4<double>, double*,
                                         const Coef<double>&, hipStream_t);
template hipError_t launch_div19<float>(const Geom&, Fields4<float>, float*, const Coef<float>&,
                                        hipStream_t);

}  // namespace fd6
