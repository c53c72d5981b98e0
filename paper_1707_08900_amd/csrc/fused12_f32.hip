// Substeps 1 and 2 fused in one launch (temporal blocking, discussion of
// Sec. 7), FP32 state and register, either state layout: the launcher of
// substep55_fused12 (16 x 16 output tiles, 22 x 22 threads).
#include "sweep_substep.hpp"

namespace fd6 {

namespace {
template <typename T, typename TW, int VS>
hipError_t launch_fused12_vs(const Geom& g, Fields4<T> in, Fields4<T> out, Fields4<TW> w,
                             const Coef<T>& c, const RKCoef<TW>& rk1, const RKCoef<TW>& rk2,
                             int zchunk, hipStream_t st) {
    constexpr int TX = 16, TY = 16, PD = 2;
    constexpr int NT = (TX + 2 * kR) * (TY + 2 * kR);
    constexpr auto kern = substep55_fused12<T, TW, TX, TY, PD, true, VS>;
    const int res = resident_blocks<kern>(NT);
    const SweepGrid sg = sweep_grid(g, TX, TY, zchunk, res);
    hipLaunchKernelGGL(kern, dim3(sg.blocks), dim3(NT), 0, st, g, in, out, w, c, rk1, rk2, sg);
    return hipGetLastError();
}
}  // namespace

template <typename T, typename TW>
hipError_t launch_fused12(const Geom& g, Fields4<T> in, Fields4<T> out, Fields4<TW> w,
                          const Coef<T>& c, const RKCoef<TW>& rk1, const RKCoef<TW>& rk2,
                          int zchunk, hipStream_t st) {
    return g.vs == 4 ? launch_fused12_vs<T, TW, 4>(g, in, out, w, c, rk1, rk2, zchunk, st)
                     : launch_fused12_vs<T, TW, 1>(g, in, out, w, c, rk1, rk2, zchunk, st);
}

namespace {
template <typename T>
__global__ __launch_bounds__(256) void unpack_w_kernel(Geom g, Fields4<T> w, Fields4<T> dst) {
    const int rows = g.ny * g.nz;
    for (int r = blockIdx.x; r < rows; r += gridDim.x) {
        const int k = r / g.ny, j = r - k * g.ny;
        const long long to = g.origin + (long long)k * g.plane + (long long)j * g.px;
        const long long from = (long long)k * g.wplane + (long long)j * g.wpx;
        for (int i = threadIdx.x; i < g.nx; i += blockDim.x)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                dst.f[q][(to + i) * g.vs] = w.f[q][(from + i) * g.vs];
    }
}
}  // namespace

template <typename T>
hipError_t launch_unpack_w(const Geom& g, Fields4<T> w, Fields4<T> dst, hipStream_t st) {
    const long long rows = (long long)g.ny * g.nz;
    const unsigned grid = (unsigned)(rows < 8192 ? rows : 8192);
    hipLaunchKernelGGL(unpack_w_kernel<T>, dim3(grid), dim3(256), 0, st, g, w, dst);
    return hipGetLastError();
}

template hipError_t launch_unpack_w<float>(const Geom&, Fields4<float>, Fields4<float>,
                                           hipStream_t);
template hipError_t launch_fused12<float, float>(const Geom&, Fields4<float>, Fields4<float>,
                                                 Fields4<float>, const Coef<float>&,
                                                 const RKCoef<float>&, const RKCoef<float>&, int,
                                                 hipStream_t);

}  // namespace fd6
