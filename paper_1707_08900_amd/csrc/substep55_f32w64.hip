// Instantiations of the z-sweep substep kernels (55-point single box and
// batch, 19-point single box) for state type float and RK3
// register type double (one translation unit per precision form keeps the
// build parallel).
#include "sweep_substep.hpp"

namespace fd6 {

template hipError_t launch_substep55<float, double>(const Geom&, Fields4<float>, Fields4<float>,
                                              Fields4<double>, const Coef<float>&,
                                              const RKCoef<double>&, int, int, int, double*, int,
                                              int*, const ForceArgs<float>*, hipStream_t);
template hipError_t launch_batch55<float, double>(const BatchBox<float, double>*, const BatchItem*, const int*,
                                            int, int, int, int, hipStream_t);
template int batch55_blocks_per_cu<float, double>(int);
template hipError_t launch_substep19<float, double>(const Geom&, Fields4<float>, Fields4<float>,
                                              Fields4<double>, const float*, const Coef<float>&,
                                              const RKCoef<double>&, int, int, int, double*, int,
                                              int*, const ForceArgs<float>*, hipStream_t);

}  // namespace fd6
