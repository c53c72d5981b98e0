// The library's host runtime (fd6_abi.cpp) over a simulated device, built by
// test_host_runtime.py with the host compiler: launches are written to a log and
// advance a simulated clock, events read that clock, memory is never touched.
#include "fd6_abi.cpp"

#include <map>
#include <sstream>

namespace {

std::ostringstream g_log;
double g_clock = 0.0;           // ms
double g_capture = 0.0;         // ms recorded by the capture in progress
bool g_capturing = false;
std::map<int, double> g_cost;   // ms per substep launch, by kernel shape
std::map<int, double> g_chunk;  // factor, by z-chunk length (boxes) or grid (ensembles)
int g_fail_tile = -100;
constexpr int kShapes = 14;

void spend(double ms) { (g_capturing ? g_capture : g_clock) += ms; }

hipError_t substep(const char* name, int s, int tile, int zchunk) {
    g_log << name << ' ' << s << ' ' << tile << ' ' << zchunk << '\n';
    if (tile == g_fail_tile) return hipErrorLaunchFailure;
    const auto c = g_cost.find(tile), z = g_chunk.find(zchunk);
    spend((c == g_cost.end() ? 1.0 : c->second) * (z == g_chunk.end() ? 1.0 : z->second));
    return hipSuccess;
}

hipError_t note(const char* name) {
    g_log << name << '\n';
    return hipSuccess;
}

}  // namespace

extern "C" {
const char* hr_log() {
    static std::string s;
    s = g_log.str();
    g_log.str("");
    return s.c_str();
}
void hr_cost(int tile, double ms) { g_cost[tile] = ms; }
void hr_chunk(int zchunk, double factor) { g_chunk[zchunk] = factor; }
void hr_fail_tile(int tile) { g_fail_tile = tile; }
// b of the three substeps, c of the last two
void hr_fp32_factors(double dt, float* f) {
    const auto r = make_rk<float, float>(dt);
    for (int s = 0; s < 3; ++s) f[s] = r[s].b;
    f[3] = r[1].c;
    f[4] = r[2].c;
}
// FP32 weights of the viscous term for spacings h: second derivatives s[3][3] and
// (4/3) s[3][3], the centre weights of the three components, that of the 19-point method
void hr_fp32_viscous(double nu, const double* h, int variant, double* out) {
    const Coef<float> c = make_coef<float>(fd6_params{nu, 1.0, h[0], h[1], h[2], 1.0}, variant, false);
    for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 3; ++k) *out++ = c.s[a][k];
    for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 3; ++k) *out++ = c.s4[a][k];
    for (int i = 0; i < 3; ++i) *out++ = c.kc[i];
    *out++ = c.kc19;
}
void hr_reset() {
    g_log.str("");
    g_clock = g_capture = 0.0;
    g_cost.clear();
    g_chunk.clear();
    g_fail_tile = -100;
}

// The device.  An event or a graph holds the clock or the time it takes.
hipError_t hipEventCreate(hipEvent_t* e) {
    *e = reinterpret_cast<hipEvent_t>(new double(0.0));
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    delete reinterpret_cast<double*>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
    *reinterpret_cast<double*>(e) = g_clock;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b) {
    *ms = (float)(*reinterpret_cast<double*>(b) - *reinterpret_cast<double*>(a));
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(8);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
    g_capturing = true;
    g_capture = 0.0;
    return note("capture");
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
    g_capturing = false;
    *g = reinterpret_cast<hipGraph_t>(new double(g_capture));
    return note("end");
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t) {
    *x = reinterpret_cast<hipGraphExec_t>(new double(*reinterpret_cast<double*>(g)));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
    delete reinterpret_cast<double*>(g);
    return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
    delete reinterpret_cast<double*>(x);
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t) {
    g_clock += *reinterpret_cast<double*>(x);
    return note("replay");
}
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) {
    *v = 256;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    std::snprintf(p->name, sizeof p->name, "simulated");
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "simulated failure"; }
}

namespace fd6 {

int substep55_tile_count() { return kShapes; }
bool substep55_reads_ghosts(int tile) { return tile == 0; }
bool substep55_aos_tile_ok(int tile) { return tile > 0 && tile < kShapes && tile != 9; }
int substep55_tile_dims(int tile, int* tx, int* ty) {
    if (tile <= 0 || tile >= kShapes) return -1;
    const bool narrow = tile == 4 || tile == 8 || tile == 13;
    *tx = narrow ? 32 : 64;
    *ty = 8;
    return 0;
}

template <typename T, typename TW>
hipError_t launch_substep55(const Geom&, Fields4<T>, Fields4<T>, Fields4<TW>, const Coef<T>&,
                            const RKCoef<TW>&, int s, int tile, int zchunk, double*, int, int*,
                            const ForceArgs<T>*, hipStream_t) {
    return substep("substep", s, tile, zchunk);
}
template <typename T, typename TW>
hipError_t launch_substep55_aos(const Geom&, Fields4<T>, Fields4<T>, Fields4<TW>,
                                const Coef<T>&, const RKCoef<TW>&, int s, int tile, int zchunk,
                                double*, int, int*, const ForceArgs<T>*, hipStream_t) {
    return substep("substep", s, tile, zchunk);
}
template <typename T, typename TW>
hipError_t launch_substep19(const Geom&, Fields4<T>, Fields4<T>, Fields4<TW>, const T*,
                            const Coef<T>&, const RKCoef<TW>&, int s, int tile, int zchunk,
                            double*, int, int*, const ForceArgs<T>*, hipStream_t) {
    return substep("substep", s, tile, zchunk);
}
template <typename T, typename TW>
hipError_t launch_batch55(const BatchBox<T, TW>*, const BatchItem*, const int*, int grid, int,
                          int s, int tile, hipStream_t) {
    return substep("batch", s, tile, grid);
}
template <typename T, typename TW>
hipError_t launch_batch55_aos(const BatchBox<T, TW>*, const BatchItem*, const int*, int grid,
                              int, int s, int tile, hipStream_t) {
    return substep("batch", s, tile, grid);
}
template <typename T, typename TW>
int batch55_blocks_per_cu(int) {
    return 2;
}
template <typename T, typename TW>
int batch55_blocks_per_cu_aos(int) {
    return 2;
}
template <typename T, typename TW>
hipError_t launch_fused12(const Geom&, Fields4<T>, Fields4<T>, Fields4<TW>, const Coef<T>&,
                          const RKCoef<TW>&, const RKCoef<TW>&, int, hipStream_t) {
    return note("fused12");
}
template <typename T>
hipError_t launch_unpack_w(const Geom&, Fields4<T>, Fields4<T>, hipStream_t) {
    return note("unpack");
}
template <typename T>
hipError_t launch_div19(const Geom&, Fields4<T>, T*, const Coef<T>&, hipStream_t) {
    return note("div");
}
template <typename T, typename TW>
hipError_t launch_pass19a(const Geom&, Fields4<T>, Fields4<T>, Fields4<TW>, T*, const Coef<T>&,
                          const RKCoef<TW>&, int, const ForceArgs<T>*, hipStream_t) {
    return note("pass19a");
}
template <typename T, typename TW>
hipError_t launch_pass19b(const Geom&, const T*, Fields4<T>, Fields4<TW>, const Coef<T>&,
                          const RKCoef<TW>&, hipStream_t) {
    return note("pass19b");
}
template <typename T>
hipError_t launch_ghost_fill(const Geom&, Fields4<T>, int, hipStream_t) {
    return note("ghosts");
}
template <typename T>
hipError_t launch_import(const Geom&, const double*, T*, long long, int, hipStream_t) {
    return hipSuccess;
}
template <typename T>
hipError_t launch_export(const Geom&, const T*, double*, long long, int, hipStream_t) {
    return hipSuccess;
}
template <typename TW>
hipError_t launch_export_w(const Geom&, const TW*, double*, int, int, hipStream_t) {
    return hipSuccess;
}
template <typename T>
hipError_t launch_import4(const Geom&, const double* const*, Fields4<T>, hipStream_t) {
    return hipSuccess;
}
template <typename T>
hipError_t launch_export4(const Geom&, Fields4<T>, double* const*, hipStream_t) {
    return hipSuccess;
}
template <typename T>
hipError_t launch_reduce(const Geom&, Fields4<T>, double*, double*, double, hipStream_t) {
    return note("reduce");
}
hipError_t launch_reduce_final(const double*, int, double*, double, hipStream_t) {
    return note("reduce_final");
}
template <typename T>
hipError_t launch_force_table(const Geom&, ForceDev<T>*, T*, const double*, double,
                              const double*, const double*, hipStream_t) {
    return note("force");
}

}  // namespace fd6
