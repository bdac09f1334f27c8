// A device made of host memory for the host side of the library (lb_api.hip):
// streams run at once, "kernels" keep only the time level of a state in its first
// value, and a captured graph never instantiates.  The program runs an adjoint
// context forward and backward and prints the time levels of the tape entries
// that the adjoint steps read, in order.
#include "lb.h"
#include "lb_internal.h"

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

namespace {
bool capturing = false;
int instantiations = 0;
std::vector<double> levels;
size_t entry = 0;  // values per tape entry
std::string route;
double* at(const void* p) { return static_cast<double*>(const_cast<void*>(p)); }
}  // namespace

extern "C" {
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(16); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(16); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { capturing = true; return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) { capturing = false; *g = nullptr; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { ++instantiations; return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
}

namespace lbk {
int step2_resident(int, int) { return -1; }
int adj_blocks(int64_t n) { return (int)((n + 255) / 256); }
hipError_t launch_init(int, const double*, const double*, const double*, void* dst, const Geom&, const Coef&, hipStream_t)
{
    *at(dst) = 0.0;
    return hipSuccess;
}
static hipError_t advance(const void* src, void* dst, void* tape, int steps)
{
    if (capturing) return hipSuccess;
    for (int j = 0; tape && j < steps; ++j) at(tape)[j * entry] = *at(src) + j;
    *at(dst) = *at(src) + steps;
    return hipSuccess;
}
hipError_t launch_tile(int, const void* src, void* dst, const TileGeom& g, const Coef&, void* tape, hipStream_t)
{
    route += " t" + std::to_string(g.steps);
    return advance(src, dst, tape, g.steps);
}
hipError_t launch_step(int, int mode, const void* src, void* dst, const Geom&, const Coef&, double* tape, hipStream_t)
{
    route += " w1";
    return mode == MODE_ENERGY ? hipSuccess : advance(src, dst, mode == MODE_STEP_TAPE ? tape : nullptr, 1);
}
hipError_t launch_step2(int, const void* src, void* dst, const Geom&, const Coef&, hipStream_t)
{
    route += " w2";
    return advance(src, dst, nullptr, 2);
}
hipError_t launch_tile_batch(int, const TileBatch& b, hipStream_t)
{
    route += " t" + std::to_string(b.steps);
    return hipSuccess;
}
hipError_t launch_step2_batch(int, bool, const BatchLattice*, const int32_t*, int, int, uint32_t, hipStream_t)
{
    route += " w2";
    return hipSuccess;
}
hipError_t launch_step_batch(int, int, int, int, int, const BatchLattice*, const int32_t*, int, int, uint32_t, double*, hipStream_t)
{
    route += " w1";
    return hipSuccess;
}
void coef_to_f32(const Coef&, float*) {}
hipError_t launch_final(const double*, int, double t, double, double* row, hipStream_t)
{
    row[0] = t;
    return hipSuccess;
}
hipError_t launch_clear(int* flag, hipStream_t)
{
    route += " clear";
    *flag = 0;
    return hipSuccess;
}
hipError_t launch_check(const double* v, int64_t n, bool positive, int* flag, hipStream_t)
{
    route += " check";
    for (int64_t i = 0; i < n; ++i)
        if (!std::isfinite(v[i]) || (positive && !(v[i] > 0.0))) *flag = 1;
    return hipSuccess;
}
hipError_t adj_tape(int, const void*, const Geom&, const AdjParams&, void*, hipStream_t) { return hipSuccess; }
hipError_t adj_area(const AdjParams&, const void*, double, void*, double*, hipStream_t) { return hipSuccess; }
hipError_t adj_seed(const AdjParams&, const void*, const void*, double, double, void*, double*, hipStream_t) { return hipSuccess; }
hipError_t adj_rho_grad(const AdjParams&, const void*, double*, hipStream_t) { return hipSuccess; }
hipError_t adj_reduce(const double*, int, int, double*, hipStream_t) { return hipSuccess; }
hipError_t adj_zero(double*, int64_t, hipStream_t) { return hipSuccess; }
hipError_t adj_steps(const AdjParams&, const AdjTile& g, const void*, const void* tape, void*, double*, hipStream_t)
{
    if (!capturing)
        for (int j = 0; j < g.steps; ++j) levels.push_back(*(at(tape) - j * entry));
    return hipSuccess;
}
}  // namespace lbk

static int fail()
{
    std::fprintf(stderr, "%s\n", lb_last_error());
    return 1;
}

static lb_params params(int storage, int nx, int ny)
{
    lb_params p{};
    p.nx = nx;
    p.ny = ny;
    p.storage = storage;
    p.tau = p.rho0 = 1.0;
    p.G1 = -4.9;
    p.rho_ref = 0.7;
    return p;
}

static void* workspace(size_t bytes) { return std::aligned_alloc(256, (bytes + 255) / 256 * 256); }

static int adjoint(int side, int64_t T, int32_t every)
{
    const lb_params p = params(LB_F64, side, side);
    entry = (size_t)4 * p.nx * p.ny;
    const size_t bytes = lb_adj_workspace_bytes(&p, T, every);
    void* ws = workspace(bytes);
    std::memset(ws, 0xff, bytes);
    std::vector<double> rho(entry / 4, 0.7), drho(entry / 4);
    lb_adj* a = nullptr;
    const lb_adj_loss loss{0.0, 0.0, 1e-6};
    double out[4], dG[2];
    if (lb_adj_init(&a, &p, T, every, ws, bytes, reinterpret_cast<void*>(32)) ||
        lb_adj_forward(a, rho.data(), 0, p.G1, p.G2, &loss, out) || lb_adj_backward(a, dG, drho.data(), 0))
        return fail();
    std::printf("%d", instantiations);
    for (double v : levels) std::printf(" %g", v);
    std::printf("\n");
    lb_adj_destroy(a);
    std::free(ws);
    return 0;
}

static int steps(const lb_params& p, int calls, char** n)
{
    const size_t bytes = lb_workspace_bytes(&p);
    void* ws = workspace(bytes);
    std::vector<double> rho((size_t)p.nx * p.ny, 0.7);
    lb_ctx* c = nullptr;
    if (lb_init(&c, &p, ws, bytes, rho.data(), nullptr, nullptr, 0, nullptr)) return fail();
    for (int i = 0; i < calls; ++i) {
        route.clear();
        if (lb_step(c, std::atoi(n[i]))) return fail();
        std::printf("%s\n", route.c_str() + 1);
    }
    lb_destroy(c);
    std::free(ws);
    return 0;
}

static int batch(const lb_params& p, int count, int calls, char** n)
{
    const std::vector<lb_params> ps(count, p);
    const size_t bytes = lb_batch_workspace_bytes(ps.data(), count);
    void* ws = workspace(bytes);
    const std::vector<double> rho((size_t)p.nx * p.ny, 0.7);
    const std::vector<const double*> rhos(count, rho.data());
    lb_batch* b = nullptr;
    if (lb_batch_init(&b, ps.data(), count, ws, bytes, rhos.data(), 0, nullptr)) return fail();
    for (int i = 0; i < calls; ++i) {
        if (n[i][0] == 'h') {
            int32_t rows = 0;
            const int rc = lb_batch_two_step_tile(b, std::atoi(n[i] + 1));
            lb_batch_two_step_shape(b, nullptr, &rows, nullptr);
            std::printf("%d %d\n", rc, rows);
            continue;
        }
        route.clear();
        if (lb_batch_step(b, std::atoi(n[i]))) return fail();
        std::printf("%s\n", route.c_str() + 1);
    }
    lb_batch_destroy(b);
    std::free(ws);
    return 0;
}

static int init(const lb_params& p, int site, double value)
{
    const size_t bytes = lb_workspace_bytes(&p);
    void* ws = workspace(bytes);
    std::vector<double> rho((size_t)p.nx * p.ny, 0.7), u(rho.size(), 0.0);
    rho[site] = value;
    lb_ctx* c = nullptr;
    const int rc = lb_init(&c, &p, ws, bytes, rho.data(), u.data(), u.data(), 1, nullptr);
    std::printf("%d%s\n%s\n", rc, route.c_str(), rc ? lb_last_error() : "");
    if (!rc) lb_destroy(c);
    std::free(ws);
    return 0;
}

int main(int argc, char** argv)
{
    const std::string mode = argc > 1 ? argv[1] : "";
    auto arg = [&](int i) { return std::atoi(argv[i]); };
    if (mode == "adjoint" && argc == 5) return adjoint(arg(2), arg(3), arg(4));
    if (mode == "steps" && argc > 5) return steps(params(arg(2), arg(3), arg(4)), argc - 5, argv + 5);
    if (mode == "batch" && argc > 6) return batch(params(arg(2), arg(4), arg(5)), arg(3), argc - 6, argv + 6);
    if (mode == "init" && argc == 7) return init(params(arg(2), arg(3), arg(4)), arg(5), std::atof(argv[6]));
    return 2;
}
