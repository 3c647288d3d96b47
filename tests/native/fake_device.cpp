// fake_device.cpp -- drives the host side of the library (grid handles, launch
// shapes, schedules, the ALI and BiCGStab drivers) without a GPU: HIP's runtime
// calls and the kernel launchers are replaced by the functions below, device
// memory is host memory with an optional limit, and streams run at once or, in a
// capture, record.  Built with g++ and AddressSanitizer, so that a launch whose
// schedule, wavelength list or partial sums were freed ends the program.
//
// usage: fake_device CASE; exits non-zero on a failed check.
#include <cstdio>
#include <functional>
#include <set>
#include <unordered_map>

#include "rt_host.hpp"

// ---------------------------------------------------------------------------
// the device
// ---------------------------------------------------------------------------
namespace dev {
std::unordered_map<void *, size_t> live;
size_t used = 0, peak = 0, limit = (size_t)1 << 36;
bool capturing = false;
hipError_t last = hipSuccess;  // sticky until hipGetLastError, as in the runtime
using Graph = std::vector<std::function<void()>>;
Graph *recording = nullptr;
int failed_allocs = 0;

hipError_t err(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}
// a kernel launch
template <typename F>
hipError_t launch(F f)
{
    if (capturing) recording->push_back(f);
    else f();
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
// reads and writes the first and last byte of a range
void touch(const void *p, size_t n)
{
    if (!p || !n) return;
    volatile char *c = static_cast<volatile char *>(const_cast<void *>(p));
    c[0] = c[0];
    c[n - 1] = c[n - 1];
}
}  // namespace dev

extern "C" {
hipError_t hipMalloc(void **p, size_t n)
{
    if (dev::capturing) return dev::err(hipErrorStreamCaptureUnsupported);
    if (dev::used + n > dev::limit) {
        ++dev::failed_allocs;
        return dev::err(hipErrorOutOfMemory);
    }
    *p = std::calloc(1, n);
    dev::live[*p] = n;
    dev::used += n;
    dev::peak = std::max(dev::peak, dev::used);
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (dev::capturing) return dev::err(hipErrorStreamCaptureUnsupported);
    dev::used -= dev::live.at(p);
    dev::live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *t = dev::limit; *f = dev::limit - dev::used; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 100000; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = 256;
    p->sharedMemPerBlock = p->maxSharedMemoryPerMultiProcessor = 160 * 1024;
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "fake device error"; }
hipError_t hipGetLastError()
{
    const hipError_t e = dev::last;
    dev::last = hipSuccess;
    return e;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = reinterpret_cast<hipStream_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
static float event_ms = 1.f;  // time of the last sweep
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = event_ms; return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    dev::recording = new dev::Graph;
    dev::capturing = true;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    dev::capturing = false;
    *g = reinterpret_cast<hipGraph_t>(dev::recording);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t g, hipGraphNode_t *, char *, size_t)
{
    *x = reinterpret_cast<hipGraphExec_t>(new dev::Graph(*reinterpret_cast<dev::Graph *>(g)));
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) { delete reinterpret_cast<dev::Graph *>(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t x) { delete reinterpret_cast<dev::Graph *>(x); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    for (auto &f : *reinterpret_cast<dev::Graph *>(x)) f();
    return hipSuccess;
}
}

// ---------------------------------------------------------------------------
// checks and what the fake kernels report
// ---------------------------------------------------------------------------
static int g_fail = 0;
#define CHECK(c)                                                                \
    do {                                                                        \
        if (!(c)) {                                                             \
            std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__); \
            ++g_fail;                                                           \
        }                                                                       \
    } while (0)

struct LastSweep {
    int lb = 0, R = 0, nb = 0, n_wg = 0;
    bool band = false;
};
static LastSweep sweep;
static std::function<float(const LastSweep &)> sweep_ms = [](const LastSweep &) { return 1.f; };
static int updates = 0;                  // operator-splitting updates so far
static std::function<double(int)> rel_of = [](int) { return 1.0; };
static int occupancy_queries = 0;
static StencilRoute route;               // of the last stencil build

static void check_lambdas(const int32_t *lam, int n)
{
    for (int i = 0; i < n; ++i) CHECK(lam[i] >= 0 && lam[i] < 4096 && (i == 0 || lam[i] > lam[i - 1]));
}

// ---------------------------------------------------------------------------
// kernel launchers
// ---------------------------------------------------------------------------
namespace rt3d {
static const FsShape kShapes[] = {{1024, 1, true, 1, false}, {1024, 2, true, 1, false}, {1024, 4, true, 1, false},
                                  {768, 6, true, 1, false},  {512, 3, false, 2, false}, {1024, 1, true, 1, true},
                                  {1024, 2, true, 1, true},  {1024, 4, true, 1, true},  {768, 6, true, 1, true}};
int fs_box_shapes(const FsShape **out)
{
    *out = kShapes;
    return (int)(sizeof kShapes / sizeof kShapes[0]);
}
int fs_box_occupancy(bool, bool, bool, bool, bool, int lb, int, int nthr, size_t lds)
{
    ++occupancy_queries;
    return std::max(1, std::min<int>(lb / nthr, (int)(160 * 1024 / std::max<size_t>(lds, 1))));
}
hipError_t fs_box_launch(const FsBoxArgs &a, bool dbl, bool wj, bool wl, bool, bool band, int lb, int R, int n_wg, int nthr,
                         size_t, hipStream_t)
{
    CHECK(nthr <= lb);
    return dev::launch([=] {
        const size_t slot = (size_t)a.n_vox * (dbl ? 8 : 4);
        for (int w = 0; w < n_wg; ++w)
            for (int k = a.wg_begin[w]; k < a.wg_begin[w + 1]; ++k) {
                const WorkItem it = a.items[k];
                if (wj) dev::touch(static_cast<char *>(a.partJ) + it.slot * slot, slot);
                if (wl) dev::touch(static_cast<char *>(a.partL) + it.slot * slot, slot);
            }
        sweep.lb = lb; sweep.R = R; sweep.nb = a.n_bundles; sweep.n_wg = n_wg; sweep.band = band;
        event_ms = sweep_ms(sweep);
    });
}
template <typename TS, typename TD>
hipError_t pad_field(const TS *, const double *, TD *, int, int, int, int, int, hipStream_t)
{
    return dev::launch([] {});
}
template hipError_t pad_field<float, float>(const float *, const double *, float *, int, int, int, int, int, hipStream_t);
template hipError_t pad_field<float, double>(const float *, const double *, double *, int, int, int, int, int, hipStream_t);
template hipError_t pad_field<double, double>(const double *, const double *, double *, int, int, int, int, int, hipStream_t);
template <typename T>
hipError_t pad_pair(const T *, const T *, T *, int, int, int, int, hipStream_t)
{
    return dev::launch([] {});
}
template hipError_t pad_pair<float>(const float *, const float *, float *, int, int, int, int, hipStream_t);
template hipError_t pad_pair<double>(const double *, const double *, double *, int, int, int, int, hipStream_t);
template <typename TP, typename TO>
hipError_t reduce_partials(const TP *part, const int32_t *slot_begin, const int32_t *slot_ids, const int32_t *lambda_of,
                           int n_batch, TO *out, int64_t n_vox, hipStream_t, bool, const TP *, TO *)
{
    return dev::launch([=] {
        check_lambdas(lambda_of, n_batch);
        for (int b = 0; b < n_batch; ++b) {
            for (int s = slot_begin[b]; s < slot_begin[b + 1]; ++s)
                dev::touch(part + (int64_t)slot_ids[s] * n_vox, (size_t)n_vox * sizeof(TP));
            dev::touch(out + (int64_t)lambda_of[b] * n_vox, (size_t)n_vox * sizeof(TO));
        }
    });
}
template hipError_t reduce_partials<float, float>(const float *, const int32_t *, const int32_t *, const int32_t *, int,
                                                  float *, int64_t, hipStream_t, bool, const float *, float *);
template hipError_t reduce_partials<double, double>(const double *, const int32_t *, const int32_t *, const int32_t *,
                                                    int, double *, int64_t, hipStream_t, bool, const double *, double *);
template <typename G, typename TN>
hipError_t source_update(const double *, const G *, const G *, double *, const double *, TN *, int, int, int64_t,
                         const int32_t *lambda_of, int n_batch, hipStream_t)
{
    return dev::launch([=] { check_lambdas(lambda_of, n_batch); });
}
template hipError_t source_update<float, float>(const double *, const float *, const float *, double *, const double *,
                                                float *, int, int, int64_t, const int32_t *, int, hipStream_t);
template hipError_t source_update<double, double>(const double *, const double *, const double *, double *,
                                                  const double *, double *, int, int, int64_t, const int32_t *, int,
                                                  hipStream_t);
template hipError_t source_update<float, double>(const double *, const float *, const float *, double *, const double *,
                                                 double *, int, int, int64_t, const int32_t *, int, hipStream_t);
template <typename TS, typename TD>
hipError_t cast_array(const TS *, TD *, int64_t, hipStream_t)
{
    return dev::launch([] {});
}
template hipError_t cast_array<float, double>(const float *, double *, int64_t, hipStream_t);
hipError_t fill_u64(unsigned long long *p, unsigned long long v, int n, hipStream_t)
{
    return dev::launch([=] { std::fill(p, p + n, v); });
}
hipError_t wall_stamp(unsigned long long *, hipStream_t) { return dev::launch([] {}); }
hipError_t ali_update(const AliUpdateArgs &a, bool dbl, bool, bool, int n_batch, hipStream_t)
{
    return dev::launch([=] {
        check_lambdas(a.lambda_of, n_batch);
        for (int b = 0; a.part && !a.rfs_in && b < n_batch; ++b)
            for (int s = a.slot_begin[b]; s < a.slot_begin[b + 1]; ++s) {
                const size_t slot = (size_t)a.n_vox * (dbl ? 8 : 4);
                dev::touch(static_cast<const char *>(a.part) + (size_t)a.slot_ids[s] * slot, slot);
            }
        if (a.rfs_out) return;
        ++updates;
        for (int b = 0; b < n_batch; ++b) a.rel_change[a.lambda_of[b]] = rel_of(a.lambda_of[b]);
    });
}
hipError_t ng_accelerate(const NgApplyArgs &a, double *, int, int n_batch, bool, hipStream_t)
{
    return dev::launch([=] { check_lambdas(a.lambda_of, n_batch); });
}
hipError_t krylov_dots(const KDots &, int64_t, int n_lambda, double *, int, double *out, hipStream_t)
{
    return dev::launch([=] { std::fill(out, out + 4 * n_lambda, 1.0); });
}
hipError_t krylov_vec(const KVec &, int, int64_t, int, bool, hipStream_t) { return dev::launch([] {}); }
hipError_t lstar_stencil_accumulate(const StencilArgs &a, bool, bool para, int n_dir, int n_batch, size_t, hipStream_t)
{
    route = stencil_route(a, para, n_dir, n_batch);
    return dev::launch([=] { check_lambdas(a.lambda_of, n_batch); });
}
hipError_t lstar_stencil_finish(const unsigned long long *, const int32_t *lambda_of, int64_t, int n_batch, const void *,
                                void *, bool, hipStream_t)
{
    return dev::launch([=] { check_lambdas(lambda_of, n_batch); });
}
hipError_t os_jacobi_sweep(const OsJacobiArgs &a, bool, bool, int n_batch, hipStream_t)
{
    return dev::launch([=] { check_lambdas(a.lambda_of, n_batch); });
}
hipError_t os_gs_sweep(const OsJacobiArgs &a, bool d, int n_batch, hipStream_t st)
{
    return os_jacobi_sweep(a, d, false, n_batch, st);
}
// not reached: spherical grids and the network
hipError_t fs_sphere_launch(const FsSphereArgs &, bool, bool, bool, bool, bool, hipStream_t) { std::abort(); }
hipError_t sphere_gather(const void *, const void *, bool, const int32_t *, const int32_t *, int64_t, int, void *, void *,
                         bool, hipStream_t)
{
    std::abort();
}
hipError_t lstar_stencil_sphere_accumulate(const SphereStencilArgs &, bool, bool, bool, hipStream_t) { std::abort(); }
std::string parse_unet(const void *, size_t, UNetSpec &) { std::abort(); }
UNetDev *unet_create(const UNetSpec &, int, int, int, std::string &) { std::abort(); }
void unet_destroy(UNetDev *) { std::abort(); }
hipError_t unet_forward(UNetDev *, const float *, float *, hipStream_t) { std::abort(); }
template <typename G>
hipError_t unet_features(const float *, double, const G *, const G *, int64_t, float *, hipStream_t)
{
    std::abort();
}
template hipError_t unet_features<float>(const float *, double, const float *, const float *, int64_t, float *, hipStream_t);
template hipError_t unet_features<double>(const float *, double, const double *, const double *, int64_t, float *,
                                          hipStream_t);
hipError_t unet_apply(const float *, double, double *, int64_t, hipStream_t) { std::abort(); }
}  // namespace rt3d

rt_status noalloc_scratch_setup(int, void **out)
{
    *out = nullptr;
    return RT_OK;
}

// ---------------------------------------------------------------------------
// cases
// ---------------------------------------------------------------------------
struct Owner {
    rt_grid_t g = nullptr;
    Owner(int nx, int ny, int nz, int n_mu, int n_phi, rt_prec prec, int n_lambda, uint32_t flags = 0)
    {
        rt_grid_desc d{};
        d.struct_size = sizeof d;
        d.geom = RT_GEOM_BOX_PERIODIC_XY;
        d.n[0] = nx; d.n[1] = ny; d.n[2] = nz;
        d.n_mu = n_mu; d.n_phi = n_phi;
        d.n_lambda_max = n_lambda;
        d.prec = prec;
        d.flags = flags;
        if (rt_create_grid(&d, &g) != RT_OK) {
            std::fprintf(stderr, "no grid: %s\n", rt_last_error());
            std::exit(2);
        }
    }
    ~Owner() { rt_destroy_grid(g); }
};

// State arrays of n wavelengths (their contents do not matter here).
struct StateArrays {
    std::vector<double> mem, rel;
    rt_state s{};
    StateArrays(const Owner &o, int n) : mem((size_t)n * o.g->n_vox * 6), rel(n)
    {
        const size_t k = (size_t)n * o.g->n_vox;
        s.struct_size = sizeof s;
        s.n_lambda = n;
        s.chi = &mem[0]; s.eps = &mem[k]; s.B = &mem[2 * k];
        s.J = &mem[3 * k]; s.S = &mem[4 * k]; s.lstar = &mem[5 * k];
        s.rel_change = rel.data();
    }
};

static rt_solve_opts options(bool graph)
{
    rt_solve_opts o{};
    o.struct_size = sizeof o;
    o.tol = 1e-3;
    o.max_iter = 400;
    o.ng_every = 4;
    o.ng_start = 4;
    o.use_graph = graph ? 1 : 0;
    return o;
}

// Solves whose wavelengths converge one at a time, in another order each time:
// every step has a wavelength list of its own, and the schedules pass the
// number that a grid keeps many times over.
static void shrinking_batches()
{
    for (rt_prec prec : {RT_FP64, RT_FP32})
        for (uint32_t flags : {0u, RT_F_BAND_TILES, RT_F_LSTAR_NONLOCAL})
            for (bool graph : {false, true}) {
                const int n = 24;
                Owner o(24, 20, 4, 4, 8, prec, n, flags);
                hipStream_t st = nullptr;
                hipStreamCreateWithFlags(&st, 0);
                for (int turn = 0; turn < 6; ++turn) {
                    const int nl = n - turn;
                    StateArrays a(o, nl);
                    updates = 0;
                    rel_of = [=](int l) { return (l * 7 + 5 * turn) % n < updates - 2 ? 0.0 : 1.0; };
                    const rt_solve_opts opt = options(graph);
                    rt_solve_report rep{};
                    CHECK(rt_solve(o.g, &a.s, &opt, &rep, st) == RT_OK);
                    CHECK(rep.n_converged == nl && rep.iters > n / 2);
                }
                CHECK(o.g->schedules.size() <= 75);
                hipStreamDestroy(st);
                rel_of = [](int) { return 1.0; };
            }
}

// Calls of many kinds on one grid, each with schedules of its own (`shift` more of
// them first, so that the limit is passed at every place of the sequence).
static void mixed_calls()
{
    for (int shift = 0; shift < 8; ++shift) {
        Owner o(24, 20, 4, 4, 8, RT_FP32, 30);
        std::vector<double> in(30 * (size_t)o.g->n_vox), out(in.size()), st(27 * in.size());
        auto some_dirs = [&](int first, int n) {
            std::vector<int32_t> dirs(n);
            for (int i = 0; i < n; ++i) dirs[i] = first + i;
            CHECK(rt_formal_solution_dirs(o.g, 1, in.data(), in.data(), nullptr, n, dirs.data(), out.data(), nullptr,
                                          nullptr) == RT_OK);
        };
        for (int i = 0; i < shift; ++i) some_dirs(i + 1, 8);
        for (int n = 1; n <= 30; ++n) {
            StateArrays a(o, n);
            rt_solve_opts opt = options(false);
            opt.method = RT_SOLVER_BICGSTAB;
            opt.max_iter = 3;
            CHECK(rt_solve(o.g, &a.s, &opt, nullptr, nullptr) == RT_E_NOT_CONVERGED);
            CHECK(rt_formal_solution(o.g, n, in.data(), in.data(), nullptr, out.data(), n % 2 ? out.data() : nullptr,
                                     nullptr) == RT_OK);
            some_dirs(0, n);
            CHECK(rt_lstar_stencil(o.g, n, in.data(), st.data(), nullptr) == RT_OK);
            CHECK(o.g->schedules.size() <= 75);
        }
    }
}

// What a grid does with the default shapes and no stencil tables fits the memory that
// this takes, also from a start with the shapes of least estimated time.
static void calls_of_a_grid(Owner &o, bool graph, bool tune)
{
    const int n = 6;
    const size_t k = (size_t)n * o.g->n_vox;
    std::vector<double> in(k), out(k), L(k), st(27 * k);
    hipStream_t stream = nullptr;
    hipStreamCreateWithFlags(&stream, 0);
    CHECK(rt_formal_solution(o.g, 1, in.data(), in.data(), nullptr, out.data(), nullptr, stream) == RT_OK);
    updates = 0;
    rel_of = [=](int l) { return l < updates - 2 ? 0.0 : 1.0; };
    StateArrays a(o, n);
    rt_solve_opts opt = options(graph);
    const rt_status rs = rt_solve(o.g, &a.s, &opt, nullptr, stream);
    if (rs != RT_OK) std::fprintf(stderr, "%s\n", rt_last_error());
    CHECK(rs == RT_OK);
    CHECK(rt_formal_solution(o.g, n, in.data(), in.data(), nullptr, out.data(), L.data(), stream) == RT_OK);
    CHECK(rt_lstar_stencil(o.g, n, in.data(), st.data(), stream) == RT_OK);
    opt.method = RT_SOLVER_BICGSTAB;
    opt.max_iter = 2;
    CHECK(rt_solve(o.g, &a.s, &opt, nullptr, stream) == RT_E_NOT_CONVERGED);
    if (tune) CHECK(rt_autotune(o.g, 1, in.data(), in.data(), nullptr, nullptr, stream) == RT_OK);
    hipStreamDestroy(stream);
}

static void short_memory()
{
    const size_t all = dev::limit;
    for (rt_prec prec : {RT_FP64, RT_FP32})
        for (uint32_t flags : {0u, RT_F_BAND_TILES, RT_F_LSTAR_NONLOCAL, RT_F_LSTAR_NONLOCAL | RT_F_LSTAR_PARABOLIC})
            for (bool graph : {false, true}) {
                size_t plain, room;
                {
                    Owner o(24, 20, 4, 4, 8, prec, 6, flags);
                    o.g->tight = true;
                    dev::peak = 0;
                    calls_of_a_grid(o, graph, false);
                    plain = dev::peak;
                }
                {
                    Owner o(24, 20, 4, 4, 8, prec, 6, flags);
                    dev::peak = 0;
                    calls_of_a_grid(o, graph, false);
                    room = dev::peak;
                }
                CHECK(room > plain || flags == RT_F_BAND_TILES);
                // half a megabyte for the schedules of two shapes
                for (size_t extra = (size_t)1 << 19; plain + extra < room; extra = 2 * extra) {
                    Owner o(24, 20, 4, 4, 8, prec, 6, flags);
                    dev::limit = plain + extra;
                    dev::failed_allocs = 0;
                    calls_of_a_grid(o, graph, true);
                    CHECK(dev::failed_allocs > 0);
                    dev::limit = all;
                }
            }
}

// The shape that a fresh grid reports can be set again, through either entry point.
static void default_shape_again()
{
    int bands = 0;
    for (int nx : {12, 33, 46, 65, 97})
        for (rt_prec prec : {RT_FP64, RT_FP32})
            for (uint32_t flags : {0u, RT_F_BAND_TILES})
                for (bool named : {false, true}) {
                    Owner o(nx, 45, 5, 4, 8, prec, 2, flags);
                    int32_t t, r, nb, band, t1, r1, nb1, band1;
                    CHECK(rt_launch_shape(o.g, &t, &r, &nb, &band) == RT_OK);
                    CHECK((named ? rt_set_launch_shape_tiles(o.g, t, r, band) : rt_set_launch_shape(o.g, t, r)) == RT_OK);
                    CHECK(rt_launch_shape(o.g, &t1, &r1, &nb1, &band1) == RT_OK);
                    CHECK(t == t1 && r == r1 && nb == nb1 && band == band1);
                    bands += band && !(flags & RT_F_BAND_TILES);
                }
    CHECK(bands > 0);  // layer grids whose default is band tiles are among them
}

// The shape that the autotuner keeps can be set again on a fresh grid, whichever is
// the fastest: it is known by threads, rays and tile kind alone.
static void tuned_shape_again()
{
    std::set<std::pair<int, int>> kept;
    for (uint32_t flags : {0u, RT_F_BAND_TILES})
        for (int fast = 0; fast < 12; ++fast) {
            sweep_ms = [=](const LastSweep &w) { return w.nb == fast ? 1.f : 2.f + w.nb; };
            std::vector<double> in(65 * 45 * 5);
            Owner o(65, 45, 5, 4, 8, RT_FP64, 1, flags), fresh(65, 45, 5, 4, 8, RT_FP64, 1, flags);
            int32_t t, r, nb, band, t1, r1, nb1, band1;
            CHECK(rt_autotune(o.g, 1, in.data(), in.data(), nullptr, nullptr, nullptr) == RT_OK);
            CHECK(rt_launch_shape(o.g, &t, &r, &nb, &band) == RT_OK);
            CHECK(rt_set_launch_shape_tiles(fresh.g, t, r, band) == RT_OK);
            CHECK(rt_launch_shape(fresh.g, &t1, &r1, &nb1, &band1) == RT_OK);
            CHECK(t == t1 && r == r1 && nb == nb1 && band == band1);
            kept.insert({t, r});
        }
    CHECK(kept.size() > 1);
    sweep_ms = [](const LastSweep &) { return 1.f; };
}

// What the runtime says of a compiled shape does not depend on the call: batches and
// shares of other sizes choose among the shapes of the first call without asking again.
static void shapes_asked_once()
{
    for (rt_prec prec : {RT_FP64, RT_FP32}) {
        Owner o(46, 45, 5, 4, 8, prec, 12);
        std::vector<double> in(12 * (size_t)o.g->n_vox), out(in.size());
        std::vector<int32_t> dirs;
        for (int n = 1; n <= 12; ++n) {
            occupancy_queries = 0;
            dirs.push_back(n);
            CHECK(rt_formal_solution(o.g, n, in.data(), in.data(), nullptr, out.data(), nullptr, nullptr) == RT_OK);
            CHECK(rt_formal_solution_dirs(o.g, n, in.data(), in.data(), nullptr, n, dirs.data(), out.data(), nullptr,
                                          nullptr) == RT_OK);
            CHECK((occupancy_queries > 0) == (n == 1));
        }
    }
}

// The slots that a schedule opens, which size the fixed scratch of the no-allocation
// formal solution.
static void slot_bound()
{
    for (int n_mu : {2, 4, 8})
        for (int n_phi : {1, 3, 16}) {
            BoxGeometry geo;
            CHECK(build_box_geometry(9, 7, 5, n_mu, n_phi, geo).empty());
            for (int nl : {1, 2, 3, 5, 11, 26})
                for (int nb : {1, 2, 3, 5})
                    for (int w = nb; w < 300; w += w < 20 ? nb : 7 * nb) {
                        std::vector<int32_t> lams(nl);
                        for (int i = 0; i < nl; ++i) lams[i] = i;
                        Schedule s;
                        build_schedule(geo, lams, w, s, nullptr, nb);
                        CHECK(s.n_slots <= std::min(w + nb * (nl - 1), nl * n_mu * n_phi * nb));
                    }
        }
}

// Stencils of many characteristics go by voxels or by rows on every quadrature, those of
// few by voxels or by characteristics.
static void stencil_routes()
{
    int ties = 0;
    for (uint32_t flags : {0u, RT_F_LSTAR_PARABOLIC})
        for (int n_mu : {2, 4, 6, 10})
            for (int n_phi = 1; n_phi <= 12; ++n_phi)
                for (int nx : {10, 456}) {
                    const bool many = nx * nx * n_mu * n_phi >= 400000;
                    Owner o(nx, nx, 2, n_mu, n_phi, RT_FP32, 1, flags);
                    std::vector<float> in(o.g->n_vox), st(27 * in.size());
                    CHECK(rt_lstar_stencil(o.g, 1, in.data(), st.data(), nullptr) == RT_OK);
                    const bool tie = o.g->nl_near <= 0;  // templates that cross two faces at once
                    CHECK(flags ? route == StencilRoute::rows
                                : route == (!tie ? StencilRoute::voxels : many ? StencilRoute::rows : StencilRoute::characteristics));
                    ties += !flags && tie && many;
                }
    CHECK(ties > 0);
}

// The workgroups that meet on one of 256 CUs (dealt in turn) add up to about the same
// number of visits everywhere.
static void balanced_cus()
{
    for (int nl : {2, 5, 8, 14})
        for (int nb : {1, 2, 4})
            for (int per_cu : {2, 4, 7}) {
                BoxGeometry geo;
                CHECK(build_box_geometry(20, 20, 30, 16, 24, geo).empty());
                std::vector<int32_t> lams(nl);
                for (int i = 0; i < nl; ++i) lams[i] = i;
                Schedule s;
                build_schedule(geo, lams, 256 * per_cu, s, nullptr, nb);
                std::vector<double> cu(256, 0.0);
                double sum = 0.0, longest = 0.0;
                for (int w = 0; w < s.n_wg; ++w) {
                    double load = 0.0;
                    for (int k = s.wg_begin[w]; k < s.wg_begin[w + 1]; ++k) load += geo.dirs[s.items[k].dir].M;
                    cu[w % 256] += load;
                    sum += load;
                    longest = std::max(longest, load);
                }
                // as far as whole workgroups allow: half of the heaviest one above the mean
                CHECK(*std::max_element(cu.begin(), cu.end()) <= std::max(longest, sum / 256 + 0.5 * longest));
            }
}

int main(int argc, char **argv)
{
    const std::string which = argc > 1 ? argv[1] : "";
    if (which == "shrinking_batches") shrinking_batches();
    else if (which == "mixed_calls") mixed_calls();
    else if (which == "short_memory") short_memory();
    else if (which == "default_shape_again") default_shape_again();
    else if (which == "tuned_shape_again") tuned_shape_again();
    else if (which == "shapes_asked_once") shapes_asked_once();
    else if (which == "slot_bound") slot_bound();
    else if (which == "stencil_routes") stencil_routes();
    else if (which == "balanced_cus") balanced_cus();
    else return 2;
    if (g_fail == 0) std::printf("%s passed\n", which.c_str());
    return g_fail == 0 ? 0 : 1;
}
