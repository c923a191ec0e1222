// The library's host code (api.cpp, adaptive.cpp, device_cache.cpp, tables.cpp, host_tree.cpp) over a HIP
// runtime of this file's own: device memory is host memory, allocations can be made to fail,
// kernel launchers check the arrays they are handed and compute nothing.  Each check runs in a
// child process of its own and names what it found.
//
// Usage: fake_runtime CHECK
#include <sys/wait.h>
#include <unistd.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../include/fmm2d.h"
#include "../include/fmm2d_adaptive.h"
#include "../paper_1008_2410_amd/csrc/adaptive_internal.h"
#include "../paper_1008_2410_amd/csrc/build_prims.h"
#include "../paper_1008_2410_amd/csrc/cost_order.h"
#include "../paper_1008_2410_amd/csrc/fmm_internal.h"

#define REQUIRE(cond)                                                                  \
    do {                                                                               \
        if (!(cond)) {                                                                 \
            printf("%s:%d: %s\n", __FILE__, __LINE__, #cond);                          \
            fflush(stdout);                                                            \
            _exit(1);                                                                  \
        }                                                                              \
    } while (0)

// Host allocations fail from this one on (-1: none does).
static int64_t g_new_left = -1;
void *operator new(size_t n)
{
    if (g_new_left == 0) throw std::bad_alloc();
    if (g_new_left > 0) --g_new_left;
    return malloc(n ? n : 1);
}
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }

// ---------------------------------------------------------------------------------
// The runtime
// ---------------------------------------------------------------------------------
namespace {
std::map<char *, size_t> g_live;  // device allocations
size_t g_used = 0;
int64_t g_allocs = 0, g_frees = 0, g_waits = 0;  // calls that a stream capture refuses
int64_t g_memsets = 0;                           // and that must not become nodes of a graph
int64_t g_fail_from = -1;                        // allocations from this one on fail
size_t g_capacity = SIZE_MAX;                    // so do those that would exceed this
size_t g_pool_used = 0, g_pool_idle = 0;         // of the stream-ordered pool

hipError_t take(void **p, size_t bytes)
{
    *p = nullptr;
    const int64_t number = g_allocs++;
    if ((g_fail_from >= 0 && number >= g_fail_from) || g_used + g_pool_idle + bytes > g_capacity) return hipErrorOutOfMemory;
    *p = calloc(1, bytes ? bytes : 1);
    const int64_t left = g_new_left;  // (this runtime's own entries are not the library's)
    g_new_left = -1;
    g_live[(char *)*p] = bytes;
    g_new_left = left;
    g_used += bytes;
    return hipSuccess;
}

hipError_t give(void *p)
{
    if (!p) return hipSuccess;
    ++g_frees;
    auto it = g_live.find((char *)p);
    REQUIRE(it != g_live.end());  // freed twice, or not device memory
    g_used -= it->second;
    g_live.erase(it);
    free(p);
    return hipSuccess;
}

bool on_device(const void *p, size_t bytes)
{
    auto it = g_live.upper_bound((char *)p);
    if (it == g_live.begin()) return false;
    --it;
    return (char *)p + bytes <= it->first + it->second;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { return take(p, n); }
hipError_t hipFree(void *p) { return give(p); }
// The stream-ordered pool: what is given back stays reserved until it is trimmed (a release
// threshold without limit).
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t)
{
    const size_t reuse = std::min(n, g_pool_idle);
    g_pool_idle -= reuse;
    const hipError_t e = take(p, n);
    if (e != hipSuccess) g_pool_idle += reuse;
    else g_pool_used += n;
    return e;
}
hipError_t hipFreeAsync(void *p, hipStream_t)
{
    const size_t n = g_live.count((char *)p) ? g_live[(char *)p] : 0;
    g_pool_used -= n;
    g_pool_idle += n;
    return give(p);
}
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t *p, int) { *p = (hipMemPool_t)&g_pool_idle; return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMemPoolGetAttribute(hipMemPool_t, hipMemPoolAttr a, void *v)
{
    if (a == hipMemPoolAttrUsedMemCurrent) *(uint64_t *)v = g_pool_used;
    else if (a == hipMemPoolAttrReservedMemCurrent) *(uint64_t *)v = g_pool_used + g_pool_idle;
    else return hipErrorInvalidValue;
    return hipSuccess;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t keep)
{
    g_pool_idle = std::min(g_pool_idle, keep > g_pool_used ? keep - g_pool_used : 0);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { ++g_waits; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { ++g_waits; return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemset(void *d, int v, size_t n)
{
    REQUIRE(on_device(d, n));
    memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t)
{
    ++g_memsets;
    return hipMemset(d, v, n);
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)malloc(1); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { free((void *)s); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { free((void *)e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
}

// ---------------------------------------------------------------------------------
// The device builds and the launchers
// ---------------------------------------------------------------------------------
namespace fmm {

static bool g_mutual = true;  // whether the trees' plans have mutual items

// A tree that cannot be evaluated, with arrays of g_tree_bytes from where the device build takes them.
static size_t g_tree_bytes = 1 << 20;
int build_tree_device(fmm_tree *t, const double *, const double *, hipStream_t s, std::string &, int64_t &,
                      const std::function<void()> &)
{
    t->pooled = true;
    return pool_malloc((void **)&t->slab, g_tree_bytes, s) == hipSuccess ? FMM_OK : FMM_ENOMEM;
}
int build_near_plan_device(fmm_tree *t, hipStream_t, std::string &)
{
    t->nmut = g_mutual ? 1 : 0;
    t->nnear_work = 1;
    return FMM_OK;
}
int build_atree_device(fmm_atree *t, const double *, const double *, hipStream_t, std::string &, int64_t &)
{
    t->pooled = true;
    return block_alloc((void **)&t->d.perm, g_tree_bytes) == hipSuccess ? FMM_OK : FMM_ENOMEM;
}
// (a list of the tree's own, made with an allocation and a wait)
static int make_list(int **p, int64_t count)
{
    if (hipMalloc((void **)p, (size_t)count * sizeof(int)) != hipSuccess) return FMM_ENOMEM;
    return hipStreamSynchronize(nullptr) == hipSuccess ? FMM_OK : FMM_EDEVICE;
}
static std::vector<int *> g_lists;
int build_atree_adjoint_units(fmm_atree *t, hipStream_t, std::string &)
{
    int *p = nullptr;
    if (int rc = make_list(&p, t->ntiles)) return rc;
    g_lists.push_back(p);
    t->nbwd_units = t->ntiles;
    return FMM_OK;
}
int build_atree_m2l_plan(fmm_atree *t, const int4 *, hipStream_t, std::string &)
{
    int *p = nullptr;
    if (int rc = make_list(&p, 1)) return rc;
    g_lists.push_back(p);
    t->m2l_plan = true;
    return FMM_OK;
}
int static_workspace(int, char **base)
{
    static char *scratch = nullptr;
    if (!scratch) {
        scratch = (char *)calloc(1, kStaticWorkspaceBytes);
        g_live[scratch] = kStaticWorkspaceBytes;
    }
    *base = scratch;
    return 0;
}

static size_t real_bytes(int is_double) { return is_double ? sizeof(double) : sizeof(float); }

static void check_far(const FarArgs &a)
{
    const int L = a.t->depth;
    if (L < 2) return;
    const int64_t d = level_base(std::min(a.split, L) + 1), f = level_base(L + 1) - d;
    REQUIRE(on_device(a.mp_d, d * a.p * sizeof(double2)) && on_device(a.lo_d, d * a.p * sizeof(double2)));
    if (f > 0) REQUIRE(on_device(a.mp_f, f * a.p * sizeof(float2)) && on_device(a.lo_f, f * a.p * sizeof(float2)));
    if (a.adj) REQUIRE(on_device(a.adj, a.t->n * sizeof(double2)));
}

void launch_zero(void *p, size_t bytes, hipStream_t)
{
    REQUIRE(on_device(p, bytes) && bytes % 8 == 0);
    memset(p, 0, bytes);
}
void launch_widen_perm(const fmm_tree *, int64_t *, int32_t *, hipStream_t) {}
GammaRows launch_stage_in(const fmm_tree *t, const double *gamma, int64_t row, hipStream_t)
{
    if (direct_rows(t->n, row)) return GammaRows{t->d_perm, gamma};
    return GammaRows{t->d_gpos2, t->d_st1};
}
void launch_pack(const fmm_tree *t, const GammaRows &, int is_double, void *gam, hipStream_t)
{
    REQUIRE(on_device(gam, t->n * real_bytes(is_double)));
}
void launch_leaf_coords(const fmm_tree *t, int is_double, void *pos, hipStream_t)
{
    REQUIRE(on_device(pos, t->n * 2 * real_bytes(is_double)));
}
void launch_p2p_forward(const fmm_tree *t, const void *pos, const void *gam, int is_double, double, double2 *near,
                        void *slots, hipStream_t)
{
    REQUIRE(on_device(pos, t->n * 2 * real_bytes(is_double)) && on_device(gam, t->n * real_bytes(is_double)));
    REQUIRE(on_device(near, t->n * sizeof(double2)));
    if (slots) REQUIRE(on_device(slots, 18 * t->n * real_bytes(is_double)));
}
void launch_far_chain(const FarArgs &a, hipStream_t, const FarArgs *b)
{
    check_far(a);
    if (b) {
        REQUIRE(b->adj);
        check_far(*b);
    }
}
void launch_finalize(const fmm_tree *t, const FarArgs &, const double2 *near, const void *, int, double, double *,
                     double *, double *, void *stage, const double *, double, hipStream_t)
{
    REQUIRE(on_device(near, t->n * sizeof(double2)) && on_device(stage, t->n * sizeof(double2)));
}
void launch_adjoint_range(int64_t, const double *, const double *, double, double2 *range, hipStream_t)
{
    REQUIRE(on_device(range, (kRangeBlocks + 1) * sizeof(double2)));
}
void launch_pack_adjoint(const fmm_tree *t, const double *, double, double2 *adj, void *qt, int is_double, double2 *,
                         const double2 *, double *, hipStream_t)
{
    REQUIRE(on_device(adj, t->n * sizeof(double2)));
    if (!is_double) REQUIRE(on_device(qt, t->n * sizeof(float2)));
}
void launch_p2p_force(const fmm_tree *t, const void *, const void *, const void *qv, const double2 *adj,
                      const GammaRows &, int is_double, double, const ForceNear &near, hipStream_t)
{
    REQUIRE(on_device(qv, t->n * 2 * real_bytes(is_double)) && on_device(adj, t->n * sizeof(double2)));
    REQUIRE(on_device(near.near, t->n * sizeof(double2)));
    if (near.slots) REQUIRE(on_device(near.slots, 18 * t->n * real_bytes(is_double)));
    if (near.phi_slots) REQUIRE(on_device(near.phi_slots, 9 * t->n * real_bytes(is_double)));
}
void launch_finalize_force(const fmm_tree *, const FarArgs &c, const FarArgs &q, const double2 *, const ForceNear &,
                           int, double, const AdjointOut &, hipStream_t)
{
    check_far(c);
    check_far(q);
}
void launch_p2p_backward(const fmm_tree *t, const void *, const void *, const void *qv, int is_double, double,
                         double4 *pa, double4 *src, hipStream_t)
{
    REQUIRE(on_device(qv, t->n * 2 * real_bytes(is_double)) && on_device(pa, t->n * sizeof(double4)));
    if (src) REQUIRE(on_device(src, t->n * sizeof(double4)));
}
void launch_finalize_backward(const fmm_tree *, const FarArgs &c, const FarArgs &q, const double4 *, const double2 *,
                              const double4 *, int, double, const AdjointOut &, double *, double *, double *,
                              hipStream_t)
{
    check_far(c);
    check_far(q);
}
hipError_t find_nonfinite(const double *, int64_t, int, int *, hipStream_t, int64_t &bad)
{
    bad = -1;
    return hipSuccess;
}

static void check_atree(const AtreeCall &c, bool adjoint)
{
    const AtreeWs &w = *c.t->wsp;
    const size_t coef = (size_t)c.t->ncells * c.p * sizeof(double2);
    REQUIRE(on_device(w.mp, coef) && on_device(w.lo, coef));
    if (adjoint) REQUIRE(on_device(w.mp2, coef) && on_device(w.lo2, coef) && on_device(w.adj, c.t->n * sizeof(double2)));
}
void launch_atree_pack(const AtreeCall &c, const double *, hipStream_t)
{
    REQUIRE(on_device(c.t->wsp->gam, c.t->n * real_bytes(c.is_double)));
}
void launch_atree_coords(const fmm_atree *t, int is_double, void *pos, hipStream_t)
{
    REQUIRE(on_device(pos, t->n * 2 * real_bytes(is_double)));
}
void launch_atree_far(const AtreeCall &c, hipStream_t, bool both) { check_atree(c, both); }
void launch_atree_pack_adjoint(const AtreeCall &c, const double *, double, hipStream_t)
{
    REQUIRE(on_device(c.t->wsp->qt, c.t->n * 2 * real_bytes(c.is_double)));
}
void launch_atree_force(const AtreeCall &c, const ForceNear &near, hipStream_t)
{
    REQUIRE(on_device(near.slots, 18 * c.t->n * sizeof(double)));
    if (near.phi) REQUIRE(on_device(near.phi_slots, 9 * c.t->n * sizeof(double)));
}
void launch_atree_finalize_force(const AtreeCall &c, const ForceNear &, const AdjointOut &, hipStream_t)
{
    check_atree(c, true);
}
void launch_atree_backward_near(const AtreeCall &c, bool src, hipStream_t)
{
    REQUIRE(c.t->nbwd_units > 0 && on_device(c.t->wsp->pa, c.t->n * sizeof(double4)));
    if (src) REQUIRE(on_device(c.t->wsp->psrc, c.t->n * sizeof(double4)));
}
void launch_atree_finalize_backward(const AtreeCall &c, const AdjointOut &, hipStream_t) { check_atree(c, true); }
void launch_atree_near(const AtreeCall &c, hipStream_t)
{
    REQUIRE(on_device(c.t->wsp->near, c.t->n * sizeof(double2)));
}
void launch_atree_finalize(const AtreeCall &c, double *, double *, double *, const double *, double, hipStream_t)
{
    check_atree(c, false);
}

}  // namespace fmm

// ---------------------------------------------------------------------------------
// The checks
// ---------------------------------------------------------------------------------
namespace {

using namespace fmm;

// Runs f in a child process; whether it ended well.
bool child(const std::function<void()> &f)
{
    fflush(stdout);
    const pid_t pid = fork();
    if (pid == 0) {
        f();
        fflush(stdout);
        _exit(0);
    }
    int status = 0;
    waitpid(pid, &status, 0);
    return WIFEXITED(status) && WEXITSTATUS(status) == 0;
}

std::vector<double> points(int64_t n)
{
    std::vector<double> xy(2 * (size_t)n);
    uint64_t s = 12345;
    for (double &v : xy) {
        s = s * 6364136223846793005ull + 1442695040888963407ull;
        v = (double)(s >> 11) / 9007199254740992.0;
    }
    return xy;
}
const double kUnit[3] = {0.0, 0.0, 1.0};

fmm_tree *uniform_tree(int64_t n, int depth)
{
    const std::vector<double> xy = points(n);
    fmm_tree *t = nullptr;
    REQUIRE(fmm_build_tree_host(xy.data(), n, depth, kUnit, nullptr, &t) == FMM_OK);
    return t;
}
fmm_atree *adaptive_tree(int64_t n)
{
    const std::vector<double> xy = points(n);
    fmm_atree *t = nullptr;
    REQUIRE(fmm_atree_build_host(xy.data(), n, 20, 8, kUnit, nullptr, &t) == FMM_OK);
    return t;
}

// A call out of memory at its k-th allocation fails cleanly: the next one has every array.
void call_memory()
{
    bool bad = false;
    for (int kind = 0; kind < 2; ++kind)
        for (int precision : {FMM_FP64, FMM_MIXED})
            for (int adjoint = 0; adjoint < 2; ++adjoint)
                for (int k = 0; k < 12; ++k)
                    bad |= !child([&] {
                        const int64_t n = 3000;
                        std::vector<double> g(n, 1.0), dl(2 * n, 1.0), dg(n), dx(2 * n), uv(2 * n);
                        auto check = [&](auto t, auto velocity, auto vjp) {
                            auto call = [&](int which) {
                                return which ? vjp(t, g.data(), 0.01, 9, precision, dl.data(), 1.0, 0, nullptr, nullptr,
                                                   dg.data(), dx.data())
                                             : velocity(t, g.data(), 0.01, 9, precision, nullptr, nullptr, uv.data());
                            };
                            if (adjoint) REQUIRE(call(0) == FMM_OK);
                            g_fail_from = g_allocs + k;
                            const int rc = call(adjoint);
                            REQUIRE(rc == FMM_OK || rc == FMM_ENOMEM);
                            g_fail_from = -1;
                            printf("kind %d precision %d adjoint %d allocation %d: ", kind, precision, adjoint, k);
                            REQUIRE(call(adjoint) == FMM_OK && call(!adjoint) == FMM_OK);
                            printf("ok\n");
                        };
                        if (kind == 0) check(uniform_tree(n, 7), fmm_velocity, fmm_transport_vjp);
                        else check(adaptive_tree(n), fmm_atree_velocity, fmm_atree_transport_vjp);
                    });
    REQUIRE(!bad);
}

// After one adjoint call for the position derivative, of either route, and also where memory was
// short of what one of the routes would like to have, every other call of that precision allocates
// nothing and waits for nothing: it can be captured.
void warm_calls()
{
    bool bad = false;
    for (int kind = 0; kind < 2; ++kind)
        for (int precision : {FMM_FP64, FMM_MIXED})
            for (int first = 0; first < 3; ++first)
                for (int k = -1; k < 12; ++k)
                    bad |= !child([&] {
                        const int64_t n = 3000;
                        std::vector<double> g(n, 1.0), dl(2 * n, 1.0), dg(n), dx(2 * n), ds(2 * n), uv(2 * n);
                        auto check = [&](auto t, auto velocity, auto backward, auto vjp) {
                            auto call = [&](int which) {
                                double *const o = nullptr;
                                if (which == 0)
                                    return vjp(t, g.data(), 0.01, 9, precision, dl.data(), 1.0, 0, nullptr, nullptr, o,
                                               dx.data());
                                if (which == 1)
                                    return vjp(t, g.data(), 0.01, 9, precision, dl.data(), 1.0, 0, nullptr, nullptr,
                                               dg.data(), dx.data());
                                if (which == 2)
                                    return backward(t, g.data(), 0.01, 9, precision, dl.data(), nullptr, nullptr,
                                                    dg.data(), dx.data(), ds.data(), o);
                                if (which == 3)
                                    return backward(t, g.data(), 0.01, 9, precision, dl.data(), nullptr, nullptr,
                                                    dg.data(), o, o, o);
                                return velocity(t, g.data(), 0.01, 9, precision, nullptr, nullptr, uv.data());
                            };
                            REQUIRE(call(4) == FMM_OK);
                            if (k >= 0) g_fail_from = g_allocs + k;
                            if (call(first) != FMM_OK) return;  // (memory needed by every route)
                            const int64_t a = g_allocs, f = g_frees, w = g_waits;
                            for (int which = 0; which < 5; ++which) {
                                printf("kind %d precision %d first %d without %d, call %d: ", kind, precision, first, k, which);
                                REQUIRE(call(which) == FMM_OK && g_allocs == a && g_frees == f && g_waits == w);
                                printf("ok\n");
                            }
                        };
                        if (kind == 0)
                            check(uniform_tree(n, 7), fmm_velocity, fmm_velocity_backward, fmm_transport_vjp);
                        else
                            check(adaptive_tree(n), fmm_atree_velocity, fmm_atree_velocity_backward,
                                  fmm_atree_transport_vjp);
                    });
    REQUIRE(!bad);
}

// What stays reserved after trees are destroyed is bounded, whatever they were and in any order.
void held_memory()
{
    const size_t MiB = size_t(1) << 20;
    for (const std::vector<int> &sizes : {std::vector<int>{3000}, {-3000}, {900, -900}, {-900, 900}, {700, -700, 700, -200},
                                          {500, 500, -500, 500}})
        REQUIRE(child([&] {
            const double xy[2] = {0.5, 0.5};
            for (int pass = 0; pass < 2; ++pass)
                for (int size : sizes) {
                    fmm::g_tree_bytes = (size_t)std::abs(size) * MiB;
                    fmm_tree *t = nullptr;
                    fmm_atree *a = nullptr;
                    if (size > 0) REQUIRE(fmm_build_tree(xy, 1, 4, kUnit, nullptr, &t) == FMM_OK);
                    else REQUIRE(fmm_atree_build(xy, 1, 4, 4, kUnit, nullptr, &a) == FMM_OK);
                    fmm_destroy_tree(t);
                    fmm_atree_destroy(a);
                    printf("after %d MiB: %zu MiB held, %zu in the pool\n", size, (g_used + g_pool_idle) / MiB,
                           g_pool_idle / MiB);
                    REQUIRE(g_used + g_pool_idle <= fmm::kIdleBytes + 64 * MiB);  // (and the caller's tables)
                }
        }));
}

// Where memory is short, what the library holds idle goes back before a call fails.
void idle_released()
{
    const size_t MiB = size_t(1) << 20;
    bool bad = false;
    for (int pool = 0; pool < 2; ++pool)
        for (int what = 0; what < 5; ++what)
            bad |= !child([&] {
                const double one[2] = {0.5, 0.5};
                const int64_t n = 100000;
                std::vector<double> g(n, 1.0), uv(2 * n);
                fmm_tree *kept = uniform_tree(n, 6), *t = nullptr;
                REQUIRE(fmm_velocity(kept, g.data(), 0.01, 9, FMM_MIXED, nullptr, nullptr, uv.data()) == FMM_OK);
                fmm::g_tree_bytes = 600 * MiB;
                fmm_atree *a = nullptr;
                if (pool) REQUIRE(fmm_build_tree(one, 1, 4, kUnit, nullptr, &t) == FMM_OK);
                else REQUIRE(fmm_atree_build(one, 1, 4, 4, kUnit, nullptr, &a) == FMM_OK);
                fmm_destroy_tree(t);
                fmm_atree_destroy(a);
                REQUIRE(g_pool_idle > 0 || !pool);
                // room for the trees' small arrays only
                g_capacity = g_used + g_pool_idle;
                printf("idle in the %s, allocation %d: ", pool ? "pool" : "cache", what);
                int rc = FMM_OK;
                if (what == 0) rc = fmm_velocity(kept, g.data(), 0.01, 31, FMM_MIXED, nullptr, nullptr, uv.data());  // tables
                if (what == 1) rc = fmm_velocity(kept, g.data(), 0.01, 9, FMM_FP64, nullptr, nullptr, uv.data());
                if (what == 2) uniform_tree(n, 5);
                if (what == 3) rc = fmm_set_option(kept, FMM_OPT_VALIDATE, 1) != FMM_OK ? FMM_EINVAL
                                    : fmm_velocity(kept, g.data(), 0.01, 9, FMM_MIXED, nullptr, nullptr, uv.data());
                fmm::g_tree_bytes = 100 * MiB;
                if (what == 4) rc = pool ? fmm_atree_build(one, 1, 4, 4, kUnit, nullptr, &a)
                                         : fmm_build_tree(one, 1, 4, kUnit, nullptr, &t);
                REQUIRE(rc == FMM_OK);
                printf("ok\n");
            });
    REQUIRE(!bad);
}

// Without host memory the cache hands out nothing or a block, gives back what it is given and
// throws nothing (it is called from destructors and behind the C interface).
void host_memory()
{
    bool bad = false;
    for (int k = 0; k < 12; ++k)
        bad |= !child([&] {
            const size_t MiB = size_t(1) << 20;
            std::vector<void *> kept, got(8, nullptr);
            for (int j = 0; j < 6; ++j) {
                void *p = nullptr;
                REQUIRE(fmm::block_alloc(&p, (200 + j) * MiB) == hipSuccess);
                kept.push_back(p);
            }
            fmm::SideStream side;
            REQUIRE(fmm::side_stream_take(0, side) == hipSuccess);
            fmm::BuildScope *scope = new fmm::BuildScope(nullptr);
            void *step = nullptr;
            REQUIRE(fmm::build_alloc(&step, MiB, nullptr) == hipSuccess);
            g_new_left = k;
            fmm::side_stream_give(0, side);
            fmm::build_free(step, MiB, nullptr);
            for (void *p : kept) fmm::block_free(p);
            for (size_t j = 0; j < got.size(); ++j)
                REQUIRE((fmm::block_alloc(&got[j], (300 + j) * MiB) == hipSuccess) == (got[j] != nullptr));
            for (void *p : got) fmm::block_free(p);
            g_new_left = -1;
            delete scope;
            printf("allocation %d: %zu MiB held\n", k, g_used / MiB);
            REQUIRE(g_used <= fmm::kIdleBytes);
        });
    REQUIRE(!bad);
}

// The host builds order their work by the device builds' key (cost_order), ties in the order of
// the leaves.
void work_order()
{
    std::vector<double> xy = points(9000);
    for (size_t k = 0; k < 4000; ++k) xy[k] = 0.3 + 0.05 * xy[k];
    fmm_tree *t = nullptr;
    REQUIRE(fmm_build_tree_host(xy.data(), 9000, 5, kUnit, nullptr, &t) == FMM_OK);
    std::vector<std::pair<uint64_t, int>> keys;
    for (int64_t k = 0; k < t->nunits; ++k) {
        const int4 u = t->d_units[k];
        int64_t nsrc = 0;
        const int x = (int)morton_x((uint32_t)u.x), y = (int)morton_y((uint32_t)u.x);
        for (int dy = -1; dy <= 1; ++dy)
            for (int dx = -1; dx <= 1; ++dx)
                if (x + dx >= 0 && y + dy >= 0 && x + dx < 32 && y + dy < 32) {
                    const uint32_t c = morton_encode((uint32_t)(x + dx), (uint32_t)(y + dy));
                    nsrc += t->d_leaf_start[c + 1] - t->d_leaf_start[c];
                }
        const int64_t stride = 64 >> u.w;
        keys.emplace_back(cost_order((uint64_t)((nsrc + stride - 1) / stride)), u.y);
    }
    REQUIRE(std::is_sorted(keys.begin(), keys.end()) && keys.front().first < keys.back().first);

    fmm_atree *a = nullptr;
    REQUIRE(fmm_atree_build_host(xy.data(), 9000, 60, 8, kUnit, nullptr, &a) == FMM_OK);
    uint64_t last = 0;
    int units = 0, items = 0;
    for (int64_t k = 0; k < a->nwork; ++k) {
        const int4 u = a->d.work[k];
        int64_t cost = 0;
        if (u.w & kMutualItem) {
            ++items;
            const int64_t s = a->d.leaf_start[u.x + 1] - a->d.leaf_start[u.x];
            const int64_t r = a->d.leaf_start[u.y + 1] - a->d.leaf_start[u.y];
            cost = u.x == u.y ? at_self_cost(s) : 3 * at_pair_steps(s, r);
        } else {
            ++units;
            const int4 c = a->d.cell[u.x];
            int64_t nsrc = 0;
            for (int e = a->d.u_off[u.x]; e < a->d.u_off[u.x + 1]; ++e) {
                const int S = a->d.u_idx[e];
                if (!((u.w >> 4) && a->d.cell[S].x == c.x && a->d.range[S].y >= a->dense_leaf)) nsrc += a->d.range[S].y;
            }
            cost = at_unit_cost(nsrc, u.z);
        }
        REQUIRE(cost_order((uint64_t)cost) >= last);
        last = cost_order((uint64_t)cost);
    }
    REQUIRE(units > 0 && items > 0);
}

// Trees that take turns with one workspace: a call clears what the other tree left in the multipoles,
// with a kernel (a call may be captured, and a memset is not to become a node of a graph).
void shared_workspace()
{
    for (int precision : {FMM_FP64, FMM_MIXED}) {
        const int64_t n = 3000;
        std::vector<double> g(n, 1.0), dl(2 * n, 1.0), dx(2 * n), uv(2 * n);
        fmm_tree *t[2] = {uniform_tree(n, 7), uniform_tree(n, 7)};
        REQUIRE(fmm_share_workspace(t[1], t[0]) == FMM_OK);
        auto calls = [&](fmm_tree *tree) {
            REQUIRE(fmm_velocity(tree, g.data(), 0.01, 9, precision, nullptr, nullptr, uv.data()) == FMM_OK);
            REQUIRE(fmm_transport_vjp(tree, g.data(), 0.01, 9, precision, dl.data(), 1.0, 0, nullptr, nullptr, nullptr,
                                      dx.data()) == FMM_OK);
        };
        for (fmm_tree *tree : t) calls(tree);
        const int64_t a = g_allocs, w = g_waits, m = g_memsets;
        Workspace &ws = *t[0]->wsp;
        for (int k = 0; k < 4; ++k) {
            auto *left = (double *)(precision == FMM_FP64 ? (void *)ws.mp_d : (void *)ws.mp_f);
            left[100] = 1.0;  // (a cell that the next tree leaves empty)
            ws.mp2_d[50].x = 1.0;
            calls(t[k % 2]);
            REQUIRE(left[100] == 0.0 && ws.mp2_d[50].x == 0.0);
            REQUIRE(g_allocs == a && g_waits == w && g_memsets == m);
        }
    }
}

}  // namespace

int main(int argc, char **argv)
{
    const std::map<std::string, void (*)()> checks = {{"call_memory", call_memory}, {"warm_calls", warm_calls}, {"held_memory", held_memory},
                                                              {"idle_released", idle_released},
                                                              {"host_memory", host_memory},
                                                              {"work_order", work_order},
                                                              {"shared_workspace", shared_workspace}};
    const auto it = checks.find(argc > 1 ? argv[1] : "");
    REQUIRE(it != checks.end());
    REQUIRE(child(it->second));
    printf("%s passed\n", argv[1]);
    return 0;
}
