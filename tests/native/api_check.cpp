// api_check.cpp -- the host side of the C-ABI (paper_1604_01829_amd/csrc/lbrb_api.cpp) on a HIP
// runtime of this file's own: memory is host memory, a launch is an entry of a list, advances a
// clock that the events read and can be made to fail.  Built and run by tests/test_host_calls.py:
//
//   api_check tune      the autotuner times what a step does: the moving-wall links too
//   api_check replay    a launch that fails in the reverse pass's replays is reported
//   api_check observe   lb_observables allocates nothing
//
// Exits 0 when every check holds; prints the first failure.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/lbrb.h"
#include "../../paper_1604_01829_amd/csrc/lbrb_analysis.h"
#include "../../paper_1604_01829_amd/csrc/lbrb_layout.h"
#include "../../paper_1604_01829_amd/csrc/lbrb_walls.h"

using namespace lbrb;

#define CHECK(cond)                                                            \
    do {                                                                       \
        if (!(cond)) {                                                         \
            std::fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                      \
        }                                                                      \
    } while (0)

// ------------------------------------------------------------------ the runtime

static hipError_t g_last = hipSuccess;
static double g_clock = 0.0;                    // us
static std::vector<std::string> g_launches;
static std::string g_fail;                      // the launch of this name that fails ...
static int g_fail_after = -1;                   // ... after so many of that name
static int g_allocations = 0;
static bool g_no_memory = false;

static void launched(const char* name, double us)
{
    g_launches.push_back(name);
    g_clock += us;
    if (g_fail == name && g_fail_after-- == 0) g_last = hipErrorLaunchFailure;
}

extern "C" {
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError()
{
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
hipError_t hipPeekAtLastError() { return g_last; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int)
{
    std::memset(p, 0, sizeof *p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memmove(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memmove(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    ++g_allocations;
    if (g_no_memory) return hipErrorOutOfMemory;
    *p = std::malloc(n);
    return hipSuccess;
}
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t*, unsigned) { return hipErrorNotSupported; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t*) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t*, hipGraph_t, hipGraphNode_t*, char*, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t) new double(0.0); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete (double*)e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { *(double*)e = g_clock; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(1e-3 * (*(double*)b - *(double*)a));
    return hipSuccess;
}
int roctxRangePushA(const char*) { return 0; }
int roctxRangePop() { return 0; }
}

// ------------------------------------------------------------------ the launches

namespace lbrb {
void noalloc_prepare() {}
template <typename Real>
void launch_couple(const StepArgs<Real>&, const CoupleArgs&, hipStream_t, const LaunchEvents&, const BodyArgs*)
{
    launched("couple", 5.0);
}
// 100 us, 5 % less with workgroups of several tiles
template <typename Real>
void launch_node_step(const StepArgs<Real>& a, bool, bool, const BodyArgs*, hipStream_t, const LaunchEvents&)
{
    launched("node", a.tiles_per_wg == 1 ? 100.0 : 95.0);
}
template <typename Real>
void launch_wall_links(Real*, const WallLink*, int64_t, hipStream_t) { launched("links", 20.0); }
template <typename Real>
void launch_init_equilibrium(Real*, int64_t, const ReplicaDesc*, const NodeTile*, int32_t, Real, const double*, hipStream_t) {}
template <typename Real>
void launch_observe(const StepArgs<Real>&, bool, int32_t, int32_t, int32_t, int64_t, Real*, double*, double*, hipStream_t)
{
    launched("observe", 5.0);
}
void launch_observe_out(const double*, int, const DeviceHeader*, const Body*, int n_bodies, int, const ObserveOut& out,
                        hipStream_t)
{
    launched("observe_out", 5.0);
    for (int k = 0; k < 6; ++k) out.totals[k] = 0.0;
    for (int k = 0; k < n_bodies * kObserveBodyWords; ++k) out.bodies[k] = k;
}
template <typename Real>
void launch_mirror_holes(Real*, const ReplicaDesc*, const RowDesc*, const RowDesc*, const NodeTile*, int32_t,
                         const uint8_t*, hipStream_t)
{
    launched("mirror", 5.0);
}
template <typename Real>
void launch_mirror_holes_transposed(Real*, const ReplicaDesc*, const RowDesc*, const RowDesc*, const NodeTile*, int32_t,
                                    const uint8_t*, hipStream_t)
{
    launched("mirror", 5.0);
}
template <typename Real>
void launch_adjoint_step(const AdjArgs<Real>&, bool, hipStream_t) { launched("adjoint", 5.0); }
template <typename Real>
void launch_adjoint_beads(const AdjArgs<Real>&, hipStream_t) { launched("adjoint_beads", 5.0); }
template <typename Real>
void launch_couple_adj_bead(const StepArgs<Real>&, const CoupleArgs&, const AdjArgs<Real>&, hipStream_t)
{
    launched("couple_adj_bead", 5.0);
}
void launch_body_predict(const BodyArgs&, int, hipStream_t) { launched("predict", 5.0); }
void launch_body_substep(const BodyArgs&, const int64_t*, int64_t, int, hipStream_t) { launched("substep", 5.0); }
void launch_set_step(int64_t* p, int64_t v, hipStream_t) { *p = v; }
void launch_record_poses(const Body*, int, double*, hipStream_t) {}
void launch_adjoint_body_post(const Body*, const Body*, int, const double*, const double*, double*, double*, double*, int,
                              hipStream_t) { launched("body_post", 5.0); }
void launch_adjoint_wca(const BodyArgs&, int, const double*, const double*, double*, int, hipStream_t) {}
void launch_records_from_poses(const Body*, int, const Bead*, BeadRec*, int, hipStream_t) { launched("records", 5.0); }

#define INSTANTIATE(R)                                                                                                 \
    template void launch_couple<R>(const StepArgs<R>&, const CoupleArgs&, hipStream_t, const LaunchEvents&, const BodyArgs*); \
    template void launch_node_step<R>(const StepArgs<R>&, bool, bool, const BodyArgs*, hipStream_t, const LaunchEvents&); \
    template void launch_wall_links<R>(R*, const WallLink*, int64_t, hipStream_t);                                     \
    template void launch_init_equilibrium<R>(R*, int64_t, const ReplicaDesc*, const NodeTile*, int32_t, R, const double*, \
                                             hipStream_t);                                                             \
    template void launch_observe<R>(const StepArgs<R>&, bool, int32_t, int32_t, int32_t, int64_t, R*, double*, double*, \
                                    hipStream_t);                                                                      \
    template void launch_mirror_holes<R>(R*, const ReplicaDesc*, const RowDesc*, const RowDesc*, const NodeTile*, int32_t, \
                                         const uint8_t*, hipStream_t);                                                 \
    template void launch_mirror_holes_transposed<R>(R*, const ReplicaDesc*, const RowDesc*, const RowDesc*,            \
                                                    const NodeTile*, int32_t, const uint8_t*, hipStream_t);            \
    template void launch_adjoint_step<R>(const AdjArgs<R>&, bool, hipStream_t);                                        \
    template void launch_adjoint_beads<R>(const AdjArgs<R>&, hipStream_t);                                             \
    template void launch_couple_adj_bead<R>(const StepArgs<R>&, const CoupleArgs&, const AdjArgs<R>&, hipStream_t);
INSTANTIATE(float)
INSTANTIATE(double)
}  // namespace lbrb

// ------------------------------------------------------------------ a channel

constexpr int kSide = 12;

// 12^3 nodes, walls 1 and 2 on the y faces, the second moving or not; `bodies` bodies of 2 beads
struct Channel {
    lb_params p{};
    lb_replica rep{kSide, kSide, kSide, 5};
    void* ws = nullptr;
    lb_ctx* c = nullptr;

    Channel(bool moving, int bodies, bool fixed = true)
    {
        p.precision = LB_PRECISION_F64;
        p.rho0 = p.tau_shear = p.tau_bulk = p.tau_odd = p.tau_even = 1.0;
        p.max_bodies = 4;
        p.max_beads = 8;
        p.max_wall_links = 18 * kSide * kSide;
        const size_t bytes = lb_workspace_bytes(&p, &rep, 1);
        CHECK(bytes > 0);
        ws = std::aligned_alloc(256, bytes);
        if (lb_init(&p, &rep, 1, ws, bytes, nullptr, &c) != LB_OK) return;
        std::vector<uint8_t> mask((size_t)kSide * kSide * kSide, 0);
        for (int z = 0; z < kSide; ++z)
            for (int x = 0; x < kSide; ++x) {
                mask[x + (size_t)kSide * kSide * z] = 1;
                mask[x + (size_t)kSide * (kSide - 1 + (size_t)kSide * z)] = 2;
            }
        CHECK(lb_set_boundary_mask(c, 0, mask.data()) == LB_OK);
        const double u[3] = {moving ? 0.01 : 0.0, 0.0, 0.0};
        CHECK(lb_set_wall_velocity(c, 0, 2, u) == LB_OK);
        for (int b = 0; b < bodies; ++b) add(fixed);
    }
    void add(bool fixed)
    {
        const double off[6] = {0, 0, 0, 1, 0, 0}, in[3] = {1, 1, 1}, pos[3] = {6, 6, 6}, q[4] = {1, 0, 0, 0},
                     zero[3] = {0, 0, 0};
        int32_t id = -1;
        CHECK(rb_add_raspberry(c, 0, off, 2, 1.0, in, pos, q, zero, zero, 1.0, fixed ? 1 : 0, &id) == LB_OK);
    }
    ~Channel()
    {
        lb_destroy(c);
        std::free(ws);
    }
};

static int tiles_per_wg(lb_ctx* c)
{
    lb_tuning t{};
    CHECK(lb_get_tuning(c, &t) == LB_OK);
    return t.tiles_per_wg;
}

// Walls at rest: the wide workgroups are 5 % faster and taken.  Moving walls: they leave the links
// to a launch of 20 us in every step, so one tile per workgroup is.  A context of the same sizes
// without moving walls, timed first, does not decide for it.
static void tune()
{
    for (int first_at_rest = 0; first_at_rest < 2; ++first_at_rest) {
        Channel rest(false, 0), moving(true, 0);
        if (first_at_rest) {
            CHECK(lb_autotune(rest.c, 2) == LB_OK);
            CHECK(tiles_per_wg(rest.c) == 4);
        }
        CHECK(lb_autotune(moving.c, first_at_rest ? 0 : 2) == LB_OK);
        CHECK(tiles_per_wg(moving.c) == 1);
        CHECK(lb_autotune(rest.c, 0) == LB_OK);
        CHECK(tiles_per_wg(rest.c) == 4);
    }
}

static int adjoint(Channel& h, int steps, int every)
{
    const size_t bytes = lb_adjoint_workspace_bytes(h.c, steps, every);
    CHECK(bytes > 0);
    void* ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    std::vector<double> w(3 * 4 * (size_t)steps, 0.0), dg(4), dr(3 * 8);
    double J = 0.0;
    const int rc = lb_rb_adjoint(h.c, steps, every, ws, bytes, w.data(), &J, dg.data(), dr.data());
    std::free(ws);
    return rc;
}

// Steps 0 ... 3, one segment: 4 forward launches of each kind, then 3 in the replays.  The failing
// launch is one of the replays, with wide workgroups, moving walls or both.
static void replay()
{
    for (int moving = 0; moving < 2; ++moving)
        for (int wide = 0; wide < 2; ++wide)
            for (int fixed = 0; fixed < 2; ++fixed)
                for (const char* name : {"", "node", "couple", "links"}) {
                    const bool links = moving && wide;
                    if (!std::strcmp(name, "links") && !links) continue;
                    Channel h(moving != 0, 1, fixed != 0);
                    lb_tuning t{};
                    t.tiles_per_wg = wide ? 4 : 1;
                    CHECK(lb_set_tuning(h.c, &t) == LB_OK);
                    g_launches.clear();
                    g_fail = name;
                    g_fail_after = 5;
                    const int rc = adjoint(h, 4, 4);
                    g_fail.clear();
                    std::printf("moving %d wide %d fixed %d failing '%s': %d\n", moving, wide, fixed, name, rc);
                    CHECK(rc == (*name ? LB_ERR_HIP : LB_OK));
                    if (links && !*name) {
                        int n = 0;
                        for (const std::string& s : g_launches) n += s == "links";
                        CHECK(n == 4 + 3);
                    }
                }
}

static void observe()
{
    Channel h(false, 1);
    CHECK(h.c != nullptr);
    const int before = g_allocations;
    lb_totals tot{};
    rb_state s[4];
    CHECK(lb_observables(h.c, 0, &tot, s, nullptr) == LB_OK);
    for (int b = 1; b < 4; ++b) h.add(true);
    CHECK(lb_observables(h.c, 0, &tot, s, nullptr) == LB_OK);
    CHECK(s[3].pos[0] == 3.0 * kObserveBodyWords);
    CHECK(g_allocations == before);
    g_no_memory = true;
    Channel none(false, 0);
    CHECK(none.c == nullptr);   // refused when the context is made
    g_no_memory = false;
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "tune") tune();
    else if (what == "replay") replay();
    else if (what == "observe") observe();
    else return 2;
    std::printf("%s ok\n", what.c_str());
    return 0;
}
