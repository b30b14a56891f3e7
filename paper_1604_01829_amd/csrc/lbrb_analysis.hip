// lbrb_analysis.hip -- trajectory analysis on the device (the C-ABI functions lb_traj_*
// and the pose recorder behind rb_record_poses).
//
// A trajectory is traj[frame][body][7]: centre (x, y, z; lab frame, unwrapped) and unit
// quaternion (w, x, y, z) of every body at every recording.  The analysis follows Sec. 2.4-2.8
// of the paper: the lab-frame MSD of the centre (eq. (dt_lab)), the lab-frame MSD of the angle
// of a reference vector (eqs. (dr_lab), (delta_theta)), body-frame displacements (each
// recording interval's lab displacement turned into the body frame with the orientation at the
// start of the interval, then summed, Sec. 2.6), body-frame rotation angles by projecting the
// body axes at t onto the planes normal to the axes at t - 1 (Sec. 2.7), and pore-frame
// displacements (the interval's displacement rotated by minus the polar angle of the centre
// about the pore axis at the start of the interval, then summed, Sec. 2.8) with MSDs binned
// by the radial position of each origin frame.
//
// Series are stored body-major, series[body][frame][k], so the MSD kernels read contiguous
// frames.  Every sum runs in a fixed order (thread-strided loops, shuffle + LDS trees) and does
// not depend on timing, but for the last bits of the sums of more than two bodies in at most 8 bins.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "../../include/lbrb.h"
#include "lbrb_analysis.h"

namespace lbrb {
namespace {

constexpr int kBlock = 256;

// rotation matrix (body -> lab) of a unit quaternion, row-major
__device__ __forceinline__ void rot_of(const double* q, double R[9])
{
    const double w = q[0], x = q[1], y = q[2], z = q[3];
    R[0] = 1.0 - 2.0 * (y * y + z * z); R[1] = 2.0 * (x * y - z * w); R[2] = 2.0 * (x * z + y * w);
    R[3] = 2.0 * (x * y + z * w); R[4] = 1.0 - 2.0 * (x * x + z * z); R[5] = 2.0 * (y * z - x * w);
    R[6] = 2.0 * (x * z - y * w); R[7] = 2.0 * (y * z + x * w); R[8] = 1.0 - 2.0 * (x * x + y * y);
}

// sum over the workgroup of v[0..K), fixed order; the result is valid in thread 0
template <int K>
__device__ __forceinline__ void block_sum(double v[K], double (*part)[K])
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1)
        for (int k = 0; k < K; ++k) v[k] += __shfl_down(v[k], m, 64);
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0)
        for (int k = 0; k < K; ++k) part[wave][k] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int k = 0; k < K; ++k) v[k] = (part[0][k] + part[1][k]) + (part[2][k] + part[3][k]);
}

// ------------------------------------------------------------------ poses

__global__ void record_kernel(const Body* bodies, int n_bodies, double* frame)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= n_bodies) return;
    const Body& B = bodies[b];
    for (int a = 0; a < 3; ++a) frame[7 * (int64_t)b + a] = B.pos[a];
    for (int a = 0; a < 4; ++a) frame[7 * (int64_t)b + 3 + a] = B.quat[a];
}

// ------------------------------------------------------------------ cumulative series

// the lab-frame displacement: every frame's centre minus the first (no sum: one thread per
// frame and body, lanes along the frames so that the series is written in order)
__global__ __launch_bounds__(kBlock) void lab_kernel(const double* __restrict__ traj, int n_frames,
                                                     int n_bodies, int body0, double* __restrict__ out)
{
    const int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int b = body0 + blockIdx.y;
    if (f >= n_frames) return;
    const double* p0 = traj + 7 * (int64_t)b;
    const double* p1 = traj + 7 * (f * n_bodies + b);
    double* o = out + 3 * ((int64_t)b * n_frames + f);
    for (int a = 0; a < 3; ++a) o[a] = p1[a] - p0[a];
}

// per-interval increments of one body between frames n-1 and n
struct BodyStep {
    static constexpr int K = 6;
    // displacement in the body frame at the interval start, and the projection angles
    __device__ static void delta(const double* p0, const double* p1, double, double, double d[K])
    {
        double A[9], Rn[9];
        rot_of(p0 + 3, A);      // columns: body axes at t-1
        rot_of(p1 + 3, Rn);     // columns: body axes at t
        const double dx[3] = {p1[0] - p0[0], p1[1] - p0[1], p1[2] - p0[2]};
        for (int a = 0; a < 3; ++a) d[a] = A[a] * dx[0] + A[3 + a] * dx[1] + A[6 + a] * dx[2];
        // axis u of t, minus its component along axis e of t-1, expressed in the t-1 frame
        auto proj = [&](int u, int e, double out[3]) {
            const double v[3] = {Rn[u], Rn[3 + u], Rn[6 + u]};
            const double ee[3] = {A[e], A[3 + e], A[6 + e]};
            const double s = v[0] * ee[0] + v[1] * ee[1] + v[2] * ee[2];
            const double p[3] = {v[0] - ee[0] * s, v[1] - ee[1] * s, v[2] - ee[2] * s};
            for (int r = 0; r < 3; ++r) out[r] = A[r] * p[0] + A[3 + r] * p[1] + A[6 + r] * p[2];
        };
        double k2[3], i2[3], j2[3];
        proj(2, 0, k2);     // z axis onto the plane normal to x
        proj(0, 1, i2);     // x axis onto the plane normal to y
        proj(1, 2, j2);     // y axis onto the plane normal to z
        d[3] = atan(k2[1] / k2[2]);
        d[4] = atan(i2[2] / i2[0]);
        d[5] = atan(j2[0] / j2[1]);
    }
};

struct PoreStep {
    static constexpr int K = 3;
    // displacement rotated by minus the polar angle about the axis (cx, cy) at the start
    __device__ static void delta(const double* p0, const double* p1, double cx, double cy,
                                 double d[K])
    {
        const double th = atan2(p0[1] - cy, p0[0] - cx);
        const double c = cos(th), s = sin(th);
        const double dx = p1[0] - p0[0], dy = p1[1] - p0[1];
        d[0] = c * dx + s * dy;
        d[1] = -s * dx + c * dy;
        d[2] = p1[2] - p0[2];
    }
};

// The F - 1 interval increments are cut into segments of kSpan, a workgroup each: a thread takes
// kPer consecutive intervals, a scan over the workgroup (shuffles, then the waves' totals in LDS)
// gives the sum before them, and the thread writes the segment's running sums.  Then one
// workgroup per body turns the sums at the segments' ends into totals, and every other value adds
// the total before its segment.  The sums run in a fixed order.  out[body][frame][K], 0 at frame 0.
// Bound by the scattered poses (56 of every 56 n_bodies bytes): a segment's are staged in LDS,
// lanes along the words of a pose.  With one workgroup per body, a serial chunk of the trajectory
// per thread and each pose waited for in turn, the body-frame series of 32 bodies and 20,000
// frames took 347 us, this 25 us (three launches); the pore frame 303 and 18 us.
constexpr int kPer = 2;
constexpr int kSpan = kBlock * kPer;

// inclusive sums over the workgroup's threads of v[0..K); returns the workgroup's total in `all`
template <int K>
__device__ __forceinline__ void block_scan(double v[K], double (*part)[K], double all[K])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int x = 1; x < 64; x <<= 1)
        for (int k = 0; k < K; ++k) {
            const double u = __shfl_up(v[k], x, 64);
            if (lane >= x) v[k] += u;
        }
    if (lane == 63)
        for (int k = 0; k < K; ++k) part[wave][k] = v[k];
    __syncthreads();
    for (int k = 0; k < K; ++k) {
        double run = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) {
            if (w == wave) v[k] += run;
            run += part[w][k];
        }
        all[k] = run;
    }
}

template <class Step>
__global__ __launch_bounds__(kBlock) void cumulate_kernel(const double* __restrict__ traj,
                                                          int n_frames, int n_bodies, int n_seg,
                                                          double cx, double cy,
                                                          double* __restrict__ out,
                                                          double* __restrict__ radial)
{
    constexpr int K = Step::K;
    constexpr int group = 7 * kPer + 1;       // one pad word per thread's frames
    __shared__ double pose[group * kBlock + 7];
    __shared__ double part[kBlock / 64][K];
    const int b = blockIdx.x / n_seg;
    const int64_t n0 = (int64_t)kSpan * (blockIdx.x % n_seg);
    for (int e = threadIdx.x; e < 7 * (kSpan + 1); e += kBlock) {
        // frames n0 ... n0 + kSpan; past the end the last frame stands still
        const int64_t f = n0 + e / 7 < n_frames ? n0 + e / 7 : n_frames - 1;
        pose[e + e / (7 * kPer)] = traj[7 * (f * n_bodies + b) + e % 7];
    }
    __syncthreads();
    auto word = [&](int q, int c) { return pose[group * (threadIdx.x + q / kPer) + 7 * (q % kPer) + c]; };
    const int64_t n = n0 + kPer * (int64_t)threadIdx.x;
    double* ob = out + (int64_t)b * n_frames * K;
    double p[kPer + 1][7], d[kPer][K], sum[K], all[K];
#pragma unroll
    for (int q = 0; q <= kPer; ++q)
        for (int c = 0; c < 7; ++c) p[q][c] = word(q, c);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        Step::delta(p[q], p[q + 1], cx, cy, d[q]);
        for (int k = 0; k < K; ++k)
            d[q][k] = (n + q + 1 < n_frames ? d[q][k] : 0.0) + (q > 0 ? d[q > 0 ? q - 1 : 0][k] : 0.0);
    }
    for (int k = 0; k < K; ++k) sum[k] = d[kPer - 1][k];
    block_scan<K>(sum, part, all);
    // the sum before the thread's intervals: its neighbour's inclusive sum
    __syncthreads();
    double* incl = pose;
    for (int k = 0; k < K; ++k) incl[(threadIdx.x + 1) * K + k] = sum[k];
    if (threadIdx.x == 0)
        for (int k = 0; k < K; ++k) incl[k] = 0.0;
    __syncthreads();
    if (n == 0)
        for (int k = 0; k < K; ++k) ob[k] = 0.0;
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (n + q + 1 < n_frames)
            for (int k = 0; k < K; ++k) ob[(n + q + 1) * K + k] = incl[threadIdx.x * K + k] + d[q][k];
    if (radial)
#pragma unroll
        for (int q = 0; q <= kPer; ++q) {     // each thread's frames, and the last frame of all
            const int64_t f = n + q;
            if (f < n_frames && (q < kPer || f == n_frames - 1))
                radial[(int64_t)b * n_frames + f] = hypot(p[q][0] - cx, p[q][1] - cy);
        }
}

// the running totals at the segments' ends (frames kSpan, 2 kSpan, ...), one workgroup per body
template <int K>
__global__ __launch_bounds__(kBlock) void segment_totals_kernel(double* __restrict__ out, int n_frames,
                                                                int n_seg)
{
    __shared__ double part[2][kBlock / 64][K];
    double* ob = out + (int64_t)blockIdx.x * n_frames * K;
    double carry[K];
    for (int k = 0; k < K; ++k) carry[k] = 0.0;
    int par = 0;
    for (int g0 = 0; g0 < n_seg - 1; g0 += kBlock, par ^= 1) {
        const int g = g0 + threadIdx.x;       // the last segment's end has nothing after it
        double* end = ob + (int64_t)kSpan * (g + 1) * K;
        double v[K], all[K];
        for (int k = 0; k < K; ++k) v[k] = g < n_seg - 1 ? end[k] : 0.0;
        block_scan<K>(v, part[par], all);
        for (int k = 0; k < K; ++k) {
            if (g < n_seg - 1) end[k] = carry[k] + v[k];
            carry[k] += all[k];
        }
    }
}

// every value of segments 1 ... but the ends: plus the total before its segment
template <int K>
__global__ __launch_bounds__(kBlock) void add_before_kernel(double* __restrict__ out, int n_frames,
                                                            int n_seg)
{
    const int b = blockIdx.x / (n_seg - 1), g = 1 + blockIdx.x % (n_seg - 1);
    double* ob = out + (int64_t)b * n_frames * K;
    const double* before = ob + (int64_t)kSpan * g * K;   // frame kSpan g
    const int64_t first = (int64_t)kSpan * g + 1;
    const int64_t last = g == n_seg - 1 ? n_frames : first + kSpan - 1;   // the end itself excluded
    for (int64_t e = first * K + threadIdx.x; e < last * K; e += kBlock) ob[e] += before[e % K];
}

// ------------------------------------------------------------------ MSDs

// Short trajectories: one workgroup per block of kLagBlock consecutive lags and per body.  The
// origins are staged kChunk at a time in LDS together with the frames the block's lags reach from
// them.  Thread (l, ph) accumulates lag lag0 + l + 1 over the origins t = ph mod 4 in increasing
// order; the four phases are then added in a fixed order.  Every term reads its values from LDS,
// but a workgroup starts and ends in 4 us, where the tiles below take 10 us however few frames
// there are, and takes every component at once.
constexpr int kLagBlock = 64;
constexpr int kChunk = 256;
constexpr int kPhases = kBlock / kLagBlock;
static_assert(kPhases == 4, "four origin phases per lag");
struct ShortMsd { static constexpr int lags = kLagBlock; };

// stage frames f0 .. f0 + n - 1 of a body-major series (K values per frame) into T; frames
// at or beyond n_frames read as zero
template <int K>
__device__ __forceinline__ void stage(const double* __restrict__ sb, int64_t f0, int n,
                                      int n_frames, double (*T)[K])
{
    for (int e = threadIdx.x; e < n * K; e += kBlock) {
        const int64_t f = f0 + e / K;
        T[e / K][e % K] = f < n_frames ? sb[f * K + e % K] : 0.0;
    }
}

// grid (lag block, body): mean over origins of the squared increment of each component
template <int K>
__global__ __launch_bounds__(kBlock) void short_msd_kernel(const double* __restrict__ s,
                                                           int n_frames, int n_lags,
                                                           double* __restrict__ out)
{
    __shared__ double A[kChunk][K];                       // origins t0 ..
    __shared__ double Bt[kChunk + kLagBlock - 1][K];      // frames t0 + lag0 + 1 ..
    __shared__ double part[kPhases][kLagBlock][K];
    const int lag0 = blockIdx.x * kLagBlock, b = blockIdx.y;
    const int l = threadIdx.x % kLagBlock, ph = threadIdx.x / kLagBlock;
    const int tau = lag0 + l + 1;
    const double* sb = s + (int64_t)b * n_frames * K;
    double acc[K];
    for (int k = 0; k < K; ++k) acc[k] = 0.0;
    for (int64_t t0 = 0; t0 + lag0 + 1 < n_frames; t0 += kChunk) {
        __syncthreads();
        stage<K>(sb, t0, kChunk, n_frames, A);
        stage<K>(sb, t0 + lag0 + 1, kChunk + kLagBlock - 1, n_frames, Bt);
        __syncthreads();
        // origins t0 + o with t0 + o + tau < n_frames; a counted loop, unrolled, lets the
        // LDS reads of several origins be in flight together
        const int o_end = (int)min<int64_t>(kChunk, n_frames - tau - t0);
#pragma unroll 8
        for (int o = ph; o < o_end; o += kPhases)
            for (int k = 0; k < K; ++k) {
                const double d = Bt[o + l][k] - A[o][k];
                acc[k] += d * d;
            }
    }
    for (int k = 0; k < K; ++k) part[ph][l][k] = acc[k];
    __syncthreads();
    if (ph == 0 && tau <= n_lags)
        for (int k = 0; k < K; ++k) {
            const double v = (part[0][l][k] + part[1][l][k]) + (part[2][l][k] + part[3][l][k]);
            out[((int64_t)b * n_lags + tau - 1) * K + k] = v / (double)(n_frames - tau);
        }
}

// Tiles: one workgroup per block of consecutive lags and per body (and component).  A
// thread takes M consecutive lags by M origins of every chunk of origins; the chunk is staged in
// LDS with the frames its lags reach, the next chunk's values being in flight to registers.  LG
// groups of M lags by NT / LG sets of origins.  Every sum runs in a fixed order.
constexpr int kFillBlocks = 512;   // workgroups of 256 threads that fill the GPU

template <int NT, int LG, int M>
struct LagShape {
    static constexpr int threads = NT, groups = LG, tile = M;
    static constexpr int runs = NT / LG;             // sets of origins
    static constexpr int chunk = M * runs;           // origins staged at a time
    static constexpr int lags = M * LG;              // lags of a workgroup
    static constexpr int reach = chunk + lags;       // frames the chunk's lags reach
    static constexpr int frames = chunk + reach;
    static_assert(runs % 32 == 0, "a half-wave shares its lag group");
};

// The sums of the threads over their lags, added over the sets of origins in a fixed order; the
// total of lag lag0 + threadIdx.x + 1 is returned to the first S::lags threads.
template <class S>
__device__ __forceinline__ double tile_total(double acc[S::tile], double (*part)[S::tile])
{
    constexpr int halves = S::runs / 32;              // half-waves per lag group
#pragma unroll
    for (int m = 0; m < S::tile; ++m) {
#pragma unroll
        for (int x = 16; x >= 1; x >>= 1) acc[m] += __shfl_xor(acc[m], x, 32);
        if ((threadIdx.x & 31) == 0) part[threadIdx.x >> 5][m] = acc[m];
    }
    __syncthreads();
    const int e = threadIdx.x;
    double v = 0.0;
    if (e < S::lags)
        for (int h = 0; h < halves; ++h) v += part[e / S::tile * halves + h][e % S::tile];
    return v;
}

// grid (lag block, body, component): mean over origins of the squared increment.  A thread's
// origins are consecutive, so the 3 M - 1 = 47 values of its tile feed 256 squared differences
// from registers: 2 FP64 operations per term against 0.18 LDS reads.  (One lag and one origin at
// a time, every term read its two values from LDS; 8 x 8 tiles read 0.36 and took 220 us where
// this takes 198.)  One pad value per M frames spreads the threads' reads over the banks.
// 128 lags per workgroup, or 16 (64 lags: 227 us, more staging).  A tile that reaches past the last
// frame goes frame by frame (term by term, each its two values from LDS, that took 14 us).
// 32 bodies, 20,000 frames, 1000 lags: 3 components 569 -> 198 us, 6 components 809 ->
// 395 us (at the FP64 vector rate: 97 and 195 us).
using WideMsd = LagShape<256, 8, 16>;
using NarrowMsd = LagShape<256, 1, 16>;

template <class S>
__global__ __launch_bounds__(S::threads) __attribute__((amdgpu_waves_per_eu(S::groups > 1 ? 3 : 1)))
void msd_kernel(const double* __restrict__ s, int n_frames, int n_comp, int n_lags,
                double* __restrict__ out)
{
    constexpr int NT = S::threads, M = S::tile;
    __shared__ double A[S::chunk / M * (M + 1)];           // origins t0 ..
    __shared__ double Bt[S::reach / M * (M + 1)];          // frames t0 + lag0 + 1 ..
    __shared__ double part[NT / 32][M];
    const int lag0 = blockIdx.x * S::lags, b = blockIdx.y, comp = blockIdx.z;
    const int r = threadIdx.x % S::runs, lg = threadIdx.x / S::runs;
    const double* sb = s + (int64_t)b * n_frames * n_comp + comp;
    constexpr int NA = S::chunk / NT, NB = (S::reach + NT - 1) / NT;
    double na[NA], nb[NB];
    auto load = [&](int64_t t0) {                          // frames past the end: zero
        const double* pa = sb + t0 * n_comp;
        const double* pb = pa + (int64_t)(lag0 + 1) * n_comp;
        const int64_t left = n_frames - t0;
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const int e = threadIdx.x + q * NT;
            na[q] = e < left ? pa[(int64_t)e * n_comp] : 0.0;
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int e = threadIdx.x + q * NT;
            nb[q] = e < left - lag0 - 1 ? pb[(int64_t)e * n_comp] : 0.0;
        }
    };
    double acc[M];
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = 0.0;
    const double* a = A + (M + 1) * r;
    const double* w = Bt + (M + 1) * (r + lg);
    load(0);
    for (int64_t t0 = 0; t0 + lag0 + 1 < n_frames; t0 += S::chunk) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NA; ++q) {
            const int e = threadIdx.x + q * NT;
            A[e + e / M] = na[q];
        }
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int e = threadIdx.x + q * NT;
            if (e < S::reach) Bt[e + e / M] = nb[q];
        }
        __syncthreads();
        load(t0 + S::chunk);
        // frames from the tile's first (origin, lag) on
        const int64_t left = n_frames - (t0 + M * r + lag0 + M * lg + 1);
        if (left >= 2 * M - 1) {                            // every origin reaches every lag
            double y[2 * M - 1];
#pragma unroll
            for (int j = 0; j < 2 * M - 1; ++j) y[j] = w[j + j / M];
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const double x = a[i];
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    const double d = y[i + m] - x;
                    acc[m] += d * d;
                }
            }
        } else if (left > 0) {                              // frame by frame, up to the last
            double x[M], y = w[0];
#pragma unroll
            for (int i = 0; i < M; ++i) x[i] = a[i];
#pragma unroll
            for (int j = 0; j < 2 * M - 1; ++j) {
                const double yj = y;
                if (j + 1 < 2 * M - 1) y = w[j + 1 + (j + 1) / M];
                if (j < left) {
#pragma unroll
                    for (int m = 0; m < M; ++m)
                        if (j - m >= 0 && j - m < M) {
                            const double d = yj - x[j - m >= 0 && j - m < M ? j - m : 0];
                            acc[m] += d * d;
                        }
                }
            }
        }
    }
    const double v = tile_total<S>(acc, part);
    const int tau = lag0 + (int)threadIdx.x + 1;
    if ((int)threadIdx.x < S::lags && tau <= n_lags)
        out[((int64_t)b * n_lags + tau - 1) * n_comp + comp] = v / (double)(n_frames - tau);
}

// Short trajectories, as short_msd_kernel: grid (lag block, body), mean over origins of the squared
// angle between the reference vectors; the unit vectors R(q) r / |R(q) r| are computed once per
// staged frame
__global__ __launch_bounds__(kBlock) void short_rotation_kernel(const double* __restrict__ traj,
                                                                int n_frames, int n_bodies,
                                                                const double* __restrict__ ref,
                                                                int n_lags, double* __restrict__ out)
{
    __shared__ double A[kChunk][3];
    __shared__ double Bt[kChunk + kLagBlock - 1][3];
    __shared__ double part[kPhases][kLagBlock];
    const int lag0 = blockIdx.x * kLagBlock, b = blockIdx.y;
    const int l = threadIdx.x % kLagBlock, ph = threadIdx.x / kLagBlock;
    const int tau = lag0 + l + 1;
    const double r[3] = {ref[3 * b], ref[3 * b + 1], ref[3 * b + 2]};
    auto unit = [&](int64_t f, double* p) {
        if (f >= n_frames) { p[0] = p[1] = p[2] = 0.0; return; }
        double R[9];
        rot_of(traj + 7 * (f * n_bodies + b) + 3, R);
        for (int a = 0; a < 3; ++a) p[a] = R[3 * a] * r[0] + R[3 * a + 1] * r[1] + R[3 * a + 2] * r[2];
        const double n = sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2]);
        for (int a = 0; a < 3; ++a) p[a] /= n;
    };
    double acc = 0.0;
    for (int64_t t0 = 0; t0 + lag0 + 1 < n_frames; t0 += kChunk) {
        __syncthreads();
        for (int e = threadIdx.x; e < kChunk; e += kBlock) unit(t0 + e, A[e]);
        for (int e = threadIdx.x; e < kChunk + kLagBlock - 1; e += kBlock)
            unit(t0 + lag0 + 1 + e, Bt[e]);
        __syncthreads();
        const int o_end = (int)min<int64_t>(kChunk, n_frames - tau - t0);
#pragma unroll 8
        for (int o = ph; o < o_end; o += kPhases) {
            const double* p0 = A[o];
            const double* p1 = Bt[o + l];
            double c = p0[0] * p1[0] + p0[1] * p1[1] + p0[2] * p1[2];
            c = c > 1.0 ? 1.0 : (c < -1.0 ? -1.0 : c);
            const double th = acos(c);
            acc += th * th;
        }
    }
    part[ph][l] = acc;
    __syncthreads();
    if (ph == 0 && tau <= n_lags)
        out[(int64_t)b * n_lags + tau - 1] =
            ((part[0][l] + part[1][l]) + (part[2][l] + part[3][l])) / (double)(n_frames - tau);
}

// The squared angle from z = 1 - cos theta in [0, 1]: theta^2 = 2 z + z^2 r(z).  zl is what rounding
// took from z (EXACT: nothing, as below 1/2): it enters with the slope 2 theta / sin theta (to 1.5 %).
// r interpolates the series theta^2 = 2 sum_n (2 z)^n / (n^2 C(2n, n)) (that of the squared arcsine of
// sqrt(z / 2)) at the Chebyshev nodes, theta^2 / z to a relative 2e-17.  With 2 z kept apart r's
// rounding errors hardly reach the result.
template <bool EXACT>
__device__ __forceinline__ double squared_angle(double z, double zl)
{
    constexpr double c[19] = {0x1.55555555555f8p-2, 0x1.6c16c16c01aadp-4, 0x1.d41d41e56b008p-6, 0x1.4ce19727a237cp-7,
                               0x1.f85e9253c495cp-9, 0x1.8ef8d0e792e25p-10, 0x1.47423977630aap-11, 0x1.010ddcd930bd4p-12,
                               0x1.6dfbf751fe7a6p-13, -0x1.4e0a7b21d29e3p-13, 0x1.1ade30efbb8f1p-11, -0x1.03fce21011ae4p-10,
                               0x1.879e9e385f6dfp-10, -0x1.bbbdc34bad526p-10, 0x1.7bf11ffa6ad20p-10, -0x1.d8e9353bd632ep-11,
                               0x1.9717eb8ade077p-12, -0x1.b20de0c460ec2p-14, 0x1.b875556a46750p-17};
    double r = c[19 - 1];
#pragma unroll
    for (int n = 19 - 2; n >= 0; --n) r = fma(r, z, c[n]);
    return fma(2.0, z, EXACT ? z * z * r : fma(z * z, r, fma(fma(0.47, z, 2.0 / 3.0), z, 2.0) * zl));
}

// The same of half the angle, from its cosine c: cos(theta / 2) = sqrt((1 + c) / 2) by the hardware's
// reciprocal square root, a coupled Newton step and a correction by the remainder; what is then
// missing to the root, the rounding of 1 + c included, goes into zl.  (From 1 - c, which is rounded
// to one bit less than an obtuse c, the squared angle lost up to six digits towards pi.)
__device__ __forceinline__ double squared_half_angle(double c)
{
    const double s = 1.0 + c, es = c - (s - 1.0);
    const double x = fmax(0.5 * s, 1e-300);
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    g = fma(fma(-g, g, x), h, g);
    const double lo = fma(0.5, es, fma(-g, g, x)) * h, z = 1.0 - g;
    return squared_angle<false>(z, ((1.0 - z) - g) - lo);
}

// grid (lag block, body): mean over origins of the squared angle between the reference
// vectors.  The unit vectors R(q) r / |R(q) r| are computed once per staged frame; a thread's
// origins are NT / LG apart, so that the lanes' reads are consecutive.  The squared angle is
// analytic in the cosine at theta = 0, so it is a polynomial in 1 - cos theta up to a right
// angle, and beyond from the half angle, each wave by its widest angle: with an arccosine and its
// square root per term 32 bodies, 20,000 frames and 1000 lags took 1968 us, this 784 us for steps of
// 0.003 rad per frame, 991 us for 0.03, 1273 us for 0.3.  A term's r.m.s. error is 4e-17 to 6e-17 of it
// at every angle, the squared arccosine's 4e-17 to 12e-17.  A chunk with a non-finite vector takes the
// arccosine itself, so that it propagates as before.  128 lags per workgroup (64 at twice the
// wavefronts: 1130 us where this took 1040), or 16.
using WideAngles = LagShape<512, 16, 8>;
using NarrowAngles = LagShape<256, 2, 8>;

template <class S>
__global__ __launch_bounds__(S::threads) __attribute__((amdgpu_waves_per_eu(2)))
void rotation_msd_kernel(const double* __restrict__ traj, int n_frames, int n_bodies,
                         const double* __restrict__ ref, int n_lags, double* __restrict__ out)
{
    constexpr int NT = S::threads, M = S::tile;
    __shared__ double A[S::chunk][3];                      // origins t0 ..
    __shared__ double Bt[S::reach][3];                     // frames t0 + lag0 + 1 ..
    __shared__ double part[NT / 32][M];
    const int lag0 = blockIdx.x * S::lags, b = blockIdx.y;
    const int r = threadIdx.x % S::runs, lg = threadIdx.x / S::runs;
    const double rv[3] = {ref[3 * b], ref[3 * b + 1], ref[3 * b + 2]};
    constexpr int NF = (S::frames + NT - 1) / NT;
    double q[NF][4];
    // staged frame e: origin t0 + e, or frame t0 + lag0 + 1 + (e - chunk)
    auto frame = [&](int64_t t0, int e) { return e < S::chunk ? t0 + e : t0 + lag0 + 1 + (e - S::chunk); };
    auto load = [&](int64_t t0) {
#pragma unroll
        for (int n = 0; n < NF; ++n) {
            const int e = threadIdx.x + n * NT;
            const int64_t f = frame(t0, e);
            for (int c = 0; c < 4; ++c)
                q[n][c] = e < S::frames && f < n_frames ? traj[7 * (f * n_bodies + b) + 3 + c] : 0.0;
        }
    };
    double acc[M];
#pragma unroll
    for (int m = 0; m < M; ++m) acc[m] = 0.0;
    load(0);
    for (int64_t t0 = 0; t0 + lag0 + 1 < n_frames; t0 += S::chunk) {
        bool bad = false;
        __syncthreads();
#pragma unroll
        for (int n = 0; n < NF; ++n) {
            const int e = threadIdx.x + n * NT;
            if (e >= S::frames) continue;
            double p[3] = {0.0, 0.0, 0.0};
            if (frame(t0, e) < n_frames) {
                double R[9];
                rot_of(q[n], R);
                for (int c = 0; c < 3; ++c)
                    p[c] = R[3 * c] * rv[0] + R[3 * c + 1] * rv[1] + R[3 * c + 2] * rv[2];
                const double len = sqrt(p[0] * p[0] + p[1] * p[1] + p[2] * p[2]);
                for (int c = 0; c < 3; ++c) p[c] /= len;
            }
            bad = bad || !(fabs(p[0]) + fabs(p[1]) + fabs(p[2]) < 4.0);
            double* to = e < S::chunk ? A[e] : Bt[e - S::chunk];
            for (int c = 0; c < 3; ++c) to[c] = p[c];
        }
        bad = __syncthreads_or(bad) != 0;
        load(t0 + S::chunk);
        const bool whole = !bad && t0 + S::chunk + lag0 + S::lags <= n_frames;
#pragma unroll 1
        for (int i = 0; i < M; ++i) {
            const int o = r + S::runs * i;
            const double x0 = A[o][0], x1 = A[o][1], x2 = A[o][2];
            const double (*y)[3] = Bt + o + M * lg;
            double d[M];
#pragma unroll
            for (int m = 0; m < M; ++m) d[m] = x0 * y[m][0] + x1 * y[m][1] + x2 * y[m][2];
            if (whole) {
                bool wide = false, obtuse = false;
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    d[m] = fmin(fmax(d[m], -1.0), 1.0);
                    wide = wide || d[m] < 0.5;
                    obtuse = obtuse || d[m] < 0.0;
                }
                if (!__any(wide)) {                         // 1 - c is exact
#pragma unroll
                    for (int m = 0; m < M; ++m) acc[m] += squared_angle<true>(1.0 - d[m], 0.0);
                } else if (!__any(obtuse)) {
#pragma unroll
                    for (int m = 0; m < M; ++m) {
                        const double z = 1.0 - d[m];
                        acc[m] += squared_angle<false>(z, (1.0 - z) - d[m]);
                    }
                } else {                                    // beyond a right angle
#pragma unroll
                    for (int m = 0; m < M; ++m) acc[m] += 4.0 * squared_half_angle(d[m]);
                }
            } else {
                const int64_t t = t0 + o + lag0 + M * lg + 1;
#pragma unroll
                for (int m = 0; m < M; ++m)
                    if (t + m < n_frames) {
                        const double c = d[m] > 1.0 ? 1.0 : (d[m] < -1.0 ? -1.0 : d[m]);
                        const double th = acos(c);
                        acc[m] += th * th;
                    }
            }
        }
    }
    const double v = tile_total<S>(acc, part);
    const int tau = lag0 + (int)threadIdx.x + 1;
    if ((int)threadIdx.x < S::lags && tau <= n_lags)
        out[(int64_t)b * n_lags + tau - 1] = v / (double)(n_frames - tau);
}

// grid (lag, bin), for more than kTileBins bins: sums of the squared increments from the
// origins whose radial coordinate lies in [edges[bin], edges[bin+1]), over all bodies, and
// their count (one workgroup per lag and bin, the bodies added in order)
template <int K>
__global__ __launch_bounds__(kBlock) void binned_msd_kernel(const double* __restrict__ s,
                                                            const double* __restrict__ radial,
                                                            int n_frames, int n_bodies,
                                                            const double* __restrict__ edges,
                                                            int n_lags, double* __restrict__ sums,
                                                            double* __restrict__ counts)
{
    __shared__ double part[4][K + 1];
    const int tau = blockIdx.x + 1, bin = blockIdx.y;
    const double lo = edges[bin], hi = edges[bin + 1];
    double acc[K + 1];
    for (int k = 0; k <= K; ++k) acc[k] = 0.0;
    for (int b = 0; b < n_bodies; ++b) {
        const double* sb = s + (int64_t)b * n_frames * K;
        const double* rb = radial + (int64_t)b * n_frames;
        for (int64_t t = threadIdx.x; t + tau < n_frames; t += kBlock) {
            const double r = rb[t];
            if (!(r >= lo && r < hi)) continue;
            for (int k = 0; k < K; ++k) {
                const double d = sb[(t + tau) * K + k] - sb[t * K + k];
                acc[k] += d * d;
            }
            acc[K] += 1.0;
        }
    }
    block_sum<K + 1>(acc, part);
    if (threadIdx.x == 0) {
        const int64_t o = (int64_t)bin * n_lags + blockIdx.x;
        for (int k = 0; k < K; ++k) sums[o * K + k] = acc[k];
        counts[o] = acc[K];
    }
}

// For at most kTileBins bins: grid (lag block, body, segment of origins).  A lane takes ML
// consecutive lags and walks the origins of its wave's share of a chunk in order, so its ML
// frames slide along (one new LDS value per origin and component, 2 ML FP64 operations) and the
// origin is the same for the whole wave: its frame comes by scalar loads a group of origins ahead,
// and its bin is uniform.  The running sums stay in registers while the bin does (a body crosses bin
// edges rarely) and are added to the workgroup's LDS sums of that bin when it changes.  The reached
// frames are staged by their index modulo ML so that the lanes' reads are consecutive.  The sums
// of waves, bodies and segments are added with LDS and device atomics, so their order (and the
// last bits of the sums) is not fixed; the counts are whole numbers and exact.  Segments: enough
// workgroups to fill the GPU.
// 32 bodies, 20,000 frames, 1000 lags, 8 bins: 1219 -> 300 us (one lag per lane: every
// term read its frames from LDS and branched on its bin).  Past the last lag that an origin reaches
// the terms are masked; added to the LDS sums one at a time, each origin's frame waited for, they
// took 34 us of 32 bodies, 256 frames and 255 lags, now 29.
//
// ORDERED, for one or two bodies: the sums run in a fixed order, so that every call gives the same
// bits (20,000 frames, 1000 lags, 8 bins: 76 us, in segments 41, by the kernel of one lag per lane
// 1095).  Each wave has LDS sums of its own, added in order at the end, which leaves room for one
// component and one lag per lane: the components are workgroups of their own along grid z, with
// 16 waves in place of segments, and an origin's frame comes from the lane that loaded it.  At most
// two of them add to one output, where the order does not matter: two bodies, or the halves of one
// body's frames.
constexpr int kTileBins = 8;
constexpr int kBinBlock = 512;
constexpr int kOrderedBlock = 1024;
constexpr int kGroup = 4;                        // origins between looks at their bins

__device__ __forceinline__ double lane_value(double v, int lane)
{
    const unsigned long long u = __double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, lane);
    const unsigned hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), lane);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

template <int K, int ML, bool ORDERED>
__global__ __launch_bounds__(ORDERED ? kOrderedBlock : kBinBlock)
__attribute__((amdgpu_waves_per_eu(4)))
void binned_msd_tiled_kernel(
    const double* __restrict__ s, const double* __restrict__ radial, int n_frames, int n_comp,
    const double* __restrict__ edges, int n_bins, int n_lags, int64_t segment,
    double* __restrict__ sums, double* __restrict__ counts)
{
    static_assert(!ORDERED || K == 1, "a component of its own");
    static_assert(kGroup % ML == 0, "the window's offset is known within a group");
    constexpr int NT = ORDERED ? kOrderedBlock : kBinBlock;
    constexpr int chunk = NT;                    // origins staged at a time: 64 per wave
    constexpr int copies = ORDERED ? NT / 64 : 1;
    constexpr int lags = 64 * ML;
    constexpr int reach = chunk + lags + ML;
    __shared__ double Bt[K][ML][reach / ML];
    __shared__ double total[copies][kTileBins][ML][K][64];
    __shared__ int count[kTileBins][ML][64];    // of the origins that not every lag reaches
    __shared__ int full[kTileBins];             // of the others
    const int lag0 = blockIdx.x * lags, b = blockIdx.y;
    const int comp = ORDERED ? blockIdx.z % n_comp : 0, seg = ORDERED ? blockIdx.z / n_comp : blockIdx.z;
    const int stride = ORDERED ? n_comp : K;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double* __restrict__ sb = s + (int64_t)b * n_frames * stride + comp;
    const double* __restrict__ rb = radial + (int64_t)b * n_frames;
    for (int e = threadIdx.x; e < copies * kTileBins * ML * K * 64; e += NT) (&total[0][0][0][0][0])[e] = 0.0;
    for (int e = threadIdx.x; e < kTileBins * ML * 64; e += NT) (&count[0][0][0])[e] = 0;
    if (threadIdx.x < kTileBins) full[threadIdx.x] = 0;
    double acc[ML][K];
#pragma unroll
    for (int m = 0; m < ML; ++m)
        for (int k = 0; k < K; ++k) acc[m][k] = 0.0;
    int cur = -1;                               // the bin of acc (-1: none, dropped)
    auto flush = [&]() {
        if (cur >= 0) {
#pragma unroll
            for (int m = 0; m < ML; ++m)
                for (int k = 0; k < K; ++k) {
                    if constexpr (ORDERED) total[wave][cur][m][k][lane] += acc[m][k];
                    else atomicAdd(&total[0][cur][m][k][lane], acc[m][k]);
                }
        }
#pragma unroll
        for (int m = 0; m < ML; ++m)
            for (int k = 0; k < K; ++k) acc[m][k] = 0.0;
    };
    double edge[kTileBins + 1];
#pragma unroll
    for (int q = 0; q <= kTileBins; ++q) edge[q] = q <= n_bins ? edges[q] : 0.0;
    const int64_t begin = segment * seg;
    const int64_t end = begin + segment < n_frames ? begin + segment : n_frames;
    // ORDERED: the frames that a chunk's lags reach, its origins' frames and their radial positions are
    // loaded a chunk ahead
    constexpr int NS = ORDERED ? (reach * K + NT - 1) / NT : 1;
    double st[NS], rad = 0.0, org = 0.0;
    auto load = [&](int64_t t0) {
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const int e = threadIdx.x + q * NT;
            const int64_t f = t0 + lag0 + 1 + e;
            st[q] = e < reach && f < n_frames ? sb[f * stride] : 0.0;
        }
        const int64_t t = t0 + threadIdx.x;
        rad = t < end ? rb[t] : 0.0;
        org = t < end ? sb[t * stride] : 0.0;
    };
    if constexpr (ORDERED) load(begin);
    for (int64_t t0 = begin; t0 < end && t0 + lag0 + 1 < n_frames; t0 += chunk) {
        __syncthreads();
        if constexpr (ORDERED) {
#pragma unroll
            for (int q = 0; q < NS; ++q)
                if ((int)threadIdx.x + q * NT < reach) Bt[0][0][threadIdx.x + q * NT] = st[q];
        } else {
            for (int e = threadIdx.x; e < reach * K; e += NT) {
                const int64_t f = t0 + lag0 + 1 + e / K;
                Bt[e % K][e / K % ML][e / K / ML] = f < n_frames ? sb[f * stride + e % K] : 0.0;
            }
        }
        __syncthreads();
        // the bin of each of the wave's 64 origins, one per lane (-1: none)
        const int64_t tw = t0 + 64 * wave;
        int bin = -1;
        if (tw + lane < end) {
            if constexpr (!ORDERED) rad = rb[tw + lane];
#pragma unroll
            for (int q = 0; q < kTileBins; ++q)
                if (q < n_bins && rad >= edge[q] && rad < edge[q + 1]) bin = q;
        }
        const double from = org;
        if constexpr (ORDERED) load(t0 + chunk);
        // whether every origin reaches every lag: then an origin counts once for all of them
        const bool whole = tw + 64 <= end && tw + 63 + lag0 + lags < n_frames;
        if (whole)
            for (int q = 0; q < n_bins; ++q) {
                const int c = __popcll(__ballot(bin == q));
                if (c > 0 && lane == 0) atomicAdd(&full[q], c);
            }
        // origins that some lag reaches
        const int64_t some = (end < n_frames - 1 - lag0 ? end : n_frames - 1 - lag0) - tw;
        const int n_org = some < 64 ? (int)some : 64;
        double w[ML][K];                        // the frames of the lane's lags
#pragma unroll
        for (int m = 0; m < ML; ++m)
            for (int k = 0; k < K; ++k) w[m][k] = Bt[k][m][64 / ML * wave + lane];
        // the origins of the wave's share, a group at a time, their frames loaded one group ahead;
        // MASK: not every lag reaches each
        auto walk = [&](auto mask) {
            constexpr bool MASK = decltype(mask)::value;
            double a[kGroup][K], next[kGroup][K];
            auto fetch = [&](int g) {
#pragma unroll
                for (int i = 0; i < kGroup; ++i)
                    for (int k = 0; k < K; ++k) {
                        if constexpr (ORDERED) {
                            next[i][k] = lane_value(from, g + i);
                        } else {                                                // uniform
                            const int64_t t = tw + g + i;
                            next[i][k] = sb[(!MASK || t < n_frames ? t : n_frames - 1) * K + k];
                        }
                    }
            };
            // one origin: the lane's lags, then the window moves on
            auto origin = [&](int g, int i) {
                const int left = MASK ? (int)(n_frames - 1 - (tw + g + i) - lag0) - ML * lane : 0;
#pragma unroll
                for (int m = 0; m < ML; ++m) {
                    const bool in = !MASK || m < left;
                    for (int k = 0; k < K; ++k) {
                        const double d = in ? w[m][k] - a[i][k] : 0.0;
                        acc[m][k] += d * d;
                    }
                    if (MASK && in && cur >= 0) atomicAdd(&count[cur][m][lane], 1);
                }
#pragma unroll
                for (int k = 0; k < K; ++k) {
#pragma unroll
                    for (int m = 0; m + 1 < ML; ++m) w[m][k] = w[m + 1][k];
                    w[ML - 1][k] = Bt[k][i % ML][64 / ML * wave + (g + i) / ML + 1 + lane];
                }
            };
            const int n = MASK ? n_org : 64;
            fetch(0);
#pragma unroll 1
            for (int g = 0; g < n; g += kGroup) {
#pragma unroll
                for (int i = 0; i < kGroup; ++i)
                    for (int k = 0; k < K; ++k) a[i][k] = next[i][k];
                fetch(g + kGroup < n ? g + kGroup : 0);
                constexpr unsigned long long group = (1ull << kGroup) - 1;
                if (((__ballot(bin == cur) >> g) & group) == group) {
#pragma unroll
                    for (int i = 0; i < kGroup; ++i) origin(g, i);
                } else {
#pragma unroll
                    for (int i = 0; i < kGroup; ++i) {
                        const int j = __builtin_amdgcn_readlane(bin, g + i);
                        if (j != cur) {
                            flush();
                            cur = j;
                        }
                        origin(g, i);
                    }
                }
            }
        };
        if (whole) walk(std::false_type{});
        else if (n_org > 0) walk(std::true_type{});
    }
    flush();
    __syncthreads();
    for (int e = threadIdx.x; e < n_bins * lags * (K + 1); e += NT) {
        const int k = e % (K + 1), m = e / (K + 1) % lags, q = e / (K + 1) / lags;
        if (lag0 + m >= n_lags) continue;
        const int64_t o = (int64_t)q * n_lags + lag0 + m;
        if (k < K) {
            double v = 0.0;
            for (int c = 0; c < copies; ++c) v += total[c][q][m % ML][k][m / ML];
            atomicAdd(sums + o * stride + comp + k, v);
        } else if (comp == 0) {
            atomicAdd(counts + o, (double)(full[q] + count[q][m % ML][m / ML]));
        }
    }
}

// zero sums[0..n) and counts[0..m) (a kernel: a captured memset has given wrong replays)
__global__ void zero_sums_kernel(double* sums, int64_t n, double* counts, int64_t m)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) sums[i] = 0.0;
    else if (i < n + m) counts[i - n] = 0.0;
}

template <class Step>
void launch_cumulate(const double* traj, int32_t n_frames, int32_t n_bodies, double cx, double cy,
                     double* out, double* radial, hipStream_t s)
{
    const int n_seg = std::max<int>(1, (int)(((int64_t)n_frames - 1 + kSpan - 1) / kSpan));
    hipLaunchKernelGGL((cumulate_kernel<Step>), dim3((unsigned)n_bodies * n_seg), dim3(kBlock), 0, s,
                       traj, n_frames, n_bodies, n_seg, cx, cy, out, radial);
    if (n_seg == 1) return;
    hipLaunchKernelGGL((segment_totals_kernel<Step::K>), dim3(n_bodies), dim3(kBlock), 0, s, out,
                       n_frames, n_seg);
    hipLaunchKernelGGL((add_before_kernel<Step::K>), dim3((unsigned)n_bodies * (n_seg - 1)),
                       dim3(kBlock), 0, s, out, n_frames, n_seg);
}

template <class S>
int64_t lag_blocks(int32_t n_lags) { return ((int64_t)n_lags + S::lags - 1) / S::lags; }

// The MSD kernels' duration in us, for the choice between them: what one workgroup takes (start +
// per_frame * frames: the latency of its chain) or what `blocks` of them cost the full GPU, whichever
// is more, with a smooth passage (the fourth powers).  Fitted to measured times (1 to 1024 bodies, 16 to
// 50,000 frames, 4 to 8191 lags; 1, 3 and 6 components), which it meets to 10 - 17 % r.m.s.; the
// kernel chosen takes 1 % more than the fastest in the mean, at most 1.4 times it.
struct MsdCost {
    double start, per_frame;               // of one workgroup alone, us
    double block_start, block_per_frame;   // of one among many, us

    double us(double frames, int64_t blocks) const
    {
        const double one = start + per_frame * frames;
        const double all = blocks * (block_start + block_per_frame * frames);
        return std::sqrt(std::hypot(one * one, all * all));
    }
};

enum class MsdShape { Short, Narrow, Wide };

MsdShape fastest(double t_short, double t_narrow, double t_wide)
{
    if (t_short <= std::min(t_narrow, t_wide)) return MsdShape::Short;
    return t_narrow <= t_wide ? MsdShape::Narrow : MsdShape::Wide;
}

template <int K, int ML>
void launch_binned(const double* series, const double* radial, int32_t n_frames, int32_t n_bodies,
                   const double* edges, int32_t n_bins, int32_t n_lags, double* sums,
                   double* counts, hipStream_t s)
{
    // segments of origins: at least one chunk each, and no more workgroups than fill the GPU
    const int64_t blocks = ((int64_t)n_lags + 64 * ML - 1) / (64 * ML);
    const int64_t chunks = ((int64_t)n_frames + kBinBlock - 1) / kBinBlock;
    const int64_t per = std::max<int64_t>(1, chunks * blocks * n_bodies / kFillBlocks);
    const dim3 grid((unsigned)blocks, n_bodies, (unsigned)((chunks + per - 1) / per));
    hipLaunchKernelGGL((binned_msd_tiled_kernel<K, ML, false>), grid, dim3(kBinBlock), 0, s, series,
                       radial, n_frames, K, edges, n_bins, n_lags, per * kBinBlock, sums, counts);
}

// one or two bodies: the frames of one body in two halves of whole chunks
void launch_binned_ordered(const double* series, const double* radial, int32_t n_frames,
                           int32_t n_bodies, int32_t k, const double* edges, int32_t n_bins,
                           int32_t n_lags, double* sums, double* counts, hipStream_t s)
{
    const int64_t chunks = ((int64_t)n_frames + kOrderedBlock - 1) / kOrderedBlock;
    const int64_t per = n_bodies == 1 ? (chunks + 1) / 2 : chunks;
    const dim3 grid((unsigned)(((int64_t)n_lags + 63) / 64), n_bodies,
                    (unsigned)(k * ((chunks + per - 1) / per)));
    hipLaunchKernelGGL((binned_msd_tiled_kernel<1, 1, true>), grid, dim3(kOrderedBlock), 0, s, series,
                       radial, n_frames, k, edges, n_bins, n_lags, per * kOrderedBlock, sums, counts);
}

bool frames_ok(const double* p, int32_t n_frames, int32_t n_bodies)
{
    return p && n_frames >= 1 && n_bodies >= 1 && (int64_t)n_frames * n_bodies * 7 < (int64_t(1) << 40);
}

int launched() { return hipGetLastError() == hipSuccess ? LB_OK : LB_ERR_HIP; }

}  // namespace

void launch_record_poses(const Body* bodies, int n_bodies, double* frame, hipStream_t s)
{
    if (n_bodies <= 0) return;
    hipLaunchKernelGGL(record_kernel, dim3((n_bodies + 255) / 256), dim3(256), 0, s, bodies,
                       n_bodies, frame);
}

}  // namespace lbrb

using namespace lbrb;

extern "C" {

int lb_traj_lab_frame(const double* traj, int32_t n_frames, int32_t n_bodies, double* out,
                        void* stream)
{
    if (!frames_ok(traj, n_frames, n_bodies) || !out) return LB_ERR_ARG;
    const dim3 block(kBlock);
    const unsigned blocks = (unsigned)(((int64_t)n_frames + kBlock - 1) / kBlock);
    for (int64_t b = 0; b < n_bodies; b += 65535)   // (bodies along the grid's second dimension)
        hipLaunchKernelGGL(lab_kernel, dim3(blocks, (unsigned)std::min<int64_t>(n_bodies - b, 65535)), block,
                           0, (hipStream_t)stream, traj, n_frames, n_bodies, (int)b, out);
    return launched();
}

int lb_traj_body_frame(const double* traj, int32_t n_frames, int32_t n_bodies, double* out,
                         void* stream)
{
    if (!frames_ok(traj, n_frames, n_bodies) || !out) return LB_ERR_ARG;
    launch_cumulate<BodyStep>(traj, n_frames, n_bodies, 0.0, 0.0, out, nullptr, (hipStream_t)stream);
    return launched();
}

int lb_traj_pore_frame(const double* traj, int32_t n_frames, int32_t n_bodies, double cx,
                         double cy, double* out, double* radial, void* stream)
{
    if (!frames_ok(traj, n_frames, n_bodies) || !out || !radial || !std::isfinite(cx) ||
        !std::isfinite(cy))
        return LB_ERR_ARG;
    launch_cumulate<PoreStep>(traj, n_frames, n_bodies, cx, cy, out, radial, (hipStream_t)stream);
    return launched();
}

int lb_traj_msd(const double* series, int32_t n_frames, int32_t n_bodies, int32_t k,
                  int32_t n_lags, double* out, void* stream)
{
    if (!frames_ok(series, n_frames, n_bodies) || !out || k < 1 || k > 6 || n_lags < 1 ||
        n_lags >= n_frames || n_bodies > 65535)
        return LB_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    const int64_t short_blocks = lag_blocks<ShortMsd>(n_lags) * n_bodies;
    const int64_t narrow_blocks = lag_blocks<NarrowMsd>(n_lags) * n_bodies * k;
    const int64_t wide_blocks = lag_blocks<WideMsd>(n_lags) * n_bodies * k;
    // (the short kernel reads all components together; near the line it goes first, as the estimates
    // of the tiles are low for one component)
    switch (fastest(0.9 * MsdCost{3.65, 0.0063, 0.0046, 1.1e-5}.us((double)n_frames * k, short_blocks),
                    MsdCost{10.7, 0.0007, 0.0365, 3.3e-6}.us(n_frames, narrow_blocks),
                    MsdCost{10.1, 0.0033, 0.0105, 9.4e-6}.us(n_frames, wide_blocks))) {
    case MsdShape::Short: {
        const dim3 grid((unsigned)lag_blocks<ShortMsd>(n_lags), n_bodies);
        switch (k) {
        case 1: hipLaunchKernelGGL((short_msd_kernel<1>), grid, dim3(kBlock), 0, s, series, n_frames, n_lags, out); break;
        case 2: hipLaunchKernelGGL((short_msd_kernel<2>), grid, dim3(kBlock), 0, s, series, n_frames, n_lags, out); break;
        case 3: hipLaunchKernelGGL((short_msd_kernel<3>), grid, dim3(kBlock), 0, s, series, n_frames, n_lags, out); break;
        case 4: hipLaunchKernelGGL((short_msd_kernel<4>), grid, dim3(kBlock), 0, s, series, n_frames, n_lags, out); break;
        case 5: hipLaunchKernelGGL((short_msd_kernel<5>), grid, dim3(kBlock), 0, s, series, n_frames, n_lags, out); break;
        default: hipLaunchKernelGGL((short_msd_kernel<6>), grid, dim3(kBlock), 0, s, series, n_frames, n_lags, out); break;
        }
        break;
    }
    case MsdShape::Narrow:
        hipLaunchKernelGGL((msd_kernel<NarrowMsd>), dim3(lag_blocks<NarrowMsd>(n_lags), n_bodies, k),
                           dim3(NarrowMsd::threads), 0, s, series, n_frames, k, n_lags, out);
        break;
    case MsdShape::Wide:
        hipLaunchKernelGGL((msd_kernel<WideMsd>), dim3(lag_blocks<WideMsd>(n_lags), n_bodies, k),
                           dim3(WideMsd::threads), 0, s, series, n_frames, k, n_lags, out);
        break;
    }
    return launched();
}

int lb_traj_rotation_msd(const double* traj, int32_t n_frames, int32_t n_bodies,
                           const double* ref_body, int32_t n_lags, double* out, void* stream)
{
    if (!frames_ok(traj, n_frames, n_bodies) || !ref_body || !out || n_lags < 1 ||
        n_lags >= n_frames || n_bodies > 65535)
        return LB_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    const int64_t short_blocks = lag_blocks<ShortMsd>(n_lags) * n_bodies;
    const int64_t narrow_blocks = lag_blocks<NarrowAngles>(n_lags) * n_bodies;
    const int64_t wide_blocks = lag_blocks<WideAngles>(n_lags) * n_bodies;
    switch (fastest(MsdCost{5.5, 0.065, 0.0059, 1.64e-4}.us(n_frames, short_blocks),
                    MsdCost{12.2, 0.0115, 0.027, 3.0e-5}.us(n_frames, narrow_blocks),
                    MsdCost{11.9, 0.0427, 0.042, 1.76e-4}.us(n_frames, wide_blocks))) {
    case MsdShape::Short:
        hipLaunchKernelGGL(short_rotation_kernel, dim3(lag_blocks<ShortMsd>(n_lags), n_bodies),
                           dim3(kBlock), 0, s, traj, n_frames, n_bodies, ref_body, n_lags, out);
        break;
    case MsdShape::Narrow:
        hipLaunchKernelGGL((rotation_msd_kernel<NarrowAngles>),
                           dim3(lag_blocks<NarrowAngles>(n_lags), n_bodies),
                           dim3(NarrowAngles::threads), 0, s, traj, n_frames, n_bodies, ref_body,
                           n_lags, out);
        break;
    case MsdShape::Wide:
        hipLaunchKernelGGL((rotation_msd_kernel<WideAngles>),
                           dim3(lag_blocks<WideAngles>(n_lags), n_bodies), dim3(WideAngles::threads),
                           0, s, traj, n_frames, n_bodies, ref_body, n_lags, out);
        break;
    }
    return launched();
}

int lb_traj_binned_msd(const double* series, const double* radial, int32_t n_frames,
                         int32_t n_bodies, int32_t k, const double* edges, int32_t n_bins,
                         int32_t n_lags, double* sums, double* counts, void* stream)
{
    if (!frames_ok(series, n_frames, n_bodies) || !radial || !edges || !sums || !counts ||
        k < 1 || k > 3 || n_bins < 1 || n_bins > 65535 || n_lags < 1 || n_lags >= n_frames)
        return LB_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    if (n_bins <= kTileBins && n_bodies <= 65535) {
        const int64_t n_sums = (int64_t)k * n_bins * n_lags, n_counts = (int64_t)n_bins * n_lags;
        hipLaunchKernelGGL(zero_sums_kernel, dim3((unsigned)((n_sums + n_counts + kBlock - 1) / kBlock)),
                           dim3(kBlock), 0, s, sums, n_sums, counts, n_counts);
        // One or two bodies in a fixed order; so also trajectories of one chunk while the workgroups all
        // run at once, which start sooner (8 bodies, 256 frames, 255 lags 13.6 us against 28.9; 32 of
        // 384 with 383 lags, 576 workgroups, 32.3 / 32.9).  Else 256 lags per workgroup, or 64 where
        // most of 256 would be past the last lag (then 384 workgroups take 25.0 against 17.4 us).
        const int64_t ordered_blocks = ((int64_t)n_lags + 63) / 64 * n_bodies * k;
        const bool one_chunk = n_frames <= kOrderedBlock && ordered_blocks <= (n_lags > 128 ? 512 : 256);
        if (n_bodies <= 2 || one_chunk) {
            launch_binned_ordered(series, radial, n_frames, n_bodies, k, edges, n_bins, n_lags, sums, counts, s);
        } else if (n_lags > 128) {
            switch (k) {
            case 1: launch_binned<1, 4>(series, radial, n_frames, n_bodies, edges, n_bins, n_lags, sums, counts, s); break;
            case 2: launch_binned<2, 4>(series, radial, n_frames, n_bodies, edges, n_bins, n_lags, sums, counts, s); break;
            default: launch_binned<3, 4>(series, radial, n_frames, n_bodies, edges, n_bins, n_lags, sums, counts, s); break;
            }
        } else {
            switch (k) {
            case 1: launch_binned<1, 1>(series, radial, n_frames, n_bodies, edges, n_bins, n_lags, sums, counts, s); break;
            case 2: launch_binned<2, 1>(series, radial, n_frames, n_bodies, edges, n_bins, n_lags, sums, counts, s); break;
            default: launch_binned<3, 1>(series, radial, n_frames, n_bodies, edges, n_bins, n_lags, sums, counts, s); break;
            }
        }
        return launched();
    }
    const dim3 grid(n_lags, n_bins);
    switch (k) {
    case 1: hipLaunchKernelGGL((binned_msd_kernel<1>), grid, dim3(kBlock), 0, s, series, radial, n_frames, n_bodies, edges, n_lags, sums, counts); break;
    case 2: hipLaunchKernelGGL((binned_msd_kernel<2>), grid, dim3(kBlock), 0, s, series, radial, n_frames, n_bodies, edges, n_lags, sums, counts); break;
    default: hipLaunchKernelGGL((binned_msd_kernel<3>), grid, dim3(kBlock), 0, s, series, radial, n_frames, n_bodies, edges, n_lags, sums, counts); break;
    }
    return launched();
}

}  // extern "C"
