// tube.hip -- D1Q3, up to 32 steps per launch with the nodes in registers.
//
// A wave holds a window of 64 N consecutive nodes, N in each lane, and takes
// up to 32 steps without touching memory: a node's neighbours are the lane's
// own other nodes, and one value per lane and side comes from the neighbouring
// lane by a wave shift.  The nodes within one step of the window's ends go
// stale each step, so the wave owns the 64 N - 64 nodes in the middle; at a
// lattice end the window is cut and the end node pulls from itself.  No LDS
// and no barrier, and N independent nodes per lane hide the latency of one.
// Every value is rounded to the storage type after every step and every node
// takes the same arithmetic, so results are bitwise equal to single steps.
//
// Bound by VALU issue: about 32 operations per node and step in FP64, 40 with
// FP16 deviations (66 and 54 in a form that kept 1024-node segments in LDS,
// read and written there every step, with a barrier).  Nodes per lane: more
// repeat fewer window nodes (64 of 64 N) and hide more latency, fewer spread a
// short lattice over more waves; 16 need so many registers that too few waves
// remain.  Measured, segments in LDS -> here: 4096 tubes FP64 472,000 -> 838,000
// MLUPS, FP16 deviations 895,000 -> 1,050,000, 1024 tubes FP32 870,000 ->
// 1,480,000; 800 nodes FP64 0.64 -> 0.33 us per step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdint.h>
#include <type_traits>

#include "device.hpp"
#include "kernels.hpp"

namespace lbm {

constexpr int kTubeSteps = 32;  // steps a window is good for (whole vectors of every storage type)
constexpr int tube_own(int n) { return 64 * n - 2 * kTubeSteps; }

// The stability criterion of Sec. IV.G on one value, as one class test: +-0,
// positive denormal or positive normal (not negative, not infinite, not NaN).
__device__ __forceinline__ bool stable3(double v) { return __builtin_amdgcn_class(v, 0x1e0); }
__device__ __forceinline__ bool stable3(float v) { return __builtin_amdgcn_classf(v, 0x1e0); }

// Register budget (waves per SIMD asked of the compiler): with eight FP64 nodes
// per lane it otherwise takes 181 registers, 2 waves.  At 3 waves it spills 60
// bytes a lane, stored and loaded once per launch (the 4096-tube batch then writes
// 1.34 times its populations' bytes), and the 1024-tube batch still runs at 808,000
// MLUPS instead of 764,000; at 4 waves at 728,000.  No budget helps the other
// forms.
constexpr int tube_waves(int st, int n) { return st == ST_F64 && n == 8 ? 3 : 1; }

template <int ST, int N, bool BATCH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(tube_waves(ST, N)))) void k_d1q3_regs(const typename Form<ST>::T *__restrict__ src_all,
                                                   typename Form<ST>::T *__restrict__ dst_all, StepArgs a)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    constexpr int W = 64 * N, S = tube_own(N);
    constexpr int V = 16 / sizeof(T);  // elements of a 16-byte access
    const int tile = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (tile >= a.ntiles) return;  // wave-uniform
    const int ii = BATCH ? a.tile_inst[tile] : 0;
    const Inst &in = BATCH ? a.inst[ii] : a.one;
    const int n = in.nx;
    const int64_t P = in.plane;
    const int x0 = BATCH ? a.tile_first[tile] : tile * S;  // first own node
    const int sn = min(S, n - x0);
    const T *src = src_all + (BATCH ? in.offset : 0);
    T *dst = dst_all + (BATCH ? in.offset : 0);
    const bool wrap = a.bc == BC_PERIODIC;
    const int lane = (int)(threadIdx.x & 63);

    // Steps this launch takes here (wave-uniform): fewer for a batch instance
    // that reaches its step limit, none for one that has.
    const int64_t s0 = a.step + (a.step_base ? *a.step_base : 0);
    int kdo = min(a.max_steps, kTubeSteps);
    if constexpr (BATCH) kdo = (int)max((int64_t)0, min((int64_t)kdo, in.stop - s0));
    if (kdo <= 0) {
        for (int k = lane; k < sn; k += 64) carry_node(src, dst, P, 3, x0 + k);
        return;
    }
    // The window starts on a vector (planes, instances and own ranges start on 64
    // elements), at least as many nodes before the own ones as there are steps:
    // a launch of any number of steps then loads vectors (ten million nodes, us per
    // launch, windows that start at the first node needed / on a vector: three
    // steps FP64 346 / 121, FP32 107 / 40, two steps FP16 deviations 57 / 29).
    const int lead = (kdo + V - 1) / V * V;
    const int ws = wrap ? x0 - lead : max(0, x0 - lead);  // first node of the window
    const int x = ws + lane * N;                          // first node of this lane
    const bool inside = ws >= 0 && ws + W <= n;
    const bool vec = N % V == 0 && inside;  // a lane's nodes are whole vectors
    T f0[N], fp[N], fm[N];
    if (vec) {
        const T *p = src + x;
#pragma unroll
        for (int c = 0; c < N / V; ++c) {
            const Chunk<T> v0 = __builtin_bit_cast(Chunk<T>, *(const u32x4 *)(p + c * V));
            const Chunk<T> v1 = __builtin_bit_cast(Chunk<T>, *(const u32x4 *)(p + P + c * V));
            const Chunk<T> v2 = __builtin_bit_cast(Chunk<T>, *(const u32x4 *)(p + 2 * P + c * V));
#pragma unroll
            for (int e = 0; e < V; ++e) {
                f0[c * V + e] = v0.e[e];
                fp[c * V + e] = v1.e[e];
                fm[c * V + e] = v2.e[e];
            }
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            int g = x + j;
            if (wrap) g = ((g % n) + n) % n;
            else g = min(g, n - 1);
            f0[j] = src[g];
            fp[j] = src[P + g];
            fm[j] = src[2 * P + g];
        }
    }
    const C r0 = C(2.0 / 3.0) * C(in.rho0), r1 = C(1.0 / 6.0) * C(in.rho0);
    const C omega = C(in.omega);
    uint64_t own[N];  // lanes whose node j is the wave's own
#pragma unroll
    for (int j = 0; j < N; ++j) own[j] = __ballot(x + j >= x0 && x + j < x0 + sn);
    int bad_step = -1, bad_x = 0;

    auto steps = [&](auto ends) __attribute__((always_inline)) {
        constexpr bool ENDS = decltype(ends)::value;  // the window holds a wall node
        for (int s = 0; s < kdo; ++s) {
            const T from_left = lane_shift<true>(fp[N - 1]), from_right = lane_shift<false>(fm[0]);
            T below = from_left;  // plane 1 of the node to the left, before this step
            uint64_t bad[N], any = 0;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                T pin = below, min_ = j < N - 1 ? fm[j < N - 1 ? j + 1 : j] : from_right;
                below = fp[j];
                bool wall = false;
                if constexpr (ENDS) {
                    const bool first = x + j == 0, last = x + j == n - 1;
                    wall = first || last;
                    pin = first ? fp[j] : pin;
                    min_ = last ? fm[j] : min_;
                }
                C g0 = load<ST>(&f0[j], r0, a.fp16_iscale);
                C gp = load<ST>(&pin, r1, a.fp16_iscale);
                C gm = load<ST>(&min_, r1, a.fp16_iscale);
                const C w0 = g0, wp = gm, wm = gp;  // a wall swaps what it pulled
                collide3(g0, gp, gm, omega);
                bool ok = stable3(g0) && stable3(gp) && stable3(gm);
                if constexpr (ENDS) {
                    g0 = wall ? w0 : g0;
                    gp = wall ? wp : gp;
                    gm = wall ? wm : gm;
                    ok = ok || wall;
                }
                bad[j] = ~__ballot(ok) & own[j];
                any |= bad[j];
                f0[j] = to_storage<ST>(g0, r0, a.fp16_scale);
                fp[j] = to_storage<ST>(gp, r1, a.fp16_scale);
                fm[j] = to_storage<ST>(gm, r1, a.fp16_scale);
            }
            if (any != 0) {  // rare; the lane's first event, its smallest node
#pragma unroll
                for (int j = 0; j < N; ++j)
                    if (bad_step < 0 && ((bad[j] >> lane) & 1)) {
                        bad_step = s;
                        bad_x = x + j;
                    }
            }
        }
    };
    if (!wrap && (ws == 0 || ws + W >= n)) steps(std::true_type{});
    else steps(std::false_type{});

    const bool all = x >= x0 && x + N <= x0 + sn;
    if (vec && all) {
        T *p = dst + x;
#pragma unroll
        for (int c = 0; c < N / V; ++c) {
            Chunk<T> v0, v1, v2;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                v0.e[e] = f0[c * V + e];
                v1.e[e] = fp[c * V + e];
                v2.e[e] = fm[c * V + e];
            }
            *(u32x4 *)(p + c * V) = __builtin_bit_cast(u32x4, v0);
            *(u32x4 *)(p + P + c * V) = __builtin_bit_cast(u32x4, v1);
            *(u32x4 *)(p + 2 * P + c * V) = __builtin_bit_cast(u32x4, v2);
        }
    } else {
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const int g = x + j;
            if (g >= x0 && g < x0 + sn) {
                dst[g] = f0[j];
                dst[P + g] = fp[j];
                dst[2 * P + g] = fm[j];
            }
        }
    }
    if (__ballot(bad_step >= 0) != 0ull)
        report_key(a.status + ii, bad_step >= 0 ? event_key(s0 + bad_step, bad_x) : ~0ull);
}

namespace {

template <int ST, int N>
hipError_t tube_go(int batch, const void *src, void *dst, StepArgs a, hipStream_t s)
{
    using T = typename Form<ST>::T;
    if (!batch) a.ntiles = (a.one.nx + tube_own(N) - 1) / tube_own(N);
    const dim3 blocks((a.ntiles + 3) / 4);
    if (batch) hipLaunchKernelGGL((k_d1q3_regs<ST, N, true>), blocks, dim3(256), 0, s, (const T *)src, (T *)dst, a);
    else hipLaunchKernelGGL((k_d1q3_regs<ST, N, false>), blocks, dim3(256), 0, s, (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST>
hipError_t tube_n(int n, int batch, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    switch (n) {
    case 2: return tube_go<ST, 2>(batch, src, dst, a, s);
    case 4: return tube_go<ST, 4>(batch, src, dst, a, s);
    case 8: return tube_go<ST, 8>(batch, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_d1q3_regs(int st, int n, int batch, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    switch (st) {
    case ST_F64: return tube_n<ST_F64>(n, batch, src, dst, a, s);
    case ST_F32N64: return tube_n<ST_F32N64>(n, batch, src, dst, a, s);
    case ST_F32: return tube_n<ST_F32>(n, batch, src, dst, a, s);
    case ST_F16DEV: return tube_n<ST_F16DEV>(n, batch, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
