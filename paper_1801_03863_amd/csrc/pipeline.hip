// pipeline.hip -- launchers of the register-pipeline shapes (pipeline.hpp) of
// one collision rule; compiled once per rule (LBM_PIPE_CO).
#include "pipeline.hpp"

namespace lbm {

namespace {

// Plain loads and stores: tiles are not whole cache lines wide, and two waves
// share the lines at a tile's sides.  Non-temporal stores write those lines
// in parts and non-temporal loads fetch them twice (4096^2, us per step,
// plain / non-temporal stores / both: SRT FP32 4 steps 87 / 101 / 109, FP32
// MinxEnt4 3 steps 127 / 135 / 141, FP64 2 steps 305 / 323 / 334).
template <int ST, int CO, int K, bool BATCH>
hipError_t rp_go(const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int blocks = (a.ntiles + 3) / 4;
    hipLaunchKernelGGL((k_d2q9_rp<ST, CO, K, BATCH>), dim3(blocks), dim3(256), 0, s, (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST, int CO, bool BATCH>
hipError_t rp_k(int k, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    switch (k) {
    case 2: return rp_go<ST, CO, 2, BATCH>(src, dst, a, s);
    case 3: return rp_go<ST, CO, 3, BATCH>(src, dst, a, s);
    case 4: return rp_go<ST, CO, 4, BATCH>(src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

template <int ST, int CO>
hipError_t rp_b(int k, int batch, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    return batch ? rp_k<ST, CO, true>(k, src, dst, a, s) : rp_k<ST, CO, false>(k, src, dst, a, s);
}

}  // namespace

#define LBM_CAT2(a, b) a##b
#define LBM_CAT(a, b) LBM_CAT2(a, b)
hipError_t LBM_CAT(launch_d2q9_pipe_, LBM_PIPE_CO)(int st, int k, int batch, const void *src, void *dst, const StepArgs &a,
                                                 hipStream_t s)
{
    switch (st) {
    case ST_F64: return rp_b<ST_F64, LBM_PIPE_CO>(k, batch, src, dst, a, s);
    case ST_F32N64: return rp_b<ST_F32N64, LBM_PIPE_CO>(k, batch, src, dst, a, s);
    case ST_F32: return rp_b<ST_F32, LBM_PIPE_CO>(k, batch, src, dst, a, s);
    case ST_F16DEV: return rp_b<ST_F16DEV, LBM_PIPE_CO>(k, batch, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
