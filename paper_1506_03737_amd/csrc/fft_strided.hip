// The strided complex passes of liblpc's 3-D FFTs (see fft.hip).
#include <hip/hip_runtime.h>

#include <utility>

#include "fft_plans.h"

namespace lpc {
namespace kern {

namespace {

// ---------------------------------------------------------------------------------------------------------------
// Strided complex pass (in place). A tile is B consecutive columns (contiguous in memory) x n points along the
// axis. Within a component, tiles are XCD-remapped so that neighbouring tiles (which share cache lines at their
// edges) run on the same XCD. Each thread owns at most EPT points of its column (n B <= EPT kFftNT); with EPT <= 8
// the kernel fits in 80 VGPRs (three workgroups of 8 waves per CU where the LDS tile allows it); larger EPT gets
// 128 (a cap of 96 would also give two workgroups per CU, and spills).
template <bool INV, int B, int EPT, bool RT>
__global__ __launch_bounds__(kFftNT, (EPT <= 8) ? 6 : 4) void k_fft_axis(const AxisJob* __restrict__ jobs,
                                                        const int* __restrict__ offs, int njob, int total) {
  extern __shared__ float2 smem[];
  {
    const int w = blockIdx.x;
    const int tid = threadIdx.x;
    if (w >= total) return;
    const int jb = __builtin_amdgcn_readfirstlane(find_job(to_const(offs), njob, w));
    const LPC_CONST AxisJob& J = to_const(jobs)[jb];
    const int local = w - offs[jb];
    const int comp = local / J.per_comp;
    // XCD-contiguous chunks of 32 items rather than eighths (forward y 0.785 -> 0.759 ms at 768^3; the other strided
    // passes and the z passes measured no better that way)
    const int t = xcd_chunk_remap(local - comp * J.per_comp, J.per_comp, 32);
    const int outer = t / J.ntc, ct = t - outer * J.ntc;
    const int n = J.n;
    if (outer >= n) return;  // padding item
    const int c0 = ct * B, bw = min(B, J.ncols - c0);
    float2* tile = smem;
    float2* tw = smem + n * strided_pitch(B);
    LPC_GLOBAL float2* ptr = to_global(J.base + comp * J.cstr + outer * J.ostr + c0);
    const uint32_t astr = static_cast<uint32_t>(J.astr);  // j astr < 2^32 for every mesh up to 1024
    // the first stage reads the columns from HBM and the last writes them back: the tile holds only the stages between
    const TableRegs<float2> twr = table_load(J.tw, n, tid);
    auto load = [&](int j, int b) { return ptr[static_cast<uint32_t>(j) * astr + min(b, bw - 1)]; };
    auto mid = [&]() { table_store(tw, twr, n, tid); };
    auto store = [&](int j, int b, float2 v) {
      if (b < bw) ptr[static_cast<uint32_t>(j) * astr + b] = v;
    };
    auto none = [](int, float2 x) { return x; };
    fft_io_fast<INV, EPT, B, strided_pitch(B), true, true, false, RT>(tile, tw, J.pl, tid, load, none, mid, store);
  }
}

struct Init {
  Init() {
    allow_big_lds(k_fft_axis<false, 8, 8, false>);
    allow_big_lds(k_fft_axis<false, 8, 8, true>);
    allow_big_lds(k_fft_axis<false, 8, 12, false>);
    allow_big_lds(k_fft_axis<false, 8, 12, true>);
    allow_big_lds(k_fft_axis<false, 8, 16, false>);
    allow_big_lds(k_fft_axis<false, 8, 16, true>);
    allow_big_lds(k_fft_axis<false, 16, 8, false>);
    allow_big_lds(k_fft_axis<false, 16, 8, true>);
    allow_big_lds(k_fft_axis<false, 16, 12, false>);
    allow_big_lds(k_fft_axis<false, 16, 12, true>);
    allow_big_lds(k_fft_axis<false, 16, 16, false>);
    allow_big_lds(k_fft_axis<false, 16, 16, true>);
    allow_big_lds(k_fft_axis<false, 32, 8, false>);
    allow_big_lds(k_fft_axis<false, 32, 8, true>);
    allow_big_lds(k_fft_axis<false, 32, 12, false>);
    allow_big_lds(k_fft_axis<false, 32, 12, true>);
    allow_big_lds(k_fft_axis<false, 32, 16, false>);
    allow_big_lds(k_fft_axis<false, 32, 16, true>);
    allow_big_lds(k_fft_axis<true, 8, 8, false>);
    allow_big_lds(k_fft_axis<true, 8, 8, true>);
    allow_big_lds(k_fft_axis<true, 8, 12, false>);
    allow_big_lds(k_fft_axis<true, 8, 12, true>);
    allow_big_lds(k_fft_axis<true, 8, 16, false>);
    allow_big_lds(k_fft_axis<true, 8, 16, true>);
    allow_big_lds(k_fft_axis<true, 16, 8, false>);
    allow_big_lds(k_fft_axis<true, 16, 8, true>);
    allow_big_lds(k_fft_axis<true, 16, 12, false>);
    allow_big_lds(k_fft_axis<true, 16, 12, true>);
    allow_big_lds(k_fft_axis<true, 16, 16, false>);
    allow_big_lds(k_fft_axis<true, 16, 16, true>);
    allow_big_lds(k_fft_axis<true, 32, 8, false>);
    allow_big_lds(k_fft_axis<true, 32, 8, true>);
    allow_big_lds(k_fft_axis<true, 32, 12, false>);
    allow_big_lds(k_fft_axis<true, 32, 12, true>);
    allow_big_lds(k_fft_axis<true, 32, 16, false>);
    allow_big_lds(k_fft_axis<true, 32, 16, true>);
  }
};

}  // namespace

void init_axis() { static Init once; }

hipError_t launch_axis(const AxisJob* jobs, WorkTable wt, bool inverse, int B, int P, bool fixed_plans, size_t lds,
                       hipStream_t s) {
  init_axis();
  if (wt.total <= 0) return hipSuccess;
  const unsigned g = static_cast<unsigned>(wt.total);
#define LPC_AXIS(INV, BB, PP)                                                                              \
  {                                                                                                        \
    if (fixed_plans)                                                                                       \
      k_fft_axis<INV, BB, PP, false><<<g, kFftNT, lds, s>>>(jobs, wt.offs, wt.njob, wt.total);             \
    else                                                                                                   \
      k_fft_axis<INV, BB, PP, true><<<g, kFftNT, lds, s>>>(jobs, wt.offs, wt.njob, wt.total);              \
  }
#define LPC_AXIS_P(INV, BB) \
  if (P == 8) LPC_AXIS(INV, BB, 8) else if (P == 12) LPC_AXIS(INV, BB, 12) else if (P == 16) LPC_AXIS(INV, BB, 16) \
  else return hipErrorInvalidValue;
  if (inverse) {
    if (B == 8) { LPC_AXIS_P(true, 8) } else if (B == 16) { LPC_AXIS_P(true, 16) } else if (B == 32) { LPC_AXIS_P(true, 32) }
    else return hipErrorInvalidValue;
  } else {
    if (B == 8) { LPC_AXIS_P(false, 8) } else if (B == 16) { LPC_AXIS_P(false, 16) } else if (B == 32) { LPC_AXIS_P(false, 32) }
    else return hipErrorInvalidValue;
  }
#undef LPC_AXIS_P
#undef LPC_AXIS
  return hipGetLastError();
}

}  // namespace kern
}  // namespace lpc
