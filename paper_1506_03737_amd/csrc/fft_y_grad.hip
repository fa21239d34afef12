// The inverse y pass of the force (see fft.hip).
#include <hip/hip_runtime.h>

#include <utility>

#include "fft_plans.h"

namespace lpc {
namespace kern {

namespace {

// ---------------------------------------------------------------------------------------------------------------
// Inverse y pass of the force. Items of component 0 transform a tile of B columns of A (the x gradient) in place.
// Items of component 1 take B / 2 columns of the x-transformed potential psi from C and stack them twice in their
// tile, as i k_y psi (columns b) and as psi (columns B / 2 + b): one B-column transform gives the y gradient, stored
// to B, and psi, stored back to C (k_z is constant along y; the z pass applies i k_z as it loads C). An item reads and
// writes only its own columns, so items do not race. At 80 registers the 8-point instances with run-time stages spill 2, which
// costs less than a wave per SIMD: without the cap 100^3 takes 15.7 us instead of 12.9, 200^3 (16 columns) 47 instead of 44.
template <int B, int EPT, bool RT>
__global__ __launch_bounds__(kFftNT, EPT <= 8 ? 6 : 4) void k_fft_y_grad(
    const YGradJob* __restrict__ jobs, const int* __restrict__ offs, int njob, int total) {
  constexpr int BP = strided_pitch(B), BH = B / 2;
  extern __shared__ float2 smem[];
  const int w = blockIdx.x;
  const int tid = threadIdx.x;
  if (w >= total) return;
  const int jb = __builtin_amdgcn_readfirstlane(find_job(to_const(offs), njob, w));
  const LPC_CONST YGradJob& J = to_const(jobs)[jb];
  const int local = w - offs[jb];
  const int n = J.n;
  float2* tile = smem;
  float2* tw = smem + n * BP;
  const TableRegs<float2> twr = table_load(J.tw, n, tid);
  auto mid = [&]() { table_store(tw, twr, n, tid); };
  if (local < J.per_comp) {  // component 0 (uniform)
    const int t = xcd_remap(local, J.per_comp);
    const int outer = t / J.ntc, ct = t - outer * J.ntc;
    if (outer >= n) return;  // padding item
    const int c0 = ct * B, bw = min(B, J.ncols - c0);
    LPC_GLOBAL float2* ptr = to_global(J.A + static_cast<int64_t>(outer) * J.ostr + c0);
    const uint32_t astr = static_cast<uint32_t>(J.astr);
    auto load = [&](int j, int b) { return ptr[static_cast<uint32_t>(j) * astr + min(b, bw - 1)]; };
    auto store = [&](int j, int b, float2 v) {
      if (b < bw) ptr[static_cast<uint32_t>(j) * astr + b] = v;
    };
    auto none = [](int, float2 x) { return x; };
    fft_io_fast<true, EPT, B, BP, true, true, false, RT>(tile, tw, J.pl, tid, load, none, mid, store);
    return;
  }
  const int t = xcd_remap(local - J.per_comp, J.per_comp1);
  const int outer = t / J.ntc1, ct = t - outer * J.ntc1;
  if (outer >= n) return;  // padding item
  const int c0 = ct * BH, bw = min(BH, J.ncols - c0);
  const int64_t off = static_cast<int64_t>(outer) * J.ostr + c0;
  LPC_GLOBAL const float2* src = to_global(J.C + off);
  LPC_GLOBAL float2* dB = to_global(J.B + off);
  LPC_GLOBAL float2* dC = to_global(J.C + off);
  const uint32_t astr = static_cast<uint32_t>(J.astr);
  const int half = n / 2;
  const float kf = J.kf;
  // tile column b < BH holds i k_y psi of psi's column b, column BH + b psi itself; they go to B and back to C.
  // Each psi value is loaded once and feeds both columns.
  auto load = [&](int j, int bh) { return src[static_cast<uint32_t>(j) * astr + min(bh, bw - 1)]; };
  auto iky = [&](int j, float2 v) {
    const float ky = (j == half) ? 0.f : kf * static_cast<float>(j <= half ? j : j - n);
    return make_float2(-ky * v.y, ky * v.x);
  };
  auto store = [&](int j, int b, float2 v) {
    const int bh = b % BH;
    if (bh < bw) (b < BH ? dB : dC)[static_cast<uint32_t>(j) * astr + bh] = v;
  };
  fft_io_fast<true, EPT, B, BP, true, true, true, RT>(tile, tw, J.pl, tid, load, iky, mid, store);
}

struct Init {
  Init() {
    allow_big_lds(k_fft_y_grad<8, 8, false>);
    allow_big_lds(k_fft_y_grad<8, 8, true>);
    allow_big_lds(k_fft_y_grad<8, 12, false>);
    allow_big_lds(k_fft_y_grad<8, 12, true>);
    allow_big_lds(k_fft_y_grad<8, 16, false>);
    allow_big_lds(k_fft_y_grad<8, 16, true>);
    allow_big_lds(k_fft_y_grad<16, 8, false>);
    allow_big_lds(k_fft_y_grad<16, 8, true>);
    allow_big_lds(k_fft_y_grad<16, 12, false>);
    allow_big_lds(k_fft_y_grad<16, 12, true>);
    allow_big_lds(k_fft_y_grad<16, 16, false>);
    allow_big_lds(k_fft_y_grad<16, 16, true>);
    allow_big_lds(k_fft_y_grad<32, 8, false>);
    allow_big_lds(k_fft_y_grad<32, 8, true>);
    allow_big_lds(k_fft_y_grad<32, 12, false>);
    allow_big_lds(k_fft_y_grad<32, 12, true>);
    allow_big_lds(k_fft_y_grad<32, 16, false>);
    allow_big_lds(k_fft_y_grad<32, 16, true>);
  }
};

}  // namespace

void init_y_grad() { static Init once; }

hipError_t launch_y_grad(const YGradJob* jobs, WorkTable wt, int B, int P, bool fixed_plans, size_t lds, hipStream_t s) {
  init_y_grad();
  if (wt.total <= 0) return hipSuccess;
  const unsigned g = static_cast<unsigned>(wt.total);
#define LPC_YG(BB, PP)                                                                            \
  {                                                                                               \
    if (fixed_plans)                                                                              \
      k_fft_y_grad<BB, PP, false><<<g, kFftNT, lds, s>>>(jobs, wt.offs, wt.njob, wt.total);       \
    else                                                                                          \
      k_fft_y_grad<BB, PP, true><<<g, kFftNT, lds, s>>>(jobs, wt.offs, wt.njob, wt.total);        \
  }
#define LPC_YG_P(BB) \
  if (P == 8) LPC_YG(BB, 8) else if (P == 12) LPC_YG(BB, 12) else if (P == 16) LPC_YG(BB, 16) \
  else return hipErrorInvalidValue;
  if (B == 8) { LPC_YG_P(8) } else if (B == 16) { LPC_YG_P(16) } else if (B == 32) { LPC_YG_P(32) }
  else return hipErrorInvalidValue;
#undef LPC_YG_P
#undef LPC_YG
  return hipGetLastError();
}

}  // namespace kern
}  // namespace lpc
