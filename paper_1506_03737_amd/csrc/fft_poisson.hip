// The fused x pass of the force (see fft.hip): forward x transform, Poisson factor, two inverse x transforms.
#include <hip/hip_runtime.h>

#include <utility>

#include "fft_plans.h"

namespace lpc {
namespace kern {

namespace {

// ---------------------------------------------------------------------------------------------------------------
// A compile-time plan (radices Rs in order, or reversed with REV): stage s has radix r(s), sub-transform length p(s)
// and its twiddles at off(s) of the plan's table (the layout make_plan gives it).
template <bool REV, int... Rs>
struct ChainPlan {
  static constexpr int K = sizeof...(Rs);
  static constexpr int N = (Rs * ...);
  static constexpr int fwd[K] = {Rs...};
  static constexpr int r(int s) { return REV ? fwd[K - 1 - s] : fwd[s]; }
  static constexpr int p(int s) {
    int q = 1;
    for (int t = 0; t < s; ++t) q *= r(t);
    return q;
  }
  static constexpr int off(int s) {
    int o = 0;
    for (int t = 0; t < s; ++t) o += p(t) * (r(t) - 1);
    return o;
  }
};

// Stages 1 .. K - 2 of plan CP in the tile.
template <class CP, bool INV, int EPT, int B, int BP, int... S>
__device__ __forceinline__ void chain_mid_stages(float2* tile, const float2* tw, int tid,
                                                 std::integer_sequence<int, S...>) {
  (fft_stage_c<CP::r(S + 1), INV, EPT, CP::N, CP::p(S + 1), B, BP>(tile, tw + CP::off(S + 1), tid), ...);
}

// The fused x pass on 8-column tiles with its three transforms chained through registers, for the plans 8 x 8 x R
// (R = 12, 5, 4, 3: meshes 768, 320, 256, 192) and 4 x 4 x 8 x 8 (1024). The forward transform's last stage (radix
// RL) leaves each thread's MB butterflies in its registers: thread (i, b) = (tid / 8, tid % 8) holds rows
// i + m 64 + r N / RL of column b, in natural order (MB = 1 for 8 x 8 x R, 2 for 1024). factor(row, g, ph) turns each
// into psi_hat (ph) and i k_x psi_hat (g) there. Both inverse transforms run the plan in reverse order, whose first
// stage (radix RL) takes exactly those rows, so neither spectrum goes back through the tile between the transforms:
// for 768, 12 LDS passes and 9 barriers per tile instead of 18 and 15. The reversed plan's twiddles wait in registers
// (r_twr) and replace the forward ones in LDS once the forward transform has read them, so one table's worth of LDS
// serves both (at 1024 that lets two workgroups share a CU).
template <int M, int... Rs, class PL, class Load, class Mid, class MakeFactor, class StoreA, class StoreC>
__device__ __forceinline__ bool x_poisson_chained(float2* tile, float2* tw, const TableRegs<float2>& r_twr,
                                                  const PL& pl, int tid, Load load, Mid mid, MakeFactor make_factor,
                                                  StoreA store_a, StoreC store_c) {
  constexpr int B = 8, BP = strided_pitch(B);
  using Fwd = FixedFFT<false, M, B, BP, Rs...>;
  if constexpr (!Fwd::kFits) {
    return false;
  } else {
    if (!Fwd::matches(pl)) return false;
    using F = ChainPlan<false, Rs...>;
    using V = ChainPlan<true, Rs...>;
    constexpr int N = F::N, K = F::K, RF = F::r(0), RL = F::r(K - 1);
    constexpr int MB = (N / RL) * B / kFftNT;
    static_assert(MB * kFftNT == (N / RL) * B, "the last stage's butterflies split evenly over the threads");
    using Mids = std::make_integer_sequence<int, K - 2>;
    // forward: the first stage from HBM, the middle stages in the tile, the last into registers
    fft_stage_from_global<RF, false, M, N, B, BP>(tile, load, mid, tid);
    __syncthreads();
    chain_mid_stages<F, false, M, B, BP>(tile, tw, tid, Mids{});
    float2 g[MB][RL], ph[MB][RL];
    fft_stage_to_regs<RL, false, N, F::p(K - 1), B, BP, MB>(tile, tw + F::off(K - 1), tid, g);
    {
      const auto factor = make_factor();
      const int i0 = tid / B;
#pragma unroll
      for (int m = 0; m < MB; ++m) {
#pragma unroll
        for (int r = 0; r < RL; ++r) factor(i0 + m * (kFftNT / B) + r * (N / RL), g[m][r], ph[m][r]);
      }
    }
    __syncthreads();  // the tile and the forward twiddles have been read
    table_store(tw, r_twr, N, tid);
    // first inverse: i k_x psi_hat -> the x gradient in A
    fft_stage_from_regs<RL, true, N, B, BP, MB>(tile, g, tid);
    __syncthreads();
    chain_mid_stages<V, true, M, B, BP>(tile, tw, tid, Mids{});
    fft_stage_to_global<RF, true, M, N, V::p(K - 1), B, BP>(tile, tw + V::off(K - 1), store_a, tid);
    __syncthreads();
    // second inverse: psi_hat -> the x-transformed potential in C
    fft_stage_from_regs<RL, true, N, B, BP, MB>(tile, ph, tid);
    __syncthreads();
    chain_mid_stages<V, true, M, B, BP>(tile, tw, tid, Mids{});
    fft_stage_to_global<RF, true, M, N, V::p(K - 1), B, BP>(tile, tw + V::off(K - 1), store_c, tid);
    return true;
  }
}

// Fused x pass of the force. With psi_hat = -delta_hat / (k^2 W^p Nm^3) (zero at k = 0; W = prod_d sinc^2(pi n_d /
// Nm); the 1/Nm^3 of the inverse transform folded in), the gradient spectra are g_hat_j = i k_j psi_hat, zero on the
// Nyquist plane of axis j. Along the x transform k_y and k_z are constant (per tile and per column), so
//   IFFT_x(g_hat_x) = IFFT_x(i k_x psi_hat) -> A,   IFFT_x(g_hat_{y,z}) = i k_{y,z} IFFT_x(psi_hat), IFFT_x(psi_hat) -> C:
// one forward and two inverse transforms per tile, two spectra written. psi_hat is kept between them. The CHAIN
// instances (B = 8, M <= 12) run every job's transforms chained through registers (x_poisson_chained): the host
// launches them only when every job's plan is 8 x 8 x R (poisson_chainable). Otherwise each thread owns the points of
// column b at rows j0 + m S, at most M of them (M = n B / kFftNT rounded up to 8, 12 or 16): with M <= 12 they stay
// in the thread's registers, so the workgroup needs one LDS tile and two workgroups fit on a CU; with M = 16 a second
// LDS tile holds them (the registers would spill). The two forms are separate instances because the generic form's
// register allocation would otherwise cover the chained form's too (and spill). The chained M = 8 instance (the
// 192-320 meshes) is capped at 80 VGPRs, so that three workgroups fit on a CU (48-box step 30.86 -> 30.25 ms).
// RT false: every job's plan is compiled in (has_fixed_plan), and the instance has no run-time stages, whose registers cost
// the compiled ones theirs (384^3, the one such mesh side that does not chain: 204 -> 193 us).
template <int B, int M, bool CHAIN, bool RT>
__global__ __launch_bounds__(kFftNT, (CHAIN && M <= 8) ? 6 : ((CHAIN || M <= 12) ? 4 : 2)) void k_fft_x_poisson(
    const PoissonJob* __restrict__ jobs, const int* __restrict__ offs, int njob, int total) {
  constexpr int BP = strided_pitch(B), S = kFftNT / B;
  constexpr bool kRegs = CHAIN || M <= 12;  // psi_hat in registers (else a second LDS tile)
  extern __shared__ float2 smem[];
  {
    const int w = blockIdx.x;
    const int tid = threadIdx.x;
    if (w >= total) return;
    const int jb = __builtin_amdgcn_readfirstlane(find_job(to_const(offs), njob, w));
    const LPC_CONST PoissonJob& J = to_const(jobs)[jb];
    const int n = J.nm, nm = J.nm, nh = nm / 2 + 1, pitch = J.pitch;
    const int t = xcd_remap(w - offs[jb], offs[jb + 1] - offs[jb]);
    const int y = t / J.ntc, ct = t - y * J.ntc;
    if (y >= n) return;  // padding item
    float2* tile = smem;
    float2* ph_lds = tile + n * BP;  // psi_hat when !kRegs
    float2* tw = tile + (kRegs ? 1 : 2) * n * BP;
    float* win = reinterpret_cast<float*>(tw + n);  // sinc^2(pi m / n), m <= n / 2 (even in m)
    const int c0 = ct * B, bw = min(B, nh - c0);
    const uint32_t astr = static_cast<uint32_t>(nm) * static_cast<uint32_t>(pitch);  // j astr < 2^32 (Nm <= 1024)
    const int64_t off = static_cast<int64_t>(y) * pitch + c0;
    LPC_GLOBAL float2* gA = to_global(J.A + off);
    LPC_GLOBAL float2* gC = to_global(J.C + off);
    const int half = nm / 2;
    const int ny = (y <= half) ? y : y - nm;
    const float kf = J.kf, inv_m3 = J.inv_m3;
    const int deconv = J.deconv;
    // The Poisson factor of this thread's column b = tid % B (read once the window table is in LDS):
    // factor(j, g, ph) takes the forward spectrum at row j in g and leaves psi_hat in ph and i k_x psi_hat in g.
    auto make_factor = [&]() {
      const int b = tid % B, nz = c0 + b;
      const bool col_ok = b < bw;
      const float wyz = win[min(y, n - y)] * win[min(nz, half)];
      const int nyz2 = ny * ny + nz * nz;
      return [=](int j, float2& g, float2& ph) {
        const int nx = (j <= half) ? j : j - nm;
        const float k2 = kf * kf * static_cast<float>(nx * nx + nyz2);
        float sc = 0.f;
        if (k2 > 0.f && col_ok) {
          const float W = win[min(j, n - j)] * wyz;
          const float wp = (deconv == 0) ? 1.f : (deconv == 1 ? W : W * W);
          sc = -inv_m3 * __builtin_amdgcn_rcpf(k2 * wp);  // hardware reciprocal (1 ulp) instead of a division
        }
        ph = make_float2(sc * g.x, sc * g.y);
        const float kx = (nx == half) ? 0.f : kf * static_cast<float>(nx);
        g = make_float2(-kx * ph.y, kx * ph.x);
      };
    };
    auto load = [&](int j, int b) { return gA[static_cast<uint32_t>(j) * astr + min(b, bw - 1)]; };
    auto store_a = [&](int j, int b, float2 v) {
      if (b < bw) gA[static_cast<uint32_t>(j) * astr + b] = v;
    };
    auto store_c = [&](int j, int b, float2 v) {
      if (b < bw) gC[static_cast<uint32_t>(j) * astr + b] = v;
    };
    if constexpr (CHAIN) {
      static_assert(B == 8, "the chained form takes 8-column tiles");
      // the tables' loads go out first; mid() writes the forward twiddles and the window to LDS while the first
      // stage's loads are in flight, the reversed plan's twiddles stay in registers until the forward pass is done
      const TableRegs<float2> r_tw = table_load(J.tw, n, tid), r_twr = table_load(J.tw_rev, n, tid);
      const TableRegs<float> r_win = table_load(J.win, n / 2 + 1, tid);
      auto mid = [&]() {
        table_store(tw, r_tw, n, tid);
        table_store(win, r_win, n / 2 + 1, tid);
      };
#define LPC_CHAIN(...) \
  if (x_poisson_chained<M, __VA_ARGS__>(tile, tw, r_twr, J.pl, tid, load, mid, make_factor, store_a, store_c)) return;
      LPC_CHAINED_PLANS(LPC_CHAIN)
#undef LPC_CHAIN
      return;
    } else {
      auto none = [](int, float2 x) { return x; };
      auto nothing = []() {};
      auto no_load = [](int, int) { return make_float2(0.f, 0.f); };
      auto no_store = [](int, int, float2) {};
      {
        // forward transform: the first stage reads delta_hat from HBM; the tables are copied while its loads are in
        // flight; the result stays in the tile (natural order)
        const TableRegs<float2> r_tw = table_load(J.tw, n, tid);
        const TableRegs<float> r_win = table_load(J.win, n / 2 + 1, tid);
        auto mid = [&]() {
          table_store(tw, r_tw, n, tid);
          table_store(win, r_win, n / 2 + 1, tid);
        };
        fft_io_fast<false, M, B, BP, true, false, false, RT>(tile, tw, J.pl, tid, load, none, mid, no_store);
      }

      // Each thread touches only its own points between the barriers that bracket the inverse transforms.
      float2 ph[kRegs ? M : 1];
      {
        const auto factor = make_factor();
        const int b = tid % B, j0 = tid / B;
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int j = j0 + m * S;
          if (j >= n) continue;
          float2 g = tile[j * BP + b], psi;
          factor(j, g, psi);
          if (kRegs)
            ph[kRegs ? m : 0] = psi;
          else
            ph_lds[j * BP + b] = psi;
          tile[j * BP + b] = g;  // i k_x psi_hat
        }
      }
      __syncthreads();
      // first inverse transform: the last stage writes the x gradient to A
      fft_io_fast<true, M, B, BP, false, true, false, RT>(tile, tw, J.pl, tid, no_load, none, nothing, store_a);
      __syncthreads();
      {
        // (the empty asm keeps the comp-invariant indices of the first inverse transform from staying live)
        int ltid = tid;
        asm volatile("" : "+v"(ltid));
        const int b = ltid % B, j0 = ltid / B;
#pragma unroll
        for (int m = 0; m < M; ++m) {
          const int j = j0 + m * S;
          if (j < n) tile[j * BP + b] = kRegs ? ph[kRegs ? m : 0] : ph_lds[j * BP + b];
        }
        __syncthreads();
        // the x-transformed potential: the y and z gradients are i k_y and i k_z times it (applied by the y and z
        // passes); the last stage writes it to C
        fft_io_fast<true, M, B, BP, false, true, false, RT>(tile, tw, J.pl, ltid, no_load, none, nothing, store_c);
      }
    }
  }
}

struct Init {
  Init() {
    allow_big_lds(k_fft_x_poisson<8, 8, true, false>);
    allow_big_lds(k_fft_x_poisson<8, 12, true, false>);
    allow_big_lds(k_fft_x_poisson<8, 16, true, false>);
    allow_big_lds(k_fft_x_poisson<4, 8, false, false>);
    allow_big_lds(k_fft_x_poisson<4, 8, false, true>);
    allow_big_lds(k_fft_x_poisson<8, 8, false, false>);
    allow_big_lds(k_fft_x_poisson<8, 8, false, true>);
    allow_big_lds(k_fft_x_poisson<8, 12, false, false>);
    allow_big_lds(k_fft_x_poisson<8, 12, false, true>);
    allow_big_lds(k_fft_x_poisson<8, 16, false, false>);
    allow_big_lds(k_fft_x_poisson<8, 16, false, true>);
    allow_big_lds(k_fft_x_poisson<16, 8, false, false>);
    allow_big_lds(k_fft_x_poisson<16, 8, false, true>);
    allow_big_lds(k_fft_x_poisson<16, 12, false, false>);
    allow_big_lds(k_fft_x_poisson<16, 12, false, true>);
    allow_big_lds(k_fft_x_poisson<16, 16, false, false>);
    allow_big_lds(k_fft_x_poisson<16, 16, false, true>);
  }
};

}  // namespace

void init_poisson() { static Init once; }

hipError_t launch_poisson(const PoissonJob* jobs, WorkTable wt, int B, int M, bool chained, bool fixed_plans, size_t lds,
                          hipStream_t s) {
  init_poisson();
  if (wt.total <= 0) return hipSuccess;
  const unsigned g = static_cast<unsigned>(wt.total);
#define LPC_POIS(BB, MM, CC, RR) k_fft_x_poisson<BB, MM, CC, RR><<<g, kFftNT, lds, s>>>(jobs, wt.offs, wt.njob, wt.total)
#define LPC_POIS_P(BB, MM)                  \
  {                                         \
    if (fixed_plans)                        \
      LPC_POIS(BB, MM, false, false);       \
    else                                    \
      LPC_POIS(BB, MM, false, true);        \
  }
  if (chained) {
    if (B == 8 && M == 8) LPC_POIS(8, 8, true, false);
    else if (B == 8 && M == 12) LPC_POIS(8, 12, true, false);
    else if (B == 8 && M == 16) LPC_POIS(8, 16, true, false);
    else return hipErrorInvalidValue;
  }
  else if (B == 4 && M == 8) LPC_POIS_P(4, 8)
  else if (B == 8 && M == 8) LPC_POIS_P(8, 8)
  else if (B == 8 && M == 12) LPC_POIS_P(8, 12)
  else if (B == 8 && M == 16) LPC_POIS_P(8, 16)
  else if (B == 16 && M == 8) LPC_POIS_P(16, 8)
  else if (B == 16 && M == 12) LPC_POIS_P(16, 12)
  else if (B == 16 && M == 16) LPC_POIS_P(16, 16)
  else return hipErrorInvalidValue;
#undef LPC_POIS_P
#undef LPC_POIS
  return hipGetLastError();
}

}  // namespace kern
}  // namespace lpc
