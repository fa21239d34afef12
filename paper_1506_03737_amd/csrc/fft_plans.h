// Shared device code of the FFT passes (fft.hip, fft_strided.hip, fft_poisson.hip): the transforms with compile-time plans
// and the lookup of a work item's job. Included by those sources only.
#pragma once

#include <hip/hip_runtime.h>

#include "fft_device.h"

namespace lpc {
namespace kern {

// Lets the kernel take up to 160 KB of dynamic LDS. If the attribute cannot be set, a launch that asks for more than
// the default fails, and the launcher reports it through hipGetLastError.
template <class K>
inline void allow_big_lds(K kernel) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024);
}

// The transforms of the workloads' meshes (768 for the single box and the learned form's fine run, 192 / 256 / 320 for
// the batched form and the coarse run) with compile-time plans when the job's plan is one of them and the tile can
// hold it, fft_tile otherwise; both compute the same stages with the same twiddle table. HALF selects the plans of the
// half-length z transforms, otherwise those of the full-length x and y transforms; a kernel carries only its own kind.
template <class F, class PL>
__device__ __forceinline__ bool try_fixed(float2* tile, const float2* tw, const PL& pl, int tid) {
  if (!F::matches(pl)) return false;
  F::run(tile, tw, tid);
  return true;
}

template <bool INV, int EPT, int B, int BP, bool HALF, bool R12 = true, class PL>
__device__ __forceinline__ void fft_tile_fast(float2* tile, const float2* tw, const PL& pl, int tid) {
  // full-length plans (make_plan): 768 = 8 x 8 x 12, 320 = 8 x 8 x 5, 256 = 8 x 8 x 4, 192 = 8 x 8 x 3;
  // half-length with radix 12: 384 = 4 x 8 x 12, 160 = 8 x 4 x 5, 128 = 4 x 4 x 8, 96 = 8 x 12;
  // half-length without radix 12: 384 = 4 x 4 x 8 x 3, 160, 128 as above, 96 = 8 x 4 x 3
  if constexpr (!HALF) {
    if (try_fixed<FixedFFT<INV, EPT, B, BP, 8, 8, 12>>(tile, tw, pl, tid)) return;
    if (try_fixed<FixedFFT<INV, EPT, B, BP, 8, 8, 5>>(tile, tw, pl, tid)) return;
    if (try_fixed<FixedFFT<INV, EPT, B, BP, 8, 8, 4>>(tile, tw, pl, tid)) return;
    if (try_fixed<FixedFFT<INV, EPT, B, BP, 8, 8, 3>>(tile, tw, pl, tid)) return;
  } else {
    if constexpr (R12) {
      if (try_fixed<FixedFFT<INV, EPT, B, BP, 4, 8, 12>>(tile, tw, pl, tid)) return;
      if (try_fixed<FixedFFT<INV, EPT, B, BP, 8, 12>>(tile, tw, pl, tid)) return;
    } else {
      if (try_fixed<FixedFFT<INV, EPT, B, BP, 4, 4, 8, 3>>(tile, tw, pl, tid)) return;
      if (try_fixed<FixedFFT<INV, EPT, B, BP, 8, 4, 3>>(tile, tw, pl, tid)) return;
    }
    if (try_fixed<FixedFFT<INV, EPT, B, BP, 8, 4, 5>>(tile, tw, pl, tid)) return;
    if (try_fixed<FixedFFT<INV, EPT, B, BP, 4, 4, 8>>(tile, tw, pl, tid)) return;
  }
  fft_tile<INV, EPT, R12>(tile, tw, pl, B, BP, tid);
}

// fft_io_fast for any plan, with run-time stages. (Filling the tile, transforming it in place and storing it from there
// took two more passes over it and two more barriers; per force evaluation at 270^3 the inverse y pass 164 -> 142 us, at
// 512^3 1021 -> 663, at 600^3 1892 -> 1425; the forward y pass 5 to 12 % less.)
template <bool INV, int EPT, int B, int BP, bool GIN, bool GOUT, bool PAIRS, class PL, class Load, class Pair, class Mid,
          class Store>
__device__ __forceinline__ void fft_io_runtime(float2* tile, const float2* tw, const PL& pl, int tid, Load load, Pair pair,
                                               Mid mid, Store store) {
  const int n = pl.n, last = pl.nst - 1;
  const TileGeom g(B, BP, tid);
  int s0 = 0, s1 = pl.nst;
  if (last == 0) {  // a single stage (8 and 12 points) fills the tile and stores from it
    const int count = n * B;
    if constexpr (GIN) {
      for (int e = tid; e < count; e += kFftNT) {
        const int j = e / B, b = e % B;
        if constexpr (PAIRS) {
          const float2 x = load(j, b % (B / 2));
          tile[j * BP + b] = (b < B / 2) ? pair(j, x) : x;
        } else {
          tile[j * BP + b] = load(j, b);
        }
      }
      mid();
      __syncthreads();
    }
    fft_tile<INV, EPT, true>(tile, tw, pl, B, BP, tid);
    if constexpr (GOUT)
      for (int e = tid; e < count; e += kFftNT) store(e / B, e % B, tile[(e / B) * BP + (e % B)]);
    return;
  }
  if constexpr (GIN) {
    s0 = 1;
#define LPC_FIRST(R)                                                                  \
  {                                                                                   \
    if constexpr (PAIRS)                                                              \
      fft_stage_load_pairs<R, INV, EPT>(tile, n, B, BP, tid, load, pair, mid);        \
    else                                                                              \
      fft_stage_load<R, INV, EPT>(tile, n, g, load, mid);                             \
    break;                                                                            \
  }
    switch (pl.radix[0]) {
      case 8: LPC_FIRST(8)
      case 12: LPC_FIRST(12)
      case 4: LPC_FIRST(4)
      case 2: LPC_FIRST(2)
      case 3: LPC_FIRST(3)
      default: LPC_FIRST(5)
    }
#undef LPC_FIRST
  }
  if constexpr (GOUT) s1 = last;
  fft_tile_stages<INV, EPT, true>(tile, tw, pl, B, BP, tid, s0, s1);
  if constexpr (GOUT) {
    const float2* tws = tw + pl.tw_off[last];
    const int p = pl.p[last], pm = pl.pmask[last];
    switch (pl.radix[last]) {
      case 8: fft_stage_store<8, INV, EPT>(tile, tws, n, p, pm, g, store); break;
      case 12: fft_stage_store<12, INV, EPT>(tile, tws, n, p, pm, g, store); break;
      case 4: fft_stage_store<4, INV, EPT>(tile, tws, n, p, pm, g, store); break;
      case 2: fft_stage_store<2, INV, EPT>(tile, tws, n, p, pm, g, store); break;
      case 3: fft_stage_store<3, INV, EPT>(tile, tws, n, p, pm, g, store); break;
      default: fft_stage_store<5, INV, EPT>(tile, tws, n, p, pm, g, store); break;
    }
  }
}

// fft_tile_fast with the tile's fill and drain folded into the first and last stages: with GIN the input comes from
// load(row, col) (the tile is not filled first; mid() runs while the first loads are in flight), with GOUT the
// output goes to store(row, col, value). Full-length transforms; plans other than the compiled ones run the same stages
// with run-time lengths. The twiddles in tw must be in LDS by the first barrier (mid() may write them).
template <class F, class PL, bool GIN, bool GOUT, bool PAIRS, class Load, class Pair, class Mid, class Store>
__device__ __forceinline__ bool try_fixed_io(float2* tile, const float2* tw, const PL& pl, int tid, Load load,
                                             Pair pair, Mid mid, Store store) {
  if (!F::matches(pl)) return false;
  F::template run_io<GIN, GOUT, PAIRS>(tile, tw, tid, load, pair, mid, store);
  return true;
}

// PAIRS: tile column b < B / 2 is pair(row, x) and column b + B / 2 is x itself, for x = load(row, b) of a B / 2
// column source (load takes source columns only). Columns transform independently, so for a column that store skips
// (past the mesh edge) load may return any finite value: the kernels reload the item's last column there instead of
// predicating the load and clearing its register.
// RT false: only the compiled plans (has_fixed_plan) are in the instance; the run-time stages' registers would otherwise
// cost those plans' kernels their own (768^3: forward y 0.753 -> 0.795 ms, inverse y 2.24 -> 2.31).
template <bool INV, int EPT, int B, int BP, bool GIN, bool GOUT, bool PAIRS = false, bool RT = true, class PL, class Load,
          class Pair, class Mid, class Store>
__device__ __forceinline__ void fft_io_fast(float2* tile, const float2* tw, const PL& pl, int tid, Load load, Pair pair,
                                            Mid mid, Store store) {
#define LPC_TRY_IO(...)                                                                                          \
  if (try_fixed_io<FixedFFT<INV, EPT, B, BP, __VA_ARGS__>, PL, GIN, GOUT, PAIRS>(tile, tw, pl, tid, load, pair, mid, \
                                                                             store))                             \
    return;
  LPC_FIXED_PLANS(LPC_TRY_IO)
#undef LPC_TRY_IO
  if constexpr (RT)
    fft_io_runtime<INV, EPT, B, BP, GIN, GOUT, PAIRS>(tile, tw, pl, tid, load, pair, mid, store);
}

// Job of work item w: the last j with offs[j] <= w (binary search; offs is uniform, so scalar loads).
__device__ __forceinline__ int find_job(const LPC_CONST int* __restrict__ offs, int njob, int w) {
  int lo = 0, hi = njob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (offs[mid] <= w)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

}  // namespace kern
}  // namespace lpc
