// Clustering statistics of a periodic box, from the half spectrum delta_hat of the CIC density contrast:
//  * the binned power spectrum (the cubic-box form of the FKP estimator used in Sec. 7.1 of Howlett, Manera &
//    Percival 2015): P = V |delta_hat|^2 / (Nm^6 W^2) per mode with one CIC window W = prod sinc^2 removed, averaged
//    in linear |k| bins. Per-bin sums are FP64 and the mode counts exact integers;
//  * the FFT shell estimator of the reduced bispectrum (Sec. 7.2): inverse transforms of shell-filtered spectra
//    (delta_hat / W or the shell indicator), block sums of the product of three of those fields, and block sums of the
//    shell power. Every block writes its own FP64 partial sum and the partial sums are added in a fixed order, so the
//    totals do not depend on scheduling.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "fft_device.h"

namespace lpc {
namespace kern {

namespace {

// Binning: a thread takes kRun consecutive kz of the modes (+-nx, +-ny, kz), which share |k|, the bin and the window, and
// adds up a run of one bin in registers before it goes to the block's bins in LDS. (One mode at a time, each with its own
// FP64 root, division and three LDS atomics, whose lanes mostly met in a few bins, 512^3 took 0.29 ms; the reading of
// the spectrum alone takes 0.11.)
constexpr int kRun = 8;
constexpr int kRunsPerThread = 2;

__global__ __launch_bounds__(kNT) void k_pk_bin(const float2* __restrict__ spec, const double* __restrict__ window, int nm,
                                                int pitch, double kf, double dk, int n_bins, double pscale,
                                                double* __restrict__ sums, unsigned long long* __restrict__ counts) {
  extern __shared__ double lds[];
  const int half = nm / 2, nh = half + 1;
  double* sk = lds;
  double* sp = sk + n_bins;
  double* win = sp + n_bins;
  unsigned* sc = reinterpret_cast<unsigned*>(win + nh);
  for (int b = threadIdx.x; b < n_bins; b += kNT) {
    sk[b] = 0.0;
    sp[b] = 0.0;
    sc[b] = 0u;
  }
  for (int m = threadIdx.x; m < nh; m += kNT) win[m] = window[m];
  __syncthreads();
  const int nseg = (nh + kRun - 1) / kRun, items = nh * nh * nseg;
  for (int t = 0; t < kRunsPerThread; ++t) {
    const int e = (static_cast<int>(blockIdx.x) * kRunsPerThread + t) * kNT + static_cast<int>(threadIdx.x);
    if (e >= items) break;
    const int r = e / nseg, kz0 = (e - r * nseg) * kRun;
    const int nx = r / nh, ny = r - nx * nh;
    // the rows of (+-nx, +-ny); a sign that gives the same row again is left out
    const int ex = (nx == 0 || nx == half) ? 1 : 2, ey = (ny == 0 || ny == half) ? 1 : 2;
    const float4* row[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kx = (q >> 1) && ex == 2 ? nm - nx : nx, ky = (q & 1) && ey == 2 ? nm - ny : ny;
      row[q] = reinterpret_cast<const float4*>(spec + (static_cast<size_t>(kx) * nm + ky) * pitch + kz0);
    }
    const double wxy = win[nx] * win[ny];
    const int nxy2 = nx * nx + ny * ny, modes = ex * ey;
    int bin = -1;
    double ak = 0.0, ap = 0.0;
    unsigned ac = 0;
    auto flush = [&]() {
      if (bin >= 0) {
        atomicAdd(sk + bin, ak);
        atomicAdd(sp + bin, ap);
        atomicAdd(sc + bin, ac);
      }
    };
#pragma unroll
    for (int j = 0; j < kRun / 2; ++j) {
      float4 v[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = row[q][j];  // (rows are padded to whole runs)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int kz = kz0 + 2 * j + i;
        const int n2 = nxy2 + kz * kz;
        if (kz > half || n2 == 0) continue;
        const double k = kf * sqrt(static_cast<double>(n2));
        const int b = static_cast<int>(floor(k / dk));
        if (b >= n_bins) break;  // |k| grows along the run
        double p2 = 0.0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (((q >> 1) && ex == 1) || ((q & 1) && ey == 1)) continue;
          const double re = i ? v[q].z : v[q].x, im = i ? v[q].w : v[q].y;
          p2 += re * re + im * im;
        }
        const double W = wxy * win[kz];
        const int mult = (kz > 0 && kz < half) ? 2 : 1;
        if (b != bin) {
          flush();
          bin = b;
          ak = ap = 0.0;
          ac = 0u;
        }
        ak += mult * modes * k;
        ap += mult * pscale * p2 / (W * W);
        ac += static_cast<unsigned>(mult * modes);
      }
    }
    flush();
  }
  __syncthreads();
  for (int b = threadIdx.x; b < n_bins; b += kNT) {
    if (sc[b] != 0u) {
      atomicAdd(sums + 2 * b, sk[b]);
      atomicAdd(sums + 2 * b + 1, sp[b]);
      atomicAdd(counts + b, static_cast<unsigned long long>(sc[b]));
    }
  }
}

constexpr int kSumBlocks = 256;  // blocks (and FP64 partial sums) of the reductions below

// ---------------------------------------------------------------------------------------------------------------
// Shell-filtered fields of the bispectrum. A field is one distinct (shell, filter) pair of a group of triangles; the
// inverse transforms of all of a group's fields run as one launch per axis, and a triangle's product is summed in the z
// pass, so that no real field is stored. (One triangle at a time, with a filling pass, three transform passes and a
// product pass per field, six triangles on 128^3 took 174 launches and 2.2 ms: launches, not bytes, bound them.)
// A shell holds modes with |n| <= nmax only: the x pass leaves the columns outside it alone, the y pass takes them as
// zero, and no pass touches kz > nmax.

// Columns of a tile at length n: 16 up to 256 points (8 points per thread), then 8 (8 to 512, 16 to 1024).
__host__ __device__ constexpr int shell_cols(int n) { return n <= 256 ? 16 : 8; }

// The x pass of field blockIdx.y: delta_hat / W (or 1) inside the shell, transformed along x, for the columns of one ky.
template <int B, int M>
__global__ __launch_bounds__(kFftNT, M <= 8 ? 4 : 2) void k_shell_x(ShellPasses a, const ShellField* __restrict__ fields) {
  constexpr int BP = strided_pitch(B), S = kFftNT / B;
  extern __shared__ float2 smem[];
  const LPC_CONST ShellField& f = to_const(fields)[blockIdx.y];
  const int tid = threadIdx.x, n = a.n, half = n / 2;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const int y = t / a.ntc, c0 = (t - y * a.ntc) * B;
  const int ny = y <= half ? y : y - n;
  if (c0 > f.nmax || ny * ny + c0 * c0 >= f.n2hi) return;  // no mode of the shell (uniform)
  float2* tile = smem;
  float2* tw = tile + n * BP;
  const TableRegs<float2> r_tw = table_load(a.tw, n, tid);
  const int b = tid % B, j0 = tid / B, nz = c0 + b;
  const uint32_t astr = static_cast<uint32_t>(n) * static_cast<uint32_t>(a.pitch);
  const size_t off = static_cast<size_t>(y) * a.pitch + nz;
  const int nyz2 = ny * ny + nz * nz;
  float2 v[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int j = j0 + m * S;
    v[m] = make_float2(0.f, 0.f);
    const int nx = j <= half ? j : j - n;
    const int n2 = nx * nx + nyz2;
    if (j < n && nz <= half && n2 >= f.n2lo && n2 < f.n2hi) {
      v[m].x = 1.f;
      if (!f.indicator) {
        const float2 d = a.spec[off + static_cast<uint32_t>(j) * astr];
        const double W = a.win[min(j, n - j)] * a.win[min(y, n - y)] * a.win[nz];
        v[m] = make_float2(static_cast<float>(static_cast<double>(d.x) / W),
                           static_cast<float>(static_cast<double>(d.y) / W));
      }
    }
  }
  table_store(tw, r_tw, n, tid);
#pragma unroll
  for (int m = 0; m < M; ++m)
    if (j0 + m * S < n) tile[(j0 + m * S) * BP + b] = v[m];
  __syncthreads();
  fft_tile<true, M>(tile, tw, a.pl, B, BP, tid);
  const bool col = nz <= min(f.nmax, half);
  LPC_GLOBAL float2* out = to_global(f.mesh);
#pragma unroll
  for (int m = 0; m < M; ++m)
    if (j0 + m * S < n && col) out[off + static_cast<uint32_t>(j0 + m * S) * astr] = tile[(j0 + m * S) * BP + b];
}

// The y pass of field blockIdx.y, in place, for the columns of one x.
template <int B, int M>
__global__ __launch_bounds__(kFftNT, M <= 8 ? 4 : 2) void k_shell_y(ShellPasses a, const ShellField* __restrict__ fields) {
  constexpr int BP = strided_pitch(B), S = kFftNT / B;
  extern __shared__ float2 smem[];
  const LPC_CONST ShellField& f = to_const(fields)[blockIdx.y];
  const int tid = threadIdx.x, n = a.n, half = n / 2;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const int x = t / a.ntc, c0 = (t - x * a.ntc) * B;
  if (c0 > f.nmax) return;  // no column of the shell (uniform)
  float2* tile = smem;
  float2* tw = tile + n * BP;
  const TableRegs<float2> r_tw = table_load(a.tw, n, tid);
  const int b = tid % B, j0 = tid / B, nz = c0 + b;
  const bool col = nz <= min(f.nmax, half);
  LPC_GLOBAL float2* mesh = to_global(f.mesh) + static_cast<size_t>(x) * n * a.pitch + nz;
  float2 v[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int j = j0 + m * S;
    const int ny = j <= half ? j : j - n;
    v[m] = make_float2(0.f, 0.f);  // where the x pass left the column alone
    if (j < n && col && ny * ny + c0 * c0 < f.n2hi) v[m] = mesh[static_cast<uint32_t>(j) * a.pitch];
  }
  table_store(tw, r_tw, n, tid);
#pragma unroll
  for (int m = 0; m < M; ++m)
    if (j0 + m * S < n) tile[(j0 + m * S) * BP + b] = v[m];
  __syncthreads();
  fft_tile<true, M>(tile, tw, a.pl, B, BP, tid);
#pragma unroll
  for (int m = 0; m < M; ++m)
    if (j0 + m * S < n && col) mesh[static_cast<uint32_t>(j0 + m * S) * a.pitch] = tile[(j0 + m * S) * BP + b];
}

// The z pass and the product sum of triple blockIdx.y: R rows of its nc distinct fields at a time become real rows in the
// tile (column r nc + c), whose product over the triple is summed in FP64. Block b takes every kSumBlocks-th group of
// rows from b on and writes one partial sum. Each thread owns at most kShellUnits (row, point pair) units.
constexpr int kShellUnits = 2;
__global__ __launch_bounds__(kFftNT, 4) void k_shell_z(ShellPasses a, const ShellField* __restrict__ fields,
                                                       const ShellTriple* __restrict__ triples) {
  extern __shared__ float2 smem[];
  __shared__ double sums[kFftNT / 64];
  const LPC_CONST ShellTriple& q = to_const(triples)[blockIdx.y];
  const int tid = threadIdx.x, n = a.n, h = n / 2, nrows = n * n, R = a.R, nc = q.nc;
  const int B = nc * R, BP = B | 1;
  float2* tile = smem;               // (h + 1) x BP
  float2* tw = tile + (h + 1) * BP;
  float2* roots = tw + h;
  const TableRegs<float2> r_tw = table_load(a.twh, h, tid), r_roots = table_load(a.roots, h + 1, tid);
  table_store(tw, r_tw, h, tid);
  table_store(roots, r_roots, h + 1, tid);
  double acc = 0.0;
  for (int row0 = blockIdx.x * R; row0 < nrows; row0 += kSumBlocks * R) {
    const int rows = min(R, nrows - row0);
    __syncthreads();  // the previous rows have been summed
    for (int c = 0; c < nc; ++c) {
      const LPC_CONST ShellField& f = to_const(fields)[q.field[c]];
      LPC_GLOBAL const float2* mesh = to_global(f.mesh) + static_cast<size_t>(row0) * a.pitch;
      const int nmax = f.nmax;
      for (int e = tid; e < rows * (h + 1); e += kFftNT) {
        const int r = e / (h + 1), k = e - r * (h + 1);
        float2 v = make_float2(0.f, 0.f);
        if (k <= nmax) v = mesh[static_cast<size_t>(r) * a.pitch + k];
        tile[k * BP + r * nc + c] = v;
      }
    }
    __syncthreads();
    const int hk = h / 2 + 1;
    for (int e = tid; e < rows * nc * hk; e += kFftNT) {  // half-length packing, as in k_fft_z_c2r
      const int c = e / hk, k = e - c * hk;
      const float2 xk = tile[k * BP + c], xm = tile[(h - k) * BP + c];
      const float2 s = cadd(xk, cconj(xm));
      const float2 u = rot<true>(cmulc(csub(xk, cconj(xm)), roots[k]));
      if (k != 0 && 2 * k != h) tile[(h - k) * BP + c] = cconj(csub(s, u));
      tile[k * BP + c] = cadd(s, u);
    }
    __syncthreads();
    fft_tile<true, 8>(tile, tw, a.plh, B, BP, tid);
#pragma unroll
    for (int u = 0; u < kShellUnits; ++u) {
      const int e = tid + u * kFftNT;
      if (e < rows * h) {
        const int r = e / h, m = e - r * h;
        const float2* z = tile + m * BP + r * nc;
        const float2 f0 = z[q.column[0]], f1 = z[q.column[1]], f2 = z[q.column[2]];
        acc += static_cast<double>(f0.x) * f1.x * f2.x;
        acc += static_cast<double>(f0.y) * f1.y * f2.y;
      }
    }
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if ((tid & 63) == 0) sums[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int w = 0; w < kFftNT / 64; ++w) s += sums[w];
    q.parts[blockIdx.x] = s;
  }
}

// Block reduction of one FP64 value per thread into part[blockIdx.x].
__device__ __forceinline__ void block_sum(double v, double* __restrict__ part) {
  __shared__ double sh[kNT];
  __syncthreads();  // sh may still be read by a previous reduction
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int off = kNT / 2; off > 0; off >>= 1) {
    if (static_cast<int>(threadIdx.x) < off) sh[threadIdx.x] += sh[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// Per-block sums over shell blockIdx.y's modes of mult |delta_hat|^2 / W^2 and of mult (exact in FP64), with mult = 2 for
// 0 < kz < Nm / 2 (the mode and its conjugate) and 1 on the kz = 0 and Nyquist planes. Walks the cube |n_d| <= nmax.
__global__ __launch_bounds__(kNT) void k_shell_power(ShellPasses a, const ShellPower* __restrict__ shells) {
  const LPC_CONST ShellPower& q = to_const(shells)[blockIdx.y];
  const int n = a.n, half = n / 2, nmax = min(q.nmax, half), nz = nmax + 1, side = min(2 * nmax + 1, n);
  const int64_t count = static_cast<int64_t>(side) * side * nz;
  double p = 0.0, cnt = 0.0;
  for (int64_t e = static_cast<int64_t>(blockIdx.x) * kNT + threadIdx.x; e < count;
       e += static_cast<int64_t>(kSumBlocks) * kNT) {
    const int64_t r = e / nz;
    const int kz = static_cast<int>(e - r * nz);
    const int iy = static_cast<int>(r % side), ix = static_cast<int>(r / side);
    const int nx = ix <= nmax ? ix : ix - side, ny = iy <= nmax ? iy : iy - side;
    const int n2 = nx * nx + ny * ny + kz * kz;
    if (n2 < q.n2lo || n2 >= q.n2hi) continue;
    const int kx = nx < 0 ? nx + n : nx, ky = ny < 0 ? ny + n : ny;
    const float2 d = a.spec[(static_cast<size_t>(kx) * n + ky) * a.pitch + kz];
    const double W = a.win[abs(nx)] * a.win[abs(ny)] * a.win[kz];
    const double mult = (kz > 0 && kz < half) ? 2.0 : 1.0;
    p += mult * (static_cast<double>(d.x) * d.x + static_cast<double>(d.y) * d.y) / (W * W);
    cnt += mult;
  }
  block_sum(p, q.parts);
  block_sum(cnt, q.parts + kSumBlocks);
}

// out[row] = the sum of row's kSumBlocks partial sums, in a fixed order.
__global__ __launch_bounds__(kNT) void k_sum_parts(const double* __restrict__ parts, double* __restrict__ out) {
  static_assert(kSumBlocks == kNT, "one partial sum per thread");
  block_sum(parts[static_cast<size_t>(blockIdx.x) * kSumBlocks + threadIdx.x], out);
}

template <class K>
void shell_big_lds(K kernel) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            144 * 1024);
}
struct ShellInit {
  ShellInit() {
    shell_big_lds(k_shell_x<16, 8>);
    shell_big_lds(k_shell_x<8, 8>);
    shell_big_lds(k_shell_x<8, 16>);
    shell_big_lds(k_shell_y<16, 8>);
    shell_big_lds(k_shell_y<8, 8>);
    shell_big_lds(k_shell_y<8, 16>);
    shell_big_lds(k_shell_z);
  }
};
void shell_init() { static ShellInit once; }

}  // namespace

hipError_t shell_fields(ShellPasses a, const ShellField* fields, int nfield, const ShellTriple* triples, int ntriple,
                        hipStream_t s) {
  if (nfield < 1 || ntriple < 1) return hipErrorInvalidValue;
  shell_init();
  const int n = a.n, h = n / 2, B = shell_cols(n);
  a.ntc = (h + B) / B;  // columns kz = 0 .. n / 2
  const dim3 grid(static_cast<unsigned>(n * a.ntc), static_cast<unsigned>(nfield));
  const size_t lds = sizeof(float2) * (static_cast<size_t>(n) * strided_pitch(B) + n);
  if (n <= 256) {
    k_shell_x<16, 8><<<grid, kFftNT, lds, s>>>(a, fields);
    k_shell_y<16, 8><<<grid, kFftNT, lds, s>>>(a, fields);
  } else if (n <= 512) {
    k_shell_x<8, 8><<<grid, kFftNT, lds, s>>>(a, fields);
    k_shell_y<8, 8><<<grid, kFftNT, lds, s>>>(a, fields);
  } else {
    k_shell_x<8, 16><<<grid, kFftNT, lds, s>>>(a, fields);
    k_shell_y<8, 16><<<grid, kFftNT, lds, s>>>(a, fields);
  }
  // rows per tile: at most kShellUnits point pairs per thread, 8 points of a column per thread (three fields a row)
  auto fits = [h](int R) { return R * h <= kShellUnits * kFftNT && 3 * R <= kFftNT && h <= 8 * (kFftNT / (3 * R)); };
  a.R = std::max(1, std::min(kFftNT / 3, kShellUnits * kFftNT / h));
  while (a.R > 1 && !fits(a.R)) --a.R;
  if (!fits(a.R)) return hipErrorInvalidValue;
  const size_t lds_z = sizeof(float2) * (static_cast<size_t>(h + 1) * ((3 * a.R) | 1) + h + h + 1);
  k_shell_z<<<dim3(kSumBlocks, static_cast<unsigned>(ntriple)), kFftNT, lds_z, s>>>(a, fields, triples);
  return hipGetLastError();
}

hipError_t shell_power(const ShellPasses& a, const ShellPower* shells, int nshell, hipStream_t s) {
  if (nshell < 1) return hipErrorInvalidValue;
  k_shell_power<<<dim3(kSumBlocks, static_cast<unsigned>(nshell)), kNT, 0, s>>>(a, shells);
  return hipGetLastError();
}

hipError_t sum_parts(const double* parts, int rows, double* out, hipStream_t s) {
  if (rows < 1) return hipErrorInvalidValue;
  k_sum_parts<<<static_cast<unsigned>(rows), kNT, 0, s>>>(parts, out);
  return hipGetLastError();
}

int sum_blocks() { return kSumBlocks; }

hipError_t pk_bin(const float2* spec, const double* window, int nm, int pitch, double box, double k_max, int n_bins,
                  double pscale, double* sums, unsigned long long* counts, hipStream_t s) {
  const int nh = nm / 2 + 1, nseg = (nh + kRun - 1) / kRun;
  static_assert(kRun == 8, "the rows' pitch is a multiple of 8 values");
  const int items = nh * nh * nseg, per_block = kNT * kRunsPerThread;
  const size_t lds = static_cast<size_t>(n_bins) * (2 * sizeof(double) + sizeof(unsigned)) + sizeof(double) * nh;
  k_pk_bin<<<static_cast<unsigned>((items + per_block - 1) / per_block), kNT, lds, s>>>(
      spec, window, nm, pitch, 2.0 * M_PI / box, k_max / n_bins, n_bins, pscale, sums, counts);
  return hipGetLastError();
}

}  // namespace kern
}  // namespace lpc
