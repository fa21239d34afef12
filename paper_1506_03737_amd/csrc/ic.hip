// Initial-condition kernels of liblpc (Sec. 2.1 Eqs. 5-10 and Sec. 5 of Howlett, Manera & Percival 2015):
// counter-based white noise, scaling by the linear spectrum, the spectral derivatives that give Psi1, the second
// derivatives of phi1 that form the 2LPT source, and the final assembly of positions and momenta on the lattice.
//
// The construction runs as nine passes over half-spectrum meshes instead of fourteen separate 3-D transforms. Every
// field of a group is a product of the axes' wavenumbers times one spectrum phi = delta / k^2, so the inverse
// transforms share their inner axes: along x the three spectra phi, i kx phi and kx^2 phi, along y six (kinds xx, x,
// xy, 1, y, yy), and only the z pass, which holds all six of a row, forms the nine real rows (Psi1 and the six phi_ij),
// the source and its forward z transform. The spectrum is zero on every Nyquist plane, so the passes leave the kz = N/2
// column out. Per lattice site (256^3, bytes): 14 transforms with their factor passes moved about 540, these passes
// about 210, which is 0.71 ms at the card's copy rate. The passes take 1.14 ms: the y passes run at 0.85 of that rate, the x
// passes at 0.55, the first z pass (343 us for 135 us of bytes) is bound by the VALU and LDS work of its nine run-time
// transforms a row and by the 0.6 GB that its spilled registers add, and the white noise by its FP64 arithmetic.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "fft_device.h"

namespace lpc {
namespace kern {

namespace {

// SplitMix64 (Steele, Lea & Flood 2014): the c-th output of a stream whose state starts at `seed`.
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t c) {
  uint64_t z = seed + (c + 1ull) * 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

__device__ __forceinline__ double uniform_open(uint64_t seed, uint64_t c) {
  return (static_cast<double>(splitmix64(seed, c) >> 11) + 0.5) * 0x1.0p-53;
}

// Unit Gaussian of lattice point idx (Box-Muller in FP64).
__device__ __forceinline__ float white_noise(uint64_t seed, uint64_t idx) {
  const double u1 = uniform_open(seed, 2 * idx), u2 = uniform_open(seed, 2 * idx + 1);
  return static_cast<float>(sqrt(-2.0 * log(u1)) * cospi(2.0 * u2));
}

// BBKS transfer function (Bardeen et al. 1986), q = k / (Om h).
__device__ __forceinline__ double bbks(double k, double om_h) {
  const double q = k / om_h, x = 2.34 * q;
  const double a = 16.1 * q, b = 5.46 * q, d = 6.71 * q;
  const double poly = 1.0 + 3.89 * q + a * a + b * b * b + d * d * d * d;
  return log1p(x) / x / sqrt(sqrt(poly));
}

// Top-hat window of radius x / k, and the integrand of sigma(8)^2 over ln k for unit amplitude.
__device__ __forceinline__ double tophat(double x) {
  if (fabs(x) < 1e-3) return 1.0 - x * x / 10.0;
  return 3.0 * (sin(x) - x * cos(x)) / (x * x * x);
}

// 2 pi^2 sigma(8)^2 of the spectrum k^ns T^2, by kIcPieces Gauss-Legendre rules of 64 nodes over ln k in [ln 1e-7, ln 1e3]
// (the quadrature of the host's pk_amplitude): one wave per piece. On the host its 25600 integrands took 0.6 ms of a call
// whose passes take 0.6 (160^3) to 1.2 ms (256^3).
__global__ __launch_bounds__(64) void k_ic_sigma8(const double* __restrict__ gl, double n_s, double om_h,
                                                  double* __restrict__ parts) {
  const double lo = log(1e-7), step = (log(1e3) - lo) / kIcPieces;
  const double r = 0.5 * step, mid = lo + (blockIdx.x + 0.5) * step;
  const double k = exp(mid + r * gl[threadIdx.x]);
  const double t = bbks(k, om_h), w = tophat(8.0 * k);
  double v = r * gl[64 + threadIdx.x] * (k * k * k * pow(k, n_s) * t * t * w * w);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  if (threadIdx.x == 0) parts[blockIdx.x] = v;
}

// Spectral weights by the integer |n|^2 of a mode (k = kf |n|): the FP64 powers and logarithms are taken once per
// distinct |n|^2 (0.75 N^2 of them) instead of once per mode (N^3 / 2; 0.14 ms at 256^3).
__global__ __launch_bounds__(kNT) void k_ic_weights(IcWeights w) {
  const IcWeight& q = w.spec[blockIdx.y];
  double amp = 1.0;  // the amplitude sigma8^2 / sigma(8)^2 of the linear spectrum
  if (q.amplitude) {
    __shared__ double sh[kNT];
    double part = 0.0;
    for (int p = threadIdx.x; p < kIcPieces; p += kNT) part += w.sigma8_parts[p];
    sh[threadIdx.x] = part;
    __syncthreads();
    for (int off = kNT / 2; off > 0; off >>= 1) {
      if (static_cast<int>(threadIdx.x) < off) sh[threadIdx.x] += sh[threadIdx.x + off];
      __syncthreads();
    }
    amp = w.sigma8 * w.sigma8 / (sh[0] / (2.0 * M_PI * M_PI));
  }
  const int n2 = blockIdx.x * kNT + threadIdx.x;
  if (n2 >= w.count) return;
  double v = 0.0;
  if (n2 > 0) {
    const double k = w.kf * sqrt(static_cast<double>(n2));
    v = amp * q.coef * pow(k, q.expo);
    if (q.transfer) {
      const double t = bbks(k, w.om_h);
      v *= q.transfer == 2 ? t * t : t;
    }
    if (q.root) v = sqrt(v);
  }
  w.table[static_cast<size_t>(blockIdx.y) * w.count + n2] = v;
}

// Forward z pass of real rows made on the fly: the white noise, or the products sum_t c fa fb of a group of
// non-Gaussian terms (grid.y). R rows per workgroup; the layout and the even/odd split are those of k_fft_z_r2c.
template <bool NOISE, int R>
__global__ __launch_bounds__(kFftNT, 4) void k_ic_r2c(IcR2C a) {
  constexpr int BP = R + 1;
  extern __shared__ float2 smem[];
  const int tid = threadIdx.x, N = a.N, h = N / 2, nrows = N * N;
  const int row0 = xcd_remap(blockIdx.x, gridDim.x) * R;
  float2* tile = smem;
  float2* tw = tile + h * BP;
  float2* roots = tw + h;
  const TableRegs<float2> r_tw = table_load(a.tw, h, tid), r_roots = table_load(a.roots, h + 1, tid);
  table_store(tw, r_tw, h, tid);
  table_store(roots, r_roots, h + 1, tid);
  const int units = min(R, nrows - row0) * h;
  {
    const int dq = kFftNT / h, dr = kFftNT - dq * h;
    int b = tid / h, j = tid - b * h;
    for (int u = tid; u < units; u += kFftNT) {
      const size_t at = static_cast<size_t>(row0) * N + 2 * static_cast<size_t>(u);
      float2 v = make_float2(0.f, 0.f);
      if constexpr (NOISE) {
        v = make_float2(white_noise(a.seed, at), white_noise(a.seed, at + 1));
      } else {
        const PngProducts& pp = a.pp[blockIdx.y];
        for (int t = 0; t < pp.n; ++t) {
          v.x += pp.c[t] * (pp.fa[t][at] * pp.fb[t][at]);
          v.y += pp.c[t] * (pp.fa[t][at + 1] * pp.fb[t][at + 1]);
        }
      }
      tile[j * BP + b] = v;
      b += dq;
      j += dr;
      if (j >= h) {
        j -= h;
        ++b;
      }
    }
  }
  __syncthreads();
  fft_tile<false, 8>(tile, tw, a.pl, R, BP, tid);
  float2* out = a.out[blockIdx.y];
  const int hk = h / 2 + 1, npair = min(R, nrows - row0) * hk;
  const int dq = kFftNT / hk, dr = kFftNT - dq * hk;
  int b = tid / hk, k = tid - b * hk;
  for (int u = tid; u < npair; u += kFftNT) {
    const float2 zk = tile[k * BP + b], zm = tile[(k == 0 ? 0 : h - k) * BP + b];
    const float2 E = cscale(cadd(zk, cconj(zm)), 0.5f), O = cscale(rot<false>(csub(zk, cconj(zm))), 0.5f);
    const float2 t = cmul(roots[k], O);
    float2* o = out + static_cast<size_t>(row0 + b) * a.pitch;
    o[k] = cadd(E, t);
    if (k != 0 && 2 * k != h) o[h - k] = cconj(csub(E, t));  // (the kz = N / 2 column is dropped)
    b += dq;
    k += dr;
    if (k >= hk) {
      k -= hk;
      ++b;
    }
  }
}

// A column tile's transform, with compile-time stages for the plans of 256 and 512 points (the commonest lattices).
template <bool INV, int M, int B, int BP, class PL>
__device__ __forceinline__ void fft_tile_fixed(float2* tile, const float2* tw, const PL& pl, int tid) {
  using F256 = FixedFFT<INV, M, B, BP, 8, 8, 4>;
  using F512 = FixedFFT<INV, M, B, BP, 8, 8, 8>;
  if (F256::matches(pl)) {
    F256::run(tile, tw, tid);
  } else if (F512::matches(pl)) {
    F512::run(tile, tw, tid);
  } else {
    fft_tile<INV, M>(tile, tw, pl, B, BP, tid);
  }
}

// i, with HIDE as a value that the compiler does not know: indices formed from it are not kept in registers from one phase
// to the next.
template <bool HIDE>
__device__ __forceinline__ int opaque(int i) {
  if constexpr (HIDE) asm volatile("" : "+v"(i));
  return i;
}

// The x pass. A tile is B columns (kz) of one ky. delta(k) = wbase base + sum_i w_i FFT_x(in_i), zero at k = 0 and on
// the Nyquist planes, stays in the threads' registers (thread (j0, b) owns rows j0 + m S, S = kFftNT / B); each output
// is the inverse x transform of a factor times it. A workgroup reads and writes its own columns only, so the outputs may
// be the inputs' buffers.
// SUM: delta has more than one term. The sum is formed in FP64 and rounded once, since the terms of a non-Gaussian field may
// exceed it by far. An instance of its own: its accumulators live through the transforms, and only without the indices that
// the compiler would carry along does it keep the register cap (160^3 equilateral, the three x passes: sum in FP32 147 us,
// in FP64 with 15 spilled registers 161, without a cap 191, so 149; the single-term instance is 1.5 % slower that way).
template <int B, int M, bool SUM>
__global__ __launch_bounds__(kFftNT, M <= 8 ? 4 : 2) void k_ic_x(IcX a) {
  constexpr int BP = strided_pitch(B), S = kFftNT / B;
  extern __shared__ float2 smem[];
  const int tid = threadIdx.x, n = a.N, half = n / 2;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const int y = t / a.ntc, c0 = (t - y * a.ntc) * B;
  const int b = tid % B, j0 = tid / B, nz = c0 + b;
  float2* tile = smem;
  float2* tw = tile + n * BP;
  const uint32_t astr = static_cast<uint32_t>(n) * static_cast<uint32_t>(a.pitch);
  const bool col = nz < half;
  const size_t off = static_cast<size_t>(y) * a.pitch + min(nz, half - 1);
  const int ny = y <= half ? y : y - n, nyz2 = ny * ny + nz * nz;
  const TableRegs<float2> r_tw = table_load(a.tw, n, tid);
  float2 d[M];
  double sx[SUM ? M : 1], sy[SUM ? M : 1];
  if constexpr (SUM) {
#pragma unroll
    for (int m = 0; m < M; ++m) sx[m] = sy[m] = 0.0;
  }
  auto add = [&](int m, float2 v, double w) {
    if constexpr (SUM) {
      sx[m] += v.x * w;
      sy[m] += v.y * w;
    } else {
      d[m] = make_float2(static_cast<float>(v.x * w), static_cast<float>(v.y * w));
    }
  };
  auto mode2 = [&](int j) {  // |n|^2 of row j, 0 for a dropped mode
    const int nx = j <= half ? j : j - n;
    return (col && nx != half && ny != half) ? nx * nx + nyz2 : 0;
  };
  table_store(tw, r_tw, n, tid);
  for (int i = 0; i < a.nin; ++i) {
    const float2* in = a.in[i];
    const int j2 = opaque<SUM>(j0);
    float2 v[M];
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = in[off + static_cast<uint32_t>(min(j2 + m * S, n - 1)) * astr];
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (j2 + m * S < n) tile[(j2 + m * S) * BP + b] = v[m];
    __syncthreads();
    fft_tile_fixed<false, M, B, BP>(tile, tw, a.pl, tid);
    const double* w = a.w[i];
    const int j1 = opaque<SUM>(j0);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int j = j1 + m * S;
      if (j < n) {
        const float2 x = tile[j * BP + b];
        const int n2 = mode2(j);
        add(m, x, w ? w[n2] : (n2 ? 1.0 : 0.0));
      }
    }
  }
  if (a.base) {
    const int j1 = opaque<SUM>(j0);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int j = j1 + m * S;
      if (j < n) {
        const float2 v = a.base[off + static_cast<uint32_t>(j) * astr];
        const int n2 = mode2(j);
        const double w = a.wbase ? a.wbase[n2] : (n2 ? 1.0 : 0.0);
        add(m, v, w);
      }
    }
  }
  if constexpr (SUM) {
#pragma unroll
    for (int m = 0; m < M; ++m) d[m] = make_float2(static_cast<float>(sx[m]), static_cast<float>(sy[m]));
  }
  if (a.keep) {
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (j0 + m * S < n && col) a.keep[off + static_cast<uint32_t>(j0 + m * S) * astr] = d[m];
  }
  const float kf = a.kf, ky = kf * static_cast<float>(ny), kz = kf * static_cast<float>(nz);
  for (int o = 0; o < a.nout; ++o) {
    const int kind = a.kind[o];
    const double* w = a.wout[o];
    const int j1 = opaque<SUM>(j0);
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int j = j1 + m * S;
      if (j < n) {
        const int n2 = mode2(j);
        const float kx = kf * static_cast<float>(j <= half ? j : j - n);
        float2 v = make_float2(0.f, 0.f);
        if (n2) {
          if (w) {
            const double f = w[n2];
            v = make_float2(static_cast<float>(d[m].x * f), static_cast<float>(d[m].y * f));
          } else {
            const float inv_k2 = a.sign / (kx * kx + ky * ky + kz * kz);
            const float s = (kind == 0 ? 1.f : (kind == 1 ? kx : kx * kx)) * inv_k2;
            v = kind == 1 ? make_float2(-s * d[m].y, s * d[m].x) : make_float2(s * d[m].x, s * d[m].y);
          }
        }
        tile[j * BP + b] = v;
      }
    }
    __syncthreads();
    fft_tile_fixed<true, M, B, BP>(tile, tw, a.pl, tid);
    float2* out = a.out[o];
    const int j2 = opaque<SUM>(j0);
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (j2 + m * S < n && col) out[off + static_cast<uint32_t>(j2 + m * S) * astr] = tile[(j2 + m * S) * BP + b];
  }
}

// The inverse y pass of the first group: kind 0 takes kx^2 phi to xx, kind 1 i kx phi to x (in place) and xy, kind 2 phi
// to itself, y and yy. The source columns are read once into registers; each output is one transform of a factor times
// them. A workgroup reads and writes its own columns only.
template <int B, int M>
__global__ __launch_bounds__(kFftNT, M <= 8 ? 4 : 2) void k_ic_y(IcY a) {
  constexpr int BP = strided_pitch(B), S = kFftNT / B;
  extern __shared__ float2 smem[];
  const int tid = threadIdx.x, n = a.N, half = n / 2;
  const int kind = blockIdx.y;
  const int t = xcd_remap(blockIdx.x, gridDim.x);
  const int x = t / a.ntc, c0 = (t - x * a.ntc) * B;
  const int b = tid % B, j0 = tid / B;
  float2* tile = smem;
  float2* tw = tile + n * BP;
  const bool col = c0 + b < half;
  const size_t off = static_cast<size_t>(x) * n * a.pitch + min(c0 + b, half - 1);
  const uint32_t astr = static_cast<uint32_t>(a.pitch);
  const TableRegs<float2> r_tw = table_load(a.tw, n, tid);
  const float2* in = a.in[kind];
  float2 v[M];
#pragma unroll
  for (int m = 0; m < M; ++m) v[m] = in[off + static_cast<uint32_t>(min(j0 + m * S, n - 1)) * astr];
  table_store(tw, r_tw, n, tid);
  for (int o = 0; o <= kind; ++o) {
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int j = j0 + m * S;
      if (j < n) {
        const float ky = a.kf * static_cast<float>(j <= half ? j : j - n);  // (the spectrum is zero at ky = N / 2)
        float2 u = v[m];
        if (o == 1) {  // i kx phi -> kx ky phi (kind 1); phi -> i ky phi (kind 2)
          const float s = kind == 1 ? -ky : ky;
          u = make_float2(-s * v[m].y, s * v[m].x);
        } else if (o == 2) {
          u = make_float2(ky * ky * v[m].x, ky * ky * v[m].y);
        }
        tile[j * BP + b] = u;
      }
    }
    __syncthreads();
    fft_tile_fixed<true, M, B, BP>(tile, tw, a.pl, tid);
    float2* out = a.out[kind][o];
#pragma unroll
    for (int m = 0; m < M; ++m)
      if (j0 + m * S < n && col) out[off + static_cast<uint32_t>(j0 + m * S) * astr] = tile[(j0 + m * S) * BP + b];
  }
}

// The inverse z pass: R rows per workgroup, NC columns of the tile per row.
//  kIcFirst:  the six spectra (xx, x, xy, 1, y, yy) of a row become nine real rows; Psi1 is written, the source
//             sum_{i>j} (phi_ii phi_jj - phi_ij^2) is formed in registers and leaves as its forward z transform.
//  kIcSecond: the three gradient spectra become Psi2, and with Psi1 the particles (positions, momenta, ids).
//  kIcPlain:  one spectrum per grid.y becomes a real field.
// R rows per workgroup hold at most E point pairs, and each thread of a column takes at most EPT of its points.
template <int MODE>
struct IcZShape;
template <>
struct IcZShape<kIcFirst> {
  static constexpr int NS = 6, NC = 9, E = 512, EPT = 12;
};
template <>
struct IcZShape<kIcSecond> {
  static constexpr int NS = 3, NC = 3, E = 1024, EPT = 8;
};
template <>
struct IcZShape<kIcPlain> {
  static constexpr int NS = 1, NC = 1, E = 2048, EPT = 8;
};

__device__ __forceinline__ float2 times_i(float2 v, float s) { return make_float2(-s * v.y, s * v.x); }  // i s v

// The cap of 80 registers spills 17 (kIcFirst) and 7 (kIcSecond) of them, and is still the better one: without spills, at 5
// waves per SIMD, the first group takes 45 us instead of 41 at 128^3, 86 and 80 at 160^3, 131 and 140 at 192^3, 345 and 343
// at 256^3, 521 and 434 at 270^3, 2700 and 2591 at 512^3; the second 281 and 301 at 270^3, 1760 and 1777 at 512^3.
template <int MODE>
__global__ __launch_bounds__(kFftNT, 6) void k_ic_z(IcZ a) {
  using Sh = IcZShape<MODE>;
  constexpr int NS = Sh::NS, NC = Sh::NC;
  constexpr int U = Sh::E / kFftNT;  // (row, point pair) units per thread
  extern __shared__ float2 smem[];
  const int tid = threadIdx.x, N = a.N, h = N / 2, R = a.R, nrows = N * N;
  const int B = NC * R, BP = B | 1;
  const int row0 = xcd_remap(blockIdx.x, gridDim.x) * R;
  const int rows = min(R, nrows - row0);
  float2* tile = smem;               // (h + 1) x BP
  float2* tw = tile + (h + 1) * BP;
  float2* roots = tw + h;
  const TableRegs<float2> r_tw = table_load(a.tw, h, tid), r_roots = table_load(a.roots, h + 1, tid);
  const int units = rows * h;
  {
    float2 v[U][NS];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = min(tid + u * kFftNT, units - 1);
      const int r = e / h, k = e - r * h;
      const size_t at = static_cast<size_t>(row0 + r) * a.pitch + k;
#pragma unroll
      for (int s = 0; s < NS; ++s) v[u][s] = a.in[MODE == kIcPlain ? blockIdx.y : s][at];
    }
    table_store(tw, r_tw, h, tid);
    table_store(roots, r_roots, h + 1, tid);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int e = tid + u * kFftNT;
      if (e >= units) continue;
      const int r = e / h, k = e - r * h;
      const float kz = a.kf * static_cast<float>(k);
      float2* o = tile + k * BP + r * NC;
      if constexpr (MODE == kIcFirst) {
        o[0] = v[u][1];                                                    // Psi_x
        o[1] = v[u][4];                                                    // Psi_y
        o[2] = times_i(v[u][3], kz);                                       // Psi_z
        o[3] = v[u][0];                                                    // xx
        o[4] = v[u][5];                                                    // yy
        o[5] = make_float2(kz * kz * v[u][3].x, kz * kz * v[u][3].y);      // zz
        o[6] = v[u][2];                                                    // xy
        o[7] = times_i(v[u][1], -kz);                                      // xz
        o[8] = times_i(v[u][4], -kz);                                      // yz
      } else if constexpr (MODE == kIcSecond) {
        o[0] = v[u][0];
        o[1] = v[u][1];
        o[2] = times_i(v[u][2], kz);
      } else {
        o[0] = v[u][0];
      }
    }
    for (int c = tid; c < B; c += kFftNT) tile[h * BP + c] = make_float2(0.f, 0.f);  // the dropped kz = N / 2 column
  }
  const int64_t n = static_cast<int64_t>(nrows) * N;
  float2 q1[U][3];  // the second group's Psi1, on its way during the transform
  if constexpr (MODE == kIcSecond) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t at = static_cast<size_t>(row0) * N + 2 * static_cast<size_t>(min(tid + u * kFftNT, units - 1));
#pragma unroll
      for (int d = 0; d < 3; ++d) q1[u][d] = make_float2(a.psi1[d * n + at], a.psi1[d * n + at + 1]);
    }
  }
  __syncthreads();
  {
    // half-length packing of the real transforms, as in k_fft_z_c2r (columns of rows past the last stay unread)
    const int hk = h / 2 + 1;
    const int dq = kFftNT / hk, dr = kFftNT - dq * hk;
    int c = tid / hk, k = tid - c * hk;
    for (int e = tid; e < hk * rows * NC; e += kFftNT) {
      const float2 xk = tile[k * BP + c], xm = tile[(h - k) * BP + c];
      const float2 s = cadd(xk, cconj(xm));
      const float2 u = rot<true>(cmulc(csub(xk, cconj(xm)), roots[k]));
      if (k != 0 && 2 * k != h) tile[(h - k) * BP + c] = cconj(csub(s, u));
      tile[k * BP + c] = cadd(s, u);
      c += dq;
      k += dr;
      if (k >= hk) {
        k -= hk;
        ++c;
      }
    }
  }
  __syncthreads();
  fft_tile<true, Sh::EPT>(tile, tw, a.pl, B, BP, tid);
  // unit (row r, pair m): points 2 m and 2 m + 1 of every field of the row
  float2 src = make_float2(0.f, 0.f);
  const bool pairs = a.aligned;  // the output arrays take 8-byte stores
  auto put = [&](float* p, size_t at, float2 x) {
    if (pairs) {
      *reinterpret_cast<float2*>(p + at) = x;
    } else {
      p[at] = x.x;
      p[at + 1] = x.y;
    }
  };
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = tid + u * kFftNT;
    if (e >= units) continue;
    const int r = e / h, m = e - r * h, row = row0 + r;
    const size_t at = static_cast<size_t>(row) * N + 2 * static_cast<size_t>(m);
    const float2* z = tile + m * BP + r * NC;
    float2 f[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) f[c] = cscale(z[c], a.scale);
    if constexpr (MODE == kIcFirst) {
#pragma unroll
      for (int d = 0; d < 3; ++d) put(a.psi1 + d * n, at, f[d]);
      auto source = [](float xx, float yy, float zz, float xy, float xz, float yz) {
        float s = xx * yy + xx * zz + yy * zz;
        s -= xy * xy;
        s -= xz * xz;
        return s - yz * yz;
      };
      src = make_float2(source(f[3].x, f[4].x, f[5].x, f[6].x, f[7].x, f[8].x),
                        source(f[3].y, f[4].y, f[5].y, f[6].y, f[7].y, f[8].y));
    } else if constexpr (MODE == kIcSecond) {
      const int lat[3] = {row / N, row % N, 2 * m};
      const double spacing = a.box / N;
      const float fbox = static_cast<float>(a.box);
      auto position = [&](int l, float p1, float p2) {
        double x = (l + 0.5) * spacing + static_cast<double>(a.d1) * p1 + static_cast<double>(a.d2) * p2;
        if (!(x >= 0.0 && x < a.box)) x -= a.box * floor(x / a.box);  // (floor is 0 inside the box)
        const float xf = static_cast<float>(x);
        return xf >= fbox ? xf - fbox : xf;
      };
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        const float2 p1 = q1[u][d], p2 = f[d];
        put(a.psi2 + d * n, at, p2);
        put(a.pos + d * n, at,
            make_float2(position(lat[d], p1.x, p2.x), position(lat[d] + (d == 2 ? 1 : 0), p1.y, p2.y)));
        put(a.vel + d * n, at, make_float2(a.f1 * p1.x + a.f2 * p2.x, a.f1 * p1.y + a.f2 * p2.y));
      }
      a.id[at] = static_cast<int32_t>(at);
      a.id[at + 1] = static_cast<int32_t>(at + 1);
    } else {
      put(a.real[blockIdx.y], at, f[0]);
    }
  }
  if constexpr (MODE == kIcFirst) {
    // the source's forward z transform: its rows take the tile's first R columns
    __syncthreads();
    if (tid < units) {
      const int r = tid / h, m = tid - r * h;
      tile[m * BP + r] = src;
    }
    __syncthreads();
    fft_tile<false, Sh::EPT>(tile, tw, a.pl, R, BP, tid);
    const int hk = h / 2 + 1;
    for (int e = tid; e < rows * hk; e += kFftNT) {
      const int r = e / hk, k = e - r * hk;
      const float2 zk = tile[k * BP + r], zm = tile[(k == 0 ? 0 : h - k) * BP + r];
      const float2 E = cscale(cadd(zk, cconj(zm)), 0.5f), O = cscale(rot<false>(csub(zk, cconj(zm))), 0.5f);
      const float2 t = cmul(roots[k], O);
      float2* o = a.source + static_cast<size_t>(row0 + r) * a.pitch;
      o[k] = cadd(E, t);
      if (k != 0 && 2 * k != h) o[h - k] = cconj(csub(E, t));
    }
  }
}

constexpr size_t kIcMaxLds = 160 * 1024;
template <class K>
void big_lds(K kernel) {
  (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(kIcMaxLds));
}
struct IcInit {
  IcInit() {
    big_lds(k_ic_r2c<true, 8>);
    big_lds(k_ic_r2c<true, 16>);
    big_lds(k_ic_r2c<true, 32>);
    big_lds(k_ic_r2c<false, 8>);
    big_lds(k_ic_r2c<false, 16>);
    big_lds(k_ic_r2c<false, 32>);
    big_lds(k_ic_x<16, 8, false>);
    big_lds(k_ic_x<16, 8, true>);
    big_lds(k_ic_x<8, 8, false>);
    big_lds(k_ic_x<8, 8, true>);
    big_lds(k_ic_x<8, 16, false>);
    big_lds(k_ic_x<8, 16, true>);
    big_lds(k_ic_y<16, 8>);
    big_lds(k_ic_y<8, 8>);
    big_lds(k_ic_y<8, 16>);
    big_lds(k_ic_z<kIcFirst>);
    big_lds(k_ic_z<kIcSecond>);
    big_lds(k_ic_z<kIcPlain>);
  }
};
void ic_init() { static IcInit once; }

// Columns of an x or y tile: 16 up to 256 points (8 points per thread), then 8 (8 per thread to 512, 16 to 1024).
int ic_cols(int n) { return n <= 256 ? 16 : 8; }
size_t ic_cols_lds(int n) { return sizeof(float2) * (static_cast<size_t>(n) * strided_pitch(ic_cols(n)) + n); }

template <int MODE>
hipError_t launch_ic_z(IcZ a, int ny, hipStream_t s) {
  ic_init();
  using Sh = IcZShape<MODE>;
  const int h = a.N / 2, nrows = a.N * a.N;
  auto fits = [&](int R) { return R * h <= Sh::E && R * Sh::NC <= kFftNT && h <= Sh::EPT * (kFftNT / (R * Sh::NC)); };
  a.R = std::max(1, std::min(kFftNT / Sh::NC, Sh::E / h));
  while (a.R > 1 && !fits(a.R)) --a.R;
  if (!fits(a.R)) return hipErrorInvalidValue;
  const int B = Sh::NC * a.R;
  const size_t lds = sizeof(float2) * (static_cast<size_t>(h + 1) * (B | 1) + h + h + 1);
  if (lds > kIcMaxLds) return hipErrorInvalidValue;
  k_ic_z<MODE><<<dim3(static_cast<unsigned>((nrows + a.R - 1) / a.R), static_cast<unsigned>(ny)), kFftNT, lds, s>>>(a);
  return hipGetLastError();
}

}  // namespace

hipError_t ic_sigma8(const double* gl, double n_s, double om_h, double* parts, hipStream_t s) {
  k_ic_sigma8<<<kIcPieces, 64, 0, s>>>(gl, n_s, om_h, parts);
  return hipGetLastError();
}

hipError_t ic_weights(const IcWeights& w, int tables, hipStream_t s) {
  if (tables < 1 || tables > kIcMaxWeights) return hipErrorInvalidValue;
  k_ic_weights<<<dim3(static_cast<unsigned>((w.count + kNT - 1) / kNT), static_cast<unsigned>(tables)), kNT, 0, s>>>(w);
  return hipGetLastError();
}

hipError_t ic_r2c(const IcR2C& a, bool noise, int groups, hipStream_t s) {
  ic_init();
  const int h = a.N / 2, nrows = a.N * a.N;
  const int R = h <= 128 ? 32 : (h <= 256 ? 16 : 8);  // 8 points of a column per thread
  const size_t lds = sizeof(float2) * (static_cast<size_t>(h) * (R + 1) + h + h + 1);
  const dim3 grid(static_cast<unsigned>((nrows + R - 1) / R), static_cast<unsigned>(noise ? 1 : groups));
#define LPC_IC_R2C(F, RR) k_ic_r2c<F, RR><<<grid, kFftNT, lds, s>>>(a)
  if (noise) {
    if (R == 32) LPC_IC_R2C(true, 32); else if (R == 16) LPC_IC_R2C(true, 16); else LPC_IC_R2C(true, 8);
  } else {
    if (R == 32) LPC_IC_R2C(false, 32); else if (R == 16) LPC_IC_R2C(false, 16); else LPC_IC_R2C(false, 8);
  }
#undef LPC_IC_R2C
  return hipGetLastError();
}

hipError_t ic_x(IcX a, hipStream_t s) {
  ic_init();
  const int B = ic_cols(a.N);
  a.ntc = (a.N / 2 + B - 1) / B;
  const unsigned grid = static_cast<unsigned>(a.N * a.ntc);
  const size_t lds = ic_cols_lds(a.N);
  const int terms = a.nin + (a.base ? 1 : 0);
  if (terms < 1) return hipErrorInvalidValue;
#define LPC_IC_X(BB, MM)                                                  \
  {                                                                       \
    if (terms > 1) k_ic_x<BB, MM, true><<<grid, kFftNT, lds, s>>>(a);     \
    else k_ic_x<BB, MM, false><<<grid, kFftNT, lds, s>>>(a);              \
  }
  if (B == 16) LPC_IC_X(16, 8)
  else if (a.N <= 512) LPC_IC_X(8, 8)
  else LPC_IC_X(8, 16)
#undef LPC_IC_X
  return hipGetLastError();
}

hipError_t ic_y(IcY a, hipStream_t s) {
  ic_init();
  const int B = ic_cols(a.N);
  a.ntc = (a.N / 2 + B - 1) / B;
  const dim3 grid(static_cast<unsigned>(a.N * a.ntc), 3u);
  const size_t lds = ic_cols_lds(a.N);
  if (B == 16) k_ic_y<16, 8><<<grid, kFftNT, lds, s>>>(a);
  else if (a.N <= 512) k_ic_y<8, 8><<<grid, kFftNT, lds, s>>>(a);
  else k_ic_y<8, 16><<<grid, kFftNT, lds, s>>>(a);
  return hipGetLastError();
}

hipError_t ic_z(const IcZ& a, int mode, int fields, hipStream_t s) {
  if (mode == kIcFirst) return launch_ic_z<kIcFirst>(a, 1, s);
  if (mode == kIcSecond) return launch_ic_z<kIcSecond>(a, 1, s);
  return launch_ic_z<kIcPlain>(a, fields, s);
}

}  // namespace kern
}  // namespace lpc
