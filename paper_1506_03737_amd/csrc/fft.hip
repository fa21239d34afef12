// 3-D real FFTs of liblpc as three LDS-staged passes over HBM (Sec. 2.4 steps 2-3 of Howlett, Manera & Percival
// 2015: forward FFT of the density, Poisson solve and gradient in k-space, inverse FFT per force component).
//
// Layout: a real mesh is x-major float[n][n][n]; its half spectrum is float2[n][n][pitch] with kz = 0..n/2 used
// (pitch = n/2 + 1 rounded up to 8 complex values, 64 bytes, so every row starts on a 64-byte boundary).
// Forward: z pass (r2c of each row via a length-n/2 complex FFT and the even/odd split), y pass, x pass.
// Inverse: x pass, y pass, z pass (c2r via the same split). The force path fuses the forward x pass, the Poisson /
// deconvolution multiply and the inverse x transforms into one kernel, so the density spectrum is read once and never
// written back; it stores the x gradient and the potential, whose y and z gradients the y and z passes apply.
//
// Every kernel is batched: workgroup w takes item w of a work table of (job, tile) items, where a job is one mesh of
// one box, so one launch per pass serves any number of boxes of uneven sizes (see WorkTable). (A persistent
// grid-stride loop over the items measured slower: it raised register pressure past the four-waves-per-SIMD limit.)
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <initializer_list>
#include <utility>

#include "fft_plans.h"

namespace lpc {
namespace kern {

// p[s], pmask[s] and tw_off[s] of a plan whose radices are set
static void set_strides(Plan1D* p);

bool make_plan(int n, Plan1D* p, bool radix12) {
  if (n < 1) return false;
  int m = n, ns = 0;
  int odd[kMaxStages];
  for (int r : {5, 3}) {
    while (m % r == 0) {
      if (ns >= kMaxStages) return false;
      odd[ns++] = r;
      m /= r;
    }
  }
  int k = 0;
  while (m % 2 == 0) {
    m /= 2;
    ++k;
  }
  if (m != 1) return false;
  // powers of two: radix-8 stages, the remainder as one radix-4 or radix-2 stage (8 x 2 becomes 4 x 4)
  int pow2[kMaxStages], np = 0;
  int n8 = k / 3, rem = k % 3;
  if (rem == 1 && n8 > 0) {
    --n8;
    pow2[np++] = 4;
    pow2[np++] = 4;
    rem = 0;
  }
  for (int i = 0; i < n8; ++i) pow2[np++] = 8;
  if (rem == 1) pow2[np++] = 2;
  if (rem == 2) pow2[np++] = 4;
  // a radix-4 and a radix-3 stage merge into one radix-12 stage (one LDS round trip fewer)
  int i4 = -1, i3 = -1;
  for (int i = 0; i < np; ++i)
    if (pow2[i] == 4) i4 = i;
  for (int i = 0; i < ns; ++i)
    if (odd[i] == 3) i3 = i;
  const bool r12 = radix12 && i4 >= 0 && i3 >= 0;
  if (ns + np - (r12 ? 1 : 0) > kMaxStages) return false;
  p->n = n;
  p->nst = 0;
  for (int i = 0; i < np; ++i)
    if (!(r12 && i == i4)) p->radix[p->nst++] = pow2[i];
  if (r12) p->radix[p->nst++] = 12;
  for (int i = 0; i < ns; ++i)
    if (!(r12 && i == i3)) p->radix[p->nst++] = odd[i];
  set_strides(p);
  return true;
}

Plan1D reversed_plan(const Plan1D& p) {
  Plan1D r = p;
  for (int s = 0; s < p.nst; ++s) r.radix[s] = p.radix[p.nst - 1 - s];
  set_strides(&r);
  return r;
}

static void set_strides(Plan1D* p) {
  int prod = 1, off = 0;
  for (int s = 0; s < p->nst; ++s) {
    p->p[s] = prod;
    p->pmask[s] = ((prod & (prod - 1)) == 0) ? prod - 1 : -1;
    p->tw_off[s] = off;
    off += prod * (p->radix[s] - 1);
    prod *= p->radix[s];
  }
}

int mesh_pitch(int n) { return ((n / 2 + 1) + 7) / 8 * 8; }

namespace {

// ---------------------------------------------------------------------------------------------------------------
// Every kernel stages its global loads through registers in fully unrolled batches before writing the LDS tile: a
// runtime-bounded load loop would wait out the HBM latency once per element.

// z pass, forward r2c. An item transforms B consecutive rows of n reals. Each row is read as h = n/2 complex values
// z[m] = x[2m] + i x[2m+1]; after the length-h FFT, X[k] = E[k] + exp(-2 pi i k / n) O[k] with
// E[k] = (Z[k] + conj Z[h-k]) / 2 and O[k] = (Z[k] - conj Z[h-k]) / (2 i), for k = 0..h.
template <bool FIXED, int B, int EPT>
__global__ __launch_bounds__(kFftNT, 4) void k_fft_z_r2c(const ZR2CJob* __restrict__ jobs,
                                                         const int* __restrict__ offs, int njob, int total,
                                                         int* __restrict__ flags) {
  constexpr int BP = B + 1;
  extern __shared__ float2 smem[];
  {
    const int w = blockIdx.x;
    const int tid = threadIdx.x;
    if (w >= total) return;
    const int jb = __builtin_amdgcn_readfirstlane(find_job(to_const(offs), njob, w));
    const LPC_CONST ZR2CJob& J = to_const(jobs)[jb];
    const int n = J.n, h = n / 2, nrows = J.nrows;
    // each XCD takes a contiguous range of row blocks (r2c 0.72 -> 0.68 ms, c2r 2.25 -> 2.20 ms at 768^3)
    const int row0 = xcd_remap(w - offs[jb], offs[jb + 1] - offs[jb]) * B;
    if (row0 >= nrows) return;  // padding item (uniform; no LDS touched)
    float2* tile = smem;
    float2* tw = tile + h * BP;
    float2* roots = tw + h;
    const int count = h * B;
    // Element e = tid + m kFftNT of the tile is (row b, point j) = divmod(e, h): one division per thread, then steps
    // of kFftNT = dq h + dr.
    const int dq = kFftNT / h, dr = kFftNT - dq * h;
    const int b0 = tid / h, j0 = tid - b0 * h;
    // The item's rows are contiguous in the input, so element e is at offset row0 h + e (in complex values); rows past
    // the last are not read.
    const int valid = min(count, (nrows - row0) * h);
    // the tables' loads go out first, so that writing them to LDS waits for them only
    const TableRegs<float2> r_tw = table_load(J.tw, h, tid), r_roots = table_load(J.roots, h + 1, tid);
    if (FIXED) {
      LPC_GLOBAL const ulonglong2* in =
          reinterpret_cast<LPC_GLOBAL const ulonglong2*>(to_global(static_cast<const uint64_t*>(J.in))) +
          static_cast<size_t>(row0) * h;
      constexpr int H = EPT / 2;
      int bb = b0, jj = j0;
#pragma unroll 1
      for (int half = 0; half < 2; ++half) {
        ulonglong2 raw[H];
        int b = bb, j = jj;
#pragma unroll
        for (int m = 0; m < H; ++m) {
          const int e = tid + (half * H + m) * kFftNT;
          raw[m] = make_ulonglong2(0ull, 0ull);
          if (e < valid) raw[m] = in[e];
        }
        if (half == 0) {
          table_store(tw, r_tw, h, tid);
          table_store(roots, r_roots, h + 1, tid);
        }
        bool overflow = false;
        b = bb;
        j = jj;
#pragma unroll
        for (int m = 0; m < H; ++m) {
          const int e = tid + (half * H + m) * kFftNT;
          if (e < count) {
            overflow |= ((raw[m].x | raw[m].y) >> 63) != 0;
            float2 v = make_float2(0.f, 0.f);
            if (row0 + b < nrows) {
              v.x = static_cast<float>(static_cast<double>(raw[m].x) * J.mscale - 1.0);
              v.y = static_cast<float>(static_cast<double>(raw[m].y) * J.mscale - 1.0);
            }
            tile[j * BP + b] = v;
          }
          b += dq;
          j += dr;
          if (j >= h) {
            j -= h;
            ++b;
          }
        }
        bb = b;
        jj = j;
        if (overflow) atomicOr(flags + kFlagOverflow, 1);
      }
    } else {
      LPC_GLOBAL const float2* in = to_global(static_cast<const float2*>(J.in)) + static_cast<size_t>(row0) * h;
      float2 v[EPT];
#pragma unroll
      for (int m = 0; m < EPT; ++m) {
        const int e = tid + m * kFftNT;
        v[m] = make_float2(0.f, 0.f);
        if (e < valid) v[m] = in[e];
      }
      table_store(tw, r_tw, h, tid);
      table_store(roots, r_roots, h + 1, tid);
      int b = b0, j = j0;
#pragma unroll
      for (int m = 0; m < EPT; ++m) {
        const int e = tid + m * kFftNT;
        if (e < count) tile[j * BP + b] = v[m];
        b += dq;
        j += dr;
        if (j >= h) {
          j -= h;
          ++b;
        }
      }
    }
    __syncthreads();
    fft_tile_fast<false, EPT, B, BP, true>(tile, tw, J.pl, tid);
    LPC_GLOBAL float2* out = to_global(J.out);
    const int pitch = J.pitch;
    // Output in pairs (k, h - k), k <= h / 2, of each row: with E = (Z[k] + conj Z[h-k]) / 2,
    // O = (Z[k] - conj Z[h-k]) / (2 i) and t = exp(-2 pi i k / n) O, X[k] = E + t and X[h-k] = conj(E - t)
    // (Z[h] = Z[0]). Unit u = (row b, pair k) = divmod(u, h / 2 + 1): one division per thread, then steps.
    const int hk = h / 2 + 1, npair = B * hk;
    const int dqp = kFftNT / hk, drp = kFftNT - dqp * hk;
    int b = tid / hk, k = tid - (tid / hk) * hk;
    for (int u = tid; u < npair; u += kFftNT) {
      const int row = row0 + b;
      if (row < nrows) {
        const float2 zk = tile[k * BP + b];
        const float2 zm = tile[(k == 0 ? 0 : h - k) * BP + b];
        const float2 E = cscale(cadd(zk, cconj(zm)), 0.5f);
        const float2 O = cscale(rot<false>(csub(zk, cconj(zm))), 0.5f);  // (zk - conj zm) / (2 i)
        const float2 t = cmul(roots[k], O);
        LPC_GLOBAL float2* o = out + static_cast<size_t>(row) * pitch;
        o[k] = cadd(E, t);
        if (2 * k != h) o[h - k] = cconj(csub(E, t));
      }
      b += dqp;
      k += drp;
      if (k >= hk) {
        k -= hk;
        ++b;
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------------------------
// z pass, inverse c2r. An item transforms R rows of each of NC spectra; tile column r NC + c holds spectrum c of
// row r (B = NC R columns). With X the half spectrum of a real row,
//   Z[k] = (X[k] + conj X[h-k]) + i exp(+2 pi i k / n) (X[k] - conj X[h-k]),  h = n/2, k < h,
// and the unnormalised length-h inverse FFT of Z gives x[2m] + i x[2m+1]. Output rows are NC-interleaved.
// Each thread owns at most EPT points of a column (h <= EPT S); with EPT <= 12 the kernel fits in 80 VGPRs, so
// LDS-light tiles run three workgroups per CU.
template <int NC, int R, int EPT>
__global__ __launch_bounds__(kFftNT, (EPT <= 12) ? 6 : 4) void k_fft_z_c2r(const ZC2RJob* __restrict__ jobs,
                                                         const int* __restrict__ offs, int njob, int total) {
  constexpr int B = NC * R, BP = B + 1;
  extern __shared__ float2 smem[];
  {
    const int w = blockIdx.x;
    const int tid = threadIdx.x;
    if (w >= total) return;
    const int jb = __builtin_amdgcn_readfirstlane(find_job(to_const(offs), njob, w));
    const LPC_CONST ZC2RJob& J = to_const(jobs)[jb];
    const int n = J.n, h = n / 2, nrows = J.nrows, pitch = J.pitch;
    const int row0 = xcd_remap(w - offs[jb], offs[jb + 1] - offs[jb]) * R;  // as in the r2c: XCD-contiguous rows
    if (row0 >= nrows) return;  // padding item
    float2* tile = smem;                 // (h + 1) x BP
    float2* tw = tile + (h + 1) * BP;    // stage twiddles (h)
    float2* roots = tw + h;              // exp(-2 pi i k / n), k <= h
    LPC_GLOBAL const float2* in0 = to_global(J.in0);
    LPC_GLOBAL const float2* in1 = to_global(J.in1);
    LPC_GLOBAL const float2* in2 = to_global(J.in2);
    const float kz3 = J.kz3;
    // Loads, spectrum by spectrum: element e = tid + m kFftNT of a spectrum's R rows below the Nyquist point is
    // (row r, frequency k) = divmod(e, h), the same for every spectrum, so the offsets are stepped once (one division
    // per thread, then steps of kFftNT = dq h + dr) and each spectrum's base pointer is a compile-time choice. R h <=
    // B h / NC <= EPT kFftNT / NC, so MC loads per thread and spectrum cover it. The R NC Nyquist points (k = h) are
    // one load each for the first R NC threads. Tile column of (row r, spectrum c): r NC + c.
    constexpr int MC = (EPT + NC - 1) / NC;
    const int per = R * h;
    const int dq = kFftNT / h, dr = kFftNT - dq * h;
    // the tables' loads go out first, so that writing them to LDS waits for them only
    const TableRegs<float2> r_tw = table_load(J.tw, h, tid), r_roots = table_load(J.roots, h + 1, tid);
    {
      int64_t goff[MC];  // global element offset (row0 + r) pitch + k, or -1 for no element
      int loff[MC];      // tile offset k BP + r NC
      int kk[MC];
      {
        int r = tid / h, k = tid - (tid / h) * h;
#pragma unroll
        for (int m = 0; m < MC; ++m) {
          const bool ok = tid + m * kFftNT < per && row0 + r < nrows;
          goff[m] = ok ? static_cast<int64_t>(row0 + r) * pitch + k : -1;
          loff[m] = k * BP + r * NC;
          kk[m] = k;
          r += dq;
          k += dr;
          if (k >= h) {
            k -= h;
            ++r;
          }
        }
      }
      float2 v[NC][MC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        LPC_GLOBAL const float2* src = (c == 0) ? in0 : (c == 1 ? in1 : in2);
#pragma unroll
        for (int m = 0; m < MC; ++m) {
          v[c][m] = make_float2(0.f, 0.f);
          if (goff[m] >= 0) v[c][m] = src[goff[m]];
        }
      }
      const int nyq_r = tid / NC, nyq_c = tid - nyq_r * NC;  // Nyquist point of tile column tid
      float2 nyq = make_float2(0.f, 0.f);
      if (tid < B && row0 + nyq_r < nrows) {
        LPC_GLOBAL const float2* src = (nyq_c == 0) ? in0 : (nyq_c == 1 ? in1 : in2);
        nyq = src[static_cast<size_t>(row0 + nyq_r) * pitch + h];
      }
      // the tables are written while the loads are in flight
      table_store(tw, r_tw, h, tid);
      table_store(roots, r_roots, h + 1, tid);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
#pragma unroll
        for (int m = 0; m < MC; ++m) {
          if (tid + m * kFftNT < per) {
            float2 x = v[c][m];
            // the third spectrum is psi: i k_z psi (applied here, once every load is issued)
            if (NC == 3 && c == 2 && kz3 != 0.f) {
              const float kz = kz3 * static_cast<float>(kk[m]);
              x = make_float2(-kz * x.y, kz * x.x);
            }
            tile[loff[m] + c] = x;
          }
        }
      }
      // i k_z psi is zero on the Nyquist plane
      if (tid < B) tile[h * BP + tid] = (NC == 3 && nyq_c == 2 && kz3 != 0.f) ? make_float2(0.f, 0.f) : nyq;
    }
    __syncthreads();
    {
      const int hk = h / 2 + 1;
      const int dqk = kFftNT / hk, drk = kFftNT - dqk * hk;
      int col = tid / hk, k = tid - (tid / hk) * hk;
      for (int e = tid; e < hk * B; e += kFftNT) {
        const float2 xk = tile[k * BP + col];
        const float2 xm = tile[(h - k) * BP + col];
        const float2 t = roots[k];
        // Z[k] = (xk + conj xm) + i conj(t) (xk - conj xm) = S + u, and
        // Z[h-k] = (xm + conj xk) - i t (xm - conj xk) = conj(S - u)
        const float2 S = cadd(xk, cconj(xm));
        const float2 u = rot<true>(cmulc(csub(xk, cconj(xm)), t));
        if (k != 0 && 2 * k != h) tile[(h - k) * BP + col] = cconj(csub(S, u));
        tile[k * BP + col] = cadd(S, u);
        col += dqk;
        k += drk;
        if (k >= hk) {
          k -= hk;
          ++col;
        }
      }
    }
    __syncthreads();
    fft_tile_fast<true, EPT, B, BP, true, NC != 3>(tile, tw, J.pl, tid);  // NC = 3: plans without radix 12
    // Output: tile row m of row r holds points 2m and 2m + 1 of every spectrum (columns r NC .. r NC + NC - 1),
    // i.e. 2 NC consecutive floats of the NC-interleaved output row. One (row, m) unit per thread: NC 8-byte LDS
    // reads at a stride of BP float2 between lanes (conflict-free for odd BP) and NC 8-byte stores, contiguous across
    // lanes.
    const int rowlen = NC * n, hm = n / 2;
    const float scale = J.scale;
    const int units = min(R, nrows - row0) * hm;
    LPC_GLOBAL float* dst = to_global(J.out) + static_cast<size_t>(row0) * rowlen;
    // (the empty asm keeps the store loop's per-thread indices from being computed before the transform)
    int stid = tid;
    asm volatile("" : "+v"(stid));
    if ((reinterpret_cast<uintptr_t>(J.out) & 7) == 0) {
      // unit u = r hm + m: one division per thread, then steps of kFftNT = dqs hm + drs
      const int dqs = kFftNT / hm, drs = kFftNT - dqs * hm;
      int r = stid / hm, m = stid - r * hm;
#pragma unroll 1
      for (int u = stid; u < units; u += kFftNT) {
        const float2* src = tile + m * BP + r * NC;
        LPC_GLOBAL float2* o = reinterpret_cast<LPC_GLOBAL float2*>(dst + static_cast<size_t>(r) * rowlen + 2 * NC * m);
        if (NC == 3) {
          const float2 a = src[0], b = src[1], c = src[2];
          o[0] = make_float2(a.x * scale, b.x * scale);
          o[1] = make_float2(c.x * scale, a.y * scale);
          o[2] = make_float2(b.y * scale, c.y * scale);
        } else {
          const float2 a = src[0];
          o[0] = make_float2(a.x * scale, a.y * scale);
        }
        r += dqs;
        m += drs;
        if (m >= hm) {
          m -= hm;
          ++r;
        }
      }
    } else {
      for (int f = stid; f < units * 2 * NC; f += kFftNT) {
        const int r = f / rowlen, q = f - r * rowlen;
        const int jj = q / NC, c = q - jj * NC;
        const float2 z = tile[(jj >> 1) * BP + r * NC + c];
        dst[f] = ((jj & 1) ? z.y : z.x) * scale;
      }
    }
  }
}

struct Init {
  Init() {
    allow_big_lds(k_fft_z_r2c<true, 8, 8>);
    allow_big_lds(k_fft_z_r2c<true, 8, 12>);
    allow_big_lds(k_fft_z_r2c<true, 8, 16>);
    allow_big_lds(k_fft_z_r2c<true, 16, 8>);
    allow_big_lds(k_fft_z_r2c<true, 16, 12>);
    allow_big_lds(k_fft_z_r2c<true, 16, 16>);
    allow_big_lds(k_fft_z_r2c<true, 32, 8>);
    allow_big_lds(k_fft_z_r2c<true, 32, 12>);
    allow_big_lds(k_fft_z_r2c<true, 32, 16>);
    allow_big_lds(k_fft_z_r2c<false, 8, 8>);
    allow_big_lds(k_fft_z_r2c<false, 8, 12>);
    allow_big_lds(k_fft_z_r2c<false, 8, 16>);
    allow_big_lds(k_fft_z_r2c<false, 16, 8>);
    allow_big_lds(k_fft_z_r2c<false, 16, 12>);
    allow_big_lds(k_fft_z_r2c<false, 16, 16>);
    allow_big_lds(k_fft_z_r2c<false, 32, 8>);
    allow_big_lds(k_fft_z_r2c<false, 32, 12>);
    allow_big_lds(k_fft_z_r2c<false, 32, 16>);
    allow_big_lds(k_fft_z_c2r<1, 8, kEPT>);
    allow_big_lds(k_fft_z_c2r<1, 16, kEPT>);
    allow_big_lds(k_fft_z_c2r<1, 32, kEPT>);
    allow_big_lds(k_fft_z_c2r<3, 4, 8>);
    allow_big_lds(k_fft_z_c2r<3, 4, 12>);
    allow_big_lds(k_fft_z_c2r<3, 4, 16>);
    allow_big_lds(k_fft_z_c2r<3, 8, 8>);
    allow_big_lds(k_fft_z_c2r<3, 8, 12>);
    allow_big_lds(k_fft_z_c2r<3, 8, 16>);
    allow_big_lds(k_fft_z_c2r<3, 16, 8>);
    allow_big_lds(k_fft_z_c2r<3, 16, 12>);
    allow_big_lds(k_fft_z_c2r<3, 16, 16>);
  }
};

void ensure_init() { static Init once; }

// One workgroup per work item (the table's total is a multiple of 8, so blockIdx.x % 8 is the item's XCD slot).
unsigned item_grid(int total) { return total > 0 ? static_cast<unsigned>(total) : 0u; }


}  // namespace

size_t lds_z_r2c(int n, int B) { return sizeof(float2) * (static_cast<size_t>(n / 2) * (B + 1) + n / 2 + n / 2 + 1); }
size_t lds_axis(int n, int B) { return sizeof(float2) * (static_cast<size_t>(n) * strided_pitch(B) + n); }
// Points per thread of a strided tile of B columns at length n (n B / kFftNT), rounded up to 8, 12 or 16.
int axis_points(int n, int B) {
  const long pts = (static_cast<long>(n) * B + kFftNT - 1) / kFftNT;
  return pts <= 8 ? 8 : (pts <= 12 ? 12 : 16);
}

// Points per thread of a forward r2c z tile of B rows (B columns of length n / 2), rounded up to 8, 12 or 16.
int r2c_points(int n, int B) {
  const long pts = (static_cast<long>(n / 2) * B + kFftNT - 1) / kFftNT;
  return pts <= 8 ? 8 : (pts <= 12 ? 12 : 16);
}

// Points per thread of a three-spectrum c2r z tile of R rows (B = 3 R columns of length n / 2, S = kFftNT / B
// threads per column), rounded up to 8, 12 or 16 (the kernel's EPT).
int c2r_points(int n, int R) {
  const int S = kFftNT / (3 * R);
  const int pts = (n / 2 + S - 1) / S;
  return pts <= 8 ? 8 : (pts <= 12 ? 12 : 16);
}

// Points per thread of the fused x + Poisson tile, n B / kFftNT rounded up to 8, 12 or 16 (the kernel's M).
int poisson_points(int n, int B) {
  const long pts = (static_cast<long>(n) * B + kFftNT - 1) / kFftNT;
  return pts <= 8 ? 8 : (pts <= 12 ? 12 : 16);
}

namespace {
bool same_plan(const Plan1D& pl, std::initializer_list<int> radices) {
  return pl.nst == static_cast<int>(radices.size()) && std::equal(radices.begin(), radices.end(), pl.radix);
}
}  // namespace

bool has_fixed_plan(const Plan1D& pl, int B, int P) {
#define LPC_SAME(...) same_plan(pl, {__VA_ARGS__}) ||
  return plan_fits(pl.n, pl.nst, B, P) && (LPC_FIXED_PLANS(LPC_SAME) false);
}

bool poisson_chainable(const Plan1D& pl) {
  return plan_fits(pl.n, pl.nst, 8, poisson_points(pl.n, 8)) && (LPC_CHAINED_PLANS(LPC_SAME) false);
#undef LPC_SAME
}

size_t lds_x_poisson(int n, int B, int M, bool chained) {
  const size_t tiles = (chained || M <= 12) ? 1 : 2;
  // tile(s), the stage twiddles (the chained form's two tables take turns), the window
  return sizeof(float2) * (tiles * static_cast<size_t>(n) * strided_pitch(B) + n) + sizeof(float) * (n / 2 + 1);
}
size_t lds_z_c2r(int n, int B) {
  return sizeof(float2) * (static_cast<size_t>(n / 2 + 1) * (B + 1) + n / 2 + n / 2 + 1);
}

// Columns of a strided tile: the most of 8, 16, 32 with n * B <= kTileElems (8 for n > 512), and at most `most`.
int strided_cols(int n, int most) { return std::min(most, (n <= 256) ? 32 : (n <= 512 ? 16 : 8)); }

namespace {

// A z-pass tile of B interleaved columns (rows times spectra) at length n: the loads cover B (h + 1) values with
// kEPT + 1 per thread, and each of the S = kFftNT / B threads of a column takes at most kEPT points per stage.
bool rows_fit(int n, int B) {
  const long h = n / 2;
  return B >= 1 && B <= kFftNT && B * (h + 1) <= kTileElems + kFftNT &&
         h * B <= static_cast<long>(kEPT) * (kFftNT / B) * B;
}

// A strided tile of B columns at length n: n B values loaded with kEPT per thread, kEPT points per thread per stage.
bool cols_fit(int n, int B) {
  return B >= 1 && B <= kFftNT && static_cast<long>(n) * B <= static_cast<long>(kEPT) * (kFftNT / B) * B;
}

constexpr size_t kMaxLds = 160 * 1024;

}  // namespace

// Rows of a z-pass tile for NC interleaved spectra: the largest power of two up to 32 that fits (rows_fit).
int z_rows(int n, int nc) {
  int best = 1;
  for (int r = 1; r <= 32; r *= 2) {
    if (!rows_fit(n, nc * r)) break;
    best = r;
  }
  return best;
}

bool tile_ok(TileKind kind, int n, int w) {
  switch (kind) {
    case TileKind::kZRows:  // forward r2c and single-spectrum c2r z passes (instances 8, 16, 32)
      return (w == 8 || w == 16 || w == 32) && rows_fit(n, w) && lds_z_r2c(n, w) <= kMaxLds &&
             lds_z_c2r(n, w) <= kMaxLds;
    case TileKind::kAxisCols:  // strided y / x passes (instances 8, 16, 32)
      return (w == 8 || w == 16 || w == 32) && cols_fit(n, w) && lds_axis(n, w) <= kMaxLds;
    case TileKind::kPoissonCols:  // fused x + Poisson pass (instances 4, 8, 16)
      return (w == 4 || w == 8 || w == 16) && cols_fit(n, w) &&
             lds_x_poisson(n, w, poisson_points(n, w), false) <= kMaxLds;
    case TileKind::kForceC2RRows:  // three-component c2r z pass (instances 4, 8, 16)
      return (w == 4 || w == 8 || w == 16) && rows_fit(n, 3 * w) && lds_z_c2r(n, 3 * w) <= kMaxLds;
  }
  return false;
}

void init_kernels() {
  ensure_init();
  init_axis();
  init_y_grad();
  init_poisson();
}

hipError_t launch_z_r2c(const ZR2CJob* jobs, WorkTable wt, bool fixed, int B, int P, size_t lds, int* flags,
                        hipStream_t s) {
  ensure_init();
  const unsigned g = item_grid(wt.total);
  if (g == 0) return hipSuccess;
  if ((B != 8 && B != 16 && B != 32) || (P != 8 && P != 12 && P != 16)) return hipErrorInvalidValue;
#define LPC_ZR2C(F, BB, PP) k_fft_z_r2c<F, BB, PP><<<g, kFftNT, lds, s>>>(jobs, wt.offs, wt.njob, wt.total, flags)
#define LPC_ZR2C_P(F, BB) \
  if (P == 8) LPC_ZR2C(F, BB, 8); else if (P == 12) LPC_ZR2C(F, BB, 12); else LPC_ZR2C(F, BB, 16)
  if (fixed) {
    if (B == 8) { LPC_ZR2C_P(true, 8); } else if (B == 16) { LPC_ZR2C_P(true, 16); } else { LPC_ZR2C_P(true, 32); }
  } else {
    if (B == 8) { LPC_ZR2C_P(false, 8); } else if (B == 16) { LPC_ZR2C_P(false, 16); } else { LPC_ZR2C_P(false, 32); }
  }
#undef LPC_ZR2C_P
#undef LPC_ZR2C
  return hipGetLastError();
}

hipError_t launch_z_c2r(const ZC2RJob* jobs, WorkTable wt, int nc, int R, int P, size_t lds, hipStream_t s) {
  ensure_init();
  const unsigned g = item_grid(wt.total);
  if (g == 0) return hipSuccess;
#define LPC_ZC2R(NC, RR, PP) k_fft_z_c2r<NC, RR, PP><<<g, kFftNT, lds, s>>>(jobs, wt.offs, wt.njob, wt.total)
  if (nc == 1) {
    if (R == 8) LPC_ZC2R(1, 8, kEPT); else if (R == 16) LPC_ZC2R(1, 16, kEPT); else if (R == 32) LPC_ZC2R(1, 32, kEPT);
    else return hipErrorInvalidValue;
  } else if (nc == 3) {
    if (R == 4 && P == 8) LPC_ZC2R(3, 4, 8);
    else if (R == 4 && P == 12) LPC_ZC2R(3, 4, 12);
    else if (R == 4 && P == 16) LPC_ZC2R(3, 4, 16);
    else if (R == 8 && P == 8) LPC_ZC2R(3, 8, 8);
    else if (R == 8 && P == 12) LPC_ZC2R(3, 8, 12);
    else if (R == 8 && P == 16) LPC_ZC2R(3, 8, 16);
    else if (R == 16 && P == 8) LPC_ZC2R(3, 16, 8);
    else if (R == 16 && P == 12) LPC_ZC2R(3, 16, 12);
    else if (R == 16 && P == 16) LPC_ZC2R(3, 16, 16);
    else return hipErrorInvalidValue;
  } else {
    return hipErrorInvalidValue;
  }
#undef LPC_ZC2R
  return hipGetLastError();
}

}  // namespace kern
}  // namespace lpc
