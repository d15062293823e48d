// DIAM kernels for gfx950.  Every kernel is written for 64-wide wavefronts;
// dense contractions run on MFMA through the tile engines of gemm.h.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "gemm.h"
#include "kernels.h"

using namespace gemm;

namespace dk {

// x' = x_ref + rho (x - x_ref) + xi, one rounding sequence used everywhere
// the proposal of a state is formed (propose and accept must agree bitwise).
DEV double propose1(double xr, double x, double rho, double xi) { return __fma_rn(rho, x - xr, xr) + xi; }

// ============================================================================
// (b) target log-density: Gaussian, Y = R (x - mu) on MFMA, then column sums
// of Y^2 in FP64 per 64-row block (the caller adds the blocks in order).
// ============================================================================
// One output tile: rows [bx BM, +BM) of Y, chains [by BN, +BN); the tile's
// FP64 partial sums go to part[j * ldp + bx] (chain-major: a chain's ldp
// row-block partials are contiguous for the reader).
template <typename T, int BK, int BM, int BN, int KG>
DEV void tgt_gauss_tile(const T* __restrict__ R, const T* __restrict__ V, int d, int P, int bx, int by,
                        double* __restrict__ part, int ldp, const double* __restrict__ twist = nullptr) {
  __shared__ T lds[KG * e_lds_elems<T, BM, BN, BK>()];
  __shared__ double red[2][BN];
  const int i0 = bx * BM, j0 = by * BN;
  EFrag<T, BM, BN> f;
  f.zero();
  e_gemm<T, BM, BN, BK, true, true, KG>(f, R, d, d, V, d, P, i0, j0, 0, d, lds);
  const bool g0 = threadIdx.x < NT;
  const int lane = threadIdx.x & 63, w = (threadIdx.x & (NT - 1)) >> 6, wm = w & 1, wn = w >> 1;
  if (g0) {
#pragma unroll
    for (int n = 0; n < EFrag<T, BM, BN>::FN; ++n) {
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < EFrag<T, BM, BN>::FM; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double y = (double)f.c[m][n][r];
          if (twist) {
            // twisted target: row 2k+1 gets c y_{2k}^2 added before squaring.  Its
            // partner row sits in the same lane (FP32 layout: rows 4q + r) or in
            // lane ^ 16 (FP64 layout: rows 4r + q)
            const double yp = (sizeof(T) == 8) ? lane_xor_f64<16>(y) : (double)f.c[m][n][r & ~1];
            int ti, tj;
            frag_coords<BM, BN, T>(m, n, r, ti, tj);
            const int i = i0 + ti;
            if ((i & 1) && i < d) y = __fma_rn(twist[i], yp * yp, y);
          }
          s = __fma_rn(y, y, s);
        }
      s += lane_xor_f64<16>(s);
      s += lane_xor_f64<32>(s);
      if (lane < 16) red[wm][wn * (BN / 2) + n * 16 + lane] = s;
    }
  }
  __syncthreads();
  if (threadIdx.x < BN) {
    const int j = j0 + threadIdx.x;
    if (j < P) part[(long)j * ldp + bx] = -0.5 * (red[0][threadIdx.x] + red[1][threadIdx.x]);
  }
}

template <typename T, int BK>
__global__ __launch_bounds__(512) void k_tgt_gauss(const T* __restrict__ R, const T* __restrict__ V, int d, int P,
                                                   double* __restrict__ part, const double* __restrict__ twist) {
  tgt_gauss_tile<T, BK, 64, 64, 2>(R, V, d, P, blockIdx.x, blockIdx.y, part, gridDim.x, twist);
}

// The same on the direct-to-LDS engine: rows [bx BM, +BM) x chains [by BN, +BN)
// by WGM x WGN waves and SETS interleaved chains of 128-byte slices of K (two
// in FP32, as the tile above).  Every two waves' rows make one partial, so a
// tile writes WGM / 2 of them per chain (ldp per chain in all); FP32 tiles with
// the same rows per wave and chains write the element engine's partials bit for
// bit.  FP64 (one chain, pairs of consecutive k) sums in another order.
template <typename T, int BM, int BN, int WGM, int WGN, int ST, int SETS>
DEV void tgt_tile_t(const T* __restrict__ R, const T* __restrict__ V, int d, int P, int bx, int by,
                    double* __restrict__ part, int ldp, const double* __restrict__ twist = nullptr) {
  typedef TFrag<T, BM, BN, WGM, WGN> F;
  constexpr int NTH = 64 * WGM * WGN, NS = WGM / 2;
  static_assert(WGM % 2 == 0 && 2 * WGM * BN <= t_lds_elems<T, BM, BN, ST>(), "two waves' rows per partial");
  __shared__ __attribute__((aligned(1024))) T lds[t_lds_elems<T, BM, BN, ST>()];
  const int i0 = bx * BM, j0 = by * BN;
  F f[SETS];
#pragma unroll
  for (int x = 0; x < SETS; ++x) f[x].zero();
  t_gemm<T, BM, BN, WGM, WGN, ST, true, true, sizeof(T) == 8, SETS>(f, R, d, d, V, d, P, i0, j0, 0, d, lds);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, wm = w % WGM, wn = w / WGM;
  double (*red)[BN] = (double (*)[BN])lds;
  __syncthreads();  // the ring's last reads are done
#pragma unroll
  for (int n = 0; n < F::FN; ++n) {
    double s = 0.0;
#pragma unroll
    for (int m = 0; m < F::FM; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int ti, tj;
        t_coords<T, BM, BN, WGM, WGN>(m, n, r, ti, tj);
        const int i = i0 + ti;
        auto total = [&](int rr) {
          T t = f[0].c[m][n][rr];
#pragma unroll
          for (int x = 1; x < SETS; ++x) t += f[x].c[m][n][rr];
          return (double)t;
        };
        double y = total(r);
        if (twist) {
          // a twisted row's partner: this lane (FP32) or lane ^ 16 (FP64), as above
          const double yp = (sizeof(T) == 8) ? lane_xor_f64<16>(y) : total(r & ~1);
          if ((i & 1) && i < d) y = __fma_rn(twist[i], yp * yp, y);
        }
        // rows past the operand repeat its last one
        if (i < d) s = __fma_rn(y, y, s);
      }
    s += lane_xor_f64<16>(s);
    s += lane_xor_f64<32>(s);
    if (lane < 16) red[wm][wn * (BN / WGN) + n * 16 + lane] = s;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < BN * NS; e += NTH) {
    const int c = e % BN, q = e / BN, j = j0 + c;
    if (j < P && bx * NS + q < ldp) part[(long)j * ldp + bx * NS + q] = -0.5 * (red[2 * q][c] + red[2 * q + 1][c]);
  }
}

template <int BM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_tgt_gauss_t(
    const double* __restrict__ R, const double* __restrict__ V, int d, int P, double* __restrict__ part,
    const double* __restrict__ twist) {
  tgt_tile_t<double, BM, 32, 2, 2, 4, 1>(R, V, d, P, blockIdx.x, blockIdx.y, part, gridDim.x, twist);
}

// The same contraction where 64 x 64 tiles would leave most of the chip idle
// (16 tiles at d = 1024, P = 64): one workgroup per 16 rows x 16 chains, K
// split over its wavefronts, each with its own accumulator.  A unit of K is
// 128 bytes per row: a wavefront loads it with eight lanes per row (fragments
// straight from global memory would meet 16 rows per quarter-wavefront, four
// times slower), turns it round in an LDS block of its own, so that the K loop
// has no barrier, and multiplies while the next units are in flight.  FP32
// keeps the two interleaved chains of 32-deep slices of the tile kernel (its
// two k-groups) and the order of k inside them, so every product sum is
// bitwise the tile kernel's; FP64 takes eight chains.  The 16 rows are 8 + 8
// rows 16 apart, the rows whose squares the tile kernel adds up in one lane:
// its row-block sum splits into such quarters exactly.  Loads are
// bounds-checked buffer loads: rows, chains and units outside return zero, and
// rows need no alignment.  The chain tiles of the same rows run on one XCD,
// which keeps its part of R (1 MB of 8 at d = 1024 in FP64) in its L2 from
// step to step.  d = 1024, P = 64: FP64 40.3 to 7.6 us, FP32 22.8 to 8.7 us;
// P = 256: 39.6 to 18.6 and 22.8 to 12.3 us.
template <typename T> struct TS {
  static constexpr int KW = sizeof(T) == 8 ? 8 : 2;  // chains of K, one wavefront each
  static constexpr int D = sizeof(T) == 8 ? 2 : 4;   // units in flight beside the one multiplied
};
template <typename T>
struct TSUnit {
  u32x4_t a[2], b[2];
};

template <typename T>
__global__ __launch_bounds__(64 * TS<T>::KW) void k_tgt_split(const T* __restrict__ R, const T* __restrict__ V, int d,
                                                              int P, double* __restrict__ part, int nh, int nct,
                                                              const double* __restrict__ twist) {
  constexpr int KW = TS<T>::KW, D = TS<T>::D, UK = tbk<T>(), VEC = 16 / (int)sizeof(T);
  __shared__ __attribute__((aligned(16))) T stage[KW][2][16 * UK];
  __shared__ T ys[KW][16][17];
  const int xcd = blockIdx.x & 7, kb = blockIdx.x >> 3;
  const int hb = (kb / nct) * 8 + xcd, ct = kb % nct;
  if (hb >= nh) return;  // uniform per workgroup, before any barrier
  const int lane = threadIdx.x & 63, g = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int i0 = (hb >> 1) * 32 + (hb & 1) * 8, j0 = ct * 16;
  const int mc = min(16, P - j0);
  const T* A = R + (long)i0 * d;
  const T* B = V + (long)j0 * d;
  const __amdgpu_buffer_rsrc_t ra =
      __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, (int)(max(0, min(24, d - i0)) * (long)d * sizeof(T)), 0x00027000);
  const __amdgpu_buffer_rsrc_t rb =
      __builtin_amdgcn_make_buffer_rsrc((void*)B, 0, (int)((long)mc * d * sizeof(T)), 0x00027000);
  // this lane's part of a unit: two 16-byte chunks of each operand (8 rows x
  // 128 bytes per load), and where they go in the wavefront's LDS block
  uint32_t oa[2], ob[2];
  int sw[2];
  const int ch = lane & 7;
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int t = v * 8 + (lane >> 3);
    oa[v] = (uint32_t)((((t & 7) + 2 * (t & 8)) * (long)d + ch * VEC) * (long)sizeof(T));
    ob[v] = (uint32_t)((t * (long)d + ch * VEC) * (long)sizeof(T));
    sw[v] = t * UK + ((ch ^ tswz(t)) * VEC);
  }
  T* sa = stage[g][0];
  T* sb = stage[g][1];
  const int nfull = d / UK;
  // whole units of this wavefront; past them loads lie outside and give zeros
  const int cnt = nfull > g ? (nfull - g + KW - 1) / KW : 0;
  auto load = [&](TSUnit<T>& u, int n) {
    const uint32_t k = n < cnt ? (uint32_t)((g + KW * n) * UK * (int)sizeof(T)) : 0x80000000u;
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      u.a[v] = __builtin_amdgcn_raw_buffer_load_b128(ra, oa[v] + k, 0, 0);
      u.b[v] = __builtin_amdgcn_raw_buffer_load_b128(rb, ob[v] + k, 0, 0);
    }
  };
  typename EAcc<T>::V c = {T(0), T(0), T(0), T(0)};
  // LDS instructions of a wavefront run in order, so its block needs no wait
  // between the reads of one unit and the writes of the next
  auto mma = [&](const TSUnit<T>& u) {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      *(u32x4_t*)(sa + sw[v]) = u.a[v];
      *(u32x4_t*)(sb + sw[v]) = u.b[v];
    }
    asm volatile("" ::: "memory");
    if (sizeof(T) == 8) {
      // a lane's two chunks of consecutive k feed four products
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        const int p = lr * UK + (((lk + 4 * v) ^ tswz(lr)) * VEC);
        T av[VEC], bv[VEC];
        *(u32x4_t*)av = *(const u32x4_t*)(sa + p);
        *(u32x4_t*)bv = *(const u32x4_t*)(sb + p);
#pragma unroll
        for (int e = 0; e < VEC; ++e) c = mfma_e<T>(av[e], bv[e], c);
      }
    } else {
      T av[UK / 4], bv[UK / 4];
#pragma unroll
      for (int q = 0; q < UK / 4; ++q) {
        const int p = t_index_kc<T>(lr, 4 * q + lk);
        av[q] = sa[p];
        bv[q] = sb[p];
      }
#pragma unroll
      for (int q = 0; q < UK / 4; ++q) c = mfma_e<T>(av[q], bv[q], c);
    }
    asm volatile("" ::: "memory");
  };
  const bool has_tail = d % UK != 0 && nfull % KW == g;
  TSUnit<T> tail;
  if (has_tail) {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      const int t = v * 8 + (lane >> 3), ar = (t & 7) + 2 * (t & 8), k0 = nfull * UK + ch * VEC;
      T ta[VEC], tb[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        ta[e] = (i0 + ar < d && k0 + e < d) ? A[(long)ar * d + k0 + e] : T(0);
        tb[e] = (t < mc && k0 + e < d) ? B[(long)t * d + k0 + e] : T(0);
      }
      tail.a[v] = *(const u32x4_t*)ta;
      tail.b[v] = *(const u32x4_t*)tb;
    }
  }
  TSUnit<T> st[D];
#pragma unroll
  for (int x = 0; x < D; ++x) load(st[x], x);
  for (int n = 0; n < cnt; n += D) {
#pragma unroll
    for (int x = 0; x < D; ++x) {
      if (n + x < cnt) mma(st[x]);
      load(st[x], n + x + D);
    }
  }
  if (has_tail) mma(tail);
#pragma unroll
  for (int r = 0; r < 4; ++r) ys[g][sizeof(T) == 8 ? 4 * r + lk : 4 * lk + r][lr] = c[r];
  __syncthreads();
  if (g != 0) return;
  // lane (lk, lr): rows 8 (hb % 2) + 4 (lk % 2) + r of both 16-row blocks of
  // chain lr, in the tile kernel's order; a twisted row's partner is its own
  double s = 0.0;
#pragma unroll
  for (int mm = 0; mm < 2; ++mm) {
    double prev = 0.0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = mm * 8 + 4 * (lk & 1) + r, i = i0 + (t & 7) + 2 * (t & 8);
      T y0 = ys[0][t][lr];
#pragma unroll
      for (int q = 1; q < KW; ++q) y0 += ys[q][t][lr];
      double y = (double)y0;
      if (twist && (r & 1) && i < d) y = __fma_rn(twist[i], prev * prev, y);
      prev = (double)y0;
      s = __fma_rn(y, y, s);
    }
  }
  s += lane_xor_f64<16>(s);
  if (lane < mc) part[(long)(j0 + lane) * nh + hb] = -0.5 * s;
}

// ---- two-part half target (mixed form): Y = R V with both operands split
// into two IEEE half parts (products with the accuracy of FP32, see h2_gemm).
// Half precision needs operands in its range, so both are scaled by powers of
// two, exactly: coordinate k of x - mu by 2^s_k (vsc), chosen from the
// largest deviation of the current states and the current factor's row norm
// so that values up to 1024 times those stay finite (the step kernel flags
// any beyond); row i of R by
// 2^(a_i - s_k) so that its largest entry lies in [2^14, 2^15).  Then
// (R' V')_i = 2^a_i (R V)_i and the reduction multiplies by 2^-a_i (rsc).
// 64- or 128-wide tiles, K split in H2_KSPLIT ranges whose FP32 partial Y are
// summed in FP64 by the reduction, which squares and sums 64-row blocks
// (chain-major partials).
constexpr int H2_KSPLIT = 4;
// scaled V entries at or above this magnitude round to infinity in half
constexpr double H2_RANGE = 65520.0;

// vsc[k] = 2^(6 - e_k) with sigma_k < 2^e_k (frexp), sigma_k the larger of
// max_p |x_kp - mu_k| and the 2-norm of row k of the lower factor L
// (column-major; the spread of the proposals), or the former alone for an
// evaluation of the states themselves; e_k clamped to [-100, 100].  64 rows per block, one per
// lane; the 16 waves split the columns of L and the chains.
__global__ __launch_bounds__(1024) void k_h2_vscale(const double* __restrict__ X, const double* __restrict__ mu,
                                                    const double* __restrict__ L, int d, int P, int states_only,
                                                    float* __restrict__ vsc) {
  __shared__ double sdev[16][64], srn[16][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int k = blockIdx.x * 64 + lane;
  double dev = 0.0, rn = 0.0;
  if (k < d) {
    const double mk = mu[k];
    for (int p = w; p < P; p += 16) dev = fmax(dev, fabs(X[k + (long)p * d] - mk));
    for (int j = w; j <= k; j += 16) {
      const double l = L[k + (long)j * d];
      rn = __fma_rn(l, l, rn);
    }
  }
  sdev[w][lane] = dev;
  srn[w][lane] = rn;
  __syncthreads();
  if (w != 0 || k >= d) return;
  for (int q = 1; q < 16; ++q) {
    dev = fmax(dev, sdev[q][lane]);
    rn += srn[q][lane];
  }
  // states_only (the evaluation of the states themselves): their spread
  // alone, the factor's row norm only where they do not spread
  const double sig = (states_only && dev > 0.0) ? dev : fmax(dev, sqrt(rn));
  int e = 0;
  if (sig > 0.0 && isfinite(sig)) {
    frexp(sig, &e);  // sig < 2^e
    e = 6 - e;
  }
  e = e < -100 ? -100 : (e > 100 ? 100 : e);
  vsc[k] = ldexpf(1.0f, e);
}

// Row i of R: a_i from the largest |R_ik / vsc[k]|, then both half parts of
// R_ik 2^a_i / vsc[k] into R2 (d x d each, in the tiled order h2_gemm reads,
// h2_tile_index) and rsc[i] = 2^-a_i.
__global__ __launch_bounds__(256) void k_h2_split_r(const float* __restrict__ R, const float* __restrict__ vsc, int d,
                                                    u16* __restrict__ R2, double* __restrict__ rsc) {
  __shared__ float red[4];
  const int i = blockIdx.x, t = threadIdx.x;
  const float* row = R + (long)i * d;
  float mx = 0.0f;
  for (int k = t; k < d; k += 256) mx = fmaxf(mx, fabsf(row[k] / vsc[k]));
  mx = wave_max_f32(mx);
  if ((t & 63) == 0) red[t >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  int e = 0;
  if (mx > 0.0f && isfinite(mx)) {
    frexpf(mx, &e);  // mx < 2^e
    e = 15 - e;
  }
  const long n = (long)d * d;
  const int arb = d / 16;
  for (int k = t; k < d; k += 256) {
    const double v = ldexp((double)row[k] / (double)vsc[k], e);
    u16 h, l;
    split_f16(v, h, l);
    const long q = h2_tile_index(i, k, arb);
    R2[q] = h;
    R2[n + q] = l;
  }
  if (t == 0) rsc[i] = ldexp(1.0, -e);
}

// Both half parts of (x - mu) vsc into V2 (d x P each, column-major).
__global__ __launch_bounds__(256) void k_h2_split_v(const double* __restrict__ X, const double* __restrict__ mu,
                                                    const float* __restrict__ vsc, int d, long n,
                                                    u16* __restrict__ V2) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= n) return;
  const int k = (int)(e % d);
  u16 h, l;
  split_f16((X[e] - mu[k]) * (double)vsc[k], h, l);
  V2[e] = h;
  V2[n + e] = l;
}

hipError_t h2_scales(const double* X, const double* mu, const double* L, const float* R, int d, int P, float* vsc,
                     uint16_t* R2, double* rsc, hipStream_t s, int states_only) {
  hipLaunchKernelGGL(k_h2_vscale, dim3((unsigned)((d + 63) / 64)), dim3(1024), 0, s, X, mu, L, d, P, states_only,
                     vsc);
  hipLaunchKernelGGL(k_h2_split_r, dim3(d), dim3(256), 0, s, R, (const float*)vsc, d, (u16*)R2, rsc);
  return hipGetLastError();
}

hipError_t h2_split_v(const double* X, const double* mu, const float* vsc, int d, int P, uint16_t* V2,
                      hipStream_t s) {
  const long n = (long)d * P;
  hipLaunchKernelGGL(k_h2_split_v, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, X, mu, vsc, d, n, (u16*)V2);
  return hipGetLastError();
}

template <int BM, int BN, int WGM, int WGN, int ST>
__global__ __launch_bounds__(64 * WGM * WGN) void k_tgt_h2(const u16* __restrict__ R2, const u16* __restrict__ V2,
                                                          int d, int P, float* __restrict__ Yp) {
  typedef W32Frag<BM, BN, WGM, WGN> F;
  __shared__ __attribute__((aligned(1024))) u16 lds[h2_lds_elems<BM, BN, ST>()];
  int i0 = blockIdx.x * BM, j0 = blockIdx.y * BN, ks = blockIdx.z;
  if (gridDim.y == 1 && gridDim.z == 1) {
    // one-dimensional grid: workgroups go round-robin to the eight XCDs, and
    // XCDs x and x + 4 take K range x mod 4, each half of the (row, chain)
    // tiles, a row block's chain tiles adjacent; an XCD then reads only its
    // quarter of x - mu and each tile of R once (requires the split into 4
    // and an even number of (row, chain) tiles, checked by the launcher)
    const int ncb = P / BN, half = (d / BM) * ncb / 2;
    const int xcd = blockIdx.x & 7, q = (xcd >> 2) * half + (blockIdx.x >> 3);
    ks = xcd & 3;
    i0 = (q / ncb) * BM;
    j0 = (q % ncb) * BN;
  }
  const int kl = d / H2_KSPLIT;
  // the output pointer is loaded before the loop: a scalar load left in
  // flight there would make every LDS wait of the pipelined loop a full one
  float* Y = Yp + (long)ks * P * d;
  asm volatile("" ::"s"(Y));
  F f;
  f.zero();
  h2_gemm<BM, BN, WGM, WGN, ST>(f, R2, (long)d * d, d / 16, V2, (long)d * P, d, i0, j0, ks * kl, (ks + 1) * kl,
                                lds);
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        int ti, tj;
        w32_coords<BM, BN, WGM, WGN>(m, n, g, ti, tj);
        // four consecutive rows of one chain: one 16-byte store
        const f4_t v = {f.c[m][n][4 * g], f.c[m][n][4 * g + 1], f.c[m][n][4 * g + 2], f.c[m][n][4 * g + 3]};
        *(f4_t*)(Y + (long)(j0 + tj) * d + i0 + ti) = v;
      }
}

// part[j][rb] = -1/2 sum over rows of block rb of (rsc_i sum_s Yp[s])^2.  One
// wave per chain and four 64-row blocks: lane l takes rows 4l .. 4l + 3 of the
// wave's 256 (16-byte loads), sixteen lanes make one block (d is a multiple
// of 64, so a block is wholly inside or outside).
// Rows 256 q4 .. 256 q4 + 255 of chain j on one wavefront: the four row-block
// terms go to part; every lane returns its block's term.
DEV double h2_reduce_wave(const float* __restrict__ Yp, const double* __restrict__ rsc, int d, int P, int nrb,
                          double* __restrict__ part, const double* __restrict__ twist, int j, int q4) {
  const int lane = threadIdx.x & 63;
  const int i = q4 * 256 + 4 * lane;
  double q = 0.0;
  if (i < d) {
    double y[4] = {0.0, 0.0, 0.0, 0.0};
    for (int s = 0; s < H2_KSPLIT; ++s) {
      const f4_t v = *(const f4_t*)(Yp + ((long)s * P + j) * d + i);
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] += (double)v[r];
    }
    const double2 r01 = *(const double2*)(rsc + i), r23 = *(const double2*)(rsc + i + 2);
    y[0] *= r01.x;
    y[1] *= r01.y;
    y[2] *= r23.x;
    y[3] *= r23.y;
    if (twist) {
      // twisted target: row 2k+1 gets c y_{2k}^2 (pairs lie within a lane)
      y[1] = __fma_rn(twist[i + 1], y[0] * y[0], y[1]);
      y[3] = __fma_rn(twist[i + 3], y[2] * y[2], y[3]);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) q = __fma_rn(y[r], y[r], q);
  }
  q = row16_sum_f64(q);
  const int rb = q4 * 4 + (lane >> 4);
  if ((lane & 15) == 0 && i < d) part[(long)j * nrb + rb] = -0.5 * q;
  return -0.5 * q;
}

__global__ __launch_bounds__(256) void k_tgt_h2_reduce(const float* __restrict__ Yp, const double* __restrict__ rsc,
                                                       int d, int P, int nrb, double* __restrict__ part,
                                                       const double* __restrict__ twist) {
  const int nq = (nrb + 3) / 4;
  const long wid = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (wid >= (long)P * nq) return;
  h2_reduce_wave(Yp, rsc, d, P, nrb, part, twist, (int)(wid / nq), (int)(wid % nq));
}

#ifndef TGT_H2_XMAP
#define TGT_H2_XMAP 1
#endif
bool tgt_h2_ok(int d, int P) { return d % (H2_KSPLIT * 32) == 0 && d % 64 == 0 && P % 64 == 0; }

size_t tgt_h2_scratch_bytes(int d, int P) { return (size_t)H2_KSPLIT * d * P * sizeof(float); }

hipError_t tgt_gauss_h2(const uint16_t* R2, const uint16_t* V2, const double* rsc, int d, int P, float* Yp,
                        double* part, hipStream_t s, const double* twist) {
  // 128 x 128 tiles on 8 waves where they fit
  static_assert(H2_KSPLIT == 4, "the XCD mapping pairs the eight XCDs with four K ranges");
  if (d % 128 == 0 && P % 128 == 0 && (d / 128) * (P / 128) % 2 == 0 && TGT_H2_XMAP)
    hipLaunchKernelGGL((k_tgt_h2<128, 128, 4, 2, 4>), dim3((d / 128) * (P / 128) * H2_KSPLIT), dim3(512), 0, s,
                       (const u16*)R2, (const u16*)V2, d, P, Yp);
  else if (d % 128 == 0 && P % 128 == 0)
    hipLaunchKernelGGL((k_tgt_h2<128, 128, 4, 2, 4>), dim3(d / 128, P / 128, H2_KSPLIT), dim3(512), 0, s,
                       (const u16*)R2, (const u16*)V2, d, P, Yp);
  else
    hipLaunchKernelGGL((k_tgt_h2<64, 64, 2, 2, 4>), dim3(d / 64, P / 64, H2_KSPLIT), dim3(256), 0, s,
                       (const u16*)R2, (const u16*)V2, d, P, Yp);
  if (!part) return hipGetLastError();  // the reduction runs inside the step (step_h2)
  const int nrb = tgt_row_blocks(d);
  const long waves = (long)P * ((nrb + 3) / 4);
  hipLaunchKernelGGL(k_tgt_h2_reduce, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, (const float*)Yp, rsc, d,
                     P, nrb, part, twist);
  return hipGetLastError();
}

// Which kernel, by the split kernel's workgroups w (16 rows x 16 chains, its
// time in proportion to them beyond one per CU) and the number n of 64 x 64
// tiles (the tile kernels take the time of one tile up to n = 256, twice that
// where the tile is not whole).  us between events, about 2 more than a kernel:
//   d, P           n    w      FP64: split  32 x 32  64 x 32    FP32: split  tile kernel
//   64, 1024       16   256          6.2    6.2      6.2              6.2    6.3
//   64, 8192       128  2048         19.2   6.3      6.3              12.4   6.3
//   128, 1024      32   512          7.0    6.3      7.6              6.4    7.7
//   256, 512       32   512          8.0    8.2      10.5             7.1    10.0
//   256, 2048      128  2048         18.2   10.1     10.7             11.1   10.5
//   512, 384       48   768          11.7   11.9     16.5             10.0   15.5
//   512, 1024      128  2048         24.1   14.6     16.7             14.0   15.5
//   700, 384       66   1056         20.4   18.4     21.2             16.2   29.0
//   700, 1024      176  2816         46.7   25.2     29.9             26.1   29.3
//   1024, 192      48   768          16.7   19.3     28.1             14.4   25.2
//   1024, 256      64   1024         22.2   19.5     27.9             15.3   25.0
//   1024, 768      192  3072         53.2   32.7     39.8             30.6   25.1
//   2048, 128      64   1024         34.9   33.9     51.4             24.4   44.9
//   3000, 256      188  3008         140    93.6     111              77.6   112
//   4096, 16       64   256          31.6   62.1     98.3
//   4096, 64       64   1024         62.8   63.7     98.3             40.8   84.3
//   8192, 32       128  1024         162    147      196
//   4096, 256      256  4096         210    150      141              121    84.8
//   odd d          n    w      FP64: split, tile kernel
//   65, 2048       64   768          9.1    9.8
//   129, 2048      96   1280         15.0   12.7
//   511, 1024      128  2048         28.2   28.7
//   1023, 768      192  3072         66.4   52.3
// The engine (32 x 32, 64 x 32) needs rows of 16-byte multiples; in FP32, whose
// two chains double its accumulators, it is behind (99.3 us at d = 4096, P =
// 256).
int tgt_gauss_sub(Prec prec, int d, int P) {
  const long w = (long)tgt_quarters(d) * cdiv(P, 16), n = (long)cdiv(d, TGT_BM) * cdiv(P, 64);
  const bool small = d < 384;  // few slices of K: the split has less to share out
  if (prec == P64 && d % 2 == 0) {
    if (small ? P <= 1024 && w <= max(256, 2 * d) : w <= (P <= 64 && d <= 4096 ? 1024 : P <= 128 ? 960 : 768)) return 4;
    return n < 256 ? 2 : 1;
  }
  if (prec == P64) return w <= 2048 && (P <= 1024 || w <= 768) ? 4 : 1;
  if (d % 64 == 0 && P % 64 == 0)  // whole tiles
    return (small ? P <= 2048 && w <= 1280 : P <= 1024 && w <= 2048) ? 4 : 1;
  return P <= 2048 && w <= (small ? 2048 : 3072) ? 4 : 1;
}

// FP64 on the engine's tiles of BM rows; false: rows not aligned for it
template <int BM>
static bool tgt_gauss_t(const void* R, const void* V, int d, int P, double* part, const double* twist, hipStream_t s) {
  if (!t_gemm_ok<double, true, true>(R, d, d, V, d, P, d)) return false;
  hipLaunchKernelGGL((k_tgt_gauss_t<BM>), dim3(cdiv(d, BM), cdiv(P, 32)), dim3(256), 0, s, (const double*)R,
                     (const double*)V, d, P, part, twist);
  return true;
}

hipError_t tgt_gauss(Prec prec, const void* R, const void* V, int d, int P, double* part, hipStream_t s,
                     const double* twist, int sub) {
  if (sub == 4) {
    const int nh = tgt_quarters(d), nct = cdiv(P, 16), groups = (nh + 7) / 8;
    if (prec == P64)
      hipLaunchKernelGGL((k_tgt_split<double>), dim3(groups * 8 * nct), dim3(64 * TS<double>::KW), 0, s,
                         (const double*)R, (const double*)V, d, P, part, nh, nct, twist);
    else
      hipLaunchKernelGGL((k_tgt_split<float>), dim3(groups * 8 * nct), dim3(64 * TS<float>::KW), 0, s,
                         (const float*)R, (const float*)V, d, P, part, nh, nct, twist);
    return hipGetLastError();
  }
  if (sub == 2) {
    if (prec != P64 || !tgt_gauss_t<32>(R, V, d, P, part, twist, s)) return hipErrorInvalidValue;
    return hipGetLastError();
  }
  if (prec == P64 && tgt_gauss_t<64>(R, V, d, P, part, twist, s)) return hipGetLastError();
  dim3 grid(cdiv(d, TGT_BM), cdiv(P, 64));
  if (prec == P64)
    hipLaunchKernelGGL((k_tgt_gauss<double, 16>), grid, dim3(512), 0, s, (const double*)R, (const double*)V, d, P, part,
                       twist);
  else
    hipLaunchKernelGGL((k_tgt_gauss<float, 32>), grid, dim3(512), 0, s, (const float*)R, (const float*)V, d, P, part,
                       twist);
  return hipGetLastError();
}

// ============================================================================
// (a) proposal contraction Xi = c L W, L lower triangular: the K range of a
// row tile stops at its last row.
// ============================================================================
// On the direct-to-LDS engine, Xi^T = W^T L^T so that lanes run along the rows
// of Xi (128-byte stores).  BJ columns of W by
// BI rows of L per workgroup.  64 x 64 tiles, three stages, three workgroups
// per CU measured best at middle sizes (d = 1024, 12800 columns: FP64 565 to
// 306 us, FP32 276 to 179 us).  With many tiles FP64 runs at the chip's power
// limit (about 1.95 GHz), where 128 x 64 tiles, which move less per product,
// are ahead at large d: d = 4096, 65536 columns 29.9 to 17.4 ms against 17.7
// with 64 x 64 (62 TFLOP/s; a large library product reaches 68 there), 32768
// columns 8.7 against 9.2.  At 8192 tiles, where the rule changes over, the two
// differ by -4 to +3 % (64 x 64 / 128 x 64, ms: d = 451 0.44 / 0.46, 1024 0.68 /
// 0.69, 2048 1.21 / 1.23, 4096 2.26 / 2.19), at 4096 tiles by -7 to +7 % (d =
// 512 0.22 / 0.23, 1024 0.35 / 0.37, 4096 1.18 / 1.10), below that 64 x 64 is
// ahead by 10 % at d = 1024.  32 x 32 tiles where 64 x 64 would not give every CU two.
template <typename T, int BJ, int BI, int ST, bool NARROW = false>
DEV void trigemm_tile_t(const T* __restrict__ L, const T* __restrict__ W, T* __restrict__ Xi, int d, int ncols, double c,
                        int bi, int bj) {
  typedef TFrag<T, BJ, BI, 2, 2> F;
  __shared__ __attribute__((aligned(1024))) T lds[t_lds_elems<T, BJ, BI, ST>()];
  const int i0 = bi * BI, j0 = bj * BJ;
  F f;
  f.zero();
  t_gemm<T, BJ, BI, 2, 2, ST, true, false, false, 1, 1, false, NARROW>(*(F(*)[1]) & f, W, d, ncols, L, d, d, j0, i0, 0,
                                                                       min(d, i0 + BI), lds);
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int ti, tj;
        t_coords<T, BJ, BI, 2, 2>(m, n, r, tj, ti);
        const int i = i0 + ti, j = j0 + tj;
        if (i < d && j < ncols) Xi[i + (long)j * d] = (T)(c * (double)f.c[m][n][r]);
      }
}

// Workgroup ids are dealt round-robin to the 8 XCDs: ids xcd + 8 k on one XCD
// take the row blocks of one column block of W, longest K range first, so that
// slice of W is fetched into the XCD's L2 once.
template <typename T, int BJ, int BI, int ST, bool NARROW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_trigemm_t(
    const T* __restrict__ L, const T* __restrict__ W, T* __restrict__ Xi, int d, int ncols, double c, int nj, int ni) {
  const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3;
  const int jb = (k / ni) * 8 + xcd;
  if (jb >= nj) return;
  trigemm_tile_t<T, BJ, BI, ST, NARROW>(L, W, Xi, d, ncols, c, ni - 1 - k % ni, jb);
}

template <typename T, int BJ, int BI, int ST, bool NARROW>
static void trigemm_t_launch(const void* L, const void* W, void* Xi, int d, long ncols, double c, hipStream_t s) {
  const int nj = cdiv(ncols, BJ), ni = cdiv(d, BI);
  hipLaunchKernelGGL((k_trigemm_t<T, BJ, BI, ST, NARROW>), dim3((unsigned)((nj + 7) / 8 * 8) * ni), dim3(256), 0, s,
                     (const T*)L, (const T*)W, (T*)Xi, d, (int)ncols, c, nj, ni);
}

// Operands without 16-byte rows take the engine's narrow copies (d = 75, 3200
// columns: 8.3 us on the element engine, 5.3 so).
template <typename T, bool NARROW>
static void trigemm_t(const void* L, const void* W, void* Xi, int d, long ncols, double c, hipStream_t s) {
  const long tiles = (long)cdiv(d, 64) * cdiv(ncols, 64);
  if (tiles < 512) trigemm_t_launch<T, 32, 32, 6, NARROW>(L, W, Xi, d, ncols, c, s);
  else if (sizeof(T) == 8 && tiles >= 8192) trigemm_t_launch<T, 128, 64, 3, NARROW>(L, W, Xi, d, ncols, c, s);
  else trigemm_t_launch<T, 64, 64, 3, NARROW>(L, W, Xi, d, ncols, c, s);
}
template <typename T>
static hipError_t trigemm_e(const void* L, const void* W, void* Xi, int d, long ncols, double c, hipStream_t s) {
  if (t_gemm_ok<T, true, false>(W, d, (int)ncols, L, d, d, d)) trigemm_t<T, false>(L, W, Xi, d, ncols, c, s);
  else if (d < 1 << 20) trigemm_t<T, true>(L, W, Xi, d, ncols, c, s);  // 32-bit offsets in a tile's slice
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// bf16: Xi^T = W~^T L~^T with the roles swapped so that lanes run along the
// rows i of Xi (coalesced stores): A operand = W (rows = columns j of W,
// k-contiguous), B operand = L~ (rows i, k-contiguous, row-major factor).
// W~ = W_hi + W_lo and L~ = L_hi + L_lo; the four bf16 products run as one
// segmented, pipelined K loop into the same fp32 registers.
// Tile order: workgroup ids are dealt round-robin to the 8 XCDs, so ids
// xcd + 8 k on one XCD take the ni row blocks of one column block of W
// (longest K range first): that slice of W is fetched into the XCD's L2 once.
// Wide variant: TBM (j) x TBN (i) tiles, WGM x WGN wavefronts, 64-deep K slices.
template <int TBM, int TBN, int WGM, int WGN>
__global__ __launch_bounds__(64 * WGM * WGN) void k_trigemm_bf16w(const u16* __restrict__ Lhi,
                                                                 const u16* __restrict__ Whi, long dW,
                                                                 float* __restrict__ Xi, int d, int ncols, float c,
                                                                 int vec_ok, int nj, int ni) {
  typedef WFrag<TBM, TBN, WGM, WGN> F;
  __shared__ u16 lds[w_lds_elems<TBM, TBN>()];
  const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3;
  const int jb = (k / ni) * 8 + xcd;
  if (jb >= nj) return;
  const int ib = ni - 1 - (k % ni);
  const int j0 = jb * TBM, i0 = ib * TBN;
  const int kend = min(d, i0 + TBN);
  F f;
  f.zero();
  w_gemm_seg<TBM, TBN, WGM, WGN>(f, Whi, dW, d, ncols, Lhi, (long)d * d, d, d, vec_ok, j0, i0, 0, kend, 4, lds);
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int tj, ti;
        w_coords<TBM, TBN, WGM, WGN>(m, n, r, tj, ti);
        const int i = i0 + ti, j = j0 + tj;
        if (i < d && j < ncols) Xi[i + (long)j * d] = c * f.c[m][n][r];
      }
}
// Direct-to-LDS hi/lo variant for operands that fill whole tiles (d a
// multiple of 2 TBN, ncols of TBM; 256 x 128 tiles on 8 waves, 3-stage ring): the K range of a row tile ends at its
// last row, so row tiles ib and ni - 1 - ib together cost the same for every
// pair; each workgroup takes one such pair of one column block of W (the
// pairs of a column block run on one XCD, which keeps that block of W in its
// L2).  The four products accumulate per 32-deep slice.
template <int TBM, int TBN, int WGM, int WGN, int ST>
__global__ __launch_bounds__(64 * WGM * WGN) void k_trigemm_hl(const u16* __restrict__ Lhi, const u16* __restrict__ Whi,
                                                              long dW, float* __restrict__ Xi, int d, int ncols, float c,
                                                              int nj, int ni) {
  typedef WFrag<TBM, TBN, WGM, WGN> F;
  __shared__ __attribute__((aligned(1024))) u16 lds[h_lds_elems<TBM, TBN, ST>()];
  const int npair = ni / 2;
  const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3;
  const int jb = (k / npair) * 8 + xcd;
  if (jb >= nj) return;
  const int q = k % npair;
  const int j0 = jb * TBM;
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int ib = h ? q : ni - 1 - q;
    const int i0 = ib * TBN;
    const int kend = min(d, i0 + TBN);
    F f;
    f.zero();
    h_gemm<TBM, TBN, WGM, WGN, ST>(f, Whi, dW, d, Lhi, (long)d * d, d, j0, i0, kend, lds);
#pragma unroll
    for (int m = 0; m < F::FM; ++m)
#pragma unroll
      for (int n = 0; n < F::FN; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int tj, ti;
          w_coords<TBM, TBN, WGM, WGN>(m, n, r, tj, ti);
          Xi[(i0 + ti) + (long)(j0 + tj) * d] = c * f.c[m][n][r];
        }
  }
}

// tile shape of the wide proposal kernel
constexpr int TW_BM = 256, TW_BN = 128, TW_WGM = 4, TW_WGN = 2;

hipError_t trigemm(Prec prec, const void* L, const void* W, const void* Wlo, void* Xi, int d, long ncols, double c,
                   hipStream_t s) {
  if (ncols <= 0) return hipSuccess;
  if (prec == P64) return trigemm_e<double>(L, W, Xi, d, ncols, c, s);
  if (prec == P32) return trigemm_e<float>(L, W, Xi, d, ncols, c, s);
  {
    const u16* Lhi = (const u16*)L;
    const long dW = (const u16*)Wlo - (const u16*)W;
    const int vec_ok = (d % 8 == 0) && ((uintptr_t)L % 16 == 0) && ((uintptr_t)W % 16 == 0) && ((uintptr_t)Wlo % 16 == 0);
    const bool whole = vec_ok && (ncols % 256 == 0);
    if (whole && d % 512 == 0) {
      const int nj = ncols / 256, ni = d / 256, groups = (nj + 7) / 8;
      hipLaunchKernelGGL((k_trigemm_hl<256, 256, 2, 4, 2>), dim3(groups * 8 * (ni / 2)), dim3(512), 0, s, Lhi,
                         (const u16*)W, dW, (float*)Xi, d, (int)ncols, (float)c, nj, ni);
      return hipGetLastError();
    }
    if (whole && d % 256 == 0) {
      const int nj = ncols / 256, ni = d / 128, groups = (nj + 7) / 8;
      hipLaunchKernelGGL((k_trigemm_hl<256, 128, 4, 2, 3>), dim3(groups * 8 * (ni / 2)), dim3(512), 0, s, Lhi,
                         (const u16*)W, dW, (float*)Xi, d, (int)ncols, (float)c, nj, ni);
      return hipGetLastError();
    }
    const int nj = cdiv(ncols, TW_BM), ni = cdiv(d, TW_BN), groups = (nj + 7) / 8;
    hipLaunchKernelGGL((k_trigemm_bf16w<TW_BM, TW_BN, TW_WGM, TW_WGN>), dim3(groups * 8 * ni),
                       dim3(64 * TW_WGM * TW_WGN), 0, s, Lhi, (const u16*)W, dW, (float*)Xi, d, (int)ncols, (float)c,
                       vec_ok, nj, ni);
  }
  return hipGetLastError();
}

// ============================================================================
// (d) window scatter G = sum_k xs_k xs_k^T (lower tiles) and row sums h.
// ============================================================================
DEV void tile_pair(int t, int& bi, int& bj) {
  // t enumerates (bi >= bj) row by row: t = bi (bi + 1)/2 + bj
  int b = (int)((sqrt(8.0 * (double)t + 1.0) - 1.0) * 0.5);
  while ((b + 1) * (b + 2) / 2 <= t) ++b;
  while (b * (b + 1) / 2 > t) --b;
  bi = b;
  bj = t - b * (b + 1) / 2;
}

constexpr int FOLD_K = 4096;  // fp32 accumulation span before folding into fp64

// Lower tile t (row-by-row enumeration) of the scatter over K split ksp, on the
// direct-to-LDS engine (leading dimension ld); lanes
// run along j, so the stores are 128-byte runs of a column of G.
template <typename T, int BT, int ST, bool NARROW = false>
DEV void syrk_tile_t(const T* __restrict__ Xs, int ld, int d, int K, int kchunk, int t, int ksp,
                     double* __restrict__ Gpart, T* lds) {
  typedef TFrag<T, BT, BT, 2, 2> F;
  int bi, bj;
  tile_pair(t, bi, bj);
  const int i0 = bi * BT, j0 = bj * BT;
  const int kb = ksp * kchunk, ke = min(K, kb + kchunk);
  double acc[F::FM][F::FN][4];
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[m][n][r] = 0.0;
  const int span = (sizeof(T) == 8) ? kchunk : FOLD_K;
  for (int k0 = kb; k0 < ke; k0 += span) {
    F f;
    f.zero();
    t_gemm<T, BT, BT, 2, 2, ST, false, false, false, 1, 1, false, NARROW>(*(F(*)[1]) & f, Xs, ld, ld, Xs, ld, ld, i0, j0, k0,
                                                                       min(ke, k0 + span), lds);
#pragma unroll
    for (int m = 0; m < F::FM; ++m)
#pragma unroll
      for (int n = 0; n < F::FN; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m][n][r] += (double)f.c[m][n][r];
  }
  double* G = Gpart + (long)ksp * d * d;
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int ti, tj;
        t_coords<T, BT, BT, 2, 2>(m, n, r, ti, tj);
        const int i = i0 + ti, j = j0 + tj;
        if (i < d && j < d) G[j + (long)i * d] = acc[m][n][r];  // G(i,j) at (row j, col i): upper
      }
}

// Row sums over K of the window.  COLMAJOR: element (i, k) at X[i + k d];
// otherwise at X[i K + k] (bf16 transposed window).
// Each of the four threads of a row adds its values in turn, ROWSUM_U loads in
// flight at a time (one by one the chain took 133 us at d = 100, K = 3200).
constexpr int ROWSUM_U = 32;

template <typename T, bool COLMAJOR>
DEV void rowsum_block(const T* __restrict__ X, int d, long ld, int K, int kchunk, int bx, int by,
                      double* __restrict__ hpart, double (*red)[64]) {
  const int kb = by * kchunk, ke = min(K, kb + kchunk);
  if (COLMAJOR) {
    const int r = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int i = bx * 64 + r;
    double s = 0.0;
    if (i < d) {
      const T* p = X + i;
      int k = kb + q;
      if (k + 4 * (ROWSUM_U - 1) < ke) {
        T v[ROWSUM_U], w[ROWSUM_U];
#pragma unroll
        for (int u = 0; u < ROWSUM_U; ++u) v[u] = p[(long)(k + 4 * u) * ld];
        for (k += 4 * ROWSUM_U; k + 4 * (ROWSUM_U - 1) < ke; k += 4 * ROWSUM_U) {
#pragma unroll
          for (int u = 0; u < ROWSUM_U; ++u) w[u] = p[(long)(k + 4 * u) * ld];
#pragma unroll
          for (int u = 0; u < ROWSUM_U; ++u) s += (double)v[u];
#pragma unroll
          for (int u = 0; u < ROWSUM_U; ++u) v[u] = w[u];
        }
#pragma unroll
        for (int u = 0; u < ROWSUM_U; ++u) s += (double)v[u];
      }
      for (; k < ke; k += 4) s += (double)p[(long)k * ld];
    }
    red[q][r] = s;
    __syncthreads();
    if (threadIdx.x < 64 && i < d)
      hpart[(long)by * d + i] = (red[0][r] + red[1][r]) + (red[2][r] + red[3][r]);
  } else {
    // one row per wavefront, 4 rows per block
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = bx * 4 + w;
    if (i >= d) return;
    double s = 0.0;
    for (int k = kb + lane; k < ke; k += 64) s += (double)bf16_bits_to_f32(((const u16*)X)[(long)i * K + k]);
    s = wave_sum_f64(s);
    if (lane == 0) hpart[(long)by * d + i] = s;
  }
}

// The window's scatter and, in FP64, on the first nrb nh workgroups of split 0
// its row sums: a chain of loads of its own (26 us at d = 1024), beside the
// products.  The loads in flight take registers, which FP32 products need for
// their occupancy (173 + 21 us apart, 231 together, at d = 1024, K = 12800).
template <typename T, int BT, int ST, bool NARROW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_syrk_t(
    const T* __restrict__ Xs, int d, int K, int kchunk, double* __restrict__ Gpart, int nrb, int nh, int hchunk,
    double* __restrict__ hpart) {
  __shared__ __attribute__((aligned(1024))) T lds[t_lds_elems<T, BT, BT, ST>()];
  const int b = blockIdx.x;
  if constexpr (sizeof(T) == 8)
    if (b < nrb * nh) {
      if (blockIdx.y == 0) rowsum_block<T, true>(Xs, d, d, K, hchunk, b % nrb, b / nrb, hpart, (double (*)[64])lds);
      return;
    }
  syrk_tile_t<T, BT, ST, NARROW>(Xs, d, d, K, kchunk, b - nrb * nh, blockIdx.y, Gpart, lds);
}

// 64-row tiles (FP64 d = 4096, K = 65536: 22.5 to 21.1 ms, 2080 tiles being
// 8.1 per CU; d = 1024, K = 12800: 415 to 320 us, FP32 195 to 168 us), 32-row
// ones where those would not give every CU one (d = 100, K = 3200: 6 tiles).
// Columns without 16-byte strides take the engine's narrow copies (d = 75, K =
// 3200: 66.8 us on the element engine and 12 for the row sums, 24.8 together).
template <typename T, bool NARROW>
static void syrk_t(const void* Xs, int d, long K, int ns, int kchunk, double* Gpart, int nh, int hchunk,
                   double* hpart, hipStream_t s) {
  const int n64 = cdiv(d, 64), n32 = cdiv(d, 32);
  if (sizeof(T) != 8) nh = 0;
  if ((long)n64 * (n64 + 1) / 2 * ns < 256)
    hipLaunchKernelGGL((k_syrk_t<T, 32, 6, NARROW>), dim3(n64 * nh + n32 * (n32 + 1) / 2, ns), dim3(256), 0, s, (const T*)Xs,
                       d, (int)K, kchunk, Gpart, n64, nh, hchunk, hpart);
  else
    hipLaunchKernelGGL((k_syrk_t<T, 64, 3, NARROW>), dim3(n64 * nh + n64 * (n64 + 1) / 2, ns), dim3(256), 0, s, (const T*)Xs,
                       d, (int)K, kchunk, Gpart, n64, nh, hchunk, hpart);
}

template <typename T>
static hipError_t syrk_e(const void* Xs, int d, long K, int ns, int kchunk, double* Gpart, int nh, int hchunk,
                         double* hpart, hipStream_t s) {
  if (t_gemm_ok<T, false, false>(Xs, d, d, Xs, d, d, K)) syrk_t<T, false>(Xs, d, K, ns, kchunk, Gpart, nh, hchunk, hpart, s);
  else if (d < 1 << 20) syrk_t<T, true>(Xs, d, K, ns, kchunk, Gpart, nh, hchunk, hpart, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// bf16: Xt is the transposed window (d x K row-major, ld = K).  Tiles are
// 128 rows (i) x 64 columns (j) covering the lower triangle: in row block bi
// the column blocks bj < 2 (bi + 1).  fp32 accumulation is folded into fp64
// every FOLD_BF16 columns of K.
constexpr int FOLD_BF16 = 2048;

DEV void syrk_tile_128x64(int t, int nbj, int& bi, int& bj) {
  int b = 0, c0 = 0;
  for (;;) {
    const int n = min(2 * b + 2, nbj);
    if (t < c0 + n) break;
    c0 += n;
    ++b;
  }
  bi = b;
  bj = t - c0;
}

__global__ __launch_bounds__(256) void k_syrk_bf16(const u16* __restrict__ Xt, int d, int K, int kchunk, int vec_ok,
                                                   double* __restrict__ Gpart) {
  constexpr int BM = 128, BN = 64;
  __shared__ u16 lds[b_lds_elems<BM, BN>()];
  int bi, bj;
  syrk_tile_128x64(blockIdx.x, (d + 63) / 64, bi, bj);
  const int i0 = bi * BM, j0 = bj * BN;
  const int kb = blockIdx.y * kchunk, ke = min(K, kb + kchunk);
  double acc[BFrag<BM, BN>::FM][BFrag<BM, BN>::FN][4];
#pragma unroll
  for (int m = 0; m < BFrag<BM, BN>::FM; ++m)
#pragma unroll
    for (int n = 0; n < BFrag<BM, BN>::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[m][n][r] = 0.0;
  for (int k0 = kb; k0 < ke; k0 += FOLD_BF16) {
    BFrag<BM, BN> f;
    f.zero();
    b_gemm<BM, BN>(f, Xt, K, d, vec_ok, Xt, K, d, vec_ok, i0, j0, k0, min(ke, k0 + FOLD_BF16), lds);
#pragma unroll
    for (int m = 0; m < BFrag<BM, BN>::FM; ++m)
#pragma unroll
      for (int n = 0; n < BFrag<BM, BN>::FN; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m][n][r] += (double)f.c[m][n][r];
  }
  double* G = Gpart + (long)blockIdx.y * d * d;
#pragma unroll
  for (int m = 0; m < BFrag<BM, BN>::FM; ++m)
#pragma unroll
    for (int n = 0; n < BFrag<BM, BN>::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int ti, tj;
        frag_coords<BM, BN>(m, n, r, ti, tj);
        const int i = i0 + ti, j = j0 + tj;
        if (i < d && j < d) G[j + (long)i * d] = acc[m][n][r];  // G(i,j) at (row j, col i): upper
      }
}

// Direct-to-LDS variant for whole tiles (d a multiple of 256, K chunks of
// 64): 256 (i) x 128 (j) tiles covering the lower triangle (bj < 2 (bi + 1)),
// fp32 accumulation folded into fp64 every FOLD_BF16 columns.
DEV void syrk_tile_256x128(int t, int nbj, int& bi, int& bj) {
  int b = 0, c0 = 0;
  for (;;) {
    const int n = min(2 * b + 2, nbj);
    if (t < c0 + n) break;
    c0 += n;
    ++b;
  }
  bi = b;
  bj = t - c0;
}

__global__ __launch_bounds__(512) void k_syrk_pl(const u16* __restrict__ Xt, int d, int K, int kchunk,
                                                 double* __restrict__ Gpart) {
  constexpr int BM = 256, BN = 128, WGM = 4, WGN = 2, ST = 3;
  typedef WFrag<BM, BN, WGM, WGN> F;
  __shared__ __attribute__((aligned(1024))) u16 lds[p_lds_elems<BM, BN, ST>()];
  int bi, bj;
  syrk_tile_256x128(blockIdx.x, d / 128, bi, bj);
  const int i0 = bi * BM, j0 = bj * BN;
  const int kb = blockIdx.y * kchunk, ke = min(K, kb + kchunk);
  double acc[F::FM][F::FN][4];
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[m][n][r] = 0.0;
  for (int k0 = kb; k0 < ke; k0 += FOLD_BF16) {
    F f;
    f.zero();
    p_gemm<BM, BN, WGM, WGN, ST>(f, Xt, K, Xt, K, i0, j0, k0, min(ke, k0 + FOLD_BF16), lds);
#pragma unroll
    for (int m = 0; m < F::FM; ++m)
#pragma unroll
      for (int n = 0; n < F::FN; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[m][n][r] += (double)f.c[m][n][r];
  }
  double* G = Gpart + (long)blockIdx.y * d * d;
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int ti, tj;
        w_coords<BM, BN, WGM, WGN>(m, n, r, ti, tj);
        G[(j0 + tj) + (long)(i0 + ti) * d] = acc[m][n][r];  // G(i,j) at (row j, col i): upper
      }
}

template <typename T, bool COLMAJOR>
__global__ __launch_bounds__(256) void k_rowsum(const T* __restrict__ X, int d, int K, int kchunk,
                                                double* __restrict__ hpart) {
  __shared__ double red[4][64];
  rowsum_block<T, COLMAJOR>(X, d, d, K, kchunk, blockIdx.x, blockIdx.y, hpart, red);
}

// col-major d x K bf16 -> row-major d x K (ld K)
__global__ __launch_bounds__(256) void k_transpose_bf16(const u16* __restrict__ in, u16* __restrict__ out, int d,
                                                        long K) {
  __shared__ u16 tile[64][66];
  const long k0 = (long)blockIdx.x * 64;
  const int i0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int kk = ty; kk < 64; kk += 4) {
    const long k = k0 + kk;
    const int i = i0 + tx;
    tile[kk][tx] = (k < K && i < d) ? in[i + k * d] : (u16)0;
  }
  __syncthreads();
  for (int ii = ty; ii < 64; ii += 4) {
    const int i = i0 + ii;
    const long k = k0 + tx;
    if (i < d && k < K) out[(long)i * K + k] = tile[tx][ii];
  }
}

// Transposition of the col-major d x K bf16 window into row-major (ld K) with
// the row sums over K taken on the way (whole 64 x 64 tiles: d and K multiples
// of 64).  Workgroup (bx, by) owns rows 64 bx .. 64 bx + 63 and the K range of
// chunk by; its four wavefronts take the chunk's 64-column tiles in turn.  In
// a tile, lane (g, q) = (lane % 8, lane / 8) reads columns 8 q .. 8 q + 7 of
// rows 8 g .. 8 g + 7 as eight 16-byte loads, transposes the 8 x 8 block in
// registers and writes it as eight 16-byte row pieces.  The bf16 values are
// summed in FP64 in a fixed order (exact while a row's values span less than
// 2^29 in magnitude: each has 8 significant bits).
DEV uint32_t pack_lo16(uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); }
DEV uint32_t pack_hi16(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); }

__global__ __launch_bounds__(256) void k_transpose_rowsum_bf16(const u16* __restrict__ in, u16* __restrict__ out,
                                                               int d, long K, long kchunk,
                                                               double* __restrict__ hpart) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int g = lane & 7, q = lane >> 3;
  const int i0 = blockIdx.x * 64 + 8 * g;
  const long kb = (long)blockIdx.y * kchunk, ke = kb + kchunk < K ? kb + kchunk : K;
  double hs[8];
#pragma unroll
  for (int r = 0; r < 8; ++r) hs[r] = 0.0;
  for (long k0 = kb + 64 * w; k0 < ke; k0 += 256) {
    uint32_t v[8][4];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint4 x = *(const uint4*)(in + i0 + (k0 + 8 * q + j) * d);
      v[j][0] = x.x; v[j][1] = x.y; v[j][2] = x.z; v[j][3] = x.w;
    }
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const int c = r >> 1;
      uint32_t o[4];
#pragma unroll
      for (int m = 0; m < 4; ++m)
        o[m] = (r & 1) ? pack_hi16(v[2 * m][c], v[2 * m + 1][c]) : pack_lo16(v[2 * m][c], v[2 * m + 1][c]);
      *(uint4*)(out + (long)(i0 + r) * K + k0 + 8 * q) = make_uint4(o[0], o[1], o[2], o[3]);
#pragma unroll
      for (int j = 0; j < 8; ++j)
        hs[r] += (double)__uint_as_float((r & 1) ? (v[j][c] & 0xffff0000u) : (v[j][c] << 16));
    }
  }
  // lanes of one row group (same g) hold the sums of its eight column groups
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    double s = hs[r];
    s += lane_xor_f64<8>(s);
    s += lane_xor_f64<16>(s);
    s += lane_xor_f64<32>(s);
    if (q == 0) red[w][8 * g + r] = s;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int i = blockIdx.x * 64 + threadIdx.x;
    hpart[(long)blockIdx.y * d + i] = (red[0][threadIdx.x] + red[1][threadIdx.x]) +
                                      (red[2][threadIdx.x] + red[3][threadIdx.x]);
  }
}

// Output tiles of the scatter: 64 x 64 lower pairs (f64/f32) or 128 x 64
// lower-covering tiles (bf16).
// bf16 windows whose tiles are whole take the direct-to-LDS kernel
static bool syrk_pl(int prec, int d, long K) { return prec == PMIX && d % 256 == 0 && K % 64 == 0; }

static int syrk_tiles(int prec, int d, long K) {
  if (prec != PMIX) return cdiv(d, 64) * (cdiv(d, 64) + 1) / 2;
  const int bi_rows = syrk_pl(prec, d, K) ? 256 : 128, bj_cols = bi_rows / 2;
  const int nbi = cdiv(d, bi_rows), nbj = cdiv(d, bj_cols);
  int n = 0;
  for (int b = 0; b < nbi; ++b) n += min(2 * b + 2, nbj);
  return n;
}

// K is split until about 512 workgroups run, but into parts of no less than
// 2048 columns (so a small window's scatter runs on few of them: 20 at d = 100, K
// = 3200); chunks are whole multiples of 64 columns (keeps the bf16 vector loads
// 16-byte aligned).
// FP32 chunks are whole multiples of the FP32 span FOLD_K: a window of at
// most FOLD_K samples is then one chunk, accumulated exactly as the grouped
// scatter of the batched form accumulates it (same FP32 sums, same FP64 fold).
static long syrk_kchunk(int prec, int d, long K) {
  const int nt = syrk_tiles(prec, d, K);
  int ns = cdiv(512, nt);
  const int maxs = (int)((K + 2047) / 2048);
  if (ns > maxs) ns = maxs;
  if (ns < 1) ns = 1;
  long kc = (K + ns - 1) / ns;
  if (prec == P32) return ((kc + FOLD_K - 1) / FOLD_K) * FOLD_K;
  return ((kc + 63) / 64) * 64;
}
static int syrk_splits(int prec, int d, long K) {
  const long kc = syrk_kchunk(prec, d, K);
  const long ns = (K + kc - 1) / kc;
  return ns < 1 ? 1 : (int)ns;
}

size_t syrk_scratch_bytes(int prec, int d, long K) {
  const int ns = syrk_splits(prec, d, K);
  return (size_t)ns * d * d * sizeof(double) + (size_t)64 * d * sizeof(double);
}

hipError_t syrk_window(Prec prec, const void* Xw, void* Xt, int d, long K, void* scratch, Scatter* out,
                       hipStream_t s) {
  const int ns = syrk_splits(prec, d, K);
  const int kchunk = (int)syrk_kchunk(prec, d, K);
  double* Gpart = (double*)scratch;
  double* hpart = Gpart + (size_t)ns * d * d;
  // row sums: at most 64 K-chunks
  int nh = (int)((K + 4095) / 4096) < 64 ? (int)((K + 4095) / 4096) : 64;
  int hchunk = (int)((K + nh - 1) / nh);
  // the bf16 window is scattered from its row-major copy (K contiguous per
  // coordinate); whole tiles take the transposition with the row sums fused
  const void* Xs = Xw;
  bool h_done = false;
  if (prec == PMIX) {
    if (d % 64 == 0 && K % 64 == 0 && (uintptr_t)Xw % 16 == 0 && (uintptr_t)Xt % 16 == 0) {
      const long hc = (K / 64 + nh - 1) / nh * 64;
      nh = (int)((K + hc - 1) / hc);
      hchunk = (int)hc;
      hipLaunchKernelGGL(k_transpose_rowsum_bf16, dim3(d / 64, nh), dim3(256), 0, s, (const u16*)Xw, (u16*)Xt, d, K,
                         hc, hpart);
      h_done = true;
    } else {
      hipLaunchKernelGGL(k_transpose_bf16, dim3((unsigned)((K + 63) / 64), cdiv(d, 64)), dim3(256), 0, s,
                         (const u16*)Xw, (u16*)Xt, d, K);
    }
    Xs = Xt;
  }
  const int nt = syrk_tiles(prec, d, K);
  dim3 grid(nt, ns);
  hipError_t e = hipSuccess;
  if (prec == P64) e = syrk_e<double>(Xs, d, K, ns, kchunk, Gpart, nh, hchunk, hpart, s);
  else if (prec == P32) e = syrk_e<float>(Xs, d, K, ns, kchunk, Gpart, nh, hchunk, hpart, s);
  else if (syrk_pl(prec, d, K) && (uintptr_t)Xs % 16 == 0)
    hipLaunchKernelGGL(k_syrk_pl, grid, dim3(512), 0, s, (const u16*)Xs, d, (int)K, kchunk, Gpart);
  else {
    const int vec_ok = (K % 8 == 0) && ((uintptr_t)Xs % 16 == 0);
    hipLaunchKernelGGL(k_syrk_bf16, grid, dim3(256), 0, s, (const u16*)Xs, d, (int)K, kchunk, vec_ok, Gpart);
  }
  if (e != hipSuccess) return e;
  if (prec == P32)
    hipLaunchKernelGGL((k_rowsum<float, true>), dim3(cdiv(d, 64), nh), dim3(256), 0, s, (const float*)Xs, d, (int)K,
                       hchunk, hpart);
  else if (prec == PMIX && !h_done)
    hipLaunchKernelGGL((k_rowsum<u16, false>), dim3(cdiv(d, 4), nh), dim3(256), 0, s, (const u16*)Xs, d, (int)K,
                       hchunk, hpart);
  *out = {Gpart, hpart, ns, nh};
  return hipGetLastError();
}

// ============================================================================
// moment fold (eqs. mom2g / mom1g with sample counts), covariance assembly
// ============================================================================
DEV void fold_mean_elem(const double* __restrict__ h, const double* __restrict__ sft, double N, double n,
                        double* __restrict__ m, int i) {
  m[i] = (N * m[i] + (h[i] + n * sft[i])) / (N + n);
}

DEV void fold_S_elem(const double* __restrict__ G, const double* __restrict__ h, const double* __restrict__ sft,
                     double N, double n, double* __restrict__ S, int d, long e) {
  const int i = (int)(e % d), j = (int)(e / d);
  const int a = i > j ? i : j, b = i > j ? j : i;
  const double g = G[b + (long)a * d];  // upper storage
  const double sxx = g + sft[a] * h[b] + h[a] * sft[b] + n * sft[a] * sft[b];
  S[e] = (N * S[e] + sxx) / (N + n);
}

// The merge: the scatter's splits added up in order and folded into S and m,
// one workgroup per pair of 64 x 64 tiles of S (tile (bi, bj), bi >= bj, and
// its mirror image).  The scatter's upper-storage tile is read along its
// columns into LDS, so the tile below the diagonal does not read it at a
// stride of d; each element's arithmetic is fold_S_elem's.  One launch and one
// trip through the splits in place of three (d = 1024: 20 + 7 + 4 us, now 13).
constexpr int MERGE_TY = 16;
__global__ __launch_bounds__(64 * MERGE_TY) __attribute__((amdgpu_waves_per_eu(8))) void k_merge(Scatter g, const double* __restrict__ sft, double N, double n,
                                                         double* __restrict__ S, double* __restrict__ m, int d) {
  __shared__ double T[64][65], hs[2][64];
  int bi, bj;
  tile_pair(blockIdx.x, bi, bj);
  const int r0 = 64 * bj, c0 = 64 * bi;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  const long dd = (long)d * d;
  if (ty < 2) {
    const int i = (ty ? c0 : r0) + tx;
    double s = 0.0;
    if (i < d) {
#pragma unroll 8
      for (int q = 0; q < g.nh; ++q) s += g.h[(long)q * d + i];
    }
    hs[ty][tx] = s;
    if (ty == 0 && bi == bj && i < d) m[i] = (N * m[i] + (s + n * sft[i])) / (N + n);
  }
  // The thread's columns side by side and four splits at a time: a load at a
  // time, column after column, was a chain of 64 / MERGE_TY x ns of them (d =
  // 64, 64 splits, one workgroup: 89 us, now 39; d = 256 47 and 24).  64
  // registers, for two workgroups a CU: with one, d = 4096 takes 82 us in place
  // of 69.
  constexpr int MC = 64 / MERGE_TY;
  double v[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c) v[c] = 0.0;
  // bytes from the tile's first element; past the edge the last row or column
  uint32_t o[MC];
#pragma unroll
  for (int c = 0; c < MC; ++c)
    o[c] = (uint32_t)(8 * (min(tx, d - 1 - r0) + (long)min(ty + c * MERGE_TY, d - 1 - c0) * d));
  const char* part = (const char*)(g.G + r0 + (long)c0 * d);
  auto add = [&](auto count) {
    constexpr int NQ = decltype(count)::value;
    double x[NQ][MC];
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int c = 0; c < MC; ++c) x[q][c] = *(const double*)(part + 8 * q * dd + o[c]);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
      for (int c = 0; c < MC; ++c) v[c] += x[q][c];
    part += 8 * NQ * dd;
  };
  int q = 0;
  for (; q + 4 <= g.ns; q += 4) add(std::integral_constant<int, 4>());
  for (; q < g.ns; ++q) add(std::integral_constant<int, 1>());
#pragma unroll
  for (int c = 0; c < MC; ++c) T[tx][ty + c * MERGE_TY] = v[c];
  __syncthreads();
  auto fold = [&](int i, int j, double v, int a, double ha, int b, double hb) {
    const long e = i + (long)j * d;
    const double sxx = v + sft[a] * hb + ha * sft[b] + n * sft[a] * sft[b];
    S[e] = (N * S[e] + sxx) / (N + n);
  };
#pragma unroll
  for (int jj = ty; jj < 64; jj += MERGE_TY) {
    const int i = c0 + tx, j = r0 + jj;
    if (i < d && j < d) {
      if (i >= j) fold(i, j, T[jj][tx], i, hs[1][tx], j, hs[0][jj]);
      else fold(i, j, T[tx][jj], j, hs[0][jj], i, hs[1][tx]);  // diagonal tile, upper part
    }
    if (bi != bj) {
      const int iu = r0 + tx, ju = c0 + jj;
      if (iu < d && ju < d) fold(iu, ju, T[tx][jj], ju, hs[1][jj], iu, hs[0][tx]);
    }
  }
}

hipError_t fold_moments(const Scatter& g, const double* sft, double N, long K, double* S, double* m, int d,
                        hipStream_t s) {
  const int nt = cdiv(d, 64);
  hipLaunchKernelGGL(k_merge, dim3(nt * (nt + 1) / 2), dim3(64 * MERGE_TY), 0, s, g, sft, N, (double)K, S, m, d);
  return hipGetLastError();
}

DEV void cov_elem(const double* __restrict__ S, const double* __restrict__ m, double eps, double* __restrict__ C,
                  int d, long e) {
  const int i = (int)(e % d), j = (int)(e / d);
  double v = 0.0;
  if (i >= j) {
    v = S[e] - m[i] * m[j];
    if (i == j) v += eps;
  }
  C[e] = v;
}

DEV void trace_block(const double* __restrict__ S, const double* __restrict__ m, int d, double* __restrict__ tr) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += 256) s += S[i + (long)i * d] - m[i] * m[i];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) *tr = red[0];
}

// The last workgroup forms the trace and clears the factorisation's words.
__global__ __launch_bounds__(256) void k_cov(const double* __restrict__ S, const double* __restrict__ m, double eps,
                                             double* __restrict__ C, int d, double* __restrict__ tr,
                                             int* __restrict__ info, int* __restrict__ cnt, int P) {
  if (blockIdx.x == gridDim.x - 1) {
    if (tr) trace_block(S, m, d, tr);
    if (info && threadIdx.x == 0) *info = 0;
    if (cnt)
      for (int p = threadIdx.x; p < P; p += 256) cnt[p] = 0;
    return;
  }
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e < (long)d * d) cov_elem(S, m, eps, C, d, e);
}

hipError_t cov_assemble(const double* S, const double* m, double eps, double* C, double* tr, int* info, int* cnt, int P,
                        int d, hipStream_t s) {
  hipLaunchKernelGGL(k_cov, dim3(cdiv((long)d * d, 256) + 1), dim3(256), 0, s, S, m, eps, C, d, tr, info, cnt, P);
  return hipGetLastError();
}

// ============================================================================
// (e) blocked right-looking Cholesky, FP64, block 64.
//   k_chol_diag   four wavefronts factor the first 64 x 64 diagonal block with
//                 its rows in registers and form the block's inverse;
//   k_chol_panel  MFMA: A_ij <- A_ij L_jj^-T as a product with that inverse;
//   k_chol_update_diag MFMA: trailing lower tiles A_ik -= A_ij A_kj^T, for up
//                 to two block columns j in one pass over the tiles, and the
//                 next diagonal block factored by the workgroup that updated it.
// ============================================================================

// lane's value v broadcast from lane `src` (a compile-time lane after unrolling)
DEV double readlane_f64(double v, int src) {
  const unsigned long long u = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, src);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), src);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The diagonal block on a workgroup of four wavefronts.  Lane r of every
// wavefront holds row r; wavefront w holds columns 16 w .. 16 w + 15 of it.
// Column c is published through a double-buffered LDS vector; after one
// workgroup barrier every wavefront that owns columns right of c applies the
// rank-1 update to its part of each row, without per-element masks (entries
// right of the diagonal collect values that are never read).  Blocks of
// CHOL_CB columns with look-ahead: the wavefront owning the next block
// applies the block just published to that block first, factors its CB
// columns in turn (each updating the later ones of the block from its own
// registers and the pivot row's value by readlane) and publishes them before
// its other updates, so one barrier per CB columns separates consecutive
// blocks.  The pivot step forms y ~ 1/sqrt(pivot) by the hardware reciprocal
// square root refined with two Newton-Raphson steps, then L(c, c) = pivot y and
// L(r, c) = a(r, c) y; a pivot that is not > 0 (or NaN) gives a diagonal that
// is not > 0.  Each entry of the lower triangle sees the updates in the same
// order as a right-looking factorisation.  The block inverse is formed as [[A,
// 0], [B, C]]^-1 = [[A^-1, 0], [-C^-1 B A^-1, C^-1]] twice: each wavefront
// inverts one 16 x 16 diagonal block by substitution, then the 16 x 16 and 32 x
// 32 products run on the matrix cores, whose FP64 product is the chain of fused
// multiply-adds over k, bit for bit.
// All of it is latency, in clock cycles: loads 1000 (2400 one at a time), the
// 64 pivot steps 19000 (all of a wavefront's 16 columns by readlane, without
// LDS: 30000), substitution 2800 (4400 with a column per lane), the products
// 2300 (11000 on the vector unit), stores.
// LDS: two buffers of CB columns, the factored block, the four 16 x 16
// inverses, the lower-left blocks of the two 32 x 32 inverses, the 32 x 32
// product.
constexpr int CHOL_DIAG_THREADS = 256;
constexpr int CHOL_CB = 4;  // columns published per workgroup barrier
static_assert((CHOL_NB / 4) % CHOL_CB == 0, "a column block lies within one wavefront's columns");
constexpr int TRI_INV_LDS = 4 * 16 * 17 + 2 * 16 * 17 + 32 * 33;                               // doubles
constexpr int CHOL_DIAG_LDS = 2 * CHOL_CB * CHOL_NB + CHOL_NB * (CHOL_NB + 1) + TRI_INV_LDS;  // doubles

// 1/sqrt(x): hardware estimate, then two Newton-Raphson steps
// y <- y + y (1 - x y^2) / 2 (NaN for x < 0 or NaN, +inf for x = 0)
DEV double rsqrt_nr(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = __fma_rn(-x * y, y, 1.0);
    y = __fma_rn(0.5 * y, e, y);
  }
  return y;
}

// The inverse of a lower-triangular 16 x 16 block by forward substitution on
// one wavefront, Ls its first entry in LDS, rd the reciprocal of the diagonal
// of row o + r in lane o + r.  Each entry is a sum in four parts (column q in
// part q mod 4): lane 4 c + g forms part g of column c, the parts meet by quad
// permutations, so a row is one dependent product, two sums and the scaling.
DEV void tri_inverse16(const double (*Ls)[CHOL_NB + 1], double rd, int o, double (*Di)[17]) {
  const int lane = threadIdx.x & 63, c = lane >> 2, g = lane & 3;
  double l[16][4], x[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int rr = 1; rr < 16; ++rr)
#pragma unroll
    for (int m = 0; 4 * m < rr; ++m) l[rr][m] = Ls[rr][4 * m + g];
#pragma unroll
  for (int rr = 0; rr < 16; ++rr) {
    double s = (g == 0 && rr == c) ? 1.0 : 0.0;
#pragma unroll
    for (int m = 0; 4 * m < rr; ++m) {
      // the parts' last columns differ; an entry past them meets x = 0
      const double v = (4 * m + 3 < rr || 4 * m + g < rr) ? l[rr][m] : 0.0;
      s = __fma_rn(-v, x[m], s);
    }
    s += lane_xor_f64<1>(s);
    s += lane_xor_f64<2>(s);
    s *= readlane_f64(rd, o + rr);
    x[rr >> 2] = (g == (rr & 3)) ? s : x[rr >> 2];
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) Di[4 * m + g][c] = x[m];
}

// The inverse of the lower-triangular block Ls (identity past the matrix
// edge) by four wavefronts from Di, the inverses of its 16 x 16 diagonal
// blocks (rows x columns, zeros above the diagonal) at the start of sh
// (TRI_INV_LDS); Ls and Di are published here.
DEV void tri_inverse_core(const double (*Ls)[CHOL_NB + 1], double* sh, double* __restrict__ Linv) {
  double (*Di)[16][17] = (double (*)[16][17])sh;
  double (*Xh)[16][17] = Di + 4;
  double (*T)[33] = (double (*)[33])(sh + 6 * 16 * 17);
  const int t = threadIdx.x, lane = t & 63, lr = lane & 15, lk = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  __syncthreads();
  // the two 32 x 32 halves, [[D0, 0], [E, D1]]^-1 = [[D0^-1, 0], [-D1^-1 E
  // D0^-1, D1^-1]]: a product's result registers are the next one's operand
  if ((w & 1) == 0) {
    const int hh = w >> 1, o = 32 * hh;
    d4_t e = {0.0, 0.0, 0.0, 0.0}, x = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; ++s) e = mfma_f64(Ls[o + 16 + lr][o + 4 * s + lk], Di[2 * hh][4 * s + lk][lr], e);
#pragma unroll
    for (int s = 0; s < 4; ++s) x = mfma_f64(-Di[2 * hh + 1][lr][4 * s + lk], e[s], x);
#pragma unroll
    for (int r = 0; r < 4; ++r) Xh[hh][4 * r + lk][lr] = x[r];
  }
  __syncthreads();
  // T = B A^-1 (B = rows 32 .. 63, columns 0 .. 31 of L), then -C^-1 T: one 16
  // x 16 block (bi, bj) per wavefront
  const int bi = w >> 1, bj = w & 1;
  {
    d4_t c = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int q = 4 * s + lk, qq = q & 15;
      const double inv = s < 4 ? (bj == 0 ? Di[0][qq][lr] : 0.0) : (bj == 0 ? Xh[0][qq][lr] : Di[1][qq][lr]);
      c = mfma_f64(Ls[32 + 16 * bi + lr][q], inv, c);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) T[16 * bi + 4 * r + lk][16 * bj + lr] = c[r];
  }
  __syncthreads();
  d4_t xl = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int q = 4 * s + lk, qq = q & 15;
    const double inv = s < 4 ? (bi == 0 ? Di[2][lr][qq] : Xh[1][lr][qq]) : (bi == 0 ? 0.0 : Di[3][lr][qq]);
    xl = mfma_f64(-inv, T[q][16 * bj + lr], xl);
  }
  // inverse out, column-major: Linv[q + c 64] = (L^-1)(q, c): the lower-left
  // block from registers, the rest from LDS in column runs
#pragma unroll
  for (int r = 0; r < 4; ++r) Linv[(32 + 16 * bi + 4 * r + lk) + (16 * bj + lr) * CHOL_NB] = xl[r];
#pragma unroll
  for (int k = 0; k < CHOL_NB * CHOL_NB / CHOL_DIAG_THREADS; ++k) {
    const int e = t + k * CHOL_DIAG_THREADS;
    const int q = e & (CHOL_NB - 1), c = e >> 6, bq = q >> 4, bc = c >> 4;
    if (bq >= 2 && bc < 2) continue;
    Linv[e] = bq < bc ? 0.0 : (bq == bc ? Di[bq] : Xh[bq >> 1])[q & 15][c & 15];
  }
}

// Row r of columns 16 w .. 16 w + 15 of a lower-triangular 64 x 64 block of
// which jn rows and columns exist: zeros right of the diagonal, identity past
// the edge.  Clamped addresses, so that all 16 loads are in flight.
DEV void load_block_columns(const double* __restrict__ A, int d, int jn, int w, int r, double* a) {
  constexpr int H = CHOL_NB / 4;
  const int i = min(r, jn - 1);
#pragma unroll
  for (int k = 0; k < H; ++k) a[k] = A[i + (long)min(w * H + k, jn - 1) * d];
#pragma unroll
  for (int k = 0; k < H; ++k) {
    const int c = w * H + k;
    a[k] = (c <= r && r < jn) ? a[k] : (c == r) ? 1.0 : 0.0;
  }
}

DEV void chol_diag_core(double* __restrict__ A, int d, int j0, int jn, double* __restrict__ Linv,
                        int* __restrict__ info, double* sh) {
  constexpr int H = CHOL_NB / 4;  // columns per wavefront
  double (*colp)[CHOL_CB][CHOL_NB] = (double (*)[CHOL_CB][CHOL_NB])sh;  // [parity][column of block][row]
  double (*Ls)[CHOL_NB + 1] = (double (*)[CHOL_NB + 1])(sh + 2 * CHOL_CB * CHOL_NB);
  double* inv = sh + 2 * CHOL_CB * CHOL_NB + CHOL_NB * (CHOL_NB + 1);
  const int t = threadIdx.x, r = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  double a[H];
  load_block_columns(A + j0 + (long)j0 * d, d, jn, w, r, a);
  // pivot step of column c by the wavefront holding it (its local column kc)
  auto pivot = [&](int c, int kc, double* dst) {
    const double piv = readlane_f64(a[kc], c);
    const double y = rsqrt_nr(piv);
    const double l = (r == c) ? piv * y : a[kc] * y;
    a[kc] = l;
    dst[r] = (r >= c) ? l : 0.0;
  };
  // the owner of block (n .. n + CB - 1) factors its columns in turn, each
  // updating the later ones of the block from its own registers and the
  // pivot row's value (readlane), and publishes them
  auto own_block = [&](int n, int buf) {
    const int k0 = n % H;
#pragma unroll
    for (int t = 0; t < CHOL_CB; ++t) {
      pivot(n + t, k0 + t, colp[buf][t]);
      const double lt = (r >= n + t) ? a[k0 + t] : 0.0;
#pragma unroll
      for (int u = t + 1; u < CHOL_CB; ++u) a[k0 + u] = __fma_rn(-lt, readlane_f64(a[k0 + t], n + u), a[k0 + u]);
    }
  };
  if (w == 0) own_block(0, 0);
#pragma unroll
  for (int q = 0; q < CHOL_NB / CHOL_CB; ++q) {
    const int c0 = CHOL_CB * q, wc = c0 / H, n0 = c0 + CHOL_CB, wn = n0 / H;
    const int buf = q & 1;
    if (c0 >= jn) break;  // uniform: identity from here on, its own factor
    __syncthreads();
    if (n0 < CHOL_NB && w == wn) {
      // owner of the next block: the published block applied to its columns,
      // that block factored and published, then the rest of its columns
      double lb[CHOL_CB];
#pragma unroll
      for (int t = 0; t < CHOL_CB; ++t) lb[t] = colp[buf][t][r];
      const int k0 = n0 % H;
#pragma unroll
      for (int u = 0; u < CHOL_CB; ++u)
#pragma unroll
        for (int t = 0; t < CHOL_CB; ++t) a[k0 + u] = __fma_rn(-lb[t], colp[buf][t][n0 + u], a[k0 + u]);
      own_block(n0, buf ^ 1);
#pragma unroll
      for (int k = (wn == wc) ? k0 + CHOL_CB : CHOL_CB; k < H; ++k)
#pragma unroll
        for (int t = 0; t < CHOL_CB; ++t) a[k] = __fma_rn(-lb[t], colp[buf][t][w * H + k], a[k]);
    } else if (w > wc) {
      double lb[CHOL_CB];
#pragma unroll
      for (int t = 0; t < CHOL_CB; ++t) lb[t] = colp[buf][t][r];
#pragma unroll
      for (int k = 0; k < H; ++k)
#pragma unroll
        for (int t = 0; t < CHOL_CB; ++t) a[k] = __fma_rn(-lb[t], colp[buf][t][w * H + k], a[k]);
    }
  }
  double diag = 1.0;
#pragma unroll
  for (int k = 0; k < H; ++k) {
    const int c = w * H + k;
    Ls[r][c] = (c <= r) ? a[k] : 0.0;
    diag = (r == c) ? a[k] : diag;
  }
  // the inverses of the four 16 x 16 diagonal blocks, one per wavefront
  tri_inverse16((const double (*)[CHOL_NB + 1]) & Ls[w * H][w * H], 1.0 / diag, w * H, ((double (*)[16][17])inv)[w]);
  tri_inverse_core(Ls, inv, Linv);
  // the factor last: a barrier waits for the stores before it
#pragma unroll
  for (int k = 0; k < H; ++k) {
    const int c = w * H + k;
    if (r < jn && c < jn) A[(j0 + r) + (long)(j0 + c) * d] = (c <= r) ? a[k] : 0.0;
  }
  if (w == 0) {
    // a pivot that is not > 0 (or NaN) leaves a diagonal root that is not > 0,
    // and every later pivot inherits the failure: the first bad column is the
    // lowest such lane
    const unsigned long long bad = __ballot(r < jn && !(Ls[r][r] > 0.0));
    if (r == 0 && bad && *info == 0) *info = j0 + __ffsll((long long)bad);
  }
}

DEV void chol_diag_block(double* __restrict__ A, int d, int j0, int jn, double* __restrict__ Linv,
                         int* __restrict__ info) {
  __shared__ double sh[CHOL_DIAG_LDS];
  chol_diag_core(A, d, j0, jn, Linv, info, sh);
}

__global__ __launch_bounds__(CHOL_DIAG_THREADS) void k_chol_diag(double* __restrict__ A, int d, int j0, int jn,
                                                                 double* __restrict__ Linv, int* __restrict__ info) {
  chol_diag_block(A, d, j0, jn, Linv, info);
}

// Inverses of all (already factored) diagonal blocks of L, one workgroup per
// block: the block is read once and inverted as in the factorisation (7 us,
// a serial chain in code that is cold once a window; 20 to 34 us when each
// lane of one wavefront substituted for a whole column).  Only for a factor
// rounded since; the factorisation leaves the unrounded blocks' inverses.
DEV void tri_inv_block(const double* __restrict__ L, int d, double* __restrict__ Linv, int bx) {
  __shared__ double sh[CHOL_NB * (CHOL_NB + 1) + TRI_INV_LDS];
  double (*Ls)[CHOL_NB + 1] = (double (*)[CHOL_NB + 1])sh;
  double* inv = sh + CHOL_NB * (CHOL_NB + 1);
  constexpr int H = CHOL_NB / 4;
  const int r = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int j0 = bx * CHOL_NB, jn = min(CHOL_NB, d - j0);
  double a[H], diag = 1.0;
  load_block_columns(L + j0 + (long)j0 * d, d, jn, w, r, a);
#pragma unroll
  for (int k = 0; k < H; ++k) {
    Ls[r][w * H + k] = a[k];
    diag = (r == w * H + k) ? a[k] : diag;
  }
  tri_inverse16((const double (*)[CHOL_NB + 1]) & Ls[w * H][w * H], 1.0 / diag, w * H, ((double (*)[16][17])inv)[w]);
  tri_inverse_core(Ls, inv, Linv + (long)bx * CHOL_NB * CHOL_NB);
}

__global__ __launch_bounds__(256) void k_tri_inv(const double* __restrict__ L, int d, double* __restrict__ Linv) {
  tri_inv_block(L, d, Linv, blockIdx.x);
}

// Panel rows below the diagonal block: A(i, j0 + c) <- sum_q A(i, j0 + q)
// Linv(c, q), 32 rows per workgroup (few rows, so latency counts) on the
// direct-to-LDS engine (narrow copies for odd d) with all of K in flight, transposed so that lanes run
// along the columns of memory: 7.3 us on the element engine, now 4.8.
constexpr int CHOL_ST = 5;  // four slices of 16 in flight: a block column
constexpr int CHOL_PANEL_LDS = t_lds_elems<double, CHOL_NB, CHOL_PANEL_ROWS, CHOL_ST>();

DEV bool chol_aligned(const double* A, int d) { return d % 2 == 0 && (uintptr_t)A % 16 == 0; }

DEV void chol_panel_tile(double* __restrict__ A, int d, int j0, int jn, const double* __restrict__ Linv, int bx) {
  __shared__ __attribute__((aligned(1024))) double lds[CHOL_PANEL_LDS];
  const int i0 = j0 + jn + bx * CHOL_PANEL_ROWS;
  if (i0 >= d) return;  // uniform: the second half of a block of at most 32 rows
  double* Pc = A + (long)j0 * d;
  constexpr int BN = CHOL_PANEL_ROWS;
  typedef TFrag<double, CHOL_NB, BN, 2, 2> F;
  F f;
  f.zero();
  if (chol_aligned(A, d))
    t_gemm<double, CHOL_NB, BN, 2, 2, CHOL_ST, false, false>(f, Linv, CHOL_NB, CHOL_NB, Pc, d, d, 0, i0, 0, CHOL_NB,
                                                             lds);
  else
    t_gemm<double, CHOL_NB, BN, 2, 2, CHOL_ST, false, false, false, 1, 1, false, true>(
        *(F(*)[1]) & f, Linv, CHOL_NB, CHOL_NB, Pc, d, d, 0, i0, 0, CHOL_NB, lds);
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int c, ti;
        t_coords<double, CHOL_NB, BN, 2, 2>(m, n, r, c, ti);
        if (i0 + ti < d) Pc[i0 + ti + (long)c * d] = f.c[m][n][r];
      }
}

__global__ __launch_bounds__(256) void k_chol_panel(double* __restrict__ A, int d, int j0, int jn,
                                                    const double* __restrict__ Linv) {
  chol_panel_tile(A, d, j0, jn, Linv, blockIdx.x);
}

// Updates of the trailing lower tiles, A(i, k) -= sum_c A(i, c) A(k, c), two
// block columns at a time: after an even block column jb only block column jb
// + 1, which is factored next, and the diagonal tile after it are updated;
// after an odd one the whole trailing part takes both columns' products, one
// after the other, in one trip through memory.  Every entry sees the same
// operations in the same order as with an update per block column, whose
// trips bound the factorisation of many or large matrices: per block column of
// 64 of 1024 x 1024 95 us, now 60, of one of 4096 x 4096 33 and 24 (22 and 20
// at 1024 x 1024, where the diagonal core bounds it).
int chol_update_tiles(int nb, int jb) {
  const int m = nb - jb - 1;
  return jb % 2 == 0 ? m + (m >= 2) : m * (m + 1) / 2;
}
constexpr int CHOL_UPD_LDS = t_lds_elems<double, 64, 64, CHOL_ST>();  // doubles

// block columns [c0, c0 + 64 NC) on tile (i0, k0)
template <int NC>
DEV void chol_update_part(double* __restrict__ A, int d, int c0, int i0, int k0, double* lds) {
  const double* Pc = A + (long)c0 * d;
  typedef TFrag<double, 64, 64, 2, 2> F;
  // the tile itself, on its way during the products
  double c[F::FM][F::FN][4];
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int tk, ti;
        t_coords<double, 64, 64, 2, 2>(m, n, r, tk, ti);
        c[m][n][r] = A[min(i0 + ti, d - 1) + (long)min(k0 + tk, d - 1) * d];
      }
  F f[NC];
#pragma unroll
  for (int x = 0; x < NC; ++x) f[x].zero();
  if (chol_aligned(A, d))
    t_gemm<double, 64, 64, 2, 2, CHOL_ST, false, false, false, NC, 1, true>(f, Pc, d, d, Pc, d, d, k0, i0, 0,
                                                                            CHOL_NB * NC, lds);
  else
    t_gemm<double, 64, 64, 2, 2, CHOL_ST, false, false, false, NC, 1, true, true>(f, Pc, d, d, Pc, d, d, k0, i0, 0,
                                                                                  CHOL_NB * NC, lds);
#pragma unroll
  for (int m = 0; m < F::FM; ++m)
#pragma unroll
    for (int n = 0; n < F::FN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int tk, ti;
        t_coords<double, 64, 64, 2, 2>(m, n, r, tk, ti);
        double v = c[m][n][r];
#pragma unroll
        for (int x = 0; x < NC; ++x) v -= f[x].c[m][n][r];
        if (i0 + ti < d && k0 + tk < d) A[i0 + ti + (long)(k0 + tk) * d] = v;
      }
}

// tile t of the update after block column jb
DEV void chol_update_core(double* __restrict__ A, int d, int jb, int t, double* lds) {
  const int nb = (d + CHOL_NB - 1) / CHOL_NB, t0 = jb + 1;
  if (jb % 2 == 0) {
    const int bi = t < nb - t0 ? t : 1, bk = t < nb - t0 ? 0 : 1;
    chol_update_part<1>(A, d, jb * CHOL_NB, (t0 + bi) * CHOL_NB, (t0 + bk) * CHOL_NB, lds);
  } else if (t == 0) {  // the next diagonal block: the first column's part is done
    chol_update_part<1>(A, d, jb * CHOL_NB, t0 * CHOL_NB, t0 * CHOL_NB, lds);
  } else {
    int bi, bk;
    tile_pair(t, bi, bk);
    chol_update_part<2>(A, d, (jb - 1) * CHOL_NB, (t0 + bi) * CHOL_NB, (t0 + bk) * CHOL_NB, lds);
  }
}

size_t chol_scratch_bytes(int d) { return (size_t)cdiv(d, CHOL_NB) * CHOL_NB * CHOL_NB * sizeof(double); }

// The update after block column jb fused with the factorisation of the next
// diagonal block: workgroup 0 updates that block, the first tile, and then
// factors it while the other workgroups finish the update.  The barrier at the start of
// the factorisation orders the tile's stores before its loads (one
// workgroup); nothing else reads the block before the next launch.
// Both phases use the same LDS buffer.
__global__ __launch_bounds__(256) void k_chol_update_diag(double* __restrict__ A, int d, int jb,
                                                          double* __restrict__ Linv_next, int* __restrict__ info) {
  constexpr int NLDS = CHOL_UPD_LDS > CHOL_DIAG_LDS ? CHOL_UPD_LDS : CHOL_DIAG_LDS;
  __shared__ __attribute__((aligned(1024))) double lds[NLDS];
  chol_update_core(A, d, jb, blockIdx.x, lds);
  if (blockIdx.x == 0) {
    __syncthreads();
    const int j1 = (jb + 1) * CHOL_NB;
    chol_diag_core(A, d, j1, min(CHOL_NB, d - j1), Linv_next, info, lds);
  }
}

hipError_t potrf(double* A, int d, int* info, double* Linv, hipStream_t s) {
  const int nb = cdiv(d, CHOL_NB);
  hipLaunchKernelGGL(k_chol_diag, dim3(1), dim3(CHOL_DIAG_THREADS), 0, s, A, d, 0, min(CHOL_NB, d), Linv, info);
  for (int jb = 0; jb + 1 < nb; ++jb) {
    const int j0 = jb * CHOL_NB, jn = CHOL_NB;
    const double* Li = Linv + (long)jb * CHOL_NB * CHOL_NB;
    const int m = nb - jb - 1;
    hipLaunchKernelGGL(k_chol_panel, dim3(m * (CHOL_NB / CHOL_PANEL_ROWS)), dim3(256), 0, s, A, d, j0, jn, Li);
    hipLaunchKernelGGL(k_chol_update_diag, dim3(chol_update_tiles(nb, jb)), dim3(256), 0, s, A, d, jb,
                       Linv + (long)(jb + 1) * CHOL_NB * CHOL_NB, info);
  }
  return hipGetLastError();
}

DEV void round_factor_elem(int prec, double* __restrict__ L, void* __restrict__ Llow, int d, long e) {
  const int i = (int)(e % d), j = (int)(e / d);
  const double v = (i >= j) ? L[e] : 0.0;
  if (prec == P32) {
    const float f = (float)v;
    L[e] = (double)f;
    ((float*)Llow)[e] = f;
  } else {
    // L~ = hi + lo, both bf16, row-major copies (k-contiguous for the MFMA)
    const u16 hi = f32_to_bf16_bits((float)v);
    const double rem = v - (double)bf16_bits_to_f32(hi);
    const u16 lo = f32_to_bf16_bits((float)rem);
    L[e] = (double)bf16_bits_to_f32(hi) + (double)bf16_bits_to_f32(lo);
    ((u16*)Llow)[(long)i * d + j] = hi;
    ((u16*)Llow)[(long)d * d + (long)i * d + j] = lo;
  }
}

__global__ __launch_bounds__(256) void k_round_factor(int prec, double* __restrict__ L, void* __restrict__ Llow, int d) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e < (long)d * d) round_factor_elem(prec, L, Llow, d, e);
}

// The mixed form's rounding by 64 x 64 tiles: the column-major factor is
// read and written back along its columns, and the row-major hi and lo
// copies leave through an LDS transpose along their rows (each element's
// arithmetic is round_factor_elem's).
__global__ __launch_bounds__(256) void k_round_factor_hl(double* __restrict__ L, u16* __restrict__ Llow, int d) {
  __shared__ u16 th[64][66], tl[64][66];  // [column][row] of the tile
  const int i0 = blockIdx.x * 64, j0 = blockIdx.y * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int jj = ty; jj < 64; jj += 4) {
    const int i = i0 + tx, j = j0 + jj;
    u16 hi = 0, lo = 0;
    if (i < d && j < d) {
      const long e = i + (long)j * d;
      const double v = (i >= j) ? L[e] : 0.0;
      hi = f32_to_bf16_bits((float)v);
      const double rem = v - (double)bf16_bits_to_f32(hi);
      lo = f32_to_bf16_bits((float)rem);
      L[e] = (double)bf16_bits_to_f32(hi) + (double)bf16_bits_to_f32(lo);
    }
    th[jj][tx] = hi;
    tl[jj][tx] = lo;
  }
  __syncthreads();
  for (int ii = ty; ii < 64; ii += 4) {
    const int i = i0 + ii, j = j0 + tx;
    if (i < d && j < d) {
      Llow[(long)i * d + j] = th[tx][ii];
      Llow[(long)d * d + (long)i * d + j] = tl[tx][ii];
    }
  }
}

hipError_t round_factor(Prec prec, double* L, void* Llow, int d, hipStream_t s) {
  if (prec == P64) return hipSuccess;
  if (prec == PMIX)
    hipLaunchKernelGGL(k_round_factor_hl, dim3(cdiv(d, 64), cdiv(d, 64)), dim3(256), 0, s, L, (u16*)Llow, d);
  else
    hipLaunchKernelGGL(k_round_factor, dim3(cdiv((long)d * d, 256)), dim3(256), 0, s, (int)prec, L, Llow, d);
  return hipGetLastError();
}

// ============================================================================
// Potential scale reduction factor (Section 2.4.2, eqs. winco, btwco, psrf,
// M = 1).  Per chain p and coordinate i the running mean and the sum of
// squared deviations of the visited states, merged window by window from the
// window store (state = pivot of the window + stored shift, in the store's
// precision) with the pairwise update of Chan, Golub and LeVeque (1979), so
// no raw second moment is ever formed.
// ============================================================================
// V consecutive stored values from element e (e a multiple of V; V = 1, 2 or 4)
template <int PR, int V>
DEV void load_win_v(const void* win, long e, double* v) {
  if (V == 1) {
    if (PR == P64) v[0] = ((const double*)win)[e];
    else if (PR == P32) v[0] = (double)((const float*)win)[e];
    else v[0] = (double)bf16_bits_to_f32(((const u16*)win)[e]);
  } else if (V == 2) {
    if (PR == P64) {
      const double2 a = *(const double2*)((const double*)win + e);
      v[0] = a.x; v[1] = a.y;
    } else if (PR == P32) {
      const float2 a = *(const float2*)((const float*)win + e);
      v[0] = a.x; v[1] = a.y;
    } else {
      const uint32_t a = *(const uint32_t*)((const u16*)win + e);
      v[0] = (double)bf16_bits_to_f32((u16)(a & 0xffff));
      v[1] = (double)bf16_bits_to_f32((u16)(a >> 16));
    }
  } else if (PR == P64) {
    const double2 a = *(const double2*)((const double*)win + e), b = *(const double2*)((const double*)win + e + 2);
    v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
  } else if (PR == P32) {
    const float4 a = *(const float4*)((const float*)win + e);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  } else {
    const uint2 a = *(const uint2*)((const u16*)win + e);
    v[0] = (double)bf16_bits_to_f32((u16)(a.x & 0xffff));
    v[1] = (double)bf16_bits_to_f32((u16)(a.x >> 16));
    v[2] = (double)bf16_bits_to_f32((u16)(a.y & 0xffff));
    v[3] = (double)bf16_bits_to_f32((u16)(a.y >> 16));
  }
}

// elements e = i + d p, V consecutive coordinates of one chain per thread
// (V = 4 needs d % 4 == 0); window column of chain p at step t: p + P t
template <int PR, int V>
__global__ __launch_bounds__(256) void k_psrf_acc(const void* __restrict__ win, int d, int P, int nw,
                                                  const double* __restrict__ xr, double n0, double* __restrict__ mean,
                                                  double* __restrict__ m2) {
  const long e0 = ((long)blockIdx.x * 256 + threadIdx.x) * V;
  if (e0 >= (long)d * P) return;
  const int i0 = (int)(e0 % d), p = (int)(e0 / d);
  double s1[V], s2[V];
#pragma unroll
  for (int k = 0; k < V; ++k) s1[k] = s2[k] = 0.0;
  // loads of 16 steps in flight per thread for 4-wide rows (measured best at
  // d = 4096, P = 256: 71 % of the HBM peak), 4 for single coordinates
  constexpr int UNR = V == 4 ? 16 : 4;
#pragma unroll UNR
  for (int t = 0; t < nw; ++t) {
    double v[V];
    load_win_v<PR, V>(win, i0 + (long)(p + (long)P * t) * d, v);
#pragma unroll
    for (int k = 0; k < V; ++k) {
      s1[k] += v[k];
      s2[k] = __fma_rn(v[k], v[k], s2[k]);
    }
  }
#pragma unroll
  for (int k = 0; k < V; ++k) {
    const long e = e0 + k;
    const double mw = s1[k] / nw;
    const double qw = __fma_rn(-s1[k], mw, s2[k]);  // sum over the window of (v - mw)^2
    const double xm = xr[i0 + k] + mw;              // the window's mean state
    if (n0 == 0.0) {
      mean[e] = xm;
      m2[e] = qw;
    } else {
      const double nt = n0 + (double)nw;
      const double delta = xm - mean[e];
      mean[e] = __fma_rn(delta, (double)nw / nt, mean[e]);
      m2[e] = m2[e] + qw + delta * delta * (n0 * (double)nw / nt);
    }
  }
}

template <int PR>
static void psrf_acc_launch(const void* win, int d, int P, int nw, const double* xr, double n0, double* mean,
                            double* m2, hipStream_t s) {
  const long n = (long)d * P;
  if (d % 4 == 0 && (uintptr_t)win % 16 == 0)
    hipLaunchKernelGGL((k_psrf_acc<PR, 4>), dim3(cdiv(n / 4, 256)), dim3(256), 0, s, win, d, P, nw, xr, n0, mean, m2);
  else
    hipLaunchKernelGGL((k_psrf_acc<PR, 1>), dim3(cdiv(n, 256)), dim3(256), 0, s, win, d, P, nw, xr, n0, mean, m2);
}

hipError_t psrf_accumulate(Prec prec, const void* win, int d, int P, int nw, const double* xr, double n0, double* mean,
                           double* m2, hipStream_t s) {
  if (prec == P64) psrf_acc_launch<P64>(win, d, P, nw, xr, n0, mean, m2, s);
  else if (prec == P32) psrf_acc_launch<P32>(win, d, P, nw, xr, n0, mean, m2, s);
  else psrf_acc_launch<PMIX>(win, d, P, nw, xr, n0, mean, m2, s);
  return hipGetLastError();
}

// out[i] = sqrt(R_i): B_i = n/(P-1) sum_p (m^p - mbar)_i^2 with mbar the mean
// of the chain means, W_i = sum_p m2[i, p] / ((n - 1) P) (the average of the
// chains' 1/n variances times n/(n-1)), R_i = (n-1)/n + (P+1)/(P n) B_i/W_i.
__global__ __launch_bounds__(256) void k_psrf_final(const double* __restrict__ mean, const double* __restrict__ m2,
                                                    int d, int P, double n, double* __restrict__ out) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= d) return;
  double sm = 0.0, sq = 0.0;
  for (int p = 0; p < P; ++p) {
    sm += mean[i + (long)p * d];
    sq += m2[i + (long)p * d];
  }
  const double mbar = sm / P;
  double sb = 0.0;
  for (int p = 0; p < P; ++p) {
    const double u = mean[i + (long)p * d] - mbar;
    sb = __fma_rn(u, u, sb);
  }
  const double B = n / (double)(P - 1) * sb;
  const double W = sq / ((n - 1.0) * (double)P);
  const double R = (n - 1.0) / n + (double)(P + 1) / ((double)P * n) * (B / W);
  out[i] = sqrt(R);
}

hipError_t psrf_finalize(const double* mean, const double* m2, int d, int P, double n, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_psrf_final, dim3(cdiv(d, 256)), dim3(256), 0, s, mean, m2, d, P, n, out);
  return hipGetLastError();
}

// ---- whitening Z = L^-1 (X - xr) ------------------------------------------
// Rows r0 .. r0 + rows - 1 of Z for 16 columns on one workgroup, with those
// rows of all 16 columns in LDS: per 64-row block j, four wavefronts form z_j =
// Linv_j r_j, then all eight subtract L_ij z_j from the rows below, a 16-row
// tile of L at a time straight from memory (column-major: a quarter wavefront
// reads 128 contiguous bytes) with the next tile's loads in flight.  The solve
// is a chain of rows / 64 dependent blocks; a launch per block made a link of
// it 14 us, in LDS it is 5 to 8 us, the latency of the L tiles (rows^2 / 2 per
// workgroup, mostly from L2): 39 us at 512 rows and 122 at 1024, where the
// launches took 150 and 260; 20000 columns of 512 rows 5.5 ms to 0.16.  X
// null: the rows already hold the right-hand side in Z.  zq (whole columns
// only): column norms.
constexpr int WHITEN_MAX = 1024;  // rows whose 16 columns fit the LDS: 128 KB

// Above that, equal pieces of at most 512 rows with one product per piece for
// the rows below it.
__host__ __device__ int whiten_rows(int d) {
  const int nb = (d + CHOL_NB - 1) / CHOL_NB;
  if (nb * CHOL_NB <= WHITEN_MAX) return nb * CHOL_NB;
  const int pieces = (nb + 7) / 8;
  return (nb + pieces - 1) / pieces * CHOL_NB;
}

DEV void whiten_tile(const double* __restrict__ L, const double* __restrict__ Linv, const double* __restrict__ X,
                     const double* __restrict__ xr, double* __restrict__ Z, double* __restrict__ zq, int d, int P,
                     int r0, int rows, int bx) {
  __shared__ double sh[(WHITEN_MAX + CHOL_NB) * 16];
  // row i, column c at zs[16 i + (c + i) % 16]: a row is one 128-byte line for
  // the products, 64 rows of a column cover the banks for the copies
  double* zs = sh;
  double (*zj)[16] = (double (*)[16])(sh + WHITEN_MAX * 16);
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
  const int q = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int c0 = bx * 16, m = min(rows, d - r0);  // rows that exist
  const int nb = (m + CHOL_NB - 1) / CHOL_NB;
  for (int e = tid; e < nb * CHOL_NB * 16; e += 512) {
    const int i = (e & 63) | ((e >> 10) << 6), c = (e >> 6) & 15;
    double v = 0.0;
    if (i < m && c0 + c < P) {
      const long g = r0 + i + (long)(c0 + c) * d;
      v = X ? X[g] - xr[r0 + i] : Z[g];
    }
    zs[16 * i + ((c + i) & 15)] = v;
  }
  const double* Lb = L + (long)r0 * d + r0;  // the diagonal piece
  const int ntile = (m + 15) / 16;
  const int off = lk * d + lr;
  // 16 rows from 16 t, the 64 columns of block j
  auto load = [&](double* a, int j, int t) {
    const double* b = Lb + (long)(CHOL_NB * j) * d + 16 * t;
    if (16 * t + 16 <= m) {
#pragma unroll
      for (int s = 0; s < 16; ++s) a[s] = (b + (long)(4 * s) * d)[off];
    } else {
      const bool in = 16 * t + lr < m;
      const int o = in ? off : lk * d;
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const double v = (b + (long)(4 * s) * d)[o];
        a[s] = in ? v : 0.0;
      }
    }
  };
  double ad[16], a0[16], a1[16], b[16];
  auto load_diag = [&](int j) {
    const double* p = Linv + (long)(r0 / CHOL_NB + j) * CHOL_NB * CHOL_NB + 16 * q;
#pragma unroll
    for (int s = 0; s < 16; ++s) ad[s] = p[(4 * s + lk) * CHOL_NB + lr];
  };
  auto first = [&](int j) { return 4 * (j + 1) + q; };  // this wavefront's first tile below block j
  auto update = [&](const double* a, int t) {
    d4_t acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 16; ++s) acc = mfma_f64(a[s], b[s], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double* p = &zs[16 * (16 * t + 4 * r + lk) + ((lr + 4 * r + lk) & 15)];
      *p -= acc[r];
    }
  };
  if (q < 4) load_diag(0);
  if (first(0) < ntile) load(a0, 0, first(0));
  __syncthreads();
  for (int j = 0; j < nb; ++j) {
    d4_t z = {0.0, 0.0, 0.0, 0.0};
    if (q < 4) {
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const int k = 4 * s + lk;
        z = mfma_f64(ad[s], zs[16 * (CHOL_NB * j + k) + ((lr + k) & 15)], z);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) zj[16 * q + 4 * r + lk][lr] = z[r];
      if (j + 1 < nb) load_diag(j + 1);
    }
    __syncthreads();  // z_j formed from all of r_j
    if (q < 4) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = CHOL_NB * j + 16 * q + 4 * r + lk;
        zs[16 * i + ((lr + i) & 15)] = z[r];
      }
    }
    if (first(j) < ntile) {
#pragma unroll
      for (int s = 0; s < 16; ++s) b[s] = zj[4 * s + lk][lr];
      for (int t = first(j); t < ntile; t += 16) {
        if (t + 8 < ntile) load(a1, j, t + 8);
        update(a0, t);
        if (t + 16 < ntile) load(a0, j, t + 16);
        else if (first(j + 1) < ntile) load(a0, j + 1, first(j + 1));
        if (t + 8 < ntile) update(a1, t + 8);
      }
    }
    __syncthreads();  // r_(j+1); z_j's copy read
  }
  if (Z)
    for (int e = tid; e < nb * CHOL_NB * 16; e += 512) {
      const int i = (e & 63) | ((e >> 10) << 6), c = (e >> 6) & 15;
      if (i < m && c0 + c < P) Z[r0 + i + (long)(c0 + c) * d] = zs[16 * i + ((c + i) & 15)];
    }
  if (zq)
    for (int c = q; c < 16 && c0 + c < P; c += 8) {
      // rows 256 apart per partial sum, then their tree: the order of colnorm_block
      double p[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        p[u] = 0.0;
        for (int i = lane + 64 * u; i < m; i += 256) {
          const double v = zs[16 * i + ((c + i) & 15)];
          p[u] = __fma_rn(v, v, p[u]);
        }
      }
      const double n2 = wave_sum_f64((p[0] + p[2]) + (p[1] + p[3]));
      if (lane == 0) zq[c0 + c] = n2;
    }
}

__global__ __launch_bounds__(512) void k_whiten(const double* __restrict__ L, const double* __restrict__ Linv,
                                                const double* __restrict__ X, const double* __restrict__ xr,
                                                double* __restrict__ Z, double* __restrict__ zq, int d, int P, int r0,
                                                int rows, double* __restrict__ xr_copy) {
  if (xr_copy && blockIdx.x == 0)
    for (int i = threadIdx.x; i < d; i += 512) xr_copy[i] = xr[i];
  whiten_tile(L, Linv, X, xr, Z, zq, d, P, r0, rows, blockIdx.x);
}

// Rows below a piece: Z_i <- (X_i - xr_i, or Z_i where X is null) - L_i,piece Z_piece
DEV void whiten_update_tile(const double* __restrict__ L, const double* __restrict__ X, const double* __restrict__ xr,
                            double* __restrict__ Z, int d, int P, int j0, int jn, int bx, int by) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ double lds[e_lds_elems<double, BM, BN, BK>()];
  const int i0 = j0 + jn + bx * BM, p0 = by * BN;
  EFrag<double, BM, BN> f;
  f.zero();
  e_gemm<double, BM, BN, BK, false, true>(f, L + (long)j0 * d, d, d, Z + j0, d, P, i0, p0, 0, jn, lds);
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        int ti, tj;
        frag_coords<BM, BN, double>(m, n, r, ti, tj);
        const int i = i0 + ti, p = p0 + tj;
        if (i >= d || p >= P) continue;
        const long e = i + (long)p * d;
        Z[e] = (X ? X[e] - xr[i] : Z[e]) - f.c[m][n][r];
      }
}

__global__ __launch_bounds__(256) void k_whiten_update(const double* __restrict__ L, const double* __restrict__ X,
                                                       const double* __restrict__ xr, double* __restrict__ Z, int d,
                                                       int P, int j0, int jn) {
  whiten_update_tile(L, X, xr, Z, d, P, j0, jn, blockIdx.x, blockIdx.y);
}

DEV void colnorm_block(const double* __restrict__ Z, int d, double* __restrict__ zq, int p) {
  __shared__ double red[256];
  double s = 0.0;
  for (int i = threadIdx.x; i < d; i += 256) {
    const double z = Z[i + (long)p * d];
    s = __fma_rn(z, z, s);
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) zq[p] = red[0];
}

__global__ __launch_bounds__(256) void k_colnorm(const double* __restrict__ Z, int d, double* __restrict__ zq) {
  colnorm_block(Z, d, zq, blockIdx.x);
}

hipError_t trsm_inverses(const double* L, double* Linv, int d, hipStream_t s) {
  hipLaunchKernelGGL(k_tri_inv, dim3(cdiv(d, CHOL_NB)), dim3(256), 0, s, L, d, Linv);
  return hipGetLastError();
}

hipError_t trsm_whiten(const double* L, const double* X, const double* xr, double* Z, double* zq, const double* Linv,
                       int d, int P, double* xr_copy, hipStream_t s) {
  const int rows = whiten_rows(d);
  const bool whole = rows >= d;
  for (int r0 = 0; r0 < d; r0 += rows) {
    const double* x = r0 ? nullptr : X;
    hipLaunchKernelGGL(k_whiten, dim3(cdiv(P, 16)), dim3(512), 0, s, L, Linv, x, xr, Z, whole ? zq : (double*)nullptr,
                       d, P, r0, rows, r0 ? (double*)nullptr : xr_copy);
    const int rem = d - (r0 + rows);
    if (rem > 0)
      hipLaunchKernelGGL(k_whiten_update, dim3(cdiv(rem, 64), cdiv(P, 64)), dim3(256), 0, s, L, x, xr, Z, d, P, r0,
                         rows);
  }
  if (zq && !whole) hipLaunchKernelGGL(k_colnorm, dim3(P), dim3(256), 0, s, Z, d, zq);
  return hipGetLastError();
}

// ---- batches of independent factorisations and whitenings -------------------
// One problem per blockIdx.z (the per-chain pairs of the local-global
// logistics), through the same device cores as potrf / trsm_whiten, so every
// problem's arithmetic is bitwise that of a separate call.  Problem z owns A
// + z sA, Linv + z sL, info[z]; the whitening works on column z of X and Z.
// skip (whitening): problem z is left untouched when skip[z] != 0.
__global__ __launch_bounds__(CHOL_DIAG_THREADS) void kb_chol_diag(double* __restrict__ A, long sA, int d, int j0, int jn,
                                                   double* __restrict__ Linv, long sL, int* __restrict__ info) {
  const int z = blockIdx.z;
  chol_diag_block(A + z * sA, d, j0, jn, Linv + z * sL, info + z);
}

__global__ __launch_bounds__(256) void kb_chol_panel(double* __restrict__ A, long sA, int d, int j0, int jn,
                                                     const double* __restrict__ Linv, long sL) {
  const int z = blockIdx.z;
  chol_panel_tile(A + z * sA, d, j0, jn, Linv + z * sL, blockIdx.x);
}

__global__ __launch_bounds__(256) void kb_chol_update_diag(double* __restrict__ A, long sA, int d, int jb,
                                                           double* __restrict__ Linv_next, long sL,
                                                           int* __restrict__ info) {
  constexpr int NLDS = CHOL_UPD_LDS > CHOL_DIAG_LDS ? CHOL_UPD_LDS : CHOL_DIAG_LDS;
  __shared__ __attribute__((aligned(1024))) double lds[NLDS];
  const int z = blockIdx.z;
  double* Az = A + z * sA;
  chol_update_core(Az, d, jb, blockIdx.x, lds);
  if (blockIdx.x == 0) {
    __syncthreads();
    const int j1 = (jb + 1) * CHOL_NB;
    chol_diag_core(Az, d, j1, min(CHOL_NB, d - j1), Linv_next + z * sL, info + z, lds);
  }
}

hipError_t potrf_batched(double* A, long sA, int d, int* info, double* Linv, long sL, int nprob, hipStream_t s) {
  if (nprob < 1 || nprob > 65535) return hipErrorInvalidValue;
  const int nb = cdiv(d, CHOL_NB);
  hipLaunchKernelGGL(kb_chol_diag, dim3(1, 1, nprob), dim3(CHOL_DIAG_THREADS), 0, s, A, sA, d, 0, min(CHOL_NB, d),
                     Linv, sL, info);
  for (int jb = 0; jb + 1 < nb; ++jb) {
    const int j0 = jb * CHOL_NB, jn = CHOL_NB;
    const int m = nb - jb - 1;
    hipLaunchKernelGGL(kb_chol_panel, dim3(m * (CHOL_NB / CHOL_PANEL_ROWS), 1, nprob), dim3(256), 0, s, A, sA, d, j0,
                       jn, (const double*)(Linv + (long)jb * CHOL_NB * CHOL_NB), sL);
    hipLaunchKernelGGL(kb_chol_update_diag, dim3(chol_update_tiles(nb, jb), 1, nprob), dim3(256), 0, s, A, sA, d, jb,
                       Linv + (long)(jb + 1) * CHOL_NB * CHOL_NB, sL, info);
  }
  return hipGetLastError();
}

__global__ __launch_bounds__(512) void kb_whiten(const double* __restrict__ L, long sA, const double* __restrict__ Linv,
                                                 long sL, const double* __restrict__ X,
                                                 const double* __restrict__ xrp, double* __restrict__ Z,
                                                 double* __restrict__ zq, int d, int r0, int rows,
                                                 const int* __restrict__ skip) {
  const int z = blockIdx.z;
  if (skip[z]) return;
  const long o = (long)z * d;
  whiten_tile(L + z * sA, Linv + z * sL, X ? X + o : nullptr, xrp + o, Z + o, zq ? zq + z : nullptr, d, 1, r0,
                    rows, 0);
}

__global__ __launch_bounds__(256) void kb_whiten_update(const double* __restrict__ L, long sA,
                                                        const double* __restrict__ X, const double* __restrict__ xrp,
                                                        double* __restrict__ Z, int d, int j0, int jn,
                                                        const int* __restrict__ skip) {
  const int z = blockIdx.z;
  if (skip[z]) return;
  const long o = (long)z * d;
  whiten_update_tile(L + z * sA, X ? X + o : nullptr, xrp + o, Z + o, d, 1, j0, jn, blockIdx.x, 0);
}

__global__ __launch_bounds__(256) void kb_colnorm(const double* __restrict__ Z, int d, double* __restrict__ zq,
                                                  const int* __restrict__ skip) {
  if (skip[blockIdx.x]) return;
  colnorm_block(Z, d, zq, blockIdx.x);
}

hipError_t trsm_whiten_batched(const double* L, long sA, const double* X, const double* xrp, double* Z, double* zq,
                               const double* Linv, long sL, int d, int P, const int* skip, hipStream_t s) {
  if (P < 1 || P > 65535) return hipErrorInvalidValue;
  const int rows = whiten_rows(d);
  const bool whole = rows >= d;
  for (int r0 = 0; r0 < d; r0 += rows) {
    const double* x = r0 ? nullptr : X;
    hipLaunchKernelGGL(kb_whiten, dim3(1, 1, P), dim3(512), 0, s, L, sA, Linv, sL, x, xrp, Z,
                  whole ? zq : (double*)nullptr, d, r0, rows, skip);
    const int rem = d - (r0 + rows);
    if (rem > 0)
      hipLaunchKernelGGL(kb_whiten_update, dim3(cdiv(rem, 64), 1, P), dim3(256), 0, s, L, sA, x, xrp, Z, d, r0, rows,
                         skip);
  }
  if (!whole) hipLaunchKernelGGL(kb_colnorm, dim3(P), dim3(256), 0, s, Z, d, zq, skip);
  return hipGetLastError();
}

// ============================================================================
// random numbers: Philox4x32-10 counters (stream 0 = W, 1 + g = U stage g)
// ============================================================================
// Four FP32 normals from counter ctr of the stream (Box-Muller on the four
// 24-bit uniforms of one Philox block).
DEV void normals4_f32(uint32_t k0, uint32_t k1, uint64_t ctr, float* v) {
  const u4_t r = philox4x32_10({(uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u}, k0, k1);
  const float ua = u01_f32(r.x), ub = u01_f32(r.y), uc = u01_f32(r.z), ud = u01_f32(r.w);
  const float ra = sqrtf(-2.0f * logf(ua)), rc = sqrtf(-2.0f * logf(uc));
  float s1, c1, s2, c2;
  sincosf(6.28318530717958647692f * ub, &s1, &c1);
  sincosf(6.28318530717958647692f * ud, &s2, &c2);
  v[0] = ra * c1;
  v[1] = ra * s1;
  v[2] = rc * c2;
  v[3] = rc * s2;
}

DEV void uniform_elem(uint32_t k0, uint32_t k1, long s0, int P, int stages, double* __restrict__ U, long e) {
  const int p = (int)(e % P);
  const long tg = e / P;
  const int g = (int)(tg % stages);
  const uint64_t st = (uint64_t)(s0 + tg / stages);
  const u4_t r = philox4x32_10({(uint32_t)st, (uint32_t)(st >> 32), 1u + (uint32_t)g, (uint32_t)(p >> 1)}, k0, k1);
  U[e] = (p & 1) ? u01_f64(r.z, r.w) : u01_f64(r.x, r.y);
}

// The workgroups from nblk on draw the call's nu uniforms.
__global__ __launch_bounds__(256) void k_normals(int prec, uint32_t k0, uint32_t k1, long g0, long total,
                                                 void* __restrict__ W, void* __restrict__ Wlo, int nblk, long s0, int P,
                                                 int stages, long nu, double* __restrict__ U) {
  if ((int)blockIdx.x >= nblk) {
    const long e = (long)(blockIdx.x - nblk) * 256 + threadIdx.x;
    if (e < nu) uniform_elem(k0, k1, s0, P, stages, U, e);
    return;
  }
  const long stride = (long)nblk * 256;
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  if (prec == P64) {
    for (long q = gid; 2 * q < total; q += stride) {
      const uint64_t ctr = (uint64_t)(g0 + 2 * q);
      const u4_t r = philox4x32_10({(uint32_t)ctr, (uint32_t)(ctr >> 32), 0u, 0u}, k0, k1);
      const double u1 = u01_f64(r.x, r.y), u2 = u01_f64(r.z, r.w);
      const double rad = sqrt(-2.0 * log(u1));
      double sn, cs;
      sincos(6.283185307179586476925286766559 * u2, &sn, &cs);
      double* w = (double*)W;
      w[2 * q] = rad * cs;
      if (2 * q + 1 < total) w[2 * q + 1] = rad * sn;
    }
  } else {
    const bool vec = (uintptr_t)W % 16 == 0 && (prec == P32 || (uintptr_t)Wlo % 8 == 0);
    for (long q = gid; 4 * q < total; q += stride) {
      float v[4];
      normals4_f32(k0, k1, (uint64_t)(g0 + 4 * q), v);
      if (4 * q + 3 < total && vec) {
        // the thread's four values as one 16-byte (FP32) or two 8-byte stores
        if (prec == P32) {
          *(float4*)((float*)W + 4 * q) = make_float4(v[0], v[1], v[2], v[3]);
        } else {
          u16 hi[4], lo[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) split_bf16(v[e], hi[e], lo[e]);
          *(uint2*)((u16*)W + 4 * q) = make_uint2(hi[0] | ((uint32_t)hi[1] << 16), hi[2] | ((uint32_t)hi[3] << 16));
          *(uint2*)((u16*)Wlo + 4 * q) = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
        }
        continue;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const long idx = 4 * q + e;
        if (idx < total) {
          if (prec == P32) {
            ((float*)W)[idx] = v[e];
          } else {
            u16 hi, lo;
            split_bf16(v[e], hi, lo);
            ((u16*)W)[idx] = hi;
            ((u16*)Wlo)[idx] = lo;
          }
        }
      }
    }
  }
}

hipError_t draws(Prec prec, uint64_t seed, long s0, int n, int d, int P, int stages, void* W, void* Wlo, double* U,
                 hipStream_t s) {
  const long total = W ? (long)n * P * d : 0, nu = U ? (long)n * stages * P : 0;
  if (total + nu <= 0) return hipSuccess;
  const long per = (prec == P64) ? 2 : 4;
  const long nq = (total + per - 1) / per;
  const int nb = (int)std::min((nq + 255) / 256, 4096L);
  hipLaunchKernelGGL(k_normals, dim3((unsigned)(nb + (nu + 255) / 256)), dim3(256), 0, s, (int)prec, (uint32_t)seed,
                     (uint32_t)(seed >> 32), s0 * (long)P * d, total, W, Wlo, nb, s0, P, stages, nu, U);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_convert_normals(int prec, const double* __restrict__ W64, long count,
                                                         void* __restrict__ W, void* __restrict__ Wlo) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= count) return;
  const float f = (float)W64[e];
  if (prec == P32) {
    ((float*)W)[e] = f;
  } else {
    u16 hi, lo;
    split_bf16(f, hi, lo);
    ((u16*)W)[e] = hi;
    ((u16*)Wlo)[e] = lo;
  }
}

hipError_t convert_normals(Prec prec, const double* W64, long count, void* W, void* Wlo, hipStream_t s) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_convert_normals, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, (int)prec, W64, count,
                     W, Wlo);
  return hipGetLastError();
}

// ============================================================================
// (c) accept / reject of step t fused with the proposal of step t+1.
// One wavefront per (chain, 512-row chunk); the chain's decision is formed
// redundantly by every wavefront of that chain from the same partial sums in
// the same order, so all of them agree bitwise.
// ============================================================================
template <int PR> struct StepT;
template <> struct StepT<P64> { typedef double XI; typedef double WT; typedef double VT; typedef double WIN; };
template <> struct StepT<P32> { typedef float XI; typedef float WT; typedef float VT; typedef float WIN; };
template <> struct StepT<PMIX> { typedef float XI; typedef u16 WT; typedef float VT; typedef u16 WIN; };

template <int PR>
DEV double load_w(const void* w, const void* wlo, long e) {
  if (PR == P64) return ((const double*)w)[e];
  if (PR == P32) return (double)((const float*)w)[e];
  return (double)bf16_bits_to_f32(((const u16*)w)[e]) + (double)bf16_bits_to_f32(((const u16*)wlo)[e]);
}

template <int PR>
DEV void store_win(void* win, long e, double v) {
  if (PR == P64) ((double*)win)[e] = v;
  else if (PR == P32) ((float*)win)[e] = (float)v;
  else ((u16*)win)[e] = f32_to_bf16_bits((float)v);
}

constexpr int MAXPROJ = 4;

// chunk ch of nch (STEP_RCH rows each) of chains 4 pq .. 4 pq + 3, one wave each.
// MODE 0: decision and state update in one pass (every chunk's wave
// recomputes its chain's decision); MODE 1: decision only (one wave per
// chain, ch = 0), written to acc_out and the per-chain scalars; MODE 2: state
// update and next proposal only, reading the decision from acc_out.
template <int PR, int MODE = 0>
DEV void step_body(const StepArgs& a, int ch, int nch, int pq) {
  typedef typename StepT<PR>::XI XI;
  typedef typename StepT<PR>::VT VT;
  constexpr int RPL = STEP_RCH / 64;  // rows per lane
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int p = pq * 4 + w;
  if (p >= a.P) return;
  const int d = a.d, P = a.P;
  const int r0 = ch * STEP_RCH;
  const XI* xi_cur = (const XI*)a.xi_cur;
  const XI* xi_nxt = (const XI*)a.xi_nxt;
  VT* V = (VT*)a.V;
  // issue every row load of this lane first; the chain's decision (which
  // needs two reductions and a log) overlaps their latency
  double x[RPL], z[RPL], xr[RPL], xc[RPL], wc[RPL], xn[RPL], wn[RPL], mu[RPL];
  bool in[RPL];
#pragma unroll
  for (int q = 0; q < RPL && MODE != 1; ++q) {
    const int i = r0 + q * 64 + lane;
    in[q] = i < d;
    const long e = i + (long)p * d;
    x[q] = z[q] = xr[q] = xc[q] = wc[q] = xn[q] = wn[q] = mu[q] = 0.0;
    if (in[q]) {
      x[q] = a.X[e];
      z[q] = a.Z[e];
      xr[q] = a.xr[i];
      const long ew = i + (long)p * (a.ldw ? a.ldw : d);
      if (a.do_accept) {
        xc[q] = (double)xi_cur[ew];
        wc[q] = load_w<PR>(a.w_cur, a.wlo_cur, ew);
      }
      if (a.do_propose) {
        xn[q] = (double)xi_nxt[ew];
        wn[q] = load_w<PR>(a.w_nxt, a.wlo_nxt, ew);
        mu[q] = a.mu ? a.mu[i] : 0.0;
      }
    }
  }
  bool acc = false;
  if (MODE == 2 && a.do_accept) acc = a.acc_out[p] != 0;
  if (MODE != 2 && a.do_accept) {
    // exact log density of the proposal: target partials (of this chain, or
    // of its survivor slot under delayed acceptance) plus the prior
    const bool live = !a.da || a.pass1[p];
    const int col = a.da ? a.slot[p] : p;
    double s = 0.0;
    if (live)
      for (int q = lane; q < a.nrb; q += 64) s += a.lpp_part[(long)col * a.nrb + q];
    s = wave_sum_f64(s);
    if (a.prior_w > 0.0) {
      double pq = 0.0;
      for (int q = lane; q < nch; q += 64) pq += a.pq_part_cur[(long)p * nch + q];
      pq = wave_sum_f64(pq);
      s = __fma_rn(-a.prior_w, pq, s);
    }
    const double lpp = s;
    double zs = 0.0;
    for (int q = lane; q < nch; q += 64) zs += a.zq_part_cur[(long)p * nch + q];
    zs = wave_sum_f64(zs);
    const double lp = a.lp_cur[p], zq = a.zq_cur[p];
    double la;
    if (!a.da) {
      la = (lpp + zs * a.inv2a2) - (lp + zq * a.inv2a2);
      acc = log(a.u[p]) < la;  // NaN compares false: rejected
    } else {
      // second stage: log alpha_2 = (log pi(x') - log pi(x)) - (s(x') - s(x)),
      // with s = r - |z|^2/(2 alpha^2) in the residual form (r = network)
      double l2 = (lpp - lp) - (a.s_new[p] - a.s_in[p]);
      if (a.da_resid) l2 += (zs - zq) * a.inv2a2;
      la = live ? l2 : -INFINITY;
      acc = live && (log(a.u2[p]) < la);
    }
    if (ch == 0 && lane == 0) {
      a.lp_nxt[p] = acc ? lpp : lp;
      a.zq_nxt[p] = acc ? zs : zq;
      a.nacc[p] += acc ? 1 : 0;
      if (a.wacc) a.wacc[p] += acc ? 1 : 0;
      a.la_out[p] = la;
      a.acc_out[p] = acc ? 1 : 0;
      if (a.da) a.s_out[p] = acc ? a.s_new[p] : a.s_in[p];
      if (a.trace_lp) a.trace_lp[p] = acc ? lpp : lp;
      if (live && isinf(lpp) && lpp > 0.0) atomicOr(a.err, 1);
    }
  }
  if (MODE == 1) return;
  double zacc = 0.0, xacc = 0.0;
  double pacc[MAXPROJ] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < RPL; ++q) {
    if (!in[q]) continue;
    const int i = r0 + q * 64 + lane;
    const long e = i + (long)p * d;
    double xv = x[q], zv = z[q];
    if (a.do_accept) {
      if (acc) {
        xv = propose1(xr[q], xv, a.rho, xc[q]);
        zv = __fma_rn(a.c, wc[q], a.rho * zv);
        a.X[e] = xv;
        a.Z[e] = zv;
      }
      store_win<PR>(a.win, i + (a.win_col0 + p) * (long)(a.ldwin ? a.ldwin : d), xv - xr[q]);
      for (int k = 0; k < a.nproj; ++k) pacc[k] = __fma_rn(a.proj[i + (long)k * d], xv, pacc[k]);
    }
    if (a.do_propose) {
      const double xp = propose1(xr[q], xv, a.rho, xn[q]);
      if (a.vh) {
        u16 h, l;
        const double sv = (xp - mu[q]) * (double)a.vsc[i];
        if (fabs(sv) >= H2_RANGE) atomicOr(a.err, 2);
        split_f16(sv, h, l);
        a.vh[e] = h;
        a.vh[(long)d * P + e] = l;
      } else {
        const long ev = i + (long)p * (a.ldv ? a.ldv : d);
        if (a.v32) ((float*)a.V)[ev] = (float)(xp - mu[q]);
        else V[ev] = (VT)(xp - mu[q]);
      }
      const double zp = __fma_rn(a.c, wn[q], a.rho * zv);
      zacc = __fma_rn(zp, zp, zacc);
      xacc = __fma_rn(xp, xp, xacc);
    }
  }
  if (a.do_propose) {
    zacc = wave_sum_f64(zacc);
    if (lane == 0) a.zq_part_nxt[(long)p * nch + ch] = zacc;
    if (a.prior_w > 0.0) {
      xacc = wave_sum_f64(xacc);
      if (lane == 0) a.pq_part_nxt[(long)p * nch + ch] = xacc;
    }
  }
  if (a.do_accept && a.nproj > 0) {
    for (int k = 0; k < a.nproj; ++k) {
      const double v = wave_sum_f64(pacc[k]);
      if (lane == 0) a.proj_part[((long)ch * a.nproj + k) * P + p] = v;
    }
  }
}

// Sum over the 256 threads of a workgroup in a fixed order (every thread
// gets the result).  red: 4 doubles of LDS.
DEV double block_sum_f64(double v, double* red) {
  v = wave_sum_f64(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  __syncthreads();
  if (lane == 0) red[w] = v;
  __syncthreads();
  return (red[0] + red[1]) + (red[2] + red[3]);
}

// Stopping errors of the experiments (Section 3.3): |S - m m^T - Sigma|_F^2,
// |Sigma|_F^2 and |m - mu|^2, as per-block FP64 partial sums (fixed order)
// reduced by one more block: deterministic (MERR_BLOCKS in kernels.h).

__global__ __launch_bounds__(256) void k_moment_err(const double* __restrict__ S, const double* __restrict__ m,
                                                    const double* __restrict__ Sigma, const double* __restrict__ mu,
                                                    int d, double* __restrict__ part) {
  __shared__ double red[4];
  const long n = (long)d * d;
  double a = 0.0, b = 0.0, c = 0.0;
  for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
    const int i = (int)(e % d), j = (int)(e / d);
    const double sg = Sigma[e];
    const double u = (S[e] - m[i] * m[j]) - sg;
    a = __fma_rn(u, u, a);
    b = __fma_rn(sg, sg, b);
  }
  if (mu)
    for (int i = blockIdx.x * 256 + threadIdx.x; i < d; i += gridDim.x * 256) {
      const double u = m[i] - mu[i];
      c = __fma_rn(u, u, c);
    }
  a = block_sum_f64(a, red);
  b = block_sum_f64(b, red);
  c = block_sum_f64(c, red);
  if (threadIdx.x == 0) {
    part[3 * blockIdx.x] = a;
    part[3 * blockIdx.x + 1] = b;
    part[3 * blockIdx.x + 2] = c;
  }
}

__global__ __launch_bounds__(256) void k_moment_err_final(const double* __restrict__ part, int nb,
                                                          double* __restrict__ out) {
  __shared__ double red[4];
  double a = 0.0, b = 0.0, c = 0.0;
  for (int k = threadIdx.x; k < nb; k += 256) {
    a += part[3 * k];
    b += part[3 * k + 1];
    c += part[3 * k + 2];
  }
  a = block_sum_f64(a, red);
  b = block_sum_f64(b, red);
  c = block_sum_f64(c, red);
  if (threadIdx.x == 0) {
    out[0] = sqrt(a / b);
    out[1] = sqrt(c);
  }
}

size_t moment_err_scratch_bytes() { return MERR_SCRATCH_DOUBLES * sizeof(double); }

hipError_t moment_error(const double* S, const double* m, const double* Sigma, const double* mu, int d, double* scratch,
                        hipStream_t s) {
  const int nb = min(MERR_BLOCKS, cdiv((long)d * d, 256));
  hipLaunchKernelGGL(k_moment_err, dim3(nb), dim3(256), 0, s, S, m, Sigma, mu, d, scratch + 2);
  hipLaunchKernelGGL(k_moment_err_final, dim3(1), dim3(256), 0, s, (const double*)(scratch + 2), nb, scratch);
  return hipGetLastError();
}


// Target partials of chain col, and row block q's term (the sum of its halves
// or quarters where the target kernel wrote those).
DEV const double* chain_parts(const StepArgs& a, int col) {
  return a.lpp_part + (long)col * (a.sub == 4 ? tgt_quarters(a.d) : a.sub == 2 ? (a.d + 31) / 32 : a.nrb);
}
DEV double row_block_part(const StepArgs& a, const double* parts, int q) {
  if (a.sub <= 1) return parts[q];
  const bool two = 64 * q + 32 < a.d;  // the block has a second half
  if (a.sub == 2) return parts[2 * q] + (two ? parts[2 * q + 1] : 0.0);
  const double* f = parts + 4 * q;
  return (f[0] + f[1]) + (two ? f[2] + f[3] : 0.0);
}

// Decision of chain p by one workgroup of 256 threads: the target partials
// (thousands of row blocks for the logistic target) are summed by all
// threads, then MH (or the second stage of delayed acceptance) decides.
DEV void decide_block(const StepArgs& a, int nch, int p) {
  __shared__ double red[4];
  const int t = threadIdx.x;
  const bool live = !a.da || a.pass1[p];
  const int col = a.da ? a.slot[p] : p;
  double s = 0.0;
  if (live)
    for (int q = t; q < a.nrb; q += 256) s += row_block_part(a, chain_parts(a, col), q);
  s = block_sum_f64(s, red);
  if (a.prior_w > 0.0) {
    double pq = 0.0;
    for (int q = t; q < nch; q += 256) pq += a.pq_part_cur[(long)p * nch + q];
    pq = block_sum_f64(pq, red);
    s = __fma_rn(-a.prior_w, pq, s);
  }
  const double lpp = s;
  double zs = 0.0;
  for (int q = t; q < nch; q += 256) zs += a.zq_part_cur[(long)p * nch + q];
  zs = block_sum_f64(zs, red);
  if (t != 0) return;
  const double lp = a.lp_cur[p], zq = a.zq_cur[p];
  double la;
  bool acc;
  if (!a.da) {
    la = (lpp + zs * a.inv2a2) - (lp + zq * a.inv2a2);
    acc = log(a.u[p]) < la;  // NaN compares false: rejected
  } else {
    // second stage: log alpha_2 = (log pi(x') - log pi(x)) - (s(x') - s(x)),
    // with s = r - |z|^2/(2 alpha^2) in the residual form (r = network)
    double l2 = (lpp - lp) - (a.s_new[p] - a.s_in[p]);
    if (a.da_resid) l2 += (zs - zq) * a.inv2a2;
    la = live ? l2 : -INFINITY;
    acc = live && (log(a.u2[p]) < la);
  }
  a.lp_nxt[p] = acc ? lpp : lp;
  a.zq_nxt[p] = acc ? zs : zq;
  a.nacc[p] += acc ? 1 : 0;
  if (a.wacc) a.wacc[p] += acc ? 1 : 0;
  a.la_out[p] = la;
  a.acc_out[p] = acc ? 1 : 0;
  if (a.da) a.s_out[p] = acc ? a.s_new[p] : a.s_in[p];
  if (a.trace_lp) a.trace_lp[p] = acc ? lpp : lp;
  if (live && isinf(lpp) && lpp > 0.0) atomicOr(a.err, 1);
}

__global__ __launch_bounds__(256) void k_decide(StepArgs a, int nch) { decide_block(a, nch, blockIdx.x); }

// The decision of chain p taken by one wavefront inside the update launch
// (no delayed acceptance; at most 64 target row blocks and 64 row chunks).
// With that many partials decide_block's block sums reduce to wave 0's
// shuffle sum plus exact zeros, so these sums, log alpha and the verdict are
// bitwise decide_block's.  Every row-chunk workgroup of the chain takes the
// (cheap, L2-resident) decision; only `write` stores its outputs.
// parts: the chain's nrb target partials (global memory or LDS).
// The decision's inputs other than the target's row-block terms, all written
// by earlier launches: this lane's z-norm (and prior) partial of the
// proposal, the current state's log pi and z-norm, and the uniform.  A kernel
// that waits for the target's terms can load these first.
struct DecIn {
  double zs, pq, lp, zq, u;
  int nacc, wacc;  // the chain's counters, for the wavefront that writes them
};

DEV DecIn decide_inputs(const StepArgs& a, int nch, int p, bool write) {
  const int lane = threadIdx.x & 63;
  DecIn in;
  in.nacc = in.wacc = 0;
  if (write) {
    in.nacc = a.nacc[p];
    if (a.wacc) in.wacc = a.wacc[p];
  }
  in.zs = lane < nch ? 0.0 + a.zq_part_cur[(long)p * nch + lane] : 0.0;
  in.pq = (a.prior_w > 0.0 && lane < nch) ? 0.0 + a.pq_part_cur[(long)p * nch + lane] : 0.0;
  in.lp = a.lp_cur[p];
  in.zq = a.zq_cur[p];
  in.u = a.u[p];
  return in;
}

DEV double lane_part(const StepArgs& a, const double* parts) {
  const int lane = threadIdx.x & 63;
  return lane < a.nrb ? 0.0 + row_block_part(a, parts, lane) : 0.0;
}

DEV bool decide_wave(const StepArgs& a, int p, bool write, double part, const DecIn& in) {
  const int lane = threadIdx.x & 63;
  const double lu = log(in.u);
  double s = wave_sum_f64(part);
  if (a.prior_w > 0.0) {
    const double pq = wave_sum_f64(in.pq);
    s = __fma_rn(-a.prior_w, pq, s);
  }
  const double lpp = s;
  const double zs = wave_sum_f64(in.zs);
  const double lp = in.lp, zq = in.zq;
  const double la = (lpp + zs * a.inv2a2) - (lp + zq * a.inv2a2);
  const bool acc = lu < la;  // NaN compares false: rejected
  if (write && lane == 0) {
    a.lp_nxt[p] = acc ? lpp : lp;
    a.zq_nxt[p] = acc ? zs : zq;
    a.nacc[p] = in.nacc + (acc ? 1 : 0);
    if (a.wacc) a.wacc[p] = in.wacc + (acc ? 1 : 0);
    a.la_out[p] = la;
    a.acc_out[p] = acc ? 1 : 0;
    if (a.trace_lp) a.trace_lp[p] = acc ? lpp : lp;
    if (isinf(lpp) && lpp > 0.0) atomicOr(a.err, 1);
  }
  return acc;
}

DEV bool decide_wave(const StepArgs& a, int nch, int p, bool write, const double* parts) {
  return decide_wave(a, p, write, lane_part(a, parts), decide_inputs(a, nch, p, write));
}

// Paired-row loads and stores for the update half (d even, so that every
// chain's column starts on an even element): lane l owns rows 2l, 2l + 1 of
// its 128-row chunk and moves them with 16-, 8- or 4-byte accesses.
// 128-row chunks per wavefront of the update (two: half the wavefronts take
// the same decision; one or four ran slower at d = 4096, P = 256)
#ifndef STEP_CPW
#define STEP_CPW 2
#endif
template <int PR> struct Pair2;
template <> struct Pair2<P64> { typedef double2 XI; typedef double2 W; };
template <> struct Pair2<P32> { typedef float2 XI; typedef float2 W; };
template <> struct Pair2<PMIX> { typedef float2 XI; typedef uint32_t W; };

template <int PR>
DEV void store_win2(void* win, long e, double v0, double v1) {
  if (PR == P64) {
    *(double2*)((double*)win + e) = make_double2(v0, v1);
  } else if (PR == P32) {
    *(float2*)((float*)win + e) = make_float2((float)v0, (float)v1);
  } else {
    *(uint32_t*)((u16*)win + e) = (uint32_t)f32_to_bf16_bits((float)v0) | ((uint32_t)f32_to_bf16_bits((float)v1) << 16);
  }
}

// The update of chain p over row chunks CPW cb .. CPW cb + CPW - 1 (STEP_RCH
// rows each; chunks past nch are skipped), one wavefront, in two phases:
// upd_load issues every load that does not depend on the chain's decision
// (keeping the raw bits, so nothing waits for them there), upd_finish takes
// the decision, loads the accepted proposal's Xi and W for every chunk
// before it converts any, and stores.  One partial per chunk, so the partials are those of one chunk
// per wavefront whatever CPW is.
// A row pair of a proposal's Xi and W as loaded (both bf16 parts of W in the
// mixed form); the conversion to double (raw_xi, raw_w; W = hi + lo in the
// mixed form) is left to where the values are used, so that the loads stay
// in flight until then instead of being waited for at once.
template <int PR> struct Raw2;
template <> struct Raw2<P64> { double2 xi, w; };
template <> struct Raw2<P32> { float2 xi, w; };
template <> struct Raw2<PMIX> { float2 xi; uint32_t wh, wl; };

DEV void raw_zero(Raw2<P64>& r) { r.xi = make_double2(0.0, 0.0); r.w = make_double2(0.0, 0.0); }
DEV void raw_zero(Raw2<P32>& r) { r.xi = make_float2(0.f, 0.f); r.w = make_float2(0.f, 0.f); }
DEV void raw_zero(Raw2<PMIX>& r) { r.xi = make_float2(0.f, 0.f); r.wh = r.wl = 0u; }

DEV void raw_load(Raw2<P64>& r, const void* xi, const void* w, const void*, long e) {
  r.xi = *(const double2*)((const double*)xi + e);
  r.w = *(const double2*)((const double*)w + e);
}
DEV void raw_load(Raw2<P32>& r, const void* xi, const void* w, const void*, long e) {
  r.xi = *(const float2*)((const float*)xi + e);
  r.w = *(const float2*)((const float*)w + e);
}
DEV void raw_load(Raw2<PMIX>& r, const void* xi, const void* w, const void* wlo, long e) {
  r.xi = *(const float2*)((const float*)xi + e);
  r.wh = *(const uint32_t*)((const u16*)w + e);
  r.wl = *(const uint32_t*)((const u16*)wlo + e);
}

DEV void raw_xi(const Raw2<P64>& r, double& v0, double& v1) { v0 = r.xi.x; v1 = r.xi.y; }
DEV void raw_xi(const Raw2<P32>& r, double& v0, double& v1) { v0 = r.xi.x; v1 = r.xi.y; }
DEV void raw_xi(const Raw2<PMIX>& r, double& v0, double& v1) { v0 = r.xi.x; v1 = r.xi.y; }
DEV void raw_w(const Raw2<P64>& r, double& w0, double& w1) { w0 = r.w.x; w1 = r.w.y; }
DEV void raw_w(const Raw2<P32>& r, double& w0, double& w1) { w0 = r.w.x; w1 = r.w.y; }
DEV void raw_w(const Raw2<PMIX>& r, double& w0, double& w1) {
  w0 = (double)bf16_bits_to_f32((u16)(r.wh & 0xffff)) + (double)bf16_bits_to_f32((u16)(r.wl & 0xffff));
  w1 = (double)bf16_bits_to_f32((u16)(r.wh >> 16)) + (double)bf16_bits_to_f32((u16)(r.wl >> 16));
}

template <int PR, int CPW>
struct UpdRegs {
  int ii[CPW];
  bool in[CPW];
  double x0[CPW], x1[CPW], z0[CPW], z1[CPW], r0[CPW], r1[CPW];
  double m0[CPW], m1[CPW];
  Raw2<PR> nw[CPW];  // the next proposal's Xi and W
  Raw2<PR> cw[CPW];  // the accepted proposal's Xi and W
  float2 sv[CPW];
};

template <int PR, int CPW>
DEV void upd_load(const StepArgs& a, int p, int cb, int nch, UpdRegs<PR, CPW>& g) {
  const int lane = threadIdx.x & 63;
  const int d = a.d;
  const long ldw = a.ldw ? a.ldw : d;
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    const int ch = cb * CPW + c;
    g.ii[c] = ch * STEP_RCH + 2 * lane;
    g.in[c] = ch < nch && g.ii[c] < d;  // d even: the pair lies wholly inside or outside
    g.x0[c] = g.x1[c] = g.z0[c] = g.z1[c] = g.r0[c] = g.r1[c] = 0.0;
    g.m0[c] = g.m1[c] = 0.0;
    raw_zero(g.nw[c]);
    g.sv[c] = make_float2(0.f, 0.f);
    if (g.in[c]) {
      const int i = g.ii[c];
      const long e = i + (long)p * d, ew = i + (long)p * ldw;
      const double2 xv = *(const double2*)(a.X + e), zv = *(const double2*)(a.Z + e);
      const double2 rv = *(const double2*)(a.xr + i);
      g.x0[c] = xv.x; g.x1[c] = xv.y; g.z0[c] = zv.x; g.z1[c] = zv.y; g.r0[c] = rv.x; g.r1[c] = rv.y;
      if (a.do_propose) {
        raw_load(g.nw[c], a.xi_nxt, a.w_nxt, a.wlo_nxt, ew);
        if (a.mu) {
          const double2 mv = *(const double2*)(a.mu + i);
          g.m0[c] = mv.x; g.m1[c] = mv.y;
        }
        if (a.vh) g.sv[c] = *(const float2*)(a.vsc + i);
      }
    }
  }
}

// The loads of an accepting and proposing step without branches: lanes past d
// read the chunk's first row, a target without a mean the pivot (neither is
// used), and both proposals are read whatever the decision will be.
template <int PR, int CPW>
DEV void upd_load_run(const StepArgs& a, int p, int cb, int nch, UpdRegs<PR, CPW>& g) {
  const int lane = threadIdx.x & 63;
  const int d = a.d;
  const long ldw = a.ldw ? a.ldw : d;
  const double* mu = a.mu ? a.mu : a.xr;
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    const int ch = cb * CPW + c;
    g.ii[c] = ch * STEP_RCH + 2 * lane;
    g.in[c] = g.ii[c] < d;  // ch < nch in its launch
    const int i = g.in[c] ? g.ii[c] : ch * STEP_RCH;
    const long e = i + (long)p * d, ew = i + (long)p * ldw;
    const double2 xv = *(const double2*)(a.X + e), zv = *(const double2*)(a.Z + e);
    raw_load(g.cw[c], a.xi_cur, a.w_cur, a.wlo_cur, ew);
    raw_load(g.nw[c], a.xi_nxt, a.w_nxt, a.wlo_nxt, ew);
    const double2 rv = *(const double2*)(a.xr + i), mv = *(const double2*)(mu + i);
    g.x0[c] = xv.x; g.x1[c] = xv.y; g.z0[c] = zv.x; g.z1[c] = zv.y; g.r0[c] = rv.x; g.r1[c] = rv.y;
    g.m0[c] = mv.x; g.m1[c] = mv.y;
  }
}

// RUN: the step accepts and proposes, and g comes from upd_load_run.
template <int PR, int CPW, bool RUN = false>
DEV void upd_finish(const StepArgs& a, int p, int cb, int nch, bool acc, UpdRegs<PR, CPW>& g) {
  const int lane = threadIdx.x & 63;
  const int d = a.d, P = a.P;
  const long ldw = a.ldw ? a.ldw : d;
  const bool do_accept = RUN || a.do_accept, do_propose = RUN || a.do_propose;
  if (!RUN)
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      raw_zero(g.cw[c]);
      if (g.in[c] && acc) raw_load(g.cw[c], a.xi_cur, a.w_cur, a.wlo_cur, g.ii[c] + (long)p * ldw);
    }
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    const int ch = cb * CPW + c;
    if (ch >= nch) break;
    const int i = g.ii[c];
    const long e = i + (long)p * d;
    double zacc = 0.0, xacc = 0.0;
    double pacc[MAXPROJ] = {0.0, 0.0, 0.0, 0.0};
    if (g.in[c]) {
      double xa = g.x0[c], xb = g.x1[c], za = g.z0[c], zb = g.z1[c];
      const double ra = g.r0[c], rb = g.r1[c];
      if (do_accept) {
        if (acc) {
          double c0, c1, wc0, wc1;
          raw_xi(g.cw[c], c0, c1);
          raw_w(g.cw[c], wc0, wc1);
          xa = propose1(ra, xa, a.rho, c0);
          xb = propose1(rb, xb, a.rho, c1);
          za = __fma_rn(a.c, wc0, a.rho * za);
          zb = __fma_rn(a.c, wc1, a.rho * zb);
          *(double2*)(a.X + e) = make_double2(xa, xb);
          *(double2*)(a.Z + e) = make_double2(za, zb);
        }
        store_win2<PR>(a.win, i + (a.win_col0 + p) * (long)(a.ldwin ? a.ldwin : d), xa - ra, xb - rb);
        for (int k = 0; k < a.nproj; ++k) {
          const double2 pv = *(const double2*)(a.proj + i + (long)k * d);
          pacc[k] = __fma_rn(pv.y, xb, __fma_rn(pv.x, xa, pacc[k]));
        }
      }
      if (do_propose) {
        double n0, n1, wn0, wn1;
        raw_xi(g.nw[c], n0, n1);
        raw_w(g.nw[c], wn0, wn1);
        const double xp0 = propose1(ra, xa, a.rho, n0), xp1 = propose1(rb, xb, a.rho, n1);
        const double m0 = RUN && !a.mu ? 0.0 : g.m0[c], m1 = RUN && !a.mu ? 0.0 : g.m1[c];
        if (!RUN && a.vh) {
          u16 h0, l0, h1, l1;
          const double s0 = (xp0 - m0) * (double)g.sv[c].x, s1 = (xp1 - m1) * (double)g.sv[c].y;
          if (fmax(fabs(s0), fabs(s1)) >= H2_RANGE) atomicOr(a.err, 2);
          split_f16(s0, h0, l0);
          split_f16(s1, h1, l1);
          *(uint32_t*)(a.vh + e) = (uint32_t)h0 | ((uint32_t)h1 << 16);
          *(uint32_t*)(a.vh + (long)d * P + e) = (uint32_t)l0 | ((uint32_t)l1 << 16);
        } else {
          const long ev = i + (long)p * (a.ldv ? a.ldv : d);
          if (a.v32 || PR != P64)
            *(float2*)((float*)a.V + ev) = make_float2((float)(xp0 - m0), (float)(xp1 - m1));
          else *(double2*)((double*)a.V + ev) = make_double2(xp0 - m0, xp1 - m1);
        }
        const double zp0 = __fma_rn(a.c, wn0, a.rho * za), zp1 = __fma_rn(a.c, wn1, a.rho * zb);
        zacc = __fma_rn(zp1, zp1, __fma_rn(zp0, zp0, 0.0));
        xacc = __fma_rn(xp1, xp1, __fma_rn(xp0, xp0, 0.0));
      }
    }
    if (do_propose) {
      zacc = wave_sum_f64(zacc);
      if (lane == 0) a.zq_part_nxt[(long)p * nch + ch] = zacc;
      if (a.prior_w > 0.0) {
        xacc = wave_sum_f64(xacc);
        if (lane == 0) a.pq_part_nxt[(long)p * nch + ch] = xacc;
      }
    }
    if (do_accept && a.nproj > 0) {
      for (int k = 0; k < a.nproj; ++k) {
        const double v = wave_sum_f64(pacc[k]);
        if (lane == 0) a.proj_part[((long)ch * a.nproj + k) * P + p] = v;
      }
    }
  }
}

// The update of chain 4 pq + (wave) over the chunks of cb.
template <int PR, int CPW = 1>
DEV void step_update2(const StepArgs& a, int cb, int nch, int pq) {
  const int w = threadIdx.x >> 6;
  const int p = pq * 4 + w;
  if (p >= a.P) return;
  UpdRegs<PR, CPW> g;
  upd_load<PR, CPW>(a, p, cb, nch, g);
  const bool acc =
      a.do_accept && (a.fuse_dec ? decide_wave(a, nch, p, cb == 0, chain_parts(a, p)) : a.acc_out[p] != 0);
  upd_finish<PR, CPW>(a, p, cb, nch, acc, g);
}

// The update half of k_step_h2, where every 128-row chunk lies inside d (d a
// multiple of 256, two chunks per wavefront), the target's mean and the
// proposal's scales are set, and PROP tells whether the step proposes.  Its
// loads are issued without branches and kept raw, so the compiler keeps them
// in flight until their first use (the shared upd_load and upd_finish wait
// for each chunk's loads at the branches that guard them); the arithmetic and
// the stores are those of upd_finish.
template <bool PROP>
DEV void upd_load_h2(const StepArgs& a, int p, int cb, UpdRegs<PMIX, 2>& g) {
  const int lane = threadIdx.x & 63;
  const int d = a.d;
  const long ldw = a.ldw ? a.ldw : d;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int i = (cb * 2 + c) * STEP_RCH + 2 * lane;
    g.ii[c] = i;
    g.in[c] = true;
    const long e = i + (long)p * d, ew = i + (long)p * ldw;
    const double2 xv = *(const double2*)(a.X + e), zv = *(const double2*)(a.Z + e);
    const double2 rv = *(const double2*)(a.xr + i);
    g.x0[c] = xv.x; g.x1[c] = xv.y; g.z0[c] = zv.x; g.z1[c] = zv.y; g.r0[c] = rv.x; g.r1[c] = rv.y;
    if (PROP) {
      raw_load(g.nw[c], a.xi_nxt, a.w_nxt, a.wlo_nxt, ew);
      const double2 mv = *(const double2*)(a.mu + i);
      g.m0[c] = mv.x; g.m1[c] = mv.y;
      g.sv[c] = *(const float2*)(a.vsc + i);
    } else {
      raw_zero(g.nw[c]);
      g.m0[c] = g.m1[c] = 0.0;
      g.sv[c] = make_float2(0.f, 0.f);
    }
  }
}

template <bool PROP>
DEV void upd_finish_h2(const StepArgs& a, int p, int cb, int nch, bool acc, const UpdRegs<PMIX, 2>& g) {
  const int lane = threadIdx.x & 63;
  const int d = a.d, P = a.P;
  const long ldw = a.ldw ? a.ldw : d;
  double xa[2], xb[2], za[2], zb[2];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    xa[c] = g.x0[c]; xb[c] = g.x1[c]; za[c] = g.z0[c]; zb[c] = g.z1[c];
  }
  if (acc) {
    // both chunks' accepted Xi and W in flight before either is converted
    Raw2<PMIX> cw[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) raw_load(cw[c], a.xi_cur, a.w_cur, a.wlo_cur, g.ii[c] + (long)p * ldw);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      double c0, c1, wc0, wc1;
      raw_xi(cw[c], c0, c1);
      raw_w(cw[c], wc0, wc1);
      xa[c] = propose1(g.r0[c], xa[c], a.rho, c0);
      xb[c] = propose1(g.r1[c], xb[c], a.rho, c1);
      za[c] = __fma_rn(a.c, wc0, a.rho * za[c]);
      zb[c] = __fma_rn(a.c, wc1, a.rho * zb[c]);
      const long e = g.ii[c] + (long)p * d;
      *(double2*)(a.X + e) = make_double2(xa[c], xb[c]);
      *(double2*)(a.Z + e) = make_double2(za[c], zb[c]);
    }
  }
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int ch = cb * 2 + c;
    const int i = g.ii[c];
    const long e = i + (long)p * d;
    const double ra = g.r0[c], rb = g.r1[c];
    store_win2<PMIX>(a.win, i + (a.win_col0 + p) * (long)d, xa[c] - ra, xb[c] - rb);
    double pacc[MAXPROJ] = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < a.nproj; ++k) {
      const double2 pv = *(const double2*)(a.proj + i + (long)k * d);
      pacc[k] = __fma_rn(pv.y, xb[c], __fma_rn(pv.x, xa[c], pacc[k]));
    }
    if (PROP) {
      double n0, n1, wn0, wn1;
      raw_xi(g.nw[c], n0, n1);
      raw_w(g.nw[c], wn0, wn1);
      const double xp0 = propose1(ra, xa[c], a.rho, n0), xp1 = propose1(rb, xb[c], a.rho, n1);
      u16 h0, l0, h1, l1;
      const double s0 = (xp0 - g.m0[c]) * (double)g.sv[c].x, s1 = (xp1 - g.m1[c]) * (double)g.sv[c].y;
      if (fmax(fabs(s0), fabs(s1)) >= H2_RANGE) atomicOr(a.err, 2);
      split_f16(s0, h0, l0);
      split_f16(s1, h1, l1);
      *(uint32_t*)(a.vh + e) = (uint32_t)h0 | ((uint32_t)h1 << 16);
      *(uint32_t*)(a.vh + (long)d * P + e) = (uint32_t)l0 | ((uint32_t)l1 << 16);
      const double zp0 = __fma_rn(a.c, wn0, a.rho * za[c]), zp1 = __fma_rn(a.c, wn1, a.rho * zb[c]);
      double zacc = __fma_rn(zp1, zp1, __fma_rn(zp0, zp0, 0.0));
      double xacc = __fma_rn(xp1, xp1, __fma_rn(xp0, xp0, 0.0));
      zacc = wave_sum_f64(zacc);
      if (lane == 0) a.zq_part_nxt[(long)p * nch + ch] = zacc;
      if (a.prior_w > 0.0) {
        xacc = wave_sum_f64(xacc);
        if (lane == 0) a.pq_part_nxt[(long)p * nch + ch] = xacc;
      }
    }
    if (a.nproj > 0) {
      for (int k = 0; k < a.nproj; ++k) {
        const double v = wave_sum_f64(pacc[k]);
        if (lane == 0) a.proj_part[((long)ch * a.nproj + k) * P + p] = v;
      }
    }
  }
}

// One step of the mixed form with the half target's reduction folded in:
// workgroup p (d / 256 wavefronts) issues its update loads, reduces the
// K-split partial products of its rows into the row-block terms of log pi
// (stored to part as the separate reduction does, and kept in LDS), then
// every wavefront takes the chain's decision from the LDS terms (bitwise the
// sums of the separate path) and updates its two 128-row chunks; wavefront 0
// writes the decision's outputs.
template <bool PROP>
__global__ __launch_bounds__(1024) void k_step_h2(StepArgs a, int nch, const float* __restrict__ Yp,
                                                  const double* __restrict__ rsc, double* __restrict__ part,
                                                  const double* __restrict__ twist) {
  __shared__ double lpp[64];
  const int p = blockIdx.x, v = threadIdx.x >> 6, lane = threadIdx.x & 63;
  UpdRegs<PMIX, 2> g;
  upd_load_h2<PROP>(a, p, v, g);
  const DecIn din = decide_inputs(a, nch, p, v == 0);
  const double q = h2_reduce_wave(Yp, rsc, a.d, a.P, a.nrb, part, twist, p, v);
  if ((lane & 15) == 0) lpp[v * 4 + (lane >> 4)] = q;
  __syncthreads();
  const bool acc = decide_wave(a, p, v == 0, lane_part(a, lpp), din);
  upd_finish_h2<PROP>(a, p, v, nch, acc, g);
}

// STEP_CPW chunks per wavefront and 8 / STEP_CPW waves per SIMD: the
// P * d / (128 STEP_CPW) wavefronts of a step at P = 256, d = 4096 fit the
// chip in one round (the argument block alone would hold it below that)
template <int PR, int MODE>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8 / STEP_CPW))) void k_step(StepArgs a, int nch) {
  if (MODE == 2 && (a.d & 1) == 0) step_update2<PR, STEP_CPW>(a, blockIdx.x, nch, blockIdx.y);
  else step_body<PR, MODE>(a, blockIdx.x, nch, blockIdx.y);
}

// A step that takes its decision and proposes the next one, for the sizes
// where latency bounds it: one chunk per wavefront, and every load that either
// verdict may need in flight before the first wait, instead of a wait for the
// state's loads, one for the decision's and one for the accepted proposal's.
// d = 1024, P = 64: 5.7 -> 3.9 us (FP64), 5.6 -> 4.2 (FP32); d = 750, P = 50,
// mixed: 5.7 -> 3.9.
template <int PR>
__global__ __launch_bounds__(256) void k_step_run(StepArgs a, int nch) {
  // a word from each line of the arguments, so that the lines arrive together
  asm volatile("" ::"s"(a.d), "s"(a.nrb), "s"(a.nproj), "s"(a.v32), "s"(a.ldw));
  const int lane = threadIdx.x & 63;
  const int p = blockIdx.y * 4 + (threadIdx.x >> 6), cb = blockIdx.x;
  if (p >= a.P) return;
  UpdRegs<PR, 1> g;
  upd_load_run<PR, 1>(a, p, cb, nch, g);
  // lanes without a row block or chunk read the chain's first; of a row
  // block's partials those that it lacks are replaced by its first
  const double* parts = chain_parts(a, p);
  const int q = lane < a.nrb ? lane : 0, sub = a.sub > 1 ? a.sub : 1;
  const bool two = 64 * q + 32 < a.d;
  const int have = sub > 1 && !two ? sub / 2 : sub;
  double f[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) f[k] = parts[sub * q + (k < have ? k : 0)];
  const double zs = a.zq_part_cur[(long)p * nch + (lane < nch ? lane : 0)];
  DecIn din;
  din.lp = a.lp_cur[p];
  din.zq = a.zq_cur[p];
  din.u = a.u[p];
  const int* wacc = a.wacc ? a.wacc : a.nacc;
  din.nacc = din.wacc = 0;
  if (cb == 0) {
    din.nacc = a.nacc[p];
    din.wacc = wacc[p];
  }
  din.pq = 0.0;
  if (a.prior_w > 0.0 && lane < nch) din.pq = 0.0 + a.pq_part_cur[(long)p * nch + lane];
  din.zs = lane < nch ? 0.0 + zs : 0.0;
  const double part = sub == 1 ? f[0] : sub == 2 ? f[0] + (two ? f[1] : 0.0) : (f[0] + f[1]) + (two ? f[2] + f[3] : 0.0);
  const bool acc = decide_wave(a, p, cb == 0, lane < a.nrb ? 0.0 + part : 0.0, din);
  upd_finish<PR, 1, true>(a, p, cb, nch, acc, g);
}

// A step with an accept half runs as a decision launch (one wave per chain)
// followed by the streaming update; the first proposal of a call has no
// decision.
hipError_t step(const StepArgs& a, hipStream_t s) {
  const int nch = step_chunks(a.d);
  const dim3 gupd((a.d & 1) == 0 ? cdiv(nch, STEP_CPW) : nch, cdiv(a.P, 4));
  // the decision moves into the update launch where one wavefront can take it
  StepArgs b = a;
  b.fuse_dec = a.do_accept && !a.da && a.nrb <= 64 && nch <= 64 && (a.d & 1) == 0;
  // up to 4096 wavefronts; beyond, reading both proposals whatever the verdict
  // costs more than the waits.  k_step_run against k_step, us: P nch = 2048
  // 7.0 / 8.2 FP64, 4.8 / 6.9 FP32; 4096 9.8 / 10.4, 8.3 / 9.9; 8192
  // 16.7 / 15.4, 13.6 / 13.0.
  if (b.fuse_dec && a.do_propose && !a.vh && (long)a.P * nch <= 4096) {
    const dim3 grun(nch, cdiv(a.P, 4));
    if (a.prec == P64) hipLaunchKernelGGL((k_step_run<P64>), grun, dim3(256), 0, s, b, nch);
    else if (a.prec == P32) hipLaunchKernelGGL((k_step_run<P32>), grun, dim3(256), 0, s, b, nch);
    else hipLaunchKernelGGL((k_step_run<PMIX>), grun, dim3(256), 0, s, b, nch);
    return hipGetLastError();
  }
  if (a.do_accept && !b.fuse_dec) hipLaunchKernelGGL(k_decide, dim3(a.P), dim3(256), 0, s, b, nch);
  if (a.prec == P64) hipLaunchKernelGGL((k_step<P64, 2>), gupd, dim3(256), 0, s, b, nch);
  else if (a.prec == P32) hipLaunchKernelGGL((k_step<P32, 2>), gupd, dim3(256), 0, s, b, nch);
  else hipLaunchKernelGGL((k_step<PMIX, 2>), gupd, dim3(256), 0, s, b, nch);
  return hipGetLastError();
}

bool step_h2_ok(int d, int P, int nrb) {
  return d % 256 == 0 && d <= 4096 && nrb == d / 64 && step_chunks(d) <= 64 && tgt_h2_ok(d, P);
}

hipError_t step_h2(const StepArgs& a, const float* Yp, const double* rsc, double* part, const double* twist,
                   hipStream_t s) {
  if (a.prec != PMIX || !a.vh || !a.mu || !a.vsc || !a.do_accept || a.da || !step_h2_ok(a.d, a.P, a.nrb))
    return hipErrorInvalidValue;
  StepArgs b = a;
  b.fuse_dec = 1;
  if (a.do_propose)
    hipLaunchKernelGGL(k_step_h2<true>, dim3(a.P), dim3(64 * (a.d / 256)), 0, s, b, step_chunks(a.d), Yp, rsc, part,
                       twist);
  else
    hipLaunchKernelGGL(k_step_h2<false>, dim3(a.P), dim3(64 * (a.d / 256)), 0, s, b, step_chunks(a.d), Yp, rsc,
                       part, twist);
  return hipGetLastError();
}

// ---- the steps of a call with the target matrix in registers --------------------
// Between merges the chains do not meet, so one workgroup runs all n steps of
// one chain.  Waves 1 .. KS hold R in registers (wave q columns (q - 1) KPT ..
// of all rows, lane l rows l, l + 64, ..), wave 0 the chain's state; a step is
// two barriers: wave 0 proposes and writes x' - mu to LDS, the others form
// their columns' part of y = R (x' - mu), wave 0 adds the parts, sums the
// squares, decides and proposes again.  The steps' search directions and
// normals are loaded RES_PF steps ahead (more spills at d = 192), log u for 64
// steps at a time and the traced projections are formed by the other waves
// while wave 0 decides.  Bound by that chain: LDS round trip, KPT dependent
// products, LDS round trip, the wave sum.  One launch replaces 2 or 3 per step,
// whose dispatch and round trips cost 9 to 13 us a step at d <= 128 whatever
// the work; the loop takes 0.55, 0.82 and 1.13 us a step at d = 32, 100 and
// 192 (one chain per CU).
constexpr int RES_PF = 2;

template <int RPT, int KS, int KPT>
__global__ __launch_bounds__(64 * (KS + 1)) void k_steps_resident(ResidentArgs a) {
  constexpr int DR = 64 * RPT;
  static_assert(KS * KPT >= DR && KPT % 2 == 0, "every column has a wave");
  __shared__ __attribute__((aligned(16))) double vs[KS * KPT];
  __shared__ double ys[KS][DR], xs[2][DR], lu[2][64], pj[MAXPROJ][DR];
  const int lane = threadIdx.x & 63, q = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int p = blockIdx.x, d = a.d, P = a.P, n = a.n;
  const long dP = (long)d * P;
  const int nproj = a.trace ? a.nfun - 1 : 0;
  for (int e = threadIdx.x; e < nproj * DR; e += 64 * (KS + 1))
    pj[e / DR][e % DR] = e % DR < d ? a.proj[(long)(e / DR) * d + e % DR] : 0.0;
  for (int e = threadIdx.x; e < KS * KPT; e += 64 * (KS + 1)) vs[e] = 0.0;  // columns past d
  if (q != 0) {
    double rk[RPT][KPT];
#pragma unroll
    for (int j = 0; j < KPT; ++j) {
      const int k = (q - 1) * KPT + j;
      const double* col = a.R + (k < d ? k : d - 1);
#pragma unroll
      for (int r = 0; r < RPT; ++r) {
        const int i = lane + 64 * r;
        const double v = col[(unsigned)((i < d ? i : d - 1) * d)];
        rk[r][j] = (i < d && k < d) ? v : 0.0;
      }
    }
    auto log_uniforms = [&](int t0) {
      if (t0 + lane < n) lu[(t0 >> 6) & 1][lane] = log(a.u[(long)(t0 + lane) * P + p]);
    };
    // projections of the state after step t (xs[t & 1] is written again two
    // decisions later)
    auto project = [&](int t) {
      for (int k = q - 1; k < nproj; k += KS) {
        double s = 0.0;
#pragma unroll
        for (int r = 0; r < RPT; ++r) s = __fma_rn(pj[k][lane + 64 * r], xs[t & 1][lane + 64 * r], s);
        s = wave_sum_f64(s);
        if (lane == 0) a.trace[((long)t * a.nfun + 1 + k) * P + p] = s;
      }
    };
    if (q == 1) log_uniforms(0);
    __syncthreads();  // vs cleared, pj and lu written
    for (int t = 0; t < n; ++t) {
      if (q == 1 && (t & 63) == 32) log_uniforms((t & ~63) + 64);
      __syncthreads();  // x' - mu
      double y0[RPT], y1[RPT];
#pragma unroll
      for (int r = 0; r < RPT; ++r) y0[r] = y1[r] = 0.0;
#pragma unroll
      for (int j = 0; j < KPT; j += 2) {
        const double2 v = *(const double2*)&vs[(q - 1) * KPT + j];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          y0[r] = __fma_rn(rk[r][j], v.x, y0[r]);
          y1[r] = __fma_rn(rk[r][j + 1], v.y, y1[r]);
        }
      }
#pragma unroll
      for (int r = 0; r < RPT; ++r) ys[q - 1][lane + 64 * r] = y0[r] + y1[r];
      __syncthreads();  // parts of y
      if (t > 0) project(t - 1);
    }
    __syncthreads();  // the last state
    project(n - 1);
    return;
  }
  double x[RPT], z[RPT], xr[RPT], mu[RPT], tw[RPT];
  double fx[RES_PF][RPT], fw[RES_PF][RPT];
  bool in[RPT];
  const long e0 = (long)p * d + lane;
  auto fetch = [&](int t, double* bx, double* bw) {
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      bx[r] = bw[r] = 0.0;
      if (in[r] && t < n) {
        bx[r] = a.xi[t * dP + e0 + 64 * r];
        bw[r] = a.w[t * dP + e0 + 64 * r];
      }
    }
  };
#pragma unroll
  for (int r = 0; r < RPT; ++r) {
    const int i = lane + 64 * r;
    in[r] = i < d;
    x[r] = in[r] ? a.X[e0 + 64 * r] : 0.0;
    z[r] = in[r] ? a.Z[e0 + 64 * r] : 0.0;
    xr[r] = in[r] ? a.xr[i] : 0.0;
    mu[r] = in[r] ? a.mu[i] : 0.0;
    tw[r] = (a.twist && (i & 1) && in[r]) ? a.twist[i] : 0.0;
  }
  double lp = a.lp[p], zq = a.zq[p];
  int nacc = 0;
#pragma unroll
  for (int b = 0; b < RES_PF; ++b) fetch(b, fx[b], fw[b]);
  __syncthreads();  // vs cleared, pj and lu written
  auto step = [&](int t, double* bx, double* bw) {
    double xp[RPT], zp[RPT], zacc = 0.0;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      xp[r] = propose1(xr[r], x[r], a.rho, bx[r]);
      zp[r] = __fma_rn(a.c, bw[r], a.rho * z[r]);
      if (in[r]) vs[lane + 64 * r] = xp[r] - mu[r];
    }
    __syncthreads();  // x' - mu
    fetch(t + RES_PF, bx, bw);
#pragma unroll
    for (int r = 0; r < RPT; ++r) zacc = __fma_rn(zp[r], zp[r], zacc);
    const double zs = wave_sum_f64(zacc);
    const double logu = lu[(t >> 6) & 1][t & 63];
    __syncthreads();  // parts of y
    double s = 0.0;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      double v = ys[0][lane + 64 * r];
#pragma unroll
      for (int g = 1; g < KS; ++g) v += ys[g][lane + 64 * r];
      if (a.twist) {
        const double e = lane_xor_f64<1>(v);  // row 2k of a twisted row 2k + 1
        if (lane & 1) v = __fma_rn(tw[r], e * e, v);
      }
      s = in[r] ? __fma_rn(v, v, s) : s;  // not 0 x infinity of the rows past d
    }
    const double lpp = -0.5 * wave_sum_f64(s);
    const double la = (lpp + zs * a.inv2a2) - (lp + zq * a.inv2a2);
    const bool acc = logu < la;  // NaN compares false: rejected
    if (acc) {
      lp = lpp;
      zq = zs;
      ++nacc;
    }
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      x[r] = acc ? xp[r] : x[r];
      z[r] = acc ? zp[r] : z[r];
      if (in[r]) a.win[t * dP + e0 + 64 * r] = x[r] - xr[r];
      if (nproj) xs[t & 1][lane + 64 * r] = x[r];
    }
    if (lane == 0) {
      a.la[(long)t * P + p] = la;
      a.acc[(long)t * P + p] = acc ? 1 : 0;
      if (a.trace) a.trace[(long)t * a.nfun * P + p] = lp;
      if (isinf(lpp) && lpp > 0.0) atomicOr(a.err, 1);
    }
  };
  for (int t = 0; t < n; t += RES_PF) {
#pragma unroll
    for (int b = 0; b < RES_PF; ++b)
      if (t + b < n) step(t + b, fx[b], fw[b]);
  }
  __syncthreads();  // the last state
#pragma unroll
  for (int r = 0; r < RPT; ++r)
    if (in[r]) {
      a.X[e0 + 64 * r] = x[r];
      a.Z[e0 + 64 * r] = z[r];
    }
  if (lane == 0) {
    a.lp_out[p] = lp;
    a.zq_out[p] = zq;
    a.nacc[p] += nacc;
    if (a.wacc) a.wacc[p] += nacc;
  }
}

// Above d = 192 the columns pass a lane's 256 registers.  Every chain's CU reads
// R anew, so a call of many chains begins with P / 256 rounds of that, which
// its steps have to earn back; long calls of very many chains lose to the tiled
// target in the end.  us a call of n steps, launches per step / this loop:
//   d     P      n = 1     n = 4      n = 8      n = 16     n = 64
//   64    64     20 / 15   42 / 16    75 / 18    129 / 23   478 / 50
//   64    4096   23 / 48   63 / 68    107 / 86   198 / 124  802 / 362
//   64    16384  48 / 165  148 / 212  274 / 277  578 / 496
//   64    65536  138 / 601 512 / 890  995 / 1277
//   128   64     22 / 20   46 / 23    77 / 27    140 / 34   516 / 78
//   128   256    21 / 28   44 / 32    79 / 37    145 / 48   535 / 106
//   128   1024   21 / 72   53 / 85    97 / 103   174 / 126  649 / 255
//   128   8192   44 / 509  140 / 553  264 / 614  530 / 770
//   192   64     23 / 32   48 / 36    79 / 40    143 / 51   533 / 115
//   192   256    23 / 52   51 / 58    86 / 67    157 / 82   561 / 157
//   192   1024   26 / 173  69 / 196   120 / 224  215 / 271  832 / 569
// Up to 64 chains the loop runs whatever the length, so that a window's bits do
// not depend on how it is cut into calls; beyond, from the length on at which
// it is ahead.
bool steps_resident_ok(int d, int P, int n) {
  const long per_step = d <= 64 ? 700 : d <= 128 ? 100 : 40;  // chains that one step earns back
  return (d <= 64 || (d <= 128 && P <= 8192) || (d <= 192 && P <= 1024)) && (P <= 64 || n * per_step >= P);
}

hipError_t steps_resident(const ResidentArgs& a, hipStream_t s) {
  if (a.d < 1 || !steps_resident_ok(a.d, a.P, a.n) || a.P < 1 || a.n < 1 || a.nfun - 1 > MAXPROJ)
    return hipErrorInvalidValue;
  if (a.d <= 64) hipLaunchKernelGGL((k_steps_resident<1, 3, 22>), dim3(a.P), dim3(256), 0, s, a);
  else if (a.d <= 128) hipLaunchKernelGGL((k_steps_resident<2, 7, 20>), dim3(a.P), dim3(512), 0, s, a);
  else hipLaunchKernelGGL((k_steps_resident<3, 7, 28>), dim3(a.P), dim3(512), 0, s, a);
  return hipGetLastError();
}

DEV void init_eval_elem(int v64, const double* __restrict__ X, const double* __restrict__ mu, void* __restrict__ V,
                        double* __restrict__ Z, int d, long e) {
  const double x = X[e];
  const double v = x - (mu ? mu[e % d] : 0.0);
  if (v64) ((double*)V)[e] = v;
  else ((float*)V)[e] = (float)v;
  Z[e] = x;
}

__global__ __launch_bounds__(256) void k_init_eval(int v64, const double* __restrict__ X, const double* __restrict__ mu,
                                                   void* __restrict__ V, double* __restrict__ Z, int d, long n) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e < n) init_eval_elem(v64, X, mu, V, Z, d, e);
}

hipError_t init_eval(int v64, const double* X, const double* mu, void* V, double* Z, int d, int P, hipStream_t s) {
  const long n = (long)d * P;
  hipLaunchKernelGGL(k_init_eval, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, v64, X, mu, V, Z, d, n);
  return hipGetLastError();
}

// lp[p] = sum_rb part[rb][p] - prior_w |x_p|^2 (one block per chain)
DEV void init_finish_block(const double* __restrict__ part, int nrb, int P, const double* __restrict__ X, int d,
                           double prior_w, double* __restrict__ lp, int p) {
  __shared__ double red[2][256];
  double s = 0.0, q = 0.0;
  for (int k = threadIdx.x; k < nrb; k += 256) s += part[(long)p * nrb + k];
  if (prior_w > 0.0)
    for (int i = threadIdx.x; i < d; i += 256) {
      const double x = X[i + (long)p * d];
      q = __fma_rn(x, x, q);
    }
  red[0][threadIdx.x] = s;
  red[1][threadIdx.x] = q;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      red[0][threadIdx.x] += red[0][threadIdx.x + o];
      red[1][threadIdx.x] += red[1][threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) lp[p] = (prior_w > 0.0) ? __fma_rn(-prior_w, red[1][0], red[0][0]) : red[0][0];
}

__global__ __launch_bounds__(256) void k_init_finish(const double* __restrict__ part, int nrb, int P,
                                                     const double* __restrict__ X, int d, double prior_w,
                                                     double* __restrict__ lp) {
  init_finish_block(part, nrb, P, X, d, prior_w, lp, blockIdx.x);
}

hipError_t init_finish(const double* part, int nrb, const double* Z, const double* X, double prior_w, double* lp,
                       double* zq, int d, int P, hipStream_t s) {
  hipLaunchKernelGGL(k_init_finish, dim3(P), dim3(256), 0, s, part, nrb, P, X, d, prior_w, lp);
  hipLaunchKernelGGL(k_colnorm, dim3(P), dim3(256), 0, s, Z, d, zq);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_proj_reduce(const double* __restrict__ proj_part, int n, int nch, int nproj,
                                                     int P, double* __restrict__ trace, int nfun) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long)n * nproj * P) return;
  const int p = (int)(e % P);
  const int k = (int)((e / P) % nproj);
  const long t = e / ((long)P * nproj);
  double s = 0.0;
  for (int c = 0; c < nch; ++c) s += proj_part[((t * nch + c) * nproj + k) * P + p];
  trace[(t * nfun + 1 + k) * P + p] = s;
}

hipError_t proj_reduce(const double* proj_part, int n, int nch, int nproj, int P, double* trace, int nfun,
                       hipStream_t s) {
  const long total = (long)n * nproj * P;
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_proj_reduce, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, proj_part, n, nch, nproj, P,
                     trace, nfun);
  return hipGetLastError();
}

// ============================================================================
// Batched form: G independent Gaussian problems of uneven d with P chains
// each (FP32 path, FP64 state and Cholesky).  Every launch below serves all
// problems at once: a host-built tile list maps blockIdx.x to (problem, tile),
// and the tile runs the same body as the single-problem kernel, so results
// are bitwise those of separate runs with the same tile shapes.
// ============================================================================
__global__ __launch_bounds__(256) void gk_normals(uint32_t k0, uint32_t k1, const long* __restrict__ win,
                                                  long per_window, long total, float* __restrict__ W) {
  const long g0 = *win * per_window;
  const long stride = (long)gridDim.x * 256;
  const bool vec = (uintptr_t)W % 16 == 0;
  for (long q = (long)blockIdx.x * 256 + threadIdx.x; 4 * q < total; q += stride) {
    float v[4];
    normals4_f32(k0, k1, (uint64_t)(g0 + 4 * q), v);
    if (vec && 4 * q + 3 < total) {
      *(float4*)(W + 4 * q) = make_float4(v[0], v[1], v[2], v[3]);
      continue;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (4 * q + e < total) W[4 * q + e] = v[e];
  }
}

// U[e], e = (g n + t) P + p: Philox stream 1, counter (window, problem-step, p/2)
__global__ __launch_bounds__(256) void gk_uniforms(uint32_t k0, uint32_t k1, const long* __restrict__ win, long total,
                                                   int P, double* __restrict__ U) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= total) return;
  const int p = (int)(e % P);
  const long gt = e / P;
  const uint64_t w = (uint64_t)*win;
  const u4_t r = philox4x32_10({(uint32_t)w, (uint32_t)gt, 1u, (uint32_t)(p >> 1)}, k0, k1);
  U[e] = (p & 1) ? u01_f64(r.z, r.w) : u01_f64(r.x, r.y);
}

__global__ void gk_bump(long* win, double* N, double K) {
  if (threadIdx.x == 0) {
    *win += 1;
    *N += K;
  }
}

template <int BM, int KG>
__global__ __launch_bounds__(256 * KG) void gk_tgt(const BProb* __restrict__ pr, const BTile* __restrict__ tl, int P) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  tgt_gauss_tile<float, 32, BM, 32, KG>(b.Rp, b.Vp, b.ld, P, t.a, t.b, b.lpp_part, b.nrb);
}

// Shapes 64 x 2 and 32 x 4 on the direct-to-LDS engine, 64-row tiles for both
// (the latter writes two 32-row partials), bitwise the tiles above.  Four
// wavefronts take the k-groups one after the other where the tiles above have
// four wavefronts each, so a tile takes longer and more of them run per CU;
// g_tgt_engine chooses.  The 271 MB of R of the 48 problems do not fit the 256
// MB Infinity Cache, so R streams from HBM every step: 93 us in either shape as
// the lists stood, 81 and 77 us with the largest problems first, 67 us (4.0
// TB/s) with the engine too.
template <int WGM, int WGN, int SETS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gk_tgt_t(const BProb* __restrict__ pr,
                                                                                      const BTile* __restrict__ tl,
                                                                                      int P) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  tgt_tile_t<float, 64, 32, WGM, WGN, 6, SETS>(b.Rp, b.Vp, b.ld, P, t.a, t.b, b.lpp_part, b.nrb);
}

// Which kernel serves shapes 64 x 2 and 32 x 4, by the number n of 64 x 32 tiles
// of the problem set; a tile at an edge takes 1.5 (rows) to 2 times (chains) as
// long in the tile kernel, no longer on the engine.  us, tile kernel / engine:
//   d; P                    n      64 x 2         32 x 4
//   1024; 32                16     15.1 / 21.0    9.2 / 18.6
//   3072; 32                48     41.1 / 59.0    25.0 / 51.1
//   8 of 1024; 32           128    15.7 / 21.1    11.3 / 19.4
//   64 of 256; 32           256    6.0 / 7.3      7.0 / 6.8
//   8 of 2048; 32           256    30.7 / 40.7    31.0 / 36.6
//   16 of 2048; 32          512    51.6 / 56.5    58.5 / 54.4
//   64 of 1024; 32          1024   52.6 / 61.4    62.1 / 59.0
//   256 of 64; 32           256    3.3 / 3.6      5.0 / 3.5
//   2048, 65, 33; 32        35     27.9 / 40.0    17.5 / 34.6
//   2000, 2048; 32          64     37.3 / 39.2    29.5 / 35.4
//   8 of 1000; 32           128    22.9 / 22.0    13.3 / 20.2
//   32 of 1000; 32          512    40.8 / 33.4    40.6 / 32.4
//   48, 64 .. 1091; 32      310    24.4 / 26.8    18.9 / 25.1
//   48, 64 .. 2708; 32      579    64.0 / 61.5    52.2 / 57.2
//   8, 64 .. 1038; 24       64     27.1 / 22.2    17.6 / 19.8
//   32, 64 .. 1134; 24      215    32.2 / 24.3    23.6 / 22.3
//   48, 64 .. 3039; 16      656    103 / 69.8     93.2 / 64.8
//   8 of 1024; 20           128    28.1 / 20.9    18.4 / 19.3
// 64 x 2: the tile kernel where no chain tile has an edge and no problem within
// a tenth of the largest has one, up to 1.5 tiles a CU, and without any edge at
// all sizes.  32 x 4: its four k-groups pay where the chip is not full.
bool g_tgt_engine(int cfg, const int* dims, int G, int P) {
  if (cfg != 2 && cfg != 4) return false;
  long n = 0;
  int dmax = 0;
  for (int g = 0; g < G; ++g) {
    n += (long)cdiv(dims[g], 64) * cdiv(P, 32);
    dmax = max(dmax, dims[g]);
  }
  if (cfg == 4) return dmax <= 128 || n > (P % 32 == 0 ? 384 : 192);
  if (P % 32 != 0) return true;
  bool edge = false, large_edge = false;
  for (int g = 0; g < G; ++g)
    if (dims[g] % 64 != 0) {
      edge = true;
      large_edge |= 10L * dims[g] > 9L * dmax;
    }
  return large_edge || (edge && n > 384);
}

hipError_t g_tgt(int cfg, bool engine, const BProb* pr, const BTile* tl, int ntiles, int P, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  if (engine) {
    if (cfg == 2) hipLaunchKernelGGL((gk_tgt_t<2, 2, 2>), dim3(ntiles), dim3(256), 0, s, pr, tl, P);
    else if (cfg == 4) hipLaunchKernelGGL((gk_tgt_t<4, 1, 4>), dim3(ntiles), dim3(256), 0, s, pr, tl, P);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  switch (cfg) {
    case 0: hipLaunchKernelGGL((gk_tgt<32, 2>), dim3(ntiles), dim3(512), 0, s, pr, tl, P); break;
    case 1: hipLaunchKernelGGL((gk_tgt<64, 1>), dim3(ntiles), dim3(256), 0, s, pr, tl, P); break;
    case 2: hipLaunchKernelGGL((gk_tgt<64, 2>), dim3(ntiles), dim3(512), 0, s, pr, tl, P); break;
    case 3: hipLaunchKernelGGL((gk_tgt<128, 2>), dim3(ntiles), dim3(512), 0, s, pr, tl, P); break;
    default: hipLaunchKernelGGL((gk_tgt<32, 4>), dim3(ntiles), dim3(1024), 0, s, pr, tl, P); break;
  }
  return hipGetLastError();
}
int g_tgt_rows(int cfg, bool engine) { return engine ? 64 : g_tgt_bm(cfg); }
int g_tgt_bm(int cfg) {
  static const int bm[G_TGT_CONFIGS] = {32, 64, 64, 128, 32};
  return bm[cfg];
}

// Step arguments of problem b for step st.t (accept step t, propose step
// t + 1; t = -1: the first proposal only).
DEV StepArgs g_step_args(const BProb& b, const BStep& st, int g) {
  const int P = st.P, d = b.d, cu = st.t & 1, nx = cu ^ 1;
  const long dP = (long)b.ld * P;  // one step's slice of W and Xi (padded rows)
  StepArgs a{};
  a.d = d;
  a.P = P;
  a.prec = P32;
  a.rho = st.rho;
  a.c = st.c;
  a.inv2a2 = st.inv2a2;
  a.xr = b.xr;
  a.mu = b.mu;
  a.X = b.X;
  a.Z = b.Z;
  a.V = b.Vp;
  a.ldv = b.ld;
  a.ldw = b.ld;
  a.nrb = b.nrb;
  a.lpp_part = b.lpp_part;
  a.nacc = b.nacc;
  a.win = b.win;
  a.ldwin = b.ld;
  a.err = st.err;
  if (st.t >= 0) {
    a.do_accept = 1;
    a.xi_cur = b.Xi + st.t * dP;
    a.w_cur = b.W + st.t * dP;
    a.wlo_cur = nullptr;
    a.zq_part_cur = b.zq_part + (long)cu * b.nch * P;
    a.lp_cur = b.lp + (long)cu * P;
    a.zq_cur = b.zq + (long)cu * P;
    a.lp_nxt = b.lp + (long)nx * P;
    a.zq_nxt = b.zq + (long)nx * P;
    a.u = st.U + ((long)g * st.n + st.t) * P;
    a.la_out = b.la + (long)st.t * P;
    a.acc_out = b.acc + (long)st.t * P;
    a.win_col0 = (long)st.t * P;
  }
  const int tn = st.t + 1;
  if (tn < st.n) {
    // the proposal of step tn is judged with the scalars of parity tn & 1
    a.do_propose = 1;
    a.xi_nxt = b.Xi + tn * dP;
    a.w_nxt = b.W + tn * dP;
    a.wlo_nxt = nullptr;
    a.zq_part_nxt = b.zq_part + (long)(tn & 1) * b.nch * P;
  }
  return a;
}

template <int MODE>
__global__ __launch_bounds__(256) void gk_step(const BProb* __restrict__ pr, const BTile* __restrict__ tl, BStep st) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  const StepArgs a = g_step_args(b, st, t.g);
  if (MODE == 1) decide_block(a, b.nch, t.b);
  else if ((b.d & 1) == 0) step_update2<P32>(a, t.a, b.nch, t.b);
  else step_body<P32, 2>(a, t.a, b.nch, t.b);
}

// decision launch over (problem, 0, chain) tiles (a workgroup per chain),
// then the update over (problem, chunk, chain quad) tiles; the first
// proposal has no decision
hipError_t g_step(const BProb* pr, const BTile* dec_tl, int ndec, const BTile* tl, int ntiles, const BStep& st,
                  hipStream_t s) {
  if (st.t >= 0) hipLaunchKernelGGL((gk_step<1>), dim3(ndec), dim3(256), 0, s, pr, dec_tl, st);
  hipLaunchKernelGGL((gk_step<2>), dim3(ntiles), dim3(256), 0, s, pr, tl, st);
  return hipGetLastError();
}

// The n_lag steps of a window for every problem in one launch (see PItem).
// Items are taken in queue order, so every item an item waits for was taken
// earlier by a running workgroup: the earliest unfinished item can always
// proceed, whatever the grid size.  A wait is bounded: after spin_max polls it
// sets bit 1 of the error word, and every workgroup then stops taking items.
// Thread 0 publishes a finished item (agent-scope release, after the
// workgroup barrier that ends the item) when it takes the next one; a waiter
// polls relaxed and then fences with an agent-scope acquire.  Every loop exit
// tests a value read back as wavefront-uniform, so all wavefronts leave (and
// pass every barrier) together.  The bodies are those of gk_tgt (64 x 2
// tiles), decide_wave (bitwise decide_block at these sizes: at most 64 row
// blocks and 64 chunks) and the update half of gk_step, so results are
// bitwise those of the per-phase launches with the default tile shape.
__global__ __launch_bounds__(PERSIST_THREADS) void gk_persist(const BProb* __restrict__ pr,
                                                              const PItem* __restrict__ items, int nitems, BStep st,
                                                              PCtl c) {
  __shared__ int s_q, s_ok;
  const int total = nitems * st.n;
  int prev_g = -1;  // problem of the item finished in the previous pass (thread 0 publishes it)
  for (;;) {
    if (threadIdx.x == 0) {
      if (prev_g >= 0) __hip_atomic_fetch_add(c.done + prev_g, 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
      int q = -1;
      if ((__hip_atomic_load(c.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 2) == 0)
        q = __hip_atomic_fetch_add(c.qctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_q = q;
    }
    __syncthreads();
    const int q = __builtin_amdgcn_readfirstlane(s_q);
    if (q < 0 || q >= total) break;
    const int t = q / nitems;
    const PItem it = items[q - t * nitems];
    if (threadIdx.x == 0) {
      const int need = t * c.per_step[it.g] + it.need;
      int ok = 1, spins = 0;
      while (__hip_atomic_load(c.done + it.g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < need) {
        if (++spins > c.spin_max || (__hip_atomic_load(c.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & 2)) {
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(2);
      }
      if (!ok) __hip_atomic_fetch_or(c.err, 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      s_ok = ok;
    }
    __syncthreads();
    if (__builtin_amdgcn_readfirstlane(s_ok) == 0) break;
    const int kind = __builtin_amdgcn_readfirstlane(it.kind), g = __builtin_amdgcn_readfirstlane(it.g);
    const BProb& b = pr[g];
    if (kind == 0) {
      tgt_gauss_tile<float, 32, 64, 32, 2>(b.Rp, b.Vp, b.ld, st.P, it.a, it.b, b.lpp_part, b.nrb);
    } else {
      BStep sp = st;
      sp.t = t;
      StepArgs a = g_step_args(b, sp, g);
      // the update items take the decision themselves where no decision item
      // was queued (the same predicate as the queue's construction)
      a.fuse_dec = kind == 2 && persist_fused_decision(b.d, b.nrb, b.nch) ? 1 : 0;
      const int w = threadIdx.x >> 6;
      if (kind == 1) {
        for (int p = w; p < st.P; p += PERSIST_THREADS / 64)
          decide_wave(a, b.nch, p, true, chain_parts(a, p));
      } else {
        // eight waves: chains 8k .. 8k + 7 per pass (the bodies take chain 4 pq + wave)
        for (int pq = 0; pq * 4 < st.P; pq += PERSIST_THREADS / 256) {
          if ((b.d & 1) == 0) step_update2<P32>(a, it.a, b.nch, pq);
          else step_body<P32, 2>(a, it.a, b.nch, pq);
        }
      }
    }
    // the item's stores, in every wavefront, complete (a workgroup barrier
    // alone does not wait for other wavefronts' stores) before thread 0
    // publishes the item with its agent-scope release
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    prev_g = g;
  }
}

hipError_t g_persist(const BProb* pr, const PItem* items, int nitems, const BStep& st, const PCtl& ctl, int grid,
                     hipStream_t s) {
  if (nitems <= 0 || st.n <= 0 || grid <= 0) return hipSuccess;
  hipLaunchKernelGGL(gk_persist, dim3(grid), dim3(PERSIST_THREADS), 0, s, pr, items, nitems, st, ctl);
  return hipGetLastError();
}

int g_persist_blocks_per_cu() {
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, gk_persist, PERSIST_THREADS, 0) != hipSuccess) return 1;
  return nb > 0 ? nb : 1;
}

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void gk_trigemm(const BProb* __restrict__ pr, const BTile* __restrict__ tl, int ncols,
                                                  double c) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  trigemm_tile_t<float, 64, 64, 3>(b.Lp, b.W, b.Xi, b.ld, ncols, c, t.a, t.b);
}

hipError_t g_trigemm(const BProb* pr, const BTile* tl, int ntiles, int ncols, double c, hipStream_t s) {
  hipLaunchKernelGGL(gk_trigemm, dim3(ntiles), dim3(256), 0, s, pr, tl, ncols, c);
  return hipGetLastError();
}

// window scatter (one K split) and row sums
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void gk_syrk(const BProb* __restrict__ pr, const BTile* __restrict__ tl, int K) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  __shared__ __attribute__((aligned(1024))) float lds[t_lds_elems<float, 64, 64, 3>()];
  syrk_tile_t<float, 64, 3>(b.win, b.ld, b.d, K, K, t.a, 0, b.G, lds);
}
__global__ __launch_bounds__(256) void gk_rowsum(const BProb* __restrict__ pr, const BTile* __restrict__ tl, int K) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  __shared__ double red[4][64];
  rowsum_block<float, true>(b.win, b.d, b.ld, K, K, t.a, 0, b.h, red);
}

hipError_t g_scatter(const BProb* pr, const BTile* syrk_tl, int nsyrk, const BTile* row_tl, int nrow, int K,
                     hipStream_t s) {
  hipLaunchKernelGGL(gk_syrk, dim3(nsyrk), dim3(256), 0, s, pr, syrk_tl, K);
  hipLaunchKernelGGL(gk_rowsum, dim3(nrow), dim3(256), 0, s, pr, row_tl, K);
  return hipGetLastError();
}

// Element-wise phases over per-problem index spaces: tile (g, block) covers
// elements [256 block, 256 block + 256) of problem g.
__global__ __launch_bounds__(256) void gk_fold(const BProb* __restrict__ pr, const BTile* __restrict__ dd_tl,
                                               const double* __restrict__ N, double K) {
  const BTile t = dd_tl[blockIdx.x];
  const BProb& b = pr[t.g];
  const long e = (long)t.a * 256 + threadIdx.x;
  const double n0 = *N;
  if (e < (long)b.d * b.d) fold_S_elem(b.G, b.h, b.xr, n0, K, b.S, b.d, e);
}
__global__ __launch_bounds__(256) void gk_fold_mean(const BProb* __restrict__ pr, const BTile* __restrict__ d_tl,
                                                    const double* __restrict__ N, double K) {
  const BTile t = d_tl[blockIdx.x];
  const BProb& b = pr[t.g];
  const int i = t.a * 256 + threadIdx.x;
  if (i < b.d) fold_mean_elem(b.h, b.xr, *N, K, b.m, i);
}

hipError_t g_fold(const BProb* pr, const BTile* dd_tl, int ndd, const BTile* d_tl, int nd, const double* N, double K,
                  hipStream_t s) {
  hipLaunchKernelGGL(gk_fold, dim3(ndd), dim3(256), 0, s, pr, dd_tl, N, K);
  hipLaunchKernelGGL(gk_fold_mean, dim3(nd), dim3(256), 0, s, pr, d_tl, N, K);
  return hipGetLastError();
}

// covariance (no jitter) into C; clears the problem's Cholesky status
__global__ __launch_bounds__(256) void gk_cov(const BProb* __restrict__ pr, const BTile* __restrict__ dd_tl) {
  const BTile t = dd_tl[blockIdx.x];
  const BProb& b = pr[t.g];
  const long e = (long)t.a * 256 + threadIdx.x;
  if (e < (long)b.d * b.d) cov_elem(b.S, b.m, 0.0, b.C, b.d, e);
  if (t.a == 0 && threadIdx.x == 0) *b.info = 0;
}

hipError_t g_cov(const BProb* pr, const BTile* dd_tl, int ndd, hipStream_t s) {
  hipLaunchKernelGGL(gk_cov, dim3(ndd), dim3(256), 0, s, pr, dd_tl);
  return hipGetLastError();
}

// blocked Cholesky: every problem's first diagonal block, then per block column
// jb the panel and the update of the problems with more blocks
__global__ __launch_bounds__(CHOL_DIAG_THREADS) void gk_chol_diag(const BProb* __restrict__ pr,
                                                                  const BTile* __restrict__ tl) {
  const BProb& b = pr[tl[blockIdx.x].g];
  chol_diag_block(b.C, b.d, 0, min(CHOL_NB, b.d), b.Linv, b.info);
}
__global__ __launch_bounds__(256) void gk_chol_panel(const BProb* __restrict__ pr, const BTile* __restrict__ tl, int jb) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  const int j0 = jb * CHOL_NB, jn = min(CHOL_NB, b.d - j0);
  chol_panel_tile(b.C, b.d, j0, jn, b.Linv + (long)jb * CHOL_NB * CHOL_NB, t.a);
}
// tile t.a of the update after block column jb; tile 0 is the problem's next
// diagonal block, factored at once
__global__ __launch_bounds__(256) void gk_chol_update_diag(const BProb* __restrict__ pr,
                                                           const BTile* __restrict__ tl, int jb) {
  constexpr int NLDS = CHOL_UPD_LDS > CHOL_DIAG_LDS ? CHOL_UPD_LDS : CHOL_DIAG_LDS;
  __shared__ __attribute__((aligned(1024))) double lds[NLDS];
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  chol_update_core(b.C, b.d, jb, t.a, lds);
  if (t.a == 0) {
    __syncthreads();
    const int j1 = (jb + 1) * CHOL_NB;
    chol_diag_core(b.C, b.d, j1, min(CHOL_NB, b.d - j1), b.Linv + (long)(jb + 1) * CHOL_NB * CHOL_NB, b.info, lds);
  }
}

hipError_t g_chol_diag(const BProb* pr, const BTile* tl, int n, hipStream_t s) {
  hipLaunchKernelGGL(gk_chol_diag, dim3(n), dim3(CHOL_DIAG_THREADS), 0, s, pr, tl);
  return hipGetLastError();
}
hipError_t g_chol_step(const BProb* pr, const BTile* panel, int npanel, const BTile* upd, int nupd, int jb,
                       hipStream_t s) {
  if (npanel) hipLaunchKernelGGL(gk_chol_panel, dim3(npanel), dim3(256), 0, s, pr, panel, jb);
  if (nupd) hipLaunchKernelGGL(gk_chol_update_diag, dim3(nupd), dim3(256), 0, s, pr, upd, jb);
  return hipGetLastError();
}

// A factored problem (status 0) adopts C as its factor, rounded to FP32,
// and its merged mean as the pivot; a failed one keeps both.
__global__ __launch_bounds__(256) void gk_adopt(const BProb* __restrict__ pr, const BTile* __restrict__ dd_tl) {
  const BTile t = dd_tl[blockIdx.x];
  const BProb& b = pr[t.g];
  if (*b.info != 0) return;
  const long e = (long)t.a * 256 + threadIdx.x;
  if (e < (long)b.d * b.d) {
    b.L[e] = b.C[e];
    round_factor_elem(P32, b.L, b.Llow, b.d, e);
    b.Lp[(e % b.d) + (e / b.d) * b.ld] = b.Llow[e];
  }
  if (e < b.d) b.xr[e] = b.m[e];
}

hipError_t g_adopt(const BProb* pr, const BTile* dd_tl, int ndd, hipStream_t s) {
  hipLaunchKernelGGL(gk_adopt, dim3(ndd), dim3(256), 0, s, pr, dd_tl);
  return hipGetLastError();
}

// whitening z = L^-1 (x - x_ref) of every problem
__global__ __launch_bounds__(256) void gk_tri_inv(const BProb* __restrict__ pr, const BTile* __restrict__ tl) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  tri_inv_block(b.L, b.d, b.Linv, t.a);
}
// piece t.b of 16 columns t.a
__global__ __launch_bounds__(512) void gk_whiten(const BProb* __restrict__ pr, const BTile* __restrict__ tl, int P) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  const int rows = whiten_rows(b.d), r0 = t.b * rows;
  whiten_tile(b.L, b.Linv, t.b ? nullptr : b.X, b.xr, b.Z, rows >= b.d ? b.zq : nullptr, b.d, P, r0, rows, t.a);
}
__global__ __launch_bounds__(256) void gk_whiten_update(const BProb* __restrict__ pr, const BTile* __restrict__ tl,
                                                        int piece, int P) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  const int rows = whiten_rows(b.d);
  whiten_update_tile(b.L, piece ? nullptr : b.X, b.xr, b.Z, b.d, P, piece * rows, rows, t.a, t.b);
}
__global__ __launch_bounds__(256) void gk_colnorm(const BProb* __restrict__ pr, const BTile* __restrict__ tl) {
  const BTile t = tl[blockIdx.x];
  const BProb& b = pr[t.g];
  colnorm_block(b.Z, b.d, b.zq, t.a);  // parity 0 at a window boundary
}

hipError_t g_tri_inv(const BProb* pr, const BTile* tl, int n, hipStream_t s) {
  hipLaunchKernelGGL(gk_tri_inv, dim3(n), dim3(256), 0, s, pr, tl);
  return hipGetLastError();
}
hipError_t g_whiten(const BProb* pr, const BTile* tl, int n, const BTile* upd, int nupd, int piece, int P,
                    hipStream_t s) {
  hipLaunchKernelGGL(gk_whiten, dim3(n), dim3(512), 0, s, pr, tl, P);
  if (nupd) hipLaunchKernelGGL(gk_whiten_update, dim3(nupd), dim3(256), 0, s, pr, upd, piece, P);
  return hipGetLastError();
}
hipError_t g_colnorm(const BProb* pr, const BTile* tl, int n, hipStream_t s) {
  if (!n) return hipSuccess;
  hipLaunchKernelGGL(gk_colnorm, dim3(n), dim3(256), 0, s, pr, tl);
  return hipGetLastError();
}

hipError_t g_rng(uint64_t seed, const long* win, long nW, long nU, int P, float* W, double* U, hipStream_t s) {
  long nq = (nW + 3) / 4;
  int blocks = (int)((nq + 255) / 256);
  if (blocks > 8192) blocks = 8192;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(gk_normals, dim3(blocks), dim3(256), 0, s, (uint32_t)seed, (uint32_t)(seed >> 32), win, nW, nW, W);
  hipLaunchKernelGGL(gk_uniforms, dim3((unsigned)((nU + 255) / 256)), dim3(256), 0, s, (uint32_t)seed,
                     (uint32_t)(seed >> 32), win, nU, P, U);
  return hipGetLastError();
}

hipError_t g_bump(long* win, double* N, double K, hipStream_t s) {
  hipLaunchKernelGGL(gk_bump, dim3(1), dim3(64), 0, s, win, N, K);
  return hipGetLastError();
}

}  // namespace dk
