// Learned-part form: Bayesian logistic-regression target, the MLP surrogate
// of log pi (forward, backward, Adam; all on FP32 MFMA) and the kernels of
// two-stage delayed acceptance (Christen & Fox 2005): surrogate screen,
// survivor compaction, exact target on the survivors only.
#include <math.h>

#include "gemm.h"
#include "kernels.h"

using namespace gemm;

namespace dk {

// ============================================================================
// Logistic target: T = A X' (n_obs x d by d x P) on FP32 MFMA, then per
// element y t - softplus(t) and FP64 sums over 64-row blocks:
//   part[p][rb] = sum_{j in rb} [ y_j t_jp - softplus(t_jp) ]   (chain-major)
// Columns p >= *nact are skipped (their tiles exit at once).  Workgroup ids
// are dealt round-robin to the 8 XCDs; the column tiles of one row block are
// given consecutive ids on one XCD so that its rows of A are fetched once.
// ============================================================================
DEV float softplus_f(float t) { return fmaxf(t, 0.f) + log1pf(expf(-fabsf(t))); }

template <int BN>
__global__ __launch_bounds__(512) void k_tgt_logreg(const float* __restrict__ A, const float* __restrict__ y, int n_obs,
                                                    const float* __restrict__ V, int d, int P,
                                                    const int* __restrict__ nact_ptr, int nrb, int nct,
                                                    double* __restrict__ part) {
  constexpr int BM = 64, BK = 32, KG = 2;
  __shared__ float lds[KG * e_lds_elems<float, BM, BN, BK>()];
  __shared__ double red[2][BN];
  const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3;
  const int rb = (k / nct) * 8 + xcd, ct = k % nct;
  const int nact = nact_ptr ? *nact_ptr : P;
  const int i0 = rb * BM, j0 = ct * BN;
  if (rb >= nrb || j0 >= nact) return;  // uniform per workgroup, before any barrier
  EFrag<float, BM, BN> f;
  f.zero();
  // V always holds P columns (under delayed acceptance the survivors packed
  // first, the rest stale but readable), so the loads are bounded by P and a
  // partly filled last tile keeps the unguarded vector path; only columns
  // below nact are written
  e_gemm<float, BM, BN, BK, true, true, KG>(f, A, d, n_obs, V, d, P, i0, j0, 0, d, lds);
  const bool g0 = threadIdx.x < NT;
  const int lane = threadIdx.x & 63, w = (threadIdx.x & (NT - 1)) >> 6, wm = w & 1, wn = w >> 1;
  if (g0) {
#pragma unroll
    for (int n = 0; n < EFrag<float, BM, BN>::FN; ++n) {
      double s = 0.0;
#pragma unroll
      for (int m = 0; m < EFrag<float, BM, BN>::FM; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int ti, tj;
          frag_coords<BM, BN>(m, n, r, ti, tj);
          const int i = i0 + ti;
          if (i < n_obs) {
            const float t = f.c[m][n][r];
            s += (double)(y[i] * t - softplus_f(t));
          }
        }
      s += lane_xor_f64<16>(s);
      s += lane_xor_f64<32>(s);
      if (lane < 16) red[wm][wn * (BN / 2) + n * 16 + lane] = s;
    }
  }
  __syncthreads();
  if (threadIdx.x < BN) {
    const int j = j0 + threadIdx.x;
    if (j < nact) part[(long)j * nrb + rb] = red[0][threadIdx.x] + red[1][threadIdx.x];
  }
}

// The same on the direct-to-LDS engine, 64 observations x 64 chains by 2 x 2
// waves of 32 x 32, two interleaved chains of slices of K as the two k-groups
// above, the term bitwise the tile's.  Two stages of LDS: five workgroups a CU
// overlap one's softplus terms (72 us of n = 200000, d = 512, P = 128) with
// the others' products; 342 us in the tile above, 333 so, 348 with three
// stages, 341 with 128 x 64 tiles.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_tgt_logreg_t(
    const float* __restrict__ A, const float* __restrict__ y, int n_obs, const float* __restrict__ V, int d, int P,
    const int* __restrict__ nact_ptr, int nrb, int nct, double* __restrict__ part) {
  constexpr int BM = 64, BN = 64, WGM = 2, ST = 2;
  typedef TFrag<float, BM, BN, WGM, 2> F;
  static_assert(F::FM == 2, "32 rows per wave: two waves per 64-row term");
  __shared__ __attribute__((aligned(1024))) float lds[t_lds_elems<float, BM, BN, ST>()];
  const int xcd = blockIdx.x & 7, k = blockIdx.x >> 3;
  const int rb = (k / nct) * 8 + xcd, ct = k % nct;
  const int nact = nact_ptr ? *nact_ptr : P;
  const int i0 = rb * BM, j0 = ct * BN;
  if (i0 >= n_obs || j0 >= nact) return;  // uniform per workgroup, before any barrier
  F f[2];
  f[0].zero();
  f[1].zero();
  t_gemm<float, BM, BN, WGM, 2, ST, true, true, false, 2>(f, A, d, n_obs, V, d, P, i0, j0, 0, d, lds);
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
        t_coords<float, BM, BN, WGM, 2>(m, n, r, ti, tj);
        const int i = i0 + ti;
        if (i < n_obs) {
          const float t = f[0].c[m][n][r] + f[1].c[m][n][r];
          s += (double)(y[i] * t - softplus_f(t));
        }
      }
    s += lane_xor_f64<16>(s);
    s += lane_xor_f64<32>(s);
    if (lane < 16) red[wm][wn * (BN / 2) + n * 16 + lane] = s;
  }
  __syncthreads();
  if (threadIdx.x < BN) {
    const int j = j0 + threadIdx.x;
    if (j < nact) part[(long)j * nrb + rb] = red[0][threadIdx.x] + red[1][threadIdx.x];
  }
}

int logreg_row_blocks(long n_obs) { return (int)((n_obs + 63) / 64); }

// Column tiles of 64 chains; under delayed acceptance (nact set) the tiles
// past the survivor count exit at once.  (32-chain tiles were measured 1.5x
// less efficient per chain, more than their finer granularity saves.)
// The engine's two stages need the other workgroups of a CU to cover a slice's
// latency, and it reads an edge at full speed; up to two tiles a CU and without
// an edge the tile kernel's eight wavefronts are ahead.  us a step, tile kernel /
// engine, by n_obs, d, P (tiles): 4096, 512, 64 (64) 22.8 / 24.6; 16000, 512, 64
// (250) 29.0 / 30.6; 12800, 512, 128 (400) 39.3 / 41.0; 32768, 1024, 64 (512)
// 59.7 / 62.9; 16000, 4096, 64 (250) 115 / 135; 51200, 512, 64 (800) 63.4 / 63.8;
// 38400, 1024, 64 (600) 92.4 / 82.8; with an edge 16001, 1024, 64 (251) 42.7 / 44.1,
// 20000, 512, 64 (313) 42.1 / 40.8, 12800, 512, 50 (200) 35.6 / 30.5; with few
// slices of K 12800, 200, 64 (200) 23.5 / 23.5.
hipError_t tgt_logreg(const float* A, const float* y, long n_obs, const float* V, int d, int P, const int* nact,
                      double* part, hipStream_t s) {
  const int nrb = logreg_row_blocks(n_obs), groups = (nrb + 7) / 8;
  const int nct = cdiv(P, 64);
  const bool few_whole = n_obs % 64 == 0 && P % 64 == 0 && d >= 256 && (long)nrb * nct <= 512;
  if (!few_whole && t_gemm_ok<float, true, true>(A, d, (int)n_obs, V, d, P, d)) {
    hipLaunchKernelGGL(k_tgt_logreg_t, dim3(groups * 8 * nct), dim3(256), 0, s, A, y, (int)n_obs, V, d, P, nact, nrb,
                       nct, part);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_tgt_logreg<64>, dim3(groups * 8 * nct), dim3(512), 0, s, A, y, (int)n_obs, V, d, P, nact, nrb,
                     nct, part);
  return hipGetLastError();
}

// ============================================================================
// MLP surrogate: s(x) = out_std * (W3 h2 + b3) + out_mean,
// h2 = gelu(W2 h1 + b2), h1 = gelu(W1 xs + b1), xs = (x - in_mean) * in_scale.
// Weights used in the forward pass are the bf16 roundings of the FP32 master
// weights (stored as FP32 values); Adam updates the masters.  Activations
// are column-major: column s is sample s.
// ============================================================================
DEV float gelu_f(float a) { return a * 0.5f * (1.f + erff(a * 0.70710678118654752f)); }
DEV float gelu_grad_f(float a) {
  return 0.5f * (1.f + erff(a * 0.70710678118654752f)) + a * 0.39894228040143268f * expf(-0.5f * a * a);
}

// Products of the network: C(p, q) = sum_k A(p, k) B(q, k), epi(p, q, C) per
// element (lanes of a quarter wavefront along q).  The layers are small (256 x
// 256 outputs, K = 256 or 512, at the default minibatch), so a product is one
// chain of K / 4 matrix instructions and the time to fill it.  MLP_T32: 32 x 32
// tiles of the direct-to-LDS engine, one 16 x 16 block and one chain per
// wavefront; MLP_CHAIN: the same with four slices of K per barrier and 96 KB
// in flight (of a ring of 128), where no CU gets a second tile and K is whole stages (a forward
// layer 6.6 us against 7.9); MLP_T64: its 64 x 64 tiles, where those give every
// CU two; MLP_E: the element engine for unaligned operands.  All take k in the
// same order, so the results are bitwise the same (64 x 64 tiles of the element
// engine, 16 workgroups: 17.4 us a forward layer of 256 samples).
enum { MLP_CHAIN, MLP_T32, MLP_T64, MLP_E };
constexpr int mlp_tile(int cfg) { return cfg == MLP_CHAIN || cfg == MLP_T32 ? 32 : 64; }
constexpr int MLP_GRP = 4, MLP_CHAIN_ST = 4;
constexpr int mlp_lds(int cfg) {
  return cfg == MLP_CHAIN ? t_lds_elems<float, 32, 32, MLP_GRP * MLP_CHAIN_ST>()
       : cfg == MLP_T32   ? t_lds_elems<float, 32, 32, 6>()
       : cfg == MLP_T64   ? t_lds_elems<float, 64, 64, 3>()
                          : e_lds_elems<float, 64, 64, 32>();
}

template <int CFG, bool AKC, bool BKC, typename E>
DEV void mlp_product(const float* __restrict__ A, int lda, int M, const float* __restrict__ B, int ldb, int N, int K,
                     int bx, int by, float* lds, E epi) {
  if constexpr (CFG == MLP_E) {
    constexpr int BM = 64, BN = 64;
    EFrag<float, BM, BN> f;
    f.zero();
    e_gemm<float, BM, BN, 32, AKC, BKC>(f, A, lda, M, B, ldb, N, bx * BM, by * BN, 0, K, lds);
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int tp, tq;
          frag_coords<BM, BN>(m, n, r, tp, tq);
          if (bx * BM + tp < M && by * BN + tq < N) epi(bx * BM + tp, by * BN + tq, f.c[m][n][r]);
        }
  } else {
    constexpr int BM = mlp_tile(CFG), ST = CFG == MLP_CHAIN ? MLP_CHAIN_ST : CFG == MLP_T32 ? 6 : 3;
    constexpr int GRP = CFG == MLP_CHAIN ? MLP_GRP : 1;
    typedef TFrag<float, BM, BM, 2, 2> F;
    F f;
    f.zero();
    t_gemm<float, BM, BM, 2, 2, ST, AKC, BKC, false, 1, GRP>(*(F(*)[1]) & f, A, lda, M, B, ldb, N, bx * BM, by * BM, 0,
                                                             K, lds);
#pragma unroll
    for (int m = 0; m < F::FM; ++m)
#pragma unroll
      for (int n = 0; n < F::FN; ++n)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          int tp, tq;
          t_coords<float, BM, BM, 2, 2>(m, n, r, tp, tq);
          if (bx * BM + tp < M && by * BM + tq < N) epi(bx * BM + tp, by * BM + tq, f.c[m][n][r]);
        }
  }
}

// blocks of a product of M x N outputs
static int mlp_blocks(int cfg, int M, int N) { return cdiv(M, mlp_tile(cfg)) * cdiv(N, mlp_tile(cfg)); }
template <bool AKC, bool BKC>
static int mlp_cfg(const float* A, int lda, int M, const float* B, int ldb, int N, int K) {
  if (!t_gemm_ok<float, AKC, BKC>(A, lda, M, B, ldb, N, K)) return MLP_E;
  if ((long)cdiv(M, 64) * cdiv(N, 64) >= 512) return MLP_T64;
  return K % (MLP_GRP * tbk<float>()) == 0 && (long)cdiv(M, 32) * cdiv(N, 32) <= 256 ? MLP_CHAIN : MLP_T32;
}

// Forward layer of n samples: a = W x + bias, h = gelu(a) (O outputs, I inputs)
template <int CFG>
__global__ __launch_bounds__(256) void k_mlp_layer(const float* __restrict__ x, int I, int n,
                                                   const float* __restrict__ W, int O, const float* __restrict__ bias,
                                                   float* __restrict__ a, float* __restrict__ h) {
  __shared__ __attribute__((aligned(1024))) float lds[mlp_lds(CFG)];
  constexpr int T = mlp_tile(CFG);
  const int nq = (O + T - 1) / T;
  mlp_product<CFG, true, true>(x, I, n, W, I, O, I, blockIdx.x / nq, blockIdx.x % nq, lds,
                               [&](int s, int o, float c) {
                                 const float v = c + bias[o];
                                 a[o + (long)s * O] = v;
                                 h[o + (long)s * O] = gelu_f(v);
                               });
}

static void mlp_layer(const float* x, int I, int n, const float* W, int O, const float* bias, float* a, float* h,
                      hipStream_t s) {
  const int cfg = mlp_cfg<true, true>(x, I, n, W, I, O, I);
  const dim3 grid(mlp_blocks(cfg, n, O));
  if (cfg == MLP_CHAIN) hipLaunchKernelGGL(k_mlp_layer<MLP_CHAIN>, grid, dim3(256), 0, s, x, I, n, W, O, bias, a, h);
  else if (cfg == MLP_T32) hipLaunchKernelGGL(k_mlp_layer<MLP_T32>, grid, dim3(256), 0, s, x, I, n, W, O, bias, a, h);
  else if (cfg == MLP_T64) hipLaunchKernelGGL(k_mlp_layer<MLP_T64>, grid, dim3(256), 0, s, x, I, n, W, O, bias, a, h);
  else hipLaunchKernelGGL(k_mlp_layer<MLP_E>, grid, dim3(256), 0, s, x, I, n, W, O, bias, a, h);
}

// out[s] = sum_o w3[o] h2[o, s] + b3 (one wavefront per sample)
__global__ __launch_bounds__(256) void k_mlp_out(const float* __restrict__ w3, const float* __restrict__ b3,
                                                 const float* __restrict__ h2, int H, int n, float* __restrict__ out) {
  const int lane = threadIdx.x & 63, s = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (s >= n) return;
  float acc = 0.f;
  for (int o = lane; o < H; o += 64) acc = fmaf(w3[o], h2[o + (long)s * H], acc);
  acc = wave_sum_f32(acc);
  if (lane == 0) out[s] = acc + b3[0];
}

// xs[:, s] = (x_s - in_mean) * in_scale from FP64 (X64) or FP32 (X32) states
__global__ __launch_bounds__(256) void k_mlp_standardize(const double* __restrict__ X64, const float* __restrict__ X32,
                                                         const float* __restrict__ in_mean,
                                                         const float* __restrict__ in_scale, int D, long n,
                                                         float* __restrict__ xs) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= (long)D * n) return;
  const int i = (int)(e % D);
  const float x = X64 ? (float)X64[e] : X32[e];
  xs[e] = (x - in_mean[i]) * in_scale[i];
}

// surrogate log density (FP64) from the FP32 network output
__global__ __launch_bounds__(256) void k_mlp_denorm(const float* __restrict__ out, const float* __restrict__ stats, int n,
                                                    double* __restrict__ s_out) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < n) s_out[e] = (double)out[e] * (double)stats[1] + (double)stats[0];
}

// per-coordinate mean and 1/std over n samples (FP64 inputs, column-major d x n)
__global__ __launch_bounds__(256) void k_mlp_in_stats(const double* __restrict__ X, int d, long n,
                                                      float* __restrict__ in_mean, float* __restrict__ in_scale) {
  __shared__ double red[2][256];
  const int i = blockIdx.x;
  double s = 0.0, q = 0.0;
  for (long k = threadIdx.x; k < n; k += 256) {
    const double x = X[i + k * d];
    s += x;
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
  if (threadIdx.x == 0) {
    const double mean = red[0][0] / n;
    const double var = fmax(red[1][0] / n - mean * mean, 0.0);
    in_mean[i] = (float)mean;
    in_scale[i] = (float)(1.0 / fmax(sqrt(var), 1e-12));
  }
}

// stats[0] = mean, stats[1] = std of the n log densities; ts = standardised
__global__ __launch_bounds__(256) void k_mlp_out_stats(const double* __restrict__ lp, long n, float* __restrict__ stats,
                                                       float* __restrict__ ts) {
  __shared__ double red[2][256];
  __shared__ double mean_s, std_s;
  double s = 0.0, q = 0.0;
  for (long k = threadIdx.x; k < n; k += 256) {
    s += lp[k];
    q = __fma_rn(lp[k], lp[k], q);
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
  if (threadIdx.x == 0) {
    const double mean = red[0][0] / n;
    mean_s = mean;
    std_s = fmax(sqrt(fmax(red[1][0] / n - mean * mean, 0.0)), 1e-12);
    stats[0] = (float)mean;
    stats[1] = (float)std_s;
  }
  __syncthreads();
  for (long k = threadIdx.x; k < n; k += 256) ts[k] = (float)((lp[k] - mean_s) / std_s);
}

// He-normal init of the master weights from Philox (biases zero)
__global__ __launch_bounds__(256) void k_mlp_init(uint32_t k0, uint32_t k1, int D, int H, float* __restrict__ master,
                                                  float* __restrict__ eff, long nparam) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e >= nparam) return;
  const long oW1 = 0, ob1 = (long)H * D, oW2 = ob1 + H, ob2 = oW2 + (long)H * H, oW3 = ob2 + H, ob3 = oW3 + H;
  float scale = 0.f;
  if (e < ob1) scale = sqrtf(2.f / D);
  else if (e >= oW2 && e < ob2) scale = sqrtf(2.f / H);
  else if (e >= oW3 && e < ob3) scale = sqrtf(2.f / H);
  float v = 0.f;
  if (scale > 0.f) {
    const u4_t r = philox4x32_10({(uint32_t)e, (uint32_t)(e >> 32), 7u, 0u}, k0, k1);
    const float u1 = u01_f32(r.x), u2 = u01_f32(r.y);
    v = scale * sqrtf(-2.f * logf(u1)) * cosf(6.28318530717958647692f * u2);
  }
  master[e] = v;
  eff[e] = bf16_bits_to_f32(f32_to_bf16_bits(v));
}

// Minibatches: indices from Philox (with replacement), step tau; one block of
// 256 threads per pair.
struct BatchArgs {
  uint32_t k0, k1;
  const float *Xs, *ts;
  int D, nb;
  long n;
  float *xb, *tb;
  int* idx;
};
DEV void mlp_batch_pair(const BatchArgs& a, long tau, int j) {
  // every thread draws the index: no trip through LDS
  const u4_t r = philox4x32_10({(uint32_t)tau, (uint32_t)(tau >> 32), 8u, (uint32_t)j}, a.k0, a.k1);
  const uint64_t bits = ((uint64_t)r.x << 32) | r.y;
  const long src = (long)(bits % (uint64_t)a.n);
  if (threadIdx.x == 0) {
    a.idx[j] = (int)src;
    a.tb[j] = a.ts[src];
  }
  for (int i = threadIdx.x; i < a.D; i += 256) a.xb[i + (long)j * a.D] = a.Xs[i + src * a.D];
}
__global__ __launch_bounds__(256) void k_mlp_batch(BatchArgs a, long tau) { mlp_batch_pair(a, tau, blockIdx.x); }

// Sums over the samples of four units' values by 256 threads: thread t holds
// unit t % 4's partial sum over samples t / 4 + 64 i; combined in the order of
// a wavefront's butterfly.  Threads 0 to 3 return the totals.
DEV float unit_sum4(float v, float (*red)[4]) {
  const int l = threadIdx.x >> 2, u = threadIdx.x & 3;
  __syncthreads();
  red[l][u] = v;
  for (int o = 32; o > 0; o >>= 1) {
    __syncthreads();
    if (l < o) red[l][u] += red[l + o][u];
  }
  return red[0][u];
}

// Output layer backward for L = mean (out - t)^2, g[s] = dL/dout[s]: gW3[o] =
// sum_s g[s] h2[o,s], ga2[o,s] = w3[o] g[s] gelu'(a2[o,s]) and gb2[o] = sum_s
// ga2[o,s] per block of four units, the loss and gb3 = sum g on the last block.
// Bound by the special functions (more units a block leave CUs idle: 14 us with
// 16) and by one trip to memory.
__global__ __launch_bounds__(256) void k_mlp_out_bwd(const float* __restrict__ w3, const float* __restrict__ out,
                                                     const float* __restrict__ tb, const float* __restrict__ h2,
                                                     const float* __restrict__ a2, int H, int nb,
                                                     float* __restrict__ gW3, float* __restrict__ gb3,
                                                     float* __restrict__ ga2, float* __restrict__ gb2,
                                                     float* __restrict__ loss) {
  const int t = threadIdx.x;
  if (blockIdx.x == gridDim.x - 1) {
    __shared__ float red[256];
    float s = 0.f;
    for (int j = t; j < nb; j += 256) {
      const float r = out[j] - tb[j];
      s = fmaf(r, r, s);
    }
    red[t] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
      if (t < o) red[t] += red[t + o];
      __syncthreads();
    }
    if (t == 0) *loss = red[0] / nb;
    if (t < 64) {
      float b = 0.f;
      for (int j = t; j < nb; j += 64) b += 2.f * (out[j] - tb[j]) / nb;
      b = wave_sum_f32(b);
      if (t == 0) gb3[0] = b;
    }
    return;
  }
  __shared__ float red[64][4];
  const int o = blockIdx.x * 4 + (t & 3);
  const bool in = o < H;
  const float w = in ? w3[o] : 0.f;
  float vw = 0.f, vb = 0.f;
#pragma unroll 4
  for (int s = t >> 2; s < nb; s += 64) {
    const long e = (in ? o : 0) + (long)s * H;
    const float g = 2.f * (out[s] - tb[s]) / nb;
    const float ga = w * g * gelu_grad_f(a2[e]);
    if (in) ga2[e] = ga;
    vw = fmaf(g, h2[e], vw);
    vb += ga;
  }
  const float sw = unit_sum4(vw, red), sb = unit_sum4(vb, red);
  if (t < 4 && in) {
    gW3[o] = sw;
    gb2[o] = sb;
  }
}

// The two products on ga2: gW2 = ga2 h1^T (the first blocks) and ga1 = (W2^T
// ga2) * gelu'(a1).  Neither fills the chip; one launch runs both.
template <int CW, int CG>
__global__ __launch_bounds__(256) void k_mlp_hidden_bwd(const float* __restrict__ ga2, const float* __restrict__ h1,
                                                        const float* __restrict__ W2, const float* __restrict__ a1,
                                                        int H, int nb, float* __restrict__ gW2,
                                                        float* __restrict__ ga1) {
  constexpr int NW = mlp_lds(CW), NG = mlp_lds(CG), TW = mlp_tile(CW), TG = mlp_tile(CG);
  __shared__ __attribute__((aligned(1024))) float lds[NW > NG ? NW : NG];
  const int nw = (H + TW - 1) / TW, ng = (H + TG - 1) / TG, b = blockIdx.x;
  if (b < nw * nw) {
    mlp_product<CW, false, false>(ga2, H, H, h1, H, H, nb, b / nw, b % nw, lds,
                                  [&](int o, int i, float c) { gW2[(long)o * H + i] = c; });
  } else {
    const int k = b - nw * nw;
    mlp_product<CG, true, false>(ga2, H, nb, W2, H, H, H, k / ng, k % ng, lds, [&](int s, int i, float c) {
      const long e = i + (long)s * H;
      ga1[e] = c * gelu_grad_f(a1[e]);
    });
  }
}

// Adam (Kingma & Ba 2015), bias-corrected; eff = bf16 rounding of the master
struct AdamArgs {
  float *master, *eff, *g, *m, *v;
  float lr, b1, b2, eps, c1, c2;
};
DEV void adam_elem(const AdamArgs& a, long e, float gg) {
  const float mm = a.b1 * a.m[e] + (1.f - a.b1) * gg;
  const float vv = a.b2 * a.v[e] + (1.f - a.b2) * gg * gg;
  a.m[e] = mm;
  a.v[e] = vv;
  const float w = a.master[e] - a.lr * (mm / a.c1) / (sqrtf(vv / a.c2) + a.eps);
  a.master[e] = w;
  a.eff[e] = bf16_bits_to_f32(f32_to_bf16_bits(w));
}

// The step's last launch: gW1 = ga1 xb^T with Adam on each element as it is
// formed, then blocks of four units for gb1 = rowsum(ga1) and its step, then
// the other parameters' steps (nothing reads them until the next minibatch),
// then the next minibatch's pairs (next.nb = 0: none) into another buffer.
template <int CFG>
__global__ __launch_bounds__(256) void k_mlp_input_bwd(const float* __restrict__ ga1, const float* __restrict__ xb,
                                                       int D, int H, int nb, AdamArgs a, BatchArgs next,
                                                       long tau) {
  __shared__ __attribute__((aligned(1024))) float lds[mlp_lds(CFG)];
  constexpr int T = mlp_tile(CFG);
  const int nq = (D + T - 1) / T, np = (H + T - 1) / T, t = threadIdx.x;
  int b = blockIdx.x;
  if (b < np * nq) {
    mlp_product<CFG, false, false>(ga1, H, H, xb, D, D, nb, b / nq, b % nq, lds, [&](int o, int i, float c) {
      const long e = (long)o * D + i;
      a.g[e] = c;
      adam_elem(a, e, c);
    });
    return;
  }
  b -= np * nq;
  const long bias1 = (long)H * D, rest = bias1 + H, end = rest + (long)H * H + 2 * H + 1;
  if (b < (H + 3) / 4) {
    const int o = b * 4 + (t & 3);
    float v = 0.f;
#pragma unroll 4
    for (int s = t >> 2; s < nb; s += 64) v += o < H ? ga1[o + (long)s * H] : 0.f;
    const float sum = unit_sum4(v, (float (*)[4])lds);
    if (t < 4 && o < H) {
      a.g[bias1 + o] = sum;
      adam_elem(a, bias1 + o, sum);
    }
    return;
  }
  b -= (H + 3) / 4;
  if (b < (end - rest + 255) / 256) {
    const long e = rest + (long)b * 256 + t;
    if (e < end) adam_elem(a, e, a.g[e]);
    return;
  }
  mlp_batch_pair(next, tau + 1, b - (int)((end - rest + 255) / 256));
}

__global__ void k_fill_f32(float* p, long n) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e < n) p[e] = 0.f;
}

size_t mlp_nparam(int D, int H) { return (size_t)H * D + H + (size_t)H * H + H + H + 1; }

// Forward pass of n samples held in xs (D x n); writes a1, h1, a2, h2, out.
hipError_t mlp_forward(const MlpBufs& b, const float* xs, int n, hipStream_t s) {
  const int D = b.D, H = b.H;
  const float* W1 = b.eff;
  const float* b1 = W1 + (long)H * D;
  const float* W2 = b1 + H;
  const float* b2 = W2 + (long)H * H;
  const float* W3 = b2 + H;
  const float* b3 = W3 + H;
  mlp_layer(xs, D, n, W1, H, b1, b.a1, b.h1, s);
  mlp_layer(b.h1, H, n, W2, H, b2, b.a2, b.h2, s);
  hipLaunchKernelGGL(k_mlp_out, dim3(cdiv(n, 4)), dim3(256), 0, s, W3, b3, (const float*)b.h2, H, n, b.out);
  return hipGetLastError();
}

hipError_t mlp_eval(const MlpBufs& b, const double* X64, const float* X32, int n, double* s_out, hipStream_t s) {
  const long tot = (long)b.D * n;
  hipLaunchKernelGGL(k_mlp_standardize, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, X64, X32,
                     (const float*)b.in_mean, (const float*)b.in_scale, b.D, (long)n, b.xb);
  hipError_t e = mlp_forward(b, b.xb, n, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_denorm, dim3(cdiv(n, 256)), dim3(256), 0, s, (const float*)b.out, (const float*)b.stats, n,
                     s_out);
  return hipGetLastError();
}

hipError_t mlp_prepare(const MlpBufs& b, const double* X, const double* lp, long n, uint64_t seed, hipStream_t s) {
  const int D = b.D;
  hipLaunchKernelGGL(k_mlp_in_stats, dim3(D), dim3(256), 0, s, X, b.d_state, n, b.in_mean, b.in_scale);
  hipLaunchKernelGGL(k_mlp_out_stats, dim3(1), dim3(256), 0, s, lp, n, b.stats, b.ts);
  const long tot = (long)D * n;
  hipLaunchKernelGGL(k_mlp_standardize, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, X, (const float*)nullptr,
                     (const float*)b.in_mean, (const float*)b.in_scale, D, n, b.Xs);
  const long np = (long)mlp_nparam(D, b.H);
  hipLaunchKernelGGL(k_mlp_init, dim3((unsigned)((np + 255) / 256)), dim3(256), 0, s, (uint32_t)seed,
                     (uint32_t)(seed >> 32), D, b.H, b.master, b.eff, np);
  hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)((2 * np + 255) / 256)), dim3(256), 0, s, b.m, 2 * np);
  return hipGetLastError();
}

// One Adam step on a Philox-drawn minibatch of nb training pairs, step tau of
// `steps`.  Where two minibatches fit xb (room columns), they take its halves
// in turn and a step's last launch gathers the next step's (3 us a step as a
// launch of its own).
hipError_t mlp_train_step(const MlpBufs& b, long n, int nb, long tau, long steps, int room, uint64_t seed, float lr,
                          hipStream_t s) {
  const int D = b.D, H = b.H;
  const long np = (long)mlp_nparam(D, H);
  float* gW2 = b.grad + (long)H * D + H;
  float* gb2 = gW2 + (long)H * H;
  float* gW3 = gb2 + H;
  const float* W2 = b.eff + (long)H * D + H;
  const float* W3 = W2 + (long)H * H + H;
  const float* ga1 = b.ga1;
  const bool ahead = 2L * nb <= room;
  float* half[2] = {b.xb, ahead ? b.xb + (long)nb * D : b.xb};
  BatchArgs ba{(uint32_t)seed, (uint32_t)(seed >> 32), b.Xs, b.ts, D, nb, n, half[tau & 1], b.tb, b.bidx};
  const float* xb = ba.xb;
  if (tau == 0 || !ahead) hipLaunchKernelGGL(k_mlp_batch, dim3(nb), dim3(256), 0, s, ba, tau);
  ba.xb = half[(tau + 1) & 1];
  if (!ahead || tau + 1 >= steps) ba.nb = 0;
  hipError_t e = mlp_forward(b, xb, nb, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_mlp_out_bwd, dim3(cdiv(H, 4) + 1), dim3(256), 0, s, W3, (const float*)b.out,
                     (const float*)b.tb, (const float*)b.h2, (const float*)b.a2, H, nb, gW3, gW3 + H, b.ga2, gb2,
                     b.loss);
  const float *ga2 = b.ga2, *h1 = b.h1, *a1 = b.a1;
  const int cw = mlp_cfg<false, false>(ga2, H, H, h1, H, H, nb), cg = mlp_cfg<true, false>(ga2, H, nb, W2, H, H, H);
  const auto blocks2 = [&](int w, int g) { return dim3(mlp_blocks(w, H, H) + mlp_blocks(g, nb, H)); };
  if (cw > MLP_T32 || cg > MLP_T64) return hipErrorInvalidValue;  // H = 256: aligned, few tiles
  if (cw == MLP_CHAIN && cg == MLP_CHAIN)
    hipLaunchKernelGGL((k_mlp_hidden_bwd<MLP_CHAIN, MLP_CHAIN>), blocks2(cw, cg), dim3(256), 0, s, ga2, h1, W2, a1, H,
                       nb, gW2, b.ga1);
  else if (cg == MLP_T64)
    hipLaunchKernelGGL((k_mlp_hidden_bwd<MLP_T32, MLP_T64>), blocks2(MLP_T32, cg), dim3(256), 0, s, ga2, h1, W2, a1,
                       H, nb, gW2, b.ga1);
  else
    hipLaunchKernelGGL((k_mlp_hidden_bwd<MLP_T32, MLP_T32>), blocks2(MLP_T32, MLP_T32), dim3(256), 0, s, ga2, h1, W2,
                       a1, H, nb, gW2, b.ga1);
  AdamArgs ad{b.master, b.eff, b.grad, b.m, b.m + np, lr, 0.9f, 0.999f, 1e-8f, 0.f, 0.f};
  ad.c1 = 1.f - powf(ad.b1, (float)(tau + 1));
  ad.c2 = 1.f - powf(ad.b2, (float)(tau + 1));
  // not one tile per CU: the other blocks of this launch share the CUs
  const int cfg1 = std::max(mlp_cfg<false, false>(ga1, H, H, xb, D, D, nb), (int)MLP_T32);
  const dim3 grid1(mlp_blocks(cfg1, H, D) + cdiv(H, 4) + cdiv((long)H * H + 2 * H + 1, 256) + ba.nb);
  if (cfg1 == MLP_T32) hipLaunchKernelGGL(k_mlp_input_bwd<MLP_T32>, grid1, dim3(256), 0, s, ga1, xb, D, H, nb, ad, ba, tau);
  else if (cfg1 == MLP_T64)
    hipLaunchKernelGGL(k_mlp_input_bwd<MLP_T64>, grid1, dim3(256), 0, s, ga1, xb, D, H, nb, ad, ba, tau);
  else hipLaunchKernelGGL(k_mlp_input_bwd<MLP_E>, grid1, dim3(256), 0, s, ga1, xb, D, H, nb, ad, ba, tau);
  return hipGetLastError();
}

// ============================================================================
// Delayed acceptance, stage 1 (one workgroup of 16 waves):
//   s_new[p] = out_std * (w3 . h2[:, p] + b3) + out_mean       (network output)
//   log a1   = (s_new - s_cur) + [plain form only] (|z'|^2 - |z|^2) / (2 alpha^2)
// In the residual form the surrogate is r(x) - |z(x)|^2 / (2 alpha^2): its
// Gaussian part cancels the proposal's own correction, so stage 1 compares
// the network outputs alone.  Survivors get consecutive slots in chain
// order (wave ballots + prefix counts), so packing is deterministic.
// ============================================================================
__global__ __launch_bounds__(1024) void k_da_screen(const float* __restrict__ w3, const float* __restrict__ b3,
                                                    const float* __restrict__ h2, int H,
                                                    const float* __restrict__ stats, int P, int nch,
                                                    const double* __restrict__ s_cur,
                                                    const double* __restrict__ zq_part,
                                                    const double* __restrict__ zq, const double* __restrict__ u1,
                                                    double inv2a2, int resid, double* __restrict__ s_new,
                                                    uint8_t* __restrict__ pass, int* __restrict__ slot,
                                                    int* __restrict__ idx, int* __restrict__ nsurv,
                                                    int* __restrict__ npass) {
  __shared__ int wt[16];
  __shared__ int base;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const double om = (double)stats[0], os = (double)stats[1];
  for (int q = w; q < P; q += 16) {
    float acc = 0.f;
    for (int o = lane; o < H; o += 64) acc = fmaf(w3[o], h2[o + (long)q * H], acc);
    acc = wave_sum_f32(acc);
    if (lane == 0) s_new[q] = (double)(acc + b3[0]) * os + om;
  }
  if (threadIdx.x == 0) base = 0;
  __syncthreads();
  for (int p0 = 0; p0 < P; p0 += 1024) {
    const int p = p0 + threadIdx.x;
    int ok = 0;
    if (p < P) {
      double la1 = s_new[p] - s_cur[p];
      if (!resid) {
        double zs = 0.0;
        for (int c = 0; c < nch; ++c) zs += zq_part[(long)p * nch + c];
        la1 += (zs - zq[p]) * inv2a2;
      }
      ok = log(u1[p]) < la1 ? 1 : 0;
      pass[p] = (uint8_t)ok;
      npass[p] += ok;
    }
    const unsigned long long m = __ballot(ok);
    const int below = __popcll(m & ((1ull << lane) - 1ull));
    if (lane == 0) wt[w] = __popcll(m);
    __syncthreads();
    int off = base;
    for (int v = 0; v < w; ++v) off += wt[v];
    if (p < P) {
      slot[p] = ok ? off + below : -1;
      if (ok) idx[off + below] = p;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      int t = 0;
      for (int v = 0; v < 16; ++v) t += wt[v];
      base += t;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *nsurv = base;
}

// survivors' proposals, packed: Vs[:, j] = V[:, idx[j]] for j < nsurv
__global__ __launch_bounds__(256) void k_da_gather(const float* __restrict__ V, const int* __restrict__ idx,
                                                   const int* __restrict__ nsurv, int d, int P,
                                                   float* __restrict__ Vs) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  const int j = (int)(e / d), i = (int)(e % d);
  if (j >= P || j >= *nsurv) return;
  Vs[i + (long)j * d] = V[i + (long)idx[j] * d];
}

hipError_t da_screen(const MlpBufs& b, const float* V, int d, int P, int nch, const double* s_cur,
                     const double* zq_part, const double* zq, const double* u1, double inv2a2, int resid,
                     double* s_new, uint8_t* pass, int* slot, int* idx, int* nsurv, int* npass, float* Vs,
                     hipStream_t s) {
  const long tot = (long)b.D * P;
  hipLaunchKernelGGL(k_mlp_standardize, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, (const double*)nullptr,
                     V, (const float*)b.in_mean, (const float*)b.in_scale, b.D, (long)P, b.xb);
  const int H = b.H;
  const float* W1 = b.eff;
  const float* b1 = W1 + (long)H * b.D;
  const float* W2 = b1 + H;
  const float* b2 = W2 + (long)H * H;
  const float* W3 = b2 + H;
  const float* b3 = W3 + H;
  mlp_layer(b.xb, b.D, P, W1, H, b1, b.a1, b.h1, s);
  mlp_layer(b.h1, H, P, W2, H, b2, b.a2, b.h2, s);
  hipLaunchKernelGGL(k_da_screen, dim3(1), dim3(1024), 0, s, W3, b3, (const float*)b.h2, H, (const float*)b.stats, P,
                     nch, s_cur, zq_part, zq, u1, inv2a2, resid, s_new, pass, slot, idx, nsurv, npass);
  hipLaunchKernelGGL(k_da_gather, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, V, (const int*)idx,
                     (const int*)nsurv, d, P, Vs);
  return hipGetLastError();
}

// t[k] = lp[k] + c zq[k]  (residual-form training targets)
__global__ __launch_bounds__(256) void k_axpy_f64(const double* __restrict__ lp, const double* __restrict__ zq,
                                                  double c, long n, double* __restrict__ t) {
  const long e = (long)blockIdx.x * 256 + threadIdx.x;
  if (e < n) t[e] = __fma_rn(c, zq[e], lp[e]);
}

hipError_t axpy_f64(const double* lp, const double* zq, double c, long n, double* t, hipStream_t s) {
  hipLaunchKernelGGL(k_axpy_f64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, lp, zq, c, n, t);
  return hipGetLastError();
}

}  // namespace dk
