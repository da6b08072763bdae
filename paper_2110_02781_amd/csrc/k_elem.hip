// BatchNorm statistics / apply / backward, pooling, softmax cross-entropy,
// SGD-momentum and small utility kernels.  All are HBM-bound streaming kernels:
// each thread moves 8 consecutive channels (16 or 32 bytes) per access, rows
// are walked so that a block touches contiguous memory, and per-channel sums
// are reduced in a fixed order (per thread -> LDS across the block -> float64
// across blocks), so results are run-to-run deterministic.  Short tensors (at most
// 2048 rows) use one-launch variants in which a block owns 4 channels over all rows.
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"
#include "bn_pending.h"

namespace ftp {

#define FTP_DISPATCH(dt, ...)                   \
  do {                                          \
    if ((dt) == 0) { typedef float T; __VA_ARGS__; } \
    else { typedef bf16_t T; __VA_ARGS__; }     \
  } while (0)

static RowTile rowtile_with(size_t M, int CG, int nslab, int max_partials) {
  RowTile t;
  t.nslab = nslab;
  t.W = (CG + t.nslab - 1) / t.nslab;
  t.R = 256 / t.W;
  if (t.R < 1) t.R = 1;
  size_t want = (M + max_partials - 1) / max_partials;        // rows per block so that P <= max
  size_t rpb = ((want + t.R - 1) / t.R) * t.R;
  size_t min_rpb = (size_t)t.R * 4;                            // at least 4 iterations per block
  if (min_rpb < (size_t)kBnMinRows) min_rpb = ((kBnMinRows + t.R - 1) / t.R) * t.R;
  if (rpb < min_rpb) rpb = min_rpb;
  t.rows_per_block = rpb;
  t.P = (int)((M + rpb - 1) / rpb);
  if (t.P < 1) t.P = 1;
  return t;
}

RowTile make_rowtile(size_t M, int C, int max_partials) {
  const int CG = C / 8;
  RowTile t = rowtile_with(M, CG, (CG + 255) / 256, max_partials);
  // Few rows and many channels (6 K x 1344): the rows alone give too few blocks for 256 CUs, so the channels are cut
  // into slabs as well, down to 8 column groups (one 128-byte line per row and slab), until there are about 1024 blocks.
  // Only where the ROWS are what limits the blocks (P stopped by the minimum rows per block, not by max_partials).
  while (t.P < 256 && t.P < max_partials / 2 && (size_t)t.P * t.nslab < 1024 && (CG + t.nslab) / (t.nslab + 1) >= 8)
    t = rowtile_with(M, CG, t.nslab + 1, max_partials);
  return t;
}

// Kernels without partial sums: one round (two rows a thread) per block until there are kApplyBlocks of them, then longer blocks, whose threads
// fetch their coefficients once for more rows.  A whole training interval, blocks 512 / 2048 / 8192 against four rounds a block at least,
// and the rows dealt round-robin: MobileNetV2 at 32x32 fp32 1.011 / 1.006 / 1.004, 224x224 bfloat16 batch 32 recomputing 1.003 / 1.006 /
// 1.007, width 1.4 batch 128 0.997 / 1.002 / 1.005.
enum { kApplyBlocks = 2048, kFinishBlocks = 1024 };
static RowTile apply_rowtile(size_t M, int C) {
  RowTile t;
  const int CG = C / 8;
  t.nslab = (CG + 255) / 256;
  t.W = (CG + t.nslab - 1) / t.nslab;
  t.R = 256 / t.W;
  const size_t round = 2 * (size_t)t.R, rounds = (M + round - 1) / round, per = (rounds * t.nslab + kApplyBlocks - 1) / kApplyBlocks;
  t.rows_per_block = per * round;
  t.P = (int)((M + t.rows_per_block - 1) / t.rows_per_block);
  return t;
}

// Row chunk and channel slab of a block of a (chunks, slabs) grid, a contiguous eighth of the rows on each XCD: the GEMM and depthwise
// tiles deal their rows out the same way, so what a kernel reads was mostly written (or read) through the same L2 by the kernel before it.
struct ChunkSlab { int chunk, slab; };
__device__ __forceinline__ ChunkSlab chunk_slab() {
  const int lb = xcd_logical(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y), ns = gridDim.y;
  return ns == 1 ? ChunkSlab{lb, 0} : ChunkSlab{lb / ns, lb % ns};
}

// Column sums of a block: v[0..16) of thread (tx = column group, ty = row lane) are 8 sums and 8 second
// sums for channels cg*8..+7.  They go through LDS; then every (value, column group) pair gets its own
// thread, which adds the R row lanes in order and stores straight into partial[2][C] (the serial tail of
// one thread per column group doing all 16 values cost more than the streaming loop for short blocks).
__device__ __forceinline__ void reduce_rows_to_partial(const float (&v)[16], int tx, int ty, int W, int R, int cg0, int C,
                                                       float* smem, float* __restrict__ partial) {
#pragma unroll
  for (int e = 0; e < 16; ++e) smem[(e * R + ty) * W + tx] = v[e];
  __syncthreads();
  for (int i = threadIdx.x; i < 16 * W; i += blockDim.x) {
    const int e = i / W, x = i - e * W;
    if ((cg0 + x) * 8 >= C) continue;
    float s = 0.f;
    for (int r = 0; r < R; ++r) s += smem[(e * R + r) * W + x];
    partial[(size_t)(e >> 3) * C + (cg0 + x) * 8 + (e & 7)] = s;
  }
}

// ------------------------------------------------------------------ bn_stats
template <typename T>
__global__ void bn_stats_k(const T* __restrict__ z, size_t M, int C, int W, int R, size_t rpb,
                           float* __restrict__ partial) {
  extern __shared__ float smem[];
  const ChunkSlab at = chunk_slab();
  int tx = threadIdx.x % W, ty = threadIdx.x / W;
  int cg = at.slab * W + tx;
  float acc[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  if (cg < C / 8) {
    size_t m0 = (size_t)at.chunk * rpb, m1 = m0 + rpb < M ? m0 + rpb : M;
    // four rows per round: the loads are issued together, the sums keep a fixed order
    for (size_t m = m0 + ty; m < m1; m += 4 * (size_t)R) {
      Raw<T> rv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (m + (size_t)u * R < m1) raw_load(rv[u], z + (m + (size_t)u * R) * C + cg * 8);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (m + (size_t)u * R >= m1) break;
        float v[8];
        raw_unpack(rv[u], v);
#pragma unroll
        for (int e = 0; e < 8; ++e) { acc[e] += v[e]; acc[8 + e] = fmaf(v[e], v[e], acc[8 + e]); }
      }
    }
  }
  reduce_rows_to_partial(acc, tx, ty, W, R, at.slab * W, C, smem, partial + (size_t)at.chunk * 2 * C);
}

void bn_stats(int dt, hipStream_t st, const void* z, size_t M, int C, float* partial, int* P_out) {
  RowTile t = make_rowtile(M, C, kBnPartials);
  {
    KScope ks(st, "bn_stats", (double)M * C * (dt == 0 ? 4.0 : 2.0), 3.0 * M * C);
    dim3 grid(t.P, t.nslab), block(t.W * t.R);
    size_t sm = (size_t)16 * t.R * t.W * sizeof(float);
    FTP_DISPATCH(dt, hipLaunchKernelGGL(bn_stats_k<T>, grid, block, sm, st, (const T*)z, M, C, t.W, t.R,
                                        t.rows_per_block, partial));
  }
  *P_out = t.P;
}

// Sums of partial[p][2][C] over p in float64; kFinCh channels per block, kFinLanes lanes per channel (few channels per
// block: a layer has only C / kFinCh blocks and the partial walk is pure latency).  Threads 0 .. kFinCh - 1 return the
// sum and the second sum of channel c0 + threadIdx.x.
enum { kFinCh = 8, kFinLanes = 256 / kFinCh };
__device__ __forceinline__ void sum_partials(const float* __restrict__ partial, int P, int C, int c0, double& s0, double& s1) {
  __shared__ double sm[kFinLanes][2 * kFinCh];
  const int tid = threadIdx.x, cl = tid % kFinCh, lane = tid / kFinCh, c = c0 + cl < C ? c0 + cl : c0;
  double a = 0.0, b = 0.0;
  // sixteen partials per round (all of them, for up to 512 partials): the loads are independent and unconditional
  // (past the end: the round's first partial again, not added), the sums keep their order; a round costs one trip to
  // memory, and this kernel is nothing but such trips
  constexpr int U = 16;
  for (int p = lane; p < P; p += U * kFinLanes) {
    float v[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned o = (unsigned)(p + kFinLanes * u < P ? p + kFinLanes * u : p) * 2u * C + c;
      v[u][0] = partial[o];
      v[u][1] = partial[o + C];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (p + kFinLanes * u < P) { a += (double)v[u][0]; b += (double)v[u][1]; }
  }
  sm[lane][cl] = a;
  sm[lane][kFinCh + cl] = b;
  __syncthreads();
  s0 = s1 = 0.0;
  if (tid < 64) {                  // sixteen values, four lanes each with eight terms, then across lanes
    const int v = tid & 15, l0 = tid >> 4;
    double t0 = 0.0, t1 = 0.0;
#pragma unroll
    for (int l = 0; l < 8; l += 2) { t0 += sm[l0 * 8 + l][v]; t1 += sm[l0 * 8 + l + 1][v]; }
    t0 += t1;
    t0 += __shfl_xor(t0, 16, 64);
    t0 += __shfl_xor(t0, 32, 64);
    s0 = t0;
    s1 = __shfl_xor(t0, 8, 64);
  }
}

// What the last threads need besides the sums is requested before them.  Means over a step, us a launch (in brackets: all 256 threads added
// all lanes' sums, the parameters were fetched behind them and M was divided by in float64): MobileNetV2 at 32x32, batch 32, fp32 3.3
// (4.0), at 224x224, width 1.4, batch 128, bfloat16 4.7 (4.9); bn_bwd_finalize_k 3.1 (3.7) and 5.0 (5.7).
__global__ __launch_bounds__(256) void bn_finalize_k(const float* __restrict__ partial, int P, double inv_M, double unbias, int C,
                                                     const float* __restrict__ gamma, const float* __restrict__ beta, float* mean, float* invstd,
                                                     float* scale, float* shift, float* run_mean, float* run_var, float eps, float momentum) {
  const int c0 = xcd_logical_block() * kFinCh, tid = threadIdx.x, c = c0 + tid;     // neighbours read the same lines of the partials: one L2
  const bool fin = tid < kFinCh && c < C;
  float p_g = 0.f, p_b = 0.f, p_rm = 0.f, p_rv = 0.f;
  if (fin) { p_g = gamma[c]; p_b = beta[c]; p_rm = run_mean[c]; p_rv = run_var[c]; }
  double s0, s1;
  sum_partials(partial, P, C, c0, s0, s1);
  asm volatile("" : "+v"(p_g), "+v"(p_b), "+v"(p_rm), "+v"(p_rv));      // first use: conversions must not move up to the loads
  if (fin) {
    const double mu = s0 * inv_M;
    double var = s1 * inv_M - mu * mu;
    if (var < 0.0) var = 0.0;
    const double is = rsqrt(var + (double)eps);
    const float sc = (float)((double)p_g * is);
    mean[c] = (float)mu;
    invstd[c] = (float)is;
    scale[c] = sc;
    shift[c] = (float)((double)p_b - mu * (double)sc);
    run_mean[c] = (float)((1.0 - momentum) * p_rm + momentum * mu);
    run_var[c] = (float)((1.0 - momentum) * p_rv + momentum * (var * unbias));
  }
}

void bn_finalize(hipStream_t st, const float* partial, int P, size_t M, int C, const float* gamma,
                 const float* beta, float* mean, float* invstd, float* scale, float* shift,
                 float* run_mean, float* run_var, float eps, float momentum) {
  KScope ks(st, "bn_finalize", (double)P * 2 * C * 4 + 8.0 * C * 4, 0);
  hipLaunchKernelGGL(bn_finalize_k, dim3((C + kFinCh - 1) / kFinCh), dim3(256), 0, st, partial, P, 1.0 / (double)M,
                     M > 1 ? (double)M / (double)(M - 1) : 1.0, C, gamma, beta,
                     mean, invstd, scale, shift, run_mean, run_var, eps, momentum);
}

// ------------------------------------------------------------- bn backward
// dY = dA where the activation (compile-time ACT) passes, else 0
template <int ACT>
__device__ __forceinline__ float act_gate(float d, float z, float sc, float sh) {
  if (ACT == ACT_NONE) return d;
  const float y = fmaf(z, sc, sh);
  if (ACT == ACT_RELU) return y > 0.f ? d : 0.f;
  return (y > 0.f && y < 6.f) ? d : 0.f;
}

#define FTP_DISPATCH_ACT(dt, act, ...)                                        \
  do {                                                                        \
    if ((act) == ACT_NONE) { constexpr int ACT = ACT_NONE; FTP_DISPATCH(dt, __VA_ARGS__); }        \
    else if ((act) == ACT_RELU) { constexpr int ACT = ACT_RELU; FTP_DISPATCH(dt, __VA_ARGS__); }   \
    else { constexpr int ACT = ACT_RELU6; FTP_DISPATCH(dt, __VA_ARGS__); }    \
  } while (0)

template <typename T, int ACT>
__global__ void bn_bwd_reduce_k(const T* __restrict__ dA, const T* __restrict__ z, size_t M, int C,
                                const float* __restrict__ scale, const float* __restrict__ shift,
                                int W, int R, size_t rpb, float* __restrict__ partial) {
  extern __shared__ float smem[];
  __builtin_amdgcn_s_setprio(3);     // data-gradient chain: ahead of the weight-gradient stream's waves on a shared SIMD
  const ChunkSlab at = chunk_slab();
  int tx = threadIdx.x % W, ty = threadIdx.x / W;
  int cg = at.slab * W + tx;
  float acc[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0.f;
  if (cg < C / 8) {
    float sc[8], sh[8];
    load8(scale + cg * 8, sc);
    load8(shift + cg * 8, sh);
    size_t m0 = (size_t)at.chunk * rpb, m1 = m0 + rpb < M ? m0 + rpb : M;
    // four rows per round: the loads are issued together, the sums keep a fixed order
    for (size_t m = m0 + ty; m < m1; m += 4 * (size_t)R) {
      Raw<T> rd[4], rv[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (m + (size_t)u * R < m1) {
          raw_load(rd[u], dA + (m + (size_t)u * R) * C + cg * 8);
          raw_load(rv[u], z + (m + (size_t)u * R) * C + cg * 8);
        }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (m + (size_t)u * R >= m1) break;
        float d[8], v[8];
        raw_unpack(rd[u], d);
        raw_unpack(rv[u], v);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float dy = act_gate<ACT>(d[e], v[e], sc[e], sh[e]);
          acc[e] += dy;
          acc[8 + e] = fmaf(dy, v[e], acc[8 + e]);
        }
      }
    }
  }
  reduce_rows_to_partial(acc, tx, ty, W, R, at.slab * W, C, smem, partial + (size_t)at.chunk * 2 * C);
}

void bn_bwd_reduce(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C,
                   const float* scale, const float* shift, int act, float* partial, int* P_out) {
  RowTile t = make_rowtile(M, C, kBnPartials);
  {
    KScope ks(st, "bn_bwd_reduce", 2.0 * M * C * (dt == 0 ? 4.0 : 2.0), 6.0 * M * C, (long)M, C, act);
    dim3 grid(t.P, t.nslab), block(t.W * t.R);
    size_t sm = (size_t)16 * t.R * t.W * sizeof(float);
    FTP_DISPATCH_ACT(dt, act, hipLaunchKernelGGL((bn_bwd_reduce_k<T, ACT>), grid, block, sm, st, (const T*)dA, (const T*)z, M,
                                                 C, scale, shift, t.W, t.R, t.rows_per_block, partial));
  }
  *P_out = t.P;
}

__global__ __launch_bounds__(256) void bn_bwd_finalize_k(const float* __restrict__ partial, int P, double inv_M, int C,
                                                         const float* __restrict__ gamma, const float* __restrict__ mean,
                                                         const float* __restrict__ invstd, float* g_gamma, float* g_beta, float* coef) {
  // data-gradient chain.  Without this its few waves are the youngest on SIMDs that the weight-gradient stream's
  // long-running waves keep busy, and issue goes to the oldest wave first: measured 190 us instead of 5 next to a
  // persistent weight-gradient kernel
  __builtin_amdgcn_s_setprio(3);
  const int c0 = xcd_logical_block() * kFinCh, tid = threadIdx.x, c = c0 + tid;     // neighbours read the same lines of the partials: one L2
  const bool fin = tid < kFinCh && c < C;
  float p_mu = 0.f, p_is = 0.f, p_g = 0.f, p_gg = 0.f, p_gb = 0.f;
  if (fin) { p_mu = mean[c]; p_is = invstd[c]; p_g = gamma[c]; p_gg = g_gamma[c]; p_gb = g_beta[c]; }
  double s0, s1;
  sum_partials(partial, P, C, c0, s0, s1);
  asm volatile("" : "+v"(p_mu), "+v"(p_is), "+v"(p_g), "+v"(p_gg), "+v"(p_gb));      // first use: see bn_finalize_k
  if (fin) {
    const double mu = p_mu, is = p_is, g = p_g;
    const double dbeta = s0, dgamma = is * (s1 - mu * s0);
    g_gamma[c] = p_gg + (float)dgamma;
    g_beta[c] = p_gb + (float)dbeta;
    const double k1 = g * is, k2 = -k1 * is * dgamma * inv_M, k3 = -k1 * dbeta * inv_M - k2 * mu;
    coef[c] = (float)k1;
    coef[C + c] = (float)k2;
    coef[2 * C + c] = (float)k3;
  }
}

void bn_bwd_finalize(hipStream_t st, const float* partial, int P, size_t M, int C, const float* gamma,
                     const float* mean, const float* invstd, float* g_gamma, float* g_beta, float* coef) {
  KScope ks(st, "bn_bwd_finalize", (double)P * 2 * C * 4 + 10.0 * C * 4, 0);
  hipLaunchKernelGGL(bn_bwd_finalize_k, dim3((C + kFinCh - 1) / kFinCh), dim3(256), 0, st, partial, P, 1.0 / (double)M, C, gamma, mean,
                     invstd, g_gamma, g_beta, coef);
}

// thread = (column group, row lane): coefficients stay in registers, rows advance by R
template <typename T, int ACT>
__global__ void bn_bwd_apply_k(const T* __restrict__ dA, const T* __restrict__ z, size_t M, int C,
                               const float* __restrict__ scale, const float* __restrict__ shift,
                               const float* __restrict__ coef, int W, int R, size_t rpb, T* __restrict__ dz) {
  __builtin_amdgcn_s_setprio(3);     // data-gradient chain: ahead of the weight-gradient stream's waves on a shared SIMD
  const ChunkSlab at = chunk_slab();
  const int tx = threadIdx.x % W, ty = threadIdx.x / W;
  const int cg = at.slab * W + tx;
  if (cg >= C / 8) return;
  const int c = cg * 8;
  float sc[8], sh[8], k1[8], k2[8], k3[8];
  if (ACT != ACT_NONE) { load8(scale + c, sc); load8(shift + c, sh); }
  load8(coef + c, k1); load8(coef + C + c, k2); load8(coef + 2 * C + c, k3);
  const size_t m0 = (size_t)at.chunk * rpb, m1 = m0 + rpb < M ? m0 + rpb : M;
  for (size_t m = m0 + ty; m < m1; m += 2 * (size_t)R) {
    Raw<T> rd[2], rv[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (m + (size_t)u * R < m1) {
        raw_load(rd[u], dA + (m + (size_t)u * R) * C + c);
        raw_load(rv[u], z + (m + (size_t)u * R) * C + c);
      }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (m + (size_t)u * R >= m1) break;
      float d[8], v[8], o[8];
      raw_unpack(rd[u], d);
      raw_unpack(rv[u], v);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float dy = act_gate<ACT>(d[e], v[e], sc[e], sh[e]);
        o[e] = fmaf(k1[e], dy, fmaf(k2[e], v[e], k3[e]));
      }
      store8(dz + (m + (size_t)u * R) * C + c, o);
    }
  }
}

static inline int flat_grid(size_t n, int block) {
  size_t g = (n + block - 1) / block;
  if (g > 65536) g = 65536;
  if (g < 1) g = 1;
  return (int)g;
}

void bn_bwd_apply(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C,
                  const float* scale, const float* shift, int act, const float* coef, void* dz) {
  KScope ks(st, "bn_bwd_apply", 3.0 * M * C * (dt == 0 ? 4.0 : 2.0), 6.0 * M * C, (long)M, C, act);
  const RowTile t = apply_rowtile(M, C);
  dim3 grid(t.P, t.nslab), block(t.W * t.R);
  FTP_DISPATCH_ACT(dt, act, hipLaunchKernelGGL((bn_bwd_apply_k<T, ACT>), grid, block, 0, st, (const T*)dA, (const T*)z, M, C,
                                               scale, shift, coef, t.W, t.R, t.rows_per_block, (T*)dz));
}

// BatchNorm backward for short tensors in ONE launch: a block owns 4 channels over all M rows, so it
// can reduce, finalize and apply without any other block (the three-kernel path needs two grid-wide
// dependencies, i.e. two extra launches, which dominate when the tensor is a few hundred KB).
// Every thread keeps its rows in registers: one trip to memory, then reduce, then apply.
template <typename T, int RPT>
__global__ __launch_bounds__(1024) void bn_bwd_small_k(const T* __restrict__ dA, const T* __restrict__ z, size_t M, int C,
                                                       const float* __restrict__ scale, const float* __restrict__ shift, int act,
                                                       const float* __restrict__ gamma, const float* __restrict__ mean,
                                                       const float* __restrict__ invstd, float* g_gamma, float* g_beta,
                                                       T* __restrict__ dz) {
  __builtin_amdgcn_s_setprio(3);     // data-gradient chain: ahead of the weight-gradient stream's waves on a shared SIMD
  __shared__ float red[16][8];    // [wave][value]
  __shared__ float coef[3][4];
  const int c0 = xcd_logical_block() * 4, tid = threadIdx.x, nt = blockDim.x;   // RPT * nt >= M; neighbours share an XCD
  // requested with the rows: what the four finishing threads need after the reduction
  float f_mu = 0.f, f_is = 0.f, f_g = 0.f, f_gg = 0.f, f_gb = 0.f;
  if (tid < 4) { f_mu = mean[c0 + tid]; f_is = invstd[c0 + tid]; f_g = gamma[c0 + tid]; f_gg = g_gamma[c0 + tid]; f_gb = g_beta[c0 + tid]; }
  float4 d[RPT], v[RPT];
  const double inv_M = early_inverse((double)M);
#pragma unroll
  for (int q = 0; q < RPT; ++q) {       // unconditional, from a clamped row: rows past M are masked where they are used
    const size_t m = tid + (size_t)q * nt, mc = m < M ? m : 0;
    d[q] = load4(dA + mc * C + c0);
    v[q] = load4(z + mc * C + c0);
  }
  float sc[4], sh[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) { sc[e] = scale[c0 + e]; sh[e] = shift[c0 + e]; }
  const float lo = act_lo(act), hi = act_hi(act);
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const float y0 = fmaf(v[q].x, sc[0], sh[0]), y1 = fmaf(v[q].y, sc[1], sh[1]), y2 = fmaf(v[q].z, sc[2], sh[2]),
                y3 = fmaf(v[q].w, sc[3], sh[3]);
    const bool live = tid + (size_t)q * nt < M;
    float4 dy;                              // rows past M count as zeros
    dy.x = (live && y0 > lo && y0 < hi) ? d[q].x : 0.f;
    dy.y = (live && y1 > lo && y1 < hi) ? d[q].y : 0.f;
    dy.z = (live && y2 > lo && y2 < hi) ? d[q].z : 0.f;
    dy.w = (live && y3 > lo && y3 < hi) ? d[q].w : 0.f;
    d[q] = dy;
    acc[0] += dy.x; acc[1] += dy.y; acc[2] += dy.z; acc[3] += dy.w;
    acc[4] = fmaf(dy.x, v[q].x, acc[4]); acc[5] = fmaf(dy.y, v[q].y, acc[5]);
    acc[6] = fmaf(dy.z, v[q].z, acc[6]); acc[7] = fmaf(dy.w, v[q].w, acc[7]);
  }
  // fixed-shape reduction: inside each wave, then the waves in order
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = wave_sum_last(acc[e]);
  const int wave = tid >> 6, nw = nt >> 6;
  if ((tid & 63) == 63) {
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wave][e] = acc[e];
  }
  __syncthreads();
  // first use of the five values requested at the top: their conversions must not move up to the loads
  asm volatile("" : "+v"(f_mu), "+v"(f_is), "+v"(f_g), "+v"(f_gg), "+v"(f_gb));
  if (tid < 4) {
    const int c = c0 + tid;
    double s0 = 0.0, s1 = 0.0;
    for (int w = 0; w < nw; ++w) { s0 += red[w][tid]; s1 += red[w][4 + tid]; }
    const double mu = f_mu, is = f_is, g = f_g;
    const double dbeta = s0, dgamma = is * (s1 - mu * s0);
    g_gamma[c] = f_gg + (float)dgamma;
    g_beta[c] = f_gb + (float)dbeta;
    const double k1 = g * is, k2 = -k1 * is * dgamma * inv_M, k3 = -k1 * dbeta * inv_M - k2 * mu;
    coef[0][tid] = (float)k1; coef[1][tid] = (float)k2; coef[2][tid] = (float)k3;
  }
  __syncthreads();
  const float4 k1 = make_float4(coef[0][0], coef[0][1], coef[0][2], coef[0][3]);
  const float4 k2 = make_float4(coef[1][0], coef[1][1], coef[1][2], coef[1][3]);
  const float4 k3 = make_float4(coef[2][0], coef[2][1], coef[2][2], coef[2][3]);
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const size_t m = tid + (size_t)q * nt;
    if (m >= M) continue;
    store4(dz + m * C + c0, fma4(k1, d[q], fma4(k2, v[q], k3)));
  }
}

int bn_bwd_small_ok(size_t M, int C) { return M <= 2048 && C >= 16 && C % 4 == 0; }

void bn_bwd_small(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C, const float* scale,
                  const float* shift, int act, const float* gamma, const float* mean, const float* invstd,
                  float* g_gamma, float* g_beta, void* dz) {
  KScope ks(st, "bn_bwd_small", 3.0 * M * C * (dt == 0 ? 4.0 : 2.0), 12.0 * M * C, (long)M, C);
  const int nt = M > 512 ? 1024 : (M > 256 ? 512 : 256);
  if (M > 1024) {
    FTP_DISPATCH(dt, hipLaunchKernelGGL((bn_bwd_small_k<T, 2>), dim3(C / 4), dim3(nt), 0, st, (const T*)dA, (const T*)z, M, C, scale,
                                        shift, act, gamma, mean, invstd, g_gamma, g_beta, (T*)dz));
  } else {
    FTP_DISPATCH(dt, hipLaunchKernelGGL((bn_bwd_small_k<T, 1>), dim3(C / 4), dim3(nt), 0, st, (const T*)dA, (const T*)z, M, C, scale,
                                        shift, act, gamma, mean, invstd, g_gamma, g_beta, (T*)dz));
  }
}

// thread = (column group, row lane), rows advance by R as in bn_bwd_apply_k
template <typename T, bool VIEW, bool RES>
__global__ void bn_apply_k(View in, size_t M, int C, const T* __restrict__ res, int W, int R, size_t rpb, T* __restrict__ out) {
  const ChunkSlab at = chunk_slab();
  const int tx = threadIdx.x % W, ty = threadIdx.x / W;
  const int cg = at.slab * W + tx;
  if (cg >= C / 8) return;
  const int c = cg * 8;
  const T* z = reinterpret_cast<const T*>(in.z);
  float sc[8], sh[8];
  if (VIEW) { load8(in.scale + c, sc); load8(in.shift + c, sh); }
  const float lo = act_lo(in.act), hi = act_hi(in.act);
  const size_t m0 = (size_t)at.chunk * rpb, m1 = m0 + rpb < M ? m0 + rpb : M;
  for (size_t m = m0 + ty; m < m1; m += 2 * (size_t)R) {
    Raw<T> rv[2], rr[2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (m + (size_t)u * R < m1) {
        raw_load(rv[u], z + (m + (size_t)u * R) * C + c);
        if (RES) raw_load(rr[u], res + (m + (size_t)u * R) * C + c);
      }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (m + (size_t)u * R >= m1) break;
      float v[8], r[8];
      raw_unpack(rv[u], v);
      if (RES) raw_unpack(rr[u], r);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (VIEW) v[e] = round_to<T>(clamp_act(fmaf(v[e], sc[e], sh[e]), lo, hi));
        if (RES) v[e] += r[e];
      }
      store8(out + (m + (size_t)u * R) * C + c, v);
    }
  }
}

void bn_apply(int dt, hipStream_t st, HView in, size_t M, int C, const void* res, void* out) {
  KScope ks(st, "bn_apply", (res ? 3.0 : 2.0) * M * C * (dt == 0 ? 4.0 : 2.0), 3.0 * M * C);
  const View v{in.z, in.scale, in.shift, in.act};
  const RowTile t = apply_rowtile(M, C);
  const dim3 grid(t.P, t.nslab), block(t.W * t.R);
#define FTP_APPLY(VIEW, RES)                                                                                                  \
  FTP_DISPATCH(dt, hipLaunchKernelGGL((bn_apply_k<T, VIEW, RES>), grid, block, 0, st, v, M, C, (const T*)res, t.W, t.R,       \
                                      t.rows_per_block, (T*)out))
  if (in.scale) { if (res) FTP_APPLY(true, true); else FTP_APPLY(true, false); }
  else { if (res) FTP_APPLY(false, true); else FTP_APPLY(false, false); }
#undef FTP_APPLY
}

// ---- finish and apply in one launch ------------------------------------------------------------------------------
// (rows, slabs) blocks of up to 64 channels: each adds the partial sums of its own channels before it works off its rows, which were
// requested first.  Bound by trips to memory: a finalize launch is some 3.3 us of a chain, the sums here 1.5.
static RowTile finish_rowtile(size_t M, int C) {
  RowTile t;
  const int CG = C / 8;
  t.nslab = (CG + 7) / 8;
  t.W = (CG + t.nslab - 1) / t.nslab;
  t.nslab = (CG + t.W - 1) / t.W;
  t.R = 256 / t.W;
  const size_t round = 2 * (size_t)t.R, rounds = (M + round - 1) / round, per = (rounds * t.nslab + kFinishBlocks - 1) / kFinishBlocks;
  t.rows_per_block = per * round;
  t.P = (int)((M + t.rows_per_block - 1) / t.rows_per_block);
  return t;
}

template <typename T, int ACT>
__global__ __launch_bounds__(256) void bn_bwd_finish_apply_k(const T* __restrict__ dA, const T* __restrict__ z, size_t M, int C,
                                                             const float* __restrict__ scale, const float* __restrict__ shift, BnPending sums,
                                                             float* g_gamma, float* g_beta, int W, int R, size_t rpb, T* __restrict__ dz) {
  __shared__ double red[kSlabSumsBytes / 8];
  __shared__ __attribute__((aligned(16))) float coef[3][64];
  __builtin_amdgcn_s_setprio(3);     // data-gradient chain
  const ChunkSlab at = chunk_slab();
  const int tid = threadIdx.x, tx = tid % W, ty = tid / W, c0 = at.slab * W * 8, nc = C - c0 < W * 8 ? C - c0 : W * 8;
  const bool in = tx * 8 < nc;
  const int c = in ? c0 + tx * 8 : c0;
  const size_t m0 = (size_t)at.chunk * rpb, m1 = m0 + rpb < M ? m0 + rpb : M;
  Raw<T> rd[2], rv[2];
  auto request = [&](const size_t m) __attribute__((always_inline)) {      // past the end: the block's first row, not used
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const size_t mu = m + (size_t)u * R < m1 ? m + (size_t)u * R : m0;
      raw_load(rd[u], dA + mu * C + c);
      raw_load(rv[u], z + mu * C + c);
    }
  };
  request(m0 + ty);
  float sc[8], sh[8], k1[8], k2[8], k3[8];
  if (ACT != ACT_NONE) { load8(scale + c, sc); load8(shift + c, sh); }
  const double inv_M = early_inverse((double)M);
  const int f = c0 + (tid < nc ? tid : 0);
  const bool write = at.chunk == 0 && tid < nc;
  float p_g = sums.gamma[f], p_mu = sums.mean[f], p_is = sums.invstd[f], p_gg = 0.f, p_gb = 0.f;
  if (write) { p_gg = g_gamma[f]; p_gb = g_beta[f]; }
  double s0, s1;
  slab_sums(sums.partial, sums.P, C, c0, nc, red, s0, s1);
  asm volatile("" : "+v"(p_g), "+v"(p_mu), "+v"(p_is), "+v"(p_gg), "+v"(p_gb));      // first use: see bn_finalize_k
  if (tid < nc) {
    const BwdChannel b = backward_channel(s0, s1, p_g, p_mu, p_is, inv_M);
    coef[0][tid] = b.k1; coef[1][tid] = b.k2; coef[2][tid] = b.k3;
    if (write) { g_gamma[f] = p_gg + b.dgamma; g_beta[f] = p_gb + b.dbeta; }
  }
  __syncthreads();
  if (!in) return;
  load8(coef[0] + tx * 8, k1); load8(coef[1] + tx * 8, k2); load8(coef[2] + tx * 8, k3);
  for (size_t m = m0 + ty; m < m1; m += 2 * (size_t)R) {
    if (m != m0 + ty) request(m);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (m + (size_t)u * R >= m1) break;
      float d[8], v[8], o[8];
      raw_unpack(rd[u], d);
      raw_unpack(rv[u], v);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float dy = act_gate<ACT>(d[e], v[e], sc[e], sh[e]);
        o[e] = fmaf(k1[e], dy, fmaf(k2[e], v[e], k3[e]));
      }
      store8(dz + (m + (size_t)u * R) * C + c, o);
    }
  }
}

// Every block reads 512 bytes for each partial: up to 256 of them, and tensors whose blocks run in one turn.  Steps, ms, finalize launches for all / where there are more than
// 200 partials or more values (when the depthwise backward was passes of its own): units 15-18 at 224x224 bfloat16 batch 64 (12 steps) 4.81 / 4.60, 32x32 fp32 (10) 9.58 / 9.47,
// 161x193 width 0.5 bfloat16 (8) 8.91 / 8.79, 224x224 bfloat16 recomputing (4) 12.46 / 12.26, 224x224 fp32 (3) 10.61 / 10.54; with up to 512 partials 10.72 there and 12.41 recomputing,
// width 1.4 batch 128 (4) 29.14 / 29.17 / 29.55, with tensors of up to 64 M values too 30.0.  (The depthwise forward doing the same for its input's BatchNorm took as long as the launch
// it saved.)  With the kernels that stand here, up to 128 / 200 / 256 partials: 32x32 8.89 / 8.98 / 8.82, 97x75 fp32 6.96 / 7.00 / 6.88, 161x193 8.21 / 8.39 / 8.12, recomputing 11.56 /
// 11.55 / 11.47, the others within 0.5 % of each other.  More would need a larger buffer: a layer that leaves sums while it reads others has half of 512.
// Blocks at most (kFinishBlocks) 512 / 1024 / 2048: 32x32 8.78 / 8.82 / 9.01, 97x75 6.88 / 6.88 / 6.98, 224x224 fp32 9.38 / 9.39 / 9.44, 161x193 8.11 / 8.12 / 8.24, the others even.
int bn_finish_ok(size_t M, int C, int P) {
  return P <= 256 && M * (size_t)C <= ((size_t)16 << 20);
}
// P partial sums that a data gradient would leave, against those of a reduction pass: not where only the pass's are few enough to be finished in the layer
// that needs them (width 1.4 at 14x14, batch 128, 88 -> 528: 36 us with sums and the launch to finish them 5, without 21 and the pass 16)
int bn_left_sums_ok(size_t M, int C, int P) {
  return P <= kBnPartials && (bn_finish_ok(M, C, P) || !bn_finish_ok(M, C, make_rowtile(M, C, kBnPartials).P));
}

void bn_bwd_finish_apply(int dt, hipStream_t st, const void* dA, const void* z, size_t M, int C, const float* scale, const float* shift, int act,
                         const BnPending& sums, float* g_gamma, float* g_beta, void* dz) {
  KScope ks(st, "bn_bwd_apply", 3.0 * M * C * (dt == 0 ? 4.0 : 2.0) + (double)sums.P * 2 * C * 4, 6.0 * M * C, (long)M, C, act);
  ks.route("finish");
  const RowTile t = finish_rowtile(M, C);
  const dim3 grid(t.P, t.nslab), block(t.W * t.R);
  FTP_DISPATCH_ACT(dt, act, hipLaunchKernelGGL((bn_bwd_finish_apply_k<T, ACT>), grid, block, 0, st, (const T*)dA, (const T*)z, M, C, scale, shift,
                                               sums, g_gamma, g_beta, t.W, t.R, t.rows_per_block, (T*)dz));
}

// forward: out = act(scale * z + shift) (+ res) from the partial sums of z
template <typename T, bool RES>
__global__ __launch_bounds__(256) void bn_finish_apply_k(BnPending pend, const T* __restrict__ z, size_t M, int C, int act, float eps, float momentum,
                                                         const T* __restrict__ res, int W, int R, size_t rpb, T* __restrict__ out) {
  __shared__ double red[kSlabSumsBytes / 8];
  __shared__ __attribute__((aligned(16))) float vec[2][64];
  const ChunkSlab at = chunk_slab();
  const int tid = threadIdx.x, tx = tid % W, ty = tid / W, c0 = at.slab * W * 8, nc = C - c0 < W * 8 ? C - c0 : W * 8;
  const bool in = tx * 8 < nc;
  const int c = in ? c0 + tx * 8 : c0;
  const size_t m0 = (size_t)at.chunk * rpb, m1 = m0 + rpb < M ? m0 + rpb : M;
  Raw<T> rv[2], rr[2];
  auto request = [&](const size_t m) __attribute__((always_inline)) {      // past the end: the block's first row, not used
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const size_t mu = m + (size_t)u * R < m1 ? m + (size_t)u * R : m0;
      raw_load(rv[u], z + mu * C + c);
      if (RES) raw_load(rr[u], res + mu * C + c);
    }
  };
  request(m0 + ty);
  finish_slab(pend, C, c0, nc, eps, momentum, at.chunk == 0, red, vec[0], vec[1]);
  if (!in) return;
  float sc[8], sh[8];
  load8(vec[0] + tx * 8, sc); load8(vec[1] + tx * 8, sh);
  const float lo = act_lo(act), hi = act_hi(act);
  for (size_t m = m0 + ty; m < m1; m += 2 * (size_t)R) {
    if (m != m0 + ty) request(m);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (m + (size_t)u * R >= m1) break;
      float v[8], r[8];
      raw_unpack(rv[u], v);
      if (RES) raw_unpack(rr[u], r);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        v[e] = round_to<T>(clamp_act(fmaf(v[e], sc[e], sh[e]), lo, hi));
        if (RES) v[e] += r[e];
      }
      store8(out + (m + (size_t)u * R) * C + c, v);
    }
  }
}

void bn_finish_apply(int dt, hipStream_t st, const BnPending& pend, const void* z, size_t M, int C, int act, float eps, float momentum,
                     const void* res, void* out) {
  KScope ks(st, "bn_apply", (res ? 3.0 : 2.0) * M * C * (dt == 0 ? 4.0 : 2.0) + (double)pend.P * 2 * C * 4, 3.0 * M * C);
  ks.route("finish");
  const RowTile t = finish_rowtile(M, C);
  const dim3 grid(t.P, t.nslab), block(t.W * t.R);
  if (res) FTP_DISPATCH(dt, hipLaunchKernelGGL((bn_finish_apply_k<T, true>), grid, block, 0, st, pend, (const T*)z, M, C, act, eps, momentum,
                                               (const T*)res, t.W, t.R, t.rows_per_block, (T*)out));
  else FTP_DISPATCH(dt, hipLaunchKernelGGL((bn_finish_apply_k<T, false>), grid, block, 0, st, pend, (const T*)z, M, C, act, eps, momentum,
                                           (const T*)nullptr, t.W, t.R, t.rows_per_block, (T*)out));
}

// Finish a BatchNorm whose statistics are still partial sums and materialise its output (+ residual) in ONE
// launch, for short tensors: a block owns 4 channels over all rows.
template <typename T>
__global__ __launch_bounds__(1024) void bn_finalize_apply_small_k(BnPending pend, const T* __restrict__ z, size_t M, int C, int act,
                                                                  float eps, float momentum, const T* __restrict__ res,
                                                                  T* __restrict__ out) {
  __shared__ double pre[32][8];
  __shared__ float insc[2][4];
  const int c0 = xcd_logical_block() * 4, tid = threadIdx.x, nt = blockDim.x;
  // the rows of this thread (at most two: M <= 2048 with 1024 threads, else one) and their residuals are requested
  // before the statistics are finished, so the two round trips overlap
  float4 zv[2], rv[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const size_t m = (size_t)tid + (size_t)q * nt, mc = m < M ? m : 0;
    zv[q] = load4(z + mc * C + c0);
    rv[q] = load4((res ? res : z) + mc * C + c0);      // unconditional: without a residual the row itself, not used
  }
  finish_pending4(pend, C, c0, eps, momentum, pre, insc);
  float sc[4], sh[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) { sc[e] = insc[0][e]; sh[e] = insc[1][e]; }
  const float lo = act_lo(act), hi = act_hi(act);
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const size_t m = (size_t)tid + (size_t)q * nt;
    if (m >= M) break;
    float4 v = zv[q];
    v.x = round_to<T>(clamp_act(fmaf(v.x, sc[0], sh[0]), lo, hi));
    v.y = round_to<T>(clamp_act(fmaf(v.y, sc[1], sh[1]), lo, hi));
    v.z = round_to<T>(clamp_act(fmaf(v.z, sc[2], sh[2]), lo, hi));
    v.w = round_to<T>(clamp_act(fmaf(v.w, sc[3], sh[3]), lo, hi));
    if (res) { v.x += rv[q].x; v.y += rv[q].y; v.z += rv[q].z; v.w += rv[q].w; }
    store4(out + m * C + c0, v);
  }
}

int bn_finalize_apply_small_ok(size_t M, int C) { return M <= 2048 && C % 4 == 0; }

void bn_finalize_apply_small(int dt, hipStream_t st, const BnPending& pend, const void* z, size_t M, int C, int act, float eps,
                             float momentum, const void* res, void* out) {
  KScope ks(st, "bn_fin_apply_small", (res ? 3.0 : 2.0) * M * C * (dt == 0 ? 4.0 : 2.0) + (double)pend.P * 2 * C * 4, 3.0 * M * C);
  const int nt = M > 512 ? 1024 : (M > 256 ? 512 : 256);
  FTP_DISPATCH(dt, hipLaunchKernelGGL(bn_finalize_apply_small_k<T>, dim3(C / 4), dim3(nt), 0, st, pend, (const T*)z, M, C, act, eps,
                                      momentum, (const T*)res, (T*)out));
}

// ------------------------------------------------------------------ pooling
// block = (image n, group of 8 channels); 64 lanes walk the positions, U of them on their way together, fixed-order sum through LDS.
// One trip to memory where the image has at most 64 positions, and then U = 1: four requests a lane, three of them for nothing, and the code
// that finishes statistics in every block took 264 x 1792 channels of 9 positions, fp32, from 18.9 to 27.8 us, 73 x 1280 of 4 from 5.8 to 8.3.
// OPEN: also, per image and channel, the number of positions that the activation passes and the sum of the raw values there, open[N][2][C].  Behind an
// average the gradient is the same at all positions, so times these it is that BatchNorm's backward sums, and nobody has to read the tensor for them.
// A lane's sum over more than 64 positions is kept in float64, lanes meet two by two and images in float64: errors of the scale gradient in 2^-24 of the sum's
// r.m.s., fp32, 64 channels, 512 images of 7x7, 100 of 14x14, 16 of 40x40: a pass over the tensor 1.9, 2.0 and 1.8, lanes one behind the other and images in fp32
// 2.5, 2.4 and 3.2, so 1.2, 1.2 and 1.4.
template <typename T, bool PEND, int U, bool OPEN>
__global__ __launch_bounds__(64) void gap_fwd_k(View in, BnPending pend, float eps, float momentum, int N, int HW, int CG, T* __restrict__ out,
                                                float* __restrict__ open) {
  __shared__ float red[64][8];
  __shared__ double fin[64];
  __shared__ float vec[2][8];
  // Neighbouring groups share the lines of an image's rows: on one XCD they are fetched once.  128 images of 7x7, 1792 channels, bfloat16 27.6 -> 17.8 us (26.3 before
  // it left anything for the backward).
  const int i = xcd_logical_block(), n = i / CG, cg = i % CG, lane = threadIdx.x;
  const T* src = reinterpret_cast<const T*>(in.z) + (size_t)n * HW * CG * 8 + cg * 8;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0}, open_n[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  typename std::conditional<(U > 1), double, float>::type open_z[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  float sc[8], sh[8];
  const bool view = in.scale != nullptr;
  Raw<T> r[U];
  auto request = [&](const int p0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) raw_load(r[u], src + (size_t)(p0 + 64 * u < HW ? p0 + 64 * u : 0) * CG * 8);
  };
  request(lane);
  if constexpr (PEND) {
    finish_pending_n(pend, CG * 8, cg * 8, 8, eps, momentum, n == 0, 64, fin, vec[0], vec[1]);
#pragma unroll
    for (int e = 0; e < 8; ++e) { sc[e] = vec[0][e]; sh[e] = vec[1][e]; }
  } else if (view) {
    load8(in.scale + cg * 8, sc);
    load8(in.shift + cg * 8, sh);
  }
  const float lo = act_lo(in.act), hi = act_hi(in.act);
  for (int p0 = lane; p0 < HW; p0 += 64 * U) {
    if (p0 != lane) request(p0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (p0 + 64 * u >= HW) break;
      float v[8];
      raw_unpack(r[u], v);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float y = fmaf(v[e], sc[e], sh[e]);
        acc[e] += view ? round_to<T>(clamp_act(y, lo, hi)) : v[e];
        if constexpr (OPEN) {
          const bool on = y > lo && y < hi;
          open_n[e] += on ? 1.f : 0.f;
          open_z[e] += on ? v[e] : 0.f;
        }
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[lane][e] = acc[e];
  if constexpr (OPEN) {
    float z[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { open_n[e] = wave_sum_last(open_n[e]); z[e] = wave_sum_last((float)open_z[e]); }
    if (lane == 63) {
      float* o = open + (size_t)n * 2 * CG * 8 + cg * 8;
      store8(o, open_n);
      store8(o + CG * 8, z);
    }
  }
  __syncthreads();
  if (lane < 8) {
    float s = 0.f;
    for (int l = 0; l < 64; ++l) s += red[l][lane];
    float o = s * (1.f / (float)HW);
    out[(size_t)i * 8 + lane] = from_f32<T>(o);
  }
}

void gap_fwd(int dt, hipStream_t st, HView in, const BnPending& pend, float eps, float momentum, int N, int HW, int C, void* out, float* open) {
  View v{in.z, in.scale, in.shift, in.act};
  int n = N * (C / 8);
  KScope ks(st, "gap_fwd", ((double)N * HW * C + (double)N * C) * (dt == 0 ? 4.0 : 2.0), 3.0 * N * HW * C);
#define FTP_GAP(PEND, U)                                                                                                                          \
  do {                                                                                                                                            \
    if (open) FTP_DISPATCH(dt, hipLaunchKernelGGL((gap_fwd_k<T, PEND, U, true>), dim3(n), dim3(64), 0, st, v, pend, eps, momentum, N, HW, C / 8, (T*)out, open)); \
    else FTP_DISPATCH(dt, hipLaunchKernelGGL((gap_fwd_k<T, PEND, U, false>), dim3(n), dim3(64), 0, st, v, pend, eps, momentum, N, HW, C / 8, (T*)out, open)); \
  } while (0)
  if (pend.partial) { if (HW <= 64) FTP_GAP(true, 1); else FTP_GAP(true, 4); }
  else if (HW <= 64) FTP_GAP(false, 1);
  else FTP_GAP(false, 4);
#undef FTP_GAP
}

// Blocks from nmain on (sums != nullptr): the backward sums of the BatchNorm in front from what gap_fwd_k has left in open, sums[chunk][2][C] for
// chunks of per images
template <typename T>
__global__ void gap_bwd_k(const T* __restrict__ dOut, size_t nvec, int HW, int CG, T* __restrict__ dIn, int nmain, const float* __restrict__ open,
                          float* __restrict__ sums, int N, int per) {
  float inv = 1.f / (float)HW;
  if ((int)blockIdx.x >= nmain) {
    const int C = CG * 8, nc = (C + 255) / 256, j = blockIdx.x - nmain, c = j % nc * 256 + threadIdx.x, chunk = j / nc;
    const int n0 = chunk * per, n1 = min(n0 + per, N);
    if (c >= C) return;
    double s1 = 0.0, s2 = 0.0;
    for (int n = n0; n < n1; n += 8) {
      float o[8], cnt[8], z[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const size_t nu = n + u < n1 ? n + u : n0;
        o[u] = to_f32(dOut[nu * C + c]);
        cnt[u] = open[nu * 2 * C + c];
        z[u] = open[(nu * 2 + 1) * C + c];
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const float d = round_to<T>(o[u] * inv);          // as stored below
        const bool on = n + u < n1 && cnt[u] > 0.f;       // chosen, not multiplied: an infinite gradient of what is off stays out
        s1 += on ? (double)d * cnt[u] : 0.0;
        s2 += on ? (double)d * z[u] : 0.0;
      }
    }
    sums[((size_t)chunk * 2) * C + c] = (float)s1;
    sums[((size_t)chunk * 2 + 1) * C + c] = (float)s2;
    return;
  }
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += (size_t)nmain * blockDim.x) {
    size_t n = i / ((size_t)HW * CG);
    int cg = (int)(i % CG);
    float v[8];
    load8(dOut + (n * CG + cg) * 8, v);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] *= inv;
    store8(dIn + i * 8, v);
  }
}

void gap_bwd(int dt, hipStream_t st, const void* dOut, int N, int HW, int C, void* dIn, const float* open, float* sums, int* P_out) {
  size_t nvec = (size_t)N * HW * (C / 8);
  const int nmain = flat_grid(nvec, 256), per = N <= 512 ? 8 : (N + 63) / 64, P = (N + per - 1) / per;
  if (sums) *P_out = P;
  KScope ks(st, "gap_bwd", ((double)N * HW * C + (double)N * C) * (dt == 0 ? 4.0 : 2.0), 1.0 * N * HW * C);
  FTP_DISPATCH(dt, hipLaunchKernelGGL(gap_bwd_k<T>, dim3(nmain + (sums ? P * ((C + 255) / 256) : 0)), dim3(256), 0, st,
                                      (const T*)dOut, nvec, HW, C / 8, (T*)dIn, nmain, open, sums, N, per));
}

// ----------------------------------------------------- softmax cross-entropy
__device__ __forceinline__ float block_reduce_256(float v, bool is_max, float* smem) {
  int tid = threadIdx.x;
  smem[tid] = v;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (tid < s) smem[tid] = is_max ? fmaxf(smem[tid], smem[tid + s]) : smem[tid] + smem[tid + s];
    __syncthreads();
  }
  float r = smem[0];
  __syncthreads();
  return r;
}

// Rows too wide for a wavefront's registers: block = row, three passes over it.
template <typename T>
__global__ __launch_bounds__(256) void softmax_ce_k(const T* __restrict__ logits, const int32_t* __restrict__ labels, int B,
                             int classes, float* __restrict__ row_loss, T* __restrict__ dlogits) {
  __shared__ float smem[256];
  int b = blockIdx.x;
  const T* row = logits + (size_t)b * classes;
  float mx = -INFINITY;
  for (int j = threadIdx.x; j < classes; j += 256) mx = fmaxf(mx, to_f32(row[j]));
  mx = block_reduce_256(mx, true, smem);
  float s = 0.f;
  for (int j = threadIdx.x; j < classes; j += 256) s += expf(to_f32(row[j]) - mx);
  s = block_reduce_256(s, false, smem);
  int lab = labels[b];
  const bool lab_ok = lab >= 0 && lab < classes;   // an invalid label yields a NaN loss, never a stray read
  float invB = 1.f / (float)B, invs = 1.f / s;
  for (int j = threadIdx.x; j < classes; j += 256) {
    float p = expf(to_f32(row[j]) - mx) * invs;
    dlogits[(size_t)b * classes + j] = from_f32<T>((p - (j == lab ? 1.f : 0.f)) * invB);
  }
  if (threadIdx.x == 0) row_loss[b] = lab_ok ? -(to_f32(row[lab]) - mx - logf(s)) : NAN;
}

// G lanes (a power of two up to 64) own a row and hold it in registers, E elements each, VEC adjacent ones at a time:
// the logits are read once and the exponentials taken once.  Element e of lane l is column
// (l + G * (e / VEC)) * VEC + e % VEC; AL: every row starts on 16 bytes (without it the same columns are read one by
// one, so the sums and their results do not depend on where the caller's buffers lie).
// op over the G lanes of a group, the same result in all of them: data-parallel-primitive moves inside a row of 16 lanes
// (wave_sum), the rows through readlane or one exchange
template <int G, typename F>
__device__ __forceinline__ float group_all(float x, F op) {
  x = op(x, dpp_move<0xB1>(x));
  x = op(x, dpp_move<0x4E>(x));
  if (G > 4) x = op(x, dpp_move<0x141>(x));
  if (G > 8) x = op(x, dpp_move<0x140>(x));
  if (G == 32) x = op(x, __shfl_xor(x, 16, 64));
  if (G == 64) {
    const int xi = __builtin_bit_cast(int, x);
    const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 0)), r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 16));
    const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 32)), r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 48));
    x = op(op(r0, r1), op(r2, r3));
  }
  return x;
}
template <int G> __device__ __forceinline__ float group_max(float x) { return group_all<G>(x, [](float a, float b) { return fmaxf(a, b); }); }
template <int G> __device__ __forceinline__ float group_sum(float x) { return group_all<G>(x, [](float a, float b) { return a + b; }); }

// exp(t) for t <= 0 (NaN stays NaN), down to the smallest numbers: 2^n times 2^f, n the integer next to t * log2(e) and f what that leaves out, log2(e) in two parts.  Nine
// instructions; probabilities off by 0.615 * 2^-24 of their value, r.m.s., as with expf (0.61, thirteen); 2^(t log2(e)) times one plus a rest was
// eight and 0.74, and zero below 2^-126: 4096 x 1000 bfloat16 7.55 -> 7.67 us.
__device__ __forceinline__ float exp_below(float t) {
  t = t < -150.f ? -150.f : t;                             // zero there; -inf has no rest
  const float n = rintf(t * 1.44269502f);
  const float f = fmaf(t, 1.92596303e-8f, fmaf(t, 1.44269502f, -n));
  return ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

template <typename T, int G, int E, int VEC, bool AL>
struct CeRow {
  float v[E];
  int lab;
  __device__ __forceinline__ void fetch(const T* __restrict__ row, const int32_t* __restrict__ label, int classes, int l) {
    lab = *label;
#pragma unroll
    for (int q = 0; q < E / VEC; ++q) {
      const int c = (l + G * q) * VEC;
      const T* src = row + (c < classes ? c : 0);       // classes % VEC == 0: a vector is in or out
      if constexpr (VEC == 8 && AL) load8(src, v + q * 8);
      else
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[q * VEC + e] = to_f32(src[e]);
    }
  }
  float invs;
  // the row's loss, the same in all its lanes; what is left in v is for store().  WHOLE: the group is a wavefront, so the row, its label and what the
  // columns allow are scalar
  template <bool WHOLE>
  __device__ __forceinline__ float sums(int classes, int l) {
    float mx = -INFINITY, z = 0.f;
#pragma unroll
    for (int q = 0; q < E / VEC; ++q) {
      const int c0 = (l + G * q) * VEC;
      if (!WHOLE || G * VEC * (q + 1) > classes)            // else every lane's vector is in the row
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[q * VEC + e] = c0 < classes ? v[q * VEC + e] : -INFINITY;
#pragma unroll
      for (int e = 0; e < VEC; ++e) mx = fmaxf(mx, v[q * VEC + e]);
    }
    mx = group_max<G>(mx);
    if (WHOLE) lab = __builtin_amdgcn_readfirstlane(lab);
    const int lb = lab;
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < E / VEC; ++q) {
      const int c0 = (l + G * q) * VEC;
      const bool in = WHOLE ? lb >= G * VEC * q && lb < G * VEC * (q + 1) : true;      // the label may lie in one of these vectors
      if (in)
#pragma unroll
        for (int e = 0; e < VEC; ++e) z += c0 + e == lb ? v[q * VEC + e] - mx : 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        // past the row: exp(-inf) = 0; a row of nothing but -inf is NaN as it was
        v[q * VEC + e] = exp_below(v[q * VEC + e] - mx);
        s += v[q * VEC + e];
      }
    }
    s = group_sum<G>(s);
    z = group_sum<G>(z);
    invs = 1.f / s;
    return lb >= 0 && lb < classes ? -(z - logf(s)) : NAN;    // an invalid label yields a NaN loss, never a stray read
  }
  template <bool WHOLE>
  __device__ __forceinline__ void store(T* __restrict__ drow, int classes, int l, float invB) {
    const int lb = WHOLE ? __builtin_amdgcn_readfirstlane(lab) : lab;
#pragma unroll
    for (int q = 0; q < E / VEC; ++q) {
      const int c = (l + G * q) * VEC;
      const bool in = WHOLE ? lb >= G * VEC * q && lb < G * VEC * (q + 1) : true;
      float d[VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) d[e] = v[q * VEC + e] * invs;
      if (in)
#pragma unroll
        for (int e = 0; e < VEC; ++e) d[e] -= c + e == lb ? 1.f : 0.f;
#pragma unroll
      for (int e = 0; e < VEC; ++e) d[e] *= invB;
      if (c >= classes) continue;
      if constexpr (VEC == 8 && AL) store8(drow + c, d);
      else
#pragma unroll
        for (int e = 0; e < VEC; ++e) drow[c + e] = from_f32<T>(d[e]);
    }
  }
};

// Wavefront = row.  Bound by memory: 4096 x 1000 bfloat16 moves 16 MB; a block per row, which goes over its row three
// times with six block-wide reductions between, took 14 us.
// The mean: a block's rows are one partial, and the last block to arrive adds all of them, in order; a launch for it cost as much as the rows where
// they are few (64 x 1000 bfloat16 7.2 us a call, 4.7 so; softmax_ce_arrives has more).  partial and arrived go past the L2s (each
// XCD has its own) one by one: a fence would write a whole L2 back.  Additions to one counter take some 12 ns each, so the blocks arrive in
// kCeGroups groups and the groups at the first counter (563 blocks at one: 3.5 us more).  Whoever arrives last leaves zeros.
// 8 rows a block: with 16 the few rows take 0.6 us more, with 4 the 4096 x 1000 0.5.
template <typename T, int E, int VEC, bool AL>
__global__ __launch_bounds__(kCeRows * 64) void softmax_ce_wave_k(const T* __restrict__ logits, const int32_t* __restrict__ labels, int B, int classes,
                                                                  float* partial, unsigned* arrived, T* __restrict__ dlogits, float* __restrict__ loss) {
  __shared__ float rows[kCeRows];
  constexpr bool WHOLE = VEC > 1;
  const int l = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), b = blockIdx.x * kCeRows + wave;
  CeRow<T, 64, E, VEC, AL> r;
  if (b < B) {
    r.fetch(logits + (size_t)b * classes, labels + b, classes, l);
    const float t = r.template sums<WHOLE>(classes, l);
    if (l == 0) rows[wave] = t;
  } else if (l == 0) {
    rows[wave] = 0.f;
  }
  __syncthreads();
  unsigned before = 0, *const mine = arrived + kCeLine * (1 + blockIdx.x % kCeGroups);
  const unsigned groups = gridDim.x < kCeGroups ? gridDim.x : kCeGroups, members = (gridDim.x - blockIdx.x % kCeGroups + kCeGroups - 1) / kCeGroups;
  if (wave == 0) {
    const float t = wave_sum(l < kCeRows ? rows[l] : 0.f);
    if (l == 0) {
      __hip_atomic_store(partial + blockIdx.x, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // it is there before this block counts as arrived
      before = __hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if (b < B) r.template store<WHOLE>(dlogits + (size_t)b * classes, classes, l, 1.f / (float)B);
  if (wave != 0 || __builtin_amdgcn_readfirstlane(before) + 1 != members) return;
  if (l == 0) {
    __hip_atomic_store(mine, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    before = __hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (__builtin_amdgcn_readfirstlane(before) + 1 != groups) return;
  float s = 0.f;
  for (int i0 = l; i0 < (int)gridDim.x; i0 += 8 * 64) {        // eight loads per trip to memory
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = __hip_atomic_load(partial + (i0 + 64 * u < (int)gridDim.x ? i0 + 64 * u : i0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int u = 0; u < 8; ++u) s += i0 + 64 * u < (int)gridDim.x ? x[u] : 0.f;
  }
  s = wave_sum(s);
  if (l == 0) {
    *loss = s / (float)B;
    __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The rows alone, for a mean in a launch behind.  Four rows a block and nothing between its wavefronts; many long rows in bfloat16 eight, which are read by all before the first is
// written: 16384 x 1000 19.4 -> 18.5 us, 60000 x 1000 52 -> 49.
template <typename T, int E, int VEC, bool AL, int RPB>
__global__ __launch_bounds__(RPB * 64) void softmax_ce_rows_k(const T* __restrict__ logits, const int32_t* __restrict__ labels, int B, int classes,
                                                         float* __restrict__ row_loss, T* __restrict__ dlogits) {
  constexpr bool WHOLE = VEC > 1;
  const int l = threadIdx.x & 63, b = blockIdx.x * RPB + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (RPB == 4 && b >= B) return;
  CeRow<T, 64, E, VEC, AL> r;
  float t = 0.f;
  if (RPB == 4 || b < B) {
    r.fetch(logits + (size_t)b * classes, labels + b, classes, l);
    t = r.template sums<WHOLE>(classes, l);
  }
  if (RPB > 4) {
    __syncthreads();
    if (b >= B) return;
  }
  r.template store<WHOLE>(dlogits + (size_t)b * classes, classes, l, 1.f / (float)B);
  if (l == 0) row_loss[b] = t;
}

// Few elements: one block does all rows and their mean.  Latency only, and a second dependent launch is half of it.
template <typename T, int G, int E>
__global__ __launch_bounds__(1024) void softmax_ce_one_k(const T* __restrict__ logits, const int32_t* __restrict__ labels, int B,
                                                         int classes, T* __restrict__ dlogits, float* __restrict__ loss) {
  enum { ROWS = 1024 / G };
  __shared__ float part[16];
  const int l = threadIdx.x % G, g = threadIdx.x / G;
  const float invB = 1.f / (float)B;
  float sum = 0.f;
  CeRow<T, G, E, 1, false> r, next;
  int b = g;
  const int b0 = b < B ? b : 0;
  r.fetch(logits + (size_t)b0 * classes, labels + b0, classes, l);
  for (; b < B; b += ROWS) {
    const int bn = b + ROWS < B ? b + ROWS : b;
    next.fetch(logits + (size_t)bn * classes, labels + bn, classes, l);     // in flight while this row is worked on
    sum += r.template sums<false>(classes, l);
    r.template store<false>(dlogits + (size_t)b * classes, classes, l, invB);
    r = next;
  }
  sum = wave_sum(l == 0 ? sum : 0.f);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += part[w];
    *loss = t / (float)B;
  }
}

__global__ __launch_bounds__(1024) void mean_rows_k(const float* __restrict__ row_loss, int B, float* __restrict__ loss) {
  __shared__ float part[16];
  const int nt = blockDim.x;
  float s = 0.f;
  for (int i0 = threadIdx.x; i0 < B; i0 += 8 * nt) {        // eight loads per trip to memory
    float x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) x[u] = row_loss[i0 + nt * u < B ? i0 + nt * u : 0];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += i0 + nt * u < B ? x[u] : 0.f;
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
    for (int w = 0; w < nt / 64; ++w) t += part[w];
    *loss = t / (float)B;
  }
}

// The same in the order in which blocks that arrive add: eight rows two by two, a chain over every 64th eight, lanes.  row_loss has a multiple of eight places.
// 64 * U eights at a time.
template <int U>
__global__ __launch_bounds__(1024) void mean_arrived_k(const float* __restrict__ row_loss, int B, float* __restrict__ loss) {
  static_assert(kCeRows == 8, "load8");
  __shared__ float part[64 * U];
  const int tid = threadIdx.x, n = (B + kCeRows - 1) / kCeRows;
  float s = 0.f;
  for (int p0 = 0; p0 < n; p0 += 64 * U) {
    if (p0 > 0) __syncthreads();                                // the eights before have been added
    for (int p = tid; p < 64 * U && p0 + p < n; p += blockDim.x) {
      float r[kCeRows];
      load8(row_loss + (size_t)(p0 + p) * kCeRows, r);
#pragma unroll
      for (int u = 0; u < kCeRows; ++u) r[u] = (p0 + p) * kCeRows + u < B ? r[u] : 0.f;
      part[p] = ((r[0] + r[1]) + (r[2] + r[3])) + ((r[4] + r[5]) + (r[6] + r[7]));
    }
    __syncthreads();
    if (tid < 64) {
      float x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) x[u] = part[tid + 64 * u];    // beyond n: not used
#pragma unroll
      for (int u = 0; u < U; ++u) s += p0 + tid + 64 * u < n ? x[u] : 0.f;
    }
  }
  if (tid >= 64) return;
  s = wave_sum(s);
  if (tid == 0) *loss = s / (float)B;
}

// One block for everything where its lane groups need at most two rounds of short rows (or one of longer ones), else a wavefront per row and the
// mean by the last block or a launch behind.  Measured, us a call (block per row and a mean kernel / one block / wavefront per row and a mean kernel; the last without that
// launch, above): 64 x 100 6.3 / 4.1 / 6.4, 128 x 100 6.3 / 6.4 / 6.4, 16 x 1000 6.4 / 5.3 / 6.4, 32 x 1000 6.4 / 9.0 / 6.4, 4096 x 10 11.4 / 24 / 6.4, 4096 x
// 1000 bfloat16 16.8 / - / 7.8 (on logits that no cache holds 21.8 / - / 9.1), 16384 x 1000 bfloat16 62 / - / 19.
static int ce_lanes(int classes) { return classes <= 16 ? 8 : classes <= 64 ? 16 : classes <= 128 ? 32 : 64; }       // of a row in the one-block kernel
static bool ce_one_block(int B, int classes) { return classes <= 1024 && B <= (classes <= 256 ? 2 : 1) * (1024 / ce_lanes(classes)); }
// Arriving costs a block its wait for the partial and the counters, a launch behind the rows 2 us of the host's time and one of the GPU's.  us a call, arriving / two launches (bound by the host
// up to 6.4 or 7.2, from machine to machine): bfloat16 4096 rows of 40 classes 4.7 / 6.4, 300 6.0 / 6.4, 8192 of 40 5.9 / 6.4, 200 6.9 / 6.5, 300 8.1 / 7.6, 16384 of 40 8.4 / 7.3, 200
// 10.5 / 9.2, 300 12.5 / 11.4; long rows hide it: 1000 classes 4096 rows 7.2 / 7.2, 9000 11.8 / 12.6, 16384 16.2 / 18.5, 60000 45 / 49, fp32 even.  In captured calls, which have no counters,
// two launches take 4.0 (600 x 40), 4.5 (4096 x 40), 5.7 (4096 x 300) and 10.6 (7000 x 1000).
int softmax_ce_arrives(int B, int classes) {
  return !ce_one_block(B, classes) && classes <= 1024 && (classes > 512 || B <= 4096 || (classes <= 256 && B <= 8192));
}

template <typename T>
static void softmax_ce_launch(hipStream_t st, const T* logits, const int32_t* labels, int B, int classes, float* row_loss, T* dlogits,
                              float* loss, unsigned* arrived) {
  if (ce_one_block(B, classes)) {
#define FTP_CE_ONE(G, E) hipLaunchKernelGGL((softmax_ce_one_k<T, G, E>), dim3(1), dim3(1024), 0, st, logits, labels, B, classes, dlogits, loss)
    if (classes <= 16) FTP_CE_ONE(8, 2);
    else if (classes <= 32) FTP_CE_ONE(16, 2);
    else if (classes <= 64) FTP_CE_ONE(16, 4);
    else if (classes <= 128) FTP_CE_ONE(32, 4);
    else if (classes <= 256) FTP_CE_ONE(64, 4);
    else if (classes <= 512) FTP_CE_ONE(64, 8);
    else FTP_CE_ONE(64, 16);
#undef FTP_CE_ONE
    return;
  }
  const bool al = ((uintptr_t)logits | (uintptr_t)dlogits) % 16 == 0;      // the buffers are the caller's
  const int mean_threads = B <= 2048 ? 256 : 1024;
  if (classes > 1024) {
    hipLaunchKernelGGL(softmax_ce_k<T>, dim3(B), dim3(256), 0, st, logits, labels, B, classes, row_loss, dlogits);
    hipLaunchKernelGGL(mean_rows_k, dim3(1), dim3(mean_threads), 0, st, row_loss, B, loss);
    return;
  }
  const bool may = softmax_ce_arrives(B, classes), arrives = may && arrived;
  const bool wide = sizeof(T) == 2 && classes > 256 && B > 4096;             // eight rows a block, see softmax_ce_rows_k
#define FTP_CE_WAVE(E, VEC, AL)                                                                                                                                  \
  do {                                                                                                                                                           \
    if (arrives) hipLaunchKernelGGL((softmax_ce_wave_k<T, E, VEC, AL>), dim3((B + kCeRows - 1) / kCeRows), dim3(kCeRows * 64), 0, st, logits, labels, B, classes, \
                                    row_loss, arrived, dlogits, loss);                                                                                           \
    else if (wide) hipLaunchKernelGGL((softmax_ce_rows_k<T, E, VEC, AL, (sizeof(T) == 2 && E > 4 ? 8 : 4)>), dim3((B + 7) / 8), dim3(512), 0, st, logits, labels, B, \
                                      classes, row_loss, dlogits);                                                                                               \
    else hipLaunchKernelGGL((softmax_ce_rows_k<T, E, VEC, AL, 4>), dim3((B + 3) / 4), dim3(256), 0, st, logits, labels, B, classes, row_loss, dlogits);          \
  } while (0)
#define FTP_CE_WAVE8(E) do { if (al) FTP_CE_WAVE(E, 8, true); else FTP_CE_WAVE(E, 8, false); } while (0)
  if (classes % 8 == 0 && classes > 256) { if (classes <= 512) FTP_CE_WAVE8(8); else FTP_CE_WAVE8(16); }
  else if (classes <= 64) FTP_CE_WAVE(1, 1, false);
  else if (classes <= 128) FTP_CE_WAVE(2, 1, false);
  else if (classes <= 256) FTP_CE_WAVE(4, 1, false);
  else if (classes <= 512) FTP_CE_WAVE(8, 1, false);
  else FTP_CE_WAVE(16, 1, false);
#undef FTP_CE_WAVE8
#undef FTP_CE_WAVE
  if (arrives) return;
  if (may && B <= 1024) hipLaunchKernelGGL(mean_arrived_k<2>, dim3(1), dim3((B + 511) / 512 * 64), 0, st, row_loss, B, loss);        // no counters: bit for bit the same
  else if (may) hipLaunchKernelGGL(mean_arrived_k<16>, dim3(1), dim3(B > 7680 ? 1024 : (B + 511) / 512 * 64), 0, st, row_loss, B, loss);
  else hipLaunchKernelGGL(mean_rows_k, dim3(1), dim3(mean_threads), 0, st, row_loss, B, loss);
}

void softmax_ce(int dt, hipStream_t st, const void* logits, const int32_t* labels, int B, int classes,
                float* row_loss, void* dlogits, float* loss, unsigned* arrived) {
  KScope ks(st, "softmax_ce", 2.0 * B * classes * (dt == 0 ? 4.0 : 2.0), 8.0 * B * classes);
  if (softmax_ce_arrives(B, classes)) ks.route(arrived ? "arrival" : "two launches");
  FTP_DISPATCH(dt, softmax_ce_launch<T>(st, (const T*)logits, labels, B, classes, row_loss, (T*)dlogits, loss, arrived));
}

// block = 16 output columns x 16 row lanes; the row lanes' sums meet in LDS in a fixed order
template <typename T>
__global__ __launch_bounds__(256) void bias_grad_k(const T* __restrict__ d, int B, int Nout, float* __restrict__ g) {
  __shared__ float red[16][17];
  const int jl = threadIdx.x & 15, lane = threadIdx.x >> 4;
  const int j = blockIdx.x * 16 + jl;
  float s = 0.f;
  if (j < Nout)
    for (int b = lane; b < B; b += 16) s += to_f32(d[(size_t)b * Nout + j]);
  red[lane][jl] = s;
  __syncthreads();
  if (lane == 0 && j < Nout) {
    float t = 0.f;
#pragma unroll
    for (int l = 0; l < 16; ++l) t += red[l][jl];
    g[j] += t;
  }
}

void bias_grad(int dt, hipStream_t st, const void* d, int B, int Nout, float* g_bias) {
  KScope ks(st, "bias_grad", (double)B * Nout * (dt == 0 ? 4.0 : 2.0) + 8.0 * Nout, 1.0 * B * Nout);
  FTP_DISPATCH(dt, hipLaunchKernelGGL(bias_grad_k<T>, dim3((Nout + 15) / 16), dim3(256), 0, st, (const T*)d, B, Nout, g_bias));
}

// -------------------------------------------------------------------- SGD
__global__ void sgd_update_k(float* __restrict__ w, float* __restrict__ g, float* __restrict__ v,
                             bf16_t* __restrict__ w_lp, size_t n, float lr, float mu, float wd) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    float wi = w[i];
    float gi = fmaf(wd, wi, g[i]);
    float vi = fmaf(mu, v[i], gi);
    wi = fmaf(-lr, vi, wi);
    w[i] = wi;
    v[i] = vi;
    g[i] = 0.f;
    if (w_lp) w_lp[i] = f32_to_bf16(wi);
  }
}

void sgd_update(hipStream_t st, float* w, float* g, float* v, void* w_lp, size_t n, float lr, float mu,
                float wd) {
  KScope ks(st, "sgd_update", (w_lp ? 26.0 : 24.0) * n, 6.0 * n);
  hipLaunchKernelGGL(sgd_update_k, dim3(flat_grid(n, 256)), dim3(256), 0, st, w, g, v, (bf16_t*)w_lp, n, lr,
                     mu, wd);
}

// w[i] = (src[0][i] + src[1][i] + ... ) / n, summed in the order given; optional bfloat16 copy
__global__ void aggregate_k(float* __restrict__ w, bf16_t* __restrict__ w_lp, AggSources src, int n, size_t count) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x) {
    float acc = src.p[0][i];
    for (int j = 1; j < n; ++j) acc += src.p[j][i];
    acc = acc / (float)n;
    w[i] = acc;
    if (w_lp) w_lp[i] = from_f32<bf16_t>(acc);
  }
}

void aggregate_weights(hipStream_t st, float* w, void* w_lp, const AggSources& src, int n, size_t count) {
  KScope ks(st, "aggregate", (double)count * (4.0 * (n + 1) + (w_lp ? 2.0 : 0.0)), (double)count * n);
  hipLaunchKernelGGL(aggregate_k, dim3(flat_grid(count, 256)), dim3(256), 0, st, w, (bf16_t*)w_lp, src, n, count);
}

__global__ void fill_zero_k(uint32_t* p, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

void fill_zero(hipStream_t st, void* p, size_t bytes) {
  KScope ks(st, "fill_zero", (double)bytes, 0);
  size_t n = (bytes + 3) / 4;  // buffers are allocated in multiples of 256 bytes
  hipLaunchKernelGGL(fill_zero_k, dim3(flat_grid(n, 256)), dim3(256), 0, st, (uint32_t*)p, n);
}

// plain 16-byte-per-thread copy of known size: the yardstick hardware traffic counters are scaled by
__global__ void calibration_copy_k(const uint4* __restrict__ src, uint4* __restrict__ dst, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

void calibration_copy(hipStream_t st, const void* src, void* dst, size_t bytes) {
  size_t n = bytes / 16;
  KScope ks(st, "calibration_copy", 2.0 * n * 16, 0);
  hipLaunchKernelGGL(calibration_copy_k, dim3(flat_grid(n, 256)), dim3(256), 0, st, (const uint4*)src, (uint4*)dst, n);
}

template <typename T>
__global__ void f32_to_storage_k(const float* __restrict__ src, T* __restrict__ dst, size_t n) {
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
    dst[i] = from_f32<T>(src[i]);
}

void f32_to_storage(int dt, hipStream_t st, const float* src, void* dst, size_t n) {
  KScope ks(st, "f32_to_storage", (4.0 + (dt == 0 ? 4.0 : 2.0)) * n, 0);
  FTP_DISPATCH(dt, hipLaunchKernelGGL(f32_to_storage_k<T>, dim3(flat_grid(n, 256)), dim3(256), 0, st, src,
                                      (T*)dst, n));
}

}  // namespace ftp
