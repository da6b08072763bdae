// Device helper shared by the short-tensor kernels: finishing BatchNorm statistics that a producer left as
// partial sums, for the four channels a block owns.
#pragma once
#include "dev_common.h"
#include "kernels.h"

namespace ftp {

// one channel from its sum and second sum; write: also the vectors and running statistics in memory
__device__ __forceinline__ void finish_channel(const BnPending& pend, double inv_M, int c, double s0, double s1, float p_g, float p_b, float p_rm,
                                               float p_rv, float eps, float momentum, bool write, float& scv, float& shv) {
  const double mu = s0 * inv_M;
  double var = s1 * inv_M - mu * mu;
  if (var < 0.0) var = 0.0;
  const double is = rsqrt(var + (double)eps);
  scv = (float)((double)p_g * is);
  shv = (float)((double)p_b - mu * (double)scv);
  if (!write) return;
  pend.mean[c] = (float)mu;
  pend.invstd[c] = (float)is;
  pend.scale[c] = scv;
  pend.shift[c] = shv;
  const double unb = pend.M > 1 ? var / (1.0 - inv_M) : var;
  pend.run_mean[c] = (float)((1.0 - momentum) * p_rm + momentum * mu);
  pend.run_var[c] = (float)((1.0 - momentum) * p_rv + momentum * unb);
}

// The same for nc channels from c0 (2 * nc <= nt threads of the block), by every block that reads the tensor: a few dozen
// partials, which cost each of them one trip to memory where a launch of its own costs three (64 partials x 64 channels: 1.4 us
// more per consumer, the launch was 4.1 and the gap in front of it 1.5).  red: nt doubles, sc / sh: [nc].
// One block per channel (write) leaves the vectors and running statistics in memory; the others only use them.
__device__ __forceinline__ void finish_pending_n(const BnPending& pend, int C, int c0, int nc, float eps, float momentum, bool write, int nt,
                                                 double* red, float* sc, float* sh) {
  const int tid = threadIdx.x, nv = 2 * nc, L = nt / nv, v = tid % nv, lane = tid / nv;
  float p_g = 0.f, p_b = 0.f, p_rm = 0.f, p_rv = 0.f;
  const double inv_M = early_inverse((double)pend.M);
  if (tid < nc) { p_g = pend.gamma[c0 + tid]; p_b = pend.beta[c0 + tid]; p_rm = pend.run_mean[c0 + tid]; p_rv = pend.run_var[c0 + tid]; }
  double t = 0.0;
  if (lane < L) {
    const float* src = pend.partial + (size_t)(v >= nc ? C : 0) + c0 + (v >= nc ? v - nc : v);
    for (int q0 = lane; q0 < pend.P; q0 += 16 * L) {
      float x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = src[(size_t)(q0 + u * L < pend.P ? q0 + u * L : lane) * 2 * C];
#pragma unroll
      for (int u = 0; u < 16; ++u) t += q0 + u * L < pend.P ? (double)x[u] : 0.0;
    }
    red[lane * nv + v] = t;
  }
  __syncthreads();
  asm volatile("" : "+v"(p_g), "+v"(p_b), "+v"(p_rm), "+v"(p_rv));       // see finish_pending4
  if (tid < nc) {
    double s0 = 0.0, s1 = 0.0;
    for (int l = 0; l < L; ++l) { s0 += red[l * nv + tid]; s1 += red[l * nv + nc + tid]; }
    finish_channel(pend, inv_M, c0 + tid, s0, s1, p_g, p_b, p_rm, p_rv, eps, momentum, write, sc[tid], sh[tid]);
  }
  __syncthreads();
}

// The backward counterpart, for all C channels (2 * C <= nt): from sums of dY and dY * z, coef[0..2][c] with dz = k1 * dY + k2 * z + k3.
// sums: partial, P, M, gamma, mean, invstd; one block (write) adds to g_gamma and g_beta.
__device__ __forceinline__ void finish_backward_n(const BnPending& sums, int C, float* g_gamma, float* g_beta, bool write, int nt, double* red,
                                                  float (*coef)[64]) {
  const int tid = threadIdx.x, nv = 2 * C, L = nt / nv, v = tid % nv, lane = tid / nv;
  const double inv_M = early_inverse((double)sums.M);
  const int c = tid < C ? tid : 0;
  float p_g = sums.gamma[c], p_mu = sums.mean[c], p_is = sums.invstd[c], p_gg = g_gamma[c], p_gb = g_beta[c];
  double t = 0.0;
  if (lane < L) {
    const float* src = sums.partial + v;
    for (int q0 = lane; q0 < sums.P; q0 += 16 * L) {
      float x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = src[(size_t)(q0 + u * L < sums.P ? q0 + u * L : lane) * 2 * C];
#pragma unroll
      for (int u = 0; u < 16; ++u) t += q0 + u * L < sums.P ? (double)x[u] : 0.0;
    }
    red[lane * nv + v] = t;
  }
  __syncthreads();
  asm volatile("" : "+v"(p_g), "+v"(p_mu), "+v"(p_is), "+v"(p_gg), "+v"(p_gb));       // see finish_pending4
  if (tid < C) {
    double s0 = 0.0, s1 = 0.0;
#pragma unroll 4
    for (int l = 0; l < L; ++l) { s0 += red[l * nv + tid]; s1 += red[l * nv + C + tid]; }
    const double mu = p_mu, is = p_is, k1 = (double)p_g * is, dgamma = is * (s1 - mu * s0);
    const double k2 = -k1 * is * dgamma * inv_M, k3 = -k1 * s0 * inv_M - k2 * mu;
    coef[0][c] = (float)k1; coef[1][c] = (float)k2; coef[2][c] = (float)k3;
    if (write) { g_gamma[c] = p_gg + (float)dgamma; g_beta[c] = p_gb + (float)s0; }
  }
  __syncthreads();
}

enum { kSlabSumsBytes = 1024 * 8 };      // slab_sums' red, blocks of 256 threads
// Column sums of partial[P][2][C] for the nc channels from c0 (multiples of 4), by every block of a kernel that is cut into slabs of
// up to 64 channels: 16-byte loads, all of a thread's (up to 16) on their way together, float64 sums in a fixed order.  red: four doubles a
// thread, at most 32 a channel; on return thread t < nc has its channel's two sums (behind a barrier; red may be used again after another).
__device__ __forceinline__ void slab_sums(const float* __restrict__ partial, int P, int C, int c0, int nc, double* red, double& s0, double& s1) {
  const int tid = threadIdx.x, n4 = nc >> 2, nv = 2 * n4, most = (int)blockDim.x / nv, L = most < 16 ? most : 16, lane = tid / nv, v = tid - lane * nv;
  if (lane < L) {
    const float* src = partial + (v < n4 ? c0 + 4 * v : C + c0 + 4 * (v - n4));
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    for (int q0 = lane; q0 < P; q0 += 16 * L) {
      float4 x[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) x[u] = ld4(src + (size_t)(q0 + u * L < P ? q0 + u * L : q0) * 2 * C);
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (q0 + u * L < P) { t[0] += (double)x[u].x; t[1] += (double)x[u].y; t[2] += (double)x[u].z; t[3] += (double)x[u].w; }
    }
    double* r = red + (size_t)lane * 2 * nc + 4 * v;
    r[0] = t[0]; r[1] = t[1]; r[2] = t[2]; r[3] = t[3];
  }
  __syncthreads();
  s0 = s1 = 0.0;
  if (tid < nc) {
#pragma unroll 4
    for (int l = 0; l < L; ++l) { s0 += red[(size_t)l * 2 * nc + tid]; s1 += red[(size_t)l * 2 * nc + nc + tid]; }
  }
}

// finish pending BatchNorm statistics for nc channels from c0 by every block that reads them (see slab_sums); write: one block per channel also
// leaves the vectors and running statistics in memory.  sc / sh: [nc], behind a barrier.
__device__ __forceinline__ void finish_slab(const BnPending& pend, int C, int c0, int nc, float eps, float momentum, bool write, double* red,
                                            float* sc, float* sh) {
  const int tid = threadIdx.x, f = c0 + (tid < nc ? tid : 0);
  const double inv_M = early_inverse((double)pend.M);
  float p_g = pend.gamma[f], p_b = pend.beta[f], p_rm = 0.f, p_rv = 0.f;
  if (write && tid < nc) { p_rm = pend.run_mean[f]; p_rv = pend.run_var[f]; }
  double s0, s1;
  slab_sums(pend.partial, pend.P, C, c0, nc, red, s0, s1);
  asm volatile("" : "+v"(p_g), "+v"(p_b), "+v"(p_rm), "+v"(p_rv));       // see finish_pending4
  if (tid < nc) finish_channel(pend, inv_M, f, s0, s1, p_g, p_b, p_rm, p_rv, eps, momentum, write, sc[tid], sh[tid]);
  __syncthreads();
}

// one channel's backward from its sums of dY and dY * z: dz = k1 * dY + k2 * z + k3
struct BwdChannel { float k1, k2, k3, dgamma, dbeta; };
__device__ __forceinline__ BwdChannel backward_channel(double s0, double s1, double gamma, double mu, double is, double inv_M) {
  const double k1 = gamma * is, dgamma = is * (s1 - mu * s0), k2 = -k1 * is * dgamma * inv_M, k3 = -k1 * s0 * inv_M - k2 * mu;
  return BwdChannel{(float)k1, (float)k2, (float)k3, (float)dgamma, (float)s0};
}

// finish pending BatchNorm statistics for channels c0..c0+3 (first 256 threads), result in insc[2][4]
__device__ __forceinline__ void finish_pending4(const BnPending& pend, int C, int c0, float eps, float momentum, double (*pre)[8],
                                                float (*insc)[4]) {
  const int tid = threadIdx.x;
  // what the last four threads need at the end is requested now, and the partials four at a time from clamped
  // addresses: this runs at the head of kernels that are a chain of memory round trips and little else
  float p_g = 0.f, p_b = 0.f, p_rm = 0.f, p_rv = 0.f;
  const double inv_M = early_inverse((double)pend.M);
  if (tid < 4) { p_g = pend.gamma[c0 + tid]; p_b = pend.beta[c0 + tid]; p_rm = pend.run_mean[c0 + tid]; p_rv = pend.run_var[c0 + tid]; }
  if (tid < 256) {
    const int v = tid & 7, lane = tid >> 3;           // 4 sums, 4 second sums; 32 lanes each
    double t = 0.0;
    for (int q0 = lane; q0 < pend.P; q0 += 128) {
      float x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = q0 + 32 * u;
        x[u] = pend.partial[((size_t)(q < pend.P ? q : 0) * 2 + (v >> 2)) * C + c0 + (v & 3)];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) t += q0 + 32 * u < pend.P ? (double)x[u] : 0.0;
    }
    pre[lane][v] = t;
  }
  __syncthreads();
  // the first wavefront: eight lanes a value with four sums each, then across lanes (the same tree for every call)
  double s0 = 0.0, s1 = 0.0;
  if (tid < 64) {
    const double* f = &pre[0][0] + tid;
    double t = (f[0] + f[64]) + (f[128] + f[192]);
#pragma unroll
    for (int o = 8; o < 64; o <<= 1) t += __shfl_xor(t, o, 64);
    s0 = t;
    s1 = __shfl_xor(t, 4, 64);                       // lanes 0..3 hold the sums, 4..7 the second sums
  }
  // first use of the four values requested at the top: their conversions must not move up to the loads
  asm volatile("" : "+v"(p_g), "+v"(p_b), "+v"(p_rm), "+v"(p_rv));
  if (tid < 4) {
    const int c = c0 + tid;
    finish_channel(pend, inv_M, c, s0, s1, p_g, p_b, p_rm, p_rv, eps, momentum, true, insc[0][tid], insc[1][tid]);
  }
  __syncthreads();
}

}  // namespace ftp
