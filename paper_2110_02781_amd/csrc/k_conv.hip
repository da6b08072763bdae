// Small dense convolutions (3x3 stem, conv1d) and depthwise 3x3, NHWC.
// Inputs are read through a View, so the producer's BatchNorm + activation is
// applied on load and zero padding is inserted after it (a halo cell is 0, not
// act(bn(0))).  Depthwise layers over short tensors (at most 2048 pixels) run whole
// forward / backward sub-chains in one launch (dw_fwd_bn_small_k, dw_bwd_small_k).
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

// g[(j % C) * stride_c + (j / C) * stride_q] += sum_p ws[p * QC + j]   (float64 sum, fixed order)
__global__ void reduce_partials_flat_k(const float* __restrict__ ws, int P, size_t QC, int C, size_t stride_q,
                                       size_t stride_c, int valid_c, float* __restrict__ g) {
  size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= QC || (int)(j % C) >= valid_c) return;
  double s = 0.0;
  for (int p = 0; p < P; ++p) s += (double)ws[(size_t)p * QC + j];
  size_t o = (j % C) * stride_c + (j / C) * stride_q;
  g[o] += (float)s;
}

// many partials: 16 outputs per block, 16 lanes share the partials of one output
__global__ void reduce_partials_wide_k(const float* __restrict__ ws, int P, size_t QC, int C, size_t stride_q,
                                       size_t stride_c, int valid_c, float* __restrict__ g) {
  __shared__ double sm[16][17];
  const int jl = threadIdx.x & 15, lane = threadIdx.x >> 4;
  const size_t j = (size_t)xcd_logical_block() * 16 + jl;     // neighbours read the same lines of the partials: one L2
  double s = 0.0;
  if (j < QC) {
    int p = lane;
    // many partials: sixteen independent loads per round (a round is one trip to memory, and this kernel is nothing but
    // such trips); the sums keep their order
    for (; p + 240 < P; p += 256) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = ws[(size_t)(p + 16 * u) * QC + j];
#pragma unroll
      for (int u = 0; u < 16; ++u) s += (double)v[u];
    }
    for (; p + 48 < P; p += 64) {        // four independent loads per round
      float a = ws[(size_t)p * QC + j], b = ws[(size_t)(p + 16) * QC + j];
      float c2 = ws[(size_t)(p + 32) * QC + j], d = ws[(size_t)(p + 48) * QC + j];
      s += (double)a; s += (double)b; s += (double)c2; s += (double)d;
    }
    for (; p < P; p += 16) s += (double)ws[(size_t)p * QC + j];
  }
  sm[lane][jl] = s;
  __syncthreads();
  if (lane == 0 && j < QC && (int)(j % C) < valid_c) {
    double t = 0.0;
#pragma unroll
    for (int l = 0; l < 16; ++l) t += sm[l][jl];
    size_t o = (j % C) * stride_c + (j / C) * stride_q;
    g[o] += (float)t;
  }
}

// columns (j % C) >= valid_c are padding and are skipped
void reduce_partials(hipStream_t st, const float* ws, int P, size_t QC, int C, size_t stride_q,
                     size_t stride_c, float* g, int valid_c) {
  if (valid_c < 0) valid_c = C;
  KScope ks(st, "reduce_partials", ((double)P + 2.0) * QC * 4, (double)P * QC);
  if (P <= 8)
    hipLaunchKernelGGL(reduce_partials_flat_k, dim3((unsigned)((QC + 255) / 256)), dim3(256), 0, st, ws, P, QC, C,
                       stride_q, stride_c, valid_c, g);
  else
    hipLaunchKernelGGL(reduce_partials_wide_k, dim3((unsigned)((QC + 15) / 16)), dim3(256), 0, st, ws, P, QC, C,
                       stride_q, stride_c, valid_c, g);
}

// Several tensors' partials in one launch: a block takes 16 outputs with 16 lanes each (many partials) or 256 outputs (up to
// 16 partials).  A launch per tensor was 3-10 us, most of it ramp, a trip or two to memory and tail.
enum { kReduceJobs = 64 };
struct ReduceGroup { ReduceJob job[kReduceJobs]; int blk0[kReduceJobs + 1]; int n; };
__global__ __launch_bounds__(256) void reduce_group_k(ReduceGroup a) {
  __shared__ double sm[16][17];
  int b0;
  const ReduceJob r = a.job[group_job(a.blk0, a.n, b0)];
  const size_t QC = r.QC;
  if (r.P <= 16) {
    const int j = b0 * 256 + threadIdx.x;
    if (j >= r.QC) return;
    float v[16];
#pragma unroll
    for (int p = 0; p < 16; ++p) v[p] = r.ws[(p < r.P ? (size_t)p * QC : 0) + j];
    const int q = j / r.C, c = j - q * r.C;
    if (c >= r.valid_c) return;
    float* dst = r.g + (size_t)c * r.stride_c + (size_t)q * r.stride_q;
    const float old = *dst;
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < 16; ++p) s += p < r.P ? (double)v[p] : 0.0;
    *dst = old + (float)s;
    return;
  }
  const int jl = threadIdx.x & 15, lane = threadIdx.x >> 4, j = b0 * 16 + jl;
  double s = 0.0;
  if (j < r.QC) {
    for (int p0 = lane; p0 < r.P; p0 += 128) {          // eight loads a trip, past the end the first one again (not added)
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = r.ws[(size_t)(p0 + 16 * u < r.P ? p0 + 16 * u : lane) * QC + j];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += p0 + 16 * u < r.P ? (double)v[u] : 0.0;
    }
  }
  sm[lane][jl] = s;
  __syncthreads();
  if (lane == 0 && j < r.QC) {
    const int q = j / r.C, c = j - q * r.C;
    if (c < r.valid_c) {
      double t = 0.0;
#pragma unroll
      for (int l = 0; l < 16; ++l) t += sm[l][jl];
      r.g[(size_t)c * r.stride_c + (size_t)q * r.stride_q] += (float)t;
    }
  }
}

void reduce_group(hipStream_t st, const ReduceJob* jobs, int n) {
  while (n > 0) {
    ReduceGroup a{};
    double bytes = 0, flops = 0;
    int blocks = 0;
    for (a.n = 0; a.n < n && a.n < kReduceJobs; ++a.n) {
      const ReduceJob& r = jobs[a.n];
      a.job[a.n] = r;
      a.blk0[a.n] = blocks;
      blocks += ((r.P <= 16 ? (r.QC + 255) / 256 : (r.QC + 15) / 16) + 7) / 8 * 8;
      bytes += (r.P + 2.0) * r.QC * 4;
      flops += (double)r.P * r.QC;
    }
    a.blk0[a.n] = blocks;
    KScope ks(st, "reduce_partials", bytes, flops);
    hipLaunchKernelGGL(reduce_group_k, dim3(blocks), dim3(256), 0, st, a);
    jobs += a.n; n -= a.n;
  }
}

// ======================================================== generic direct conv
static const int kWChunkFloats = 8192;  // LDS weight chunk: 32 KB

int conv_direct_supported(const ConvGeom& g) {
  return g.Cout % 8 == 0 && g.Cout <= 1024 && (size_t)g.Cin * g.Cout <= (size_t)kWChunkFloats;
}

// thread = (output pixel, 8 output channels); weights of a few taps at a time in LDS as [k][Cout]
template <typename T>
__global__ void conv_direct_fwd_k(View in, const T* __restrict__ w, ConvGeom g, int TC, int PPB,
                                  T* __restrict__ z) {
  extern __shared__ float wl[];
  const int CGo = g.Cout / 8;
  const int pl = threadIdx.x / CGo, cg = threadIdx.x % CGo;
  const size_t total = (size_t)g.N * g.Hout * g.Wout;
  const size_t pix = (size_t)blockIdx.x * PPB + pl;
  const bool valid = pix < total;
  int n = 0, ho = 0, wo = 0;
  if (valid) {
    wo = (int)(pix % g.Wout);
    size_t r = pix / g.Wout;
    ho = (int)(r % g.Hout);
    n = (int)(r / g.Hout);
  }
  const int ntaps = g.kh * g.kw, K = ntaps * g.Cin;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int t0 = 0; t0 < ntaps; t0 += TC) {
    const int tcnt = ntaps - t0 < TC ? ntaps - t0 : TC;
    const int kc = tcnt * g.Cin;
    __syncthreads();
    for (int idx = threadIdx.x; idx < kc * g.Cout; idx += blockDim.x) {
      int co = idx / kc, k = idx % kc;
      wl[k * g.Cout + co] = to_f32(w[(size_t)co * K + t0 * g.Cin + k]);
    }
    __syncthreads();
    if (valid) {
      for (int t = 0; t < tcnt; ++t) {
        int tap = t0 + t, i = tap / g.kw, j = tap % g.kw;
        int hi = ho * g.stride + i - g.ph, wi = wo * g.stride + j - g.pw;
        if (hi < 0 || hi >= g.Hin || wi < 0 || wi >= g.Win) continue;
        size_t base = (((size_t)n * g.Hin + hi) * g.Win + wi) * g.Cin;
        for (int ci = 0; ci < g.Cin; ++ci) {
          float xv = view_at<T>(in, base + ci, ci);
          const float* wr = wl + (size_t)(t * g.Cin + ci) * g.Cout + cg * 8;
#pragma unroll
          for (int e = 0; e < 8; ++e) acc[e] = fmaf(xv, wr[e], acc[e]);
        }
      }
    }
  }
  if (valid) store8(z + pix * g.Cout + cg * 8, acc);
}

void conv_direct_fwd(int dt, hipStream_t st, HView in, const void* w, const ConvGeom& g, void* z) {
  int CGo = g.Cout / 8;
  int PPB = 256 / CGo;
  if (PPB < 1) PPB = 1;
  int TC = kWChunkFloats / (g.Cin * g.Cout);
  if (TC < 1) TC = 1;
  if (TC > g.kh * g.kw) TC = g.kh * g.kw;
  size_t total = (size_t)g.N * g.Hout * g.Wout;
  size_t sm = (size_t)TC * g.Cin * g.Cout * sizeof(float);
  View v{in.z, in.scale, in.shift, in.act};
  KScope ks(st, "conv_direct_fwd", ((double)g.N * g.Hin * g.Win * g.Cin + (double)total * g.Cout + (double)g.kh * g.kw * g.Cin * g.Cout) * (dt == 0 ? 4.0 : 2.0),
            2.0 * total * g.Cout * g.kh * g.kw * g.Cin);
  FTP_DISPATCH(dt, hipLaunchKernelGGL(conv_direct_fwd_k<T>, dim3((unsigned)((total + PPB - 1) / PPB)),
                                      dim3(PPB * CGo), sm, st, v, (const T*)w, g, TC, PPB, (T*)z));
}

// thread = (input pixel, input channel): gathers every (tap, cout) that reaches it
template <typename T>
__global__ void conv_direct_dgrad_k(const T* __restrict__ dz, const T* __restrict__ w, ConvGeom g,
                                    T* __restrict__ dIn) {
  size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  size_t total = (size_t)g.N * g.Hin * g.Win * g.Cin;
  if (idx >= total) return;
  int ci = (int)(idx % g.Cin);
  size_t r = idx / g.Cin;
  int wi = (int)(r % g.Win);
  r /= g.Win;
  int hi = (int)(r % g.Hin);
  int n = (int)(r / g.Hin);
  const int K = g.kh * g.kw * g.Cin;
  float acc = 0.f;
  for (int i = 0; i < g.kh; ++i) {
    int hn = hi + g.ph - i;
    if (hn < 0 || hn % g.stride) continue;
    int ho = hn / g.stride;
    if (ho >= g.Hout) continue;
    for (int j = 0; j < g.kw; ++j) {
      int wn = wi + g.pw - j;
      if (wn < 0 || wn % g.stride) continue;
      int wo = wn / g.stride;
      if (wo >= g.Wout) continue;
      const T* d = dz + (((size_t)n * g.Hout + ho) * g.Wout + wo) * g.Cout;
      const T* wp = w + (size_t)(i * g.kw + j) * g.Cin + ci;
      for (int co = 0; co < g.Cout; ++co) acc = fmaf(to_f32(d[co]), to_f32(wp[(size_t)co * K]), acc);
    }
  }
  dIn[idx] = from_f32<T>(acc);
}

void conv_direct_dgrad(int dt, hipStream_t st, const void* dz, const void* w, const ConvGeom& g, void* dIn) {
  size_t total = (size_t)g.N * g.Hin * g.Win * g.Cin;
  KScope ks(st, "conv_direct_dgrad", ((double)total + (double)g.N * g.Hout * g.Wout * g.Cout) * (dt == 0 ? 4.0 : 2.0),
            2.0 * g.N * g.Hout * g.Wout * g.Cout * g.kh * g.kw * g.Cin);
  FTP_DISPATCH(dt, hipLaunchKernelGGL(conv_direct_dgrad_k<T>, dim3((unsigned)((total + 255) / 256)), dim3(256),
                                      0, st, (const T*)dz, (const T*)w, g, (T*)dIn));
}

// Weight gradient of a small dense convolution: the input patches are written out once as a
// matrix A[pixel][Kpad] (k = (tap, ci), zero padded to a multiple of 8, producer BatchNorm +
// activation applied), then dW = dZ^T * A runs on the MFMA weight-gradient kernel.
// A thread keeps one group of 8 columns and walks pixels: what a column is (tap, channel, offset) is decoded once per thread, the
// pixel once per block in full and per thread relative to that, all eight loads are requested before the first is used.
// Bound by vector instructions and 2-byte gathers (it was a table read and two 64-bit products per value and four 64-bit divisions
// per pixel).  224 x 224 x 3, batch 128, bfloat16: 59.9 -> 50.5 us; 32 x 32 x 3, batch 32, fp32: 5.4 -> 5.5 us, latency.
struct Im2colArgs {
  ConvGeom g;
  size_t M;            // pixels
  int KG, K, PPT, PB;  // column groups, columns in use, pixels the block writes at once / in all
  FastDiv dKG, dC, dKw, dW, dH;
  int fast;            // Hout and Wout small enough for dW, dH over the pixels of a block
};

template <typename T>
__global__ __launch_bounds__(256) void im2col_k(View in, Im2colArgs a, T* __restrict__ out) {
  const ConvGeom& g = a.g;
  const size_t p0 = (size_t)blockIdx.x * a.PB;
  const int pl0 = a.KG <= 256 ? (int)a.dKG.div(threadIdx.x) : 0;
  if (pl0 >= a.PPT) return;
  const int np = a.M - p0 < (size_t)a.PB ? (int)(a.M - p0) : a.PB;
  const size_t hw = (size_t)g.Hout * g.Wout;
  const int n0 = (int)(a.M >> 32 ? p0 / hw : (uint32_t)p0 / (uint32_t)hw);      // a 64-bit division ahead of the first load is a tenth of a short launch
  const int r0 = (int)(p0 - n0 * hw);
  const int ho0 = r0 / g.Wout, wo0 = r0 - ho0 * g.Wout;
  const T* z = reinterpret_cast<const T*>(in.z);
  for (int kg = (int)threadIdx.x - pl0 * a.KG; kg < a.KG; kg += 256) {       // one turn unless there are more than 256 groups
    int di[8], dj[8], ch[8];
    ptrdiff_t off[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int k = kg * 8 + e, tap = (int)a.dC.div(k), ci = k - tap * g.Cin, i = (int)a.dKw.div(tap), j = tap - i * g.kw;
      di[e] = k < a.K ? i : 1 << 30;                                          // a padding column lies outside every image
      dj[e] = j;
      ch[e] = k < a.K ? ci : 0;
      off[e] = ((ptrdiff_t)i * g.Win + j) * g.Cin + ci;
    }
    for (int pl = pl0; pl < np; pl += a.PPT) {
      const uint32_t t = (uint32_t)(wo0 + pl);
      const int dr = (int)(a.fast ? a.dW.div(t) : t / (uint32_t)g.Wout), wo = (int)t - dr * g.Wout;
      const uint32_t hh = (uint32_t)(ho0 + dr);
      const int dn = (int)(a.fast ? a.dH.div(hh) : hh / (uint32_t)g.Hout), ho = (int)hh - dn * g.Hout;
      const int h0 = ho * g.stride - g.ph, w0 = wo * g.stride - g.pw;
      const ptrdiff_t base = (((ptrdiff_t)(n0 + dn) * g.Hin + h0) * g.Win + w0) * g.Cin;
      T raw[8];
      bool ok[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ok[e] = (uint32_t)(h0 + di[e]) < (uint32_t)g.Hin && (uint32_t)(w0 + dj[e]) < (uint32_t)g.Win;
        raw[e] = z[ok[e] ? base + off[e] : 0];
      }
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x = to_f32(raw[e]);
        if (in.scale) x = round_to<T>(act_apply(fmaf(x, in.scale[ch[e]], in.shift[ch[e]]), in.act));
        v[e] = ok[e] ? x : 0.f;
      }
      store8(out + ((p0 + pl) * a.KG + kg) * 8, v);
    }
  }
}

static int direct_kpad(const ConvGeom& g) { return (g.kh * g.kw * g.Cin + 7) / 8 * 8; }

static void write_patches(int dt, hipStream_t st, HView in, const ConvGeom& g, void* out) {
  Im2colArgs a{};
  a.g = g;
  a.M = (size_t)g.N * g.Hout * g.Wout;
  a.K = g.kh * g.kw * g.Cin;
  a.KG = direct_kpad(g) / 8;
  a.PPT = a.KG <= 256 ? 256 / a.KG : 1;
  // up to 8 pixels a thread, fewer where that would leave less than 2048 blocks (8 per CU)
  const size_t per = a.M / ((size_t)a.PPT * 2048);
  a.PB = a.PPT * (per < 1 ? 1 : per > 8 ? 8 : (int)per);
  a.dKG = FastDiv::of(a.KG); a.dC = FastDiv::of(g.Cin); a.dKw = FastDiv::of(g.kw); a.dW = FastDiv::of(g.Wout); a.dH = FastDiv::of(g.Hout);
  // the reciprocal is exact while dividend x divisor stays under 2^32; a block has at most 2048 pixels
  a.fast = g.Wout <= 60000 && g.Hout <= 60000;
  const View v{in.z, in.scale, in.shift, in.act};
  FTP_DISPATCH(dt, hipLaunchKernelGGL(im2col_k<T>, dim3((unsigned)((a.M + a.PB - 1) / a.PB)), dim3(256), 0, st, v, a, (T*)out));
}

size_t conv_direct_im2col_elems(const ConvGeom& g) { return (size_t)g.N * g.Hout * g.Wout * direct_kpad(g); }

size_t conv_direct_wgrad_ws(const ConvGeom& g) {
  return pw_wgrad_ws((size_t)g.N * g.Hout * g.Wout, direct_kpad(g), g.Cout);
}

void conv_direct_wgrad(int dt, hipStream_t st, const void* dz, HView in, const ConvGeom& g, void* im2col, float* ws,
                       float* g_w, bool patches_ready) {
  const int Kpad = direct_kpad(g), K = g.kh * g.kw * g.Cin;
  const size_t M = (size_t)g.N * g.Hout * g.Wout;
  if (!patches_ready) {
    const double es = dt == 0 ? 4.0 : 2.0;
    KScope ks(st, "im2col", ((double)g.N * g.Hin * g.Win * g.Cin + (double)M * Kpad) * es, 0, (long)M, Kpad, g.Cout);
    write_patches(dt, st, in, g, im2col);
  }
  pw_wgrad(dt, st, dz, HView{im2col, nullptr, nullptr, 0}, M, Kpad, g.Cout, ws, g_w, K);
}

// Forward of a small dense convolution over many pixels (the 224x224 stem) as im2col + MFMA GEMM: the patch
// matrix costs one extra write and read of M x Kpad elements but the GEMM streams at several TB/s and leaves the
// BatchNorm statistics in its epilogue, where the direct kernel issues Cin*kh*kw scalar loads per output vector.
template <typename T>
__global__ void pad_rows_k(const T* __restrict__ w, int rows, int K, int Kpad, T* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= rows * Kpad) return;
  const int r = i / Kpad, k = i - r * Kpad;
  out[i] = k < K ? w[(size_t)r * K + k] : from_f32<T>(0.f);
}

// many pixels (the 224x224 stem) or many taps x channels per output (conv1d): the direct kernel's scalar loads lose
int conv_direct_gemm_ok(const ConvGeom& g) {
  const int Kpad = direct_kpad(g);
  return g.Cout % 8 == 0 && (((size_t)g.N * g.Hout * g.Wout >= ((size_t)1 << 18) && Kpad <= 64) || (Kpad >= 40 && Kpad <= 2048));
}
size_t conv_direct_gemm_wpad_elems(const ConvGeom& g) { return (size_t)g.Cout * direct_kpad(g); }

void conv_direct_fwd_gemm(int dt, hipStream_t st, HView in, const void* w, const ConvGeom& g, void* im2col, void* wpad, void* z,
                          float* stats, int* P_out) {
  const int Kpad = direct_kpad(g), K = g.kh * g.kw * g.Cin;
  const size_t M = (size_t)g.N * g.Hout * g.Wout;
  {
    const double es = dt == 0 ? 4.0 : 2.0;
    KScope ks(st, "im2col", ((double)g.N * g.Hin * g.Win * g.Cin + (double)M * Kpad) * es, 0, (long)M, Kpad, g.Cout);
    write_patches(dt, st, in, g, im2col);
    FTP_DISPATCH(dt, hipLaunchKernelGGL(pad_rows_k<T>, dim3((g.Cout * Kpad + 255) / 256), dim3(256), 0, st, (const T*)w, g.Cout, K,
                                        Kpad, (T*)wpad));
  }
  pw_fwd(dt, st, HView{im2col, nullptr, nullptr, 0}, wpad, nullptr, M, Kpad, g.Cout, z, stats, P_out);
}

// Data gradient of a stride-1 dense convolution as a forward convolution of dz with the taps flipped and the
// channel roles swapped: dIn[hi][ci] = sum_{i',j',co} dz[hi - (kh-1-ph) + i'][co] * w[co][kh-1-i'][kw-1-j'][ci],
// run as im2col(dz) x rearranged weights on the MFMA GEMM.
template <typename T>
__global__ void dgrad_weights_k(const T* __restrict__ w, int Cout, int kh, int kw, int Cin, int Kpad, T* __restrict__ out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= Cin * Kpad) return;
  const int ci = i / Kpad, k = i - ci * Kpad;
  T v = from_f32<T>(0.f);
  if (k < kh * kw * Cout) {
    const int tap = k / Cout, co = k - tap * Cout, ti = tap / kw, tj = tap - ti * kw;
    v = w[(((size_t)co * kh + (kh - 1 - ti)) * kw + (kw - 1 - tj)) * Cin + ci];
  }
  out[i] = v;
}

static ConvGeom dgrad_as_forward(const ConvGeom& g) {
  ConvGeom d = g;
  d.Hin = g.Hout; d.Win = g.Wout; d.Cin = g.Cout;
  d.Hout = g.Hin; d.Wout = g.Win; d.Cout = g.Cin;
  d.stride = 1; d.ph = g.kh - 1 - g.ph; d.pw = g.kw - 1 - g.pw;
  return d;
}

int conv_direct_dgrad_gemm_ok(const ConvGeom& g) {
  if (g.stride != 1 || g.kh - 1 - g.ph < 0 || g.kw - 1 - g.pw < 0) return 0;
  const int Kpad = direct_kpad(dgrad_as_forward(g));
  return Kpad >= 40 && Kpad <= 4096;
}
size_t conv_direct_dgrad_gemm_im2col_elems(const ConvGeom& g) {
  return (size_t)g.N * g.Hin * g.Win * direct_kpad(dgrad_as_forward(g));
}
size_t conv_direct_dgrad_gemm_w_elems(const ConvGeom& g) { return (size_t)g.Cin * direct_kpad(dgrad_as_forward(g)); }

void conv_direct_dgrad_gemm(int dt, hipStream_t st, const void* dz, const void* w, const ConvGeom& g, void* im2col, void* wscratch,
                            void* dIn) {
  const ConvGeom d = dgrad_as_forward(g);
  const int Kpad = direct_kpad(d);
  const size_t M = (size_t)g.N * g.Hin * g.Win;
  {
    const double es = dt == 0 ? 4.0 : 2.0;
    KScope ks(st, "im2col", ((double)g.N * g.Hout * g.Wout * g.Cout + (double)M * Kpad) * es, 0, (long)M, Kpad, g.Cin);
    write_patches(dt, st, HView{dz, nullptr, nullptr, 0}, d, im2col);
    FTP_DISPATCH(dt, hipLaunchKernelGGL(dgrad_weights_k<T>, dim3((g.Cin * Kpad + 255) / 256), dim3(256), 0, st, (const T*)w, g.Cout,
                                        g.kh, g.kw, g.Cin, Kpad, (T*)wscratch));
  }
  pw_fwd(dt, st, HView{im2col, nullptr, nullptr, 0}, wscratch, nullptr, M, Kpad, g.Cin, dIn, nullptr, nullptr);
}

// ================================================================ depthwise 3x3
// A block owns a slab of CGB*8 channels (128 bytes of every pixel) of one spatial tile.  The input
// patch with its one-pixel halo is staged in LDS once in the tensor's own type, already passed through the
// producer's BatchNorm + activation and with zeros outside the image, so HBM sees every input
// element once per tile.  A thread then owns 4 channels of a horizontal run of 4 pixels: per kernel
// row it reads the 6 (stride 1) or 9 (stride 2) patch vectors under the run once and uses each for
// up to three taps, which cuts the LDS traffic of a pixel-per-thread mapping to a quarter, and it
// keeps the nine weight vectors in registers.  Tiles are numbered so that neighbours, which share
// halo pixels, run on the same XCD and meet in its L2.
struct DwPlan {
  int TH, TW, PH, PW;       // tile of the produced / walked tensor, staged patch
  int CGB, nslab, PPB;      // column groups per slab, slabs, patch pixels staged per pass
  int segw, nseg, spp;      // 4-pixel runs per tile row, per tile, and runs the block covers per pass
  int tiles_h, tiles_w, ntiles, nblocks;
  unsigned m_cgb, m_qb, m_pw, m_segw;   // reciprocals for dw_div (divisors < 64, dividends < 1024)
};
// passes of the forward kernel's patch staging at most (128 bytes of channels, a patch of 10 x 18 pixels): a load past the patch is made all the same, and
// fp32 slabs are half as many column groups
template <typename T> struct DwFill { enum { NV = sizeof(T) == 4 ? 3 : 6 }; };

// x / d for x < 1024, d < 64 with m = 65536 / d + 1: two full-rate instructions instead of the
// ~25-instruction integer division sequence (thread-index decoding was a third of the kernel's VALU work)
static unsigned dw_magic(int d) { return 65536u / (unsigned)d + 1u; }
__device__ __forceinline__ int dw_div(int x, unsigned m) { return (int)(__umul24((unsigned)x, m) >> 16); }

static DwPlan dw_plan(int C, int es, bool half_rows, int out_h, int out_w, int wide = 16) {
  DwPlan d;
  const int cgs = C / 8, cap = es == 2 ? 8 : 4;            // 128 bytes of channels per pixel
  d.nslab = (cgs + cap - 1) / cap;
  d.CGB = (cgs + d.nslab - 1) / d.nslab;
  d.PPB = 256 / d.CGB;
  d.spp = 256 / (2 * d.CGB);
  d.TH = half_rows ? 4 : 8;
  d.TW = half_rows ? 8 : wide;   // measured: 8x16 tiles beat 8x8 by 10-25 % (less halo, fewer blocks), 4x8 is best for stride 2
  if (d.TH > out_h) d.TH = out_h;
  if (d.TW > out_w) d.TW = out_w;
  d.segw = (d.TW + 3) / 4;
  d.nseg = d.TH * d.segw;
  d.tiles_h = (out_h + d.TH - 1) / d.TH;
  d.tiles_w = (out_w + d.TW - 1) / d.TW;
  d.ntiles = 0; d.nblocks = 0; d.PH = d.PW = 0;
  d.m_cgb = dw_magic(d.CGB); d.m_qb = dw_magic(2 * d.CGB); d.m_segw = dw_magic(d.segw); d.m_pw = 0;
  return d;
}

// Patch rows h0 .. h0+PH-1, cols w0 .. w0+PW-1 of image n (H x W x C), column groups cg0 .. cg0+CGB-1,
// into LDS as float [PH][PW][CGB][8].  Thread = (pixel lane, column group); fetch() issues all global
// loads, commit() applies the view and writes LDS, so a caller can keep the loads of the next tile
// in flight while it works on the current one.
template <typename T>
struct DwPatch {
  enum { NV = DwFill<T>::NV };
  Raw<T> raw[NV];
  unsigned ok;
  // image n is at most 2^31 elements: offsets inside it are 32-bit, products of 24-bit factors
  __device__ __forceinline__ void fetch(const T* __restrict__ src, int n, int h0, int w0, const DwPlan& d, int H, int W,
                                        int C, int cg0) {
    ok = 0;
    const int pl = dw_div(threadIdx.x, d.m_cgb), cg = threadIdx.x - pl * d.CGB, gcg = cg0 + cg;
    if (pl >= d.PPB || gcg >= C / 8) return;
    const T* img = src + (size_t)n * H * W * C + gcg * 8;
    const int npix = d.PH * d.PW, dph = dw_div(d.PPB, d.m_pw), dpw = d.PPB - dph * d.PW;
    int ph = dw_div(pl, d.m_pw), pw = pl - ph * d.PW;
    // Offsets first, then the loads back to back and unconditional (a pixel outside the image or the patch reads the
    // image's first pixel and is zeroed in commit): with a branch around each load, and its address computed next to
    // it, every load waited for the one before.
    unsigned off[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      const int h = h0 + ph, w = w0 + pw;
      const bool in = pl + q * d.PPB < npix && h >= 0 && h < H && w >= 0 && w < W;
      off[q] = in ? __umul24(__umul24(h, W) + w, C) : 0u;
      ok |= (in ? 1u : 0u) << q;
      ph += dph; pw += dpw;
      if (pw >= d.PW) { pw -= d.PW; ++ph; }
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) raw_load(raw[q], img + off[q]);
  }
  __device__ __forceinline__ void commit(T* patch, const View& vw, const DwPlan& d, int cg0) const {
    const int pl = dw_div(threadIdx.x, d.m_cgb), cg = threadIdx.x - pl * d.CGB;
    if (pl >= d.PPB) return;
    const int npix = d.PH * d.PW;
    float sc[8], sh[8];
    const bool view = vw.scale != nullptr && ok != 0;
    if (view) {
      load8(vw.scale + (cg0 + cg) * 8, sc);
      load8(vw.shift + (cg0 + cg) * 8, sh);
    }
    const float lo = act_lo(vw.act), hi = act_hi(vw.act);
    T* dst = patch + (pl * d.CGB + cg) * 8;            // stored in the tensor's own type: the values are already rounded to it
    const int step = d.PPB * d.CGB * 8;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      if (pl + q * d.PPB >= npix) break;
      float val[8] = {0, 0, 0, 0, 0, 0, 0, 0};
      if (ok & (1u << q)) {
        raw_unpack(raw[q], val);
        if (view) {
#pragma unroll
          for (int e = 0; e < 8; ++e) val[e] = clamp_act(fmaf(val[e], sc[e], sh[e]), lo, hi);   // store8 rounds to T
        }
      }
      store8(dst + q * step, val);
    }
  }
};

// the slab's weights as float [9][CGB][8].  All global loads are issued before the first LDS store (at most five
// per thread: 9 * 16 * 8 values over 256 threads): loaded and stored one by one, every round cost a memory round trip
// that nothing else in the block could hide.
template <typename T>
__device__ __forceinline__ void dw_stage_weights(float* wl, const T* __restrict__ w, int C, int cg0, int CGB, unsigned m_cgb) {
  constexpr int NV = 5;
  const int n = 9 * CGB * 8;
  T v[NV];                 // as loaded: a conversion next to its load makes the compiler wait for that load alone
  bool live[NV];
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int i = threadIdx.x + q * 256;
    const int e = i & 7, t = dw_div(i >> 3, m_cgb), c8 = (i >> 3) - t * CGB;      // i >> 3 < 160
    const int c = (cg0 + c8) * 8 + e;
    live[q] = i < n && c < C;
    v[q] = w[live[q] ? (size_t)c * 9 + t : 0];
  }
#pragma unroll
  for (int q = 0; q < NV; ++q) {
    const int i = threadIdx.x + q * 256;
    if (i < n) wl[i] = live[q] ? to_f32(v[q]) : 0.f;
  }
}

// out[ho][wo] = sum_{ky,kx} src[ho*S-1+ky][wo*S-1+kx] * w[ky][kx]
// RL = pixels per run: four at stride 1; two at stride 2, where a run of four keeps 9 patch vectors and 4 sums live
// (111 registers, four resident blocks per CU) and a 4 x 8 tile has work for only 96 of the 256 threads
// STATS (layers with at most kMaxPartials tiles): the block also leaves per-channel sums over its stored outputs, one
// partial per tile ([tile][2][C]): the sum and the sum of squares (what bn_stats would compute in a pass of its own).
template <typename T> __device__ __forceinline__ float4 round4(float4 v) {
  return make_float4(round_to<T>(v.x), round_to<T>(v.y), round_to<T>(v.z), round_to<T>(v.w));
}
// four of the eight channels of a raw vector
__device__ __forceinline__ float4 raw_half(const Raw<float>& r, int half) { return half ? r.b : r.a; }
__device__ __forceinline__ float4 raw_half(const Raw<bf16_t>& r, int half) {
  const uint32_t lo = half ? r.a.z : r.a.x, hi = half ? r.a.w : r.a.y;
  return make_float4(__uint_as_float(lo << 16), __uint_as_float(lo & 0xffff0000u), __uint_as_float(hi << 16), __uint_as_float(hi & 0xffff0000u));
}
struct DwPrev { const void* z; const float* scale; const float* shift; int act; };

// The runs of a channel quad are spread over spp threads: through LDS (red: [spp][QB][8]), summed in
// a fixed order by one thread per channel and value into partial[2][C]
__device__ __forceinline__ void dw_leave_sums(float4 s1, float4 s2, bool worker, int seg0, int cq, int QB, int cg0, int C, int spp, float* red,
                                              float* __restrict__ partial) {
  if (worker) {
    float* r = red + ((size_t)seg0 * QB + cq) * 8;
    r[0] = s1.x; r[1] = s1.y; r[2] = s1.z; r[3] = s1.w; r[4] = s2.x; r[5] = s2.y; r[6] = s2.z; r[7] = s2.w;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < QB * 8; i += 256) {
    const int q = i >> 3, e = i & 7, c = cg0 * 8 + q * 4 + (e & 3);
    if (c >= C) continue;
    float t = 0.f;
    for (int sgi = 0; sgi < spp; ++sgi) t += red[((size_t)sgi * QB + q) * 8 + e];
    partial[(size_t)(e >> 2) * C + c] = t;
  }
}
template <typename T, int S, bool STATS = false, int RL = (S == 2 ? 2 : 4)>
__global__ __launch_bounds__(256) void dw_conv_k(View in, const T* __restrict__ w, DwPlan d, int Hin, int Win, int Hout,
                                                 int Wout, int C, T* __restrict__ out, float* __restrict__ stats = nullptr) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  T* patch = reinterpret_cast<T*>(smem_raw);
  float* wl = reinterpret_cast<float*>(smem_raw + (((size_t)d.PH * d.PW * d.CGB * 8 * sizeof(T) + 15) / 16 * 16));
  const int lb = xcd_logical_block();
  const int slab = lb % d.nslab, tile = lb / d.nslab;     // the slabs of a tile run together: they share cache lines when a slab is not 128 bytes
  const int tw = tile % d.tiles_w, th = (tile / d.tiles_w) % d.tiles_h, n = tile / (d.tiles_w * d.tiles_h);
  const int ho0 = th * d.TH, wo0 = tw * d.TW, cg0 = slab * d.CGB;
  DwPatch<T> lp;
  lp.fetch(reinterpret_cast<const T*>(in.z), n, ho0 * S - 1, wo0 * S - 1, d, Hin, Win, C, cg0);
  dw_stage_weights(wl, w, C, cg0, d.CGB, d.m_cgb);
  lp.commit(patch, in, d, cg0);
  __syncthreads();
  const int QB = 2 * d.CGB, seg0 = dw_div(threadIdx.x, d.m_qb), cq = threadIdx.x - seg0 * QB;
  const int c4 = cq * 4, gc = cg0 * 8 + c4;
  const bool worker = seg0 < d.spp && gc < C;
  if (!STATS && !worker) return;
  float4 wr[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) wr[t] = worker ? ld4(wl + (size_t)t * d.CGB * 8 + c4) : make_float4(0.f, 0.f, 0.f, 0.f);
  const int vs = d.CGB * 8;                       // floats per patch pixel
  float4 s1 = make_float4(0.f, 0.f, 0.f, 0.f), s2 = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int sg = worker ? seg0 : d.nseg; sg < d.nseg; sg += d.spp) {
    const int hl = dw_div(sg, d.m_segw), wl0 = (sg - hl * d.segw) * RL;
    const int ho = ho0 + hl;
    if (ho >= Hout) continue;
    float4 acc[RL];
#pragma unroll
    for (int o = 0; o < RL; ++o) acc[o] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int ky = 0; ky < 3; ++ky) {
      const T* row = patch + (size_t)((hl * S + ky) * d.PW + wl0 * S) * vs + c4;
      float4 iv[(RL - 1) * S + 3];
#pragma unroll
      for (int x = 0; x < (RL - 1) * S + 3; ++x) iv[x] = load4(row + (size_t)x * vs);
#pragma unroll
      for (int kx = 0; kx < 3; ++kx)
#pragma unroll
        for (int o = 0; o < RL; ++o) acc[o] = fma4(iv[o * S + kx], wr[ky * 3 + kx], acc[o]);
    }
    T* dst = out + (((size_t)n * Hout + ho) * Wout + wo0 + wl0) * C + gc;
#pragma unroll
    for (int o = 0; o < RL; ++o)
      if (wo0 + wl0 + o < Wout) {
        store4(dst + (size_t)o * C, acc[o]);
        if (STATS) {                              // sums over the values as stored
          const float4 r = round4<T>(acc[o]);
          s1.x += r.x; s1.y += r.y; s1.z += r.z; s1.w += r.w;
          s2 = fma4(r, r, s2);
        }
      }
  }
  if (STATS) {
    __syncthreads();                    // the patch is no longer needed
    dw_leave_sums(s1, s2, worker, seg0, cq, QB, cg0, C, d.spp, reinterpret_cast<float*>(smem_raw), stats + (size_t)tile * 2 * C);
  }
}

// LDS layout: the patch as T [PH][PW][CGB][8], then (16-byte aligned) the weights as float [9][CGB][8]
static size_t dw_patch_bytes(const DwPlan& d, int es) { return (((size_t)d.PH * d.PW * d.CGB * 8 * es) + 15) / 16 * 16; }
static size_t dw_lds_bytes(const DwPlan& d, int es) { return dw_patch_bytes(d, es) + (size_t)9 * d.CGB * 8 * 4; }

// staging is unrolled for `fill` passes; dw_div needs small divisors.  The plans of every shape a model can
// describe satisfy this; if one ever does not, the launch is skipped and the stage call reports it.
static bool dw_check_plan(DwPlan& d, int fill, int rounds) {
  if (d.PH * d.PW > fill * d.PPB || d.PW > 63 || d.CGB > 16 || d.segw > 32 || d.nseg > rounds * d.spp) {
    launch_plan_failed("depthwise tile plan outside the kernels' limits");
    return false;
  }
  d.m_pw = dw_magic(d.PW);
  return true;
}

// the depthwise forward can leave the BatchNorm partial sums itself when its tiles are few enough to be the partials
int dw_fwd_stats_ok(int dt, const ConvGeom& g) {
  const int es = dt == 0 ? 4 : 2;
  const DwPlan d = dw_plan(g.Cout, es, g.stride == 2, g.Hout, g.Wout);
  return (size_t)g.N * d.tiles_h * d.tiles_w <= (size_t)kMaxPartials;
}

void dw_fwd(int dt, hipStream_t st, HView in, const void* w, const ConvGeom& g, void* z, float* stats, int* P_out) {
  const int es = dt == 0 ? 4 : 2, s = g.stride;
  DwPlan d = dw_plan(g.Cout, es, s == 2, g.Hout, g.Wout);
  const int run = s == 2 ? 2 : 4;                // pixels per run, as the kernel's RL
  d.segw = (d.TW + run - 1) / run;
  d.nseg = d.TH * d.segw;
  d.m_segw = dw_magic(d.segw);
  d.PH = (d.TH - 1) * s + 3;
  d.PW = (d.segw * run - 1) * s + 3;             // runs are whole: the patch covers the rounded-up tile width
  d.ntiles = g.N * d.tiles_h * d.tiles_w;
  if (!dw_check_plan(d, dt == 0 ? DwFill<float>::NV : DwFill<bf16_t>::NV, 2)) return;
  View v{in.z, in.scale, in.shift, in.act};
  size_t total = (size_t)g.N * g.Hout * g.Wout;
  KScope ks(st, "dw_fwd", ((double)g.N * g.Hin * g.Win * g.Cout + (double)total * g.Cout) * es, 18.0 * total * g.Cout,
            (long)total, g.Cout, g.stride);
  const unsigned grid = (unsigned)d.ntiles * d.nslab;
  if (stats) {
    if (d.ntiles > kMaxPartials) { launch_plan_failed("depthwise forward with statistics: more tiles than partial sums"); return; }
    // the reduction reuses the patch's LDS: [spp][2*CGB][8] floats
    size_t lds = dw_lds_bytes(d, es);
    const size_t red = (size_t)d.spp * 2 * d.CGB * 8 * sizeof(float);
    if (lds < red) lds = red;
    if (s == 1) {
      FTP_DISPATCH(dt, hipLaunchKernelGGL((dw_conv_k<T, 1, true>), dim3(grid), dim3(256), lds, st, v, (const T*)w, d,
                                          g.Hin, g.Win, g.Hout, g.Wout, g.Cout, (T*)z, stats));
    } else {
      FTP_DISPATCH(dt, hipLaunchKernelGGL((dw_conv_k<T, 2, true>), dim3(grid), dim3(256), lds, st, v, (const T*)w, d,
                                          g.Hin, g.Win, g.Hout, g.Wout, g.Cout, (T*)z, stats));
    }
    *P_out = d.ntiles;
    return;
  }
  if (s == 1) {
    FTP_DISPATCH(dt, hipLaunchKernelGGL((dw_conv_k<T, 1>), dim3(grid), dim3(256), dw_lds_bytes(d, es), st, v, (const T*)w, d,
                                        g.Hin, g.Win, g.Hout, g.Wout, g.Cout, (T*)z));
  } else {
    FTP_DISPATCH(dt, hipLaunchKernelGGL((dw_conv_k<T, 2>), dim3(grid), dim3(256), dw_lds_bytes(d, es), st, v, (const T*)w, d,
                                        g.Hin, g.Win, g.Hout, g.Wout, g.Cout, (T*)z));
  }
}

// ---- short tensors: whole depthwise layers in one launch ------------------------------------------------
// For tensors of a few hundred KB the separate kernels are all launch latency.  Here a block owns 4 channels
// over every pixel: the tensor that is gathered from (input in forward, dz in backward) is staged once in LDS
// as one float4 per pixel (the view applied once per element), so the nine taps are LDS reads and the
// per-channel sums never leave the block.  A pixel's row and column come from two 32-bit multiplications and a tap outside the
// image reads a zero slot, so the nine reads go out together: with 64-bit divisions and a branch per tap the backward of
// 1859 pixels x 384 channels took 19.5 us instead of 16.5 (bfloat16), the forward 10 instead of 8.1.
__device__ __forceinline__ float4 view4(float4 v, const float* sc, const float* sh, float lo, float hi) {
  return make_float4(clamp_act(fmaf(v.x, sc[0], sh[0]), lo, hi), clamp_act(fmaf(v.y, sc[1], sh[1]), lo, hi),
                     clamp_act(fmaf(v.z, sc[2], sh[2]), lo, hi), clamp_act(fmaf(v.w, sc[3], sh[3]), lo, hi));
}

// four channels of one pixel as loaded, converted at the point of use (so the load can stay in flight)
template <typename T> struct Raw4;
template <> struct Raw4<float> { float4 v; };
template <> struct Raw4<bf16_t> { uint2 v; };
__device__ __forceinline__ void raw4_load(Raw4<float>& r, const float* p) { r.v = *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void raw4_load(Raw4<bf16_t>& r, const bf16_t* p) { r.v = *reinterpret_cast<const uint2*>(p); }
__device__ __forceinline__ float4 raw4_unpack(const Raw4<float>& r) { return r.v; }
__device__ __forceinline__ float4 raw4_unpack(const Raw4<bf16_t>& r) {
  return make_float4(__uint_as_float(r.v.x << 16), __uint_as_float(r.v.x & 0xffff0000u), __uint_as_float(r.v.y << 16),
                     __uint_as_float(r.v.y & 0xffff0000u));
}

// Depthwise convolution + BatchNorm statistics + their finalisation (and, when the producer left them pending,
// the finalisation of the input's BatchNorm too).
template <typename T>
__global__ __launch_bounds__(1024) void dw_fwd_bn_small_k(View in, BnPending pend, const T* __restrict__ w, ConvGeom g, FastDiv dW,
                                                          FastDiv dH, int M, int Min, const float* __restrict__ gamma, const float* __restrict__ beta,
                                                          float* mean, float* invstd, float* scale, float* shift,
                                                          float* run_mean, float* run_var, float eps, float momentum,
                                                          T* __restrict__ z) {
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  float4* tile = reinterpret_cast<float4*>(smem_raw);           // [Min + 1], the last one zero
  __shared__ float wl[9][4];
  __shared__ float red[16][8];
  __shared__ double pre[32][8];
  __shared__ float insc[2][4];
  // adjacent channel groups share cache lines: keep them on one XCD
  const int C = g.Cout, c0 = xcd_logical_block() * 4, tid = threadIdx.x, nt = blockDim.x, s = g.stride;
  // Everything that depends on nothing is requested first: the input pixels of this block (at most three per thread,
  // raw, from a clamped address), the BatchNorm parameters and running statistics.  They then travel while the pending
  // BatchNorm of the input is finished; the kernel is a chain of memory round trips and little else.
  const T* src = reinterpret_cast<const T*>(in.z);
  Raw4<T> rv[3];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int m = tid + q * nt;
    raw4_load(rv[q], src + (size_t)(m < Min ? m : 0) * C + c0);
  }
  float bn_g = 0.f, bn_b = 0.f, bn_rm = 0.f, bn_rv = 0.f;
  const double inv_M = early_inverse((double)M);
  if (tid < 4) { bn_g = gamma[c0 + tid]; bn_b = beta[c0 + tid]; bn_rm = run_mean[c0 + tid]; bn_rv = run_var[c0 + tid]; }
  if (tid < 36) wl[tid / 4][tid % 4] = to_f32(w[(size_t)(c0 + tid % 4) * 9 + tid / 4]);
  const bool view = in.scale != nullptr;
  if (pend.partial) finish_pending4(pend, C, c0, eps, momentum, pre, insc);
  else if (tid < 4 && view) { insc[0][tid] = in.scale[c0 + tid]; insc[1][tid] = in.shift[c0 + tid]; }
  if (!pend.partial) __syncthreads();
  float sc[4] = {1.f, 1.f, 1.f, 1.f}, sh[4] = {0.f, 0.f, 0.f, 0.f};
  if (view) {
#pragma unroll
    for (int e = 0; e < 4; ++e) { sc[e] = insc[0][e]; sh[e] = insc[1][e]; }
  }
  const float lo = view ? act_lo(in.act) : -INFINITY, hi = view ? act_hi(in.act) : INFINITY;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int m = tid + q * nt;
    if (m >= Min) break;
    float4 v = raw4_unpack(rv[q]);
    if (view) v = round4<T>(view4(v, sc, sh, lo, hi));
    tile[m] = v;
  }
  if (tid == 0) tile[Min] = make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  float4 wr[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) wr[t] = make_float4(wl[t][0], wl[t][1], wl[t][2], wl[t][3]);
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int m = tid; m < M; m += nt) {
    const int r = (int)dW.div(m), wo = m - r * g.Wout, n = (int)dH.div(r), ho = r - n * g.Hout;
    // the nine values first, from the zero slot where a tap leaves the image: no branches between the reads
    float4 t[9];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int h = ho * s - 1 + i;
      const int row = (unsigned)h < (unsigned)g.Hin ? (n * g.Hin + h) * g.Win : -1;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int ww = wo * s - 1 + j;
        t[i * 3 + j] = tile[row >= 0 && (unsigned)ww < (unsigned)g.Win ? row + ww : Min];
      }
    }
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int k = 0; k < 9; ++k) o = fma4(t[k], wr[k], o);
    store4(z + (size_t)m * C + c0, o);
    const float4 sv = round4<T>(o);               // statistics of the values as stored
    acc[0] += sv.x; acc[1] += sv.y; acc[2] += sv.z; acc[3] += sv.w;
    acc[4] = fmaf(sv.x, sv.x, acc[4]); acc[5] = fmaf(sv.y, sv.y, acc[5]);
    acc[6] = fmaf(sv.z, sv.z, acc[6]); acc[7] = fmaf(sv.w, sv.w, acc[7]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = wave_sum_last(acc[e]);
  const int wave = tid >> 6, nw = nt >> 6;
  if ((tid & 63) == 63) {
#pragma unroll
    for (int e = 0; e < 8; ++e) red[wave][e] = acc[e];
  }
  __syncthreads();
  // first use of the four values requested at the top: their conversions must not move up to the loads
  asm volatile("" : "+v"(bn_g), "+v"(bn_b), "+v"(bn_rm), "+v"(bn_rv));
  if (tid < 4) {
    const int c = c0 + tid;
    double s0 = 0.0, s1 = 0.0;
    for (int q = 0; q < nw; ++q) { s0 += red[q][tid]; s1 += red[q][4 + tid]; }
    const double mu = s0 * inv_M;
    double var = s1 * inv_M - mu * mu;
    if (var < 0.0) var = 0.0;
    const double is = rsqrt(var + (double)eps);
    const float scv = (float)((double)bn_g * is);
    mean[c] = (float)mu;
    invstd[c] = (float)is;
    scale[c] = scv;
    shift[c] = (float)((double)bn_b - mu * (double)scv);
    const double unb = M > 1 ? var / (1.0 - inv_M) : var;
    run_mean[c] = (float)((1.0 - momentum) * bn_rm + momentum * mu);
    run_var[c] = (float)((1.0 - momentum) * bn_rv + momentum * unb);
  }
}

int dw_fwd_bn_small_ok(const ConvGeom& g) {
  return (size_t)g.N * g.Hout * g.Wout <= 2048 && (size_t)g.N * g.Hin * g.Win <= 3072 && g.Cout >= 32 && g.Cout % 8 == 0;
}

void dw_fwd_bn_small(int dt, hipStream_t st, HView in, const BnPending& pend, const void* w, const ConvGeom& g, const float* gamma,
                     const float* beta, float* mean, float* invstd, float* scale, float* shift, float* run_mean,
                     float* run_var, float eps, float momentum, void* z) {
  const size_t M = (size_t)g.N * g.Hout * g.Wout, Min = (size_t)g.N * g.Hin * g.Win;
  const int es = dt == 0 ? 4 : 2;
  View v{in.z, in.scale, in.shift, in.act};
  KScope ks(st, "dw_fwd_bn_small", ((double)Min * g.Cout + (double)M * g.Cout) * es, 21.0 * M * g.Cout, (long)M, g.Cout, g.stride);
  const int nt = Min > 512 ? 1024 : (Min > 256 ? 512 : 256);
  FTP_DISPATCH(dt, hipLaunchKernelGGL(dw_fwd_bn_small_k<T>, dim3(g.Cout / 4), dim3(nt), (Min + 1) * 16, st, v, pend, (const T*)w, g,
                                      FastDiv::of(g.Wout), FastDiv::of(g.Hout), (int)M, (int)Min,
                                      gamma, beta, mean, invstd, scale, shift, run_mean, run_var, eps, momentum, (T*)z));
}

// V channels of one pixel, as floats
template <int V> struct alignas(4 * V) Chans { float v[V]; };
__device__ __forceinline__ Chans<4> load_chans(const float* p, Chans<4>*) { const float4 f = *reinterpret_cast<const float4*>(p); return {{f.x, f.y, f.z, f.w}}; }
__device__ __forceinline__ Chans<4> load_chans(const bf16_t* p, Chans<4>*) { const float4 f = load4(p); return {{f.x, f.y, f.z, f.w}}; }
__device__ __forceinline__ Chans<2> load_chans(const float* p, Chans<2>*) { const float2 f = *reinterpret_cast<const float2*>(p); return {{f.x, f.y}}; }
__device__ __forceinline__ Chans<2> load_chans(const bf16_t* p, Chans<2>*) {
  const uint32_t u = *reinterpret_cast<const uint32_t*>(p);
  return {{__uint_as_float(u << 16), __uint_as_float(u & 0xffff0000u)}};
}
template <typename T> __device__ __forceinline__ void store_chans(T* p, Chans<4> c) { store4(p, make_float4(c.v[0], c.v[1], c.v[2], c.v[3])); }
__device__ __forceinline__ void store_chans(float* p, Chans<2> c) { *reinterpret_cast<float2*>(p) = make_float2(c.v[0], c.v[1]); }
__device__ __forceinline__ void store_chans(bf16_t* p, Chans<2> c) { *reinterpret_cast<uint32_t*>(p) = f32x2_to_bf16x2(c.v[0], c.v[1]); }

// Backward of a depthwise layer, of its own BatchNorm and of the BatchNorm in front of it.  A block owns V channels of all pixels, a thread RPT
// pixels.  The layer's own BatchNorm backward comes first (block-local: same channels), its dz goes into LDS and never to memory.  A thread
// gathers the dz values that reach an input pixel once and uses each twice: times the tap weight for the data gradient, times the pixel's own
// activation for the weight gradient (dW[tap] = sum_p dz[p] * a[p*s-1+tap] is the same sum walked from the input side).  The data gradient never
// leaves the registers: it is gated by the activation, reduced into the BatchNorm sums, and after the block-wide reduction turned into the
// gradient of the raw convolution output in front (dz_prev).
// Bound by the lines that a CU fetches and the instructions it issues: a block reads 16 or 8 bytes of every line of three tensors and sums 11 values a channel
// over its wavefronts.  Two channels a block (C <= 512: no more blocks than CUs) halve the instructions and leave room for twice the wavefronts: 1859 rows,
// 192 channels, bfloat16 15.6 -> 13.5 us; 512 x 384, fp32 8.5 -> 7.1; 2048 x 192 16.8 -> 14.5.  With more blocks than CUs it loses (512 x 576:
// 9.4, four channels 8.4).  All sums of a thread are formed before the last lane stores them (a branch for each sum: 256 x 960 7.0 us, now 6.1).
template <typename T, int V, int RPT, int NT>
__global__ __launch_bounds__(NT) void dw_bwd_small_k(BnBwdIn bo, const T* __restrict__ w, View in,
                                                     ConvGeom g, FastDiv dW, FastDiv dH, int M, int Mout, const float* __restrict__ gamma,
                                                     const float* __restrict__ mean, const float* __restrict__ invstd, float* g_w,
                                                     float* g_gamma, float* g_beta, T* __restrict__ dz_prev) {
  typedef Chans<V> F;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  F* tile = reinterpret_cast<F*>(smem_raw);           // dz, [Mout + 1], the last one zero
  __shared__ F wl[9];
  __shared__ __attribute__((aligned(16))) float red[NT / 64][11 * V], red2[NT / 64][2 * V];    // [wave][value]
  __shared__ F coef[3], coef2[3];
  __builtin_amdgcn_s_setprio(3);             // data-gradient chain: ahead of the weight-gradient stream's waves
  // adjacent channel groups share cache lines: keep them on one XCD
  const int C = g.Cout, c0 = xcd_logical_block() * V, tid = threadIdx.x, nt = blockDim.x, s = g.stride;
  const T* zin = reinterpret_cast<const T*>(in.z) + c0;
  const T* dA2 = reinterpret_cast<const T*>(bo.dA) + c0;
  const T* z2 = reinterpret_cast<const T*>(bo.out.z) + c0;
  F* const none = nullptr;
  // Everything that depends on nothing is requested first, unconditionally and from clamped addresses: this thread's
  // rows of the layer input, the old weight gradient, and what the finishing threads need after each reduction.
  // The kernel is a chain of memory round trips; these then overlap with the first of them.
  F zv[RPT], dy2[RPT], z2v[RPT];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int m = tid + q * nt;
    const size_t mc = m < Mout ? m : 0;
    dy2[q] = load_chans(dA2 + mc * C, none);
    z2v[q] = load_chans(z2 + mc * C, none);
  }
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int m = tid + q * nt;
    zv[q] = load_chans(zin + (size_t)(m < M ? m : 0) * C, none);
  }
  const double inv_M = early_inverse((double)M), inv_Mo = early_inverse((double)Mout);
  float gw_old = 0.f, f_mu = 0.f, f_is = 0.f, f_g = 0.f, f_gg = 0.f, f_gb = 0.f;
  float f2_mu = 0.f, f2_is = 0.f, f2_g = 0.f, f2_gg = 0.f, f2_gb = 0.f;
  if (tid < 9 * V) gw_old = g_w[(size_t)(c0 + tid % V) * 9 + tid / V];
  if (tid >= 64 && tid < 64 + V) {
    const int c = c0 + tid - 64;
    f_mu = mean[c]; f_is = invstd[c]; f_g = gamma[c]; f_gg = g_gamma[c]; f_gb = g_beta[c];
  }
  if (tid < V) {
    const int c = c0 + tid;
    f2_mu = bo.mean[c]; f2_is = bo.invstd[c]; f2_g = bo.gamma[c]; f2_gg = bo.g_gamma[c]; f2_gb = bo.g_beta[c];
  }
  const T w_raw = w[tid < 9 * V ? (size_t)(c0 + tid % V) * 9 + tid / V : 0];
  float sc[V], sh[V], sc2[V], sh2[V];
#pragma unroll
  for (int e = 0; e < V; ++e) { sc[e] = in.scale[c0 + e]; sh[e] = in.shift[c0 + e]; sc2[e] = bo.out.scale[c0 + e]; sh2[e] = bo.out.shift[c0 + e]; }
  const float lo = act_lo(in.act), hi = act_hi(in.act), lo2 = act_lo(bo.out.act), hi2 = act_hi(bo.out.act);
  const bool lead = (tid & 63) == 63;
  const int wave = tid >> 6, nw = nt >> 6;
  float b2[2 * V] = {};
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const bool row = tid + q * nt < Mout;
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const float zz = row ? z2v[q].v[e] : 0.f, y = fmaf(zz, sc2[e], sh2[e]), v = row && y > lo2 && y < hi2 ? dy2[q].v[e] : 0.f;
      z2v[q].v[e] = zz; dy2[q].v[e] = v;
      b2[e] += v;
      b2[V + e] = fmaf(v, zz, b2[V + e]);
    }
  }
#pragma unroll
  for (int e = 0; e < 2 * V; ++e) b2[e] = wave_sum_last(b2[e]);
  if (lead)
#pragma unroll
    for (int e = 0; e < 2 * V; ++e) red2[wave][e] = b2[e];
  if (tid < 9 * V) wl[tid / V].v[tid % V] = to_f32(w_raw);
  __syncthreads();
  // first use of the values requested at the top: their conversions must not move up to the loads
  asm volatile("" : "+v"(f2_mu), "+v"(f2_is), "+v"(f2_g), "+v"(f2_gg), "+v"(f2_gb));
  if (tid < V) {
    const int c = c0 + tid;
    double s0 = 0.0, s1 = 0.0;
    for (int q = 0; q < nw; ++q) { s0 += red2[q][tid]; s1 += red2[q][V + tid]; }
    const double mu = f2_mu, is = f2_is, gm = f2_g;
    const double dbeta = s0, dgamma = is * (s1 - mu * s0);
    bo.g_gamma[c] = f2_gg + (float)dgamma;
    bo.g_beta[c] = f2_gb + (float)dbeta;
    const double k1 = gm * is, k2 = -k1 * is * dgamma * inv_Mo, k3 = -k1 * dbeta * inv_Mo - k2 * mu;
    coef2[0].v[tid] = (float)k1; coef2[1].v[tid] = (float)k2; coef2[2].v[tid] = (float)k3;
  }
  __syncthreads();
  {
    const F k1 = coef2[0], k2 = coef2[1], k3 = coef2[2];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      const int m = tid + q * nt;
      F dz;
#pragma unroll
      for (int e = 0; e < V; ++e) dz.v[e] = round_to<T>(fmaf(k1.v[e], dy2[q].v[e], fmaf(k2.v[e], z2v[q].v[e], k3.v[e])));   // as a stored dz would read back
      if (m < Mout) tile[m] = dz;
    }
  }
  if (tid == 0) tile[Mout] = F{};
  __syncthreads();
  F wr[9], accw[9], dy[RPT];
#pragma unroll
  for (int t = 0; t < 9; ++t) { wr[t] = wl[t]; accw[t] = F{}; }
  float bsum[2 * V] = {};
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int m = tid + q * nt;
    dy[q] = F{};
    if (m >= M) { zv[q] = dy[q]; continue; }
    const int r = (int)dW.div(m), ww = m - r * g.Win, n = (int)dH.div(r), h = r - n * g.Hin;
    F t[9];
    // the nine values first, from the zero slot where no output pixel lies: no branches between the reads
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const int hn = h + 1 - i, ho = s == 2 ? hn >> 1 : hn;
      const int row = (unsigned)ho < (unsigned)g.Hout && !(s == 2 && (hn & 1)) ? (n * g.Hout + ho) * g.Wout : -1;
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const int wn = ww + 1 - j, wo = s == 2 ? wn >> 1 : wn;
        t[i * 3 + j] = tile[row >= 0 && (unsigned)wo < (unsigned)g.Wout && !(s == 2 && (wn & 1)) ? row + wo : Mout];
      }
    }
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const float z = zv[q].v[e], y = fmaf(z, sc[e], sh[e]), a = round_to<T>(clamp_act(y, lo, hi));
      float dA = 0.f;
#pragma unroll
      for (int k = 0; k < 9; ++k) {
        dA = fmaf(t[k].v[e], wr[k].v[e], dA);
        accw[k].v[e] = fmaf(t[k].v[e], a, accw[k].v[e]);
      }
      dA = round_to<T>(dA);                    // the data gradient as the separate kernels would store it
      const float v = y > lo && y < hi ? dA : 0.f;
      dy[q].v[e] = v;
      bsum[e] += v;
      bsum[V + e] = fmaf(v, z, bsum[V + e]);
    }
  }
  // block-wide sums in a fixed order: inside each wave, then the waves in order
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int e = 0; e < V; ++e) accw[t].v[e] = wave_sum_last(accw[t].v[e]);
#pragma unroll
  for (int e = 0; e < 2 * V; ++e) bsum[e] = wave_sum_last(bsum[e]);
  if (lead) {
#pragma unroll
    for (int t = 0; t < 9; ++t) *reinterpret_cast<F*>(&red[wave][t * V]) = accw[t];
#pragma unroll
    for (int e = 0; e < 2 * V; ++e) red[wave][9 * V + e] = bsum[e];
  }
  __syncthreads();
  asm volatile("" : "+v"(gw_old), "+v"(f_mu), "+v"(f_is), "+v"(f_g), "+v"(f_gg), "+v"(f_gb));
  if (tid < 9 * V) {
    double tot = 0.0;                        // up to sixteen wavefronts: no chain of that length in fp32
    for (int q = 0; q < nw; ++q) tot += red[q][tid];
    g_w[(size_t)(c0 + tid % V) * 9 + tid / V] = gw_old + (float)tot;
  } else if (tid >= 64 && tid < 64 + V) {
    const int e = tid - 64, c = c0 + e;
    double s0 = 0.0, s1 = 0.0;
    for (int q = 0; q < nw; ++q) { s0 += red[q][9 * V + e]; s1 += red[q][10 * V + e]; }
    const double mu = f_mu, is = f_is, gm = f_g;
    const double dbeta = s0, dgamma = is * (s1 - mu * s0);
    g_gamma[c] = f_gg + (float)dgamma;
    g_beta[c] = f_gb + (float)dbeta;
    const double k1 = gm * is, k2 = -k1 * is * dgamma * inv_M, k3 = -k1 * dbeta * inv_M - k2 * mu;
    coef[0].v[e] = (float)k1; coef[1].v[e] = (float)k2; coef[2].v[e] = (float)k3;
  }
  __syncthreads();
  const F k1 = coef[0], k2 = coef[1], k3 = coef[2];
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int m = tid + q * nt;
    if (m >= M) continue;
    F o;
#pragma unroll
    for (int e = 0; e < V; ++e) o.v[e] = fmaf(k1.v[e], dy[q].v[e], fmaf(k2.v[e], zv[q].v[e], k3.v[e]));
    store_chans(dz_prev + (size_t)m * C + c0, o);
  }
}

int dw_bwd_small_ok(const ConvGeom& g) {
  return (size_t)g.N * g.Hin * g.Win <= 2048 && g.Cout >= 32 && g.Cout % 8 == 0 && (g.stride == 1 || g.stride == 2);
}

void dw_bwd_small(int dt, hipStream_t st, const BnBwdIn& bo, const void* w, HView in, const ConvGeom& g,
                  const float* gamma, const float* mean, const float* invstd, float* g_w, float* g_gamma, float* g_beta,
                  void* dz_prev) {
  const size_t M = (size_t)g.N * g.Hin * g.Win, Mout = (size_t)g.N * g.Hout * g.Wout;
  const int es = dt == 0 ? 4 : 2;
  View v{in.z, in.scale, in.shift, in.act};
  KScope ks(st, "dw_bwd_small", ((double)M * g.Cout * 2 + (double)Mout * g.Cout * 2) * es, 42.0 * M * g.Cout, (long)M, g.Cout, g.stride);
  const FastDiv dW = FastDiv::of(g.Win), dH = FastDiv::of(g.Hin);
#define FTP_DW_SMALL(V, RPT, NT, THREADS)                                                                                       \
  FTP_DISPATCH(dt, hipLaunchKernelGGL((dw_bwd_small_k<T, V, RPT, NT>), dim3(g.Cout / V), dim3(THREADS), (Mout + 1) * 4 * V, st, bo, (const T*)w, v, g, \
                                      dW, dH, (int)M, (int)Mout, gamma, mean, invstd, g_w, g_gamma, g_beta, (T*)dz_prev))
  if (g.Cout <= 512 && M > 256) {
    if (M > 1024) FTP_DW_SMALL(2, 2, 1024, 1024);
    else FTP_DW_SMALL(2, 1, 1024, M > 512 ? 1024 : 512);
  } else if (M > 1024) FTP_DW_SMALL(4, 4, 512, 512);
  else if (M > 512) FTP_DW_SMALL(4, 2, 512, 512);
  else FTP_DW_SMALL(4, 1, 512, M > 256 ? 512 : 256);
#undef FTP_DW_SMALL
}

// ---- the whole backward of a depthwise layer in one pass ---------------------------------------------------------
// From the gradient dA of the layer's activated output (FORM: dz = k1 * gated dA + k2 * z + k3 is formed on the way into LDS and never written; else dz
// itself): data gradient, weight gradient (gw[block][9][C]: dW[tap] = sum over input pixels p of dz[the output that sees p at that tap] *
// activation[p]) and, where the input is the view prev of a raw output, the backward sums of that BatchNorm (as bn_bwd_reduce leaves them,
// sums[block][2][C]).  As passes of their own these move the expanded tensors nine times, here it is four and the halo.  A block takes `per` tiles of
// 8 x 16 pixels (bfloat16 at stride 1: 8 x 8) of 128 bytes of channels in a row, so that there are no more partials than kMaxPartials.  A thread owns four channels; stride 1: runs of four pixels
// with the six dz under each row of taps, in LDS in fp32 (converted once instead of for up to nine taps); stride 2: quads of 2 x 2 pixels, which
// four dz values reach (nine products, no parity to branch on).  The weights stay in LDS: in registers, one block less would fit a CU.
// Bound by memory at stride 2 (112x112x144, batch 64, bfloat16: 126 us, 4.7 TB/s; its passes were 18 + 48 + 106 + 70) and by vector instructions at stride 1,
// some 60 an output value in bfloat16, a third of them for the patch.  MobileNetV2 of width 1.4 at 224x224, batch 128: the 17 layers 1.8 ms a step (of kernels that run beside weight
// gradients); their data and weight gradients were 1.80 and the passes for dz and the sums another 0.9, on two streams (a step 7.27 -> 6.79 ms; 224x224 fp32 3.51 -> 3.21).
// bfloat16 tiles of 8 x 16 at stride 1: 207 registers, two blocks to a CU, or scratch with three: 1.12 and 1.24 ms for the stride-1 layers, 1.03 so.
// LEN: 0 blocks of a single tile, 1 of up to CHAIN, 2 of more (its own code, with the weights out of the way of the sums that meet inside the loop: for all, block 2 at 112x112 took 1 % longer).
// A block of a single tile requests the tile together with the weights and the partial sums.  The eleven sums of a block leave in one round
// through LDS, a wavefront to each in turn.  Both against a request after the prologue and four rounds of twelve numbers: the width-1.4 step
// 6.82 -> 6.77 ms, a 13-image step of width 0.5 at 161x193 1.070 -> 1.061.
struct DwBwdArgs {
  const void *dA, *w;       // dA: dz if nothing is to be formed
  View own;                 // the layer's own output (FORM)
  BnPending pend;           // its backward sums, if the blocks finish them (partial != nullptr), else coef[3][C]
  const float* coef;
  float *g_gamma, *g_beta;
  DwPlan d;
  int Hin, Win, Hout, Wout, C, per;
  void* dIn;                // may be nullptr, as sums
  float *sums, *gw;
  DwPrev prev;              // scale == nullptr: the input is stored as it is
};
__device__ __forceinline__ void keep_here(float4& v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }
template <typename T, int S> struct DwBwd {
  enum { F32 = sizeof(T) == 4, TW = S == 1 && !F32 ? 8 : 16,              // tiles of 8 x TW
         NR = S == 1 || F32 ? 1 : 2,                                             // rounds of a tile's runs or quads
         VS = F32 ? 32 : 64, PH = S == 1 ? 10 : 5, PW = S == 1 ? TW + 2 : 9 };          // the patch has its largest size whatever the tile: offsets are constants
  typedef typename std::conditional<S == 1, float, T>::type P;                                  // patch elements
  // the patch, or the sums of the layer's own BatchNorm; behind it the weights.  The eleven sums of all threads meet all over that, or, where another tile may follow, in front
  // of the weights.
  enum { PATCH = PH * PW * VS * sizeof(P) > kSlabSumsBytes ? PH * PW * VS * sizeof(P) : kSlabSumsBytes, RED = 11 * 256 * 16, STAGED = PATCH + 9 * VS * 4,
         LDS_ONE = STAGED > RED ? STAGED : RED, WEIGHTS = PATCH > RED ? PATCH : RED, LDS_MORE = WEIGHTS + 9 * VS * 4 };
  // Tiles whose values go through one chain of additions: at stride 1 68 for a tap or a sum, no more than in kernels of their own (a walk down strips for the weights: 12 rows
  // of two columns and more, then up to 64 strips; a pass for the sums: 75 rows, then 42 lanes); at stride 2 half as many and less for a tap, 100 to 200 for a sum.  Errors in
  // 2^-24 of the sums' r.m.s., 3.2 M rows, kernels of their own / one chain a block / this: fp32 stride 1 sums 3.0 and 4.0 / 5.0 and 4.3 / 3.0 and 2.7, weights 4.4 / 4.5 /
  // 2.8, bfloat16 weights 2.0 / 2.7 / 1.6; stride 2 sums 3.8 and 4.1 / 4.6 and 4.5 / 3.1 and 3.8, bfloat16 (whose terms have few bits) 1.2 and 3.2 / 1.2 and 2.5 / 1.0 and 1.6.
  // Width 1.4, batch 128: 105.2 us a launch, one chain a block 103.9; with chains of 12 and 8 tiles a step takes 1 % longer.
  enum { CHAIN = S == 1 ? 17 : 25 };
};
template <typename T, int S, bool FORM, int NV, int LEN>
__global__ __launch_bounds__(256, 3) void dw_bwd_k(DwBwdArgs p) {        // three blocks to a CU: 168 registers
  typedef DwBwd<T, S> X;
  typedef typename X::P PT;
  constexpr int NR = X::NR, VS = X::VS, PW = X::PW;
  constexpr bool ONE = LEN == 0;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  __shared__ __attribute__((aligned(16))) float vec[FORM ? 5 : 1][64], prv[2][64];
  __shared__ float met[LEN == 2 ? 11 : 1][64];        // sums of the chains that have met
  __builtin_amdgcn_s_setprio(3);                      // data-gradient chain: ahead of the weight-gradient stream's waves
  const DwPlan& d = p.d;
  const int C = p.C, Hin = p.Hin, Win = p.Win;
  PT* const patch = reinterpret_cast<PT*>(smem_raw);
  float* const wl = reinterpret_cast<float*>(smem_raw + (LEN == 2 ? X::WEIGHTS : X::PATCH));       // [9][VS]
  const int lb = xcd_logical_block();
  const int slab = lb % d.nslab, part = lb / d.nslab, cg0 = slab * d.CGB, t0 = part * p.per, t1 = min(t0 + p.per, d.ntiles);
  const int QB = 2 * d.CGB, seg0 = dw_div(threadIdx.x, d.m_qb), cq = threadIdx.x - seg0 * QB, c4 = cq * 4, gc = cg0 * 8 + c4;
  const int nc = min(C - cg0 * 8, d.CGB * 8);
  const bool worker = seg0 < d.spp && gc < C, viewed = p.prev.scale != nullptr;
  const float plo = act_lo(p.prev.act), phi = act_hi(p.prev.act), olo = act_lo(p.own.act), ohi = act_hi(p.own.act);
  // staging: thread = (pixel lane, column group)
  const int pl = dw_div(threadIdx.x, d.m_cgb), cg = threadIdx.x - pl * d.CGB;
  const bool stager = pl < d.PPB && cg0 + cg < C / 8;
  const int dph = dw_div(d.PPB, d.m_pw), dpw = d.PPB - dph * d.PW;
  const int ph_first = dw_div(pl, d.m_pw), pw_first = pl - ph_first * d.PW;
  int tw = t0 % d.tiles_w, th = t0 / d.tiles_w % d.tiles_h, n = t0 / (d.tiles_w * d.tiles_h);
  // a tile on its way: its patch, the input under it, and where they lie
  Raw<T> ra[NV], rz[FORM ? NV : 1];
  Raw4<T> zp[NR][4];
  unsigned ok = 0, inside = 0, at[NR];                // vectors and pixels inside the image; pixel of this thread's first run or quad
  int lds[NR], ph0 = 0, pw0 = 0;                      // where its dz lies in the patch, negative: none
  bool all_in = false;
  T* out = nullptr;
  auto request = [&]() __attribute__((always_inline)) {
    const int h0 = th * d.TH, w0 = tw * d.TW, ph_lo = S == 1 ? h0 - 1 : h0 / 2, pw_lo = S == 1 ? w0 - 1 : w0 / 2;
    // Where a thread works is decoded again for every tile: kept over the loop, the compiler holds some eighty registers of addresses
    ph0 = ph_first; pw0 = pw_first;
    int sg0 = seg0;
    asm volatile("" : "+v"(ph0), "+v"(pw0), "+v"(sg0));
    // the patch and the input under it, all requested together and unconditionally (outside: the image's first pixel, not used)
    ok = inside = 0;
    {
      const size_t img = (size_t)n * p.Hout * p.Wout * C + (stager ? (cg0 + cg) * 8 : 0);
      const T* A = reinterpret_cast<const T*>(p.dA) + img;
      const T* O = reinterpret_cast<const T*>(p.own.z) + img;
      unsigned off[NV];
      int ph = ph0, pw = pw0;
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        const int h = ph_lo + ph, x = pw_lo + pw;
        const bool in = stager && ph < d.PH && (unsigned)h < (unsigned)p.Hout && (unsigned)x < (unsigned)p.Wout;
        off[q] = in ? __umul24(__umul24(h, p.Wout) + x, C) : 0u;
        ok |= (in ? 1u : 0u) << q;
        ph += dph; pw += dpw;
        if (pw >= d.PW) { pw -= d.PW; ++ph; }
      }
#pragma unroll
      for (int q = 0; q < NV; ++q) {
        raw_load(ra[q], A + off[q]);
        if (FORM) raw_load(rz[FORM ? q : 0], O + off[q]);
      }
    }
    // nothing of the tile or its patch lies outside the image: a branch for the wavefront instead of a mask for every value
    all_in = h0 + d.TH <= Hin && w0 + d.TW <= Win && d.TW % 4 == 0 && d.TH % 2 == 0 && ph_lo >= 0 && pw_lo >= 0 && ph_lo + d.PH <= p.Hout && pw_lo + d.PW <= p.Wout;
    const size_t img = (size_t)n * Hin * Win * C + (worker ? gc : 0);
    const T* const Z = reinterpret_cast<const T*>(p.prev.z) + img;
    out = reinterpret_cast<T*>(p.dIn) + img;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int sg = sg0 + r * d.spp;
      const bool has = worker && sg < d.nseg;
      const int hl = dw_div(has ? sg : 0, d.m_segw), wl0 = (has ? sg : 0) - hl * d.segw, h = h0 + hl * S, x = w0 + wl0 * (S == 1 ? 4 : 2);
      lds[r] = has ? (hl * PW + wl0 * (S == 1 ? 4 : 1)) * VS + c4 : -1;
      at[r] = __umul24(h, Win) + x;
#pragma unroll
      for (int o = 0; o < 4; ++o) {
        const bool in = has && h + (S == 1 ? 0 : o >> 1) < Hin && x + (S == 1 ? o : o & 1) < Win;
        inside |= (in ? 1u : 0u) << (4 * r + o);
        raw4_load(zp[r][o], Z + (in ? __umul24(at[r] + (S == 1 ? o : (o >> 1) * Win + (o & 1)), C) : 0u));
      }
    }
  };
  // a block of a single tile: what depends on nothing is requested together, the tile, the weights and the sums (in front of a loop the compiler has no
  // registers for that)
  if (ONE) request();
  T w0[(9 * VS + 255) / 256];
#pragma unroll
  for (int q = 0; q < (9 * VS + 255) / 256; ++q) {
    const int i = threadIdx.x + q * 256, t = i / VS, c = i - t * VS;
    w0[q] = reinterpret_cast<const T*>(p.w)[c < nc && t < 9 ? (size_t)(cg0 * 8 + c) * 9 + t : 0];
  }
  if (viewed && (int)threadIdx.x < nc) { prv[0][threadIdx.x] = p.prev.scale[cg0 * 8 + threadIdx.x]; prv[1][threadIdx.x] = p.prev.shift[cg0 * 8 + threadIdx.x]; }
  if (FORM) {
    const int t = threadIdx.x, f = cg0 * 8 + (t < nc ? t : 0);
    const float osc = p.own.scale[f], osh = p.own.shift[f];
    if (p.pend.partial) {
      const bool write = part == 0 && t < nc;
      float g = p.pend.gamma[f], mu = p.pend.mean[f], is = p.pend.invstd[f], gg = 0.f, gb = 0.f;
      if (write) { gg = p.g_gamma[f]; gb = p.g_beta[f]; }
      const double inv_M = early_inverse((double)p.pend.M);
      double s0, s1;
      slab_sums(p.pend.partial, p.pend.P, C, cg0 * 8, nc, reinterpret_cast<double*>(smem_raw), s0, s1);
      asm volatile("" : "+v"(g), "+v"(mu), "+v"(is), "+v"(gg), "+v"(gb));
      if (t < nc) {
        const BwdChannel b = backward_channel(s0, s1, g, mu, is, inv_M);
        vec[FORM ? 2 : 0][t] = b.k1; vec[FORM ? 3 : 0][t] = b.k2; vec[FORM ? 4 : 0][t] = b.k3;
        if (write) { p.g_gamma[f] = gg + b.dgamma; p.g_beta[f] = gb + b.dbeta; }
      }
    } else if (t < nc) {
#pragma unroll
      for (int q = 0; q < 3; ++q) vec[FORM ? 2 + q : 0][t] = p.coef[q * C + f];
    }
    if (t < nc) { vec[0][t] = osc; vec[FORM ? 1 : 0][t] = osh; }
  }
#pragma unroll
  for (int q = 0; q < (9 * VS + 255) / 256; ++q) {
    const int i = threadIdx.x + q * 256, t = i / VS, c = i - t * VS;
    if (t < 9) wl[i] = c < nc ? to_f32(w0[q]) : 0.f;
  }
  __syncthreads();
  float4 aw[9], s1 = make_float4(0.f, 0.f, 0.f, 0.f), s2 = s1;
#pragma unroll
  for (int t = 0; t < 9; ++t) aw[t] = make_float4(0.f, 0.f, 0.f, 0.f);
  // The sums of a chain of tiles meet: the runs of a channel quad are spread over spp threads, eleven vectors of each go through LDS and are summed in a fixed order, a
  // wavefront to each vector in turn.
  auto meet = [&](const bool first, const bool last) __attribute__((always_inline)) {
    float4* const red = reinterpret_cast<float4*>(smem_raw);         // [11][256]
    const int tid = threadIdx.x, wave = tid >> 6, ch = tid & 63;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 9; ++t) red[t * 256 + tid] = aw[t];
    red[9 * 256 + tid] = s1;
    red[10 * 256 + tid] = s2;
    __syncthreads();
    if (ch >= nc) return;
    for (int v = wave; v < (p.sums ? 11 : 9); v += 4) {
      const float* src = reinterpret_cast<const float*>(red + v * 256) + ch;
      // four chains, 6 to 10 additions one behind the other in most layers.  In float64 the blocks of one tile took 4 to 10 % longer; as one chain in fp32 of 16 or 32 the error of fp32
      // layers with few rows was 2.0 where a pass has 1.7 (25088 x 96), so it is 1.4.
      float q[4] = {0.f, 0.f, 0.f, 0.f};
      int sgi = 0;
#pragma unroll 2
      for (; sgi + 3 < d.spp; sgi += 4)
#pragma unroll
        for (int u = 0; u < 4; ++u) q[u] += src[(sgi + u) * QB * 4];
      for (; sgi < d.spp; ++sgi) q[0] += src[sgi * QB * 4];
      float t = (q[0] + q[1]) + (q[2] + q[3]);
      if (!first) t += met[LEN == 2 ? v : 0][ch];
      float* dst = v < 9 ? p.gw + ((size_t)part * 9 + v) * C : p.sums + ((size_t)part * 2 + v - 9) * C;
      if (last) dst[cg0 * 8 + ch] = t;
      else met[LEN == 2 ? v : 0][ch] = t;
    }
  };
  for (int tile = t0; tile < (ONE ? t0 + 1 : t1); ++tile) {
    if (!ONE) request();
    if (!ONE && tile > t0) __syncthreads();           // the tile before has been read
    asm volatile("" ::: "memory");                    // the coefficients come from LDS again, not out of forty registers
    if (pl < d.PPB) {
#pragma unroll
      for (int half = 0; half < 2; ++half) {          // four channels at a time: their five coefficients are twenty registers
        const int c = cg * 8 + half * 4;
        float4 k1, k2, k3, sc, sh;
        if (FORM) { sc = ld4(vec[0] + c); sh = ld4(vec[FORM ? 1 : 0] + c); k1 = ld4(vec[FORM ? 2 : 0] + c); k2 = ld4(vec[FORM ? 3 : 0] + c); k3 = ld4(vec[FORM ? 4 : 0] + c); }
        int ph = ph0, pw = pw0;
#pragma unroll
        for (int q = 0; q < NV; ++q) {
          float4 v = raw_half(ra[q], half);
          if (FORM) {
            const float4 z = raw_half(rz[FORM ? q : 0], half), y = fma4(z, sc, sh);
            v = make_float4(y.x > olo && y.x < ohi ? v.x : 0.f, y.y > olo && y.y < ohi ? v.y : 0.f, y.z > olo && y.z < ohi ? v.z : 0.f, y.w > olo && y.w < ohi ? v.w : 0.f);
            v = round4<T>(fma4(k1, v, fma4(k2, z, k3)));  // as a stored dz would read back
          }
          if (!all_in && !(ok & (1u << q))) v = make_float4(0.f, 0.f, 0.f, 0.f);
          if (ph < d.PH) store4(patch + (ph * PW + pw) * VS + c, v);
          ph += dph; pw += dpw;
          if (pw >= d.PW) { pw -= d.PW; ++ph; }
        }
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    __syncthreads();
    if (++tw == d.tiles_w) { tw = 0; if (++th == d.tiles_h) { th = 0; ++n; } }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      // the rounds one behind the other, each with its own reads
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (lds[r] < 0) continue;
      const PT* const q = patch + lds[r];
      const float* const wt = wl + c4;
      const float4 psc = ld4(prv[0] + c4), psh = ld4(prv[1] + c4);       // not used where the input is no view
      auto input = [&](const int o) __attribute__((always_inline)) {
        const float4 z = raw4_unpack(zp[r][o]), y = fma4(z, psc, psh);
        float4 a = !viewed ? z : round4<T>(make_float4(clamp_act(y.x, plo, phi), clamp_act(y.y, plo, phi), clamp_act(y.z, plo, phi), clamp_act(y.w, plo, phi)));
        if (!all_in && !(inside >> (4 * r + o) & 1u)) a = make_float4(0.f, 0.f, 0.f, 0.f);
        return a;
      };
      auto leave = [&](const int o, const float4 v) __attribute__((always_inline)) {
        if (!(inside >> (4 * r + o) & 1u)) return;
        if (p.dIn) store4(out + __umul24(at[r] + (S == 1 ? o : (o >> 1) * Win + (o & 1)), C), v);
        const float4 g = round4<T>(v), z = raw4_unpack(zp[r][o]), y = fma4(z, psc, psh);             // sums over the values as stored
        const float4 t = make_float4(y.x > plo && y.x < phi ? g.x : 0.f, y.y > plo && y.y < phi ? g.y : 0.f, y.z > plo && y.z < phi ? g.z : 0.f,
                                     y.w > plo && y.w < phi ? g.w : 0.f);
        s1.x += t.x; s1.y += t.y; s1.z += t.z; s1.w += t.w;
        s2 = fma4(t, z, s2);
      };
      if constexpr (S == 1) {
        float4 v[4], a[4];
#pragma unroll
        for (int o = 0; o < 4; ++o) { a[o] = input(o); v[o] = make_float4(0.f, 0.f, 0.f, 0.f); }
#pragma unroll
        for (int k = 0; k < 3; ++k) {                 // row k of the patch under the run: taps 2 - k
          __builtin_amdgcn_sched_barrier(0);
          float4 g[6];
#pragma unroll
          for (int x = 0; x < 6; ++x) g[x] = load4(q + (k * PW + x) * VS);
#pragma unroll
          for (int j = 0; j < 3; ++j) {
            const int t = (2 - k) * 3 + j;
            const float4 w4 = ld4(wt + t * VS);
#pragma unroll
            for (int o = 0; o < 4; ++o) { v[o] = fma4(g[o + 2 - j], w4, v[o]); aw[t] = fma4(g[o + 2 - j], a[o], aw[t]); }
            keep_here(aw[t]);
          }
          // the products of a row of taps stay here: moved behind the branches of the results, all 27 vectors of LDS would be held until there
#pragma unroll
          for (int o = 0; o < 4; ++o) keep_here(v[o]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int o = 0; o < 4; ++o) leave(o, v[o]);
      } else {
        const float4 d00 = load4(q), d01 = load4(q + VS), d10 = load4(q + PW * VS), d11 = load4(q + (PW + 1) * VS);
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          const float4 a = input(o);
          float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
          auto tap = [&](const int t, const float4 g) __attribute__((always_inline)) { v = fma4(g, ld4(wt + t * VS), v); aw[t] = fma4(g, a, aw[t]); };
          if (o == 0) { tap(4, d00); }
          else if (o == 1) { tap(3, d01); tap(5, d00); }
          else if (o == 2) { tap(1, d10); tap(7, d00); }
          else { tap(0, d11); tap(2, d10); tap(6, d01); tap(8, d00); }
          leave(o, v);
        }
      }
    }
    if constexpr (LEN == 2) {
      const bool last = tile + 1 == t1;
      if (!last && (tile + 1 - t0) % X::CHAIN != 0) continue;
      meet(tile - t0 < X::CHAIN, last);
#pragma unroll
      for (int t = 0; t < 9; ++t) aw[t] = make_float4(0.f, 0.f, 0.f, 0.f);
      s1 = s2 = aw[0];
    }
  }
  if constexpr (LEN < 2) meet(true, true);
}

static DwPlan dw_bwd_plan(int dt, const ConvGeom& g, int* per, int* P) {
  DwPlan d = dw_plan(g.Cout, dt == 0 ? 4 : 2, false, g.Hin, g.Win, g.stride == 1 && dt != 0 ? DwBwd<bf16_t, 1>::TW : 16);       // tiles in input resolution
  // bfloat16 at stride 1: tiles of 7 rows take three passes to stage instead of four and nine tenths of the time; images of 7, 14 and 28 rows divide by them
  const int rows7 = (g.Hin + 6) / 7;
  if (g.stride == 1 && dt != 0 && d.TH == 8 && rows7 * 9 < d.tiles_h * 10) {
    d.TH = 7; d.tiles_h = rows7; d.nseg = d.TH * d.segw;
  }
  d.ntiles = g.N * d.tiles_h * d.tiles_w;
  if (g.stride == 1) {
    d.PH = d.TH + 2;
    d.PW = d.segw * 4 + 2;
  } else {
    d.segw = (d.TW + 1) / 2;
    d.nseg = (d.TH + 1) / 2 * d.segw;
    d.m_segw = dw_magic(d.segw);
    d.PH = (d.TH + 1) / 2 + 1;
    d.PW = d.segw + 1;
  }
  *per = (d.ntiles + kMaxPartials - 1) / kMaxPartials;
  *P = (d.ntiles + *per - 1) / *per;
  return d;
}
int dw_bwd_partials(int dt, const ConvGeom& g) {
  int per, P;
  dw_bwd_plan(dt, g, &per, &P);
  return P;
}
size_t dw_bwd_ws(int dt, const ConvGeom& g) { return (size_t)dw_bwd_partials(dt, g) * 9 * g.Cout; }

void dw_bwd(int dt, hipStream_t st, const void* dA, const HView* own, const BnPending* sums_in, const float* coef, float* g_gamma, float* g_beta, const void* w,
            const ConvGeom& g, void* dIn, HView in, float* sums, float* gw_part) {
  const int es = dt == 0 ? 4 : 2;
  int P;
  DwBwdArgs a{};
  a.d = dw_bwd_plan(dt, g, &a.per, &P);
  const size_t total = (size_t)g.N * g.Hin * g.Win, outs = (size_t)g.N * g.Hout * g.Wout;
  KScope ks(st, "dw_bwd", (2.0 * total + (own ? 2.0 : 1.0) * outs) * g.Cout * es + (double)P * 11 * g.Cout * 4, 36.0 * outs * g.Cout, (long)total, g.Cout, g.stride);
  // passes of the staging: a kernel for each number, so that registers are held and loads made for no more
  const int passes = (a.d.PH * a.d.PW + a.d.PPB - 1) / a.d.PPB, fill = g.stride == 2 ? (dt == 0 ? 1 : 2) : dt == 0 || passes <= 3 ? 3 : 4;
  if (!dw_check_plan(a.d, fill, dt == 0 || g.stride == 1 ? 1 : 2)) return;
  a.dA = dA; a.w = w; a.coef = coef; a.g_gamma = g_gamma; a.g_beta = g_beta;
  if (own) a.own = View{own->z, own->scale, own->shift, own->act};
  if (sums_in) a.pend = *sums_in;
  a.Hin = g.Hin; a.Win = g.Win; a.Hout = g.Hout; a.Wout = g.Wout; a.C = g.Cout;
  a.dIn = dIn; a.sums = sums; a.gw = gw_part;
  a.prev = DwPrev{in.z, in.scale, in.shift, in.act};
  if (a.d.PH > (g.stride == 1 ? 10 : 5) || a.d.PW > (g.stride == 1 ? (dt == 0 ? DwBwd<float, 1>::PW : DwBwd<bf16_t, 1>::PW) : 9)) { launch_plan_failed("depthwise backward patch beyond the kernel's"); return; }
  const dim3 grid((unsigned)P * a.d.nslab);
#define FTP_DW_BWD1(T, S, NV, LEN)                                                                            \
  do {                                                                                                        \
    const size_t lds = LEN == 2 ? DwBwd<T, S>::LDS_MORE : DwBwd<T, S>::LDS_ONE;                               \
    if (own) hipLaunchKernelGGL((dw_bwd_k<T, S, true, NV, LEN>), grid, dim3(256), lds, st, a);                \
    else hipLaunchKernelGGL((dw_bwd_k<T, S, false, NV, LEN>), grid, dim3(256), lds, st, a);                   \
  } while (0)
#define FTP_DW_BWD(T, S, NV)                                                                                  \
  do {                                                                                                        \
    if (a.per == 1) FTP_DW_BWD1(T, S, NV, 0);                                                                 \
    else if (a.per <= DwBwd<T, S>::CHAIN) FTP_DW_BWD1(T, S, NV, 1);                                           \
    else FTP_DW_BWD1(T, S, NV, 2);                                                                            \
  } while (0)
  if (g.stride == 2) { if (dt == 0) FTP_DW_BWD(float, 2, 1); else FTP_DW_BWD(bf16_t, 2, 2); }
  else if (dt == 0) FTP_DW_BWD(float, 1, 3);
  else if (fill == 3) FTP_DW_BWD(bf16_t, 1, 3);
  else FTP_DW_BWD(bf16_t, 1, 4);
#undef FTP_DW_BWD
#undef FTP_DW_BWD1
}

}  // namespace ftp
