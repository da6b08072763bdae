// Convolutions along one axis (1 x kw, stride 1, same length out as in), at most 64 channels on either side, as
// implicit GEMMs: row m of the patch matrix is kw neighbouring rows of the input, so the matrix is never written.  A tile
// of rows with its halo goes into LDS once (through the producer's BatchNorm + activation) and every tap reads it
// there at a row offset; rows are the flattened (window, position) index, so a tile may span windows of any length, and a tap
// that leaves its own window reads zero.  All products run on the fp32 MFMA (products of bfloat16 values are exact in it).
// What bounds them is that unit, 256 FLOP a cycle and CU (157 TFLOP/s): 64 -> 64 channels, 5 taps, 32768 rows is 8.5 us a pass.
#include "dev_common.h"
#include "kernels.h"
#include "bn_pending.h"

namespace ftp {

#define FTP_DISPATCH(dt, ...)                   \
  do {                                          \
    if ((dt) == 0) { typedef float T; __VA_ARGS__; } \
    else { typedef bf16_t T; __VA_ARGS__; }     \
  } while (0)

typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

struct Conv1dArgs {
  const void* x;      // the tensor read at row offsets: A (forward, weight gradient), dZ (data gradient)
  const void* w;      // [Cout][kw][Cin] (forward, data gradient); dZ (weight gradient)
  View view;          // of x: forward and weight gradient
  View prev;          // data gradient with sums: the BatchNorm + activation whose dA this is
  void* out;
  float* stats;       // [nranges][2][NC] or nullptr
  int M, W;           // rows, window length
  int C, NC;          // channels of x, output columns
  int Cin, Cout, kw, pad;   // pad: rows in front of the output row at tap 0
  int CP;             // C rounded up to 8: reduction index k = tap * CP + channel
  int itiles, jtiles, tiles_per_range;
  BnPending pend;     // few rows, forward: the BatchNorm of x is still partial sums
  float eps, momentum;
  FastDiv dC, dW;     // few rows: by C and by W
  // few rows, backward: pend.partial != nullptr: the BatchNorm + activation backward of this layer's own output is still to be done.  What is
  // given as dZ is the gradient of the activated output, own the output; dz = k1 * gated gradient + k2 * z + k3 is formed on the way
  // in, from partial sums that the layer behind has left, and never written.
  View own;
  float *g_gamma, *g_beta;
  int own_writes;
};

enum { kC1Chan = 64, kC1Taps = 9, kC1Small = 2048 };

// ---- row tiles: forward and data gradient ---------------------------------------------------------------------
// 4 wavefronts of 32 x 32 results: 64 rows x 64 columns (WC 2), or 64 x 32 with two wavefronts on each half of the reduction
// (WC 1).  Weights pass through LDS 64 reduction elements per wavefront at a time, the next chunk on its way in registers
// while one is multiplied.  64-row tiles leave two blocks per CU at 32768 rows (two wavefronts per SIMD hide each other's
// LDS reads and barriers); 64 -> 64 channels, 5 taps there: 20 us forward, 25 us data
// gradient; patch matrix + GEMM took 63 and 51.
template <typename T, bool DGRAD, int WC>
__global__ __launch_bounds__(256) void conv1d_rows_k(Conv1dArgs p) {
  constexpr int TI = 64, BC = 32 * WC, KS = 64, KC = KS * 2 / WC, WLD = KC + 4;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int LDR = (p.CP / 4) % 2 ? p.CP : p.CP + 4;       // an odd number of 16-byte units: rows fall into different banks
  const int prow = TI + p.kw - 1;                         // row prow is the zero row
  float* xs = smem;
  float* wsm = smem + (prow + 1) * LDR;                   // [2][BC][WLD]
  __shared__ float red[2][BC][2];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int wr = wave & 1, wc = WC == 2 ? wave >> 1 : 0, ks = WC == 2 ? 0 : wave >> 1;
  const int lb = xcd_logical_block();
  const int jt = lb % p.jtiles, range = lb / p.jtiles;
  const int j0 = jt * BC;
  const int KP = p.kw * p.CP, nchunk = (KP + KC - 1) / KC;
  const T* X = reinterpret_cast<const T*>(p.x);
  const T* Wt = reinterpret_cast<const T*>(p.w);
  const bool vec = p.C % 8 == 0;
  const bool view = !DGRAD && p.view.scale != nullptr;
  const float lo = act_lo(p.view.act), hi = act_hi(p.view.act);
  const int it_beg = range * p.tiles_per_range, it_end = min(it_beg + p.tiles_per_range, p.itiles);
  const unsigned cp_magic = 65536u / (unsigned)p.CP + 1u;     // k / CP, exact for k * CP < 65536: k < 9 * 64 + 128 with the last chunk's end, CP <= 64

  // weight chunk kc into registers / from there into LDS (column-major: a column's chunk is contiguous)
  constexpr int WE = BC * KC / 256;
  float wreg[WE];
  auto fetch_w = [&](int kc) {
    if (!DGRAD && vec) {
#pragma unroll
      for (int s = 0; s < WE / 8; ++s) {
        const int v = tid + 256 * s, col = v / (KC / 8), k = kc * KC + (v % (KC / 8)) * 8;
        const bool in = j0 + col < p.NC && k < KP;            // CP == C: k is the offset in a weight row
        load8(Wt + (in ? (size_t)(j0 + col) * KP + k : 0), wreg + 8 * s);
#pragma unroll
        for (int e = 0; e < 8; ++e) wreg[8 * s + e] = in ? wreg[8 * s + e] : 0.f;
      }
    } else if (DGRAD && p.NC % 4 == 0) {                      // CP == C here too: k / C is the tap, k % C the channel of dZ
#pragma unroll
      for (int s = 0; s < WE / 4; ++s) {
        const int v = tid + 256 * s, col = v % (BC / 4) * 4, k = kc * KC + v / (BC / 4);
        const int tap = (int)(((unsigned)k * cp_magic) >> 16), c = k - tap * p.CP;
        const bool in = j0 + col < p.NC && k < KP;
        const float4 x = load4(Wt + (in ? ((size_t)c * p.kw + (p.kw - 1 - tap)) * p.Cin + j0 + col : 0));
        wreg[4 * s] = in ? x.x : 0.f; wreg[4 * s + 1] = in ? x.y : 0.f; wreg[4 * s + 2] = in ? x.z : 0.f; wreg[4 * s + 3] = in ? x.w : 0.f;
      }
    } else {
#pragma unroll
      for (int s = 0; s < WE; ++s) {
        const int e = tid + 256 * s;
        const int col = DGRAD ? e % BC : e / KC, kk = DGRAD ? e / BC : e % KC;
        const int k = kc * KC + kk, tap = (int)(((unsigned)k * cp_magic) >> 16), c = k - tap * p.CP;
        const bool in = j0 + col < p.NC && k < KP && c < p.C;
        const size_t at = DGRAD ? ((size_t)c * p.kw + (p.kw - 1 - tap)) * p.Cin + j0 + col : ((size_t)(j0 + col) * p.kw + tap) * p.Cin + c;
        const float x = to_f32(Wt[in ? at : 0]);
        wreg[s] = in ? x : 0.f;
      }
    }
  };
  auto commit_w = [&](int buf) {
    float* dst = wsm + buf * BC * WLD;
    if (!DGRAD && vec) {
#pragma unroll
      for (int s = 0; s < WE / 8; ++s) {
        const int v = tid + 256 * s;
        store8(dst + v / (KC / 8) * WLD + v % (KC / 8) * 8, wreg + 8 * s);
      }
    } else if (DGRAD && p.NC % 4 == 0) {
#pragma unroll
      for (int s = 0; s < WE / 4; ++s) {
        const int v = tid + 256 * s;
#pragma unroll
        for (int f = 0; f < 4; ++f) dst[(v % (BC / 4) * 4 + f) * WLD + v / (BC / 4)] = wreg[4 * s + f];
      }
    } else {
#pragma unroll
      for (int s = 0; s < WE; ++s) {
        const int e = tid + 256 * s;
        const int col = DGRAD ? e % BC : e / KC, kk = DGRAD ? e / BC : e % KC;
        dst[col * WLD + kk] = wreg[s];
      }
    }
  };

  for (int c = tid; c < LDR; c += 256) xs[prow * LDR + c] = 0.f;
  float s1 = 0.f, s2 = 0.f;
  const int col = j0 + wc * 32 + l32;
  const bool col_ok = col < p.NC;
  float psc = 0.f, psh = 0.f;
  const bool sums = DGRAD && p.stats != nullptr;
  if (sums && col_ok) { psc = p.prev.scale[col]; psh = p.prev.shift[col]; }
  const float plo = act_lo(p.prev.act), phi = act_hi(p.prev.act);
  for (int it = it_beg; it < it_end; ++it) {
    const int m0 = it * TI;
    fetch_w(0);
    const int mb = m0 + wr * 32 + 4 * h;                // rows of this lane's results, see below
    float zp[16];
    if (sums) {
      const T* Z = reinterpret_cast<const T*>(p.prev.z);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int m = mb + 8 * (r >> 2) + (r & 3);
        zp[r] = to_f32(Z[col_ok && m < p.M ? (size_t)m * p.NC + col : 0]);
      }
    }
    __syncthreads();                                    // the tile before has been read
    if (vec) {
      const int CG = p.CP / 8, nv = prow * CG;
      for (int v0 = tid; v0 < nv; v0 += 4 * 256) {
        float val[4][8];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int v = v0 + 256 * s, r = v / CG, m = m0 - p.pad + r;
          load8(X + (v < nv && m >= 0 && m < p.M ? (size_t)m * p.C + (v - r * CG) * 8 : 0), val[s]);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int v = v0 + 256 * s, r = v / CG, cg = v - r * CG, m = m0 - p.pad + r;
          if (v >= nv) break;
          const bool in = m >= 0 && m < p.M;
          if (view) {
            float sc[8], sh[8];
            load8(p.view.scale + cg * 8, sc);
            load8(p.view.shift + cg * 8, sh);
#pragma unroll
            for (int e = 0; e < 8; ++e) val[s][e] = round_to<T>(clamp_act(fmaf(val[s][e], sc[e], sh[e]), lo, hi));
          }
#pragma unroll
          for (int e = 0; e < 8; ++e) val[s][e] = in ? val[s][e] : 0.f;
          store8(xs + r * LDR + cg * 8, val[s]);
        }
      }
    } else {
      const int n = prow * p.CP;
      for (int i0 = tid; i0 < n; i0 += 4 * 256) {
        float val[4];
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int i = i0 + 256 * s, r = i / p.CP, c = i - r * p.CP, m = m0 - p.pad + r;
          const bool in = i < n && m >= 0 && m < p.M && c < p.C;
          val[s] = to_f32(X[in ? (size_t)m * p.C + c : 0]);
          if (view) val[s] = round_to<T>(clamp_act(fmaf(val[s], p.view.scale[in ? c : 0], p.view.shift[in ? c : 0]), lo, hi));
          val[s] = in ? val[s] : 0.f;
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int i = i0 + 256 * s, r = i / p.CP;
          if (i < n) xs[r * LDR + i - r * p.CP] = val[s];
        }
      }
    }
    commit_w(0);
    __syncthreads();
    const int mrow = m0 + wr * 32 + l32;
    const int t = mrow < p.M ? (int)((unsigned)mrow % (unsigned)p.W) : -(1 << 20);   // a row past the end is outside every window
    // a chain of fp32 additions per weight chunk, not one through the whole reduction: 64 -> 64 channels, 9 taps were 4.3e-7 off the exact
    // result (2-norm), 1.6e-7 like this; the additions are a thirtieth of the matrix instructions' time
    f16v acc, tot;
#pragma unroll
    for (int e = 0; e < 16; ++e) tot[e] = 0.f;
    auto tap_row = [&](int tp) { return xs + ((unsigned)(t + tp - p.pad) < (unsigned)p.W ? wr * 32 + l32 + tp : prow) * LDR + 4 * h; };
    for (int kc = 0; kc < nchunk; ++kc) {
      if (kc + 1 < nchunk) fetch_w(kc + 1);
      const float* brow = wsm + (kc & 1) * BC * WLD + (wc * 32 + l32) * WLD + ks * KS + 4 * h;
      const int k0 = kc * KC + ks * KS, nq = min(KS, KP - k0) / 8;      // KP is a multiple of 8; may be past the end
      int tap = (int)(((unsigned)k0 * cp_magic) >> 16), c0 = k0 - tap * p.CP;
      if (tap > p.kw) tap = p.kw;
      const float* arow = tap_row(tap);
      float4 a = ld4(arow + c0), b = ld4(brow);
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.f;
      for (int q = 0; q < nq; ++q) {                    // the next operands are on their way while four products run
        c0 += 8;
        if (c0 == p.CP) { c0 = 0; ++tap; arow = tap_row(tap); }       // behind the last tap: at most the zero row, not used
        const float4 an = ld4(arow + c0), bn = ld4(brow + 8 * (q + 1 < nq ? q + 1 : q));
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
        a = an; b = bn;
      }
#pragma unroll
      for (int e = 0; e < 16; ++e) tot[e] += acc[e];
      if (kc + 1 < nchunk) {
        commit_w((kc + 1) & 1);                         // the buffer read before this chunk: all have passed the barrier behind it
        __syncthreads();
      }
    }
    if constexpr (WC == 1) {                            // the two halves of the reduction meet
      __syncthreads();
      float* half = wsm + wr * 16 * 64 + lane;
      if (ks == 1)
#pragma unroll
        for (int r = 0; r < 16; ++r) half[r * 64] = tot[r];
      __syncthreads();
      if (ks == 1) continue;
#pragma unroll
      for (int r = 0; r < 16; ++r) tot[r] += half[r * 64];
    }
    // register r: row 8 * (r / 4) + 4 * h + r % 4, column l32
    T* out = reinterpret_cast<T*>(p.out);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int m = mb + 8 * (r >> 2) + (r & 3);
      const bool ok = col_ok && m < p.M;
      if (ok) out[(size_t)m * p.NC + col] = from_f32<T>(tot[r]);
      const float v = round_to<T>(tot[r]);              // sums are those of the values as stored
      if (sums) {
        // chosen, not multiplied: a gradient that is not finite stays out of the sums of a channel that is off
        const float yp = fmaf(zp[r], psc, psh);
        const float dy = ok && (p.prev.act == ACT_NONE || (yp > plo && yp < phi)) ? v : 0.f;
        s1 += dy;
        s2 += ok ? dy * zp[r] : 0.f;
      } else {
        s1 += ok ? v : 0.f;
        s2 += ok ? v * v : 0.f;
      }
    }
  }
  if (p.stats) {
    s1 += __shfl_xor(s1, 32, 64);
    s2 += __shfl_xor(s2, 32, 64);
    if (h == 0 && ks == 0) { red[0][wc * 32 + l32][wr] = s1; red[1][wc * 32 + l32][wr] = s2; }
    __syncthreads();
    if (tid < 2 * BC) {
      const int sq = tid / BC, c = tid % BC;
      if (j0 + c < p.NC) p.stats[((size_t)range * 2 + sq) * p.NC + j0 + c] = red[sq][c][0] + red[sq][c][1];
    }
  }
}

// ---- weight gradient over row tiles ---------------------------------------------------------------------------
// A block takes a range of 64-row tiles (dZ and the input with its halo in LDS) and a set of 32 x 80 pieces of
// g_w [Cout][kw * Cin]: a wavefront keeps 2 x 5 tiles of 16 x 16 in accumulators over all its rows and reads seven LDS words for
// ten MFMAs.  Pieces that leave wavefronts over share their rows among them.  One partial per block and row share.  64 -> 64
// channels, 32768 rows: 28 us (patch matrix + GEMM 73); the next tile in registers while one is multiplied, or four row groups'
// LDS reads together, measured no faster.
struct Conv1dWgArgs {
  Conv1dArgs c;
  int nco, nkg;            // pieces along Cout (32 each) and along kw * Cin (80 each)
  int gpb, rs;             // pieces per block, wavefronts that share a piece's rows: gpb * rs <= 4
  int ngrp;                // blocks per row range
};
enum { kC1WgRows = 64, kC1RT = 2, kC1CT = 5 };

template <typename T>
__global__ __launch_bounds__(256) void conv1d_wgrad_k(Conv1dWgArgs a) {
  const Conv1dArgs& p = a.c;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  // 16 or 48 banks between rows: the four rows of an MFMA operand fall into different banks
  const int LDR = (p.Cin + 31) / 32 * 32 + 16, LDZ = (p.Cout + 31) / 32 * 32 + 16;
  const int prow = kC1WgRows + p.kw - 1;
  float* xs = smem;
  float* ds = smem + prow * LDR;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, rg = lane >> 4;
  const int grp = blockIdx.x % a.ngrp, range = blockIdx.x / a.ngrp;
  const int piece = grp * a.gpb + wave % a.gpb, rsub = wave / a.gpb;
  const bool live = piece < a.nco * a.nkg && rsub < a.rs;
  const int pco = piece % a.nco, pkg = piece / a.nco;
  const int K = p.kw * p.Cin;
  const T* X = reinterpret_cast<const T*>(p.x);
  const T* D = reinterpret_cast<const T*>(p.w);
  const bool view = p.view.scale != nullptr;
  const float lo = act_lo(p.view.act), hi = act_hi(p.view.act);
  int off[kC1CT], tj[kC1CT], doff[kC1RT];
#pragma unroll
  for (int q = 0; q < kC1CT; ++q) {
    const int k = (pkg * kC1CT + q) * 16 + l16;
    const int tap = k / p.Cin;
    off[q] = k < K ? tap * LDR + (k - tap * p.Cin) : 0;
    tj[q] = k < K ? tap - p.pad : -(1 << 20);           // a column past the end is outside every window
  }
#pragma unroll
  for (int q = 0; q < kC1RT; ++q) {
    const int co = (pco * kC1RT + q) * 16 + l16;
    doff[q] = co < p.Cout ? co : 0;                     // its results are not written
  }
  f4v acc[kC1RT][kC1CT];
#pragma unroll
  for (int i = 0; i < kC1RT; ++i)
#pragma unroll
    for (int q = 0; q < kC1CT; ++q) acc[i][q] = f4v{0.f, 0.f, 0.f, 0.f};

  const int it_end = min((range + 1) * p.tiles_per_range, p.itiles);
  for (int it = range * p.tiles_per_range; it < it_end; ++it) {
    const int m0 = it * kC1WgRows;
    __syncthreads();
    {
      const int CG = p.Cout / 8, nv = kC1WgRows * CG;
      for (int v = tid; v < nv; v += 256) {
        const int r = v / CG, cg = v - r * CG, m = m0 + r;
        const bool in = m < p.M;
        float val[8];
        load8(D + (in ? (size_t)m * p.Cout + cg * 8 : 0), val);
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = in ? val[e] : 0.f;
        store8(ds + r * LDZ + cg * 8, val);
      }
    }
    if (p.Cin % 8 == 0) {
      const int CG = p.Cin / 8, nv = prow * CG;
      for (int v = tid; v < nv; v += 256) {
        const int r = v / CG, cg = v - r * CG, m = m0 - p.pad + r;
        const bool in = m >= 0 && m < p.M;
        float val[8];
        load8(X + (in ? (size_t)m * p.Cin + cg * 8 : 0), val);
        if (view) {
          float sc[8], sh[8];
          load8(p.view.scale + cg * 8, sc);
          load8(p.view.shift + cg * 8, sh);
#pragma unroll
          for (int e = 0; e < 8; ++e) val[e] = round_to<T>(clamp_act(fmaf(val[e], sc[e], sh[e]), lo, hi));
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = in ? val[e] : 0.f;
        store8(xs + r * LDR + cg * 8, val);
      }
    } else {
      for (int i = tid; i < prow * p.Cin; i += 256) {
        const int r = i / p.Cin, c = i - r * p.Cin, m = m0 - p.pad + r;
        const bool in = m >= 0 && m < p.M;
        float x = to_f32(X[in ? (size_t)m * p.Cin + c : 0]);
        if (view) x = round_to<T>(clamp_act(fmaf(x, p.view.scale[c], p.view.shift[c]), lo, hi));
        xs[r * LDR + c] = in ? x : 0.f;
      }
    }
    __syncthreads();
    if (live) {
      const int r_step = 4 * a.rs;
      int t = (int)((unsigned)(m0 + 4 * rsub + rg) % (unsigned)p.W);
      for (int r = 4 * rsub + rg; r < kC1WgRows; r += r_step) {
        const bool row_ok = m0 + r < p.M;
        float d[kC1RT], x[kC1CT];
#pragma unroll
        for (int q = 0; q < kC1RT; ++q) d[q] = ds[r * LDZ + doff[q]];
#pragma unroll
        for (int q = 0; q < kC1CT; ++q) x[q] = xs[r * LDR + off[q]];
#pragma unroll
        for (int q = 0; q < kC1CT; ++q) x[q] = row_ok && (unsigned)(t + tj[q]) < (unsigned)p.W ? x[q] : 0.f;
#pragma unroll
        for (int q = 0; q < kC1CT; ++q)
#pragma unroll
          for (int i = 0; i < kC1RT; ++i) acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[i], x[q], acc[i][q], 0, 0, 0);
        t += r_step;                                    // at most 16, and a window has at least 16 rows
        t -= t >= p.W ? p.W : 0;
      }
    }
  }
  if (!live) return;
  float* out = reinterpret_cast<float*>(p.out) + (size_t)(range * a.rs + rsub) * p.Cout * K;
#pragma unroll
  for (int i = 0; i < kC1RT; ++i)
#pragma unroll
    for (int q = 0; q < kC1CT; ++q) {
      const int k = (pkg * kC1CT + q) * 16 + l16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int co = (pco * kC1RT + i) * 16 + 4 * rg + r;
        if (co < p.Cout && k < K) out[(size_t)co * K + k] = acc[i][q][r];
      }
    }
}

// ---- few rows: latency only ----------------------------------------------------------------------------------
// 16 x 16 results of forward or data gradient by four wavefronts that split the reduction, fragments straight from global
// memory (1024 rows, 64 -> 64 channels: 4.9 us; patch matrix, padded weights and GEMM were three launches of 11) with up to five steps in flight (64 channels x 5 taps: one trip), wavefronts meet in LDS.  CV: channels of x are
// a multiple of 4, so a lane's four reduction elements lie in one tap and in one vector.
template <typename T, bool DGRAD, bool CV, int NW, bool PRO = false>
__device__ __forceinline__ void conv1d_tile(const Conv1dArgs& p, const int bid) {
  constexpr int U = 5, GROUPS = NW / 4;
  __shared__ float red[GROUPS][4][16][17];
  __shared__ float sred[GROUPS][2][16][17];
  const int grp = threadIdx.x >> 8, wave = (threadIdx.x >> 6) & 3, lane = threadIdx.x & 63;
  const int tile = bid * GROUPS + grp;
  const bool tile_ok = tile < p.itiles * p.jtiles;
  const int jt = tile % p.jtiles, it = tile / p.jtiles;
  const int m0 = it * 16, j0 = jt * 16, l16 = lane & 15, kg = (lane >> 4) * 4;
  const int K = p.kw * p.C, nst = (K + 15) / 16, sb = wave * nst / 4, se = (wave + 1) * nst / 4;
  const int row = m0 + l16, col = j0 + l16;
  const bool row_ok = tile_ok && row < p.M, col_ok = tile_ok && col < p.NC;
  const int t = row - (int)p.dW.div(row) * p.W;
  const T* X = reinterpret_cast<const T*>(p.x);
  const T* Wt = reinterpret_cast<const T*>(p.w);
  const bool view = !DGRAD && p.view.scale != nullptr, pending = !DGRAD && p.pend.partial != nullptr;
  __shared__ double fin[DGRAD ? (PRO ? 64 * NW : 1) : 256];
  __shared__ __attribute__((aligned(16))) float vec[DGRAD ? (PRO ? 5 : 1) : 2][kC1Chan];
  const float lo = DGRAD ? act_lo(p.own.act) : act_lo(p.view.act), hi = DGRAD ? act_hi(p.own.act) : act_hi(p.view.act);
  const T* Z = reinterpret_cast<const T*>(p.own.z);
  // data gradient with sums: the prev tensor at the element this thread writes, requested now
  const int orow = (threadIdx.x >> 4) & 15, ocol = threadIdx.x & 15;
  const bool in_out = tile_ok && m0 + orow < p.M && j0 + ocol < p.NC, sums = DGRAD && p.stats != nullptr;
  T zp = T();
  float psc = 0.f, psh = 0.f;
  if (sums) {
    const int pc = in_out ? j0 + ocol : 0;
    zp = reinterpret_cast<const T*>(p.prev.z)[in_out ? (size_t)(m0 + orow) * p.NC + pc : 0];
    psc = p.prev.scale[pc]; psh = p.prev.shift[pc];
  }
  f4v acc = {0.f, 0.f, 0.f, 0.f};
  float a[U][4], b[U][4], sc[U][4], sh[U][4], zz[PRO ? U : 1][4];
  bool ok[U][4], kin[U][4];
  int ch[U][4];
  auto request = [&](const int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int e = 0; e < 4; ++e) kin[u][e] = ok[u][e] = false;
      if (s0 + u >= se) continue;                       // the wavefront as a whole
#pragma unroll
      for (int e = 0; e < 4; e += CV ? 4 : 1) {
        const int k = (s0 + u) * 16 + kg + e;
        kin[u][e] = k < K;
        const int kc = kin[u][e] ? k : 0, tap = (int)p.dC.div(kc), c = kc - tap * p.C;
        ch[u][e] = c;
        ok[u][e] = kin[u][e] && row_ok && (unsigned)(t + tap - p.pad) < (unsigned)p.W;
        const size_t xa = ok[u][e] ? (size_t)(row + tap - p.pad) * p.C + c : 0;
        const int cc = col_ok ? col : 0;
        if constexpr (CV) {
          *reinterpret_cast<float4*>(a[u]) = load4(X + xa);
          if (PRO) *reinterpret_cast<float4*>(zz[PRO ? u : 0]) = load4(Z + xa);
          if (view && !pending) { *reinterpret_cast<float4*>(sc[u]) = ld4(p.view.scale + c); *reinterpret_cast<float4*>(sh[u]) = ld4(p.view.shift + c); }
          if constexpr (!DGRAD) *reinterpret_cast<float4*>(b[u]) = load4(Wt + (size_t)cc * K + kc);
          else
#pragma unroll
            for (int f = 0; f < 4; ++f) b[u][f] = to_f32(Wt[((size_t)(c + f) * p.kw + (p.kw - 1 - tap)) * p.Cin + cc]);
        } else {
          a[u][e] = to_f32(X[xa]);
          if (view && !pending) { sc[u][e] = p.view.scale[c]; sh[u][e] = p.view.shift[c]; }
          b[u][e] = to_f32(Wt[DGRAD ? ((size_t)c * p.kw + (p.kw - 1 - tap)) * p.Cin + cc : (size_t)cc * K + kc]);
        }
      }
    }
  };
  // the first round's fragments travel while the statistics are finished
  request(sb);
  if (PRO && threadIdx.x < p.C) { vec[PRO ? 3 : 0][threadIdx.x] = p.own.scale[threadIdx.x]; vec[PRO ? 4 : 0][threadIdx.x] = p.own.shift[threadIdx.x]; }
  if (PRO) finish_backward_n(p.pend, p.C, p.g_gamma, p.g_beta, bid == 0, 64 * NW, fin, vec);
  if (pending) finish_pending_n(p.pend, p.C, 0, p.C, p.eps, p.momentum, bid == 0, 256, fin, vec[0], vec[DGRAD ? 0 : 1]);
  for (int s0 = sb; s0 < se; s0 += U) {
    if (s0 != sb) request(s0);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (s0 + u >= se) break;
      float own[PRO ? 5 : 1][4];
      if (PRO)
#pragma unroll
        for (int q = 0; q < 5; ++q) *reinterpret_cast<float4*>(own[PRO ? q : 0]) = ld4(&vec[PRO ? q : 0][ch[u][0]]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (pending) { const int c = CV ? ch[u][0] + e : ch[u][e]; sc[u][e] = vec[0][c]; sh[u][e] = vec[DGRAD ? 0 : 1][c]; }
        const bool in = ok[u][CV ? 0 : e], kn = kin[u][CV ? 0 : e];
        float x = a[u][e];
        if constexpr (PRO) {
          const float y = fmaf(zz[u][e], own[3][e], own[4][e]);
          x = round_to<T>(fmaf(own[0][e], y > lo && y < hi ? x : 0.f, fmaf(own[1][e], zz[u][e], own[2][e])));
        }
        if (view) x = round_to<T>(clamp_act(fmaf(x, sc[u][e], sh[u][e]), lo, hi));
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? x : 0.f, kn ? b[u][e] : 0.f, acc, 0, 0, 0);
      }
    }
  }
  // (a row or column outside the tensor, or a step past the end, contributed 0 x 0; a column outside is not written)
#pragma unroll
  for (int r = 0; r < 4; ++r) red[grp][wave][4 * (lane >> 4) + r][l16] = acc[r];
  __syncthreads();
  const bool in = in_out;
  const float v = red[grp][0][orow][ocol] + red[grp][1][orow][ocol] + red[grp][2][orow][ocol] + red[grp][3][orow][ocol];
  if (in) reinterpret_cast<T*>(p.out)[(size_t)(m0 + orow) * p.NC + j0 + ocol] = from_f32<T>(v);
  if (p.stats) {
    float sv = in ? round_to<T>(v) : 0.f, other = sv;
    if (DGRAD) {                            // chosen, not multiplied, as in conv1d_rows_k
      other = to_f32(zp);
      const float y = fmaf(other, psc, psh);
      sv = p.prev.act == ACT_NONE || (y > act_lo(p.prev.act) && y < act_hi(p.prev.act)) ? sv : 0.f;
    }
    sred[grp][0][orow][ocol] = sv;
    sred[grp][1][orow][ocol] = in ? sv * other : 0.f;
    __syncthreads();
    if ((threadIdx.x & 255) < 32 && tile_ok) {
      const int sq = (threadIdx.x >> 4) & 1, c = threadIdx.x & 15;
      float tot = 0.f;
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) tot += sred[grp][sq][rr][c];
      if (j0 + c < p.NC) p.stats[((size_t)it * 2 + sq) * p.NC + j0 + c] = tot;
    }
  }
}

template <typename T, bool CV>
__global__ __launch_bounds__(256) void conv1d_fwd_small_k(Conv1dArgs p) { conv1d_tile<T, false, CV, 4>(p, xcd_logical_block()); }

// 16 x 16 of g_w by 16 wavefronts that split the rows: no partial buffers, one round of sixteen row groups up to 1024 rows, two at 2048
template <typename T, bool PRO, int NW>
__device__ __forceinline__ void conv1d_wgrad_tile(const Conv1dArgs& p, float* __restrict__ g_w, const int bid) {
  constexpr int U = 16;
  __shared__ float red[NW][16][17];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15, mg = lane >> 4;
  const int K = p.kw * p.Cin, jt_n = (K + 15) / 16;
  const int jt = bid % jt_n, it = bid / jt_n;
  const int co = it * 16 + l16, k = jt * 16 + l16;
  const bool co_ok = co < p.Cout, k_ok = k < K;
  const int tap = k_ok ? k / p.Cin : 0, ci = k_ok ? k - tap * p.Cin : 0, dt = tap - p.pad;
  const T* D = reinterpret_cast<const T*>(p.w) + (co_ok ? co : 0);
  const T* X = reinterpret_cast<const T*>(p.x) + ci;
  const T* Z = reinterpret_cast<const T*>(p.own.z) + (co_ok ? co : 0);
  __shared__ double fin[PRO ? 64 * NW : 1];
  __shared__ float vec[3][kC1Chan];
  float osc = 0.f, osh = 0.f, k1 = 0.f, k2 = 0.f, k3 = 0.f;
  const float olo = act_lo(p.own.act), ohi = act_hi(p.own.act);
  if (PRO) { osc = p.own.scale[co_ok ? co : 0]; osh = p.own.shift[co_ok ? co : 0]; }
  const bool view = p.view.scale != nullptr;
  const float sc = view ? p.view.scale[ci] : 1.f, sh = view ? p.view.shift[ci] : 0.f;
  const float lo = act_lo(p.view.act), hi = act_hi(p.view.act);
  // the gradient element this thread adds to, requested now
  const int orow = (threadIdx.x >> 4) & 15, ocol = threadIdx.x & 15;
  const bool writer = threadIdx.x < 256 && it * 16 + orow < p.Cout && jt * 16 + ocol < K;
  float* dst = g_w + (writer ? (size_t)(it * 16 + orow) * K + jt * 16 + ocol : 0);
  float g_old = writer ? *dst : 0.f;
  const int per = (p.M + 4 * NW - 1) / (4 * NW) * 4, mb = wave * per, me = min(mb + per, p.M);
  f4v acc = {0.f, 0.f, 0.f, 0.f};
  int t = mb + mg - (int)p.dW.div(mb + mg) * p.W;
  T dr[U], xr[U], zr[PRO ? U : 1];
  bool xin[U];
  auto request = [&](const int m) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int mm = m + 4 * u + mg;
      xin[u] = mm < me && k_ok && (unsigned)(t + dt) < (unsigned)p.W;
      const size_t at = (size_t)(mm < me ? mm : mb < p.M ? mb : 0) * p.Cout;
      dr[u] = D[at];
      if (PRO) zr[PRO ? u : 0] = Z[at];
      xr[u] = X[xin[u] ? (size_t)(mm + dt) * p.Cin : 0];
      t += 4;
      t -= t >= p.W ? p.W : 0;
    }
  };
  request(mb);
  if constexpr (PRO) {
    finish_backward_n(p.pend, p.Cout, p.g_gamma, p.g_beta, p.own_writes && bid == 0, 64 * NW, fin, vec);
    const int c = co_ok ? co : 0;
    k1 = vec[0][c]; k2 = vec[1][c]; k3 = vec[2][c];
  }
  for (int m = mb; m < me; m += 4 * U) {
    if (m != mb) request(m);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x = to_f32(xr[u]);
      if (view) x = round_to<T>(clamp_act(fmaf(x, sc, sh), lo, hi));
      const bool din = m + 4 * u + mg < me && co_ok;
      float d = to_f32(dr[u]);
      if constexpr (PRO) {
        const float z = to_f32(zr[u]), y = fmaf(z, osc, osh);
        d = round_to<T>(fmaf(k1, y > olo && y < ohi ? d : 0.f, fmaf(k2, z, k3)));
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(din ? d : 0.f, xin[u] ? x : 0.f, acc, 0, 0, 0);
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][4 * mg + r][l16] = acc[r];
  __syncthreads();
  asm volatile("" : "+v"(g_old));
  if (writer) {
    float v = 0.f;
#pragma unroll
    for (int q = 0; q < NW; ++q) v += red[q][orow][ocol];
    *dst = g_old + v;
  }
}

// both gradients of a layer in one launch: blocks [0, n_dgrad) hold four data-gradient tiles each
// The BatchNorm backward on the way in (PRO) doubles a wavefront's instructions, and what a block of 16 takes then is four wavefronts'
// instructions on each SIMD of a CU that has no neighbour busy: 8 wavefronts.  A step of the sensor network at batch 8 (1024 rows, two such
// layers), us: BatchNorm backward in launches of its own, 16 wavefronts 68.1, 8 71.7, 4 84.1; on the way in 67.2, 64.0, 76.0.
template <typename T, bool CV, bool PRO, int NW>
__global__ __launch_bounds__(64 * NW) void conv1d_bwd_small_k(Conv1dArgs d, Conv1dArgs g, float* g_w, int n_dgrad) {
  if ((int)blockIdx.x < n_dgrad) conv1d_tile<T, true, CV, NW, PRO>(d, blockIdx.x);
  else conv1d_wgrad_tile<T, PRO, NW>(g, g_w, blockIdx.x - n_dgrad);
}

// ---- host ---------------------------------------------------------------------------------------------------
int conv1d_ok(const ConvGeom& g) {
  // windows of 16 and more: the row counters wrap at most once a step; 32-bit row and element indexes
  return g.kh == 1 && g.Hin == 1 && g.Hout == 1 && g.ph == 0 && g.stride == 1 && g.kw >= 2 && g.kw <= kC1Taps && g.kw % 2 == 1 &&
         2 * g.pw == g.kw - 1 && g.Win >= 16 && g.Cin <= kC1Chan && g.Cout <= kC1Chan && g.Cout % 8 == 0 &&
         (size_t)g.N * g.Win * kC1Chan < ((size_t)1 << 31);
}

static bool conv1d_small(const ConvGeom& g) { return (size_t)g.N * g.Win <= kC1Small; }

// Which of these layers run here, and which through patch matrices and the pointwise kernels.  Those multiply bfloat16 on its own matrix
// instructions, sixteen times the rate of the fp32 ones here, and walk narrow tensors with fewer instructions a row; what they pay is the
// matrices: one in forward, which the weight gradient reads again if no layer behind has taken the buffer, one of dz, and launches that
// layers here share with others.  A first layer (no data gradient) needs a single matrix.  A stage that forks has no buffer for
// that of dz, and its direct data gradient is slower than all else.
// Steps, us, patch matrices / here.  fp32: 64 -> 64, 5 taps, alone, 32768 rows 100 / 65; first layers alone 9 -> 32, 5 taps, 32768 50 / 55,
// 131072 77 / 84, 8 -> 32 131072 77 / 73, 3 -> 64, 3 taps, 131072 85 / 80, 262144 107 / 114; chain 8 -> 8, 3 taps, 131072 138 / 137, 262144
// 200 / 215.  bfloat16: chain 64 -> 64, 9 taps, 2304 rows 104 / 132, 8192 122 / 116, 32768 229 / 206, 7 taps, 131072 600 / 640; 48 -> 48,
// 7 taps, 2304 91 / 105, 6144 98 / 106, 131072 485 / 549; 32 -> 64, 9 taps, 4096 99 / 102, 6144 107 / 103; chain 8 -> 8, 3 taps, 65536
// 101 / 98, 131072 112 / 129, 1048576 350 / 670; 32 -> 32, 3 taps, 131072 190 / 174, 524288 522 / 580; first layers 9 -> 32, 5 taps, alone 2304
// 36 / 38, 65536 48 / 67, in front of two more 16384 180 / 179, 65536 325 / 336; 3 -> 8, 3 taps, alone 8192 41 / 38, 16384 42 / 40,
// 32768 42 / 46, 524288 76 / 162; a layer behind others alone in its stage 64 -> 64, 9 taps 4096 70 / 70, 8192 84 / 94, 24576 108 / 129, 5 taps 32768
// 97 / 98, 65536 131 / 157, 3 taps 32768 87 / 87, 65536 107 / 131; 16 -> 16, 5 taps, in front of another 32768 99 / 93, 131072 157 / 157, 524288 390 / 437.
int conv1d_pays(int dt, const ConvGeom& g, bool first, bool alone, bool forks) {
  const size_t M = (size_t)g.N * g.Win;
  const int lo = g.Cin < g.Cout ? g.Cin : g.Cout, hi = g.Cin < g.Cout ? g.Cout : g.Cin;
  const int K = g.kw * g.Cin, both = g.kw * (g.Cin + g.Cout), weights = K * g.Cout;
  const bool odd = g.Cin % 8 != 0;                    // read value by value here
  if (conv1d_small(g)) return 1;
  if (first && dt == 0) {                             // the patch matrix of a narrow input is little to write
    if (g.Cout > 32 ? odd && K <= 54 && M >= 200000 : (odd || alone) && K <= 45 && M >= 32768) return 0;
    if (odd && g.Cin < 12 && K <= 81 && (g.Cout <= 32 || K >= 45) && M >= 131072) return 0;
  }
  if (first && dt == 1) {
    if (K >= 280 && g.Cout <= 32 && M >= 8192) return 1;
    if (alone && M < 8192) return odd ? K <= 40 : K <= 240 && weights <= 5000;
    if (alone) return K <= 30 && M < 24576;
    if (M >= (weights >= 10000 ? 8192u : odd ? 32768u : 98304u)) return 0;
  }
  if (forks) return 1;
  if (dt == 0) return !(hi <= 8 && g.kw == 3 && M >= 200000);
  if (M < 8192) return M > (size_t)128 * lo || weights < 10000;      // few tiles, each a long chain of fp32 products
  if (lo >= 40) return M < (g.kw >= 7 ? (alone ? 8192u : 49152u) : alone ? 40000u : 98304u);           // bound by the fp32 products
  return !(hi <= 2 * lo && both <= 192 && M >= (size_t)1700 * both);   // narrow: columns filled up to 32
}

static Conv1dArgs conv1d_args(const ConvGeom& g, bool dgrad) {
  Conv1dArgs a{};
  a.M = g.N * g.Win; a.W = g.Win; a.Cin = g.Cin; a.Cout = g.Cout; a.kw = g.kw;
  a.pad = dgrad ? g.kw - 1 - g.pw : g.pw;
  a.C = dgrad ? g.Cout : g.Cin;
  a.NC = dgrad ? g.Cin : g.Cout;
  a.CP = (a.C + 7) / 8 * 8;
  a.dC = FastDiv::of(a.C); a.dW = FastDiv::of(a.W);
  return a;
}

static void conv1d_plan_tiles(Conv1dArgs* a) {
  a->itiles = (a->M + 15) / 16; a->jtiles = (a->NC + 15) / 16; a->tiles_per_range = 1;
}

// tile shape by the columns (a 64-wide tile over 32 columns or fewer would be half padding); at most kBnPartials row
// ranges, since each leaves one partial
template <typename T, bool DGRAD>
static void conv1d_rows(hipStream_t st, Conv1dArgs& a, int* P_out) {
  const int WC = a.NC <= 32 ? 1 : 2, TI = 64;
  a.itiles = (a.M + TI - 1) / TI;
  a.jtiles = (a.NC + 32 * WC - 1) / (32 * WC);
  a.tiles_per_range = (a.itiles + kBnPartials - 1) / kBnPartials;
  const int nr = (a.itiles + a.tiles_per_range - 1) / a.tiles_per_range;
  const int LDR = (a.CP / 4) % 2 ? a.CP : a.CP + 4;
  const size_t lds = ((size_t)(TI + a.kw) * LDR + (size_t)2 * 32 * WC * (128 / WC + 4)) * sizeof(float);
  if (lds > 65536 - 1024) { launch_plan_failed("conv1d: tile does not fit LDS"); return; }
  if (P_out) *P_out = nr;
  if (WC == 1) hipLaunchKernelGGL((conv1d_rows_k<T, DGRAD, 1>), dim3(nr * a.jtiles), dim3(256), lds, st, a);
  else hipLaunchKernelGGL((conv1d_rows_k<T, DGRAD, 2>), dim3(nr * a.jtiles), dim3(256), lds, st, a);
}

int conv1d_small_ok(const ConvGeom& g) { return conv1d_ok(g) && conv1d_small(g); }

void conv1d_fwd(int dt, hipStream_t st, HView in, const BnPending& pend, float eps, float momentum, const void* w, const ConvGeom& g, void* z,
                float* stats, int* P_out) {
  Conv1dArgs a = conv1d_args(g, false);
  a.pend = pend; a.eps = eps; a.momentum = momentum;
  a.x = in.z; a.w = w; a.view = View{in.z, in.scale, in.shift, in.act}; a.out = z; a.stats = stats;
  KScope ks(st, "conv1d_fwd", ((double)a.M * (g.Cin + g.Cout) + (double)g.Cout * g.kw * g.Cin) * (dt == 0 ? 4.0 : 2.0),
            2.0 * a.M * g.Cout * g.kw * g.Cin, a.M, g.kw * g.Cin, g.Cout);
  if (conv1d_small(g)) {
    conv1d_plan_tiles(&a);
    *P_out = a.itiles;
    const dim3 grid(a.itiles * a.jtiles);
    if (g.Cin % 4 == 0) FTP_DISPATCH(dt, hipLaunchKernelGGL((conv1d_fwd_small_k<T, true>), grid, dim3(256), 0, st, a));
    else FTP_DISPATCH(dt, hipLaunchKernelGGL((conv1d_fwd_small_k<T, false>), grid, dim3(256), 0, st, a));
    return;
  }
  FTP_DISPATCH(dt, (conv1d_rows<T, false>(st, a, P_out)));
}

void conv1d_dgrad(int dt, hipStream_t st, const void* dz, const void* w, const ConvGeom& g, void* dIn, HView prev, float* sums, int* P_out) {
  Conv1dArgs a = conv1d_args(g, true);
  a.x = dz; a.w = w; a.out = dIn; a.stats = sums; a.prev = View{prev.z, prev.scale, prev.shift, prev.act};
  KScope ks(st, "conv1d_dgrad", ((double)a.M * (g.Cin + g.Cout) + (double)g.Cout * g.kw * g.Cin) * (dt == 0 ? 4.0 : 2.0),
            2.0 * a.M * g.Cout * g.kw * g.Cin, a.M, g.kw * g.Cout, g.Cin);
  FTP_DISPATCH(dt, (conv1d_rows<T, true>(st, a, P_out)));
}

static Conv1dWgArgs conv1d_wgrad_plan(const ConvGeom& g, int* P) {
  Conv1dWgArgs a{};
  a.c = conv1d_args(g, false);
  a.nco = (g.Cout + 16 * kC1RT - 1) / (16 * kC1RT);
  a.nkg = (g.kw * g.Cin + 16 * kC1CT - 1) / (16 * kC1CT);
  const int pieces = a.nco * a.nkg;
  a.gpb = pieces >= 4 ? 4 : pieces >= 2 ? 2 : 1;
  a.rs = 4 / a.gpb;
  a.ngrp = (pieces + a.gpb - 1) / a.gpb;
  a.c.itiles = (a.c.M + kC1WgRows - 1) / kC1WgRows;
  // two blocks per CU; every row share leaves a partial of the whole gradient.  One block per CU halves the partials, but
  // its single wavefront per SIMD waits for every LDS read (64 -> 64 channels, 32768 rows: 37 us against 28)
  const int want = 512 / a.ngrp > 0 ? 512 / a.ngrp : 1;
  a.c.tiles_per_range = (a.c.itiles + want - 1) / want;
  *P = (a.c.itiles + a.c.tiles_per_range - 1) / a.c.tiles_per_range * a.rs;
  return a;
}

size_t conv1d_wgrad_ws(const ConvGeom& g) {
  if (conv1d_small(g)) return 0;
  int P;
  conv1d_wgrad_plan(g, &P);
  return (size_t)P * g.Cout * g.kw * g.Cin;
}

void conv1d_wgrad(int dt, hipStream_t st, const void* dz, HView in, const ConvGeom& g, float* ws, float* g_w,
                  std::vector<ReduceJob>* left) {
  int P;
  Conv1dWgArgs a = conv1d_wgrad_plan(g, &P);
  const int K = g.kw * g.Cin;
  a.c.x = in.z; a.c.w = dz; a.c.view = View{in.z, in.scale, in.shift, in.act};
  if (conv1d_small(g)) {
    conv1d_bwd_small(dt, st, dz, nullptr, in, g, g_w, nullptr);
    return;
  }
  {
    KScope ks(st, "conv1d_wgrad", (double)a.c.M * (g.Cin + g.Cout) * (dt == 0 ? 4.0 : 2.0) + (double)P * g.Cout * K * 4, 2.0 * a.c.M * g.Cout * K,
              a.c.M, K, g.Cout);
    a.c.out = ws;
    const int LDR = (g.Cin + 31) / 32 * 32 + 16, LDZ = (g.Cout + 31) / 32 * 32 + 16;
    const size_t lds = ((size_t)(kC1WgRows + g.kw - 1) * LDR + (size_t)kC1WgRows * LDZ) * sizeof(float);
    FTP_DISPATCH(dt, hipLaunchKernelGGL(conv1d_wgrad_k<T>, dim3(P / a.rs * a.ngrp), dim3(256), lds, st, a));
  }
  left->push_back(ReduceJob{ws, g_w, P, g.Cout * K, K, K, 1, K});
}

void conv1d_bwd_small(int dt, hipStream_t st, const void* dz, const void* w, HView in, const ConvGeom& g, float* g_w, void* dIn,
                      const BnPending* sums, const BnBwdIn* own, float* left, int* P_out) {
  Conv1dArgs d = conv1d_args(g, true), a = conv1d_args(g, false);
  d.x = dz; d.w = w; d.out = dIn;
  conv1d_plan_tiles(&d);
  a.x = in.z; a.w = dz; a.view = View{in.z, in.scale, in.shift, in.act};
  if (sums) {
    d.x = a.w = own->dA;
    d.pend = a.pend = *sums;
    d.own = a.own = View{own->out.z, own->out.scale, own->out.shift, own->out.act};
    d.g_gamma = a.g_gamma = own->g_gamma; d.g_beta = a.g_beta = own->g_beta;
  }
  if (left) {
    d.stats = left; d.prev = View{in.z, in.scale, in.shift, in.act};
    *P_out = d.itiles;
  }
  const int groups = sums ? 2 : 4;     // tiles of the data gradient to a block
  const int K = g.kw * g.Cin, nd = dIn ? (d.itiles * d.jtiles + groups - 1) / groups : 0, nw = (K + 15) / 16 * ((g.Cout + 15) / 16);
  a.own_writes = nd == 0;              // who adds to the BatchNorm's gradients: the first data-gradient block, where there is one
  KScope ks(st, dIn ? "conv1d_bwd" : "conv1d_wgrad", (double)d.M * (2.0 * g.Cin + g.Cout) * (dt == 0 ? 4.0 : 2.0) + (double)g.Cout * K * 8, 4.0 * d.M * g.Cout * K,
            d.M, K, g.Cout);
  if (sums) FTP_DISPATCH(dt, hipLaunchKernelGGL((conv1d_bwd_small_k<T, true, true, 8>), dim3(nd + nw), dim3(512), 0, st, d, a, g_w, nd));
  else FTP_DISPATCH(dt, hipLaunchKernelGGL((conv1d_bwd_small_k<T, true, false, 16>), dim3(nd + nw), dim3(1024), 0, st, d, a, g_w, nd));
}

}  // namespace ftp
