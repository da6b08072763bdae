// Convolutions along one axis (1 x kw, stride 1, same length out as in), at most 64 channels on either side, as
// implicit GEMMs: row m of the patch matrix is kw neighbouring rows of the input, so the matrix is never written.  A tile
// of rows with its halo goes into LDS once (through the producer's BatchNorm + activation) and every tap reads it
// there at a row offset; rows are the flattened (window, position) index, so a tile may span windows of any length, and a tap
// that leaves its own window reads zero.  All products run on the fp32 MFMA (products of bfloat16 values are exact in it).
// What bounds them is that unit, 256 FLOP a cycle and CU (157 TFLOP/s): 64 -> 64 channels, 5 taps, 32768 rows is 8.5 us a pass.  It does not run
// beside the vector ALU: in a loop of 16x16x4 instructions with 45 vector instructions to ten of them a step took the sum of both, also with a
// second wavefront on the SIMD.  So nothing is computed in the loops over the reduction that can be computed in front of them.
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
  int kphase;         // row tiles: reduction elements whose weights lie in LDS together
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

enum { kC1Chan = 64, kC1Taps = 9, kC1Small = 2048, kC1Blocks = 256 };

// four values as they lie in memory: converted only when they go into LDS, so that a tile on its way is not waited for
template <typename T> struct Raw4;
template <> struct Raw4<float> {
  float4 v;
  __device__ __forceinline__ void load(const float* p) { v = ld4(p); }
  __device__ __forceinline__ void set(int e, float x) { (&v.x)[e] = x; }
  __device__ __forceinline__ float4 get() const { return v; }
};
template <> struct Raw4<bf16_t> {
  uint2 v;
  __device__ __forceinline__ void load(const bf16_t* p) { v = *reinterpret_cast<const uint2*>(p); }
  __device__ __forceinline__ void set(int e, bf16_t x) {
    unsigned& w = e < 2 ? v.x : v.y;
    w = e & 1 ? (w & 0xffffu) | ((unsigned)x << 16) : (w & 0xffff0000u) | x;
  }
  __device__ __forceinline__ float4 get() const {
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u));
  }
};

// NV vectors of four channels per thread of a tile of `rows` rows of a tensor [M][C], padded to CP channels (a multiple of 4): from
// row m0 on requested by fetch, through the view and zeros outside the tensor into LDS rows of ld floats by commit.
template <typename T, int NV>
struct RowVecs {
  Raw4<T> raw[NV];
  int row[NV], chan[NV], lds[NV];        // a row far outside the tensor: padding channels
  __device__ __forceinline__ void init(const int C, const int CP, const int ld, const int rows, const int spare) {   // spare: four floats that nobody reads
    const int CG = CP / 4, nv = rows * CG;
    const unsigned magic = 65536u / (unsigned)CG + 1u;       // v / CG: exact, v * CG < 65536
#pragma unroll
    for (int s = 0; s < NV; ++s) {
      const int v = threadIdx.x + 512 * s, r = (int)(((unsigned)v * magic) >> 16), c = (v - r * CG) * 4;
      row[s] = v < nv && c < C ? r : -(1 << 28);
      chan[s] = v < nv && c < C ? c : 0;
      lds[s] = v < nv ? r * ld + c : spare;
    }
  }
  __device__ __forceinline__ void fetch(const T* __restrict__ X, const int C, const int M, const int m0) {
    if (C % 4 == 0) {
#pragma unroll
      for (int s = 0; s < NV; ++s) {
        const int m = m0 + row[s];
        raw[s].load(X + ((unsigned)m < (unsigned)M ? m * C + chan[s] : 0));
      }
      return;
    }
    T x[NV][4];
#pragma unroll
    for (int s = 0; s < NV; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int m = m0 + row[s];
        x[s][e] = X[(unsigned)m < (unsigned)M && chan[s] + e < C ? m * C + chan[s] + e : 0];
      }
#pragma unroll
    for (int s = 0; s < NV; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) raw[s].set(e, x[s][e]);
  }
  __device__ __forceinline__ void commit(float* dst, const int C, const int M, const int m0, const bool view, const float* sc, const float* sh,
                                         const float lo, const float hi) const {
    if (view) put<true>(dst, C, M, m0, sc, sh, lo, hi);
    else put<false>(dst, C, M, m0, sc, sh, lo, hi);
  }
  // no branch between the vectors: their LDS reads go out together
  template <bool VIEW>
  __device__ __forceinline__ void put(float* dst, const int C, const int M, const int m0, const float* sc, const float* sh, const float lo, const float hi) const {
    float4 a[VIEW ? NV : 1], b[VIEW ? NV : 1];
    if (VIEW)
#pragma unroll
      for (int s = 0; s < NV; ++s) { a[VIEW ? s : 0] = ld4(sc + chan[s]); b[VIEW ? s : 0] = ld4(sh + chan[s]); }
#pragma unroll
    for (int s = 0; s < NV; ++s) {
      const bool in = (unsigned)(m0 + row[s]) < (unsigned)M;
      float4 x = raw[s].get();
      float* f = &x.x;
      if (VIEW)
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = round_to<T>(clamp_act(fmaf(f[e], (&a[VIEW ? s : 0].x)[e], (&b[VIEW ? s : 0].x)[e]), lo, hi));
#pragma unroll
      for (int e = 0; e < 4; ++e) f[e] = in && chan[s] + e < C ? f[e] : 0.f;
      *reinterpret_cast<float4*>(dst + lds[s]) = x;
    }
  }
};

// ---- row tiles: forward and data gradient ---------------------------------------------------------------------
// 8 wavefronts of 32 x 32 results: WC groups of 32 columns, 8 / (WC * KSP) of 32 rows, and KSP wavefronts that split the reduction of
// each and meet in LDS, where each then finishes its share of the rows.  One block per CU: the weights pass into LDS once for all
// its tiles (in two phases a tile where they do not fit), the next tile's rows are on their way while one is multiplied, and
// the reduction runs without a barrier, at 97 % of the matrix unit's rate.  Kernel times at 5 taps, 32768 rows, before (weights in
// double-buffered chunks of 64 with a barrier each, two blocks of 4 wavefronts per CU) and now, us: 64 -> 64 forward 22.1 / 19.0, data
// gradient 26.2 / 21.5; 32 -> 64 16.7 / 13.5 and 19.2 / 14.2.  What is left over the 8.5 is the launch, the first tile's way into LDS (4) and the
// results' way out (2).  A step of the sensor network, us: 2400 rows 146 / 104, 8192 158 / 120, 32768 238 / 218, 131072 638 / 544;
// bfloat16 8192 158 / 114, 131072 566 / 527 (the weight gradient below and the sums the layers leave each other included).
enum { kC1Lds = 160 * 1024 - 4096 };
template <typename T, bool DGRAD, int WC, int KSP>
__global__ __launch_bounds__(512) void conv1d_rows_k(Conv1dArgs p) {
  constexpr int RG = 8 / (WC * KSP), TI = 32 * RG, BC = 32 * WC, SHARE = 16 / KSP, NV = ((TI + kC1Taps - 1) * (kC1Chan / 4) + 511) / 512;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  const int LDR = p.CP + 4;                               // CP is a multiple of 8: an odd number of 16-byte units, rows fall into different banks
  const int prow = TI + p.kw - 1, xbuf = (prow + 1) * LDR; // row prow is the zero row; four floats behind each buffer that nobody reads
  const int WLD = p.kphase + 4;                           // an odd number of 16-byte units too
  float* ex = smem;                                       // [8][16][64] where the reduction is split
  float* xs = smem + (KSP > 1 ? 8 * 16 * 64 : 0);         // [2][xbuf], one of them where there is a single tile
  float* wsm = xs + (p.tiles_per_range > 1 ? 2 : 1) * (xbuf + 4);   // [BC][WLD]
  __shared__ float red[2][BC][RG * KSP];
  __shared__ __attribute__((aligned(16))) float vsc[2][kC1Chan];
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, h = lane >> 5, l32 = lane & 31;
  const int ks = wave % KSP, wc = wave / KSP % WC, wr = wave / (KSP * WC);
  const int range = xcd_logical_block();
  const int KP = p.kw * p.CP;
  const T* X = reinterpret_cast<const T*>(p.x);
  const T* Wt = reinterpret_cast<const T*>(p.w);
  const bool view = !DGRAD && p.view.scale != nullptr;
  const float lo = act_lo(p.view.act), hi = act_hi(p.view.act);
  const int it_beg = range * p.tiles_per_range, it_end = min(it_beg + p.tiles_per_range, p.itiles);
  const unsigned cp_magic = 65536u / (unsigned)p.CP + 1u;     // k / CP, exact for k * CP < 65536: k <= 9 * 64, CP <= 64

  // weights of reduction elements [k0, k0 + n) into LDS, a column's elements contiguous
  auto load_w = [&](const int k0, const int n) {
    if (!DGRAD && p.C % 8 == 0) {                            // CP == C: k is the offset in a weight row
      constexpr int TC = 512 / BC, U = 10;                   // threads to a column; 64 columns, 320 elements: one round
      const int col = tid / TC, at = (tid % TC) * 4;
      const T* src = Wt + (col < p.NC ? col * KP : 0) + k0;
      for (int q0 = at; q0 < n; q0 += U * 4 * TC) {
        Raw4<T> x[U];
#pragma unroll
        for (int s = 0; s < U; ++s) x[s].load(src + (q0 + 4 * TC * s < n ? q0 + 4 * TC * s : at));
#pragma unroll
        for (int s = 0; s < U; ++s) {
          float4 f = x[s].get();
          if (col >= p.NC) f = make_float4(0.f, 0.f, 0.f, 0.f);
          if (q0 + 4 * TC * s < n) *reinterpret_cast<float4*>(wsm + col * WLD + q0 + 4 * TC * s) = f;
        }
      }
    } else if (DGRAD && p.NC % 4 == 0) {                     // CP == C here too: k / C is the tap, k % C the channel of dZ
      // a wavefront takes 16 columns of 16 elements: 64-byte pieces of memory, and all its LDS words in different banks
      constexpr int CGN = BC / 4, TK = 512 / CGN, U = 5;     // groups of four columns; elements to a round
      const int col = (tid / 16 % CGN) * 4, at = tid / (16 * CGN) * 16 + tid % 16;
      const bool col_in = col < p.NC;
      for (int q0 = at; q0 < n; q0 += U * TK) {
        Raw4<T> x[U];
#pragma unroll
        for (int s = 0; s < U; ++s) {
          const int kl = q0 + TK * s, k = k0 + (kl < n ? kl : at);
          const int tap = (int)(((unsigned)k * cp_magic) >> 16), c = k - tap * p.CP;
          x[s].load(Wt + (c * p.kw + (p.kw - 1 - tap)) * p.Cin + (col_in ? col : 0));
        }
#pragma unroll
        for (int s = 0; s < U; ++s) {
          const int kl = q0 + TK * s;
          const float4 f = x[s].get();
          if (kl < n)
#pragma unroll
            for (int e = 0; e < 4; ++e) wsm[(col + e) * WLD + kl] = col_in ? (&f.x)[e] : 0.f;
        }
      }
    } else {
      constexpr int U = 5;
      for (int e0 = tid; e0 < BC * n; e0 += U * 512) {
        T x[U];
#pragma unroll
        for (int s = 0; s < U; ++s) {
          const int e = e0 + 512 * s, col = DGRAD ? e % BC : e / n, k = k0 + (DGRAD ? e / BC : e - col * n);
          const int tap = (int)(((unsigned)k * cp_magic) >> 16), c = k - tap * p.CP;
          const bool in = e < BC * n && col < p.NC && c < p.C;
          x[s] = Wt[in ? (DGRAD ? (c * p.kw + (p.kw - 1 - tap)) * p.Cin + col : (col * p.kw + tap) * p.Cin + c) : 0];
        }
#pragma unroll
        for (int s = 0; s < U; ++s) {
          const int e = e0 + 512 * s, col = DGRAD ? e % BC : e / n, kl = DGRAD ? e / BC : e - col * n, k = k0 + kl;
          if (e >= BC * n) break;
          const int c = k - (int)(((unsigned)k * cp_magic) >> 16) * p.CP;
          wsm[col * WLD + kl] = col < p.NC && c < p.C ? to_f32(x[s]) : 0.f;
        }
      }
    }
  };

  RowVecs<T, NV> tile;
  tile.init(p.C, p.CP, LDR, prow, xbuf);
  tile.fetch(X, p.C, p.M, it_beg * TI - p.pad);
  // The BatchNorm of x still partial sums: every block adds them, on their way with its first rows, where a tile or the meeting of the wavefronts
  // will lie (256 bytes a channel; a tile is more).  A finalize launch took 4.1 us of the chain.
  const bool pending = !DGRAD && p.pend.partial != nullptr;
  if (pending) finish_slab(p.pend, p.C, 0, p.C, p.eps, p.momentum, range == 0, reinterpret_cast<double*>(smem), vsc[0], vsc[1]);
  if (view && !pending && tid < p.C) { vsc[0][tid] = p.view.scale[tid]; vsc[1][tid] = p.view.shift[tid]; }
  load_w(0, p.kphase);
  for (int c = tid; c < LDR; c += 512) {
    xs[prow * LDR + c] = 0.f;
    if (p.tiles_per_range > 1) xs[xbuf + 4 + prow * LDR + c] = 0.f;
  }
  float s1 = 0.f, s2 = 0.f;
  const int col = wc * 32 + l32;
  const bool col_ok = col < p.NC;
  float psc = 0.f, psh = 0.f;
  const bool sums = DGRAD && p.stats != nullptr;
  if (sums && col_ok) { psc = p.prev.scale[col]; psh = p.prev.shift[col]; }
  const float plo = act_lo(p.prev.act), phi = act_hi(p.prev.act);
  if (view) __syncthreads();
  tile.commit(xs, p.C, p.M, it_beg * TI - p.pad, view, vsc[0], vsc[1], lo, hi);
  if (it_beg + 1 < it_end) tile.fetch(X, p.C, p.M, (it_beg + 1) * TI - p.pad);
  __syncthreads();
  for (int it = it_beg; it < it_end; ++it) {
    const int m0 = it * TI, buf = (it - it_beg) & 1;
    const bool more = it + 1 < it_end;
    // the next tile goes into LDS, and the one behind it is requested; wavefronts 4 - 7 do that before their products, the others, which share
    // their SIMDs, behind them: the matrix unit is busy meanwhile
    auto advance = [&]() __attribute__((always_inline)) {
      if (!more) return;
      tile.commit(xs + (buf ^ 1) * (xbuf + 4), p.C, p.M, m0 + TI - p.pad, view, vsc[0], vsc[1], lo, hi);
      if (it + 2 < it_end) tile.fetch(X, p.C, p.M, m0 + 2 * TI - p.pad);
    };
    if (wave >= 4) advance();
    // registers of this wavefront's results that it finishes: ks * SHARE ..; register r is row 8 * (r / 4) + 4 * h + r % 4, column l32
    T zp[SHARE];
    if (sums) {
      const T* Z = reinterpret_cast<const T*>(p.prev.z);
#pragma unroll
      for (int i = 0; i < SHARE; ++i) {
        const int r = ks * SHARE + i, m = m0 + wr * 32 + 4 * h + 8 * (r >> 2) + (r & 3);
        zp[i] = Z[col_ok && m < p.M ? m * p.NC + col : 0];
      }
    }
    const int mrow = m0 + wr * 32 + l32;
    const int t = mrow < p.M ? (int)((unsigned)mrow % (unsigned)p.W) : -(1 << 20);   // a row past the end is outside every window
    const float* xt = xs + buf * (xbuf + 4);
    auto tap_row = [&](int tp) { return xt + ((unsigned)(t + tp - p.pad) < (unsigned)p.W ? wr * 32 + l32 + tp : prow) * LDR + 4 * h; };
    // Chains of at most 64 fp32 additions, not one through the whole reduction: 64 -> 64 channels, 9 taps were 4.3e-7 off the exact result
    // (2-norm) in one chain, 1.6e-7 in chains of 64.  32 columns and fewer: of 32, 32 -> 32 channels, 5 taps, 1.45e-7 (in chains of 80 1.67e-7).
    // The additions are a sixteenth and an eighth of the matrix instructions' time, which start a chain from a constant zero.
    constexpr int CHAIN = WC == 1 ? 4 : 8;              // steps of eight elements
    f16v acc, tot;
#pragma unroll
    for (int e = 0; e < 16; ++e) tot[e] = 0.f;
    for (int k0 = 0; k0 < KP; k0 += p.kphase) {
      const int n = min(p.kphase, KP - k0);
      if (p.kphase < KP && (k0 > 0 || it > it_beg)) {
        __syncthreads();                                // the phase before has been read
        load_w(k0, n);
        __syncthreads();
      }
      const int nq = n / 8, qe = (ks + 1) * nq / KSP;   // KP and the phase are multiples of 8
      int q = ks * nq / KSP;
      if (q == qe) continue;
      int tap = (int)(((unsigned)(k0 + 8 * q) * cp_magic) >> 16), c0 = k0 + 8 * q - tap * p.CP;
      const float* arow = tap_row(tap);
      const float* brow = wsm + (wc * 32 + l32) * WLD + 4 * h + 8 * q;
      float4 a0 = ld4(arow + c0), b0 = ld4(brow), a1, b1;
      auto next = [&](float4& a, float4& b) __attribute__((always_inline)) {
        c0 += 8;
        brow += 8;
        if (c0 == p.CP) { c0 = 0; ++tap; arow = tap_row(tap); }       // behind the last tap: at most the zero row, not used
        a = ld4(arow + c0);
        b = ld4(brow);                                  // behind the last element: padding or the next column, not used
        __builtin_amdgcn_sched_barrier(0);              // requested before the products in front of them run, not behind
      };
      auto products = [&](const float4& a, const float4& b, const bool first) __attribute__((always_inline)) {
        const f16v none = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, first ? none : acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      };
      for (; q + CHAIN <= qe; q += CHAIN) {
#pragma unroll
        for (int i = 0; i < CHAIN; i += 2) {
          next(a1, b1);
          products(a0, b0, i == 0);
          next(a0, b0);
          products(a1, b1, false);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) tot[e] += acc[e];
      }
      if (q < qe) {                                     // a shorter one
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = 0.f;
        for (; q + 2 <= qe; q += 2) {
          next(a1, b1);
          products(a0, b0, false);
          next(a0, b0);
          products(a1, b1, false);
        }
        if (q < qe) {
          next(a1, b1);
          products(a0, b0, false);
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) tot[e] += acc[e];
      }
    }
    if (wave < 4) advance();
    if constexpr (KSP > 1) {
      if (it > it_beg) __syncthreads();                 // the shares of the tile before have been read
#pragma unroll
      for (int r = 0; r < 16; ++r) ex[(wave * 16 + r) * 64 + lane] = tot[r];
    }
    if (KSP > 1 || more) __syncthreads();
    T* out = reinterpret_cast<T*>(p.out);
    auto finish = [&](const bool whole) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < SHARE; ++i) {
        const int r = ks * SHARE + i, m = m0 + wr * 32 + 4 * h + 8 * (r >> 2) + (r & 3);
        float x = KSP > 1 ? 0.f : tot[r];
        if constexpr (KSP > 1)
#pragma unroll
          for (int k2 = 0; k2 < KSP; ++k2) x += ex[((wave - ks + k2) * 16 + r) * 64 + lane];
        const bool ok = whole || (col_ok && m < p.M);
        if (ok) out[m * p.NC + col] = from_f32<T>(x);
        const float v = round_to<T>(x);                   // sums are those of the values as stored
        if (sums) {
          // chosen, not multiplied: a gradient that is not finite stays out of the sums of a channel that is off
          const float z = to_f32(zp[i]), yp = fmaf(z, psc, psh);
          const float dy = ok && (p.prev.act == ACT_NONE || (yp > plo && yp < phi)) ? v : 0.f;
          s1 += dy;
          s2 += ok ? dy * z : 0.f;
        } else {
          s1 += ok ? v : 0.f;
          s2 += ok ? v * v : 0.f;
        }
      }
    };
    if (m0 + TI <= p.M && p.NC == BC) finish(true);     // nothing to ask for each value
    else finish(false);
  }
  if (p.stats) {
    s1 += __shfl_xor(s1, 32, 64);
    s2 += __shfl_xor(s2, 32, 64);
    if (h == 0) { red[0][col][wr * KSP + ks] = s1; red[1][col][wr * KSP + ks] = s2; }
    __syncthreads();
    if (tid < 2 * BC) {
      const int sq = tid / BC, c = tid % BC;
      float v = 0.f;
#pragma unroll
      for (int q = 0; q < RG * KSP; ++q) v += red[sq][c][q];
      if (c < p.NC) p.stats[((size_t)range * 2 + sq) * p.NC + c] = v;
    }
  }
}

// ---- weight gradient over row tiles ---------------------------------------------------------------------------
// A block takes a range of row tiles (dZ and the input with its halo in LDS, the next tile on its way in registers) and a set of 32 x
// 80 pieces of g_w [Cout][kw * Cin]: a wavefront keeps 2 x 5 tiles of 16 x 16 in accumulators over all its rows and reads seven LDS
// words for ten MFMAs.  Wavefronts that share a piece's rows meet in LDS: one partial per block.  Half the pieces to a block
// where there are several: what it then loads twice is less than the partials of twice as many row ranges.  64 -> 64 channels, 32768
// rows: 25.9 us and 128 partials, added up in 5.0; four wavefronts, nothing on its way, two blocks per CU and 256
// partials 29 and 11.6.
// Partials meet in float64, and so do the wavefronts of a piece; a wavefront adds every other step of its rows to a second set of accumulators.
// Where it was one chain and the wavefronts met in fp32, 32768 rows of 16 -> 16, 3 taps, were 1.13e-7 off 64 bits (2-norm), of 64 -> 64, 5 taps, 2.10e-7;
// with each wavefront's chain a partial 0.95e-7 and 2.08e-7; so 0.89e-7 and 1.55e-7, at the same time.
struct Conv1dWgArgs {
  Conv1dArgs c;
  int nco, nkg;            // pieces along Cout (32 each) and along kw * Cin (80 each)
  int rs;                  // wavefronts that share a piece's rows: 8 / rs pieces per block
  int ngrp;                // blocks per row range
  int rows;                // rows of a tile: 64 or 32
};
// kC1WgLd: 16 banks between rows, so that the four rows of an MFMA operand fall into different banks; the same for every channel count, so that
// a step's rows are at an offset known to the compiler
enum { kC1RT = 2, kC1CT = 5, kC1Acc = kC1RT * kC1CT * 4, kC1WgLd = kC1Chan + 16 };

template <typename T, int RS, int ROWS>
__global__ __launch_bounds__(512) void conv1d_wgrad_k(Conv1dWgArgs a) {
  const Conv1dArgs& p = a.c;
  constexpr int NX = ((64 + kC1Taps - 1) * (kC1Chan / 4) + 511) / 512, ND = 64 * (kC1Chan / 4) / 512;
  extern __shared__ __attribute__((aligned(16))) float smem[];
  __shared__ __attribute__((aligned(16))) float vsc[2][kC1Chan];
  constexpr int LD = kC1WgLd, STEPS = ROWS / (4 * RS);
  const int prow = ROWS + p.kw - 1, xbuf = prow * LD, buf_n = xbuf + ROWS * LD + 4, CX = (p.Cin + 3) / 4 * 4;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, rg = lane >> 4;
  const int lb = xcd_logical_block(), grp = lb % a.ngrp, range = lb / a.ngrp;      // the blocks of a range read the same rows
  constexpr int GPB = 8 / RS;            // pieces per block
  const int slot = wave % GPB, piece = grp * GPB + slot, rsub = wave / GPB;
  const bool live = piece < a.nco * a.nkg;
  const int pco = piece / a.nkg, pkg = piece % a.nkg;
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
    off[q] = k < K ? (4 * rsub + rg + tap) * LD + (k - tap * p.Cin) : 0;
    tj[q] = k < K ? tap - p.pad : 0;                    // a column past the end is not written
  }
#pragma unroll
  for (int q = 0; q < kC1RT; ++q) {
    const int co = (pco * kC1RT + q) * 16 + l16;
    doff[q] = xbuf + (4 * rsub + rg) * LD + (live && co < p.Cout ? co : 0);    // a row past the end is not written either
  }
  constexpr int SETS = STEPS > 1 ? 2 : 1;
  f4v acc[SETS][kC1RT][kC1CT];
#pragma unroll
  for (int h = 0; h < SETS; ++h)
#pragma unroll
    for (int i = 0; i < kC1RT; ++i)
#pragma unroll
      for (int q = 0; q < kC1CT; ++q) acc[h][i][q] = f4v{0.f, 0.f, 0.f, 0.f};

  const int it_beg = range * p.tiles_per_range, it_end = min(it_beg + p.tiles_per_range, p.itiles);
  RowVecs<T, NX> xt;
  RowVecs<T, ND> dt;
  xt.init(p.Cin, CX, LD, prow, buf_n - 4);
  dt.init(p.Cout, p.Cout, LD, ROWS, ROWS * LD);         // the same four floats, at the end of a buffer
  auto fetch = [&](const int it) {
    xt.fetch(X, p.Cin, p.M, it * ROWS - p.pad);
    dt.fetch(D, p.Cout, p.M, it * ROWS);
  };
  auto commit = [&](const int it, float* dst) {
    xt.commit(dst, p.Cin, p.M, it * ROWS - p.pad, view, vsc[0], vsc[1], lo, hi);
    dt.commit(dst + xbuf, p.Cout, p.M, it * ROWS, false, nullptr, nullptr, 0.f, 0.f);
  };
  fetch(it_beg);
  if (view) {
    if (tid < p.Cin) { vsc[0][tid] = p.view.scale[tid]; vsc[1][tid] = p.view.shift[tid]; }
    __syncthreads();
  }
  commit(it_beg, smem);
  if (it_beg + 1 < it_end) fetch(it_beg + 1);
  __syncthreads();
  for (int it = it_beg; it < it_end; ++it) {
    const int m0 = it * ROWS, buf = (it - it_beg) & 1;
    const bool more = it + 1 < it_end;
    // as in conv1d_rows_k: half of the wavefronts bring in the next tile before their products, half behind them
    auto advance = [&]() __attribute__((always_inline)) {
      if (!more) return;
      commit(it + 1, smem + (buf ^ 1) * buf_n);         // read last in the tile before, a barrier ago
      if (it + 2 < it_end) fetch(it + 2);
    };
    if (wave >= 4) advance();
    const float* xs = smem + buf * buf_n;
    if (live) {
      // Row 4 * rsub + rg and every 4 * RS-th behind it; the LDS words of the next four rows are on their way while ten products run.
      // t: position in its window of the step's first row.  Only where a tap leaves a window, or the rows end, is anything masked.
      int t = (int)((unsigned)(m0 + 4 * rsub) % (unsigned)p.W), m = m0 + 4 * rsub;
      const float *px[kC1CT], *pd[kC1RT];
#pragma unroll
      for (int q = 0; q < kC1CT; ++q) px[q] = xs + off[q];
#pragma unroll
      for (int q = 0; q < kC1RT; ++q) pd[q] = xs + doff[q];
      float d[2][kC1RT], x[2][kC1CT];
      auto read = [&](const int s) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < kC1RT; ++q) d[s & 1][q] = pd[q][s * 4 * RS * LD];
#pragma unroll
        for (int q = 0; q < kC1CT; ++q) x[s & 1][q] = px[q][s * 4 * RS * LD];
        __builtin_amdgcn_sched_barrier(0);
      };
      read(0);
#pragma unroll
      for (int s = 0; s < STEPS; ++s) {
        if (s + 1 < STEPS) read(s + 1);
        if (t < p.pad || t + 3 + p.pad >= p.W || m + 3 >= p.M) {
          int tl = t + rg;
          tl = m + rg < p.M ? tl - (tl >= p.W ? p.W : 0) : -(1 << 20);
#pragma unroll
          for (int q = 0; q < kC1CT; ++q) x[s & 1][q] = (unsigned)(tl + tj[q]) < (unsigned)p.W ? x[s & 1][q] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < kC1CT; ++q)
#pragma unroll
          for (int i = 0; i < kC1RT; ++i)
            acc[s % SETS][i][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[s & 1][i], x[s & 1][q], acc[s % SETS][i][q], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        m += 4 * RS;
        t += 4 * RS;                                    // at most 32, and a window has at least 16 rows
        t -= t >= p.W ? p.W : 0;
        if (RS == 8) t -= t >= p.W ? p.W : 0;
      }
    }
    if (wave < 4) advance();
    __syncthreads();
  }
  // The wavefronts of a piece meet in float64: each adds and writes its share of the rows of the sixteen-row tiles
  float* meet = smem;                                   // [8][kC1Acc][64]
#pragma unroll
  for (int i = 0; i < kC1RT; ++i)
#pragma unroll
    for (int q = 0; q < kC1CT; ++q) {
      if (SETS > 1) acc[0][i][q] += acc[SETS - 1][i][q];
#pragma unroll
      for (int r = 0; r < 4; ++r) meet[(wave * kC1Acc + (i * kC1CT + q) * 4 + r) * 64 + lane] = acc[0][i][q][r];
    }
  __syncthreads();
  if (!live) return;
  float* out = reinterpret_cast<float*>(p.out) + (size_t)range * p.Cout * K;
  constexpr int EACH = kC1Acc / RS;                     // accumulators that a wavefront finishes
  float v[EACH];
#pragma unroll
  for (int j = 0; j < EACH; ++j) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < RS; ++w) t += (double)meet[((slot + w * GPB) * kC1Acc + rsub * EACH + j) * 64 + lane];
    v[j] = (float)t;
  }
  if (pco * 16 * kC1RT + 16 * kC1RT <= p.Cout && pkg * 16 * kC1CT + 16 * kC1CT <= K) {       // a whole piece: nothing to ask for each value
#pragma unroll
    for (int j = 0; j < EACH; ++j) {
      const int e = rsub * EACH + j, i = e / (4 * kC1CT), q = e / 4 % kC1CT, r = e % 4;
      out[((pco * kC1RT + i) * 16 + 4 * rg + r) * K + (pkg * kC1CT + q) * 16 + l16] = v[j];
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < EACH; ++j) {
    const int e = rsub * EACH + j, i = e / (4 * kC1CT), q = e / 4 % kC1CT, r = e % 4;
    const int k = (pkg * kC1CT + q) * 16 + l16, co = (pco * kC1RT + i) * 16 + 4 * rg + r;
    if (co < p.Cout && k < K) out[co * K + k] = v[j];
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

// 16 x 16 of g_w by NW wavefronts that split the rows: no partial buffers, rounds of sixteen row groups (16 wavefronts: one up to 1024 rows, two
// at 2048; the 8 with PRO twice as many).  Every wavefront adds in 16 / NW chains, so that none is longer than 16 wavefronts would have (a
// step of four rows is one addition): with one chain each the gradients of three layers in one stage were 3.2e-7 and 3.8e-7 off 64 bits at 1024 and 2048
// rows, 2.97e-7 and 3.25e-7 in launches of their own with 16 wavefronts.
template <typename T, bool PRO, int NW>
__device__ __forceinline__ void conv1d_wgrad_tile(const Conv1dArgs& p, float* __restrict__ g_w, const int bid) {
  constexpr int U = 16, CH = 16 / NW;
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
  f4v acc[CH];
#pragma unroll
  for (int c = 0; c < CH; ++c) acc[c] = f4v{0.f, 0.f, 0.f, 0.f};
  int t = mb + mg - (int)p.dW.div(mb + mg) * p.W;
  T dr[U], xr[U], zr[PRO ? U : 1];
  bool xin[U];
  auto request = [&](const int m) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int mm = m + 4 * u + mg;
      xin[u] = mm < me && k_ok && (unsigned)(t + dt) < (unsigned)p.W;
      // Rows outside are read at the nearest one inside and not used: of a select between two rows the compiler makes two loads, each behind a
      // branch, and waits for most of them on its own (two layers of 8 -> 8 channels, 2048 rows, no sums taken 25.6 / 24.3 us).  Where the sums are
      // finished behind the requests nothing waits for these, and a load that is not made is the cheaper one (sensor network, batch 8, 52.6 / 52.2).
      const int at = (PRO ? mm < me ? mm : mb < p.M ? mb : 0 : min(mm, me - 1)) * p.Cout;
      const int xat = (PRO ? xin[u] ? mm + dt : 0 : min(max(mm + dt, 0), p.M - 1)) * p.Cin;
      dr[u] = D[at];
      if (PRO) zr[PRO ? u : 0] = Z[at];
      xr[u] = X[xat];
      t += 4;
      t -= t >= p.W ? p.W : 0;
    }
  };
  if constexpr (PRO) {
    request(mb);                         // in front of the loop only where something else happens meanwhile
    finish_backward_n(p.pend, p.Cout, p.g_gamma, p.g_beta, p.own_writes && bid == 0, 64 * NW, fin, vec);
    const int c = co_ok ? co : 0;
    k1 = vec[0][c]; k2 = vec[1][c]; k3 = vec[2][c];
  }
  for (int m = mb; m < me; m += 4 * U) {
    if (!PRO || m != mb) request(m);
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
      acc[u % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(din ? d : 0.f, xin[u] ? x : 0.f, acc[u % CH], 0, 0, 0);
    }
  }
#pragma unroll
  for (int c = 1; c < CH; ++c) acc[0] += acc[c];
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][4 * mg + r][l16] = acc[0][r];
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
// First layers in front of others, a step of the stage (forward, backward, update) with an average, a fully connected layer and the loss behind, us, patch matrices /
// here, 32768, 65536, 131072 and 262144 rows.  fp32: in front of a layer of 3 taps 3 -> 16, 3 taps, 103 / 90, 122 / 114, 178 / 178, 282 / 288; 1 -> 32, 5 taps 102 / 93,
// 130 / 124, 192 / 195, 297 / 311; 5 -> 32, 9 taps 105 / 96, 139 / 127, 213 / 199, 330 / 319; 12 -> 24, 3 taps 101 / 90, 131 / 119, 203 / 186, 313 / 296; 9 -> 64, 5 taps 122 /
// 113, 168 / 157, 262 / 249, 442 / 423; the sensor network's 9 -> 32, 5 taps 199 / 192, 297 / 288, 485 / 474.  bfloat16 (odd channels +): 3 -> 16 90 / 86, 113 / 108, 159 /
// 164; 12 -> 24 96 / 86, 115 / 107, 172 / 167, 254 / 263; 9 -> 64, 5 taps 106 / 106, 139 / 144; 10 -> 64, 9 taps 112 / 111, 149 / 152; the sensor network 177 / 173, 261 / 260.
// The other lines lie where both sides were even when the row tiles took their weights through LDS in chunks; the kernels here have since gained 7 - 45 %
// and the other side nothing, so layers just beyond a line are now often faster here too (marked +: sent to the patch matrices all the same), and none is
// slower than it was.  Steps, us: fp32 64 -> 64, 5 taps, alone, 32768 rows 164 / 88; first layers alone 9 -> 32, 5 taps, 32768 41.7 / 36.0 +, 131072 79.9 / 70.3 +, 3 ->
// 64, 3 taps, 131072 97.6 / 84.3, 262144 142 / 139 +, bfloat16 3 -> 8, 3 taps, 16384 37.6 / 32.4, 32768 38.6 / 35.5 +, 524288 76 / 144, 9 -> 32, 5 taps, 2304 29.5 / 29.4,
// 65536 42.4 / 45.0; chain 8 -> 8, 3 taps, 131072 207 / 177, 262144 327 / 287 +.  bfloat16: chain
// 64 -> 64, 9 taps, 2304 rows 143 / 136 +, 8192 237 / 151, 32768 487 / 288, 7 taps, 131072 1121 / 772 +;
// 48 -> 48, 7 taps, 2304 127 / 109 +, 6144 157 / 123 +, 32768 352 / 228, 131072 893 / 637 +; 32 -> 64, 9 taps, 4096 153 / 115 +, 6144 176 / 117; chain
// 8 -> 8, 3 taps, 65536 148 / 118, 131072 181 / 169 +, 1048576 614 / 912; 32 -> 32, 3 taps, 131072 341 / 222, 524288 929 / 668 +; a layer behind others alone in
// its stage 64 -> 64, 9 taps 4096 55.3 / 56.7, 8192 72.0 / 61.6 +, 24576 106 / 104, 5 taps 32768 93.8 / 78.9, 65536 128 / 120 +, 3 taps 32768 80.0 / 66.9, 65536
// 104 / 103; 16 -> 16, 5 taps, in front of another 32768 120 / 74, 131072 219 / 144, 524288 480 / 423 +.
int conv1d_pays(int dt, const ConvGeom& g, bool first, bool alone, bool forks) {
  const size_t M = (size_t)g.N * g.Win;
  const int lo = g.Cin < g.Cout ? g.Cin : g.Cout, hi = g.Cin < g.Cout ? g.Cout : g.Cin;
  const int K = g.kw * g.Cin, both = g.kw * (g.Cin + g.Cout), weights = K * g.Cout;
  const bool odd = g.Cin % 8 != 0;                    // read value by value here
  if (conv1d_small(g)) return 1;
  if (first && dt == 0 && alone) {
    if (g.Cout > 32 ? odd && K <= 54 && M >= 200000 : K <= 45 && M >= 32768) return 0;
    if (odd && g.Cin < 12 && K <= 81 && (g.Cout <= 32 || K >= 45) && M >= 131072) return 0;
  }
  if (first && dt == 0 && !alone && odd && K < 24 && g.Cout <= 32 && M >= 98304) return 0;      // little to multiply for each row read value by value
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

// One block per CU over a range of tiles, each leaving one partial.  Tiles of 128 rows, 64 or 32, by the longest range (a tile costs as much
// as some 24 rows on top of its own): 32768 rows are one of 128 to a block, 8192 one of 32.  64 columns or 32: a 64-wide tile over 32
// columns or fewer would be half padding.
template <typename T, bool DGRAD>
static void conv1d_rows(hipStream_t st, Conv1dArgs& a, int* P_out) {
  const int WC = a.NC <= 32 ? 1 : 2;
  auto ranges = [&](int ti) { const int n = (a.M + ti - 1) / ti; return (n + kC1Blocks - 1) / kC1Blocks; };
  int TI = 128;
  for (int ti : {64, 32})
    if (ranges(ti) * (ti + 24) < ranges(TI) * (TI + 24)) TI = ti;
  a.itiles = (a.M + TI - 1) / TI;
  a.tiles_per_range = ranges(TI);
  const int nr = (a.itiles + a.tiles_per_range - 1) / a.tiles_per_range;
  const int LDR = a.CP + 4, KP = a.kw * a.CP;
  const bool split = !(WC == 2 && TI == 128);
  const size_t fixed = (split ? 8 * 16 * 64 : 0) + (size_t)(a.tiles_per_range > 1 ? 2 : 1) * ((TI + a.kw) * LDR + 4) + 8;       // floats
  const int fit = (int)((kC1Lds / sizeof(float) - fixed) / (32 * WC)) - 4, phases = (KP + fit - 1) / fit;
  a.kphase = ((KP / 8 + phases - 1) / phases) * 8;
  if (a.kphase > fit) a.kphase = fit / 8 * 8;
  const size_t lds = (fixed + (size_t)32 * WC * (a.kphase + 4)) * sizeof(float);
  if (P_out) *P_out = nr;
#define FTP_ROWS(wc, ksp) hipLaunchKernelGGL((conv1d_rows_k<T, DGRAD, wc, ksp>), dim3(nr), dim3(512), lds, st, a)
  if (WC == 1) { if (TI == 128) FTP_ROWS(1, 2); else if (TI == 64) FTP_ROWS(1, 4); else FTP_ROWS(1, 8); }
  else { if (TI == 128) FTP_ROWS(2, 1); else if (TI == 64) FTP_ROWS(2, 2); else FTP_ROWS(2, 4); }
#undef FTP_ROWS
}

int conv1d_small_ok(const ConvGeom& g) { return conv1d_ok(g) && conv1d_small(g); }

// tiles of the data gradient and of the weight gradient of a short layer
static int conv1d_bwd_tiles(const ConvGeom& g, int* weights) {
  *weights = (g.kw * g.Cin + 15) / 16 * ((g.Cout + 15) / 16);
  return (g.N * g.Win + 15) / 16 * ((g.Cin + 15) / 16);
}

// The BatchNorm backward on the way into both gradients saves a launch and costs instructions in every block: as long as each block has a CU to
// itself, and in bfloat16, whose gradient elements are read one by one, up to 1536 rows (three rounds of a weight tile's rows).  A step of a chain of
// two such layers, us, launches of their own / on the way in: fp32 64 channels, 5 taps, 1152 rows (224 blocks) 53.6 / 50.1, 1536 (272) 56.2 / 56.9, 2048 (336)
// 60.0 / 63.3, 9 taps, 512 rows (208) 45.9 / 42.6, 1024 (272) 49.8 / 52.0, 1600 (344) 61.5 / 67.8; 32 channels, 5 taps, 2048 rows (148) 51.9 / 48.9; bfloat16 1536 rows
// 46.8 / 44.3, 2048 48.4 / 48.2, 16 channels, 3 taps, 1536 rows 41.4 / 40.2, 2048 41.9 / 43.6.
int conv1d_bwd_sums_ok(int dt, const ConvGeom& g) {
  int weights;
  const int data = conv1d_bwd_tiles(g, &weights);
  return conv1d_small_ok(g) && (data + 1) / 2 + weights <= kC1Blocks && (dt == 0 || g.N * g.Win <= 1536);
}

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
int conv1d_finish_ok(const ConvGeom& g, int P) { return P <= kC1Blocks && g.Cin % 8 == 0; }

void conv1d_dgrad(int dt, hipStream_t st, const void* dz, const void* w, const ConvGeom& g, void* dIn, HView prev, float* sums, int* P_out) {
  Conv1dArgs a = conv1d_args(g, true);
  a.x = dz; a.w = w; a.out = dIn; a.stats = sums; a.prev = View{prev.z, prev.scale, prev.shift, prev.act};
  KScope ks(st, "conv1d_dgrad", ((double)a.M * (g.Cin + g.Cout) + (double)g.Cout * g.kw * g.Cin) * (dt == 0 ? 4.0 : 2.0),
            2.0 * a.M * g.Cout * g.kw * g.Cin, a.M, g.kw * g.Cout, g.Cin);
  FTP_DISPATCH(dt, (conv1d_rows<T, true>(st, a, P_out)));
}

// Pieces to a block: one, two from four pieces on, four from eight; the blocks of a range each bring in all its rows.  From four tiles to a range
// on that costs more than the partials of twice as many ranges, and a block takes twice the pieces, as long as at most one wavefront group in
// a range is left without one.  Launch and the sum of its partials, us (6 of the events), before / now: fp32 131072 rows 3 -> 64, 3 taps, 45 / 35, 32 -> 32,
// 3 taps, 44 / 35 (two pieces), 64 -> 8, 3 taps, 73 / 46 (three), 64 -> 64, 3 taps, 84 / 84 (six: 83 - 89 with four to a block), 32 -> 64, 5 taps,
// 56 / 51 (four); 32768 rows 3 -> 64, 3 taps, 21 / 19, 64 -> 8 30 / 23, 32 -> 64, 5 taps, 25 / 25; 8192 rows (one or two tiles to a range) 8 -> 64, 5 taps, 16, 17 with
// two.  bfloat16 131072 rows 3 -> 64, 3 taps, 45 / 34, 64 -> 8, 3 taps, 51 / 43, 32 -> 64, 5 taps, 50 / 46.
static Conv1dWgArgs conv1d_wgrad_plan(const ConvGeom& g, int* P) {
  Conv1dWgArgs a{};
  a.c = conv1d_args(g, false);
  a.nco = (g.Cout + 16 * kC1RT - 1) / (16 * kC1RT);
  a.nkg = (g.kw * g.Cin + 16 * kC1CT - 1) / (16 * kC1CT);
  const int pieces = a.nco * a.nkg;
  int gpb = pieces >= 8 ? 4 : pieces >= 4 ? 2 : 1;
  auto groups = [&](int n) { return (pieces + n - 1) / n; };
  auto ranges = [&](int n) { const int r = kC1Blocks / groups(n); return r > 0 ? r : 1; };
  while (gpb < 4 && gpb < pieces && groups(2 * gpb) * 2 * gpb <= pieces + 1 && ((a.c.M + 63) / 64 + ranges(gpb) - 1) / ranges(gpb) >= 4) gpb *= 2;
  a.rs = 8 / gpb;
  a.ngrp = groups(gpb);
  const int want = ranges(gpb);
  a.rows = (a.c.M + 63) / 64 * 2 <= want ? 32 : 64;      // tiles of 64 would leave half of the CUs idle
  a.c.itiles = (a.c.M + a.rows - 1) / a.rows;
  a.c.tiles_per_range = (a.c.itiles + want - 1) / want;
  *P = (a.c.itiles + a.c.tiles_per_range - 1) / a.c.tiles_per_range;
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
    const size_t tiles = (size_t)2 * ((2 * a.rows + g.kw - 1) * kC1WgLd + 4), meet = (size_t)8 * kC1Acc * 64;
    const size_t lds = (tiles > meet ? tiles : meet) * sizeof(float);
    const dim3 grid(P * a.ngrp);
#define FTP_WGRAD(rs, rows) FTP_DISPATCH(dt, hipLaunchKernelGGL((conv1d_wgrad_k<T, rs, rows>), grid, dim3(512), lds, st, a))
    if (a.rows == 64) { if (a.rs == 2) FTP_WGRAD(2, 64); else if (a.rs == 4) FTP_WGRAD(4, 64); else FTP_WGRAD(8, 64); }
    else { if (a.rs == 2) FTP_WGRAD(2, 32); else if (a.rs == 4) FTP_WGRAD(4, 32); else FTP_WGRAD(8, 32); }
#undef FTP_WGRAD
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
  const int K = g.kw * g.Cin;
  int nw;
  const int tiles = conv1d_bwd_tiles(g, &nw), nd = dIn ? (tiles + groups - 1) / groups : 0;
  a.own_writes = nd == 0;              // who adds to the BatchNorm's gradients: the first data-gradient block, where there is one
  KScope ks(st, dIn ? "conv1d_bwd" : "conv1d_wgrad", (double)d.M * (2.0 * g.Cin + g.Cout) * (dt == 0 ? 4.0 : 2.0) + (double)g.Cout * K * 8, 4.0 * d.M * g.Cout * K,
            d.M, K, g.Cout);
  if (sums) FTP_DISPATCH(dt, hipLaunchKernelGGL((conv1d_bwd_small_k<T, true, true, 8>), dim3(nd + nw), dim3(512), 0, st, d, a, g_w, nd));
  else FTP_DISPATCH(dt, hipLaunchKernelGGL((conv1d_bwd_small_k<T, true, false, 16>), dim3(nd + nw), dim3(1024), 0, st, d, a, g_w, nd));
}

}  // namespace ftp
