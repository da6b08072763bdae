// Pointwise (1x1) convolution and fully connected layers as MFMA GEMMs.
//
// One kernel computes C[i][j] = sum_r X(i, r) * Y(j, r) for the three passes:
//   forward : i = pixel m, j = cout n, r = cin k   X = A'[m][k]   Y = W[n][k]
//   dgrad   : i = pixel m, j = cin k,  r = cout n  X = dZ[m][n]   Y = W[n][k]  (read transposed)
//   wgrad   : i = cout n,  j = cin k,  r = pixel m X = dZ[m][n]   Y = A'[m][k] (both transposed,
//             the pixel range split over blocks into fp32 partials summed in a fixed order)
// A' is read through a View (the producer's BatchNorm + activation applied on load).
//
// These GEMMs stream a tall activation matrix once against a small weight matrix,
// so they are HBM-bound; the kernel is built around that:
//   * a block owns one 64-wide column tile and walks a contiguous range of row
//     tiles, so weights stay in L2 and per-column BatchNorm sums accumulate in
//     registers over the whole range (one partial per block, fixed order);
//   * the next reduction chunk is fetched from HBM into registers while the
//     current one is multiplied out of LDS (software pipeline over a flat
//     (row tile, chunk) sequence);
//   * the weight tile is stored row-permuted so that a lane's two accumulators are adjacent
//     columns: results leave straight from the MFMA registers and every store instruction
//     writes whole 128/256-byte row segments.
// Three tile shapes: 128 x 64 with the four wavefronts splitting the rows (tall problems);
// 32 x 64 with the four wavefronts splitting a 128-long reduction chunk (few row tiles, long
// reductions); and 16 x 16 with fragments loaded straight from global memory (at most 2048
// rows: pure latency, see pw_gemm_tiny_body), where data gradient and weight gradient of a
// layer share one launch and the weight gradient needs no partial buffers.
// bfloat16 uses v_mfma_f32_32x32x16_bf16 (16x16x32 in the short kernels), float uses
// v_mfma_f32_32x32x2_f32 (16x16x4).
#include <type_traits>
#include "dev_common.h"
#include "kernels.h"
#include "bn_pending.h"

namespace ftp {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

enum { BJ = 64, CLD = BJ + 4 };
enum { MODE_FWD = 0, MODE_DGRAD = 1, MODE_WGRAD = 2 };

template <bool SMALL> struct Shape {
  enum { TI = SMALL ? 32 : 128, CH = SMALL ? 128 : 32 };
};
template <typename T> struct Pad;
template <> struct Pad<float> { enum { V = 4 }; };
template <> struct Pad<bf16_t> { enum { V = 8 }; };

struct GemmArgs {
  const void* x;     // dZ (dgrad, wgrad) or A (fwd; through view)
  const void* y;     // W (fwd, dgrad) or A (wgrad; through view)
  View view;         // prologue of A' (fwd: on x, wgrad: on y)
  const float* bias; // fwd
  const void* res;   // dgrad: added to the result
  void* out;         // T (fwd, dgrad) or float partials (wgrad)
  float* stats;      // fwd: partial[nranges][2][N] column sums of the stored output, or nullptr
  size_t M;
  int K, N;
  int jtiles, itiles;
  int nranges;       // fwd/dgrad: row-tile ranges; wgrad: splits of the pixel range
  int tiles_per_range;
  size_t mchunk;     // wgrad: pixels per split
};

// One operand tile: ROWS (i or j) x CH (r).  RC = source is r-contiguous (element (i,r) at
// src[i*ld + r]); otherwise i-contiguous (element (i,r) at src[r*ld + i]) and transposed on the
// way into LDS.  The view prologue indexes scale/shift by the channel, which is r for RC
// sources and i for the others.
// PERM stores tile row n at LDS row (n & 1) * 32 + (n >> 1) (64-row tiles only), so that the two
// MFMA column sub-tiles of a lane are the adjacent columns 2*lane and 2*lane+1.
__device__ __forceinline__ int perm64(int n) { return ((n & 1) << 5) | (n >> 1); }

template <typename T, int ROWS, int CH, bool RC, bool USE_VIEW, bool PERM = false>
struct TileLoader {
  enum { NVEC = ROWS * CH / 8, PER = (NVEC + 255) / 256, LD = CH + Pad<T>::V };
  Raw<T> raw[PER];
  unsigned ok;      // bit q: raw[q] holds a full in-bounds vector

  __device__ __forceinline__ void coords(int v, int& i, int& r) const {
    if (RC) { i = v / (CH / 8); r = (v % (CH / 8)) * 8; }
    else { r = v / (ROWS / 8); i = (v % (ROWS / 8)) * 8; }
  }

  __device__ __forceinline__ void fetch(const T* __restrict__ src, size_t ld, size_t i0, size_t ni, size_t r0,
                                        size_t nr) {
    ok = 0;
    const bool vec_ok = (ld % 8) == 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      int v = threadIdx.x + q * 256;
      if (v >= NVEC) break;
      int i, r;
      coords(v, i, r);
      size_t gi = i0 + i, gr = r0 + r;
      bool full = vec_ok && (RC ? (gi < ni && gr + 8 <= nr) : (gr < nr && gi + 8 <= ni));
      if (full) {
        raw_load(raw[q], RC ? src + gi * ld + gr : src + gr * ld + gi);
        ok |= 1u << q;
      }
    }
  }

  __device__ __forceinline__ void commit(T* lds, const T* __restrict__ src, size_t ld, size_t i0, size_t ni,
                                         size_t r0, size_t nr, const View& vw) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      int v = threadIdx.x + q * 256;
      if (v >= NVEC) break;
      int i, r;
      coords(v, i, r);
      size_t gi = i0 + i, gr = r0 + r;
      float val[8];
      size_t ch = RC ? gr : gi;      // first channel of the vector
      if (ok & (1u << q)) {
        raw_unpack(raw[q], val);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          size_t ei = RC ? gi : gi + e, er = RC ? gr + e : gr;
          val[e] = (ei < ni && er < nr) ? to_f32(RC ? src[ei * ld + er] : src[er * ld + ei]) : 0.f;
        }
      }
      if (USE_VIEW && vw.scale) {
        if (ok & (1u << q)) {          // whole vector in range: channels ch .. ch+7 exist
          float sc[8], sh[8];
          load8(vw.scale + ch, sc);
          load8(vw.shift + ch, sh);
          const float lo = act_lo(vw.act), hi = act_hi(vw.act);
#pragma unroll
          for (int e = 0; e < 8; ++e) val[e] = clamp_act(fmaf(val[e], sc[e], sh[e]), lo, hi);
        } else {
          size_t nch = RC ? nr : ni;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            // out-of-range elements must stay exactly zero
            bool in = RC ? (gi < ni && gr + e < nr) : (gr < nr && gi + e < ni);
            if (in && ch + e < nch) val[e] = act_apply(fmaf(val[e], vw.scale[ch + e], vw.shift[ch + e]), vw.act);
          }
        }
      }
      if (RC) {
        store8(lds + (PERM ? perm64(i) : i) * LD + r, val);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) lds[(PERM ? perm64(i + e) : i + e) * LD + r] = from_f32<T>(val[e]);
      }
    }
  }
};

// Transposing loader for "i contiguous" sources (element (i, r) at src[r*ld + i]).  A thread takes
// two consecutive reduction rows r, r+1 of the same 8 columns and writes LDS in (r, r+1) pairs:
// one 32-bit (bfloat16) or 64-bit (float) store per column instead of two 16/32-bit ones, and for
// plain bfloat16 data the pair is assembled from the raw bits without a float round trip.
__device__ __forceinline__ void lds_put_pair(float* p, float a, float b) { *reinterpret_cast<float2*>(p) = make_float2(a, b); }
__device__ __forceinline__ void lds_put_pair(bf16_t* p, float a, float b) { *reinterpret_cast<uint32_t*>(p) = f32x2_to_bf16x2(a, b); }

template <typename T, int ROWS, int CH, bool USE_VIEW, bool PERM>
struct TransLoader {
  enum { NITEM = (ROWS / 8) * (CH / 2), PER = (NITEM + 255) / 256, LD = CH + Pad<T>::V };
  Raw<T> raw[PER][2];
  unsigned ok;      // bit 2q+u: raw[q][u] holds a full in-bounds vector

  // consecutive lanes take consecutive row pairs of the same 8 columns, so their LDS stores fall into
  // consecutive words of one LDS row (the other order would put 16 lanes on one bank)
  __device__ __forceinline__ void coords(int item, int& i, int& r) const {
    r = (item % (CH / 2)) * 2;
    i = (item / (CH / 2)) * 8;
  }

  __device__ __forceinline__ void fetch(const T* __restrict__ src, size_t ld, size_t i0, size_t ni, size_t r0,
                                        size_t nr) {
    ok = 0;
    const bool vec_ok = (ld % 8) == 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int item = threadIdx.x + q * 256;
      if (item >= NITEM) break;
      int i, r;
      coords(item, i, r);
      const size_t gi = i0 + i;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const size_t gr = r0 + r + u;
        if (vec_ok && gr < nr && gi + 8 <= ni) {
          raw_load(raw[q][u], src + gr * ld + gi);
          ok |= 1u << (2 * q + u);
        }
      }
    }
  }

  __device__ __forceinline__ void commit(T* lds, const T* __restrict__ src, size_t ld, size_t i0, size_t ni,
                                         size_t r0, size_t nr, const View& vw) const {
    const bool view = USE_VIEW && vw.scale != nullptr;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int item = threadIdx.x + q * 256;
      if (item >= NITEM) break;
      int i, r;
      coords(item, i, r);
      const size_t gi = i0 + i;
      const unsigned both = (ok >> (2 * q)) & 3u;
      if (sizeof(T) == 2 && !view && both == 3u) {
        // raw bits straight into (r, r+1) pairs
        const uint32_t* w0 = reinterpret_cast<const uint32_t*>(&raw[q][0]);
        const uint32_t* w1 = reinterpret_cast<const uint32_t*>(&raw[q][1]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t a = w0[e >> 1], b = w1[e >> 1];
          const uint32_t pr = (e & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
          *reinterpret_cast<uint32_t*>(lds + (PERM ? perm64(i + e) : i + e) * LD + r) = pr;
        }
        continue;
      }
      float val[2][8];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const size_t gr = r0 + r + u;
        if (ok & (1u << (2 * q + u))) {
          raw_unpack(raw[q][u], val[u]);
          if (view) {
            float sc[8], sh[8];
            load8(vw.scale + gi, sc);
            load8(vw.shift + gi, sh);
            const float lo = act_lo(vw.act), hi = act_hi(vw.act);
#pragma unroll
            for (int e = 0; e < 8; ++e) val[u][e] = clamp_act(fmaf(val[u][e], sc[e], sh[e]), lo, hi);
          }
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float x = 0.f;                      // out-of-range elements must stay exactly zero
            if (gr < nr && gi + e < ni) {
              x = to_f32(src[gr * ld + gi + e]);
              if (view) x = act_apply(fmaf(x, vw.scale[gi + e], vw.shift[gi + e]), vw.act);
            }
            val[u][e] = x;
          }
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) lds_put_pair(lds + (PERM ? perm64(i + e) : i + e) * LD + r, val[0][e], val[1][e]);
    }
  }
};

// Branch-free loaders for problems whose extents along the vectorised dimension are multiples of 8
// (every layer of the networks here except the classifier output): a vector is then wholly inside or
// wholly outside the tensor; outside ones are loaded from the base address, which is always valid,
// and zeroed by a select.  The generic loaders above spend most of their instructions on
// per-element bounds branches that never fire for such shapes.
template <typename T, int ROWS, int CH, bool USE_VIEW, bool PERM>
struct VecTileLoader {   // r-contiguous source
  enum { NVEC = ROWS * CH / 8, PER = NVEC / 256, LD = CH + Pad<T>::V };
  static_assert(NVEC % 256 == 0, "tile must divide over 256 threads");
  Raw<T> raw[PER];
  unsigned ok;
  float psc[USE_VIEW ? PER : 1][8], psh[USE_VIEW ? PER : 1][8];   // view vectors requested together with the tile

  // the scale / shift of the channels (= reduction indices) of the vectors that fetch() requests for the same step
  __device__ __forceinline__ void fetch_view(const View& vw, size_t r0, size_t nr) {
    if (!USE_VIEW || !vw.scale) return;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int v = threadIdx.x + q * 256;
      const int r = (v % (CH / 8)) * 8;
      const size_t ch = r0 + r < nr ? r0 + r : 0;
      load8(vw.scale + ch, psc[q]);
      load8(vw.shift + ch, psh[q]);
    }
  }
  // commit with the view vectors that fetch_view requested
  __device__ __forceinline__ void commit_pv(T* lds, int act) const {
    const float lo = act_lo(act), hi = act_hi(act);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int v = threadIdx.x + q * 256;
      const int i = v / (CH / 8), r = (v % (CH / 8)) * 8;
      const bool in = (ok >> q) & 1u;
      float val[8];
      raw_unpack(raw[q], val);
#pragma unroll
      for (int e = 0; e < 8; ++e) val[e] = in ? clamp_act(fmaf(val[e], psc[USE_VIEW ? q : 0][e], psh[USE_VIEW ? q : 0][e]), lo, hi) : 0.f;
      store8(lds + (PERM ? perm64(i) : i) * LD + r, val);
    }
  }

  __device__ __forceinline__ void fetch(const T* __restrict__ src, size_t ld, size_t i0, size_t ni, size_t r0,
                                        size_t nr) {
    ok = 0;
    // every address first, then the loads back to back: an address computed between two loads can land in a
    // register the compiler still counts as the target of an earlier load, and then each load waits for the one before
    const T* ptr[PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int v = threadIdx.x + q * 256;
      const int i = v / (CH / 8), r = (v % (CH / 8)) * 8;
      const size_t gi = i0 + i, gr = r0 + r;
      const bool in = gi < ni && gr < nr;
      ptr[q] = in ? src + gi * ld + gr : src;
      ok |= (in ? 1u : 0u) << q;
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) raw_load(raw[q], ptr[q]);
  }

  __device__ __forceinline__ void commit(T* lds, const T* __restrict__, size_t, size_t, size_t, size_t r0, size_t,
                                         const View& vw) const {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int v = threadIdx.x + q * 256;
      const int i = v / (CH / 8), r = (v % (CH / 8)) * 8;
      const bool in = (ok >> q) & 1u;
      float val[8];
      raw_unpack(raw[q], val);
      if (USE_VIEW && vw.scale) {
        const size_t ch = in ? r0 + r : 0;
        float sc[8], sh[8];
        load8(vw.scale + ch, sc);
        load8(vw.shift + ch, sh);
        const float lo = act_lo(vw.act), hi = act_hi(vw.act);
#pragma unroll
        for (int e = 0; e < 8; ++e) val[e] = clamp_act(fmaf(val[e], sc[e], sh[e]), lo, hi);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) val[e] = in ? val[e] : 0.f;
      store8(lds + (PERM ? perm64(i) : i) * LD + r, val);
    }
  }

};

template <typename T, int ROWS, int CH, bool USE_VIEW, bool PERM>
struct VecTransLoader {  // i-contiguous source, transposed into (r, r+1) pairs like TransLoader
  enum { NITEM = (ROWS / 8) * (CH / 2), PER = (NITEM + 255) / 256, LD = CH + Pad<T>::V };
  Raw<T> raw[PER][2];
  unsigned ok;
  // the view's scale / shift of this thread's columns: the same for every step of a block (the channel is the tile's
  // i index), so they are loaded once (hold_view) instead of in every commit, where the load could not be hidden
  float vsc[USE_VIEW ? PER : 1][8], vsh[USE_VIEW ? PER : 1][8];
  bool held = false;

  __device__ __forceinline__ void hold_view(const View& vw, size_t i0, size_t ni) {
    if (!USE_VIEW || !vw.scale) return;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int item = threadIdx.x + q * 256;
      const int i = (item / (CH / 2)) * 8;
      const size_t ch = (item < NITEM && i0 + i < ni) ? i0 + i : 0;      // ni is a multiple of 8 here
      load8(vw.scale + ch, vsc[q]);
      load8(vw.shift + ch, vsh[q]);
    }
    held = true;
  }

  __device__ __forceinline__ void fetch(const T* __restrict__ src, size_t ld, size_t i0, size_t ni, size_t r0,
                                        size_t nr) {
    ok = 0;
    const T* ptr[PER][2];                    // every address first, then the loads back to back (see VecTileLoader)
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int item = threadIdx.x + q * 256;
      const int r = (item % (CH / 2)) * 2, i = (item / (CH / 2)) * 8;
      const size_t gi = i0 + i;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const size_t gr = r0 + r + u;
        const bool in = item < NITEM && gr < nr && gi < ni;
        ptr[q][u] = in ? src + gr * ld + gi : src;
        ok |= (in ? 1u : 0u) << (2 * q + u);
      }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      raw_load(raw[q][0], ptr[q][0]);
      raw_load(raw[q][1], ptr[q][1]);
    }
  }

  __device__ __forceinline__ void commit(T* lds, const T* __restrict__, size_t, size_t i0, size_t, size_t, size_t,
                                         const View& vw) const {
    const bool view = USE_VIEW && vw.scale != nullptr;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int item = threadIdx.x + q * 256;
      if (item >= NITEM) break;
      const int r = (item % (CH / 2)) * 2, i = (item / (CH / 2)) * 8;
      const bool in0 = (ok >> (2 * q)) & 1u, in1 = (ok >> (2 * q + 1)) & 1u;
      if (sizeof(T) == 2 && !view) {
        // raw bits straight into (r, r+1) pairs
        const uint32_t* w0 = reinterpret_cast<const uint32_t*>(&raw[q][0]);
        const uint32_t* w1 = reinterpret_cast<const uint32_t*>(&raw[q][1]);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t a = in0 ? w0[e >> 1] : 0u, b = in1 ? w1[e >> 1] : 0u;
          const uint32_t pr = (e & 1) ? ((a >> 16) | (b & 0xffff0000u)) : ((a & 0xffffu) | (b << 16));
          *reinterpret_cast<uint32_t*>(lds + (PERM ? perm64(i + e) : i + e) * LD + r) = pr;
        }
        continue;
      }
      float val[2][8];
      raw_unpack(raw[q][0], val[0]);
      raw_unpack(raw[q][1], val[1]);
      if (view) {
        float sc[8], sh[8];
        if (held) {
#pragma unroll
          for (int e = 0; e < 8; ++e) { sc[e] = vsc[USE_VIEW ? q : 0][e]; sh[e] = vsh[USE_VIEW ? q : 0][e]; }
        } else {
          const size_t ch = (in0 || in1) ? i0 + i : 0;     // same channels for both rows
          load8(vw.scale + ch, sc);
          load8(vw.shift + ch, sh);
        }
        const float lo = act_lo(vw.act), hi = act_hi(vw.act);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          val[0][e] = clamp_act(fmaf(val[0][e], sc[e], sh[e]), lo, hi);
          val[1][e] = clamp_act(fmaf(val[1][e], sc[e], sh[e]), lo, hi);
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        lds_put_pair(lds + (PERM ? perm64(i + e) : i + e) * LD + r, in0 ? val[0][e] : 0.f, in1 ? val[1][e] : 0.f);
    }
  }
};

template <typename T, int ROWS, int CH, bool RC, bool USE_VIEW, bool PERM, bool VEC>
struct LoaderSel { typedef TileLoader<T, ROWS, CH, true, USE_VIEW, PERM> type; };
template <typename T, int ROWS, int CH, bool USE_VIEW, bool PERM>
struct LoaderSel<T, ROWS, CH, false, USE_VIEW, PERM, false> { typedef TransLoader<T, ROWS, CH, USE_VIEW, PERM> type; };
template <typename T, int ROWS, int CH, bool USE_VIEW, bool PERM>
struct LoaderSel<T, ROWS, CH, true, USE_VIEW, PERM, true> { typedef VecTileLoader<T, ROWS, CH, USE_VIEW, PERM> type; };
template <typename T, int ROWS, int CH, bool USE_VIEW, bool PERM>
struct LoaderSel<T, ROWS, CH, false, USE_VIEW, PERM, true> { typedef VecTransLoader<T, ROWS, CH, USE_VIEW, PERM> type; };

// ---- MFMA over one staged chunk of 32 reduction elements starting at column c0 -------
__device__ __forceinline__ void mma32(const bf16_t* xs, const bf16_t* ys, int LD, int irow, int lane, int c0,
                                      f16v acc[2]) {
  const int h = lane >> 5, jl = lane & 31;
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    uint4 a = *reinterpret_cast<const uint4*>(xs + irow * LD + c0 + ks * 16 + h * 8);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      uint4 b = *reinterpret_cast<const uint4*>(ys + (t * 32 + jl) * LD + c0 + ks * 16 + h * 8);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), acc[t], 0, 0, 0);
    }
  }
}

__device__ __forceinline__ void mma32(const float* xs, const float* ys, int LD, int irow, int lane, int c0,
                                      f16v acc[2]) {
  const int h = lane >> 5, jl = lane & 31;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    // lane half h holds r = 8q+4h .. +3; instruction t multiplies r = 8q+t and 8q+4+t
    float4 a = *reinterpret_cast<const float4*>(xs + irow * LD + c0 + q * 8 + h * 4);
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float4 b = *reinterpret_cast<const float4*>(ys + (t * 32 + jl) * LD + c0 + q * 8 + h * 4);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, acc[t], 0, 0, 0);
      acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, acc[t], 0, 0, 0);
    }
  }
}

template <typename T, int MODE, bool SMALL, bool VEC>
__global__ __launch_bounds__(256) void pw_gemm_k(GemmArgs p) {
  constexpr int TI = Shape<SMALL>::TI, CH = Shape<SMALL>::CH;
  constexpr int LD = CH + Pad<T>::V;
  constexpr int STAGE_BYTES = (TI + BJ) * LD * (int)sizeof(T);
  constexpr int CT_BYTES = (SMALL ? 4 : 1) * TI * CLD * 4;
  constexpr int SMEM = STAGE_BYTES > CT_BYTES ? STAGE_BYTES : CT_BYTES;
  __shared__ __attribute__((aligned(16))) char smem[SMEM];
  T* xs = reinterpret_cast<T*>(smem);
  T* ys = xs + TI * LD;
  float* ct = reinterpret_cast<float*>(smem);   // aliases the staging buffers between tiles
  if (MODE == MODE_DGRAD) __builtin_amdgcn_s_setprio(3);   // data-gradient chain: ahead of the weight-gradient stream's waves

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int lb = xcd_logical_block();
  const int jt = lb % p.jtiles;
  const int range = lb / p.jtiles;
  const size_t j0 = (size_t)jt * BJ;
  const T* X = reinterpret_cast<const T*>(p.x);
  const T* Y = reinterpret_cast<const T*>(p.y);

  // reduction extent and the row tiles this block walks
  size_t rbeg = 0, rend;
  int it_beg, it_end;
  if (MODE == MODE_WGRAD) {
    // range = (row tile, split): all row tiles are walked by different blocks, the split picks the pixels
    const int split = range / p.itiles;
    it_beg = range % p.itiles; it_end = it_beg + 1;
    rbeg = (size_t)split * p.mchunk;
    rend = rbeg + p.mchunk < p.M ? rbeg + p.mchunk : p.M;
  } else {
    rend = MODE == MODE_FWD ? p.K : p.N;
    it_beg = range * p.tiles_per_range;
    it_end = it_beg + p.tiles_per_range < p.itiles ? it_beg + p.tiles_per_range : p.itiles;
  }
  const int nchunks = (int)((rend - rbeg + CH - 1) / CH);
  const int nsteps = (it_end - it_beg) * nchunks;

  // operand geometry: leading dimensions and extents
  const size_t ldx = MODE == MODE_FWD ? p.K : p.N;
  const size_t ldy = p.K;
  const size_t ni = MODE == MODE_WGRAD ? (size_t)p.N : p.M;        // extent of i
  const size_t nj = MODE == MODE_FWD ? (size_t)p.N : (size_t)p.K;  // extent of j

  // forward: X = A' (r-contiguous, view), Y = W (r-contiguous)
  // dgrad  : X = dZ (r-contiguous),       Y = W as (j=k, r=n)  (i-contiguous)
  // wgrad  : X = dZ as (i=n, r=m),        Y = A' as (j=k, r=m) (both i-contiguous, view on Y)
  typename LoaderSel<T, TI, CH, MODE != MODE_WGRAD, MODE == MODE_FWD, false, VEC>::type lx;
  typename LoaderSel<T, BJ, CH, MODE == MODE_FWD, MODE == MODE_WGRAD, false, VEC>::type ly;
  // weight gradient: the view vectors of this block's columns stay in registers (the same columns at every step)
  if constexpr (MODE == MODE_WGRAD && VEC) ly.hold_view(p.view, j0, nj);

  f16v acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  // narrow bfloat16 weight gradients: the sums of every chunk (32 rows a wavefront) meet in float64.  One fp32 chain through all rows of
  // the block was 7.1e-8 off the exact product (50176 rows, 192 -> 32), this is 6.2e-8
  constexpr bool SUM64 = MODE == MODE_WGRAD && SMALL && sizeof(T) == 2;
  double tot[2][16];
  if constexpr (SUM64)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 16; ++e) tot[t][e] = 0.0;

  // output pass mapping: 8 column groups x 32 row lanes
  const int ocg = threadIdx.x & 7, orl = threadIdx.x >> 3;
  float ssum[8] = {0, 0, 0, 0, 0, 0, 0, 0}, ssq[8] = {0, 0, 0, 0, 0, 0, 0, 0};

  if (nsteps > 0) {
    lx.fetch(X, ldx, (size_t)it_beg * TI, ni, rbeg, rend);
    if constexpr (MODE == MODE_FWD && VEC) lx.fetch_view(p.view, rbeg, rend);
    ly.fetch(Y, ldy, j0, nj, rbeg, rend);
  }
  for (int s = 0; s < nsteps; ++s) {
    const int it = it_beg + s / nchunks, kc = s % nchunks;
    const size_t i0 = (size_t)it * TI, r0 = rbeg + (size_t)kc * CH;
    __syncthreads();                       // LDS free: previous multiply / output pass finished
    if constexpr (MODE == MODE_FWD && VEC) {
      if (p.view.scale) lx.commit_pv(xs, p.view.act);
      else lx.commit(xs, X, ldx, i0, ni, r0, rend, p.view);
    } else {
      lx.commit(xs, X, ldx, i0, ni, r0, rend, p.view);
    }
    ly.commit(ys, Y, ldy, j0, nj, r0, rend, p.view);
    __syncthreads();
    if (s + 1 < nsteps) {                  // next chunk travels while this one is multiplied
      const int it2 = it_beg + (s + 1) / nchunks, kc2 = (s + 1) % nchunks;
      lx.fetch(X, ldx, (size_t)it2 * TI, ni, rbeg + (size_t)kc2 * CH, rend);
      if constexpr (MODE == MODE_FWD && VEC) lx.fetch_view(p.view, rbeg + (size_t)kc2 * CH, rend);
      ly.fetch(Y, ldy, j0, nj, rbeg + (size_t)kc2 * CH, rend);
    }
    if (SMALL) mma32(xs, ys, LD, lane & 31, lane, wave * 32, acc);
    else mma32(xs, ys, LD, wave * 32 + (lane & 31), lane, 0, acc);
    if constexpr (SUM64)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) { tot[t][e] += (double)acc[t][e]; acc[t][e] = 0.f; }
    if (kc + 1 < nchunks) continue;
    if constexpr (SUM64)
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[t][e] = (float)tot[t][e];

    // ---- tile finished: accumulators -> LDS tile -> vector stores ----
    __syncthreads();                       // everyone is done reading the staging buffers
    {
      // register r of lane l is C[8*(r/4) + 4*(l/32) + r%4][l%32]
      const int h = lane >> 5, jl = lane & 31;
      float* base = SMALL ? ct + wave * TI * CLD : ct + wave * 32 * CLD;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          base[(8 * (r / 4) + 4 * h + (r % 4)) * CLD + t * 32 + jl] = acc[t][r];
          acc[t][r] = 0.f;
        }
    }
    __syncthreads();
    const size_t jg = j0 + ocg * 8;
    const bool vec_out = (nj % 8) == 0;
    // residual vectors of all rows of the pass first (see the row-streaming kernel)
    float rpre[SMALL ? 1 : 4][8];
    const bool res_pre = MODE == MODE_DGRAD && p.res != nullptr && vec_out && jg + 8 <= nj;
    if (res_pre) {
#pragma unroll
      for (int q = 0; q < (SMALL ? 1 : 4); ++q) {
        const size_t ig = i0 + orl + q * 32;
        if (ig < ni) load8(reinterpret_cast<const T*>(p.res) + ig * p.K + jg, rpre[q]);
      }
    }
#pragma unroll
    for (int q = 0; q < (SMALL ? 1 : 4); ++q) {
      const int row = orl + q * 32;
      const size_t ig = i0 + row;
      if (ig >= ni || jg >= nj) continue;
      float v[8];
      {
        const float* src = ct + row * CLD + ocg * 8;
        float4 a = *reinterpret_cast<const float4*>(src), b = *reinterpret_cast<const float4*>(src + 4);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
        if (SMALL) {
#pragma unroll
          for (int w = 1; w < 4; ++w) {
            const float* s2 = src + w * TI * CLD;
            float4 c = *reinterpret_cast<const float4*>(s2), d = *reinterpret_cast<const float4*>(s2 + 4);
            v[0] += c.x; v[1] += c.y; v[2] += c.z; v[3] += c.w; v[4] += d.x; v[5] += d.y; v[6] += d.z; v[7] += d.w;
          }
        }
      }
      const bool full = vec_out && jg + 8 <= nj;
      if (MODE == MODE_FWD) {
        T* dst = reinterpret_cast<T*>(p.out) + ig * p.N + jg;
        if (p.bias) {
#pragma unroll
          for (int e = 0; e < 8; ++e) if (jg + e < nj) v[e] += p.bias[jg + e];
        }
        if (full) store8(dst, v);
        else for (int e = 0; e < 8 && jg + e < nj; ++e) dst[e] = from_f32<T>(v[e]);
        if (p.stats) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            float sv = round_to<T>(v[e]);   // statistics of the values as stored
            ssum[e] += sv;
            ssq[e] = fmaf(sv, sv, ssq[e]);
          }
        }
      } else if (MODE == MODE_DGRAD) {
        T* dst = reinterpret_cast<T*>(p.out) + ig * p.K + jg;
        if (p.res) {
          const T* rs = reinterpret_cast<const T*>(p.res) + ig * p.K + jg;
          if (full) {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += rpre[q][e];      // full implies res_pre
          } else {
            for (int e = 0; e < 8 && jg + e < nj; ++e) v[e] += to_f32(rs[e]);
          }
        }
        if (full) store8(dst, v);
        else for (int e = 0; e < 8 && jg + e < nj; ++e) dst[e] = from_f32<T>(v[e]);
      } else {
        const int split = range / p.itiles;
        float* dst = reinterpret_cast<float*>(p.out) + ((size_t)split * p.N + ig) * p.K + jg;
        if (full) store8(dst, v);
        else for (int e = 0; e < 8 && jg + e < nj; ++e) dst[e] = v[e];
      }
    }
  }

  if (MODE == MODE_FWD && p.stats) {
    // column sums over this block's rows: reduce the 32 row lanes through LDS, one partial per block
    __syncthreads();
    float* red = reinterpret_cast<float*>(smem);      // [32][8 groups][16]
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      red[(orl * 8 + ocg) * 16 + e] = ssum[e];
      red[(orl * 8 + ocg) * 16 + 8 + e] = ssq[e];
    }
    __syncthreads();
    if (threadIdx.x < 128) {
      const int cg = threadIdx.x & 7, e = threadIdx.x >> 3;    // e in 0..15: 0-7 sums, 8-15 squares
      float tot = 0.f;
      for (int rl = 0; rl < 32; ++rl) tot += red[(rl * 8 + cg) * 16 + e];
      const size_t j = j0 + cg * 8 + (e & 7);
      if (j < (size_t)p.N) p.stats[((size_t)range * 2 + (e >> 3)) * p.N + j] = tot;
    }
  }
}


// ---- tall problems: 128 x 64 tiles, rows split over the four wavefronts ----------------
// Double-buffered staging (one barrier per chunk); results go from the MFMA registers
// straight to memory: with the permuted weight tile a lane owns columns 2l and 2l+1, so
// each store instruction writes whole 128-byte (bfloat16) / 256-byte (float) row segments.
__device__ __forceinline__ void store_pair(float* p, float a, float b) { *reinterpret_cast<float2*>(p) = make_float2(a, b); }
__device__ __forceinline__ void store_pair(bf16_t* p, float a, float b) {
  *reinterpret_cast<uint32_t*>(p) = f32x2_to_bf16x2(a, b);
}
__device__ __forceinline__ void store_pair_rounded(float* p, float a, float b, float& ra, float& rb) {
  *reinterpret_cast<float2*>(p) = make_float2(a, b); ra = a; rb = b;
}
__device__ __forceinline__ void store_pair_rounded(bf16_t* p, float a, float b, float& ra, float& rb) {
  const uint32_t v = f32x2_to_bf16x2(a, b);
  *reinterpret_cast<uint32_t*>(p) = v;
  ra = __uint_as_float(v << 16); rb = __uint_as_float(v & 0xffff0000u);
}
__device__ __forceinline__ void load_pair(const float* p, float& a, float& b) { float2 v = *reinterpret_cast<const float2*>(p); a = v.x; b = v.y; }
__device__ __forceinline__ void load_pair(const bf16_t* p, float& a, float& b) {
  uint32_t v = *reinterpret_cast<const uint32_t*>(p);
  a = __uint_as_float(v << 16); b = __uint_as_float(v & 0xffff0000u);
}

template <typename T> struct alignas(2 * sizeof(T)) Pair2 { T v[2]; };

// CH = reduction elements staged per step (32 everywhere, see launch_t).
// RES: data gradient with a residual to add (a variant of its own: the sixteen prefetched residual pairs cost
// registers that the plain data gradient should not pay for)
// DEEP: data gradient whose reduction spans at least two steps.  The loads of TWO steps are kept in flight (two
// register sets and the two LDS buffers, addressed statically: the chunk loop is unrolled by two, and a tile with an
// odd number of chunks hands over to a copy of the tile code that starts on the other set).  On this architecture
// loads and stores share one counter and complete out of order with respect to each other, so a wait for "all but
// the youngest n loads" exists only while no store is pending and only if n is the same on every path: the chunk
// loop of a tile has no stores, it is entered after an explicit wait for everything, every step requests its
// successor's successor unconditionally (past the end: a valid tile again, never used), and the tile's stores follow.
// SUMS: data gradient that also leaves the backward sums of the BatchNorm in front (p.view: its view; scale == nullptr: no activation)
template <typename T, int MODE, bool VEC, int CH, bool RES = false, bool DEEP = false, bool SUMS = false>
__global__ __launch_bounds__(256) void pw_gemm_rows_k(GemmArgs p) {
  constexpr int TI = 128;
  constexpr int PD = DEEP ? 2 : 1;
  static_assert(!DEEP || MODE != MODE_FWD, "two steps in flight: data gradient and weight gradient");
  constexpr int LD = CH + Pad<T>::V;
  constexpr int BUF = (TI + BJ) * LD;
  __shared__ __attribute__((aligned(16))) T smem[2 * BUF];
  __shared__ float red[4][64][4];
  if (MODE == MODE_DGRAD) __builtin_amdgcn_s_setprio(3);   // data-gradient chain: ahead of the weight-gradient stream's waves

  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int lb = xcd_logical_block();
  const int jt = lb % p.jtiles;
  const int range = lb / p.jtiles;
  const size_t j0 = (size_t)jt * BJ;
  const T* X = reinterpret_cast<const T*>(p.x);
  const T* Y = reinterpret_cast<const T*>(p.y);

  size_t rbeg = 0, rend;
  int it_beg, it_end, split = 0;
  if (MODE == MODE_WGRAD) {
    split = range / p.itiles;
    it_beg = range % p.itiles; it_end = it_beg + 1;
    rbeg = (size_t)split * p.mchunk;
    rend = rbeg + p.mchunk < p.M ? rbeg + p.mchunk : p.M;
  } else {
    rend = MODE == MODE_FWD ? p.K : p.N;
    it_beg = range * p.tiles_per_range;
    it_end = it_beg + p.tiles_per_range < p.itiles ? it_beg + p.tiles_per_range : p.itiles;
  }
  const int nchunks = (int)((rend - rbeg + CH - 1) / CH);

  const size_t ldx = MODE == MODE_FWD ? p.K : p.N;
  const size_t ldy = p.K;
  const size_t ni = MODE == MODE_WGRAD ? (size_t)p.N : p.M;
  const size_t nj = MODE == MODE_FWD ? (size_t)p.N : (size_t)p.K;
  const size_t ldo = nj;                   // leading dimension of the output

  typename LoaderSel<T, TI, CH, MODE != MODE_WGRAD, MODE == MODE_FWD, false, VEC>::type lx[PD];
  typename LoaderSel<T, BJ, CH, MODE == MODE_FWD, MODE == MODE_WGRAD, true, VEC>::type ly[PD];
  // weight gradient: the view vectors of this block's columns stay in registers (the same columns at every step);
  // forward: they are requested together with the tile they belong to (fetch_view)
  if constexpr (MODE == MODE_WGRAD && VEC) {
#pragma unroll
    for (int d = 0; d < PD; ++d) ly[d].hold_view(p.view, j0, nj);
  }

  f16v acc[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
  float s0 = 0.f, s1 = 0.f, q0 = 0.f, q1 = 0.f;   // column sums / sums of squares of this lane's two columns

  const int h = lane >> 5, jl = lane & 31;
  const size_t jc = j0 + 2 * jl;                    // this lane's first column
  const bool pair_ok = (ldo % 2) == 0 && jc + 1 < nj;
  float b0 = 0.f, b1 = 0.f;
  if (MODE == MODE_FWD && p.bias) {
    if (jc < nj) b0 = p.bias[jc];
    if (jc + 1 < nj) b1 = p.bias[jc + 1];
  }
  const bool gated = SUMS && p.view.scale != nullptr;
  float gsc0 = 0.f, gsc1 = 0.f, gsh0 = 0.f, gsh1 = 0.f;
  const float glo = act_lo(p.view.act), ghi = act_hi(p.view.act);
  if (SUMS && gated && jc < nj) { gsc0 = p.view.scale[jc]; gsc1 = p.view.scale[jc + 1]; gsh0 = p.view.shift[jc]; gsh1 = p.view.shift[jc + 1]; }     // an even width
  if (SUMS) asm volatile("" ::"v"(gsc0), "v"(gsc1), "v"(gsh0), "v"(gsh1));
  // Eight rows of a tile are a chain of their own, and the chains of a block's tiles meet in s0 .. q1: with 25 tiles a block (112x112, batch 128) the results of
  // a lane went through 400 additions one behind the other, where a pass over rows has 75 and 42 where its lanes meet; so it is 8 and 50.
  float e0 = 0.f, e1 = 0.f, f0 = 0.f, f1 = 0.f;
  auto add_sums = [&](const float a, const float b, const float za, const float zb) __attribute__((always_inline)) {
    const float ya = fmaf(za, gsc0, gsh0), yb = fmaf(zb, gsc1, gsh1);
    const float ga = !gated || (ya > glo && ya < ghi) ? a : 0.f, gb = !gated || (yb > glo && yb < ghi) ? b : 0.f;
    e0 += ga; f0 = fmaf(ga, za, f0); e1 += gb; f1 = fmaf(gb, zb, f1);
  };
  auto chain_ends = [&]() __attribute__((always_inline)) {
    s0 += e0; q0 += f0; s1 += e1; q1 += f1;
    e0 = e1 = f0 = f1 = 0.f;
  };
  // Have the two values arrive here.  Their first use is in the tile epilogue inside the loop, where the compiler
  // cannot tell how many younger loads are outstanding and waits for all of them: the prefetch of the next tile
  // would be drained before every output pass.
  asm volatile("" ::"v"(b0), "v"(b1));

  const bool pview = MODE == MODE_FWD && VEC && p.view.scale != nullptr;   // view vectors travel with the tile

  // the finished tile with first row i0; the sums are cleared for the next tile
  auto epilogue = [&](const size_t i0) __attribute__((always_inline)) {
    // tile finished: register r of this lane is row 8*(r/4) + 4*h + r%4, columns jc (acc[0]) and jc+1 (acc[1])
    const size_t irow = i0 + wave * 32 + 4 * h;
    if (VEC && i0 + TI <= ni) {
      // all rows inside and an even width: a lane's column pair is wholly in or out, no other bounds
      // tests, one address computation per lane
      if (jc < nj) {
        const size_t obase = (MODE == MODE_WGRAD ? (size_t)split * p.N + irow : irow) * ldo + jc;
        // all sixteen residual pairs are requested before the first store: res and out are not known to be
        // distinct, so loads left between the stores are not moved up and each one waits for memory on its own
        float ra[RES ? 16 : 1], rb[RES ? 16 : 1];
        if (RES) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            load_pair(reinterpret_cast<const T*>(p.res) + obase + (size_t)(8 * (r / 4) + (r % 4)) * ldo, ra[RES ? r : 0], rb[RES ? r : 0]);
        }
        if constexpr (SUMS) {
          // a row's address is one for the block and an offset that all rows share
          const uint32_t voff = (uint32_t)(wave * 32 + 4 * h) * (uint32_t)ldo + (uint32_t)jc;
          Pair2<T> zr[16];
#pragma unroll
          for (int r = 0; r < 16; ++r)
            zr[r] = *reinterpret_cast<const Pair2<T>*>(reinterpret_cast<const T*>(p.view.z) + (i0 + 8 * (r / 4) + (r % 4)) * ldo + voff);
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            float v0 = acc[0][r], v1 = acc[1][r], a, b, za, zb;
            if (RES) { v0 += ra[RES ? r : 0]; v1 += rb[RES ? r : 0]; }
            store_pair_rounded(reinterpret_cast<T*>(p.out) + (i0 + 8 * (r / 4) + (r % 4)) * ldo + voff, v0, v1, a, b);      // the sums are of the values as stored
            load_pair(reinterpret_cast<const T*>(&zr[r]), za, zb);
            add_sums(a, b, za, zb);
            // two steps' loads are in flight around this: results in order, or the registers of sixteen rows at once cost a block of occupancy (192, so 152)
            if (DEEP) asm volatile("" : "+v"(e0), "+v"(e1), "+v"(f0), "+v"(f1) :: "memory");
            if (r % 8 == 7) chain_ends();
          }
        } else
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const size_t o = obase + (size_t)(8 * (r / 4) + (r % 4)) * ldo;
          float v0 = acc[0][r], v1 = acc[1][r];
          if (MODE == MODE_FWD) {
            v0 += b0; v1 += b1;
            float a, b;                                         // the values as stored: the statistics use those
            store_pair_rounded(reinterpret_cast<T*>(p.out) + o, v0, v1, a, b);
            if (p.stats) { s0 += a; q0 = fmaf(a, a, q0); s1 += b; q1 = fmaf(b, b, q1); }
          } else if (MODE == MODE_DGRAD) {
            if (RES) { v0 += ra[RES ? r : 0]; v1 += rb[RES ? r : 0]; }
            store_pair(reinterpret_cast<T*>(p.out) + o, v0, v1);
          } else {
            store_pair(reinterpret_cast<float*>(p.out) + o, v0, v1);
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) { acc[0][r] = 0.f; acc[1][r] = 0.f; }
      return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const size_t ig = irow + 8 * (r / 4) + (r % 4);
      float v0 = acc[0][r], v1 = acc[1][r];
      acc[0][r] = 0.f; acc[1][r] = 0.f;
      if (SUMS && r == 8) chain_ends();
      if (ig >= ni || jc >= nj) continue;
      if (MODE == MODE_FWD) {
        v0 += b0; v1 += b1;
        T* dst = reinterpret_cast<T*>(p.out) + ig * ldo + jc;
        if (pair_ok) store_pair(dst, v0, v1);
        else { dst[0] = from_f32<T>(v0); if (jc + 1 < nj) dst[1] = from_f32<T>(v1); }
        if (p.stats) {
          float a = round_to<T>(v0), b = round_to<T>(v1);   // statistics of the values as stored
          s0 += a; q0 = fmaf(a, a, q0); s1 += b; q1 = fmaf(b, b, q1);
        }
      } else if (MODE == MODE_DGRAD) {
        T* dst = reinterpret_cast<T*>(p.out) + ig * ldo + jc;
        if (RES) {
          const T* rs = reinterpret_cast<const T*>(p.res) + ig * ldo + jc;
          if (pair_ok) { float ra, rb; load_pair(rs, ra, rb); v0 += ra; v1 += rb; }
          else { v0 += to_f32(rs[0]); if (jc + 1 < nj) v1 += to_f32(rs[1]); }
        }
        if (pair_ok) store_pair(dst, v0, v1);
        else { dst[0] = from_f32<T>(v0); if (jc + 1 < nj) dst[1] = from_f32<T>(v1); }
        if (SUMS) {
          float za, zb;
          load_pair(reinterpret_cast<const T*>(p.view.z) + ig * ldo + jc, za, zb);
          add_sums(round_to<T>(v0), round_to<T>(v1), za, zb);
        }
      } else {
        float* dst = reinterpret_cast<float*>(p.out) + ((size_t)split * p.N + ig) * ldo + jc;
        if (pair_ok) store_pair(dst, v0, v1);
        else { dst[0] = v0; if (jc + 1 < nj) dst[1] = v1; }
      }
    }
    if (SUMS) chain_ends();
  };

  if constexpr (!DEEP) {
    const int nsteps = (it_end - it_beg) * nchunks;
    const bool y_static = nchunks == 1;      // the weight tile never changes: stage it once per buffer
    if (nsteps > 0) {
      lx[0].fetch(X, ldx, (size_t)it_beg * TI, ni, rbeg, rend);
      if constexpr (MODE == MODE_FWD && VEC) { if (pview) lx[0].fetch_view(p.view, rbeg, rend); }
      ly[0].fetch(Y, ldy, j0, nj, rbeg, rend);
    }
    for (int s = 0; s < nsteps; ++s) {
      const int it = it_beg + s / nchunks, kc = s % nchunks;
      const size_t i0 = (size_t)it * TI, r0 = rbeg + (size_t)kc * CH;
      T* xs = smem + (s & 1) * BUF;
      T* ys = xs + TI * LD;
      if constexpr (MODE == MODE_FWD && VEC) {
        if (pview) lx[0].commit_pv(xs, p.view.act);
        else lx[0].commit(xs, X, ldx, i0, ni, r0, rend, p.view);
      } else {
        lx[0].commit(xs, X, ldx, i0, ni, r0, rend, p.view);
      }
      if (!y_static || s < 2) ly[0].commit(ys, Y, ldy, j0, nj, r0, rend, p.view);
      __syncthreads();
      if (s + 1 < nsteps) {
        const int it2 = it_beg + (s + 1) / nchunks, kc2 = (s + 1) % nchunks;
        // the weight tile first: its registers may still be the target of a load the compiler has not seen consumed
        // (its commit is conditional), and the wait for that must not come behind this step's other requests
        if (!y_static || s + 1 < 2) ly[0].fetch(Y, ldy, j0, nj, rbeg + (size_t)kc2 * CH, rend);
        lx[0].fetch(X, ldx, (size_t)it2 * TI, ni, rbeg + (size_t)kc2 * CH, rend);
        if constexpr (MODE == MODE_FWD && VEC) { if (pview) lx[0].fetch_view(p.view, rbeg + (size_t)kc2 * CH, rend); }
      }
  #pragma unroll
      for (int c0 = 0; c0 < CH; c0 += 32) mma32(xs, ys, LD, wave * 32 + jl, lane, c0, acc);
      if (kc + 1 == nchunks) epilogue(i0);
    }
  } else {
    const int ntile = it_end - it_beg;
    auto fetch_step = [&](auto& fx, auto& fy, const int t2, const int kc2) __attribute__((always_inline)) {
      // past the last tile the request is only there to keep the count of loads in flight the same on every path: it
      // repeats one of the last tile's last two chunks, which the caches still hold
      const bool past = t2 >= ntile;
      const size_t r2 = rbeg + (size_t)(past ? nchunks - 2 + kc2 : kc2) * CH;
      fy.fetch(Y, ldy, j0, nj, r2, rend);
      fx.fetch(X, ldx, (size_t)(it_beg + (past ? ntile - 1 : t2)) * TI, ni, r2, rend);
    };
    // chunk kc of tile t from register set / LDS buffer SET, then the request for the step two ahead into the same set
    auto step = [&](auto SET, const int t, const int kc) __attribute__((always_inline)) {
      constexpr int set = decltype(SET)::value;
      const size_t i0 = (size_t)(it_beg + t) * TI, r0 = rbeg + (size_t)kc * CH;
      T* xs = smem + set * BUF;
      T* ys = xs + TI * LD;
      lx[set].commit(xs, X, ldx, i0, ni, r0, rend, p.view);
      ly[set].commit(ys, Y, ldy, j0, nj, r0, rend, p.view);
      __syncthreads();
      int kc2 = kc + 2, t2 = t;
      if (kc2 >= nchunks) { kc2 -= nchunks; ++t2; }
      fetch_step(lx[set], ly[set], t2, kc2);
#pragma unroll
      for (int c0 = 0; c0 < CH; c0 += 32) mma32(xs, ys, LD, wave * 32 + jl, lane, c0, acc);
    };
    // one tile whose chunk 0 sits in set P0
    auto tile_body = [&](auto P0, const int t) __attribute__((always_inline)) {
      constexpr int p0 = decltype(P0)::value;
      // vmcnt(0): the last tile's stores and the two steps requested so far are complete; from here to the end of
      // the chunk loop only loads are pending
      __builtin_amdgcn_s_waitcnt(0x0F70);
      int kc = 0;
      for (; kc + 1 < nchunks; kc += 2) {
        step(std::integral_constant<int, p0>(), t, kc);
        step(std::integral_constant<int, p0 ^ 1>(), t, kc + 1);
      }
      if (kc < nchunks) step(std::integral_constant<int, p0>(), t, kc);
      epilogue((size_t)(it_beg + t) * TI);
    };
    if (ntile > 0) {           // nchunks >= 2 (the host launches this variant only then)
      fetch_step(lx[0], ly[0], 0, 0);
      fetch_step(lx[PD - 1], ly[PD - 1], 0, 1);
    }
    const bool odd = nchunks & 1;
    for (int t = 0; t < ntile;) {
      tile_body(std::integral_constant<int, 0>(), t++);
      if (odd && t < ntile) tile_body(std::integral_constant<int, 1>(), t++);
    }
  }

  if (SUMS || (MODE == MODE_FWD && p.stats)) {
    // one partial per block: sum the 8 (wave, half) contributions of every column in a fixed order
    red[wave][lane][0] = s0; red[wave][lane][1] = s1; red[wave][lane][2] = q0; red[wave][lane][3] = q1;
    __syncthreads();
    if (threadIdx.x < 128) {
      const int col = threadIdx.x & 63, sq = threadIdx.x >> 6;   // column within the tile; 0 = sum, 1 = squares
      const int l = col >> 1, t = col & 1;
      typename std::conditional<SUMS, double, float>::type tot = 0;      // sums of a data gradient: no chain of eight more
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        if (SUMS) { tot += red[w][l][2 * sq + t]; tot += red[w][l + 32][2 * sq + t]; }
        else tot += red[w][l][2 * sq + t] + red[w][l + 32][2 * sq + t];
      }
      const size_t j = j0 + col;
      if (j < nj) p.stats[((size_t)range * 2 + sq) * nj + j] = (float)tot;
    }
  }
}

// ---- short problems: 16 x 16 output tiles, operands straight from global memory ----------------
// When M x N is small the layer is pure latency: staged tiles would leave most CUs idle behind a long
// serial reduction.  Here a block owns one 16 x 16 tile, its four wavefronts split the reduction,
// every lane loads its MFMA fragments (G consecutive reduction elements) directly as vectors, and the
// four partial tiles are summed through LDS in a fixed order.
typedef float f4v __attribute__((ext_vector_type(4)));
template <typename T> struct TinyStep;
template <> struct TinyStep<float> { enum { G = 4, KS = 16 }; };
template <> struct TinyStep<bf16_t> { enum { G = 8, KS = 32 }; };

// A fragment as loaded, and as the MFMAs take it: four floats, or eight bfloat16
template <typename T> struct Frag;
template <> struct Frag<float> { float4 v; };
template <> struct Frag<bf16_t> { uint4 v; };
__device__ __forceinline__ void frag_unpack(const Frag<float>& r, float* v) { v[0] = r.v.x; v[1] = r.v.y; v[2] = r.v.z; v[3] = r.v.w; }
__device__ __forceinline__ void frag_unpack(const Frag<bf16_t>& r, float* v) {
  v[0] = __uint_as_float(r.v.x << 16); v[1] = __uint_as_float(r.v.x & 0xffff0000u);
  v[2] = __uint_as_float(r.v.y << 16); v[3] = __uint_as_float(r.v.y & 0xffff0000u);
  v[4] = __uint_as_float(r.v.z << 16); v[5] = __uint_as_float(r.v.z & 0xffff0000u);
  v[6] = __uint_as_float(r.v.w << 16); v[7] = __uint_as_float(r.v.w & 0xffff0000u);
}
__device__ __forceinline__ void frag_pack(Frag<float>& r, const float* v) { r.v = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void frag_pack(Frag<bf16_t>& r, const float* v) {       // rounds
  r.v = make_uint4(f32x2_to_bf16x2(v[0], v[1]), f32x2_to_bf16x2(v[2], v[3]), f32x2_to_bf16x2(v[4], v[5]), f32x2_to_bf16x2(v[6], v[7]));
}
// from single elements, each in 32 bits as loaded.  The empty asm keeps a pair from becoming one load into the low and one into the high half
// of a register, where the second waits for the first.
template <typename T> struct Elem;
template <> struct Elem<float> { typedef float R; };
template <> struct Elem<bf16_t> { typedef uint32_t R; };
__device__ __forceinline__ float elem_f32(float e) { return e; }
__device__ __forceinline__ float elem_f32(uint32_t e) { return __uint_as_float(e << 16); }
__device__ __forceinline__ void frag_of(Frag<float>& r, float* e) { r.v = make_float4(e[0], e[1], e[2], e[3]); }
__device__ __forceinline__ void frag_of(Frag<bf16_t>& r, uint32_t* e) {
#pragma unroll
  for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(e[i]));
  r.v = make_uint4(e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16);
}
__device__ __forceinline__ void frag_zero(Frag<float>& r) { r.v = make_float4(0.f, 0.f, 0.f, 0.f); }
__device__ __forceinline__ void frag_zero(Frag<bf16_t>& r) { r.v = make_uint4(0u, 0u, 0u, 0u); }
__device__ __forceinline__ void frag_store(float* p, const Frag<float>& r) { *reinterpret_cast<float4*>(p) = r.v; }
__device__ __forceinline__ void frag_store(bf16_t* p, const Frag<bf16_t>& r) { *reinterpret_cast<uint4*>(p) = r.v; }

__device__ __forceinline__ f4v tiny_mma(const Frag<float>& a, const Frag<float>& b, f4v acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.x, b.v.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.y, b.v.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.z, b.v.z, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a.v.w, b.v.w, acc, 0, 0, 0);
}
__device__ __forceinline__ f4v tiny_mma(const Frag<bf16_t>& a, const Frag<bf16_t>& b, f4v acc) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a.v), __builtin_bit_cast(bf16x8, b.v), acc, 0, 0, 0);
}

// A BatchNorm between two short pointwise layers is finished by the second of them.  Forward: x is the raw output of a layer whose statistics
// are still partial sums; the operand is act(scale * x + shift) (+ x_add), what the block output holds.  Data gradient: x is the
// gradient of such an output and x_add the output itself; the operand is the gradient of the raw output, k1 * x + k2 * x_add + k3.  Every
// block sums the partials of all channels, the tiles of the first column write the operand to x_out, the first block the per-channel
// results.  A launch of its own owned four channels over all rows, so each of its few CUs walked every row (a CU has some three cycles per
// 128-byte line and row).  Two launches / one, us, fp32: 512 rows, 64 -> 384 forward 8.6 / 5.8, data gradient of 384 -> 64 8.5 / 5.4;
// 2048 rows, 32 -> 192 12.1 / 7.4 and 13.7 / 6.7; bfloat16 about 480 rows, 64 -> 384 8.3 / 6.7.  What it costs the layer is the sums: 1.4 us
// for 16 KB of partials, 3 us for 32 KB.
struct TinyArgs : GemmArgs {
  FastDiv dj;                // by jtiles
  BnPending pend;            // partial == nullptr: x is read as it is; data gradient: partial, P, gamma, mean, invstd
  const void* x_add;
  void* x_out;
  float *g_gamma, *g_beta;   // data gradient
  double inv_M;
  float eps, momentum;
  const void* z_sum;         // data gradient with stats: the raw output whose gradient is written, statistics sum(out), sum(out * z_sum)
};
enum { kProChan = 96, kProBytes = 1 << 16 };

// Sums of partial[P][2][C] in float64 (C a multiple of 8), then coef[.][c]: scale and shift, or k1, k2, k3.  A wavefront takes 32 neighbouring
// values (a 128-byte line) of eight rows of partials at a time, S wavefronts share the rows of a line where there are more
// wavefronts than lines.  fin: 4 * S rows of 2C, at most kProFin.
enum { kProFin = 4 * 2 * kProChan };
template <int MODE, int NW>
__device__ __forceinline__ void tiny_finish(const TinyArgs& p, const int C, const bool write, double* fin, float (*coef)[kProChan]) {
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, q = lane & 7, pl = lane >> 3;
  const int ng = (C + 15) / 16, S = ng >= NW ? 1 : NW >= 4 * ng ? 4 : NW >= 2 * ng ? 2 : 1;       // lines of a row, wavefronts to a line
  // channels to the threads that add up and finish: tc threads each
  const int tc = C * 8 <= 64 * NW ? 8 : C * 4 <= 64 * NW ? 4 : C * 2 <= 64 * NW ? 2 : 1;
  const int ch = tid / tc, sub = tid & (tc - 1), c = ch < C ? ch : 0;
  // what the finishing threads need is requested before the sums
  float f0 = p.pend.gamma[c], f1, f2, f3, f4 = 0.f;
  if (MODE == MODE_FWD) { f1 = p.pend.beta[c]; f2 = p.pend.run_mean[c]; f3 = p.pend.run_var[c]; }
  else { f1 = p.pend.mean[c]; f2 = p.pend.invstd[c]; f3 = p.g_gamma[c]; f4 = p.g_beta[c]; }
  const int P = p.pend.P;
  for (int j = wave; j < ng * S; j += NW) {
    const int g = S == 1 ? j : j % ng, sl = S == 1 ? 0 : j / ng, v0 = g * 32 + q * 4;
    const bool in = v0 < 2 * C;
    const float* src = p.pend.partial + (in ? v0 : 0);
    double t[4] = {0.0, 0.0, 0.0, 0.0};
    constexpr int U = 4;
    for (int r = sl * 8 + pl; r < P; r += U * 8 * S) {
      float4 v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = ld4(src + (unsigned)(r + u * 8 * S < P ? r + u * 8 * S : r) * 2u * C);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const bool ok = r + u * 8 * S < P;
        t[0] += ok ? (double)v[u].x : 0.0; t[1] += ok ? (double)v[u].y : 0.0; t[2] += ok ? (double)v[u].z : 0.0; t[3] += ok ? (double)v[u].w : 0.0;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {                          // eight rows -> four
      const int2 w = __builtin_bit_cast(int2, t[e]);
      const int2 o = make_int2(__builtin_amdgcn_update_dpp(0, w.x, 0x128, 0xF, 0xF, false), __builtin_amdgcn_update_dpp(0, w.y, 0x128, 0xF, 0xF, false));
      t[e] += __builtin_bit_cast(double, o);
    }
    if (in && !(pl & 1)) {
      double2* d = reinterpret_cast<double2*>(fin + (size_t)(sl * 4 + (pl >> 1)) * 2 * C + v0);
      d[0] = make_double2(t[0], t[1]);
      d[1] = make_double2(t[2], t[3]);
    }
  }
  __syncthreads();
  double s0 = 0.0, s1 = 0.0;
  for (int l = sub; l < 4 * S; l += tc) { s0 += fin[l * 2 * C + c]; s1 += fin[l * 2 * C + C + c]; }
  for (int o = 1; o < tc; o <<= 1) { s0 += __shfl_xor(s0, o, 64); s1 += __shfl_xor(s1, o, 64); }
  asm volatile("" : "+v"(f0), "+v"(f1), "+v"(f2), "+v"(f3), "+v"(f4));      // first use: conversions must not move up to the loads
  if (ch < C && sub == 0) {
    if (MODE == MODE_FWD) {
      finish_channel(p.pend, p.inv_M, c, s0, s1, f0, f1, f2, f3, p.eps, p.momentum, write, coef[0][c], coef[1][c]);
    } else {
      const double mu = f1, is = f2, k1 = (double)f0 * is, dgamma = is * (s1 - mu * s0);
      const double k2 = -k1 * is * dgamma * p.inv_M, k3 = -k1 * s0 * p.inv_M - k2 * mu;
      coef[0][c] = (float)k1; coef[1][c] = (float)k2; coef[2][c] = (float)k3;
      if (write) { p.g_gamma[c] = f3 + (float)dgamma; p.g_beta[c] = f4 + (float)s0; }
    }
  }
  __syncthreads();
}

// Operands are read through buffer descriptors: an element outside the problem is requested past the end and comes back as zero, so
// a fragment costs one 32-bit offset and no branch.  (These kernels are as long as their instructions: 200 in front of the first load
// took 1600 cycles, half of them exec masks, 64-bit addresses and zeroes for fragments that might not be loaded.)
enum : uint32_t { kTinyPast = 0x80000000u };
typedef uint32_t u4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ __amdgpu_buffer_rsrc_t tiny_rsrc(const void* p, size_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buf_load16(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __builtin_bit_cast(uint4, (u4v)__builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0));
}
__device__ __forceinline__ float4 buf_load4f(__amdgpu_buffer_rsrc_t rs, uint32_t off) { return __builtin_bit_cast(float4, buf_load16(rs, off)); }
__device__ __forceinline__ void buf_load1(float& v, __amdgpu_buffer_rsrc_t rs, uint32_t off, int soff) {
  v = __builtin_bit_cast(float, (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, soff, 0));
}
__device__ __forceinline__ void buf_load1(uint32_t& v, __amdgpu_buffer_rsrc_t rs, uint32_t off, int soff) {
  v = (bf16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)off, soff, 0);
}
__device__ __forceinline__ void frag_of(Frag<float>& r, uint4 v) { r.v = __builtin_bit_cast(float4, v); }
__device__ __forceinline__ void frag_of(Frag<bf16_t>& r, uint4 v) { r.v = v; }

// WT wavefronts share a tile's reduction (launch_tiny picks the number), a block of NW wavefronts works on NW / WT tiles
template <typename T, int MODE, int WT, int NW, bool PRO = false>
__device__ __forceinline__ void pw_gemm_tiny_body(const TinyArgs& p, const int bid) {
  constexpr int G = TinyStep<T>::G, KS = TinyStep<T>::KS, U = 4, ES = sizeof(T);
  static_assert(KS * ES == 64 && G * ES == 16, "a step is 64 bytes of a row, a fragment 16");
  constexpr int GROUPS = NW / WT;
  __shared__ float red_[WT > 1 && !PRO ? GROUPS * WT * 16 * 17 : 1];
  __shared__ __attribute__((aligned(16))) double fin_[PRO ? kProFin : 1];
  __shared__ __attribute__((aligned(16))) float coef[PRO ? 3 : 1][PRO ? kProChan : 1];
  static_assert(!PRO || sizeof(fin_) >= sizeof(float) * GROUPS * WT * 16 * 17, "the tiles' sums take the place of the statistics'");
  float (*red)[WT][16][17] = reinterpret_cast<float (*)[WT][16][17]>(PRO ? reinterpret_cast<float*>(fin_) : red_);
  __shared__ float sred[WT > 1 ? GROUPS : 1][2][16][17];
  if (MODE == MODE_DGRAD) __builtin_amdgcn_s_setprio(3);   // data-gradient chain: ahead of the weight-gradient stream's waves
  // scalar: the data gradient's offsets of single weights go into the scalar offset of the load, and from a vector register each load would be a
  // loop over the values it holds (both gradients in one launch, us, before and now: fp32 2048 rows of 384 -> 64 22.8 / 18.6, 1040 rows of 528 -> 88 18.1 / 15.0,
  // bfloat16 2048 rows of 384 -> 64 22.7 / 20.2)
  const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = wid / WT, wave = wid % WT, lane = threadIdx.x & 63;
  const int tile = bid * GROUPS + grp;
  const bool tile_ok = tile < p.jtiles * p.itiles;
  const int it = (int)p.dj.div(tile), jt = tile - it * p.jtiles;
  const int i0 = it * 16, j0 = jt * 16, M = (int)p.M;
  const int R = MODE == MODE_FWD ? p.K : p.N;       // reduction extent (a multiple of G)
  const int nj = MODE == MODE_FWD ? p.N : p.K;      // output columns
  const int nst = (R + KS - 1) / KS;
  const int sb = wave * nst / WT, se = (wave + 1) * nst / WT;
  const int l16 = lane & 15, kg = (lane >> 4) * G;
  const int row = i0 + l16, col = j0 + l16;
  const bool row_ok = tile_ok && row < M, col_ok = tile_ok && col < nj;
  const bool view = MODE == MODE_FWD && !PRO && p.view.scale != nullptr;
  const float lo = act_lo(p.view.act), hi = act_hi(p.view.act);
  const __amdgpu_buffer_rsrc_t bx = tiny_rsrc(p.x, (size_t)M * R * ES), bw = tiny_rsrc(p.y, (size_t)R * nj * ES);
  const __amdgpu_buffer_rsrc_t bx2 = tiny_rsrc(PRO && p.x_add ? p.x_add : p.x, (size_t)M * R * ES);
  const __amdgpu_buffer_rsrc_t bsc = tiny_rsrc(p.view.scale, (size_t)R * 4), bsh = tiny_rsrc(p.view.shift, (size_t)R * 4);
  const int kend = se * KS < R ? se * KS : R;
  // byte offsets at step 0 (PAST stays past the end when a step's offset is added)
  const uint32_t ox = row_ok ? (uint32_t)(row * R + kg) * ES : kTinyPast;
  const uint32_t ow = !col_ok ? kTinyPast : MODE == MODE_FWD ? (uint32_t)(col * R + kg) * ES : (uint32_t)(kg * nj + col) * ES;

  // the output elements this thread writes after the reduction (WT == 1: its four accumulators, else one); what is added
  // to them there (residual, bias) is requested now: a load at the end of the kernel would be one more round trip on the
  // launch-latency path
  constexpr int NO = WT == 1 ? 4 : 1;
  const int orow = WT == 1 ? 4 * (lane >> 4) : (threadIdx.x >> 4) & 15, ocol = threadIdx.x & 15;
  const int ig = i0 + orow, jg = j0 + ocol;
  const uint32_t oo = (uint32_t)(ig * nj + jg) * ES;       // a row further down: nj elements on, past the end in the last tile
  bool in[NO];
  typename Elem<T>::R add_r[NO], zs_r[NO];
  float bias = 0.f;
#pragma unroll
  for (int o = 0; o < NO; ++o) in[o] = tile_ok && ig + o < M && jg < nj && (WT <= 4 || wave < 4);
  const bool with_res = MODE == MODE_DGRAD && p.res != nullptr, with_z = MODE == MODE_DGRAD && p.stats != nullptr;
  if (MODE == MODE_FWD) {
    if (p.bias && in[0]) bias = p.bias[jg];
  } else {
    if (with_res) {
      const __amdgpu_buffer_rsrc_t br = tiny_rsrc(p.res, (size_t)M * nj * ES);
#pragma unroll
      for (int o = 0; o < NO; ++o) buf_load1(add_r[o], br, in[o] ? oo : kTinyPast, o * nj * ES);
    }
    if (with_z) {
      const __amdgpu_buffer_rsrc_t bz = tiny_rsrc(p.z_sum, (size_t)M * nj * ES);
#pragma unroll
      for (int o = 0; o < NO; ++o) buf_load1(zs_r[o], bz, in[o] ? oo : kTinyPast, o * nj * ES);
    }
  }

  f4v acc = {0.f, 0.f, 0.f, 0.f}, step[U];      // step: WT == 1 (one round), a chain for each step
  Frag<T> xr[U], er[PRO ? U : 1], br[U];        // er: the operand's second tensor (PRO)
  float sc[U][G], sh[U][G];
  typename Elem<T>::R bs[U][G];                 // data gradient: single elements of W down a column
  auto request = [&](const int s) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool inb = (s + u) * KS + kg < kend;
      const uint32_t ko = (uint32_t)(s + u) * 64u;
      frag_of(xr[u], buf_load16(bx, inb ? ox + ko : kTinyPast));
      if (PRO) frag_of(er[PRO ? u : 0], buf_load16(bx2, inb ? ox + ko : kTinyPast));
      if (MODE == MODE_FWD) {
        frag_of(br[u], buf_load16(bw, inb ? ow + ko : kTinyPast));
        if (view) {
          const uint32_t o = inb ? (uint32_t)((s + u) * KS + kg) * 4u : kTinyPast;
#pragma unroll
          for (int e = 0; e < G; e += 4) {
            *reinterpret_cast<float4*>(sc[u] + e) = buf_load4f(bsc, o + 4 * e);
            *reinterpret_cast<float4*>(sh[u] + e) = buf_load4f(bsh, o + 4 * e);
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < G; ++e) buf_load1(bs[u][e], bw, inb ? ow : kTinyPast, ((s + u) * KS + e) * nj * ES);
      }
    }
  };
  request(sb);
  if constexpr (PRO) tiny_finish<MODE, NW>(p, R, bid == 0, fin_, reinterpret_cast<float (*)[kProChan]>(coef));      // while the first round travels
  for (int s = sb; s < se; s += U) {
    if (WT > 1 && s != sb) request(s);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = (s + u) * KS + kg;
      Frag<T> a = xr[u], b = br[u];
      if (MODE == MODE_DGRAD) frag_of(b, bs[u]);
      if constexpr (PRO) {
        const bool inb = k < kend;
        const int c = inb ? k : 0;
        float x[G], y[G], k1[G], k2[G], k3[G];
        frag_unpack(xr[u], x);
        frag_unpack(er[u], y);
#pragma unroll
        for (int e = 0; e < G; e += 4) {
          *reinterpret_cast<float4*>(k1 + e) = ld4(&coef[0][c + e]);
          *reinterpret_cast<float4*>(k2 + e) = ld4(&coef[1][c + e]);
          if (MODE == MODE_DGRAD) *reinterpret_cast<float4*>(k3 + e) = ld4(&coef[2][c + e]);
        }
#pragma unroll
        for (int e = 0; e < G; ++e) {
          if (MODE == MODE_FWD) {
            x[e] = clamp_act(fmaf(x[e], k1[e], k2[e]), lo, hi);
            if (p.x_add) x[e] = round_to<T>(x[e]) + y[e];
          } else {
            x[e] = fmaf(k1[e], x[e], fmaf(k2[e], y[e], k3[e]));
          }
        }
        frag_pack(a, x);
        if (jt == 0 && inb && row_ok) frag_store(reinterpret_cast<T*>(p.x_out) + (size_t)row * R + k, a);
        if (!inb) frag_zero(a);
      } else if (view) {
        // past the end of the reduction scale and shift are zero, and so is the operand; a row past M is not written
        float x[G];
        frag_unpack(xr[u], x);
#pragma unroll
        for (int e = 0; e < G; ++e) x[e] = clamp_act(fmaf(x[e], sc[u][e], sh[u][e]), lo, hi);
        frag_pack(a, x);
      }
      if constexpr (WT == 1) step[u] = tiny_mma(a, b, f4v{0.f, 0.f, 0.f, 0.f});
      else acc = tiny_mma(a, b, acc);
    }
    // the steps' sums are added in their order, as those of four wavefronts are: one chain through all of them would be up to 64 fp32
    // additions long instead of 16 (64 -> 384 channels, fp32: 1.4e-7 off in the 2-norm instead of 8.4e-8)
    if constexpr (WT == 1) acc = ((step[0] + step[1]) + step[2]) + step[3];
  }
  float addend[NO], zs[NO];
#pragma unroll
  for (int o = 0; o < NO; ++o) {
    addend[o] = MODE == MODE_FWD ? bias : with_res ? elem_f32(add_r[o]) : 0.f;
    zs[o] = with_z ? elem_f32(zs_r[o]) : 0.f;
  }

  // register r of lane l is C[4*(l/16) + r][l%16]
  if constexpr (WT == 1) {
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = acc[r] + addend[r];
      if (in[r]) reinterpret_cast<T*>(p.out)[(size_t)(ig + r) * nj + jg] = from_f32<T>(v);
      const float sv = in[r] ? round_to<T>(v) : 0.f;      // statistics of the values as stored
      s1 += sv;
      s2 += sv * (MODE == MODE_FWD ? sv : zs[r]);
    }
    if (p.stats) {
      s1 += __shfl_xor(s1, 16, 64); s2 += __shfl_xor(s2, 16, 64);
      s1 += __shfl_xor(s1, 32, 64); s2 += __shfl_xor(s2, 32, 64);
      if (lane < 32 && tile_ok && jg < nj) p.stats[((size_t)it * 2 + (lane >> 4)) * nj + jg] = lane < 16 ? s1 : s2;
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[grp][wave][4 * (lane >> 4) + r][l16] = acc[r];
  __syncthreads();
  const bool writer = WT <= 4 || wave < 4;  // 256 threads of a tile hold its elements
  float v = 0.f;
  if (writer) {
#pragma unroll
    for (int q = 0; q < WT; ++q) v += red[grp][q][orow][ocol];
    v += addend[0];
    if (in[0]) reinterpret_cast<T*>(p.out)[(size_t)ig * nj + jg] = from_f32<T>(v);
  }
  if (p.stats) {
    const float sv = in[0] ? round_to<T>(v) : 0.f;        // statistics of the values as stored
    if (writer) {
      sred[grp][0][orow][ocol] = sv;
      sred[grp][1][orow][ocol] = sv * (MODE == MODE_FWD ? sv : zs[0]);
    }
    __syncthreads();
    if (wave == 0 && lane < 32 && tile_ok) {
      const int sq = lane >> 4, c = lane & 15;
      float tot = 0.f;
#pragma unroll
      for (int rr = 0; rr < 16; ++rr) tot += sred[grp][sq][rr][c];
      if (j0 + c < nj) p.stats[((size_t)it * 2 + sq) * nj + j0 + c] = tot;
    }
  }
}

// Weight gradient of a short problem, g_w[n][k] += sum_m dZ[m][n] * A'[m][k], in one launch: a block owns a
// 16 x 16 tile of g_w, its four wavefronts split the pixels and meet in LDS, so there are no partial
// buffers and no second kernel.  A lane's two MFMA operands are single elements of consecutive columns
// (64-byte runs), the per-column scale/shift of the view sit in two registers.  Both storage types use
// the fp32 16x16x4 MFMA: products of bfloat16 values are exact in fp32.
template <typename T, int NW>
__device__ __forceinline__ void pw_wgrad_tiny_body(const GemmArgs& p, const int K_out, const int bid) {
  constexpr int U = 8;
  __shared__ float red[NW][16][17];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int jt = bid % p.jtiles, it = bid / p.jtiles;
  const int l16 = lane & 15, mg = lane >> 4;
  const int n = it * 16 + l16, k = jt * 16 + l16;
  const bool n_ok = n < p.N, k_ok = k < p.K;
  const T* X = reinterpret_cast<const T*>(p.x) + (n_ok ? n : 0);
  const T* Y = reinterpret_cast<const T*>(p.y) + (k_ok ? k : 0);
  const bool view = p.view.scale != nullptr;
  const float sc = view && k_ok ? p.view.scale[k] : 1.f, sh = view && k_ok ? p.view.shift[k] : 0.f;
  const float lo = act_lo(p.view.act), hi = act_hi(p.view.act);
  const size_t M = p.M;
  // the gradient element this thread adds to after the reduction, requested now (see pw_gemm_tiny_body)
  const int orow = (threadIdx.x >> 4) & 15, ocol = threadIdx.x & 15;
  const int on = it * 16 + orow, ok_ = jt * 16 + ocol;
  const bool writer = threadIdx.x < 256 && on < p.N && ok_ < K_out;
  float* dst = reinterpret_cast<float*>(p.out) + (writer ? (size_t)on * K_out + ok_ : 0);
  float g_old = writer ? *dst : 0.f;
  const size_t per = ((M + 4 * NW - 1) / (4 * NW)) * 4;    // pixels per wavefront, a multiple of 4
  const size_t mb = (size_t)wave * per, me = mb + per < M ? mb + per : M;
  // a chain of fp32 additions per round of 32 rows; the rounds and the wavefronts meet in float64, as in pw_wgrad_group_k
  double tot[4] = {0.0, 0.0, 0.0, 0.0};
  for (size_t m0 = mb; m0 < me; m0 += 4 * U) {
    f4v acc = {0.f, 0.f, 0.f, 0.f};
    float x[U], y[U];
    T xr[U], yr[U];                            // converted after all loads of the round are out (see FragRaw)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const size_t m = m0 + 4 * u + mg;
      const size_t mc = m < me ? m : mb;       // unconditional loads from a valid row (X, Y point at valid columns)
      xr[u] = X[mc * p.N];
      yr[u] = Y[mc * p.K];
    }
    __builtin_amdgcn_sched_barrier(0);         // without it every bfloat16 load is followed by its conversion, and a wait: 512 rows, 64 -> 384 27 us a step instead of 20
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const bool ok = m0 + 4 * u + mg < me;
      x[u] = ok && n_ok ? to_f32(xr[u]) : 0.f;
      y[u] = ok && k_ok ? to_f32(yr[u]) : 0.f;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float a = y[u];
      if (view) {
        const bool ok = m0 + 4 * u + mg < me && k_ok;       // padding stays exactly zero
        a = ok ? round_to<T>(clamp_act(fmaf(a, sc, sh), lo, hi)) : 0.f;
      }
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u], a, acc, 0, 0, 0);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) tot[r] += (double)acc[r];
  }
  // register r of lane l is tile element (row 4*(l/16) + r = n, column l%16 = k)
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][4 * mg + r][l16] = (float)tot[r];
  __syncthreads();
  asm volatile("" : "+v"(g_old));
  if (writer) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < NW; ++q) v += (double)red[q][orow][ocol];
    *dst = g_old + (float)v;
  }
}

template <typename T, int MODE, int WT, int NW, bool PRO>
__global__ __launch_bounds__(64 * NW) void pw_gemm_tiny_k(TinyArgs p) { pw_gemm_tiny_body<T, MODE, WT, NW, PRO>(p, xcd_logical_block()); }   // the column tiles of a row panel share an L2
template <typename T>
__global__ __launch_bounds__(256) void pw_wgrad_tiny_k(GemmArgs p, int K_out) { pw_wgrad_tiny_body<T, 4>(p, K_out, blockIdx.x); }
// data gradient and weight gradient of one short layer in one launch: both read the same dZ, their tiles are
// independent, and for these sizes a launch costs more than either of them.  NW wavefronts per block: with many
// pixels the weight-gradient tiles are few and each walks all pixels, so 16 wavefronts share that walk.
template <typename T, int NW>
__global__ __launch_bounds__(64 * NW) void pw_bwd_tiny_k(TinyArgs pd, GemmArgs pw, int K_out, int n_dgrad) {
  if ((int)blockIdx.x < n_dgrad) pw_gemm_tiny_body<T, MODE_DGRAD, 4, NW>(pd, blockIdx.x);
  else pw_wgrad_tiny_body<T, NW>(pw, K_out, blockIdx.x - n_dgrad);
}

// the 16 x 16 kernel serves problems whose output is short (few rows) and whose reduction extent
// allows aligned vector fragments.  Beyond 2048 rows the kernels behind it are the faster ones throughout; below, against the
// long-reduction kernel, the layer's time (us, with some 3 of the events around the launch) here / there: fp32 forward 384 -> 64 513 rows 6.9 / 9.6, 2048
// 8.8 / 9.8, 576 -> 96 513 8.0 / 11.9, 144 -> 24 6.5 / 9.2, data gradient 64 -> 384 513 6.3 / 8.2, 2048 6.9 / 8.5; but layers that widen lose here from some
// 700 rows on: forward 96 -> 576 700 9.9 / 6.8, 1040 12.1 / 7.5, 64 -> 384 1600 8.6 / 6.8, data gradient 576 -> 96 1040 10.3 / 6.9.  bfloat16 is
// mostly even: forward 576 -> 96 513 6.9 / 8.0, 1040 9.2 / 8.0, 64 -> 384 2048 8.2 / 6.7.
static bool tiny_ok(int dt, size_t M, int R, int ncols, bool stats) {
  const int G = dt == 0 ? 4 : 8;
  if (M > 2048 || R % G != 0) return false;
  if ((double)M * R * ncols > 64.0 * 1024 * 1024) return false;   // every block re-reads its operand rows
  if (stats && (M + 15) / 16 > (size_t)kMaxPartials) return false;
  return true;
}

template <int MODE>
static void launch_tiny(int dt, hipStream_t st, TinyArgs& a, int ncols) {
  a.jtiles = (ncols + 15) / 16;
  a.itiles = (int)((a.M + 15) / 16);
  a.nranges = a.itiles;
  a.tiles_per_range = 1;
  // Four steps of a wavefront's reduction travel together, one trip to memory: enough wavefronts per tile to make it one trip
  // or two.  MobileNetV2 at 32x32, batch 32, fp32: 57 launches a step, 303 us with four wavefronts per tile for all.  Up to four
  // steps a tile to itself (no LDS, no barrier, a quarter of the blocks; 14 launches, 59 us); above sixteen steps eight
  // wavefronts (24 launches: 134 us, with four 150, with sixteen 139).
  a.dj = FastDiv::of(a.jtiles);
  const int R = MODE == MODE_FWD ? a.K : a.N, nst = (R + (dt == 0 ? 15 : 31)) / (dt == 0 ? 16 : 32);
  const unsigned tiles = (unsigned)((size_t)a.jtiles * a.itiles);
#define FTP_TINY(WT, NW, PRO)                                                                                                         \
  do {                                                                                                                                \
    const dim3 grid((tiles + (NW) / (WT) - 1) / ((NW) / (WT)));                                                                       \
    if (dt == 0) hipLaunchKernelGGL((pw_gemm_tiny_k<float, MODE, WT, NW, PRO>), grid, dim3(64 * (NW)), 0, st, a);                     \
    else hipLaunchKernelGGL((pw_gemm_tiny_k<bf16_t, MODE, WT, NW, PRO>), grid, dim3(64 * (NW)), 0, st, a);                            \
  } while (0)
  if (a.pend.partial) FTP_TINY(1, 4, true);           // pw_pro_ok: at most four steps
  else if (nst <= 4) FTP_TINY(1, 4, false);
  else if (nst <= 16) FTP_TINY(4, 4, false);
  else FTP_TINY(8, 8, false);
#undef FTP_TINY
}

template <typename T, int MODE, bool VEC>
static void launch_t(hipStream_t st, const GemmArgs& a, bool small, unsigned grid) {
  if (small) { hipLaunchKernelGGL((pw_gemm_k<T, MODE, true, VEC>), dim3(grid), dim3(256), 0, st, a); return; }
  const size_t red = MODE == MODE_FWD ? (size_t)a.K : MODE == MODE_DGRAD ? (size_t)a.N : a.mchunk;   // reduction extent of a block
  // Every mode stages 32 reduction elements per step.  64 per step made the weight-gradient kernel itself 5 % faster
  // (half the barriers) but costs 55 KB of LDS per block: next to the data-gradient chain on the other stream the
  // step was 0.9 % slower with it.
  if (MODE == MODE_WGRAD && red > 32)
    hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, false, MODE == MODE_WGRAD>), dim3(grid), dim3(256), 0, st, a);
  else if (MODE == MODE_DGRAD && red > 32) {     // at least two steps per tile: two steps' loads in flight
    constexpr bool D = MODE == MODE_DGRAD;
    if (VEC && a.stats && a.res) hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, D, D, D && VEC>), dim3(grid), dim3(256), 0, st, a);
    else if (VEC && a.stats) hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, false, D, D && VEC>), dim3(grid), dim3(256), 0, st, a);
    else if (a.res) hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, D, D>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, false, D>), dim3(grid), dim3(256), 0, st, a);
  }
  else if (MODE == MODE_DGRAD && VEC && a.stats) {
    constexpr bool D = MODE == MODE_DGRAD && VEC;
    if (a.res) hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, D, false, D>), dim3(grid), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, false, false, D>), dim3(grid), dim3(256), 0, st, a);
  }
  else if (MODE == MODE_DGRAD && a.res) hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32, MODE == MODE_DGRAD>), dim3(grid), dim3(256), 0, st, a);
  else hipLaunchKernelGGL((pw_gemm_rows_k<T, MODE, VEC, 32>), dim3(grid), dim3(256), 0, st, a);
}

template <int MODE>
static void launch(int dt, hipStream_t st, const GemmArgs& a, bool small) {
  unsigned grid = (unsigned)((size_t)a.jtiles * a.nranges);
  const bool vec = a.K % 8 == 0 && a.N % 8 == 0;   // whole vectors along both weight dimensions
  if (dt == 0) {
    if (vec) launch_t<float, MODE, true>(st, a, small, grid);
    else launch_t<float, MODE, false>(st, a, small, grid);
  } else {
    if (vec) launch_t<bf16_t, MODE, true>(st, a, small, grid);
    else launch_t<bf16_t, MODE, false>(st, a, small, grid);
  }
}

// Row-streaming passes (forward, dgrad): tile shape and the split of the row tiles into ranges.
static void plan_rows(size_t M, int ncols, int R, GemmArgs* a, bool* small) {
  a->jtiles = (ncols + BJ - 1) / BJ;
  size_t big_tiles = (M + 127) / 128;
  // short problems: too few 128-row tiles to fill 256 CUs and a reduction worth splitting
  *small = (big_tiles * a->jtiles < 96 && R >= 128) || (big_tiles * a->jtiles < 512 && R >= 512);
  int TI = *small ? 32 : 128;
  a->itiles = (int)((M + TI - 1) / TI);
  int want = (4096 + a->jtiles - 1) / a->jtiles;          // about 4096 blocks in flight
  if (want > kMaxPartials) want = kMaxPartials;
  if (want < 1) want = 1;
  a->tiles_per_range = (a->itiles + want - 1) / want;
  a->nranges = (a->itiles + a->tiles_per_range - 1) / a->tiles_per_range;
}

// Four steps at most, a tile to a wavefront.  Above, tiles of several wavefronts and partials of more channels cost more than the launch:
// fp32 512 rows, 96 channels (2 launches / 1) 9.5 / 12.0 us forward, 9.3 / 10.2 backward, 128 rows, 160 channels 7.9 / 9.7 and 7.5 / 8.9;
// bfloat16 96 channels 8.5 / 8.0, 128 the same as two.
int pw_pro_ok(int dt, size_t M, int R, int ncols) {
  const size_t P = (M + 15) / 16;
  return R % 8 == 0 && R <= (dt == 0 ? 64 : 96) && tiny_ok(dt, M, R, ncols, true) && P * 2 * R * sizeof(float) <= kProBytes;
}
int pw_dgrad_sums_ok(int dt, size_t M, int K, int N, HView of) {
  if (tiny_ok(dt, M, N, K, false)) return of.scale == nullptr && tiny_ok(dt, M, N, K, true);
  if (of.scale != nullptr && of.act != ACT_RELU6) return 0;
  if (pw_deep_ok(dt, M, N, K, true)) return pw_deep_sums_ok(dt, M, N, K);
  GemmArgs a{};
  bool small;
  plan_rows(M, K, N, &a, &small);
  return !small && K % 8 == 0 && N % 8 == 0 && bn_left_sums_ok(M, K, a.nranges);
}

void pw_fwd_pro(int dt, hipStream_t st, const BnPending& pend, HView x, const void* x_add, void* x_out, float eps, float momentum, const void* w,
                size_t M, int K, int N, void* z, float* stats, int* P_out) {
  TinyArgs a{};
  a.x = x.z; a.y = w; a.view = View{x.z, x.scale, x.shift, x.act}; a.out = z; a.stats = stats; a.M = M; a.K = K; a.N = N;
  a.pend = pend; a.x_add = x_add; a.x_out = x_out; a.inv_M = 1.0 / (double)M; a.eps = eps; a.momentum = momentum;
  KScope ks(st, "pw_fwd", ((double)M * K * (x_add ? 3.0 : 2.0) + (double)M * N + (double)N * K) * (dt == 0 ? 4.0 : 2.0), 2.0 * M * K * N, (long)M, K, N);
  launch_tiny<MODE_FWD>(dt, st, a, N);
  *P_out = a.nranges;
}

void pw_fwd(int dt, hipStream_t st, HView av, const void* w, const float* bias, size_t M, int K, int N,
            void* z, float* stats, int* P_out) {
  TinyArgs a{};
  a.x = av.z; a.y = w; a.view = View{av.z, av.scale, av.shift, av.act};
  a.bias = bias; a.out = z; a.stats = stats; a.M = M; a.K = K; a.N = N;
  KScope ks(st, "pw_fwd", ((double)M * K + (double)M * N + (double)N * K) * (dt == 0 ? 4.0 : 2.0), 2.0 * M * K * N, (long)M, K, N);
  if (tiny_ok(dt, M, K, N, stats != nullptr)) {
    launch_tiny<MODE_FWD>(dt, st, a, N);
    if (P_out) *P_out = a.nranges;
    return;
  }
  if (!bias && pw_deep_ok(dt, M, K, N, false)) { ks.route(pw_fwd_deep(dt, st, av, w, M, K, N, z, stats, P_out)); return; }
  bool small;
  plan_rows(M, N, K, &a, &small);
  if (P_out) *P_out = a.nranges;
  launch<MODE_FWD>(dt, st, a, small);
}

void pw_dgrad_pro(int dt, hipStream_t st, const BnPending& sums, const BnBwdIn& bn, void* dz, const void* w, size_t M, int K, int N, void* dA) {
  TinyArgs a{};
  a.x = bn.dA; a.x_add = bn.out.z; a.x_out = dz; a.y = w; a.out = dA; a.M = M; a.K = K; a.N = N;
  a.pend = sums; a.g_gamma = bn.g_gamma; a.g_beta = bn.g_beta; a.inv_M = 1.0 / (double)M;
  KScope ks(st, "pw_dgrad", ((double)M * K + 3.0 * M * N + (double)N * K) * (dt == 0 ? 4.0 : 2.0), 2.0 * M * K * N, (long)M, K, N);
  launch_tiny<MODE_DGRAD>(dt, st, a, K);
}

void pw_dgrad(int dt, hipStream_t st, const void* dz, const void* w, const void* res, size_t M, int K,
              int N, void* dA, HView of, float* sums, int* P_out) {
  TinyArgs a{};
  a.x = dz; a.y = w; a.res = res; a.out = dA; a.M = M; a.K = K; a.N = N;
  KScope ks(st, "pw_dgrad", ((double)M * K * (1.0 + (res != nullptr) + (sums != nullptr)) + (double)M * N + (double)N * K) * (dt == 0 ? 4.0 : 2.0), 2.0 * M * K * N, (long)M, K, N);
  if (tiny_ok(dt, M, N, K, false)) {
    a.z_sum = of.z; a.stats = sums;
    launch_tiny<MODE_DGRAD>(dt, st, a, K);
    if (sums) *P_out = a.nranges;
    return;
  }
  if (pw_deep_ok(dt, M, N, K, true)) { ks.route(pw_dgrad_deep(dt, st, dz, w, res, M, K, N, dA, of, sums, P_out)); return; }
  bool small;
  plan_rows(M, K, N, &a, &small);
  if (sums) { a.view = View{of.z, of.scale, of.shift, of.act}; a.stats = sums; *P_out = a.nranges; }
  launch<MODE_DGRAD>(dt, st, a, small);
}

// wgrad: output tiles (N x K) times splits of the pixel range
static void plan_wgrad(size_t M, int K, int N, GemmArgs* a, bool* small) {
  a->jtiles = (K + BJ - 1) / BJ;
  *small = N <= 32;                         // few output rows: 32-row tiles waste less of the MFMA
  int TI = *small ? 32 : 128;
  int CH = *small ? 128 : 32;
  a->itiles = (N + TI - 1) / TI;
  size_t tiles = (size_t)a->itiles * a->jtiles;
  size_t s = (512 + tiles - 1) / tiles;
  size_t smax = (M + 2 * CH - 1) / (2 * CH);      // at least two reduction chunks per split
  if (s > smax) s = smax;
  if (s > (size_t)kMaxPartials) s = kMaxPartials;
  if (s < 1) s = 1;
  size_t mc = (M + s - 1) / s;
  mc = ((mc + CH - 1) / CH) * CH;
  a->mchunk = mc;
  a->nranges = (int)((M + mc - 1) / mc) * a->itiles;
  a->tiles_per_range = 1;
}

size_t pw_wgrad_ws(size_t M, int K, int N) {
  GemmArgs a{};
  bool small;
  plan_wgrad(M, K, N, &a, &small);
  const size_t own = (size_t)(a.nranges / a.itiles) * N * K, tr = pw_wgrad_tr_ws(M, K, N);   // either storage type may run
  return own > tr ? own : tr;
}

void pw_wgrad(int dt, hipStream_t st, const void* dz, HView av, size_t M, int K, int N, float* ws,
              float* g_w, int K_out) {
  GemmArgs a{};
  a.x = dz; a.y = av.z; a.view = View{av.z, av.scale, av.shift, av.act};
  a.out = ws; a.M = M; a.K = K; a.N = N;
  if (M <= 2048) {
    // short problem: straight into g_w, no partials
    KScope ks(st, "pw_wgrad", ((double)M * K + (double)M * N) * (dt == 0 ? 4.0 : 2.0) + (double)N * K * 8, 2.0 * M * K * N, (long)M, K, N);
    a.out = g_w;
    a.jtiles = (K + 15) / 16;
    a.itiles = (N + 15) / 16;
    const unsigned grid = (unsigned)a.jtiles * a.itiles;
    if (dt == 0) hipLaunchKernelGGL(pw_wgrad_tiny_k<float>, dim3(grid), dim3(256), 0, st, a, K_out < 0 ? K : K_out);
    else hipLaunchKernelGGL(pw_wgrad_tiny_k<bf16_t>, dim3(grid), dim3(256), 0, st, a, K_out < 0 ? K : K_out);
    return;
  }
  if (pw_wgrad_tr_ok(dt, M, K, N)) { pw_wgrad_tr(st, dz, av, M, K, N, ws, g_w, K_out); return; }
  bool small;
  plan_wgrad(M, K, N, &a, &small);
  int S = a.nranges / a.itiles;
  {
    KScope ks(st, "pw_wgrad", ((double)M * K + (double)M * N) * (dt == 0 ? 4.0 : 2.0) + (double)S * N * K * 4, 2.0 * M * K * N, (long)M, K, N);
    launch<MODE_WGRAD>(dt, st, a, small);
  }
  // K_out < K: the last K - K_out columns of A are padding and g_w is [N][K_out]
  if (K_out < 0) K_out = K;
  reduce_partials(st, ws, S, (size_t)N * K, K, (size_t)K_out, 1, g_w, K_out);
}

// ---- weight gradients of several layers in one launch -----------------------------------------------------------
// A backward pass over small tensors is a chain of short launches; the weight gradients are not part of the chain, so they
// are noted and all done here at its end, where their tiles together fill the chip (one layer has 10-60 of them).  A block
// takes a 128 x 64 tile of one layer's g_w over 32 to 256 rows: the wider of N and K in slices of 32 per wavefront, the
// narrower as up to four tiles of 16 (the ones past its end are not computed, so 24 channels cost 32 and not 64).  Operands lie
// in LDS as they lie in memory, widened to fp32 (products of bfloat16 values are exact in the fp32 MFMA); six LDS words
// feed eight MFMAs.  Layers of up to 256 rows are added to g_w here, the others leave a partial per block of rows (grp_rows).
// MobileNetV2, 32x32 input, batch 32, fp32: 33 us for 35 layers, where each layer's own weight gradient (next to its data gradient
// in one launch, or two launches of its own) put about 200 us on the chain; width 0.5, 161x193, batch 13, bfloat16: 38 us against 250.
// Bound by the latency of eight chunks (MFMA time about 10 us).  Blocks in the order of the jobs over the XCDs took 45 us:
// the layers' blocks differ in cost, so every layer is dealt over all of them.
enum { kGrpWide = 128, kGrpNarrow = 64, kGrpChunk = 32, kGrpRows = 256, kGrpJobs = 36 };
struct PwWgGroupJob {
  const void* x; const void* y;       // dZ [M][N], A [M][K]
  const float* scale; const float* shift;
  float* out;                         // g_w, or partials [S][N][K]
  int M, K, N, act, rows;             // rows per block
  int wtiles, ntiles;                 // tiles along the wider / narrower of N and K
  int nblk, add;
};
struct PwWgGroup { PwWgGroupJob job[kGrpJobs]; int blk0[kGrpJobs + 1]; int n; };

template <typename T>
__global__ __launch_bounds__(256, 3) void pw_wgrad_group_k(PwWgGroup a) {
  enum { LW = kGrpWide + 16, LN = kGrpNarrow + 16 };   // 16 banks from row to row: the four rows of an operand do not collide
  __shared__ __attribute__((aligned(16))) float sw[kGrpChunk * LW];
  __shared__ __attribute__((aligned(16))) float sn[kGrpChunk * LN];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, rg = lane >> 4;
  int lb;
  const PwWgGroupJob p = a.job[group_job(a.blk0, a.n, lb)];
  if (lb >= p.nblk) return;
  const int tiles = p.wtiles * p.ntiles, split = lb / tiles, tile = lb - split * tiles;
  const bool wide_n = p.N >= p.K;
  const int Cw = wide_n ? p.N : p.K, Cn = wide_n ? p.K : p.N;
  const int w0 = tile % p.wtiles * kGrpWide, n0 = tile / p.wtiles * kGrpNarrow;
  const T* W = reinterpret_cast<const T*>(wide_n ? p.x : p.y);
  const T* Nn = reinterpret_cast<const T*>(wide_n ? p.y : p.x);
  const int mb = split * p.rows, me = min(mb + p.rows, p.M);
  const bool view_w = p.scale != nullptr && !wide_n, view_n = p.scale != nullptr && wide_n;
  const float lo = act_lo(p.act), hi = act_hi(p.act);

  // 32 rows x 16 vectors of the wide operand (two per thread), 32 x 8 of the narrow one
  const int wc = (tid & 15) * 8, wr = tid >> 4, nc = (tid & 7) * 8, nr = tid >> 3;
  const bool wc_ok = w0 + wc < Cw, nc_ok = n0 + nc < Cn;
  float sc[8], sh[8];                                   // of the operand that is a view
  if (view_w || view_n) {
    const int c = view_w ? (wc_ok ? w0 + wc : 0) : (nc_ok ? n0 + nc : 0);
    load8(p.scale + c, sc);
    load8(p.shift + c, sh);
  }
  Raw<T> rw[2], rn;
  auto fetch = [&](const int m0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 2; ++q) raw_load(rw[q], W + (wc_ok && m0 + wr + 16 * q < me ? (size_t)(m0 + wr + 16 * q) * Cw + w0 + wc : 0));
    raw_load(rn, Nn + (nc_ok && m0 + nr < me ? (size_t)(m0 + nr) * Cn + n0 + nc : 0));
  };
  auto put = [&](float* dst, const Raw<T>& r, const bool in, const bool view) __attribute__((always_inline)) {
    float v[8];
    raw_unpack(r, v);
    if (view)
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = round_to<T>(clamp_act(fmaf(v[e], sc[e], sh[e]), lo, hi));
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = in ? v[e] : 0.f;
    store8(dst, v);
  };
  f4v acc[2][4];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[i][q] = f4v{0.f, 0.f, 0.f, 0.f};
  const bool live = w0 + wave * 32 < Cw;
  // A chain of fp32 additions no longer than one chunk, whatever the rows of the block: the chunks' sums meet in float64.  With all
  // 256 rows in one chain a gradient over 6272 rows was 2.8e-7 (2-norm) off the exact product of its operands; layer by layer, in
  // pieces of 64 rows, it is 1.4e-7; this is 1.1e-7.
  auto run = [&](auto NQ) __attribute__((always_inline)) {
    constexpr int nq = decltype(NQ)::value;
    double tot[2][nq][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < nq; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) tot[i][q][r] = 0.0;
    fetch(mb);
    for (int m0 = mb; m0 < me; m0 += kGrpChunk) {
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 2; ++q) put(sw + (wr + 16 * q) * LW + wc, rw[q], wc_ok && m0 + wr + 16 * q < me, view_w);
      put(sn + nr * LN + nc, rn, nc_ok && m0 + nr < me, view_n);
      __syncthreads();
      if (m0 + kGrpChunk < me) fetch(m0 + kGrpChunk);
      if (live) {
#pragma unroll
        for (int r = 0; r < kGrpChunk; r += 4) {
          float x[2], y[nq];
#pragma unroll
          for (int i = 0; i < 2; ++i) x[i] = sw[(r + rg) * LW + wave * 32 + i * 16 + l16];
#pragma unroll
          for (int q = 0; q < nq; ++q) y[q] = sn[(r + rg) * LN + q * 16 + l16];
#pragma unroll
          for (int q = 0; q < nq; ++q)
#pragma unroll
            for (int i = 0; i < 2; ++i)
              acc[i][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[q], r == 0 ? f4v{0.f, 0.f, 0.f, 0.f} : acc[i][q], 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int q = 0; q < nq; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) tot[i][q][r] += (double)acc[i][q][r];
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < nq; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][q][r] = (float)tot[i][q][r];
  };
  const int nq = min(4, (Cn - n0 + 15) / 16);
  if (nq == 1) run(std::integral_constant<int, 1>());
  else if (nq == 2) run(std::integral_constant<int, 2>());
  else if (nq == 3) run(std::integral_constant<int, 3>());
  else run(std::integral_constant<int, 4>());
  if (!live) return;
  // register r: wide index 4 * rg + r, narrow index l16: sixteen lanes (wide = N) or a lane's four registers (wide = K) are adjacent
  float* out = p.out + (p.add ? 0 : (size_t)split * p.N * p.K);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int w = w0 + wave * 32 + i * 16 + 4 * rg, c = n0 + q * 16 + l16;
      if (w >= Cw || c >= Cn) continue;                 // Cw is a multiple of 8: four at once are in or out
      if (wide_n) {
        float old[4];
        if (p.add)
#pragma unroll
          for (int r = 0; r < 4; ++r) old[r] = out[(size_t)(w + r) * p.K + c];
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(size_t)(w + r) * p.K + c] = p.add ? old[r] + acc[i][q][r] : acc[i][q][r];
      } else {
        float4* dst = reinterpret_cast<float4*>(out + (size_t)c * p.K + w);
        float4 v = make_float4(acc[i][q][0], acc[i][q][1], acc[i][q][2], acc[i][q][3]);
        if (p.add) { const float4 o = *dst; v = make_float4(o.x + v.x, o.y + v.y, o.z + v.z, o.w + v.w); }
        *dst = v;
      }
    }
}

// Rows per block: as many blocks as fill the chip together with those of the other layers (about 512), 32 to 256 rows each, and more
// where a layer would leave more than 512 partials.  A step, us, always 256 rows / this: 96 -> 24 channels, 8192 rows, alone fp32 47.9 / 40.8,
// bfloat16 42.2 / 35.0; 64 <-> 384, 6272 rows, fp32 alone 66.9 / 58.8, two layers 103 / 98; 24 <-> 144, 512 rows, 24 layers 391 / 327;
// with 32 rows throughout twelve layers of 6272 rows took 562 instead of 516.
static int grp_rows(size_t M, int K, int N, int share) {
  if (M <= kGrpRows) return kGrpRows;
  const int wide = N >= K ? N : K, narrow = N >= K ? K : N;
  const size_t tiles = (size_t)((wide + kGrpWide - 1) / kGrpWide) * ((narrow + kGrpNarrow - 1) / kGrpNarrow), want = share < 2 ? 512 : share < 512 ? 512 / share : 1;
  const auto chunks = [](size_t rows) { return (rows + kGrpChunk - 1) / kGrpChunk * kGrpChunk; };
  size_t rows = chunks((M * tiles + want - 1) / want);
  if (rows > kGrpRows) rows = kGrpRows;
  const size_t least = chunks((M + 511) / 512);
  return (int)(rows > least ? rows : least);
}

// Long bfloat16 layers run in the transposing kernel, which leaves partials; of the others those of more than grp_rows rows do, and
// shorter ones are added to g_w at once.
size_t pw_wgrad_group_ws(int dt, size_t M, int K, int N, PwShare share) {
  if (pw_wgrad_tr_ok(dt, M, K, N)) return pw_wgrad_tr_ws(M, K, N, share.tr);
  const int R = grp_rows(M, K, N, share.other);
  return M > (size_t)R ? (M + R - 1) / R * (size_t)N * K : 0;
}

void pw_wgrad_group(int dt, hipStream_t st, const PwWgradJob* jobs, int n, PwShare share, std::vector<ReduceJob>* left) {
  if (dt == 1) pw_wgrad_tr_group(st, jobs, n, share.tr, left);
  PwWgGroup a{};
  int blocks = 0;
  double bytes = 0, flops = 0;
  auto launch = [&]() {
    if (a.n == 0) return;
    a.blk0[a.n] = blocks;
    KScope ks(st, "pw_wgrad", bytes, flops);
    if (dt == 0) hipLaunchKernelGGL(pw_wgrad_group_k<float>, dim3(blocks), dim3(256), 0, st, a);
    else hipLaunchKernelGGL(pw_wgrad_group_k<bf16_t>, dim3(blocks), dim3(256), 0, st, a);
    a.n = 0; blocks = 0; bytes = flops = 0;
  };
  for (int i = 0; i < n; ++i) {
    const PwWgradJob& w = jobs[i];
    if (pw_wgrad_tr_ok(dt, w.M, w.K, w.N)) continue;
    const int R = grp_rows(w.M, w.K, w.N, share.other), S = (int)((w.M + R - 1) / R), wide = w.N >= w.K ? w.N : w.K, narrow = w.N >= w.K ? w.K : w.N;
    PwWgGroupJob j{w.dz, w.a.z, w.a.scale, w.a.shift, S == 1 ? w.g_w : w.ws, (int)w.M, w.K, w.N, w.a.act, R,
                   (wide + kGrpWide - 1) / kGrpWide, (narrow + kGrpNarrow - 1) / kGrpNarrow, 0, S == 1};
    j.nblk = j.wtiles * j.ntiles * S;
    a.blk0[a.n] = blocks;
    a.job[a.n++] = j;
    blocks += (j.nblk + 7) / 8 * 8;
    bytes += ((double)w.M * w.K + (double)w.M * w.N) * (dt == 0 ? 4.0 : 2.0) + (double)S * w.N * w.K * 4;
    flops += 2.0 * w.M * w.K * w.N;
    if (S > 1) left->push_back(ReduceJob{w.ws, w.g_w, S, w.N * w.K, w.K, w.K, 1, w.K});
    if (a.n == kGrpJobs) launch();
  }
  launch();
}

// ---- backward of a fully connected layer ------------------------------------------------------------------------
// Latency only (a few tiles over operands that the caches hold), so everything is one launch: blocks [0, nd) take 16 x 16 tiles of the
// data gradient, the others 16 x 16 tiles of g_w (and, in the first column of tiles, the bias gradient, whose terms pass through their
// registers anyway); four wavefronts split the reduction.  The class count is arbitrary, so elements are loaded one by one.
// Weight gradient, bias gradient, data gradient and the average's backward were four launches: 2.5 + 1.4 + 4.9 + 2.7 us for 8 x 64 -> 6
// fp32, 4.7 + 2.2 + 12.0 + 3.8 for 13 x 1280 -> 100 bfloat16; one: 5.3 and 5.9.
template <typename T>
__global__ __launch_bounds__(256) void fc_bwd_k(const T* __restrict__ d, View in, const T* __restrict__ w, int B, int N, int K, float* __restrict__ g_w,
                                                float* __restrict__ g_b, T* __restrict__ dIn, int HW, int nd, const float* __restrict__ open,
                                                float* __restrict__ sums) {
  constexpr int U = 4;
  __shared__ float red[4][16][17];
  __shared__ float bred[4][16];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, l16 = lane & 15, rg = lane >> 4;
  const int orow = threadIdx.x >> 4, ocol = threadIdx.x & 15, kt = (K + 15) / 16;
  const bool dgrad = (int)blockIdx.x < nd;
  const int tile = dgrad ? blockIdx.x : blockIdx.x - nd, k0 = tile % kt * 16, i0 = tile / kt * 16;
  const int k = k0 + l16, kc = k < K ? k : 0;
  f4v acc = {0.f, 0.f, 0.f, 0.f};
  if (dgrad) {                                          // rows b, reduction over n
    const int b = i0 + l16, bc = b < B ? b : 0;
    const int nst = (N + 15) / 16, sb = wave * nst / 4, se = (wave + 1) * nst / 4;
    const int ob = i0 + orow, ok = k0 + ocol;
    const bool written = ob < B && ok < K;
    float cnt = 0.f, z = 0.f;
    if (sums) {                                         // requested now, used behind the products
      const size_t at = written ? (size_t)ob * 2 * K + ok : 0;
      cnt = open[at];
      z = open[at + (written ? K : 0)];
    }
    for (int s0 = sb; s0 < se; s0 += U) {
      T x[U][4], y[U][4];
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int n = (s0 + u) * 16 + rg * 4 + e, nc = s0 + u < se && n < N ? n : 0;
          x[u][e] = d[(size_t)bc * N + nc];
          y[u][e] = w[(size_t)nc * K + kc];
        }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool ok = s0 + u < se && (s0 + u) * 16 + rg * 4 + e < N;
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ok && b < B ? to_f32(x[u][e]) : 0.f, ok && k < K ? to_f32(y[u][e]) : 0.f, acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][4 * rg + r][l16] = acc[r];
    __syncthreads();
    const float v = red[0][orow][ocol] + red[1][orow][ocol] + red[2][orow][ocol] + red[3][orow][ocol];
    if (HW == 0) { if (written) dIn[(size_t)ob * K + ok] = from_f32<T>(v); return; }
    // the mean's gradient: the pooled feature's, as stored, times 1 / HW at every position
    const T o = from_f32<T>(round_to<T>(v) * (1.f / (float)HW));
    if (sums) {
      const bool on = written && cnt > 0.f;             // chosen, not multiplied: an infinite gradient of what is off stays out
      __syncthreads();
      red[0][orow][ocol] = on ? to_f32(o) * cnt : 0.f;
      red[1][orow][ocol] = on ? to_f32(o) * z : 0.f;
      __syncthreads();
      if (threadIdx.x < 32 && k0 + (int)(threadIdx.x & 15) < K) {
        const int q = threadIdx.x >> 4, c = threadIdx.x & 15;
        double t = 0.0;                                 // images meet in float64, as in gap_bwd_k
#pragma unroll
        for (int r = 0; r < 16; ++r) t += red[q][r][c];
        sums[((size_t)(tile / kt) * 2 + q) * K + k0 + c] = (float)t;
      }
    }
    if (!written) return;
    T* dst = dIn + (size_t)ob * HW * K + ok;
    for (int p = 0; p < HW; ++p) dst[(size_t)p * K] = o;
    return;
  }
  const int n = i0 + l16, nc = n < N ? n : 0;           // rows n, reduction over b
  const bool view = in.scale != nullptr;
  const float sc = view ? in.scale[kc] : 1.f, sh = view ? in.shift[kc] : 0.f, lo = act_lo(in.act), hi = act_hi(in.act);
  const T* A = reinterpret_cast<const T*>(in.z);
  const int on = i0 + orow, ok = k0 + ocol;
  const bool writer = on < N && ok < K, bias = k0 == 0 && threadIdx.x < 16 && i0 + (int)threadIdx.x < N;
  float g_old = writer ? g_w[(size_t)on * K + ok] : 0.f, b_old = bias ? g_b[i0 + threadIdx.x] : 0.f, bs = 0.f;
  const int per = (B + 15) / 16 * 4, mb = wave * per, me = min(mb + per, B);
  for (int m0 = mb; m0 < me; m0 += 4 * 2 * U) {
    T x[2 * U], y[2 * U];
#pragma unroll
    for (int u = 0; u < 2 * U; ++u) {
      const int m = m0 + 4 * u + rg, mc = m < me ? m : mb;
      x[u] = d[(size_t)mc * N + nc];
      y[u] = A[(size_t)mc * K + kc];
    }
#pragma unroll
    for (int u = 0; u < 2 * U; ++u) {
      const bool in_m = m0 + 4 * u + rg < me;
      float a = to_f32(y[u]);
      if (view) a = round_to<T>(clamp_act(fmaf(a, sc, sh), lo, hi));
      const float dv = in_m && n < N ? to_f32(x[u]) : 0.f;
      bs += dv;
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(dv, in_m && k < K ? a : 0.f, acc, 0, 0, 0);
    }
  }
  bs += __shfl_xor(bs, 16, 64);
  bs += __shfl_xor(bs, 32, 64);
#pragma unroll
  for (int r = 0; r < 4; ++r) red[wave][4 * rg + r][l16] = acc[r];
  if (lane < 16) bred[wave][lane] = bs;
  __syncthreads();
  asm volatile("" : "+v"(g_old), "+v"(b_old));
  if (writer) g_w[(size_t)on * K + ok] = g_old + (red[0][orow][ocol] + red[1][orow][ocol] + red[2][orow][ocol] + red[3][orow][ocol]);
  if (bias) g_b[i0 + threadIdx.x] = b_old + (bred[0][threadIdx.x] + bred[1][threadIdx.x] + bred[2][threadIdx.x] + bred[3][threadIdx.x]);
}

// A wavefront walks a quarter of the rows (weight gradient) and of the classes (data gradient), 32 and 64 to a trip, and every tile fetches
// its operands itself: from about 200 M products on the tiled kernels' launches are faster.  Forward and backward, us, separate launches / one,
// fp32 (bfloat16 likewise): 512 x 64 -> 12 20 / 12, 32 x 1792 -> 1000 42 / 34, 128 x 1280 -> 1000 (164 M) 64 / 55, 512 x 384 -> 1000 (197 M)
// 53 / 47, 128 x 1792 -> 1000 (229 M) 75 / 72 and 53 / 54, 512 x 4096 -> 100 (210 M) 120 / 129, 256 x 1280 -> 1000 (328 M) 73 / 80,
// 512 x 1792 -> 1000 129 / 178.
int fc_bwd_ok(int B, int N, int K) { return B <= 512 && N <= 1024 && (size_t)N * K <= ((size_t)1 << 24) && (size_t)B * N * K <= 200000000; }
// the tiles write their 64-byte pieces position by position: for a few MB that is cheaper than a launch
int fc_bwd_gap_ok(int B, int HW, int K) { return (size_t)B * HW * K <= ((size_t)1 << 20); }

void fc_bwd(int dt, hipStream_t st, const void* d, HView in, const void* w, int B, int N, int K, float* g_w, float* g_b, void* dIn, int HW,
            const float* open, float* sums, int* P_out) {
  const int kt = (K + 15) / 16, nd = dIn ? (B + 15) / 16 * kt : 0, nw = (N + 15) / 16 * kt;
  const double es = dt == 0 ? 4.0 : 2.0;
  KScope ks(st, "fc_bwd", ((double)B * K * (1.0 + (HW > 0 ? HW : 1)) + (double)B * N + (double)N * K) * es + (double)N * K * 8, 4.0 * B * N * K, B, K, N);
  const View v{in.z, in.scale, in.shift, in.act};
  if (sums) *P_out = (B + 15) / 16;
  if (dt == 0) hipLaunchKernelGGL(fc_bwd_k<float>, dim3(nd + nw), dim3(256), 0, st, (const float*)d, v, (const float*)w, B, N, K, g_w, g_b, (float*)dIn, HW, nd, open, sums);
  else hipLaunchKernelGGL(fc_bwd_k<bf16_t>, dim3(nd + nw), dim3(256), 0, st, (const bf16_t*)d, v, (const bf16_t*)w, B, N, K, g_w, g_b, (bf16_t*)dIn, HW, nd, open, sums);
}

// wgrad then dgrad of one pointwise layer; short problems take one launch for both
void pw_bwd(int dt, hipStream_t st, const void* dz, const void* w, const void* res, HView av, size_t M, int K, int N,
            float* ws, float* g_w, void* dA) {
  if (M <= 2048 && tiny_ok(dt, M, N, K, false)) {
    TinyArgs d{};
    GemmArgs g{};
    d.x = dz; d.y = w; d.res = res; d.out = dA; d.M = M; d.K = K; d.N = N;
    d.jtiles = (K + 15) / 16; d.itiles = (int)((M + 15) / 16); d.nranges = d.itiles; d.tiles_per_range = 1; d.dj = FastDiv::of(d.jtiles);
    g.x = dz; g.y = av.z; g.view = View{av.z, av.scale, av.shift, av.act}; g.out = g_w; g.M = M; g.K = K; g.N = N;
    g.jtiles = (K + 15) / 16; g.itiles = (N + 15) / 16;
    const int nd = d.jtiles * d.itiles, nw = g.jtiles * g.itiles;
    const double es = dt == 0 ? 4.0 : 2.0;
    KScope ks(st, "pw_bwd", ((double)M * K * (res ? 3.0 : 2.0) + (double)M * N + (double)N * K) * es + (double)N * K * 8,
              4.0 * M * K * N, (long)M, K, N);
    if (M > 512) {
      const int nd4 = (nd + 3) / 4;             // four data-gradient tiles per 16-wavefront block
      if (dt == 0) hipLaunchKernelGGL((pw_bwd_tiny_k<float, 16>), dim3(nd4 + nw), dim3(1024), 0, st, d, g, K, nd4);
      else hipLaunchKernelGGL((pw_bwd_tiny_k<bf16_t, 16>), dim3(nd4 + nw), dim3(1024), 0, st, d, g, K, nd4);
    } else {
      if (dt == 0) hipLaunchKernelGGL((pw_bwd_tiny_k<float, 4>), dim3(nd + nw), dim3(256), 0, st, d, g, K, nd);
      else hipLaunchKernelGGL((pw_bwd_tiny_k<bf16_t, 4>), dim3(nd + nw), dim3(256), 0, st, d, g, K, nd);
    }
    return;
  }
  pw_wgrad(dt, st, dz, av, M, K, N, ws, g_w);
  pw_dgrad(dt, st, dz, w, res, M, K, N, dA);
}

}  // namespace ftp
