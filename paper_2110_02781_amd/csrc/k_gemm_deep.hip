// Pointwise layers with a LONG reduction and few rows: the project layers (forward) and the expand layers (data gradient) of the
// low-resolution inverted residual blocks, against a reduction of up to 2048 channels, and most shorter ones there; in fp32
// nearly all layers (deep_plan says which, in either type).  Their tensors are small (they stay in the memory-side cache) and
// their arithmetic intensity is at the MFMA / HBM balance, so what they need is a GEMM that keeps the matrix cores fed, not a streaming kernel.
// In fp32 the matrix instructions are what bounds it (they run at a sixteenth of the rate and not beside vector instructions): there a grid that
// fills the 256 CUs with small tiles, and few instructions a step, are what counts.
//   * a block owns a (32*S) x (32*T) output tile (S = 1, 2 or 4, T = 1 .. 5, see deep_plan) and walks the whole reduction in steps of 64 (fp32: 32),
//     its four wavefronts in a 2 x 2 arrangement of (16*S) x (16*T) sub-tiles of v_mfma_f32_16x16x32_bf16 or 16x16x4_f32;
//   * both operands go through double-buffered LDS (one barrier per step); the 16-byte vectors of the next two
//     steps are on their way from memory into registers while the current step is multiplied (a layer has about one
//     block per CU and a round trip to memory takes several steps: what hides it is bytes in flight per block);
//   * the weights of the data gradient are stored [reduction][column]: they are staged as they lie in memory and
//     read back through the LDS transpose read (fp32: word by word), so neither mode repacks anything;
//   * the weight operand is the MFMA's first operand: a lane then holds four CONSECUTIVE output columns of one row
//     and stores (and adds the residual, and sums the BatchNorm statistics of) them together.
// Forward applies the producer's BatchNorm + activation to the rows on their way into LDS and leaves the column sums of
// the stored output (one partial per row tile, summed in a fixed order) for the BatchNorm that follows.
#include <type_traits>

#include "dev_common.h"
#include "kernels.h"
#include "mfma_frag.h"

namespace ftp {

enum { kDeepMaxR = 2048 };
// a reduction step is 128 bytes of a row, moved in vectors of 16; an odd number of those between LDS rows
template <typename E> struct Deep { enum { V = 16 / sizeof(E), KS = 8 * V, LD = KS + V, F32 = sizeof(E) == 4 }; };
enum { DEEP_FWD = 0, DEEP_FWD_VIEW = 1, DEEP_DGRAD = 2, DEEP_DGRAD_RES = 3, DEEP_DGRAD_GATED = 4, DEEP_DGRAD_SUMS = 5 };

struct DeepArgs {
  const void* x;      // [M][R]: A as stored (forward) or dZ (data gradient)
  const void* y;      // W[N][K]: forward [column][reduction], data gradient [reduction][column]
  const float* scale;   // forward: view of x, indexed by the reduction channel (DEEP_FWD_VIEW)
  const float* shift;
  const void* res;    // [M][NC] added to the result (DEEP_DGRAD_RES; GATED, SUMS: may be nullptr)
  const void* z;      // [M][NC] the raw output that the result is the gradient behind (DEEP_DGRAD_GATED: through scale, shift, act of its columns)
  void* out;          // [M][NC]
  float* stats;         // forward: [row tiles][2][NC] column sums of the stored output and of its squares, or nullptr; GATED, SUMS: of the (gated) output and of it times z
  int act;
  int M, R, NC;         // rows, reduction extent, output columns
  int jtiles;           // column tiles; the grid is jtiles * row tiles
};

template <typename E, int S, int T, int MODE>
__global__ __launch_bounds__(256) void pw_gemm_deep_k(DeepArgs p) {
  constexpr int V = Deep<E>::V, KS = Deep<E>::KS;
  constexpr bool F32 = Deep<E>::F32;
  constexpr bool DG = MODE >= DEEP_DGRAD;
  constexpr int BM = 32 * S, BN = 32 * T, LD = Deep<E>::LD, LDY = BN + V;
  constexpr int XS = BM * LD;                               // elements of one x buffer
  constexpr int YS = DG ? KS * LDY : BN * LD;          // elements of one y buffer
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  E* xs = reinterpret_cast<E*>(smem_raw);                   // [2][BM][LD]
  E* ys = xs + 2 * XS;                                      // [2][BN][LD] or [2][KS][LDY]
  float* vw = reinterpret_cast<float*>(ys + 2 * YS);        // forward with a view: scale[RP], shift[RP], RP = R rounded up to KS
  if (DG) __builtin_amdgcn_s_setprio(3);                    // data-gradient chain

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l16 = lane & 15, G = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;
  const int lb = xcd_logical_block();
  const int jt = lb % p.jtiles, it = lb / p.jtiles;
  const int m0 = it * BM, j0 = jt * BN;
  const int M = p.M, R = p.R, NC = p.NC;

  // ---- loaders: S vectors of x and T vectors of y per thread and step ----
  // Both operands are read through buffer descriptors (base, size): a load whose byte offset lies outside the tensor
  // returns zeros, so a vector outside the operand (rows past M, columns past NC, reduction elements past R) is
  // requested at an offset past the end instead of being selected away afterwards: no selects and no branches between a
  // load and its use, one 32-bit offset register per vector, and the only waits in the loop are the counted ones in
  // front of each step.  Through the view a zero row becomes act(shift): such rows (past M) are never stored and are
  // masked out of the statistics; past R the weights are zero, so the products vanish.
  const int xkv = (tid & 7) * V, xrow = tid >> 3;           // x: 8 threads cover the reduction elements of a row
  // steps in flight: two.  A third costs about a hundred registers here, and two resident blocks per CU, which hide each
  // other's barrier and LDS phases, measured worth more than the third step.
  constexpr int D = 2;
  constexpr uint32_t kPast = 0x80000000u;                   // beyond any operand here (they are smaller than 2 GiB), also after adding a step
  constexpr uint32_t ES = sizeof(E);
  constexpr int VR = BN / V;                                // data gradient: vectors to a staged row of weights
  struct Set { uint4 x[S]; uint4 y[T]; };
  Set set[D];
  const int RP = (R + KS - 1) / KS * KS;
  const __amdgpu_buffer_rsrc_t bx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.x), 0, (int)((size_t)M * R * sizeof(E)), 0x00020000);
  const __amdgpu_buffer_rsrc_t by = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.y), 0, (int)((size_t)R * NC * sizeof(E)), 0x00020000);
  uint32_t ox[S], oy[T];                                    // byte offsets of this thread's vectors at step 0
#pragma unroll
  for (int q = 0; q < S; ++q) {
    const int m = m0 + xrow + q * 32;
    ox[q] = m < M ? (uint32_t)(m * R + xkv) * ES : kPast;
  }
#pragma unroll
  for (int q = 0; q < T; ++q) {
    if (!DG) {
      const int j = j0 + xrow + q * 32;
      oy[q] = j < NC ? (uint32_t)(j * R + xkv) * ES : kPast;
    } else {
      const int v = tid + q * 256;
      const int j = j0 + (v % VR) * V;
      oy[q] = j < NC ? (uint32_t)((v / VR) * NC + j) * ES : kPast;
    }
  }
  if (MODE == DEEP_FWD_VIEW) {
    for (int i = tid; i < RP; i += 256) {
      vw[i] = i < R ? p.scale[i] : 0.f;
      vw[RP + i] = i < R ? p.shift[i] : 0.f;
    }
  }
  typedef uint32_t u4v_t __attribute__((ext_vector_type(4)));
  auto ld = [&](const __amdgpu_buffer_rsrc_t rs, const uint32_t off) __attribute__((always_inline)) {
    const u4v_t v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
  };
  auto fetch = [&](Set& f, const int r0) __attribute__((always_inline)) {
    const bool kin = r0 + xkv < R;
#pragma unroll
    for (int q = 0; q < S; ++q) f.x[q] = ld(bx, kin ? ox[q] + (uint32_t)r0 * ES : kPast);
#pragma unroll
    for (int q = 0; q < T; ++q) {
      if (!DG) {
        f.y[q] = ld(by, kin ? oy[q] + (uint32_t)r0 * ES : kPast);
      } else {
        const int v = tid + q * 256;
        f.y[q] = ld(by, r0 + v / VR < R ? oy[q] + (uint32_t)(r0 * NC) * ES : kPast);
      }
    }
  };
  auto commit = [&](const Set& f, const int r0, E* xb, E* yb) __attribute__((always_inline)) {
    const float lo = act_lo(p.act), hi = act_hi(p.act);
    float vsc[V], vsh[V];
    if (MODE == DEEP_FWD_VIEW)             // r0 + xkv < RP: the steps stop at RP
#pragma unroll
      for (int e = 0; e < V; e += 4) {
        *reinterpret_cast<float4*>(vsc + e) = ld4(vw + r0 + xkv + e);
        *reinterpret_cast<float4*>(vsh + e) = ld4(vw + RP + r0 + xkv + e);
      }
#pragma unroll
    for (int q = 0; q < S; ++q) {
      uint4 v = f.x[q];
      if (MODE == DEEP_FWD_VIEW && F32) {
        float* t = reinterpret_cast<float*>(&v);
#pragma unroll
        for (int e = 0; e < 4; ++e) t[e] = clamp_act(fmaf(t[e], vsc[e], vsh[e]), lo, hi);
      }
      if constexpr (MODE == DEEP_FWD_VIEW && !F32) {
        Raw<bf16_t> raw;
        raw.a = v;
        float t[8];
        raw_unpack(raw, t);
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = clamp_act(fmaf(t[e], vsc[e], vsh[e]), lo, hi);
        v.x = f32x2_to_bf16x2(t[0], t[1]); v.y = f32x2_to_bf16x2(t[2], t[3]);
        v.z = f32x2_to_bf16x2(t[4], t[5]); v.w = f32x2_to_bf16x2(t[6], t[7]);
      }
      *reinterpret_cast<uint4*>(xb + (xrow + q * 32) * LD + xkv) = v;
    }
#pragma unroll
    for (int q = 0; q < T; ++q) {
      if (!DG) {
        *reinterpret_cast<uint4*>(yb + (xrow + q * 32) * LD + xkv) = f.y[q];
      } else {
        const int i = tid + q * 256;
        *reinterpret_cast<uint4*>(yb + (i / VR) * LDY + (i % VR) * V) = f.y[q];
      }
    }
  };

  f4v_t acc[S][T];
#pragma unroll
  for (int a = 0; a < S; ++a)
#pragma unroll
    for (int b = 0; b < T; ++b) acc[a][b] = f4v_t{0.f, 0.f, 0.f, 0.f};
  // fp32: a chain of additions per step, 32 reduction elements, not one through the whole reduction: the streaming kernel's wavefronts share a
  // reduction of 128 and more where rows are few, and this may not be further off.  8192 rows, 192 -> 32: 1.38e-7 off the exact product
  // (2-norm) there, 1.48e-7 in chains of 64, 1.14e-7 in these; 1568 rows, 960 -> 160: 2.8e-7, 1.63e-7, 1.46e-7.  The sums of a step are added in front of
  // the next one's products: behind its own they were waited for (6272 rows 576 -> 96 data gradient 15.5 / 14.8 us, 25088 rows forward 41.9 / 40.1).  Against chains of 64
  // within 4 % either way (those 14.7 and 41.9, 3136 rows 1280 -> 320 forward 35.6 / 36.9, 160 -> 960 data gradient 18.6 / 18.8).
  f4v_t tot[F32 ? S : 1][F32 ? T : 1];
  if constexpr (F32)
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
      for (int b = 0; b < T; ++b) tot[a][b] = f4v_t{0.f, 0.f, 0.f, 0.f};
  auto meet = [&]() __attribute__((always_inline)) {
    if constexpr (F32)
#pragma unroll
      for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) tot[a][b] += acc[a][b];
  };

  // one step: set -> LDS buffer s % 2, barrier (which also says that everyone has finished multiplying the step before
  // last, this buffer's previous contents), the set's next request (D steps ahead; past the end: zeros), multiply
  auto step = [&](Set& f, const int s) __attribute__((always_inline)) {
    E* xb = xs + (s & 1) * XS;
    E* yb = ys + (s & 1) * YS;
    commit(f, s * KS, xb, yb);
    __syncthreads();
    __builtin_amdgcn_sched_barrier(0);   // the requests stay here, D steps ahead of their use (the scheduler would move them down to it)
    fetch(f, (s + D) * KS);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (F32) {
      meet();                              // the step before: its products are long done here, behind them each addition would wait
      // a lane holds four consecutive reduction elements of both operands, one for each of four instructions
#pragma unroll
      for (int ks = 0; ks < KS / 16; ++ks) {
        float4 xf[S], yf[T];
#pragma unroll
        for (int a = 0; a < S; ++a) xf[a] = ld4(xb + (wm * 16 * S + a * 16 + l16) * LD + ks * 16 + G * 4);
#pragma unroll
        for (int b = 0; b < T; ++b) {
          if (DG) {
            const float* yr = yb + (ks * 16 + G * 4) * LDY + wn * 16 * T + b * 16 + l16;
            yf[b] = make_float4(yr[0], yr[LDY], yr[2 * LDY], yr[3 * LDY]);
          } else {
            yf[b] = ld4(yb + (wn * 16 * T + b * 16 + l16) * LD + ks * 16 + G * 4);
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int a = 0; a < S; ++a)
#pragma unroll
            for (int b = 0; b < T; ++b)
              acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32((&yf[b].x)[e], (&xf[a].x)[e], ks + e == 0 ? f4v_t{0.f, 0.f, 0.f, 0.f} : acc[a][b], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int ks = 0; ks < KS / 32; ++ks) {
        bf16x8_t xf[S], yf[T];
#pragma unroll
        for (int a = 0; a < S; ++a) xf[a] = lds_frag(xb + (wm * 16 * S + a * 16 + l16) * LD + ks * 32 + G * 8);
#pragma unroll
        for (int b = 0; b < T; ++b) {
          if (DG) yf[b] = lds_frag_tr(yb, LDY, ks * 32 + G * 8, wn * 16 * T + b * 16, l16);
          else yf[b] = lds_frag(yb + (wn * 16 * T + b * 16 + l16) * LD + ks * 32 + G * 8);
        }
#pragma unroll
        for (int a = 0; a < S; ++a)
#pragma unroll
          for (int b = 0; b < T; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yf[b], xf[a], acc[a][b], 0, 0, 0);
      }
    }
  };
  const int nsteps = RP / KS;
#pragma unroll
  for (int d = 0; d < D; ++d) {
    fetch(set[d], d * KS);
    // the sets are requested in order: a wait for set d is then a wait for "all but the youngest loads" on every path
    __builtin_amdgcn_sched_barrier(0);
  }
  // with sums a thread has V columns and every RL-th row of the tile; its part of z is requested behind the first two steps (short reductions have no others)
  // where that costs no resident block
  constexpr bool SUMS = MODE >= DEEP_DGRAD_GATED, EARLY = SUMS && S * T <= 6;
  constexpr int CG = BN / V, RL = 256 / CG, NP = SUMS ? (BM + RL - 1) / RL : 1;
  const int cg = tid % CG, rl = tid / CG, jv = j0 + cg * V;
  const bool cin = rl < RL && jv < NC;
  uint4 zq[NP];
  auto request_z = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int row = rl + q * RL, m = m0 + row;
      zq[q] = *reinterpret_cast<const uint4*>((const E*)p.z + (cin && row < BM && m < M ? (size_t)m * NC + jv : 0));
    }
  };
  if (EARLY) {
    request_z();
    __builtin_amdgcn_sched_barrier(0);
  }
  if (MODE == DEEP_FWD_VIEW) __syncthreads();                        // the view vectors are in LDS
  // whole groups of D steps without a branch inside (a path from the middle of a group back to the loop head would
  // turn every wait at the head into a wait for all loads), then the remaining steps
  int s0 = 0;
  for (; s0 + D <= nsteps; s0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) step(set[d], s0 + d);
  }
#pragma unroll
  for (int d = 0; d + 1 < D; ++d)
    if (s0 + d < nsteps) step(set[d], s0 + d);
  if constexpr (F32) {
    meet();
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
      for (int b = 0; b < T; ++b) acc[a][b] = tot[a][b];
  }

  // ---- results with sums: the rounded tile goes through LDS, so that its stores, z and the sums go by rows of 16-byte vectors.  As the accumulators lie a
  // lane has four columns, a wavefront 32 bytes of a row: 12544 rows 56 -> 336 with gate 9.9 us, so 9.0; without sums 6.7, and a pass for them 5.7 ----
  if constexpr (SUMS) {
    constexpr int LDO = BN + V;
    if (!EARLY) request_z();
    float sc[V], sh[V], s1[V], s2[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      s1[e] = s2[e] = 0.f;
      if (MODE == DEEP_DGRAD_GATED) { sc[e] = p.scale[(cin ? jv : 0) + e]; sh[e] = p.shift[(cin ? jv : 0) + e]; }
    }
    typedef typename std::conditional<F32, float4, uint2>::type Out4;
    if (p.res) {                         // added in front of the rounding; all groups are requested before the first is used
      Out4 rs[S][T];
#pragma unroll
      for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) {
          const int m = m0 + wm * 16 * S + a * 16 + l16, j = j0 + wn * 16 * T + b * 16 + 4 * G;
          rs[a][b] = *reinterpret_cast<const Out4*>((const E*)p.res + (m < M && j < NC ? (size_t)m * NC + j : 0));
        }
#pragma unroll
      for (int a = 0; a < S; ++a)
#pragma unroll
        for (int b = 0; b < T; ++b) {
          const float4 r = load4(reinterpret_cast<const E*>(&rs[a][b]));
          acc[a][b][0] += r.x; acc[a][b][1] += r.y; acc[a][b][2] += r.z; acc[a][b][3] += r.w;
        }
    }
    E* const ot = reinterpret_cast<E*>(smem_raw);
    __syncthreads();                     // the staging buffers are free
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
      for (int b = 0; b < T; ++b)
        store4(ot + (wm * 16 * S + a * 16 + l16) * LDO + wn * 16 * T + b * 16 + 4 * G, make_float4(acc[a][b][0], acc[a][b][1], acc[a][b][2], acc[a][b][3]));
    __syncthreads();
    const float lo = act_lo(p.act), hi = act_hi(p.act);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      const int row = rl + q * RL, m = m0 + row;
      if (cin && row < BM && m < M) {
        const uint4 u = *reinterpret_cast<const uint4*>(ot + row * LDO + cg * V);
        *reinterpret_cast<uint4*>((E*)p.out + (size_t)m * NC + jv) = u;
#pragma unroll
        for (int h = 0; h < V; h += 4) {
          const float4 d4 = load4(reinterpret_cast<const E*>(&u) + h), z4 = load4(reinterpret_cast<const E*>(&zq[q]) + h);
          const float d[4] = {d4.x, d4.y, d4.z, d4.w}, z[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float r = d[e];
            if (MODE == DEEP_DGRAD_GATED) {
              const float y = fmaf(z[e], sc[h + e], sh[h + e]);
              r = y > lo && y < hi ? r : 0.f;
            }
            s1[h + e] += r;
            s2[h + e] = fmaf(r, z[e], s2[h + e]);
          }
        }
      }
    }
    __syncthreads();
    float* const red = reinterpret_cast<float*>(smem_raw);             // [2][RL][BN]
    if (rl < RL)
#pragma unroll
      for (int e = 0; e < V; e += 4) {
        *reinterpret_cast<float4*>(red + rl * BN + cg * V + e) = make_float4(s1[e], s1[e + 1], s1[e + 2], s1[e + 3]);
        *reinterpret_cast<float4*>(red + (RL + rl) * BN + cg * V + e) = make_float4(s2[e], s2[e + 1], s2[e + 2], s2[e + 3]);
      }
    __syncthreads();
    for (int i = tid; i < 2 * BN; i += 256) {
      const int which = i / BN, col = i - which * BN, j = j0 + col;
      if (j >= NC) continue;
      float t = 0.f;
#pragma unroll 4
      for (int r = 0; r < RL; ++r) t += red[(which * RL + r) * BN + col];
      p.stats[((size_t)it * 2 + which) * NC + j] = t;
    }
    return;
  }
  // ---- results: acc[a][b][e] is out[m0 + wm*16S + 16a + l16][j0 + wn*16T + 16b + 4G + e] ----
  float s1[T][4], s2[T][4];
#pragma unroll
  for (int b = 0; b < T; ++b)
#pragma unroll
    for (int e = 0; e < 4; ++e) { s1[b][e] = 0.f; s2[b][e] = 0.f; }
  typedef typename std::conditional<F32, float4, uint2>::type Out4;      // four consecutive columns as stored
  Out4 rs[S][T];
  if (MODE == DEEP_DGRAD_RES) {          // all residual groups are requested before the first store
#pragma unroll
    for (int a = 0; a < S; ++a)
#pragma unroll
      for (int b = 0; b < T; ++b) {
        const int m = m0 + wm * 16 * S + a * 16 + l16, j = j0 + wn * 16 * T + b * 16 + 4 * G;
        const bool in = m < M && j < NC;
        rs[a][b] = *reinterpret_cast<const Out4*>((const E*)p.res + (in ? (size_t)m * NC + j : 0));
      }
  }
#pragma unroll
  for (int a = 0; a < S; ++a)
#pragma unroll
    for (int b = 0; b < T; ++b) {
      const int m = m0 + wm * 16 * S + a * 16 + l16, j = j0 + wn * 16 * T + b * 16 + 4 * G;
      float v0 = acc[a][b][0], v1 = acc[a][b][1], v2 = acc[a][b][2], v3 = acc[a][b][3];
      if constexpr (MODE == DEEP_DGRAD_RES) {
        const float4 r = load4(reinterpret_cast<const E*>(&rs[a][b]));
        v0 += r.x; v1 += r.y; v2 += r.z; v3 += r.w;
      }
      Out4 u;
      if constexpr (F32) {
        u = make_float4(v0, v1, v2, v3);
      } else {
        u.x = f32x2_to_bf16x2(v0, v1);
        u.y = f32x2_to_bf16x2(v2, v3);
      }
      if (m < M && j < NC) *reinterpret_cast<Out4*>((E*)p.out + (size_t)m * NC + j) = u;
      if (!DG) {                         // statistics of the values as stored; columns past NC are exact zeros, rows past M are masked
        const float4 t = load4(reinterpret_cast<const E*>(&u));
        const float v[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float r = m < M ? v[e] : 0.f;
          s1[b][e] += r;
          s2[b][e] = fmaf(r, r, s2[b][e]);
        }
      }
    }
  if (!DG && p.stats) {
    // sum over the 16 rows a 16-lane group holds (butterflies inside the group), then the two wavefronts that share
    // the columns through LDS in a fixed order: one partial per row tile
    __syncthreads();                     // the staging buffers are free
    float* red = reinterpret_cast<float*>(smem_raw);       // [2 (wm)][2 (sum, squares)][BN]
#pragma unroll
    for (int b = 0; b < T; ++b)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float a1 = s1[b][e], a2 = s2[b][e];
        a1 += dpp_move<0xB1>(a1); a1 += dpp_move<0x4E>(a1); a1 += dpp_move<0x141>(a1); a1 += dpp_move<0x140>(a1);
        a2 += dpp_move<0xB1>(a2); a2 += dpp_move<0x4E>(a2); a2 += dpp_move<0x141>(a2); a2 += dpp_move<0x140>(a2);
        if (l16 == 0) {
          const int col = wn * 16 * T + b * 16 + 4 * G + e;
          red[(wm * 2 + 0) * BN + col] = a1;
          red[(wm * 2 + 1) * BN + col] = a2;
        }
      }
    __syncthreads();
    for (int i = tid; i < 2 * BN; i += 256) {
      const int which = i / BN, col = i - which * BN;
      const int j = j0 + col;
      if (j < NC) p.stats[((size_t)it * 2 + which) * NC + j] = red[which * BN + col] + red[(2 + which) * BN + col];
    }
  }
}

// ---- host side ---------------------------------------------------------------------------------------------
struct DeepPlan { int S, T, itiles, jtiles; size_t lds; };

// rows M, reduction extent R, output columns NC
static bool deep_plan(int dt, size_t M, int R, int NC, bool dgrad, DeepPlan* d, bool sums = false) {
  // bfloat16: reductions of 192 and more as they come; shorter ones up to 32768 rows, but layers that widen them much there, whose time is the
  // output's.  us on the streaming kernels and here, forward 700 rows 960 -> 320 10.5 / 7.0, 2100 24 -> 144 6.3 / 2.9, 3136 160 -> 960 8.7 / 7.2, 6825 48 -> 288 5.7 / 5.0, 12544 40 -> 96 4.3 /
  // 3.8, 144 -> 64 6.2 / 4.2, 25088 96 -> 64 5.0 / 4.8; but 12544 64 -> 384 6.7 / 7.6, 25088 32 -> 192 5.4 / 7.5, 88 -> 528 14.8 / 16.3, 136 -> 816 26.4 / 36.4.
  // Data gradient 1568 rows of 960 -> 320 8.7 / 5.2, 2048 160 -> 960 9.9 / 6.2, 8192 96 -> 48 3.5 / 2.9, 25088 96 -> 64 4.7 / 4.1, 136 -> 816 27.5 / 24.5; but 20800
  // 96 -> 32 3.6 / 3.9, 25088 144 -> 32 4.4 / 4.8.
  // The streaming kernels take 32 reduction elements and 64 columns a step, a step here is 64 and a tile up to 160: where the layer is whole in the first
  // and has more than 4 M results, they are the faster ones from twice the width on.  These with some 3 us of the events around the launch: forward 8192 rows 96 -> 576 10.5 / 11.6, 160 -> 960 14.4 / 15.7, 16385
  // 160 -> 320 12.4 / 14.8, 25088 96 -> 288 11.9 / 14.3, 64 -> 192 9.3 / 10.0 (20480 9.2 / 8.3), 128 -> 256 12.6 / 13.5.  Data gradient (columns of 64, and a reduction of
  // one step or with half a step left over) 25088 rows 576 -> 96 16.6 / 19.7, 384 -> 96 13.5 / 16.5, 384 -> 64 12.1 / 13.4, 320 -> 160 14.2 / 16.1, 16385 576 -> 160 16.7 / 17.6; but
  // 768 -> 128 18.0 / 18.8 and 23.1 / 23.0, 528 -> 88 17.0 / 16.1, 720 -> 120 24.4 / 19.9, 480 -> 160 20.2 / 18.9.
  // fp32: everything that is not for the short kernel in front, up to 65536 rows, but forward layers that widen a short reduction, whose time is
  // the output's, and beyond 32768 rows reductions of few steps: forward 1568 rows 960 -> 160 18.9 / 12.9, 3136 960 -> 160 30.1 / 17.1, 6272 384 -> 96
  // 20.8 / 10.3, 12544 64 -> 384 13.8 / 13.6, 16384 192 -> 32 11.5 / 5.5, 50176 144 -> 32 17.9 / 16.3; but 8192 32 -> 192 4.8 / 5.1, 25088 64 -> 384 20.9 / 22.8,
  // 96 -> 576 37.3 / 37.9, 50176 32 -> 192 14.6 / 17.0, 100352 144 -> 32 33.8 / 34.3.  Data gradient 800 rows of 960 -> 320
  // 17.8 / 8.6, 6272 96 -> 576 20.8 / 12.3, 25088 69.0 / 35.2, 8192 48 -> 96 7.1 / 3.4, 50176 192 -> 64 21.3 / 20.5, 144 -> 32 13.0 / 13.1.  With the events' 3 us:
  // forward 50176 64 -> 64 12.8 / 13.9 (25088 9.5 / 9.3), 96 -> 96 24.1 / 25.3, data gradient 50176 192 -> 32 16.5 / 17.9, 65536 18.7 / 20.7, 96 -> 24 13.7 / 14.8.
  const bool many = M * (size_t)NC > ((size_t)4 << 20);
  if (M > 65536 || R > kDeepMaxR || R % 8 || NC % 8 || NC < 32) return false;
  if (dt == 0) {
    if (M <= 512 || R < 16) return false;
    if (!dgrad && ((M > 4096 && R < 64 && NC > 2 * R) || (M > 16384 && NC > R) || (M > 32768 && R <= 128 && NC > 32))) return false;
    if (dgrad && M > 32768 && R <= 32 && NC > R) return false;
  } else if (R < 192) {
    if (M <= 512 || M > 32768 || R < 16) return false;
    if (dgrad ? M > 16384 && R < 64 && NC > 2 * R : M > 8192 && NC > 3 * R) return false;
    if (many && NC >= 2 * R && (dgrad ? NC % 64 == 0 && (R == 64 || R % 64 == 32) : R % 32 == 0)) return false;
  } else if (M <= 512) {
    return false;
  }
  const int KS = dt == 0 ? 32 : 64, LD = dt == 0 ? 36 : 72, V = dt == 0 ? 4 : 8, es = dt == 0 ? 4 : 2;
  // The tile: a step of a block costs what it stages, S + T units of 4 KB (a trip through registers and LDS, in order; the products are a
  // fifth of it), and 1.4 times that if the block has its CU to itself; blocks beyond the 256 CUs take turns.  fp32: 256
  // cycles of products for each 32 x 32 results, which nothing else runs beside, some 60 for each unit staged, and 400 for the trip of a block that has its
  // CU to itself.  3136 rows, us, bfloat16:
  // 960 -> 160 forward 15.7 (2 x 5, 49 blocks), 12.3 (2 x 2, 147), 11.8 (1 x 3, 196), 10.4 (1 x 1, 490); its mirror, with residual, 13.5, 8.7, 8.5, 7.3;
  // 1280 -> 320 data gradient 16.1 (2 x 5, 98), 13.0 (2 x 3, 196), 11.3 (2 x 2, 245), 13.8 (1 x 1, 980); 320 -> 960 11.6 (2 x 5, 294), 8.9 (4 x 3, 250).
  // With sums, bfloat16: up to two.  What such a layer waits for is z, and of the larger tiles two blocks at most share a CU: width 1.4, batch 128, 4 steps
  // 26.92 ms with tiles of four, 26.85 without, recomputing at 224x224 11.48 / 11.47, units 15-18 batch 64 4.278 / 4.273, 161x193 8.12 / 8.12; 4 x 5 (one block) 25088 rows
  // 136 -> 816 67 us, 4 x 4 51, without sums 33.
  static const int kTiles[][2] = {{4, 5}, {4, 4}, {4, 3}, {4, 2}, {2, 3}, {2, 2}, {2, 1}, {1, 1}};
  int best = 0;
  for (const auto& st : kTiles) {
    const int S = st[0], T = st[1];
    const size_t itiles = (M + 32 * S - 1) / (32 * S), jtiles = (NC + 32 * T - 1) / (32 * T);
    if (itiles > kMaxPartials || (dt == 0 && S * T > 8) || (sums && dt && S == 4)) continue;      // (fp32: an accumulator more for every one)
    const size_t xs = (size_t)32 * S * LD, ys = dgrad ? (size_t)KS * (32 * T + V) : (size_t)32 * T * LD;
    const size_t lds = 2 * (xs + ys) * es + (dgrad ? 0 : 2 * (size_t)((R + KS - 1) / KS * KS) * sizeof(float));
    const int turns = (int)((itiles * jtiles + 255) / 256), alone = turns == 1 || 2 * lds > 160 * 1024;
    const int cost = dt == 0 ? turns * (256 * S * T + 60 * (S + T) + (alone ? 400 : 100)) : turns * (S + T) * (alone ? 7 : 5);
    if (best && cost >= best) continue;
    best = cost;
    const size_t red = (size_t)4 * 32 * T * sizeof(float);
    *d = DeepPlan{S, T, (int)itiles, (int)jtiles, lds > red ? lds : red};
  }
  return best > 0;
}

int pw_deep_ok(int dt, size_t M, int R, int NC, bool dgrad) {
  DeepPlan d;
  return deep_plan(dt, M, R, NC, dgrad, &d);
}

template <typename E, int S, int T>
static void deep_launch_mode(hipStream_t st, const DeepArgs& a, const DeepPlan& d, int mode) {
  const dim3 grid((unsigned)d.itiles * d.jtiles), block(256);
  switch (mode) {
    case DEEP_FWD: hipLaunchKernelGGL((pw_gemm_deep_k<E, S, T, DEEP_FWD>), grid, block, d.lds, st, a); break;
    case DEEP_FWD_VIEW: hipLaunchKernelGGL((pw_gemm_deep_k<E, S, T, DEEP_FWD_VIEW>), grid, block, d.lds, st, a); break;
    case DEEP_DGRAD: hipLaunchKernelGGL((pw_gemm_deep_k<E, S, T, DEEP_DGRAD>), grid, block, d.lds, st, a); break;
    case DEEP_DGRAD_GATED:
    case DEEP_DGRAD_SUMS:
      if constexpr (Deep<E>::F32 || S < 4) {               // deep_plan
        if (mode == DEEP_DGRAD_GATED) hipLaunchKernelGGL((pw_gemm_deep_k<E, S, T, DEEP_DGRAD_GATED>), grid, block, d.lds, st, a);
        else hipLaunchKernelGGL((pw_gemm_deep_k<E, S, T, DEEP_DGRAD_SUMS>), grid, block, d.lds, st, a);
      } else {
        launch_plan_failed("data gradient with sums: no such tile");
      }
      break;
    default: hipLaunchKernelGGL((pw_gemm_deep_k<E, S, T, DEEP_DGRAD_RES>), grid, block, d.lds, st, a); break;
  }
}

template <typename E>
static void deep_launch_tile(hipStream_t st, const DeepArgs& a, const DeepPlan& d, int mode) {
  switch (d.S * 10 + d.T) {
    case 11: deep_launch_mode<E, 1, 1>(st, a, d, mode); break;
    case 21: deep_launch_mode<E, 2, 1>(st, a, d, mode); break;
    case 22: deep_launch_mode<E, 2, 2>(st, a, d, mode); break;
    case 23: deep_launch_mode<E, 2, 3>(st, a, d, mode); break;
    case 42: deep_launch_mode<E, 4, 2>(st, a, d, mode); break;
    default:
      if constexpr (!Deep<E>::F32) {
        if (d.T == 3) deep_launch_mode<E, 4, 3>(st, a, d, mode);
        else if (d.T == 4) deep_launch_mode<E, 4, 4>(st, a, d, mode);
        else deep_launch_mode<E, 4, 5>(st, a, d, mode);
      }
  }
}

static void deep_launch(int dt, hipStream_t st, const DeepArgs& a, const DeepPlan& d, int mode) {
  if (dt == 0) deep_launch_tile<float>(st, a, d, mode);
  else deep_launch_tile<bf16_t>(st, a, d, mode);
}

static const char* deep_name(const DeepPlan& d) {
  switch (d.S * 10 + d.T) {
    case 11: return "deep 1x1";
    case 21: return "deep 2x1";
    case 22: return "deep 2x2";
    case 23: return "deep 2x3";
    case 42: return "deep 4x2";
    case 43: return "deep 4x3";
    case 44: return "deep 4x4";
    default: return "deep 4x5";
  }
}

// z[M][N] = A'[M][K] * W[N][K]^T; stats as in pw_fwd (P_out = partials written)
const char* pw_fwd_deep(int dt, hipStream_t st, HView av, const void* w, size_t M, int K, int N, void* z, float* stats, int* P_out) {
  DeepPlan d;
  if (!deep_plan(dt, M, K, N, false, &d)) { launch_plan_failed("long-reduction pointwise forward called for a shape it does not take"); return nullptr; }
  DeepArgs a{};
  a.x = av.z; a.y = w; a.scale = av.scale; a.shift = av.shift; a.act = av.act;
  a.out = z; a.stats = stats; a.M = (int)M; a.R = K; a.NC = N; a.jtiles = d.jtiles;
  if (P_out) *P_out = d.itiles;
  deep_launch(dt, st, a, d, av.scale ? DEEP_FWD_VIEW : DEEP_FWD);
  return deep_name(d);
}

int pw_deep_sums_ok(int dt, size_t M, int R, int NC) {
  DeepPlan d;
  return deep_plan(dt, M, R, NC, true, &d, true) && bn_left_sums_ok(M, NC, d.itiles);
}

// dA[M][K] = dZ[M][N] * W[N][K] (+ res); sums != nullptr: with the sums of dA and dA * of.z, dA gated by the activation that the view `of` has (P_out partials)
const char* pw_dgrad_deep(int dt, hipStream_t st, const void* dz, const void* w, const void* res, size_t M, int K, int N, void* dA, HView of, float* sums, int* P_out) {
  DeepPlan d;
  if (!deep_plan(dt, M, N, K, true, &d, sums != nullptr)) { launch_plan_failed("long-reduction pointwise data gradient called for a shape it does not take"); return nullptr; }
  DeepArgs a{};
  a.x = dz; a.y = w; a.res = res; a.out = dA;
  a.M = (int)M; a.R = N; a.NC = K; a.jtiles = d.jtiles;
  if (sums) {
    a.z = of.z; a.scale = of.scale; a.shift = of.shift; a.act = of.act; a.stats = sums;
    *P_out = d.itiles;
    deep_launch(dt, st, a, d, of.scale ? DEEP_DGRAD_GATED : DEEP_DGRAD_SUMS);
  } else {
    deep_launch(dt, st, a, d, res ? DEEP_DGRAD_RES : DEEP_DGRAD);
  }
  return deep_name(d);
}

}  // namespace ftp
