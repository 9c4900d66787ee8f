// MI355X (gfx950) kernels and C ABI of one Allegro layer around the tensor
// product.  What is computed is stated in include/allegro_layer.h.
//
// The dense contractions run in fp32 on the matrix cores: through split
// operands on v_mfma_f32_16x16x32_bf16 (mfma_split) or with
// v_mfma_f32_16x16x4_f32.  For one of the latter lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16], and accumulator register r of lane l holds
// D[4 (l / 16) + r][l % 16].  Over the steps of a sum, lane group l / 16
// either interleaves with the others (k = 4 s + l / 16) or owns a contiguous
// quarter of k, whichever keeps that kernel's LDS reads free of bank
// conflicts; A and B always use the same order, so every product pairs the
// same k.
//
//   row_gemm_kernel     C[E][N] = X[E][K] B[K][N], X staged in LDS, with an
//                       optional addend: w = h A and dh = dhm + dw A^T
//   latent_chain_kernel the latent update a = [h, s] B1, h' = h + SiLU(a) B2 or
//                       its VJP in one pass, both products in fp32 through
//                       split operands on the bf16 matrix cores
//   reduce_gemm_kernel  G[M][N] = sum_e P[e][M] Q[e][N] (dA, dB1, dB2):
//                       persistent workgroups with register accumulators,
//                       one partial per workgroup, then colsum_kernel
//   mix_kernel          per-irrep channel mixing V' = Mix_c T_c (forward) or
//                       dT = Mix_c^T dV' (backward), in fp32 through split
//                       operands on the bf16 matrix cores; each wave keeps
//                       rows of its irreps' Mix_c in registers
//   mix_wgrad_kernel    dMix_c = sum over edges and components of dV'_c T_c^T
//   colsum_kernel       fixed-order sum of the workgroups' partials
//
// Edge-major [E][U][d1] tiles are staged through LDS in a per-irrep column
// layout: column (e, m) of irrep c holds the U channels of component
// off(c) + m of edge e, columns padded so that the 64 lanes of an MFMA
// operand read hit distinct banks.  All reductions over edges have a fixed
// order and no atomics, so every output is bit-identical run to run.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "allegro_layer.h"
#include "device_common.hpp"
#include "plan.hpp"

namespace {

using namespace allegro_dev;
using allegro_internal::fail;

constexpr int kWave = 64;
constexpr int kThreads = 256;  // four waves per workgroup
constexpr int kU = 64;         // channels supported by the layer
constexpr int kBufferNonTemporal = 2;  // buffer access policy bit (streamed once)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ f32x4 mfma_16x16x4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// SiLU(a) = a / (1 + exp(-a)) and its derivative sigma(a) (1 + a (1 - sigma(a))).
__device__ __forceinline__ float silu(float a) { return a / (1.0f + expf(-a)); }
__device__ __forceinline__ float silu_grad(float a) {
  const float sg = 1.0f / (1.0f + expf(-a));
  return sg * (1.0f + a * (1.0f - sg));
}

// The x irreps of a plan: for l = 0..lmax, (l, natural parity) then, with
// full parity, (l, the other parity); sizes 2l + 1, concatenated.
template <int LMAX_, bool FULL>
struct XIrreps {
  static constexpr int LMAX = LMAX_;
  static constexpr int NX = FULL ? 2 * (LMAX_ + 1) : LMAX_ + 1;
  static constexpr int D1 = FULL ? 2 * (LMAX_ + 1) * (LMAX_ + 1) : (LMAX_ + 1) * (LMAX_ + 1);
  static constexpr int dim(int c) { return 2 * (FULL ? c / 2 : c) + 1; }
  static constexpr int off(int c) { return c == 0 ? 0 : off(c - 1) + dim(c - 1); }
};

// ------------------------------------------------------ split products
// fp32 products on the bf16 matrix cores (the three-way split of G. Henry, P. T.
// P. Tang, A. Heinecke, "Leveraging the bfloat16 artificial intelligence datatype
// for higher-precision computations", ARITH 2019).  x = h + m + l with h = bf16(x),
// m = bf16(x - h), l = x - h - m: 8 significant bits each, rounded to nearest,
// so the three hold all 24 bits of x exactly (both subtractions are exact).
// Of the nine products of two split operands the six of weight 2^-16 and more
// are summed (in fp32, by the matrix core), the small ones first; the three
// dropped are below 2^-26 of the product, a quarter of the rounding of one
// fp32 product.  The matrix core takes bf16 subnormals as zero, so both
// operands are scaled by kSplitScale first: the smallest part of any fp32
// value, 2^-149, is then a normal number.  The sum comes back through
// kSplitUnscale; what overflows for the scale (or is infinite to begin with)
// leaves a sum that is not finite, and the caller redoes it in fp32.
//
// The matrix core rounds its bf16 sums down, not to nearest: the values carry a
// mean error of about -1e-8 of their size, and every result here is later summed
// over edges (dB1's error rose from 5.1e-7 to 5.6e-7), where the mean grows with
// the count and the rest with its root.  So half of the sums are formed with the
// opposite sign.  latent_chain_kernel takes half of a sum's steps with negated
// weights into an accumulator of their own and subtracts it at the end;
// mix_kernel negates every other column, which are, as irreps have odd
// dimensions, every other edge of each component.
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

struct Split8 {
  bf16x8 h, m, l;
};

// The packed bf16 parts of two values.
__device__ __forceinline__ void split2(float x0, float x1, uint32_t &h, uint32_t &m, uint32_t &l) {
  h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x0, x1}, bf16x2));
  const f32x2 r = {x0 - __builtin_bit_cast(float, h << 16), x1 - __builtin_bit_cast(float, h & 0xffff0000u)};
  m = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
  const f32x2 q = {r.x - __builtin_bit_cast(float, m << 16), r.y - __builtin_bit_cast(float, m & 0xffff0000u)};
  l = __builtin_bit_cast(uint32_t, __builtin_convertvector(q, bf16x2));
}

__device__ __forceinline__ Split8 split8(const float (&x)[8], float scale = kSplitScale) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  u32x4 h, m, l;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t hb, mb, lb;
    split2(scale * x[2 * i], scale * x[2 * i + 1], hb, mb, lb);
    h[i] = hb;
    m[i] = mb;
    l[i] = lb;
  }
  return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

__device__ __forceinline__ f32x4 mfma_split(const Split8 &a, const Split8 &b, f32x4 c) {
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.l, b.h, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.l, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.m, b.m, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.m, b.h, c, 0, 0, 0);
  c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.m, c, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.h, b.h, c, 0, 0, 0);
}

// ------------------------------------------------------------- row GEMM
enum { kProNone = 0, kProSilu = 1 };   // elementwise step on the rows of reduce_gemm_kernel's P
enum { kEpiStore = 0, kEpiAdd = 1 };   // row_gemm_kernel's result, or with d added

struct RowGemmArgs {
  int64_t E;
  const float *x;  // [E][K]
  const float *b;  // B[k][n] = b[k * b_rs + n * b_cs]
  int b_rs, b_cs;
  const float *d;  // addend (kEpiAdd)
  float *c;
  int *ticket;     // set to zero for the mixing kernel launched after this one (may be null)
};

constexpr int kRowTile = 64;  // rows per workgroup tile

// Stages rows r0 .. r0 + 63 of x [E][KX] into columns col0 .. col0 + KX - 1 of
// an LDS tile (row stride XS), zero past the last row, with an optional
// elementwise prologue, in two halves, so that a tile's loads can be in flight
// while the previous tile is multiplied: the loads into registers, then the LDS
// writes.
template <int KX>
struct RowRegs {
  static constexpr int F4 = kRowTile * KX / 4, PER = (F4 + kThreads - 1) / kThreads;
  float4 v[PER];
  __device__ __forceinline__ void load(const float *__restrict__ x, int64_t r0, int rows, int tid) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int f = tid + kThreads * i, r = f / (KX / 4), k = 4 * (f % (KX / 4));
      v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (f < F4 && r < rows) v[i] = *reinterpret_cast<const float4 *>(x + (r0 + r) * KX + k);
    }
  }
  template <int PRO>
  __device__ __forceinline__ void put(float *xs, int XS, int col0, int tid) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int f = tid + kThreads * i, r = f / (KX / 4), k = 4 * (f % (KX / 4));
      if (f >= F4) continue;
      float4 u = v[i];
      if constexpr (PRO == kProSilu) {
        u.x = silu(u.x); u.y = silu(u.y); u.z = silu(u.z); u.w = silu(u.w);
      }
      *reinterpret_cast<float4 *>(xs + r * XS + col0 + k) = u;
    }
  }
};

// C[E][N] = X[E][K] B[K][N] over 64-row tiles.  Wave w owns the column tiles
// w + 4 j of every row tile and keeps their B operands in registers for the
// whole launch; A operands come from the LDS tile.  The products of the tile
// go back through LDS (over the X tile), so that the epilogue reads its addend
// and writes its output as whole rows, 16 bytes per lane and consecutive
// lanes along a row: written straight from the accumulators, each store
// instruction would cover 64-byte pieces of four rows.
template <int K, int N, int EPI>
__global__ __launch_bounds__(kThreads) void row_gemm_kernel(RowGemmArgs g) {
  constexpr int XS = K + 4;   // row stride: the 16 rows of an A read hit distinct banks
  constexpr int OS = N + 4;   // row stride of the product tile
  constexpr int NJ = N / 64;  // column tiles per wave
  constexpr int LDSF = kRowTile * (XS > OS ? XS : OS);
  constexpr int OF4 = kRowTile * N / 4, OPER = OF4 / kThreads;  // product float4 per thread
  static_assert(K % 16 == 0 && N % 64 == 0 && OF4 % kThreads == 0, "tile shape");
  __shared__ float4 xs4[LDSF / 4];
  float *xs = reinterpret_cast<float *>(xs4);
  const int tid = threadIdx.x, wave = tid / kWave, l = tid % kWave;
  if (g.ticket && blockIdx.x == 0 && tid == 0) *g.ticket = 0;
  // step s pairs k = 4 s + l / 16 in both operands
  float bf[NJ][K / 4];
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int s = 0; s < K / 4; ++s)
      bf[j][s] = g.b[(4 * s + l / 16) * g.b_rs + (16 * (wave + 4 * j) + l % 16) * g.b_cs];
  const int64_t n_tiles = (g.E + kRowTile - 1) / kRowTile;
  // the next tile's rows are loaded while this tile is multiplied
  RowRegs<K> xr;
  auto load = [&](int64_t t) {
    const int64_t r0 = t * kRowTile;
    xr.load(g.x, r0, int(g.E - r0 < kRowTile ? g.E - r0 : kRowTile), tid);
  };
  if (int64_t(blockIdx.x) < n_tiles) load(blockIdx.x);
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const int64_t r0 = t * kRowTile;
    const int rows = int(g.E - r0 < kRowTile ? g.E - r0 : kRowTile);
    xr.template put<kProNone>(xs, XS, 0, tid);
    lds_sync<4>();
    if (t + gridDim.x < n_tiles) load(t + gridDim.x);
    f32x4 acc[kRowTile / 16][NJ];
#pragma unroll
    for (int rt = 0; rt < kRowTile / 16; ++rt) {
      // with XS = 4 (mod 64) the 64 lanes of an A read hit distinct banks
      const float *xa = xs + (16 * rt + l % 16) * XS + l / 16;
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[rt][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int s = 0; s < K / 4; ++s) {
        const float a = xa[4 * s];
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[rt][j] = mfma_16x16x4(a, bf[j][s], acc[rt][j]);
      }
    }
    lds_sync<4>();  // every wave has read the X tile: its LDS takes the products
#pragma unroll
    for (int rt = 0; rt < kRowTile / 16; ++rt)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          xs[(16 * rt + 4 * (l / 16) + r) * OS + 16 * (wave + 4 * j) + l % 16] = acc[rt][j][r];
    lds_sync<4>();
    // epilogue by whole rows: float4 f = tid + 256 i is row f / (N / 4), columns 4 (f % (N / 4)) ..
    float4 dv[OPER];
    if constexpr (EPI == kEpiAdd) {
#pragma unroll
      for (int i = 0; i < OPER; ++i) {
        const int f = tid + kThreads * i, row = f / (N / 4), col = 4 * (f % (N / 4));
        dv[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row < rows) dv[i] = *reinterpret_cast<const float4 *>(g.d + (r0 + row) * N + col);
      }
    }
#pragma unroll
    for (int i = 0; i < OPER; ++i) {
      const int f = tid + kThreads * i, row = f / (N / 4), col = 4 * (f % (N / 4));
      if (row >= rows) continue;
      float4 v = *reinterpret_cast<const float4 *>(xs + row * OS + col);
      if constexpr (EPI == kEpiAdd) {
        v.x += dv[i].x; v.y += dv[i].y; v.z += dv[i].z; v.w += dv[i].w;
      }
      *reinterpret_cast<float4 *>(g.c + (r0 + row) * N + col) = v;
    }
    lds_sync<4>();  // the products are read: the next X tile may land
  }
}

// ---------------------------------------------------------- latent chain
// The two dense steps of the latent update, or of its VJP, in one pass:
//   forward   a = [h, s] B1,  c = h + SiLU(a) B2                (mid_out = a)
//   backward  da = (dh' B2^T) * SiLU'(a),  [c | c2] = [dh', 0] + da B1^T  (mid_out = da)
// X = [x1 | x2] is [E][K1], the middle [E][H], the result [E][N2].
struct ChainArgs {
  int64_t E;
  const float *x1, *x2;    // X = [x1 | x2], [E][K1A] and [E][K1B]
  const float *w1, *w2;    // W1[k][n] = w1[k * w1_rs + n * w1_cs], W2 likewise
  int w1_rs, w1_cs, w2_rs, w2_cs;
  const float *a;          // backward: the pre-activations [E][H]
  float *mid_out;          // [E][H]
  const float *add;        // [E][N2A], added to the first N2A columns of the result
  float *c, *c2;           // result: columns < N2A to c, the rest to c2
  int *ticket;             // set to zero for the mixing kernel launched after this one (may be null)
};

// B operands of CT = N / 16 column tiles of W [K][N] for 8 waves over a tile of
// 64 rows (four row tiles): wave w owns column tiles w + 8 i whole, and of the
// last four, if CT is not a multiple of eight, tile w % 4 for the row tiles
// 2 (w / 4) and + 1.
template <int K, int N>
struct ChainWeights {
  static constexpr int CT = N / 16, FULL = CT / 8, HALF = CT % 8 ? 1 : 0, OWN = FULL + HALF, KS = K / 32;
  static_assert(K % 32 == 0 && N % 64 == 0, "whole column tiles");
  Split8 w[OWN][KS];
  static __device__ __forceinline__ int tile(int i, int wave) { return i < FULL ? wave + 8 * i : 8 * FULL + wave % 4; }
  __device__ __forceinline__ void load(const float *__restrict__ p, int rs, int cs, int wave, int l) {
#pragma unroll
    for (int i = 0; i < OWN; ++i)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j)
          x[j] = p[(32 * ks + 8 * (l / 16) + j) * rs + (16 * tile(i, wave) + l % 16) * cs];
        // odd steps are negated and summed apart: see mfma_split
        w[i][ks] = split8(x, ks % 2 ? -kSplitScale : kSplitScale);
      }
  }
};

// The three bf16 parts of a [64][K] tile in LDS: part q of row r, column k at
// (q 64 + r) (K + 8) + k.  The row stride, 36, 68 and 100 words at K = 64, 128
// and 192, is 4 (mod 32): the 16-byte operand reads of 16 consecutive rows start
// in 16 distinct quads of banks.
template <int K>
struct ChainPlanes {
  static constexpr int STRIDE = K + 8, HALFS = 3 * 64 * STRIDE;  // HALFS: 16-bit elements
  static __device__ __forceinline__ void put(uint16_t *p, int row, int col, float4 v) {
    const float x[4] = {kSplitScale * v.x, kSplitScale * v.y, kSplitScale * v.z, kSplitScale * v.w};
    uint32_t h[2], m[2], lo[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) split2(x[2 * i], x[2 * i + 1], h[i], m[i], lo[i]);
    uint2 *d = reinterpret_cast<uint2 *>(p + row * STRIDE + col);
    d[0] = make_uint2(h[0], h[1]);
    d[64 * STRIDE / 4] = make_uint2(m[0], m[1]);
    d[2 * 64 * STRIDE / 4] = make_uint2(lo[0], lo[1]);
  }
  static __device__ __forceinline__ Split8 get(const uint16_t *p, int row, int col) {
    const bf16x8 *d = reinterpret_cast<const bf16x8 *>(p + row * STRIDE + col);
    return {d[0], d[64 * STRIDE / 8], d[2 * 64 * STRIDE / 8]};
  }
};

// out [64][OS] (fp32, LDS) = P W over the wave's column tiles; P are the planes
// of a [64][K] tile.  A row tile whose sum is not finite is redone in fp32 with
// P(row, k) and W(k, n) read through the callbacks.
template <int K, int N, class PElem, class WElem>
__device__ __forceinline__ void chain_gemm(const uint16_t *planes, const ChainWeights<K, N> &w, float *out, int OS,
                                           int wave, int l, PElem p_elem, WElem w_elem) {
  using W = ChainWeights<K, N>;
#pragma unroll
  for (int i = 0; i < W::OWN; ++i) {
    const int rts = i < W::FULL ? 4 : 2, rt0 = i < W::FULL ? 0 : 2 * (wave / 4), col = 16 * W::tile(i, wave) + l % 16;
#pragma unroll
    for (int q = 0; q < rts; ++q) {
      __builtin_amdgcn_sched_barrier(0);  // one row tile's operands at a time
      const int rt = rt0 + q;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f}, neg = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < W::KS; ++ks) {
        f32x4 &d = ks % 2 ? neg : acc;
        d = mfma_split(ChainPlanes<K>::get(planes, 16 * rt + l % 16, 32 * ks + 8 * (l / 16)), w.w[i][ks], d);
      }
      acc -= neg;
      float bad = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) bad = __builtin_fmaf(acc[r], 0.f, bad);
      acc *= kSplitUnscale;
      if (__any(bad != bad)) {
        acc = f32x4{0.f, 0.f, 0.f, 0.f};
        int lane = l;
        asm volatile("" : "+v"(lane));  // keeps these addresses out of the loop's registers
        const int n = 16 * W::tile(i, wave) + lane % 16;
#pragma unroll 1
        for (int k = lane / 16; k < K; k += 4) acc = mfma_16x16x4(p_elem(16 * rt + lane % 16, k), w_elem(k, n), acc);
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(16 * rt + 4 * (l / 16) + r) * OS + col] = acc[r];
    }
  }
}

constexpr int kChainThreads = 512, kChainRows = 64;

// One workgroup of 8 waves per compute unit over 64-row tiles; both weight
// matrices stay in registers, split (mfma_split).  Per tile: the rows of X,
// loaded one tile ahead, go to LDS as bf16 planes; first product to an fp32
// tile; middle step by whole rows (SiLU or its gradient, mid_out written, the
// middle's planes over those of X); second product; result written by whole
// rows.  The middle never returns from memory, and the matrix instructions run
// at the bf16 rate: at L = 64, H = 128 and 523,599 edges (0.67 and 0.94 GB)
// two row GEMMs on the fp32 matrix cores took 362 us forward and 461 backward
// in the same run, this 239 and 278 (2.8 and 3.4 TB/s; what is left is the
// tile's serial phases, four barriers with one workgroup on a unit).
template <int K1A, int K1B, int H, int N2, int N2A, bool BWD>
__global__ __launch_bounds__(kChainThreads) void latent_chain_kernel(ChainArgs g) {
  constexpr int K1 = K1A + K1B, T = kChainThreads, R = kChainRows;
  constexpr int PH = ChainPlanes<K1>::HALFS > ChainPlanes<H>::HALFS ? ChainPlanes<K1>::HALFS : ChainPlanes<H>::HALFS;
  constexpr int MS = H + 4, OS = N2 + 4;  // row strides of the fp32 tiles
  __shared__ uint4 planes4[PH / 8];
  __shared__ float4 mid4[R * MS / 4], out4[R * OS / 4];
  uint16_t *planes = reinterpret_cast<uint16_t *>(planes4);
  float *mid = reinterpret_cast<float *>(mid4), *out = reinterpret_cast<float *>(out4);
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid / kWave), l = tid % kWave;
  if (g.ticket && blockIdx.x == 0 && tid == 0) *g.ticket = 0;
  ChainWeights<K1, H> w1;
  ChainWeights<H, N2> w2;
  w1.load(g.w1, g.w1_rs, g.w1_cs, wave, l);
  w2.load(g.w2, g.w2_rs, g.w2_cs, wave, l);
  const int64_t n_tiles = (g.E + R - 1) / R;
  // float4 f = tid + 512 i of a [64][W] tile: row f / (W / 4), columns 4 (f % (W / 4)) ..
  constexpr int XP = R * K1 / 4 / T, MP = R * H / 4 / T, OP = R * N2 / 4 / T;
  static_assert(R * K1A / 4 % T == 0 && R * K1B / 4 % T == 0, "whole sources per thread");
  // The addend is on its way during the second product and the backward's a a
  // tile ahead, unless the result is 192 wide, where registers run out.
  constexpr bool EARLY = OP < 6;
  float4 xv[XP], av[BWD ? MP : 1];
  // the rows of tile t of an [E][width] tensor, as far as it has any (accesses
  // past the range read zeros and are dropped); within it float4 f sits at byte 16 f
  auto rows_of = [&](const float *p, int width, int64_t t) {
    const int64_t left = g.E - t * R;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(p + t * R * width), short(0),
                                             int(left < R ? left : R) * width * 4, 0x00020000);
  };
  // (the whole offset goes in voff: the scalar offset is not part of the range check)
  auto load4 = [&](__amdgpu_buffer_rsrc_t r, int voff) {
    const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, 0, 0));
    return make_float4(v.x, v.y, v.z, v.w);
  };
  auto store4 = [&](__amdgpu_buffer_rsrc_t r, int voff, float4 v) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{v.x, v.y, v.z, v.w}), r, voff, 0, 0);
  };
  auto load = [&](int64_t t) {
    constexpr int A = R * K1A / 4 / T;
    const auto r1 = rows_of(g.x1, K1A, t);
#pragma unroll
    for (int i = 0; i < A; ++i) xv[i] = load4(r1, 16 * (tid + T * i));
    if constexpr (K1B > 0) {
      const auto r2 = rows_of(g.x2, K1B, t);
#pragma unroll
      for (int i = A; i < XP; ++i) xv[i] = load4(r2, 16 * (tid + T * (i - A)));
    }
  };
  auto load_a = [&](int64_t t) {
    const auto r = rows_of(g.a, H, t);
#pragma unroll
    for (int i = 0; i < MP; ++i) av[i] = load4(r, 16 * (tid + T * i));
  };
  if (int64_t(blockIdx.x) < n_tiles) {
    load(blockIdx.x);
    if constexpr (BWD && EARLY) load_a(blockIdx.x);
  }
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const int64_t r0 = t * R;
    const int rows = int(g.E - r0 < R ? g.E - r0 : R);
#pragma unroll
    for (int i = 0; i < XP; ++i) {
      constexpr int A = R * K1A / 4 / T;
      const int f = tid + T * (i < A ? i : i - A), W4 = (i < A ? K1A : K1B) / 4;
      ChainPlanes<K1>::put(planes, f / W4, (i < A ? 0 : K1A) + 4 * (f % W4), xv[i]);
    }
    lds_sync<8>();
    if constexpr (BWD && !EARLY) load_a(t);
    if (t + gridDim.x < n_tiles) load(t + gridDim.x);
    chain_gemm<K1, H>(planes, w1, mid, MS, wave, l,
                      [&](int row, int k) {
                        if (row >= rows) return 0.f;
                        return k < K1A ? g.x1[(r0 + row) * K1A + k] : g.x2[(r0 + row) * K1B + (k - K1A)];
                      },
                      [&](int k, int n) { return g.w1[k * g.w1_rs + n * g.w1_cs]; });
    lds_sync<8>();  // the first product is there, the planes of X have been read
    const auto rm = rows_of(g.mid_out, H, t);
#pragma unroll
    for (int i = 0; i < MP; ++i) {
      const int f = tid + T * i, row = f / (H / 4), col = 4 * (f % (H / 4));
      float4 *m = reinterpret_cast<float4 *>(mid + row * MS + col);
      float4 v = *m, keep;
      if constexpr (BWD) {
        v.x *= silu_grad(av[i].x); v.y *= silu_grad(av[i].y); v.z *= silu_grad(av[i].z); v.w *= silu_grad(av[i].w);
        keep = v;
      } else {
        keep = v;
        v.x = silu(v.x); v.y = silu(v.y); v.z = silu(v.z); v.w = silu(v.w);
      }
      store4(rm, 16 * (tid + T * i), keep);
      *m = v;  // for a product that has to be redone in fp32
      ChainPlanes<H>::put(planes, row, col, v);
    }
    if constexpr (BWD && EARLY) {
      if (t + gridDim.x < n_tiles) load_a(t + gridDim.x);
    }
    float4 dv[OP];
    auto load_add = [&] {
      const auto r = rows_of(g.add, N2A, t);
#pragma unroll
      for (int i = 0; i < OP; ++i) {
        const int f = tid + T * i, row = f / (N2 / 4), col = 4 * (f % (N2 / 4));
        dv[i] = load4(r, col < N2A ? 4 * (row * N2A + col) : 4 * R * N2A);
      }
    };
    if constexpr (EARLY) load_add();
    lds_sync<8>();
    chain_gemm<H, N2>(planes, w2, out, OS, wave, l, [&](int row, int k) { return mid[row * MS + k]; },
                      [&](int k, int n) { return g.w2[k * g.w2_rs + n * g.w2_cs]; });
    if constexpr (!EARLY) load_add();
    lds_sync<8>();  // the result is there, the planes are free for the next tile
    const auto rc = rows_of(g.c, N2A, t), rc2 = rows_of(N2 > N2A ? g.c2 : g.c, N2 > N2A ? N2 - N2A : N2A, t);
#pragma unroll
    for (int i = 0; i < OP; ++i) {
      const int f = tid + T * i, row = f / (N2 / 4), col = 4 * (f % (N2 / 4));
      const float4 p = *reinterpret_cast<const float4 *>(out + row * OS + col);
      const float4 v = make_float4(p.x + dv[i].x, p.y + dv[i].y, p.z + dv[i].z, p.w + dv[i].w);
      if (N2 == N2A || col < N2A) store4(rc, 4 * (row * N2A + col), v);
      else store4(rc2, 4 * (row * (N2 - N2A) + col - N2A), v);
    }
  }
}

// ---------------------------------------------------------- reduce GEMM
constexpr int kRedTile = 64;  // edges per step

template <int M1, int M2, int N, int PRO>
__global__ __launch_bounds__(kThreads) void reduce_gemm_kernel(int64_t E, const float *__restrict__ p1,
                                                               const float *__restrict__ p2,
                                                               const float *__restrict__ q,
                                                               float *__restrict__ part) {
  constexpr int M = M1 + M2, PS = M + 16, QS = N + 16;  // strides = 16 (mod 64): conflict-free operand reads
  constexpr int MT = M / 16, NJ = N / 64;  // wave w owns column tiles nt = w + 4 j (j < NJ) of every row tile
  static_assert(M1 % 16 == 0 && M2 % 16 == 0 && N % 64 == 0, "tile shape");
  __shared__ float4 ps4[kRedTile * PS / 4], qs4[kRedTile * QS / 4];
  float *ps = reinterpret_cast<float *>(ps4), *qs = reinterpret_cast<float *>(qs4);
  const int tid = threadIdx.x, wave = tid / kWave, l = tid % kWave;
  f32x4 acc[MT][NJ];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[mt][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int64_t n_tiles = (E + kRedTile - 1) / kRedTile;
  static_assert(kRedTile == kRowTile, "tiles staged by RowRegs");
  // the next tile's loads are issued before this tile's products, into the
  // registers this tile's rows have just left
  RowRegs<M1> r1;
  RowRegs<(M2 > 0 ? M2 : 4)> r2;
  RowRegs<N> rq;
  auto load = [&](int64_t t) {
    const int64_t r0 = t * kRedTile;
    const int rows = int(E - r0 < kRedTile ? E - r0 : kRedTile);
    r1.load(p1, r0, rows, tid);
    if constexpr (M2 > 0) r2.load(p2, r0, rows, tid);
    rq.load(q, r0, rows, tid);
  };
  if (int64_t(blockIdx.x) < n_tiles) load(blockIdx.x);
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    r1.template put<PRO>(ps, PS, 0, tid);
    if constexpr (M2 > 0) r2.template put<kProNone>(ps, PS, M1, tid);
    rq.template put<kProNone>(qs, QS, 0, tid);
    lds_sync<4>();
    if (t + gridDim.x < n_tiles) load(t + gridDim.x);
    // the sum runs over the tile's edges: step s pairs edge 4 s + l / 16
    const float *pa = ps + (l / 16) * PS + l % 16;
    const float *qb = qs + (l / 16) * QS + 16 * wave + l % 16;
#pragma unroll 2
    for (int s = 0; s < kRedTile / 4; ++s) {
      float a[MT], b[NJ];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) a[mt] = pa[4 * s * PS + 16 * mt];
#pragma unroll
      for (int j = 0; j < NJ; ++j) b[j] = qb[4 * s * QS + 64 * j];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[mt][j] = mfma_16x16x4(a[mt], b[j], acc[mt][j]);
    }
    lds_sync<4>();
  }
  float *out = part + int64_t(blockIdx.x) * M * N;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(16 * mt + 4 * (l / 16) + r) * N + 16 * (wave + 4 * j) + l % 16] = acc[mt][j][r];
}

// out[c] = sum over r of part[r][c], in a fixed order: a block owns 16
// columns; thread (g, c) sums rows g, g + 16, g + 32, ... with four
// accumulators, then the 16 row groups are added in order.
constexpr int kColsumCols = 16, kColsumGroups = 16;

__global__ __launch_bounds__(256) void colsum_kernel(int R, int C, const float *__restrict__ part,
                                                     float *__restrict__ out) {
  __shared__ float sums[kColsumGroups][kColsumCols];
  const int cl = int(threadIdx.x) % kColsumCols, g = int(threadIdx.x) / kColsumCols;
  const int c = int(blockIdx.x) * kColsumCols + cl;
  float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
  if (c < C) {
    int r = g;
    constexpr int S = kColsumGroups;
    for (; r + 3 * S < R; r += 4 * S) {
      a0 += part[int64_t(r) * C + c];
      a1 += part[int64_t(r + S) * C + c];
      a2 += part[int64_t(r + 2 * S) * C + c];
      a3 += part[int64_t(r + 3 * S) * C + c];
    }
    for (; r < R; r += S) a0 += part[int64_t(r) * C + c];
  }
  sums[g][cl] = (a0 + a1) + (a2 + a3);
  __syncthreads();
  if (g == 0 && c < C) {
    float a = sums[0][cl];
    for (int k = 1; k < kColsumGroups; ++k) a += sums[k][cl];
    out[c] = a;
  }
}

// ------------------------------------------------------------ mixing
// LDS column index of component k of edge e in a tile of ne_tile edges.
template <class X>
__device__ __forceinline__ void component_column(int k, int ne_tile, int &col0, int &dim) {
  int c = 0;
#pragma unroll
  for (int i = 1; i < X::NX; ++i) c = k >= X::off(i) ? i : c;
  int o = 0, d = 1;
#pragma unroll
  for (int i = 0; i < X::NX; ++i)
    if (i == c) { o = X::off(i); d = X::dim(i); }
  col0 = ne_tile * o + (k - o);
  dim = d;
}

// Column stride (floats): 68 = 4 (mod 64), so the 16-byte accesses of one
// channel quad in 16 consecutive columns start in distinct bank quads.
constexpr int kMixCS = kU + 4;
constexpr int kMixComputeWaves = 8, kMixMemoryWaves = 4;
constexpr int kMixThreads = kWave * (kMixComputeWaves + kMixMemoryWaves);

// Channel at position p of a column: positions 4 u .. 4 u + 3 hold channels u,
// u + 16, u + 32 and u + 48, so that a memory thread moves four channels of a
// component as one 16-byte LDS access while a wave's global accesses cover
// consecutive rows.
__device__ __forceinline__ constexpr int mix_channel(int p) { return 16 * (p & 3) + (p >> 2); }

// Per-irrep channel mixing, software-pipelined over two LDS tile buffers.
// Waves 0-7 (compute) run the matrix-core products on one buffer while waves
// 8-11 (memory) store the previous tile's results from the other buffer and
// refill it with the next tile.  Per tile the two roles meet at two workgroup
// barriers: after the first the compute waves write their results into their
// buffer in place, after the second the buffers swap.  Both roles run the same
// tile sequence, so their barrier counts match.
//
// The tiles of a workgroup: the first three by its index, the rest in the order
// in which the workgroups of the whole device come to ask (ticket, zero before
// the launch), so that at any time they work on neighbouring tiles.  With a
// fixed stride per workgroup they drift apart (in a copy kernel with this tile
// size by up to 22 tiles), and HBM serves the widely spread streams at 5.4-5.7
// TB/s where the compact ones reach 6.8.  The first compute wave takes tile
// p + 3 during period p and leaves it at order[(p + 3) % 4] before B2.
//
// A compute wave owns the irreps of one pair of orders (l = 0 with 3, 1 with 2)
// at one parity, 8 of lmax 3's 32 components each, and 16 RT of the output
// channels; it holds its rows of their Mix matrices in registers, split into
// three bf16 parts (mfma_split).  A column is then read by 4 / RT waves
// instead of by all, which pays for splitting it on the way (5 vector
// operations a value), and the fp32 matrix instructions that set this kernel's
// pace (20 column tiles x 16 steps x 32 cycles per 8 edges and SIMD at lmax 3)
// become 5 x 24 x 2 x 16.  Bound now by HBM: with the products skipped the
// kernel takes as long.  Measured at lmax 3, full parity, 523,599 edges (8.6
// GB): fp32 products in fixed order 2.04 ms; these products 1.65 ms; tiles in
// order of arrival 1.37 ms (6.3 TB/s).  lmax 2, 206,624 edges: 478, 357 (14
// edges a tile instead of 8), 305 us.
template <class X>
struct MixTile {
  static constexpr int U = kU, D1 = X::D1, NX = X::NX, CS = kMixCS;
  // Edges per tile: about the 64 KB a compute unit must have in flight (at lmax 2
  // 8 edges, 36 KB, left it short of loads), and 16 where that fills the column tiles.
  static constexpr int NE = D1 == 32 ? 8 : D1 == 18 ? 14 : D1 >= 9 ? 16 : 32;
  static constexpr int COLS = NE * D1;
  static constexpr int BUF = (COLS + 16) * CS;  // +16 columns: the last irrep's padded column tile
  static constexpr int VW = D1 % 4 == 0 ? 4 : D1 % 2 == 0 ? 2 : 1;  // components per global access
  static constexpr int CH = D1 / VW;                                // accesses per row
  // memory task: VW components of the four channels u, u + 16, u + 32, u + 48 of an edge
  static constexpr int TASKS = NE * 16 * CH, PER = (TASKS + kWave * kMixMemoryWaves - 1) / (kWave * kMixMemoryWaves);
  static constexpr int PARITIES = X::NX > X::LMAX + 1 ? 2 : 1;
  static constexpr int PAIRS = X::LMAX == 1 ? 1 : 2;
  // row splits: the compute waves over the irrep groups, at least 16 channels each
  static constexpr int RS = PARITIES * PAIRS == 4 ? 2 : 4, RT = 4 / RS;
  static constexpr int BUSY = PARITIES * PAIRS * RS;
  // the two orders of pair i (-1: none)
  static constexpr int la(int i) { return X::LMAX == 2 && i == 1 ? 2 : i; }
  static constexpr int lb(int i) { return X::LMAX == 3 ? 3 - i : X::LMAX == 2 && i == 1 ? -1 : 1; }
  static constexpr int nct(int l) { return l < 0 ? 0 : (NE * (2 * l + 1) + 15) / 16; }  // column tiles
  static_assert(BUSY <= kMixComputeWaves, "compute waves");
};

// v, negated in odd columns.  A column's reads start at a multiple of 4 floats
// whose bit 2 is the column's lowest (kMixCS = 68, the lane group adds 16): made
// at each use from the offset at hand, since a register kept for it would spill.
__device__ __forceinline__ float column_sign(int rd, float v) {
  float r;
  asm volatile("v_lshl_or_b32 %0, %1, 29, %2" : "=v"(r) : "v"(rd), "s"(v));
  return r;
}

template <class X, bool BWD, int LA, int LB>
__device__ __forceinline__ void mix_compute_waves(int par, int rs, int64_t n_tiles, const float *__restrict__ mix,
                                                  float *lds, int *order, int *__restrict__ ticket) {
  using M = MixTile<X>;
  constexpr int U = M::U, CS = M::CS, NE = M::NE, RT = M::RT, NS = LB < 0 ? 1 : 2;
  constexpr int TA = M::nct(LA), NT = TA + M::nct(LB);  // column tiles of the first irrep, of both
  int l = threadIdx.x % kWave;
  asm volatile("" : "+v"(l));  // nothing derived from it is shared, and held, across the pairs' code
  const int g = l / 16, q = l % 16;
  const float scale = q % 2 ? -kSplitScale : kSplitScale;  // odd columns have the opposite sign: see mfma_split
  // The irreps, and the lane's LDS offsets in a buffer of its reads (rd) and
  // writes (wr) in their first column tile; opaque, so that the tiles' addresses
  // are immediate offsets from these and not a register each.
  const int cs[2] = {M::PARITIES * LA + par, M::PARITIES * (LB < 0 ? 0 : LB) + par};
  int rd[2], wr[2];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    constexpr int lo[2] = {LA, LB};
    // the components before irrep (l, par): l^2 of each parity, then the other parity of l
    const int col = NE * (M::PARITIES * lo[s] * lo[s] + par * (2 * lo[s] + 1)) + q;
    rd[s] = col * CS + 16 * g;
    wr[s] = col * CS + 16 * RT * rs + 4 * g;
    asm volatile("" : "+v"(rd[s]), "+v"(wr[s]));
  }
  // element (row position pr, reduction position pk) of Mix_c, transposed for the backward
  auto elem = [&](int c, int pr, int pk) {
    const int r = mix_channel(pr), k = mix_channel(pk);
    return BWD ? mix[(c * U + k) * U + r] : mix[(c * U + r) * U + k];
  };
  // step ks of lane group g covers positions 16 g + 8 ks .. + 7
  Split8 A[NS][RT][2];
#pragma unroll
  for (int s = 0; s < NS; ++s)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = elem(cs[s], 16 * (RT * rs + rt) + q, 16 * g + 8 * ks + j);
        A[s][rt][ks] = split8(x);
      }
  lds_sync<12>();  // the first tile is in buffer 0
  const bool taker = LA == 0 && par == 0 && rs == 0;
  for (int p = 0; __builtin_amdgcn_readfirstlane(order[p & 3]) < n_tiles; ++p) {
    int tile = 0;
    if (taker && l == 0) tile = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    float *b = lds + (p & 1) * M::BUF;
    f32x4 acc[NT][RT];
    float bad = 0.f;  // becomes NaN if a product is not finite
    static_for<0, NT>([&](auto it) {
      constexpr int i = decltype(it)::value, s = i < TA ? 0 : 1, ct = i < TA ? i : i - TA;
      constexpr int nq = NE * (2 * (s == 0 ? LA : LB) + 1);
      const float4 *bp = reinterpret_cast<const float4 *>(b + rd[s] + 16 * ct * CS);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) acc[i][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const float4 u = bp[2 * ks], v = bp[2 * ks + 1];
        const float x[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
        const Split8 B = split8(x, scale);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[i][rt] = mfma_split(A[s][rt][ks], B, acc[i][rt]);
      }
      if (16 * ct + q < nq) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int r = 0; r < 4; ++r) bad = __builtin_fmaf(acc[i][rt][r], 0.f, bad);
      }
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][rt][r] *= kSplitUnscale;
    });
    if (__any(bad != bad)) {
      // An infinity (or a value or sum too large for the scale) has left inf - inf:
      // redo the wave's products in fp32, which carries it through as it is.  (The
      // opaque lane index keeps these addresses out of the loop's registers.)
      int lane = l;
      asm volatile("" : "+v"(lane));
      const int go = lane / 16, qo = lane % 16;
      static_for<0, NT>([&](auto it) {
        constexpr int i = decltype(it)::value, s = i < TA ? 0 : 1, ct = i < TA ? i : i - TA;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          f32x4 a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
          for (int k = 0; k < 16; ++k)
            a = mfma_16x16x4(elem(cs[s], 16 * (RT * rs + rt) + qo, 16 * go + k),
                             b[rd[s] + 16 * ct * CS + k], a);
          acc[i][rt] = a * column_sign(rd[s], 1.f);
        }
      });
    }
    lds_sync<12>();  // B1: every compute wave has read the tile
    static_for<0, NT>([&](auto it) {
      constexpr int i = decltype(it)::value, s = i < TA ? 0 : 1, ct = i < TA ? i : i - TA;
      constexpr int nq = NE * (2 * (s == 0 ? LA : LB) + 1);
      if (16 * ct + q < nq) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          f32x4 v = acc[i][rt] * column_sign(rd[s], 1.f);
          // the 0e irrep also has the gradient of s: [edge][position] behind the tile buffers
          if (BWD && LA == 0 && s == 0 && par == 0)
            v += *reinterpret_cast<const f32x4 *>(lds + 2 * M::BUF + (16 * ct + q) * U + 16 * (RT * rs + rt) + 4 * g);
          *reinterpret_cast<f32x4 *>(b + wr[s] + 16 * ct * CS + 16 * rt) = v;
        }
      }
    });
    if (taker && l == 0) order[(p + 3) & 3] = 3 * int(gridDim.x) + tile;
    lds_sync<12>();  // B2: results are in the buffer
  }
}

template <class X, bool BWD>
__device__ __forceinline__ void mix_compute_role(int64_t n_tiles, const float *__restrict__ mix, float *lds,
                                                 int *order, int *__restrict__ ticket) {
  using M = MixTile<X>;
  // wave-uniform: row split, parity, pair of orders
  const int w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
  const int rs = w % M::RS, par = (w / M::RS) % M::PARITIES, pair = w / (M::RS * M::PARITIES);
  if (w >= M::BUSY) {  // no irreps left for this wave: it only keeps the barrier count
    lds_sync<12>();
    for (int p = 0; __builtin_amdgcn_readfirstlane(order[p & 3]) < n_tiles; ++p) {
      lds_sync<12>();
      lds_sync<12>();
    }
  } else if (pair == 0) {
    mix_compute_waves<X, BWD, M::la(0), M::lb(0)>(par, rs, n_tiles, mix, lds, order, ticket);
  } else if constexpr (M::PAIRS > 1) {
    mix_compute_waves<X, BWD, M::la(1), M::lb(1)>(par, rs, n_tiles, mix, lds, order, ticket);
  }
}

// VW consecutive floats by buffer access: past the descriptor's range loads
// give zeros and stores are dropped.
template <int VW>
using FloatVec = float __attribute__((ext_vector_type(VW)));

template <int VW>
__device__ __forceinline__ FloatVec<VW> buffer_load_f(__amdgpu_buffer_rsrc_t r, int off) {
  using V = FloatVec<VW>;
  if constexpr (VW == 4) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kBufferNonTemporal));
  else if constexpr (VW == 2) return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kBufferNonTemporal));
  else return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kBufferNonTemporal));
}

template <int VW>
__device__ __forceinline__ void buffer_store_f(__amdgpu_buffer_rsrc_t r, int off, FloatVec<VW> v) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  if constexpr (VW == 4)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, off, 0, kBufferNonTemporal);
  else if constexpr (VW == 2)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, kBufferNonTemporal);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, kBufferNonTemporal);
}

template <class X, bool BWD>
__device__ __forceinline__ void mix_memory_role(int64_t E, int64_t n_tiles, const float *__restrict__ src,
                                                const float *__restrict__ ds, float *__restrict__ dst,
                                                float *__restrict__ s_out, float *lds, const int *order) {
  using M = MixTile<X>;
  constexpr int U = M::U, D1 = M::D1, NE = M::NE, PER = M::PER, VW = M::VW, CH = M::CH;
  constexpr int THREADS = kWave * kMixMemoryWaves;
  const int mt = int(threadIdx.x) - kWave * kMixComputeWaves;
  // Task j of the thread: components VW b .. of channels u + 16 i (i = 0..3) of
  // edge e, task index (e 16 + u) CH + b = mt + 256 j: for one i consecutive
  // lanes cover consecutive bytes.  In LDS the four channels of a component
  // are one 16-byte access at addr.
  int off[PER], addr[PER][VW];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int task = mt + THREADS * j, bch = task % CH, u = (task / CH) % 16, e = task / (16 * CH);
    off[j] = 4 * ((e * U + u) * D1 + VW * bch);  // bytes within the tile; e >= NE lies past its range
#pragma unroll
    for (int q = 0; q < VW; ++q) {
      int col0, dim;
      component_column<X>(VW * bch + q, NE, col0, dim);
      addr[j][q] = task < M::TASKS ? (col0 + e * dim) * M::CS + 4 * u : 0;
    }
  }
  // tile t of an [E][U][width] tensor, as far as it has edges; empty for no tile
  auto rsrc = [&](const float *base, int width, int64_t t) {
    const bool valid = t >= 0 && t < n_tiles;
    const int64_t e0 = valid ? t * NE : 0;
    const int ne = valid ? int(E - e0 < NE ? E - e0 : NE) : 0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base + e0 * U * width), short(0),
                                             ne * U * width * 4, 0x00020000);
  };
  // The 0e component has tensors of its own, s (forward, out) and ds (backward,
  // in), both [E][U]: item k of the thread is channels u + 16 i of edge e, index
  // 16 e + u = mt + 256 k.
  constexpr int SPER = (NE * 16 + THREADS - 1) / THREADS;
  auto has_item = [&](int k) { return NE * 16 % THREADS == 0 || mt + THREADS * k < NE * 16; };
  auto item_off = [&](int k) { return 4 * ((mt / 16 + THREADS / 16 * k) * U + mt % 16); };
  FloatVec<VW> v[PER][4];
  f32x4 dsv[SPER];  // backward: ds of the next tile
  auto load = [&](__amdgpu_buffer_rsrc_t r, int j) {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[j][i] = buffer_load_f<VW>(r, off[j] + i * 64 * D1);
  };
  auto load_ds = [&](int64_t t) {
    const auto r = rsrc(ds, 1, t);
#pragma unroll
    for (int k = 0; k < SPER; ++k)
#pragma unroll
      for (int i = 0; i < 4; ++i) dsv[k][i] = buffer_load_f<1>(r, item_off(k) + 64 * i)[0];
  };
  auto put_ds = [&] {
#pragma unroll
    for (int k = 0; k < SPER; ++k)
      if (has_item(k)) reinterpret_cast<f32x4 *>(lds + 2 * M::BUF)[mt + THREADS * k] = dsv[k];
  };
  // s[e][u] = T[e][u][0]: irrep 0 (0e) has one component, so its column is e
  auto store_s = [&](int64_t t, const float *b) {
    const auto r = rsrc(s_out, 1, t);
#pragma unroll
    for (int k = 0; k < SPER; ++k) {
      if (!has_item(k)) continue;
      const f32x4 x = *reinterpret_cast<const f32x4 *>(b + (mt / 16 + THREADS / 16 * k) * M::CS + 4 * (mt % 16));
#pragma unroll
      for (int i = 0; i < 4; ++i) buffer_store_f<1>(r, item_off(k) + 64 * i, FloatVec<1>{x[i]});
    }
  };
  auto put = [&](float *b, int j) {
    // The task's registers as the loads left them: without this the transposing
    // moves are made at the end of the period before, and wait for the loads there.
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if constexpr (VW == 1) {
        float x = v[j][i][0];
        asm volatile("" : "+v"(x));
        v[j][i][0] = x;
      } else {
        asm volatile("" : "+v"(v[j][i]));
      }
    }
    if (M::TASKS % THREADS != 0 && mt + THREADS * j >= M::TASKS) return;
#pragma unroll
    for (int q = 0; q < VW; ++q)
      *reinterpret_cast<f32x4 *>(b + addr[j][q]) = f32x4{v[j][0][q], v[j][1][q], v[j][2][q], v[j][3][q]};
  };
  auto store = [&](int64_t t, const float *b) {
    const auto r = rsrc(dst, D1, t);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      f32x4 x[VW];
#pragma unroll
      for (int q = 0; q < VW; ++q) x[q] = *reinterpret_cast<const f32x4 *>(b + addr[j][q]);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        FloatVec<VW> y;
#pragma unroll
        for (int q = 0; q < VW; ++q) y[q] = x[q][i];
        buffer_store_f<VW>(r, off[j] + i * 64 * D1, y);
      }
    }
  };
  // The tile after the next one is loaded into registers one period ahead, each
  // task's loads as soon as its registers have moved to LDS, so that a compute
  // unit always has most of a tile's loads in flight.  Every period issues the
  // same accesses, those of a tile that is not there with an empty descriptor:
  // the loads and stores share one in-order counter, and behind a branch the
  // wait for a tile's loads would also wait for the stores issued after them.
  // tiles of period p - 1, p, p + 1 and p + 2
  int64_t before = -1, t = blockIdx.x, next = t + gridDim.x, after = next + gridDim.x;
  {
    const auto r0 = rsrc(src, D1, t), r1 = rsrc(src, D1, next);
#pragma unroll
    for (int j = 0; j < PER; ++j) load(r0, j);
    if constexpr (BWD) load_ds(t);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      put(lds, j);
      load(r1, j);
    }
  }
  lds_sync<12>();
  int p = 0;
  for (; t < n_tiles; ++p) {
    // each LDS element is read (store of the tile before) and then overwritten (the
    // next tile) by the same thread, so program order alone orders the two
    float *b = lds + ((p + 1) & 1) * M::BUF;
    if constexpr (BWD) put_ds();  // read by the compute waves between B1 and B2
    else store_s(t, lds + (p & 1) * M::BUF);  // overwritten by them after B1
    store(before, b);
    if constexpr (BWD) load_ds(next);
    const auto r = rsrc(src, D1, after);
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      // the loads go into the registers that put has just read: not moved above
      // it, where they would need others
      __builtin_amdgcn_sched_barrier(0);
      put(b, j);
      __builtin_amdgcn_sched_barrier(0);
      load(r, j);
    }
    lds_sync<12>();  // B1
    lds_sync<12>();  // B2: the compute waves have written this tile's results
    before = t;
    t = next;
    next = after;
    after = __builtin_amdgcn_readfirstlane(order[(p + 3) & 3]);
  }
  store(before, lds + ((p + 1) & 1) * M::BUF);
}

template <int LMAX, bool FULL, bool BWD>
__global__ __launch_bounds__(kMixThreads) void mix_kernel(int64_t E, const float *__restrict__ src,
                                                          const float *__restrict__ mix,
                                                          const float *__restrict__ ds, float *__restrict__ dst,
                                                          float *__restrict__ s_out, int *__restrict__ ticket) {
  using X = XIrreps<LMAX, FULL>;
  using M = MixTile<X>;
  __shared__ float4 lds4[(2 * M::BUF + (BWD ? M::NE * kU : 0)) / 4];  // tiles, ds
  __shared__ int order[4];
  float *lds = reinterpret_cast<float *>(lds4);
  const int64_t n_tiles = (E + M::NE - 1) / M::NE;
  if (threadIdx.x < 3) order[threadIdx.x] = int(blockIdx.x + threadIdx.x * gridDim.x);  // read after the first barrier
  if (threadIdx.x < kWave * kMixComputeWaves) mix_compute_role<X, BWD>(n_tiles, mix, lds, order, ticket);
  else mix_memory_role<X, BWD>(E, n_tiles, src, ds, dst, s_out, lds, order);
}

constexpr int kWgEdges = 4;        // edges per tile: column counts NE * (2l + 1) are multiples of 4
// Channel u of the column of component k sits at u ^ wg_swizzle(k) (bits 1-3,
// within its 16-channel block).  A memory wave's 4-byte writes of one
// instruction cover 8 components k = 4 b + q (b = 0..7) of up to 8 channels;
// the swizzle spreads them over 64 distinct banks (without it 8 lanes shared
// a bank), and the compute waves' reads of 16 consecutive channels of one
// column stay a permutation of one 16-bank block.
__host__ __device__ constexpr int wg_swizzle(int k) { return 2 * (k >> 2); }
constexpr int kWgCS = kU + 16;     // = 16 (mod 64): the four lane groups of an operand read hit distinct banks
constexpr int kWgThreads = 512;    // four compute waves, then four memory waves

// dMix_c = sum over edges and components of dV'_c T_c^T, software-pipelined
// over two LDS buffers that each hold a tile of dV' and of T in the column
// layout of the mixing kernel.  Waves 0-3 (compute) own rows 16w .. 16w+15 of
// every dMix_c as register accumulators; waves 4-7 (memory) keep the next tile
// in registers and move it into the free buffer while the compute waves work
// on the other.  One barrier per tile; both roles run the same tile sequence.
// Each workgroup writes one partial of every dMix_c.
template <class X>
struct WgTile {
  static constexpr int U = kU, D1 = X::D1, NE = kWgEdges, CS = kWgCS;
  static constexpr int COLS = NE * D1;
  static constexpr int BUF = 2 * COLS * CS;     // dV' then T
  static constexpr int F4 = NE * U * D1 / 4;    // float4 per tensor and tile
  static constexpr int PER = (F4 + 255) / 256;  // float4 per memory thread and tensor
  static_assert((U * D1) % 4 == 0, "edge rows must be whole float4");
};

template <class X>
__device__ __forceinline__ void wgrad_compute_role(int64_t n_tiles, float *lds, float *__restrict__ part) {
  using M = WgTile<X>;
  constexpr int U = M::U, CS = M::CS, NE = M::NE, NX = X::NX;
  const int tid = threadIdx.x, w = tid / kWave, l = tid % kWave;
  f32x4 acc[NX][4];
#pragma unroll
  for (int c = 0; c < NX; ++c)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) acc[c][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
  lds_sync<8>();  // the first tile is in buffer 0
  int p = 0;
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x, ++p) {
    const float *la = lds + (p & 1) * M::BUF, *lb = la + M::COLS * CS;
    // dMix_c[v][u] += sum_q dV'_c[q][v] T_c[q][u]; lane group l / 16 owns
    // the quarter of the irrep's columns q = (l / 16) * nq / 4 + s
    static_for<0, NX>([&](auto ic) {
      constexpr int c = decltype(ic)::value, nq = NE * X::dim(c), base = NE * X::off(c);
      const int q0 = base + (l / 16) * (nq / 4);
#pragma unroll
      for (int s = 0; s < nq / 4; ++s) {
        // column q0 + s holds component off(c) + s (of edge l / 16): its
        // channels sit XOR-swizzled by wg_swizzle of that component
        const int ul = (l % 16) ^ wg_swizzle(X::off(c) + s);
        const float a = la[(q0 + s) * CS + 16 * w + ul];
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[c][nt] = mfma_16x16x4(a, lb[(q0 + s) * CS + 16 * nt + ul], acc[c][nt]);
      }
    });
    lds_sync<8>();  // this buffer is free again; the other holds the next tile
  }
  float *out = part + int64_t(blockIdx.x) * NX * U * U;
#pragma unroll
  for (int c = 0; c < NX; ++c)
#pragma unroll
    for (int nt = 0; nt < 4; ++nt)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        out[(c * U + 16 * w + 4 * (l / 16) + r) * U + 16 * nt + l % 16] = acc[c][nt][r];
}

template <class X>
__device__ __forceinline__ void wgrad_memory_role(int64_t E, int64_t n_tiles, const float *__restrict__ dv,
                                                  const float *__restrict__ tt, float *lds) {
  using M = WgTile<X>;
  constexpr int U = M::U, D1 = M::D1, NE = M::NE, PER = M::PER, F4 = M::F4;
  const int mt = int(threadIdx.x) - 256;
  // the thread's float4 of a tile, 256 B apart (as in mix_memory_role)
  const int f0 = (mt / 16) * (16 * PER) + mt % 16;
  auto fi = [&](int i) { return f0 + 16 * i; };
  // LDS offset (within a tensor's tile) of each of the thread's elements
  int addr[PER][4];
#pragma unroll
  for (int i = 0; i < PER; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int idx = 4 * fi(i) + q;
      int a = 0;
      if (idx < 4 * F4) {
        const int e = idx / (U * D1), rem = idx % (U * D1), u = rem / D1, k = rem % D1;
        int col0, dim;
        component_column<X>(k, NE, col0, dim);
        a = (col0 + e * dim) * M::CS + (u ^ wg_swizzle(k));
      }
      addr[i][q] = a;
    }
  float4 va[PER], vb[PER];
  auto load = [&](int64_t t) {
    const int nf4 = int(E - t * NE < NE ? E - t * NE : NE) * (U * D1 / 4);
    const float4 *a4 = reinterpret_cast<const float4 *>(dv + t * NE * U * D1);
    const float4 *b4 = reinterpret_cast<const float4 *>(tt + t * NE * U * D1);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int f = fi(i);
      va[i] = f < nf4 ? load_stream(a4 + f) : make_float4(0.f, 0.f, 0.f, 0.f);
      vb[i] = f < nf4 ? load_stream(b4 + f) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  auto put = [&](float *b) {
    float *la = b, *lb = b + M::COLS * M::CS;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (fi(i) >= F4) continue;
      la[addr[i][0]] = va[i].x; la[addr[i][1]] = va[i].y; la[addr[i][2]] = va[i].z; la[addr[i][3]] = va[i].w;
      lb[addr[i][0]] = vb[i].x; lb[addr[i][1]] = vb[i].y; lb[addr[i][2]] = vb[i].z; lb[addr[i][3]] = vb[i].w;
    }
  };
  const int64_t G = gridDim.x;
  int64_t t = blockIdx.x;
  if (t < n_tiles) {
    load(t);
    put(lds);
  }
  if (t + G < n_tiles) load(t + G);
  lds_sync<8>();
  for (int p = 0; t < n_tiles; t += G, ++p) {
    // the compute waves read buffer p & 1; fill the other with tile t + G, then
    // start the loads of tile t + 2G
    if (t + G < n_tiles) put(lds + ((p + 1) & 1) * M::BUF);
    if (t + 2 * G < n_tiles) load(t + 2 * G);
    lds_sync<8>();
  }
}

template <int LMAX, bool FULL>
__global__ __launch_bounds__(kWgThreads) void mix_wgrad_kernel(int64_t E, const float *__restrict__ dv,
                                                               const float *__restrict__ tt,
                                                               float *__restrict__ part) {
  using X = XIrreps<LMAX, FULL>;
  __shared__ float lds[2 * WgTile<X>::BUF];
  const int64_t n_tiles = (E + kWgEdges - 1) / kWgEdges;
  if (threadIdx.x < 256) wgrad_compute_role<X>(n_tiles, lds, part);
  else wgrad_memory_role<X>(E, n_tiles, dv, tt, lds);
}

// ------------------------------------------------------------- host side
constexpr int64_t kMaxPersistent = 512;  // workgroups of the persistent kernels (2 per CU)

int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
size_t align256(size_t b) { return (b + 255) & ~size_t(255); }
int64_t red_groups(int64_t E) { return std::min<int64_t>(cdiv(E, kRedTile), kMaxPersistent); }
int64_t wgrad_groups(int64_t E) { return std::min<int64_t>(cdiv(E, kWgEdges), kMaxPersistent); }

struct Shape {
  int L = 0, H = 0, U = 0, d1 = 0, d2 = 0, P = 0, NX = 0;
  int64_t N = 0, E = 0;
};

// Byte offsets of the regions of the saved and workspace buffers.
struct SavedLayout {
  size_t w, env, T, s, a, total;
};
struct WorkLayout {
  size_t dT, da, dhm, ds, dw, genv, tpws, red, mixp, total, tpws_bytes;
};

SavedLayout saved_layout(const Shape &z) {
  SavedLayout o{};
  size_t at = 0;
  auto take = [&](size_t floats) { const size_t off = at; at += align256(floats * sizeof(float)); return off; };
  o.w = take(size_t(z.E) * z.U);
  o.env = take(size_t(z.N) * z.U * z.d2);
  o.T = take(size_t(z.E) * z.U * z.d1);
  o.s = take(size_t(z.E) * z.U);
  o.a = take(size_t(z.E) * z.H);
  o.total = at;
  return o;
}

WorkLayout work_layout(const allegro_tp_plan *plan, const Shape &z) {
  WorkLayout o{};
  size_t at = 0;
  auto take = [&](size_t bytes) { const size_t off = at; at += align256(bytes); return off; };
  const size_t f = sizeof(float);
  o.dT = take(size_t(z.E) * z.U * z.d1 * f);
  o.da = take(size_t(z.E) * z.H * f);
  o.dhm = take(size_t(z.E) * z.L * f);
  o.ds = take(size_t(z.E) * z.U * f);
  o.dw = take(size_t(z.E) * z.U * f);
  o.genv = take(size_t(z.N) * z.U * z.d2 * f);
  size_t tpws = 0;
  (void)allegro_tp_backward_workspace(plan, z.N, &tpws);
  o.tpws_bytes = tpws;
  o.tpws = take(tpws);
  const size_t mn = std::max({size_t(z.L + z.U) * z.H, size_t(z.H) * z.L, size_t(z.L) * z.U});
  o.red = take(size_t(red_groups(z.E)) * mn * f);
  o.mixp = take(size_t(wgrad_groups(z.E)) * z.NX * z.U * z.U * f);
  o.total = at;
  return o;
}

int after(const char *what) {
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess) return fail(ALLEGRO_E_HIP, "%s launch failed: %s", what, hipGetErrorString(err));
  return ALLEGRO_OK;
}

// Workgroups of `kernel` (static LDS only) that the device holds at once; at
// least one per compute unit.
int64_t resident_groups(const void *kernel, int threads) {
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu <= 0)
    per_cu = 1;
  return int64_t(cus) * per_cu;
}

void colsum(hipStream_t s, int64_t R, int C, const float *part, float *out) {
  hipLaunchKernelGGL(colsum_kernel, dim3(unsigned(cdiv(C, kColsumCols))), dim3(256), 0, s, int(R), C, part, out);
}

// Launchers of the dense contractions of a layer with latent width L and hidden width H.
template <int L, int H>
struct DenseOps {
  static constexpr int U = kU;
  // one workgroup per slot the GPU holds at once: each loads its B operands once
  template <int K, int N, int EPI>
  static void row(hipStream_t s, const RowGemmArgs &g) {
    if (g.E == 0) return;
    static const int64_t slots =
        resident_groups(reinterpret_cast<const void *>(&row_gemm_kernel<K, N, EPI>), kThreads);
    const unsigned G = unsigned(std::min<int64_t>(cdiv(g.E, kRowTile), slots));
    hipLaunchKernelGGL((row_gemm_kernel<K, N, EPI>), dim3(G), dim3(kThreads), 0, s, g);
  }
  template <int K1A, int K1B, int N2, int N2A, bool BWD>
  static void chain(hipStream_t s, const ChainArgs &g) {
    if (g.E == 0) return;
    static const int64_t slots = resident_groups(
        reinterpret_cast<const void *>(&latent_chain_kernel<K1A, K1B, H, N2, N2A, BWD>), kChainThreads);
    const unsigned G = unsigned(std::min<int64_t>(cdiv(g.E, kChainRows), slots));
    hipLaunchKernelGGL((latent_chain_kernel<K1A, K1B, H, N2, N2A, BWD>), dim3(G), dim3(kChainThreads), 0, s, g);
  }
  template <int M1, int M2, int N, int PRO>
  static void reduce(hipStream_t s, int64_t E, const float *p1, const float *p2, const float *q, float *part,
                     float *out) {
    const int64_t G = red_groups(E);
    if (G > 0)
      hipLaunchKernelGGL((reduce_gemm_kernel<M1, M2, N, PRO>), dim3(unsigned(G)), dim3(kThreads), 0, s, E, p1, p2, q,
                         part);
    colsum(s, G, (M1 + M2) * N, part, out);
  }

  // w = h A;  a = [h, s] B1 (after the mixing has written s);  h' = h + SiLU(a) B2
  static void embed_weights(hipStream_t s, int64_t E, const float *h, const float *A, float *w, int *ticket) {
    row<L, U, kEpiStore>(s, {E, h, A, U, 1, nullptr, w, ticket});
  }
  static void latent(hipStream_t s, int64_t E, const float *h, const float *sv, const float *B1, const float *B2,
                     float *a, float *h_out) {
    chain<L, U, L, L, false>(s, {E, h, sv, B1, B2, H, 1, L, 1, nullptr, a, h, h_out, nullptr, nullptr});
  }
  // da = (dh' B2^T) * SiLU'(a);  [dhm | ds] = [dh', 0] + da B1^T;  dB2, dB1
  static void latent_vjp(hipStream_t s, int64_t E, const float *h, const float *sv, const float *a,
                         const float *B1, const float *B2, const float *dh_out, float *da, float *dhm, float *ds,
                         float *part, float *dB1, float *dB2, int *ticket) {
    chain<L, 0, L + U, L, true>(s, {E, dh_out, nullptr, B2, B1, 1, L, 1, H, a, da, dh_out, dhm, ds, ticket});
    reduce<H, 0, L, kProSilu>(s, E, a, nullptr, dh_out, part, dB2);
    reduce<L, U, H, kProNone>(s, E, h, sv, da, part, dB1);
  }
  // dA = h^T dw;  dh = dhm + dw A^T
  static void embed_vjp(hipStream_t s, int64_t E, const float *h, const float *A, const float *dw, const float *dhm,
                        float *part, float *dA, float *dh) {
    reduce<L, 0, U, kProNone>(s, E, h, nullptr, dw, part, dA);
    row<U, L, kEpiAdd>(s, {E, dw, A, 1, U, dhm, dh, nullptr});
  }
};

struct DenseTable {
  void (*embed_weights)(hipStream_t, int64_t, const float *, const float *, float *, int *) = nullptr;
  void (*latent)(hipStream_t, int64_t, const float *, const float *, const float *, const float *, float *,
                 float *) = nullptr;
  void (*latent_vjp)(hipStream_t, int64_t, const float *, const float *, const float *, const float *,
                     const float *, const float *, float *, float *, float *, float *, float *, float *,
                     int *) = nullptr;
  void (*embed_vjp)(hipStream_t, int64_t, const float *, const float *, const float *, const float *, float *,
                    float *, float *) = nullptr;
};

template <int L, int H>
DenseTable dense_table() {
  using D = DenseOps<L, H>;
  return {&D::embed_weights, &D::latent, &D::latent_vjp, &D::embed_vjp};
}

DenseTable select_dense(int L, int H) {
  if (L == 64 && H == 64) return dense_table<64, 64>();
  if (L == 64 && H == 128) return dense_table<64, 128>();
  if (L == 128 && H == 64) return dense_table<128, 64>();
  if (L == 128 && H == 128) return dense_table<128, 128>();
  return {};
}

// Launchers of the mixing kernels of one (lmax, parity).
template <int LMAX, bool FULL>
struct MixOps {
  // one workgroup per tile slot the GPU holds at once
  template <bool BWD>
  static unsigned grid(int64_t E) {
    static const int64_t slots = resident_groups(reinterpret_cast<const void *>(&mix_kernel<LMAX, FULL, BWD>),
                                                 kMixThreads);
    return unsigned(std::min<int64_t>(cdiv(E, MixTile<XIrreps<LMAX, FULL>>::NE), slots));
  }
  static void forward(hipStream_t s, int64_t E, const float *T, const float *mix, float *V_out, float *sv,
                      int *ticket) {
    if (E == 0) return;
    hipLaunchKernelGGL((mix_kernel<LMAX, FULL, false>), dim3(grid<false>(E)), dim3(kMixThreads), 0, s, E, T, mix,
                       nullptr, V_out, sv, ticket);
  }
  static void backward(hipStream_t s, int64_t E, const float *dV_out, const float *T, const float *mix,
                       const float *ds, float *dT, float *part, float *dmix, int *ticket) {
    using X = XIrreps<LMAX, FULL>;
    // resident workgroups (one per compute unit), at most the partials the workspace holds
    static const int64_t slots = std::min<int64_t>(
        resident_groups(reinterpret_cast<const void *>(&mix_wgrad_kernel<LMAX, FULL>), kWgThreads), kMaxPersistent);
    const int64_t Gw = std::min<int64_t>(wgrad_groups(E), slots);
    if (E > 0) {
      hipLaunchKernelGGL((mix_kernel<LMAX, FULL, true>), dim3(grid<true>(E)), dim3(kMixThreads), 0, s, E, dV_out,
                         mix, ds, dT, nullptr, ticket);
      hipLaunchKernelGGL((mix_wgrad_kernel<LMAX, FULL>), dim3(unsigned(Gw)), dim3(kWgThreads), 0, s, E, dV_out, T,
                         part);
    }
    colsum(s, Gw, X::NX * kU * kU, part, dmix);
  }
};

struct MixTable {
  void (*forward)(hipStream_t, int64_t, const float *, const float *, float *, float *, int *) = nullptr;
  void (*backward)(hipStream_t, int64_t, const float *, const float *, const float *, const float *, float *,
                   float *, float *, int *) = nullptr;
};

template <int LMAX, bool FULL>
MixTable mix_table() {
  return {&MixOps<LMAX, FULL>::forward, &MixOps<LMAX, FULL>::backward};
}

MixTable select_mix(int lmax, bool full) {
  switch (lmax * 2 + (full ? 1 : 0)) {
    case 2: return mix_table<1, false>();
    case 3: return mix_table<1, true>();
    case 4: return mix_table<2, false>();
    case 5: return mix_table<2, true>();
    case 6: return mix_table<3, false>();
    case 7: return mix_table<3, true>();
    default: return {};
  }
}

int layer_shape(const allegro_tp_plan *plan, int L, int H, int64_t N, int64_t E, Shape &z) {
  if (!plan) return fail(ALLEGRO_E_INVALID, "plan is NULL");
  if (N < 0 || E < 0) return fail(ALLEGRO_E_INVALID, "negative size (N=%lld, E=%lld)", (long long)N, (long long)E);
  if (N == 0 && E > 0) return fail(ALLEGRO_E_INVALID, "E=%lld edges but N=0 centers", (long long)E);
  if (N >= (int64_t(1) << 31)) return fail(ALLEGRO_E_INVALID, "N=%lld exceeds 2^31-1", (long long)N);
  if (plan->U != kU) return fail(ALLEGRO_E_UNSUPPORTED, "the layer supports U=64 (plan has U=%d)", plan->U);
  if (!select_dense(L, H).latent)
    return fail(ALLEGRO_E_UNSUPPORTED, "the layer supports L, H in {64, 128} (got L=%d, H=%d)", L, H);
  const auto &t = plan->table;
  z.L = L;
  z.H = H;
  z.U = plan->U;
  z.d1 = t.d1;
  z.d2 = t.d2;
  z.P = int(t.paths.size());
  z.NX = int(t.x_irreps.size());
  z.N = N;
  z.E = E;
  return ALLEGRO_OK;
}

int check_ptr(const void *p, const char *name) {
  if (!p) return fail(ALLEGRO_E_INVALID, "%s is NULL", name);
  if (reinterpret_cast<uintptr_t>(p) & 15u) return fail(ALLEGRO_E_INVALID, "%s is not 16-byte aligned", name);
  return ALLEGRO_OK;
}

template <class T>
T *at(void *base, size_t off) {
  return reinterpret_cast<T *>(static_cast<char *>(base) + off);
}

}  // namespace

extern "C" {

int allegro_layer_buffers(const allegro_tp_plan *plan, int L, int H, int64_t N, int64_t E, size_t *saved_bytes,
                          size_t *workspace_bytes) {
  Shape z;
  int rc = layer_shape(plan, L, H, N, E, z);
  if (rc) return rc;
  if (saved_bytes) *saved_bytes = saved_layout(z).total;
  if (workspace_bytes) *workspace_bytes = work_layout(plan, z).total;
  return ALLEGRO_OK;
}

int allegro_layer_forward(const allegro_tp_plan *plan, int L, int H, int64_t N, int64_t E, const int64_t *row_ptr,
                          const float *h, const float *V, const float *Y, const float *A, const float *W,
                          const float *Mix, const float *B1, const float *B2, float *h_out, float *V_out,
                          void *saved, size_t saved_bytes, void *stream) {
  Shape z;
  int rc = layer_shape(plan, L, H, N, E, z);
  if (rc) return rc;
  if (N == 0) return ALLEGRO_OK;
  const SavedLayout sl = saved_layout(z);
  if ((rc = check_ptr(saved, "saved"))) return rc;
  if (saved_bytes < sl.total)
    return fail(ALLEGRO_E_INVALID, "saved buffer of %zu bytes is smaller than the %zu required", saved_bytes,
                sl.total);
  if ((rc = check_ptr(W, "W")) || (rc = check_ptr(A, "A")) || (rc = check_ptr(Mix, "Mix")) ||
      (rc = check_ptr(B1, "B1")) || (rc = check_ptr(B2, "B2")))
    return rc;
  if (E > 0 && ((rc = check_ptr(h, "h")) || (rc = check_ptr(V, "V")) || (rc = check_ptr(Y, "Y")) ||
                (rc = check_ptr(h_out, "h_out")) || (rc = check_ptr(V_out, "V_out"))))
    return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const DenseTable dn = select_dense(L, H);
  const MixTable mx = select_mix(plan->lmax, (plan->flags & ALLEGRO_FULL_PARITY) != 0);
  if (!mx.forward) return fail(ALLEGRO_E_UNSUPPORTED, "no mixing kernel for this plan");
  float *w = at<float>(saved, sl.w), *env = at<float>(saved, sl.env), *T = at<float>(saved, sl.T);
  float *sv = at<float>(saved, sl.s), *a = at<float>(saved, sl.a);
  int *ticket = at<int>(saved, sl.a);  // in a's region, which is written after the mixing
  dn.embed_weights(s, E, h, A, w, ticket);
  if ((rc = after("allegro_layer_forward"))) return rc;
  if ((rc = allegro_env_embed(plan, N, E, row_ptr, w, Y, env, stream))) return rc;
  if ((rc = allegro_tp_forward(plan, N, E, row_ptr, V, env, W, T, stream))) return rc;
  mx.forward(s, E, T, Mix, V_out, sv, ticket);
  dn.latent(s, E, h, sv, B1, B2, a, h_out);
  return after("allegro_layer_forward");
}

int allegro_layer_backward(const allegro_tp_plan *plan, int L, int H, int64_t N, int64_t E, const int64_t *row_ptr,
                           const float *h, const float *V, const float *Y, const float *A, const float *W,
                           const float *Mix, const float *B1, const float *B2, const void *saved, size_t saved_bytes,
                           const float *dh_out, const float *dV_out, float *dh, float *dV, float *dY, float *dA,
                           float *dW, float *dMix, float *dB1, float *dB2, void *workspace, size_t workspace_bytes,
                           void *stream) {
  Shape z;
  int rc = layer_shape(plan, L, H, N, E, z);
  if (rc) return rc;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((rc = check_ptr(dA, "dA")) || (rc = check_ptr(dW, "dW")) || (rc = check_ptr(dMix, "dMix")) ||
      (rc = check_ptr(dB1, "dB1")) || (rc = check_ptr(dB2, "dB2")) || (rc = check_ptr(W, "W")) ||
      (rc = check_ptr(A, "A")) || (rc = check_ptr(Mix, "Mix")) || (rc = check_ptr(B1, "B1")) ||
      (rc = check_ptr(B2, "B2")))
    return rc;
  if (N == 0) {  // no centers, no edges: every weight gradient is zero
    colsum(s, 0, z.L * z.U, nullptr, dA);
    colsum(s, 0, z.P * z.U, nullptr, dW);
    colsum(s, 0, z.NX * z.U * z.U, nullptr, dMix);
    colsum(s, 0, (z.L + z.U) * z.H, nullptr, dB1);
    colsum(s, 0, z.H * z.L, nullptr, dB2);
    return after("allegro_layer_backward");
  }
  const SavedLayout sl = saved_layout(z);
  const WorkLayout wl = work_layout(plan, z);
  if ((rc = check_ptr(saved, "saved")) || (rc = check_ptr(workspace, "workspace"))) return rc;
  if (saved_bytes < sl.total)
    return fail(ALLEGRO_E_INVALID, "saved buffer of %zu bytes is smaller than the %zu required", saved_bytes,
                sl.total);
  if (workspace_bytes < wl.total)
    return fail(ALLEGRO_E_INVALID, "workspace of %zu bytes is smaller than the %zu required", workspace_bytes,
                wl.total);
  if (E > 0 && ((rc = check_ptr(h, "h")) || (rc = check_ptr(V, "V")) || (rc = check_ptr(Y, "Y")) ||
                (rc = check_ptr(dh_out, "dh_out")) || (rc = check_ptr(dV_out, "dV_out")) ||
                (rc = check_ptr(dh, "dh")) || (rc = check_ptr(dV, "dV")) || (rc = check_ptr(dY, "dY"))))
    return rc;
  const DenseTable dn = select_dense(L, H);
  const MixTable mx = select_mix(plan->lmax, (plan->flags & ALLEGRO_FULL_PARITY) != 0);
  if (!mx.backward) return fail(ALLEGRO_E_UNSUPPORTED, "no mixing kernel for this plan");
  void *sv_base = const_cast<void *>(saved);
  const float *w = at<float>(sv_base, sl.w), *env = at<float>(sv_base, sl.env), *T = at<float>(sv_base, sl.T);
  const float *sv = at<float>(sv_base, sl.s), *a = at<float>(sv_base, sl.a);
  float *dT = at<float>(workspace, wl.dT), *da = at<float>(workspace, wl.da), *dhm = at<float>(workspace, wl.dhm);
  float *ds = at<float>(workspace, wl.ds), *dw = at<float>(workspace, wl.dw), *genv = at<float>(workspace, wl.genv);
  float *red = at<float>(workspace, wl.red), *mixp = at<float>(workspace, wl.mixp);
  int *ticket = at<int>(workspace, wl.dw);  // in dw's region, which is written after the mixing
  dn.latent_vjp(s, E, h, sv, a, B1, B2, dh_out, da, dhm, ds, red, dB1, dB2, ticket);
  mx.backward(s, E, dV_out, T, Mix, ds, dT, mixp, dMix, ticket);
  if ((rc = after("allegro_layer_backward"))) return rc;
  if ((rc = allegro_tp_backward_train(plan, N, E, row_ptr, V, env, W, dT, w, Y, dV, genv, dw, dY, dW,
                                      at<void>(workspace, wl.tpws), wl.tpws_bytes, stream)))
    return rc;
  dn.embed_vjp(s, E, h, A, dw, dhm, red, dA, dh);
  return after("allegro_layer_backward");
}

}  // extern "C"
