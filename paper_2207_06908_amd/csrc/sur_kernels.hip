// sur_kernels.hip -- kernels of the surrogate network on gfx950.
//
// Products are C = A B^T with both operands bfloat16, on the CDNA4 matrix
// cores (v_mfma_f32_16x16x32_bf16, FP32 accumulation).  The producers of every
// operand write it in the layout its consumer wants: the forward epilogue
// writes each activation transposed (input of the weight-gradient product),
// the backward epilogue does the same for the output-side gradient, and Adam
// keeps W and W^T copies.  So every product reads 16-byte vectors along K and
// no kernel transposes through LDS.
//
// The copies and the transposes are in fragment order (frag_off): the 16 rows
// x 32 of K that one instruction takes are 1 KB in a row, in lane order, so a
// wave's load of a fragment is one contiguous KB.  (Row by row, a fragment takes
// half of each of 16 cache lines, and with 16 waves streaming weights the
// other halves were gone from the 32 KB L1 when the next step wanted them:
// twice the traffic from L2.)  The K steps of a row fragment lie next to each
// other: with the rows of a step next to each other instead, the fused
// inference of 65,536 rows takes 181 us, not 148.
//
// Fragment layout of the 16x16x32 instruction (64 lanes): lane l supplies
// A[row l%16][k = 8(l/16) .. 8(l/16)+7] and B^T[col l%16][same k], and holds
// D[rows 4(l/16) .. 4(l/16)+3][col l%16].
//
// Reductions (loss, bias gradients, routing) use a fixed order, so every
// result is reproducible run to run.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "sur_dev.h"

namespace mi355sur {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

// FP32 -> bfloat16, round to nearest, ties to even (one instruction).
__device__ __forceinline__ uint32_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

__device__ __forceinline__ bf16x8 ld_frag(const uint16_t* p) {
  const uint4 q = *(const uint4*)p;
  return __builtin_bit_cast(bf16x8, q);
}

// A lane's piece, at byte offset lo, of what lies at a uniform address.  The
// address stays in scalar registers and the offset in one vector register
// (the asm statements keep the compiler from adding them up outside a loop).
typedef __attribute__((address_space(1))) char* gptr;
template <typename T>
__device__ __forceinline__ T ld_uni(gptr p, unsigned lo) {
  asm volatile("" : "+s"(p), "+v"(lo));
  return *(const __attribute__((address_space(1))) T*)(p + lo);
}
template <typename T>
__device__ __forceinline__ void st_uni(gptr p, unsigned lo, T v) {
  asm volatile("" : "+s"(p), "+v"(lo));
  *(__attribute__((address_space(1))) T*)(p + lo) = v;
}

// Element offset of (row, k) in a fragment-ordered operand of K columns.
__device__ __forceinline__ long long frag_off(int row, int k, int K) {
  return ((long long)(row >> 4) * (K >> 5) + (k >> 5)) * 512 + ((row & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7);
}

// Two at once, the first value in the low half.
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// Offset of the four values (m .. m + 3, n) that a lane holds of a result
// fragment, in an FP32 block of N columns kept in fragment order: 16 x 16
// patches, a lane's four values side by side (m a multiple of 4).
__device__ __forceinline__ long long acc_off(int m, int n, int N) {
  return ((long long)(m >> 4) * (N >> 4) + (n >> 4)) * 256 + (((m & 15) >> 2) * 16 + (n & 15)) * 4;
}

constexpr float kInvSqrt2Pi = 0.39894228040143268f;

// The standard normal distribution function Phi(z), and exp(-z^2 / 2), for
// the exact GELU z Phi(z) and its derivative Phi(z) + z phi(z).  Phi comes
// from the erfc approximation of Abramowitz and Stegun, formula 7.1.26
// (absolute error of erf at most 1.5e-7, against a bfloat16 step of 2^-8 in
// the activations it feeds): with x = |z| / sqrt 2 and t = 1 / (1 + p x),
// erfc(x) = t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-x^2), and
// Phi(z) = erfc(x) / 2 for z < 0, 1 - erfc(x) / 2 otherwise.  No branch, one
// reciprocal and one exponential per value.
__device__ __forceinline__ float norm_cdf(float z, float& gz) {
  constexpr float kP = 0.3275911f * 0.70710678118654752f;  // p / sqrt 2
  constexpr float c1 = 0.5f * 0.254829592f, c2 = 0.5f * -0.284496736f, c3 = 0.5f * 1.421413741f,
                  c4 = 0.5f * -1.453152027f, c5 = 0.5f * 1.061405429f;  // a_i / 2
  const float t = __builtin_amdgcn_rcpf(fmaf(kP, fabsf(z), 1.0f));
  float s = fmaf(t, c5, c4);
  s = fmaf(t, s, c3);
  s = fmaf(t, s, c2);
  s = fmaf(t, s, c1);
  s *= t;
  gz = __builtin_amdgcn_exp2f(z * z * -0.72134752044448170f);  // 2^(-z^2 log2(e) / 2)
  const float h = s * gz;  // erfc(x) / 2
  return z < 0.0f ? h : 1.0f - h;
}

// Epilogue of a wave's FM x FN fragments at (mw, nw): fragment (i, j) is
// skipped unless vm[i] and vn[j].
template <int EPI, int FM, int FN>
__device__ __forceinline__ void gemm_store(const GemmArgs& g, const f32x4 (&c)[FM][FN], int mw, int nw, int lane,
                                           const bool (&vm)[FM], const bool (&vn)[FN]) {
  const int r16 = lane & 15;
  const int rq = (lane >> 4) * 4;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    if (!vm[i]) continue;
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      if (!vn[j]) continue;
      const int m0 = mw + 16 * i + rq, n = nw + 16 * j + r16;
      constexpr bool T = EPI == EPI_GELU_TRAIN || EPI == EPI_BWD;
      uint32_t t16[4];
      f32x4 f32;
      if (EPI == EPI_BWD) f32 = *(const f32x4*)(g.o32 + acc_off(m0, n, g.N));
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + r;
        const float v = c[i][j][r];
        if (EPI == EPI_GELU_TRAIN || EPI == EPI_GELU_INFER) {
          const float z = v + g.bias[n];
          float gz;
          const float ph = norm_cdf(z, gz);
          t16[r] = f2bf(z * ph);
          f32[r] = ph + z * (gz * kInvSqrt2Pi);
        } else if (EPI == EPI_LINEAR) {
          if (m < g.m_valid) g.o32[(size_t)m * g.ld32 + n] = v + g.bias[n];
        } else {  // EPI_BWD
          f32[r] = v * f32[r];
          t16[r] = f2bf(f32[r]);
        }
        if (EPI != EPI_LINEAR) g.o16[(size_t)m * g.ld16 + n] = (uint16_t)t16[r];
      }
      if (T) {
        *(uint2*)(g.oT + frag_off(n, m0, g.M)) = make_uint2(t16[0] | (t16[1] << 16), t16[2] | (t16[3] << 16));
        *(f32x4*)(g.o32 + acc_off(m0, n, g.N)) = f32;
      }
    }
  }
}

// One (32 F) x (32 F) output tile per block of four waves; each wave owns a
// (16 F) x (16 F) quarter, F x F fragments.  F = 2 for small products (the
// training batches: more blocks), F = 4 for large ones (twice the reuse of
// every fragment loaded).  Fragments beyond M or N are skipped (the
// conditions are uniform across the wave).  Each accumulator takes its K
// steps in order, so the result does not depend on F.
template <int EPI, int F>
__global__ __launch_bounds__(256) void k_gemm(GemmArgs g) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int mw = blockIdx.y * (32 * F) + (w >> 1) * (16 * F);
  const int nw = blockIdx.x * (32 * F) + (w & 1) * (16 * F);
  if (mw >= g.M || nw >= g.N) return;
  bool vm[F], vn[F];
#pragma unroll
  for (int i = 0; i < F; ++i) {
    vm[i] = i == 0 || mw + 16 * i < g.M;
    vn[i] = i == 0 || nw + 16 * i < g.N;
  }
  const int r16 = lane & 15, kq = (lane >> 4) * 8;
  const uint16_t* pa = g.A + (size_t)(mw + r16) * g.lda + kq;
  const uint16_t* pb = g.B + (size_t)nw * g.K + lane * 8;
  const size_t sa = (size_t)16 * g.lda, sb = (size_t)16 * g.K;
  f32x4 c[F][F];
#pragma unroll
  for (int i = 0; i < F; ++i)
#pragma unroll
    for (int j = 0; j < F; ++j) c[i][j] = f32x4{0, 0, 0, 0};
  const bf16x8 zero = __builtin_bit_cast(bf16x8, make_uint4(0, 0, 0, 0));
  // U K steps at a time: all their fragment loads first, then the products,
  // so a wave waits for memory once per U steps.
  auto steps = [&](int k0, auto u_tag) {
    constexpr int U = decltype(u_tag)::value;
    bf16x8 fa[U][F], fb[U][F];
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int i = 0; i < F; ++i) {
        fa[s][i] = vm[i] ? ld_frag(pa + i * sa + k0 + 32 * s) : zero;
        fb[s][i] = vn[i] ? ld_frag(pb + i * sb + 16 * (k0 + 32 * s)) : zero;
      }
#pragma unroll
    for (int s = 0; s < U; ++s)
#pragma unroll
      for (int i = 0; i < F; ++i)
#pragma unroll
        for (int j = 0; j < F; ++j)
          c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[s][i], fb[s][j], c[i][j], 0, 0, 0);
  };
  constexpr int KU = F == 2 ? 4 : 2;
  int k0 = 0;
  for (; k0 + 32 * KU <= g.K; k0 += 32 * KU) steps(k0, std::integral_constant<int, KU>());
  for (; k0 < g.K; k0 += 32) steps(k0, std::integral_constant<int, 1>());
  gemm_store<EPI, F, F>(g, c, mw, nw, lane, vm, vn);
}

// Large aligned inference products (M and N multiples of 128, K of 64; the
// hidden layers' GELU and the output layer's linear epilogue): the 128 x 128
// output tile of k_gemm<EPI, 4>, four waves of 4 x 4 fragments each, with
// the operands staged through LDS.  K advances in tiles of 64: the block
// copies the 128 x 64 tiles of A and B into LDS once and every wave reads
// its fragments there (in k_gemm two waves fetch each fragment from L2),
// while the loads of the next K tile are in flight in registers.  Rows are
// padded by 16 bytes (144-byte pitch), so the 16 rows of a fragment start
// in 16 distinct groups of four banks.  Each accumulator takes its K steps
// in the same order with the same instruction as k_gemm, and the epilogue
// is k_gemm's: the outputs are the same bits.
constexpr int GL_BM = 128, GL_BK = 64, GL_LD = GL_BK + 8;

// k_gemm_lds's GELU epilogue: gemm_store<EPI_GELU_INFER, 4>'s arithmetic,
// with the bfloat16 outputs staged in the wave's own 64 x 64 slice of LDS
// (lt, pitch GL_LD) so that they leave in 16-byte row pieces instead of one
// 2-byte store per value.
__device__ __forceinline__ void gemm_store_gelu_lds(const GemmArgs& g, const f32x4 (&c)[4][4], int mw, int nw,
                                                    int lane, uint16_t* lt) {
  const int r16 = lane & 15, rq = (lane >> 4) * 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = nw + 16 * j + r16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float z = c[i][j][r] + g.bias[n];
        float gz;
        const float ph = norm_cdf(z, gz);
        lt[(16 * i + rq + r) * GL_LD + 16 * j + r16] = (uint16_t)f2bf(z * ph);
      }
    }
  }
  // the slice is this wave's alone: its LDS writes done, its lanes read rows
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  const int ch = (lane & 7) * 8;
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    const int row = (lane >> 3) + 8 * t;
    *(uint4*)(g.o16 + (size_t)(mw + row) * g.ld16 + nw + ch) = *(const uint4*)(lt + row * GL_LD + ch);
  }
}

template <int EPI>
__global__ __launch_bounds__(256, 3) void k_gemm_lds(GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint16_t sm[2 * GL_BM * GL_LD];
  uint16_t* const sa = sm;
  uint16_t* const sb = sm + GL_BM * GL_LD;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  // Blocks are dealt to the 8 XCDs round robin.  The column tiles of one row
  // tile go to one XCD, one after another, so that the row tile of A comes
  // from HBM once and from that XCD's L2 for the other column tiles (dealt
  // in plain order, they would land on N / 128 different XCDs, and each
  // would read it from HBM).
  const int nt = g.N / GL_BM, b = blockIdx.x;
  int mi, ni;
  if ((g.M / GL_BM) % 8 == 0) {
    const int q = b >> 3;
    ni = q % nt;
    mi = (b & 7) + 8 * (q / nt);
  } else {
    mi = b / nt;
    ni = b % nt;
  }
  const int m0 = mi * GL_BM, n0 = ni * GL_BM;
  // this thread's 16-byte pieces of a K tile: rows cr + 32 i, k offset ck
  const int cr = tid >> 3, ck = (tid & 7) * 8;
  const uint16_t* ga = g.A + (size_t)(m0 + cr) * g.lda + ck;
  // ... and of B, in fragment order: fragment (w >> 1) + 2 i, half w & 1 of
  // the K tile, this lane's piece
  const int br = 16 * (w >> 1) + (lane & 15), bk = 32 * (w & 1) + 8 * (lane >> 4);
  const uint16_t* gb = g.B + frag_off(n0 + br, bk, g.K);
  const size_t a32 = (size_t)32 * g.lda, b32 = (size_t)32 * g.K;
  uint16_t* const la = sa + cr * GL_LD + ck;
  uint16_t* const lb = sb + br * GL_LD + bk;
  // (named values, not arrays: an array would be kept in scratch memory
  // across the asm statement below)
  uint4 a0, a1, a2, a3, b0, b1, b2, b3;
#define GL_FETCH(k0)                             \
  a0 = *(const uint4*)(ga + (k0));               \
  a1 = *(const uint4*)(ga + a32 + (k0));         \
  a2 = *(const uint4*)(ga + 2 * a32 + (k0));     \
  a3 = *(const uint4*)(ga + 3 * a32 + (k0));     \
  b0 = *(const uint4*)(gb + 16 * (k0));               \
  b1 = *(const uint4*)(gb + b32 + 16 * (k0));         \
  b2 = *(const uint4*)(gb + 2 * b32 + 16 * (k0));     \
  b3 = *(const uint4*)(gb + 3 * b32 + 16 * (k0));
#define GL_STASH()                               \
  *(uint4*)(la) = a0;                            \
  *(uint4*)(la + 32 * GL_LD) = a1;               \
  *(uint4*)(la + 64 * GL_LD) = a2;               \
  *(uint4*)(la + 96 * GL_LD) = a3;               \
  *(uint4*)(lb) = b0;                            \
  *(uint4*)(lb + 32 * GL_LD) = b1;               \
  *(uint4*)(lb + 64 * GL_LD) = b2;               \
  *(uint4*)(lb + 96 * GL_LD) = b3;
  const int r16 = lane & 15, kq = (lane >> 4) * 8;
  const int wm = (w >> 1) * 64, wn = (w & 1) * 64;
  const uint16_t* fa0 = sa + (wm + r16) * GL_LD + kq;
  const uint16_t* fb0 = sb + (wn + r16) * GL_LD + kq;
  f32x4 c[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) c[i][j] = f32x4{0, 0, 0, 0};
  GL_FETCH(0)
  GL_STASH()
  __syncthreads();
  for (int k0 = 0; k0 < g.K; k0 += GL_BK) {
    const bool more = k0 + GL_BK < g.K;
    if (more) {
      GL_FETCH(k0 + GL_BK)
    }
    // keep the next tile's loads here, ahead of the products (the compiler
    // would otherwise move them down to the LDS stores that use them)
    asm volatile("" ::: "memory");
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8 fa[4], fb[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        fa[i] = ld_frag(fa0 + 16 * i * GL_LD + 32 * s);
        fb[i] = ld_frag(fb0 + 16 * i * GL_LD + 32 * s);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], fb[j], c[i][j], 0, 0, 0);
    }
    __syncthreads();  // every wave is done with this tile
    if (more) {
      GL_STASH()
      __syncthreads();
    }
  }
#undef GL_FETCH
#undef GL_STASH
  if (EPI == EPI_GELU_INFER) {
    // the last barrier of the loop has freed the tiles: wave w takes rows
    // [64 w, 64 w + 64) of them
    gemm_store_gelu_lds(g, c, m0 + wm, n0 + wn, lane, sm + w * 64 * GL_LD);
  } else {
    const bool all[4] = {true, true, true, true};
    gemm_store<EPI, 4>(g, c, m0 + wm, n0 + wn, lane, all, all);
  }
}

// Fused inference: every layer of one net over BM rows in one block.  The
// block's activations stay in LDS from layer to layer (bfloat16, rows padded
// by 16 bytes so that the 16 rows of a fragment fall in different banks);
// only the inputs, the weights (a few MB per net, L2-resident) and the last
// layer's FP32 outputs touch memory.  (Layer by layer, a 64K-row activation
// block with 512 x 512 weights moves 128 MB through HBM per layer; here it
// moves none.)  NW waves; the waves split the block's rows into NW / (32 / CF)
// groups and the 32 column fragments of a 512-wide layer (16 columns each)
// into 32 / CF groups: wave w owns the row fragments of group w / (32 / CF)
// and the column fragments c, c + 32 / CF, ... (CF of them, c = w % (32 / CF)).
// Each activation fragment a wave reads from LDS serves CF products, each
// weight fragment it reads from L2 serves RF.  The weight fragments run PD K
// steps ahead of the products.
// The K loop has no branches: rows past the last hold zero inputs, a column
// fragment past the layer's width multiplies fragment 0's weights, and neither
// result is ever stored.  Each accumulator takes its K steps in order with the
// instruction k_gemm uses, and the epilogue is k_gemm's, so the outputs equal
// the layer-by-layer products bit for bit.
// (4 waves per SIMD: 128 registers a lane.)
template <int BM, int NW, int CF, int PD>
__global__ __launch_bounds__(64 * NW, 4) void k_mlp_infer(MlpArgs a) {
  constexpr int NT = 64 * NW, NWC = 32 / CF, NWR = NW / NWC, RF = BM / 16 / NWR;
  static_assert(NWC * CF == 32 && NWR * NWC == NW && RF * NWR * 16 == BM, "block shape");
  __shared__ __attribute__((aligned(16))) uint16_t act[BM * MLP_LDA];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cg = w % NWC, r0 = (w / NWC) * RF;  // column group, first row fragment
  const int net = blockIdx.y, m0 = blockIdx.x * BM;
  const uint16_t* bfn = a.bf + (size_t)net * a.bf_stride;
  const float* pn = a.p + (size_t)net * a.p_stride;
  for (int e = tid; e < BM * 16; e += NT) {  // inputs: 32 columns, two at a time
    const int r = e >> 4, q = (e & 15) * 2;
    const float* xr = a.x + (size_t)(m0 + r) * a.kin;
    const bool in = m0 + r < a.M;
    const float v0 = in && q < a.kin ? xr[q] : 0.0f, v1 = in && q + 1 < a.kin ? xr[q + 1] : 0.0f;
    *(uint32_t*)(act + r * MLP_LDA + q) = f2bf2(v0, v1);
  }
  __syncthreads();
  const int r16 = lane & 15, kq = (lane >> 4) * 8, rq = (lane >> 4) * 4;
  const uint16_t* pa = act + (16 * r0 + r16) * MLP_LDA + kq;
  const unsigned lo = 16u * lane;  // this lane's piece of a weight fragment
#pragma unroll 1
  for (int l = 0; l < a.L; ++l) {
    const MlpLayer ly = a.lay[l];
    const int nf = ly.n >> 4;
    // a fragment past the width reads fragment 0's rows (its products are
    // never stored); uniform pointers, advanced a K step at each load
    gptr pb[CF];
#pragma unroll
    for (int j = 0; j < CF; ++j) {
      const int f = cg + NWC * j < nf ? cg + NWC * j : 0;
      pb[j] = (gptr)(bfn + ly.w16 + (size_t)f * 16 * ly.kp);
    }
    auto ld_w = [&](bf16x8* b) {
#pragma unroll
      for (int j = 0; j < CF; ++j) {
        b[j] = ld_uni<bf16x8>(pb[j], lo);
        pb[j] += 1024;
      }
    };
    f32x4 c[RF][CF];
#pragma unroll
    for (int i = 0; i < RF; ++i)
#pragma unroll
      for (int j = 0; j < CF; ++j) c[i][j] = f32x4{0, 0, 0, 0};
    // One K step: the wave's activation fragments from LDS, RF x CF products
    // with this step's weight fragments.
    auto kstep = [&](int k0, const bf16x8* b) {
      bf16x8 fa[RF];
#pragma unroll
      for (int i = 0; i < RF; ++i) fa[i] = *(const bf16x8*)(pa + 16 * i * MLP_LDA + k0);
#pragma unroll
      for (int i = 0; i < RF; ++i)
#pragma unroll
        for (int j = 0; j < CF; ++j) c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[i], b[j], c[i][j], 0, 0, 0);
    };
    // The empty asm statements between steps keep each load in the step that
    // issues it: nothing is stored in the loop, so the compiler would
    // otherwise move the loads down to the step that uses them, and every
    // step would wait for its own loads.
    if (ly.kp == MLP_KMAX) {
      // the 16 steps of a 512-wide layer unrolled: step s reads the register
      // set s % PD, so the prefetched values are never copied (a copy would
      // wait for the load)
      constexpr int NS = MLP_KMAX / 32;
      bf16x8 b[PD][CF];
#pragma unroll
      for (int q = 0; q < PD; ++q) ld_w(b[q]);
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        asm volatile("" ::: "memory");
        kstep(32 * s, b[s % PD]);
        if (s + PD < NS) ld_w(b[s % PD]);
      }
    } else {
      // other widths (the first layer, small nets): one step at a time
#pragma unroll 1
      for (int k0 = 0; k0 < ly.kp; k0 += 32) {
        asm volatile("" ::: "memory");
        bf16x8 b[CF];
        ld_w(b);
        kstep(k0, b);
      }
    }
    float bn[CF];
#pragma unroll
    for (int j = 0; j < CF; ++j) bn[j] = pn[ly.bias + (cg + NWC * j < nf ? cg + NWC * j : 0) * 16 + r16];
    __syncthreads();  // every wave has read this layer's input
    if (l + 1 < a.L) {  // hidden layer: bias, exact GELU, bfloat16 into LDS
#pragma unroll
      for (int j = 0; j < CF; ++j) {
        if (cg + NWC * j >= nf) continue;
        uint16_t* const col = act + (16 * r0 + rq) * MLP_LDA + (cg + NWC * j) * 16 + r16;
#pragma unroll
        for (int i = 0; i < RF; ++i) {
#pragma unroll
          for (int r = 0; r < 4; r += 2) {
            float gz;
            const float z0 = c[i][j][r] + bn[j], z1 = c[i][j][r + 1] + bn[j];
            const uint32_t q = f2bf2(z0 * norm_cdf(z0, gz), z1 * norm_cdf(z1, gz));
            col[(16 * i + r) * MLP_LDA] = (uint16_t)q;
            col[(16 * i + r + 1) * MLP_LDA] = (uint16_t)(q >> 16);
          }
        }
      }
    } else {  // output layer: bias, FP32 staged in LDS, then rows < M out as whole rows
      float* of = (float*)act;
#pragma unroll
      for (int j = 0; j < CF; ++j) {
        if (cg + NWC * j >= nf) continue;
        const int n = (cg + NWC * j) * 16 + r16;
#pragma unroll
        for (int i = 0; i < RF; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r) of[(16 * (r0 + i) + rq + r) * ly.n + n] = c[i][j][r] + bn[j];
      }
      __syncthreads();
      // the block's rows are contiguous (of is dense, as the output is)
      const int cnt = min(BM, a.M - m0) * (ly.n >> 2);
      float4* out = (float4*)(a.out + (size_t)net * a.ld_net + (size_t)m0 * ly.n);
      if (((uintptr_t)a.out & 15) == 0) {
        for (int e = tid; e < cnt; e += NT) out[e] = ((const float4*)of)[e];
      } else {
        for (int e = tid; e < 4 * cnt; e += NT) ((float*)out)[e] = of[e];
      }
    }
    __syncthreads();  // the next layer reads what this one wrote
  }
}

// Batch assembly: inputs to bfloat16, zero-padded to 32 columns and to M rows
// (row-major and, for training, transposed in fragment order).
__global__ void k_gather(const float* __restrict__ x, const int* __restrict__ rows, int m_valid, int M, int kin,
                         uint16_t* X16, uint16_t* XT) {
  const int stride = gridDim.x * blockDim.x;
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < M * 32; e += stride) {
    const int m = e >> 5, c = e & 31;
    float v = 0.0f;
    if (m < m_valid && c < kin) {
      const long long r = rows ? rows[m] : m;
      v = x[r * kin + c];
    }
    const uint16_t b = (uint16_t)f2bf(v);
    X16[e] = b;
    if (XT) XT[frag_off(c, m, M)] = b;
  }
}

// Mean squared error and its gradient dY = 2 (y - t) / (m_valid W), written
// as bfloat16 (row-major and transposed in fragment order) and FP32 in
// fragment order.  Each block covers 64 columns x 16 rows and leaves the sum
// of its squared errors in part[].
__global__ __launch_bounds__(256) void k_loss(const float* __restrict__ y, const float* __restrict__ t,
                                              const int* __restrict__ rows, int M, int m_valid, int W, float scale,
                                              uint16_t* g16, uint16_t* gT, float* dz, float* part) {
  __shared__ float red[256];
  const int n = blockIdx.x * 64 + (threadIdx.x & 63);
  const int m0 = blockIdx.y * 16 + (threadIdx.x >> 6) * 4;
  float s = 0.0f;
  uint32_t q[4];
  f32x4 gv;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = m0 + r;
    const size_t e = (size_t)m * W + n;
    float d = 0.0f;
    if (m < m_valid) d = y[e] - t[(long long)(rows ? rows[m] : m) * W + n];
    s += d * d;
    gv[r] = scale * d;
    q[r] = f2bf(gv[r]);
    g16[e] = (uint16_t)q[r];
  }
  *(f32x4*)(dz + acc_off(m0, n, W)) = gv;
  *(uint2*)(gT + frag_off(n, m0, M)) = make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
  red[threadIdx.x] = s;
  __syncthreads();
  for (int h = 128; h > 0; h >>= 1) {
    if (threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.y * gridDim.x + blockIdx.x] = red[0];
}

// Forward, loss and backward of one net over 16 rows of the batch per block:
// the rows are independent until the weight gradient, so a step needs no
// launch per layer.  16 waves; wave w owns the 16-column fragments 2w and
// 2w + 1 of every layer.  The row-major activations and gradients stay in LDS
// (two buffers, a barrier per layer); their transposes, the GELU derivatives
// and dZ, which replaces the derivatives in place, go to memory in fragment
// order, every store contiguous across the wave.
//
// What bounds it is the weights through the CU's L1: each block reads W and
// W^T once (3.6 MB for 4 x 512 + 256 wide layers, 27 us at 64 bytes a clock),
// so they stream without a break: fragments run PD K steps ahead, and the
// last steps of a layer load the first of the next.  Each pass costs about 2
// us more than its share of the stream, for the epilogue and the barrier.
// Measured with k_dw_adam, us a step: batches of 64 59, 256 61 (23 launches:
// 220), 1024 66, 4096 102 (one launch per layer: 81, 87, 100, 176).
// Each accumulator takes its K steps in order with the instruction k_gemm
// uses and the epilogues are k_gemm's and k_loss's: the same bits.
template <int PD>
__global__ __launch_bounds__(1024) void k_mlp_train(TrainArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t act[2][16 * MLP_LDA];
  __shared__ float red[1024];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = (lane >> 4) * 8, rq = (lane >> 4) * 4;
  const int m0 = blockIdx.x * 16, M = a.M, L = a.L, T = 2 * L - 1;
  const unsigned lo = 16u * lane;  // this lane's piece of a fragment or of a result's patch
  // ... of a transposed result: column r16 of 16, rows (m0 % 32) + rq .. + 3 of 32
  const unsigned lt = 16u * (r16 + 16 * (((m0 & 31) + rq) >> 3)) + 2u * (rq & 7);

  // Weights of pass t (0 .. L-1: forward through layer t; L .. 2L-2: backward
  // through layer 2L-1-t): K steps and the wave's fragments 2w and 2w + 1.  A
  // wave past the layer's width reads fragments 0 and 1.
  struct Stream {
    gptr p0, p1;  // the next step to load
    int ns;
  };
  auto weights = [&](int t) {
    const bool fwd = t < L;
    const TrainLayer& ly = a.lay[fwd ? t : 2 * L - 1 - t];
    const int K = fwd ? ly.kp : ly.n, N = fwd ? ly.n : ly.kp, f = 2 * w < (N >> 4) ? 2 * w : 0;
    const gptr p = (gptr)(a.bf + (fwd ? ly.w16 : ly.wt) + (size_t)f * 16 * K);
    return Stream{p, p + 32 * K, K >> 5};
  };
  bf16x8 b[PD][2];
  // the next step into b[q], while there is one (the last stays in place)
  auto ld_w = [&](int q, Stream& s, int step) {
    b[q][0] = ld_uni<bf16x8>(s.p0, lo);
    b[q][1] = ld_uni<bf16x8>(s.p1, lo);
    const int d = step + 1 < s.ns ? 1024 : 0;
    s.p0 += d;
    s.p1 += d;
  };
  Stream ws = weights(0);
#pragma unroll
  for (int q = 0; q < PD; ++q) ld_w(q, ws, q);

  if (tid < 256) {  // inputs: 16 rows x 32 columns, two at a time
    const int r = tid >> 4, c = (tid & 15) * 2, m = m0 + r;
    float v0 = 0.0f, v1 = 0.0f;
    if (m < a.m_valid) {
      const float* xr = a.x + (long long)(a.rows ? a.rows[m] : m) * a.kin;
      if (c < a.kin) v0 = xr[c];
      if (c + 1 < a.kin) v1 = xr[c + 1];
    }
    const uint32_t q = f2bf2(v0, v1);
    *(uint32_t*)(act[0] + r * MLP_LDA + c) = q;
    a.XT[frag_off(c, m, M)] = (uint16_t)q;
    a.XT[frag_off(c + 1, m, M)] = (uint16_t)(q >> 16);
  }
  __syncthreads();

  // One pass: N columns, this wave's two fragments of them.  KIND 0: hidden
  // layer forward, 1: output layer and loss, 2: backward.  tr: where the
  // result goes transposed; o32: GELU derivatives (0: written, 2: read and
  // replaced by dZ) or dZ (1).
  auto pass = [&](auto kind, int t, int N, const float* bias, uint16_t* tr, float* o32) {
    constexpr int KIND = decltype(kind)::value;
    const uint16_t* cur = act[t & 1] + r16 * MLP_LDA + kq;
    uint16_t* const nxt = act[(t & 1) ^ 1] + rq * MLP_LDA + 32 * w + r16;
    Stream wn = weights(t + 1 < T ? t + 1 : t);
    if (2 * w < (N >> 4)) {
      const gptr pz = (gptr)(o32 + (size_t)((m0 >> 4) * (N >> 4) + 2 * w) * 256);
      const gptr pt = (gptr)(tr + (size_t)(2 * w * (M >> 5) + (m0 >> 5)) * 512);
      // the epilogue's operands ahead of the products
      float bn[2];
      f32x4 ep[2];
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (KIND == 2)
          ep[j] = ld_uni<f32x4>(pz + 1024 * j, lo);
        else
          bn[j] = bias[32 * w + 16 * j + r16];
      }
      f32x4 c[2] = {f32x4{0, 0, 0, 0}, f32x4{0, 0, 0, 0}};
      auto kstep = [&](int q, int step) {
        const bf16x8 fa = *(const bf16x8*)(cur + 32 * step);
        c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, b[q][0], c[0], 0, 0, 0);
        c[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa, b[q][1], c[1], 0, 0, 0);
      };
      int s0 = 0;
#pragma unroll 1
      for (; s0 + PD < ws.ns; s0 += PD) {
#pragma unroll
        for (int q = 0; q < PD; ++q) {
          kstep(q, s0 + q);
          ld_w(q, ws, s0 + PD + q);
          asm volatile("" ::: "memory");
        }
      }
      if (KIND == 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + rq + r;
          const float* tp = a.t + (long long)(a.rows ? a.rows[min(m, a.m_valid - 1)] : min(m, a.m_valid - 1)) * N +
                            32 * w + r16;
          ep[0][r] = tp[0];
          ep[1][r] = tp[16];
        }
      }
#pragma unroll
      for (int q = 0; q < PD; ++q) {  // the last steps; the next pass's first fragments
        if (s0 + q < ws.ns) kstep(q, s0 + q);
        ld_w(q, wn, q);
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        __builtin_amdgcn_sched_barrier(0);
        f32x4 o;
        float h[4], se = 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          if (KIND == 0) {
            const float z = c[j][r] + bn[j];
            float g;
            const float ph = norm_cdf(z, g);
            h[r] = z * ph;
            o[r] = ph + z * (g * kInvSqrt2Pi);
          } else if (KIND == 1) {
            const float d = m0 + rq + r < a.m_valid ? (c[j][r] + bn[j]) - ep[j][r] : 0.0f;
            se += d * d;
            o[r] = h[r] = a.scale * d;
          } else {
            o[r] = h[r] = c[j][r] * ep[j][r];
          }
        }
        if (KIND == 1) red[(w >> 1) * 256 + (rq >> 2) * 64 + ((32 * w + 16 * j) & 63) + r16] = se;
        const uint32_t h01 = f2bf2(h[0], h[1]), h23 = f2bf2(h[2], h[3]);
        nxt[16 * j] = (uint16_t)h01;
        nxt[16 * j + MLP_LDA] = (uint16_t)(h01 >> 16);
        nxt[16 * j + 2 * MLP_LDA] = (uint16_t)h23;
        nxt[16 * j + 3 * MLP_LDA] = (uint16_t)(h23 >> 16);
        st_uni(pt + j * 32 * M, lt, u32x2{h01, h23});
        st_uni(pz + 1024 * j, lo, o);
      }
    } else {
#pragma unroll
      for (int q = 0; q < PD; ++q) ld_w(q, wn, q);
    }
    ws = wn;
    __syncthreads();  // the next pass reads what this one wrote
  };
#pragma unroll 1
  for (int l = 0; l + 1 < L; ++l) {
    const TrainLayer& ly = a.lay[l];
    pass(std::integral_constant<int, 0>(), l, ly.n, a.p + ly.bias, ly.aT, ly.gz);
  }
  {
    const TrainLayer& ly = a.lay[L - 1];
    pass(std::integral_constant<int, 1>(), L - 1, ly.n, a.p + ly.bias, ly.gT, ly.gz);
    if (w < (ly.n >> 6)) {  // k_loss's tree over 64 columns x 16 rows
      const float* q = red + w * 256 + lane;
      float s = (q[0] + q[128]) + (q[64] + q[192]);
      for (int h = 32; h > 0; h >>= 1) s += __shfl_down(s, h, 64);
      if (lane == 0) a.part[blockIdx.x * (ly.n >> 6) + w] = s;
    }
  }
#pragma unroll 1
  for (int l = L - 1; l > 0; --l) {
    const TrainLayer& ly = a.lay[l - 1];  // (of the columns this pass makes)
    pass(std::integral_constant<int, 2>(), 2 * L - 1 - l, ly.n, nullptr, ly.gT, ly.gz);
  }
}

__device__ __forceinline__ float adam1(const DwArgs& a, float g, float p, float& m, float& v) {
  m = a.b1 * m + (1.0f - a.b1) * g;
  v = a.b2 * v + (1.0f - a.b2) * (g * g);
  return p - a.lr * (m / a.c1) / (sqrtf(v / a.c2) + a.eps);
}

// Everything of a training step after dZ of every layer is known, in one
// launch: weight gradients dW = dZ^T A with Adam and the refresh of the
// bfloat16 copies in the epilogue (blocks 0 .. n_tile - 1, one 32 x 16 tile of
// some layer's W^T per wave), bias gradients with theirs (n_col blocks of 64
// columns x 4 row slices, added in a fixed order), and the loss.  The tile's
// parameters and moments are loaded before the products; a lane holds four
// adjacent columns of W, so all of it moves in 16-byte pieces.  Bound by the
// parameters and moments: 32 bytes a weight, 30 MB for 0.93 M weights.
template <int KF, int NF, int U>
__global__ __launch_bounds__(256) void k_dw_adam(DwArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), M = a.M;
  if ((int)blockIdx.x >= a.n_tile + a.n_col) {  // the loss, from the blocks' parts
    __shared__ float red[256];
    float s = 0.0f;
    for (int i = tid; i < a.n_part; i += 256) s += a.part[i];
    red[tid] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
      if (tid < h) red[tid] += red[tid + h];
      __syncthreads();
    }
    if (tid == 0) *a.loss = red[0] * a.inv;
    return;
  }
  int l = 0;
  if ((int)blockIdx.x >= a.n_tile) {  // bias gradients
    __shared__ float sl[4][64];
    const int blk = (int)blockIdx.x - a.n_tile;
    while (l + 1 < a.nl && blk >= a.L[l + 1].c0) ++l;
    const DwLayer& y = a.L[l];
    const int n = (blk - y.c0) * 64 + lane, q = M / 64;  // row blocks of a slice
    float acc = 0.0f;
#pragma unroll 4
    for (int b = w * q; b < (w + 1) * q; ++b) {
      const float* d = y.dz + acc_off(16 * b, n, y.n);
      f32x4 v[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = *(const f32x4*)(d + 64 * i);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc += v[i][r];
    }
    sl[w][lane] = acc;
    __syncthreads();
    if (w == 0) {
      const int e = y.off + y.n * y.k + n;
      const float g = ((sl[0][lane] + sl[1][lane]) + sl[2][lane]) + sl[3][lane];
      a.g[e] = g;
      if (a.update) {
        float m = a.m[e], v = a.v[e];
        a.p[e] = adam1(a, g, a.p[e], m, v);
        a.m[e] = m;
        a.v[e] = v;
      }
    }
    return;
  }
  const int wt = (int)blockIdx.x * 4 + w;
  if (wt >= a.n_wave) return;
  while (l + 1 < a.nl && wt >= a.L[l + 1].t0) ++l;
  const DwLayer& y = a.L[l];
  const int q = wt - y.t0, nk = y.kp / (16 * KF), k0 = 16 * KF * (q % nk), n0 = 16 * NF * (q / nk);
  const int r16 = lane & 15, rq = (lane >> 4) * 4;
  const bool vec = (y.k & 3) == 0;  // (offsets of the layers are multiples of 64)
  // a lane's elements of fragment (i, j): columns k0 + 16 i + rq .. + 3 of row n0 + 16 j + r16
  f32x4 p[KF][NF], m[KF][NF], v[KF][NF];
  auto elem = [&](int i, int j) { return y.off + (n0 + 16 * j + r16) * y.k + k0 + 16 * i + rq; };
  auto get = [&](const float* src, int i, int j) {
    f32x4 x = f32x4{0, 0, 0, 0};
    const int e = elem(i, j);
    if (vec) {
      if (k0 + 16 * i + rq < y.k) x = *(const f32x4*)(src + e);
      return x;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (k0 + 16 * i + rq + r < y.k) x[r] = src[e + r];
    return x;
  };
  auto put = [&](float* dst, int i, int j, f32x4 x) {
    const int e = elem(i, j);
    if (vec) {
      if (k0 + 16 * i + rq < y.k) *(f32x4*)(dst + e) = x;
      return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if (k0 + 16 * i + rq + r < y.k) dst[e + r] = x[r];
  };
  if (a.update)
#pragma unroll
    for (int i = 0; i < KF; ++i)
#pragma unroll
      for (int j = 0; j < NF; ++j) {
        p[i][j] = get(a.p, i, j);
        m[i][j] = get(a.m, i, j);
        v[i][j] = get(a.v, i, j);
      }
  const size_t fs = (size_t)16 * M;  // a row fragment of the transposes
  const uint16_t* pa = y.aT + (k0 >> 4) * fs + lane * 8;
  const uint16_t* pb = y.gT + (n0 >> 4) * fs + lane * 8;
  f32x4 c[KF][NF];
#pragma unroll
  for (int i = 0; i < KF; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j) c[i][j] = f32x4{0, 0, 0, 0};
  auto steps = [&](int s, auto u_tag) {
    constexpr int V = decltype(u_tag)::value;
    bf16x8 fa[V][KF], fb[V][NF];
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int i = 0; i < KF; ++i) fa[u][i] = ld_frag(pa + i * fs + 512 * (s + u));
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int j = 0; j < NF; ++j) fb[u][j] = ld_frag(pb + j * fs + 512 * (s + u));
#pragma unroll
    for (int u = 0; u < V; ++u)
#pragma unroll
      for (int i = 0; i < KF; ++i)
#pragma unroll
        for (int j = 0; j < NF; ++j)
          c[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[u][i], fb[u][j], c[i][j], 0, 0, 0);
  };
  const int S = M >> 5;
  int s = 0;
  for (; s + U <= S; s += U) steps(s, std::integral_constant<int, U>());
  for (; s < S; s += 2) steps(s, std::integral_constant<int, 2>());
#pragma unroll
  for (int i = 0; i < KF; ++i)
#pragma unroll
    for (int j = 0; j < NF; ++j) {
      put(a.g, i, j, c[i][j]);
      if (!a.update) continue;
      f32x4 x;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float mr = m[i][j][r], vr = v[i][j][r];
        x[r] = adam1(a, c[i][j][r], p[i][j][r], mr, vr);
        m[i][j][r] = mr;
        v[i][j][r] = vr;
      }
      put(a.m, i, j, m[i][j]);
      put(a.v, i, j, v[i][j]);
      put(a.p, i, j, x);
      const int n = n0 + 16 * j + r16, k = k0 + 16 * i + rq;
      uint16_t h[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) h[r] = k + r < y.k ? (uint16_t)f2bf(x[r]) : (uint16_t)0;  // padding stays zero
      *(uint2*)(a.bf + y.w16 + frag_off(n, k, y.kp)) =
          make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
#pragma unroll
      for (int r = 0; r < 4; ++r) a.bf[y.wt + frag_off(k + r, n, y.n)] = h[r];
    }
}

// The bfloat16 copies W [n x kp] and W^T [kp x n], in fragment order, of newly
// set parameters (k_dw_adam keeps them from then on; the padding is zero).
__global__ __launch_bounds__(256) void k_copies(CopyArgs a) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= a.P) return;
  int l = 0;
  while (l + 1 < a.nl && e >= a.L[l + 1].off) ++l;
  const CopyLayer& L = a.L[l];
  const int i = e - L.off;
  if (i < L.n * L.k) {
    const int row = i / L.k, col = i - row * L.k;
    const uint16_t b = (uint16_t)f2bf(a.p[e]);
    a.bf[L.w16 + frag_off(row, col, L.kp)] = b;
    a.bf[L.wt + frag_off(col, row, L.n)] = b;
  }
}

// Ensemble reduction of one chunk: one wave per row, one pass over the nets'
// outputs ys ([net][row][col], net stride ld_net).  Each lane keeps the
// running sum of its columns (nets added in order) and the running peak of
// the net in hand; the spread is (max - min) / |mean| of the nets' peaks, the
// peaks summed in net order.  Rows with an input outside [-xbound, xbound]
// get an infinite spread.
__global__ __launch_bounds__(256) void k_route(const float* __restrict__ ys, int nets, long long ld_net, int m, int W,
                                               const float* __restrict__ x, int kin, float xbound, float* ymean,
                                               float* spread) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= m) return;
  // an input outside [-xbound, xbound] routes the row whatever the spread
  const bool out = lane < kin && !(fabsf(x[(long long)row * kin + lane]) <= xbound);
  const bool any_out = __ballot(out) != 0;
  constexpr int CMAX = 8;  // columns per lane per group of 512 held in registers
  float pkq[16];           // per net (nets <= 16): the lane's running peak
#pragma unroll
  for (int q = 0; q < 16; ++q) pkq[q] = -INFINITY;
  for (int c0 = 0; c0 < W; c0 += 64 * CMAX) {
    float s[CMAX];
#pragma unroll
    for (int t = 0; t < CMAX; ++t) s[t] = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      if (q < nets) {
        const float* yq = ys + q * ld_net + (long long)row * W;
#pragma unroll
        for (int t = 0; t < CMAX; ++t) {
          const int c = c0 + lane + 64 * t;
          if (c < W) {
            const float v = yq[c];
            s[t] += v;
            pkq[q] = fmaxf(pkq[q], v);
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < CMAX; ++t) {
      const int c = c0 + lane + 64 * t;
      if (c < W) ymean[(long long)row * W + c] = s[t] / (float)nets;
    }
  }
  float pmax = -INFINITY, pmin = INFINITY, psum = 0.0f;
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    if (q < nets) {
      float pk = pkq[q];
      for (int o = 32; o > 0; o >>= 1) pk = fmaxf(pk, __shfl_xor(pk, o, 64));
      pmax = fmaxf(pmax, pk);
      pmin = fminf(pmin, pk);
      psum += pk;
    }
  }
  if (lane == 0) spread[row] = any_out ? INFINITY : (pmax - pmin) / fabsf(psum / (float)nets);
}

// k_route for four nets and W a multiple of 4: a lane takes 4 adjacent
// columns, with 16-byte loads and no branch around them.  Each column's sum
// runs over the nets in the same order from 0, the peaks are exact maxima,
// and the spread is formed as in k_route: the same bits.
__global__ __launch_bounds__(256) void k_route4(const float* __restrict__ ys, long long ld_net, int m, int W,
                                                const float* __restrict__ x, int kin, float xbound, float* ymean,
                                                float* spread) {
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= m) return;
  const bool out = lane < kin && !(fabsf(x[(long long)row * kin + lane]) <= xbound);
  const bool any_out = __ballot(out) != 0;
  float pk0 = -INFINITY, pk1 = -INFINITY, pk2 = -INFINITY, pk3 = -INFINITY;
  const float* y0 = ys + (long long)row * W;
  for (int c = 4 * lane; c < W; c += 256) {
    const float4 v0 = *(const float4*)(y0 + c);
    const float4 v1 = *(const float4*)(y0 + ld_net + c);
    const float4 v2 = *(const float4*)(y0 + 2 * ld_net + c);
    const float4 v3 = *(const float4*)(y0 + 3 * ld_net + c);
    float4 sm;
    sm.x = (((0.0f + v0.x) + v1.x) + v2.x) + v3.x;
    sm.y = (((0.0f + v0.y) + v1.y) + v2.y) + v3.y;
    sm.z = (((0.0f + v0.z) + v1.z) + v2.z) + v3.z;
    sm.w = (((0.0f + v0.w) + v1.w) + v2.w) + v3.w;
    *(float4*)(ymean + (long long)row * W + c) =
        make_float4(sm.x / 4.0f, sm.y / 4.0f, sm.z / 4.0f, sm.w / 4.0f);
    pk0 = fmaxf(pk0, fmaxf(fmaxf(v0.x, v0.y), fmaxf(v0.z, v0.w)));
    pk1 = fmaxf(pk1, fmaxf(fmaxf(v1.x, v1.y), fmaxf(v1.z, v1.w)));
    pk2 = fmaxf(pk2, fmaxf(fmaxf(v2.x, v2.y), fmaxf(v2.z, v2.w)));
    pk3 = fmaxf(pk3, fmaxf(fmaxf(v3.x, v3.y), fmaxf(v3.z, v3.w)));
  }
  for (int o = 32; o > 0; o >>= 1) {
    pk0 = fmaxf(pk0, __shfl_xor(pk0, o, 64));
    pk1 = fmaxf(pk1, __shfl_xor(pk1, o, 64));
    pk2 = fmaxf(pk2, __shfl_xor(pk2, o, 64));
    pk3 = fmaxf(pk3, __shfl_xor(pk3, o, 64));
  }
  float pmax = -INFINITY, pmin = INFINITY, psum = 0.0f;
  pmax = fmaxf(pmax, pk0), pmin = fminf(pmin, pk0), psum += pk0;
  pmax = fmaxf(pmax, pk1), pmin = fminf(pmin, pk1), psum += pk1;
  pmax = fmaxf(pmax, pk2), pmin = fminf(pmin, pk2), psum += pk2;
  pmax = fmaxf(pmax, pk3), pmin = fminf(pmin, pk3), psum += pk3;
  if (lane == 0) spread[row] = any_out ? INFINITY : (pmax - pmin) / fabsf(psum / 4.0f);
}

// Ordered list of the rows whose spread is above the threshold or not
// finite, in one block of 1024 threads.  Thread t owns the contiguous rows
// [t L, t L + L), L a multiple of 64 (64 for up to 65,536 rows).  It flags
// them 64 at a time into a bit mask (16 16-byte loads issued together), and
// a block scan of the counts gives each thread's first position.  The thread
// then writes its rows in order from the masks (the first segment's mask is
// kept, later ones are read again).
__device__ __forceinline__ unsigned long long flag_mask(const float* __restrict__ spread, int s, int b, float thr) {
  unsigned long long m = 0;
  if (s + 64 <= b) {
    float4 v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = *(const float4*)(spread + s + 4 * j);
#pragma unroll
    for (int j = 0; j < 16; ++j)
      m |= ((unsigned long long)!(v[j].x <= thr) << (4 * j)) | ((unsigned long long)!(v[j].y <= thr) << (4 * j + 1)) |
           ((unsigned long long)!(v[j].z <= thr) << (4 * j + 2)) | ((unsigned long long)!(v[j].w <= thr) << (4 * j + 3));
  } else {
    for (int r = s; r < b; ++r) m |= (unsigned long long)!(spread[r] <= thr) << (r - s);
  }
  return m;
}

__global__ __launch_bounds__(1024) void k_compact_chunks(const float* __restrict__ spread, int n, float thr,
                                                         int* __restrict__ ids, int* __restrict__ count) {
  __shared__ int wsum[16];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int L = (((n + 1023) / 1024) + 63) & ~63;
  const int a = min(t * L, n), b = min(a + L, n);
  const unsigned long long m0 = a < b ? flag_mask(spread, a, b, thr) : 0ull;
  int c = __popcll(m0);
  for (int s = a + 64; s < b; s += 64) c += __popcll(flag_mask(spread, s, b, thr));
  int incl = c;  // inclusive scan within the wave
  for (int o = 1; o < 64; o <<= 1) {
    const int y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  if (lane == 63) wsum[w] = incl;
  __syncthreads();
  int base = 0;
  for (int q = 0; q < w; ++q) base += wsum[q];
  if (t == 1023) *count = base + incl;
  int pos = base + incl - c;
  for (int s = a; s < b; s += 64) {
    unsigned long long m = s == a ? m0 : flag_mask(spread, s, b, thr);
    while (m) {
      ids[pos++] = s + __builtin_ctzll(m);
      m &= m - 1;
    }
  }
}

// Ordered list of the rows whose spread is above the threshold or not finite,
// in one block of 16 waves: the spreads are read 64 at a time (one per lane,
// coalesced), counted by ballot, the counts of the 64-row pieces scanned in
// LDS, and the rows written at their piece's offset plus their rank in it.
__global__ __launch_bounds__(1024) void k_compact(const float* __restrict__ spread, int n, float thr, int* ids,
                                                  int* count) {
  __shared__ int cnt[1024];
  __shared__ int off[1024];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int pieces = (n + 63) / 64;
  const int per = (pieces + 1023) / 1024;   // pieces per scan slot
  for (int s = threadIdx.x; s < 1024; s += 1024) cnt[s] = 0;
  __syncthreads();
  for (int p = w; p < pieces; p += 16) {
    const int i = p * 64 + lane;
    const bool f = i < n && !(spread[i] <= thr);
    const int c = __popcll(__ballot(f));
    if (lane == 0) atomicAdd(&cnt[p / per], c);
  }
  __syncthreads();
  const int mine = cnt[threadIdx.x];
  int v = mine;
  for (int o = 1; o < 1024; o <<= 1) {  // inclusive Hillis-Steele scan
    __syncthreads();
    off[threadIdx.x] = v;
    __syncthreads();
    if (threadIdx.x >= o) v += off[threadIdx.x - o];
  }
  __syncthreads();
  off[threadIdx.x] = v - mine;  // exclusive offset of scan slot
  __syncthreads();
  if (threadIdx.x == 1023) *count = v;
  // each scan slot's pieces in order, by one wave
  for (int slot = w; slot < 1024; slot += 16) {
    int pos = off[slot];
    for (int p = slot * per; p < min(pieces, (slot + 1) * per); ++p) {
      const int i = p * 64 + lane;
      const bool f = i < n && !(spread[i] <= thr);
      const unsigned long long b = __ballot(f);
      if (f) ids[pos + __popcll(b & ((1ull << lane) - 1ull))] = i;
      pos += __popcll(b);
    }
  }
}

static int last() { return (int)hipGetLastError(); }

template <int F>
void launch_gemm_f(int epi, const GemmArgs& a, hipStream_t s) {
  const dim3 grid((a.N + 32 * F - 1) / (32 * F), (a.M + 32 * F - 1) / (32 * F)), block(256);
  switch (epi) {
    case EPI_GELU_TRAIN: k_gemm<EPI_GELU_TRAIN, F><<<grid, block, 0, s>>>(a); break;
    case EPI_GELU_INFER: k_gemm<EPI_GELU_INFER, F><<<grid, block, 0, s>>>(a); break;
    case EPI_LINEAR: k_gemm<EPI_LINEAR, F><<<grid, block, 0, s>>>(a); break;
    default: k_gemm<EPI_BWD, F><<<grid, block, 0, s>>>(a); break;
  }
}

int launch_gemm(int epi, const GemmArgs& a, void* stream) {
  const hipStream_t s = (hipStream_t)stream;
  // 128 x 128 block tiles once they still give every CU a few blocks; the
  // inference products staged through LDS where the shape is aligned to the
  // tiles
  if ((long long)((a.M + 127) / 128) * ((a.N + 127) / 128) >= 1024) {
    const bool infer = epi == EPI_GELU_INFER || epi == EPI_LINEAR;
    if (infer && a.M % GL_BM == 0 && a.N % GL_BM == 0 && a.K % GL_BK == 0 && a.K > 0 &&
        (epi == EPI_LINEAR || a.ld16 % 8 == 0)) {
      const dim3 grid((a.N / GL_BM) * (a.M / GL_BM)), block(256);
      if (epi == EPI_GELU_INFER)
        k_gemm_lds<EPI_GELU_INFER><<<grid, block, 0, s>>>(a);
      else
        k_gemm_lds<EPI_LINEAR><<<grid, block, 0, s>>>(a);
    } else {
      launch_gemm_f<4>(epi, a, s);
    }
  } else {
    launch_gemm_f<2>(epi, a, s);
  }
  return last();
}

// Block shape by the number of blocks it makes.  While 16-row blocks do not
// outnumber the CUs, each takes one (23 us for 4 x 512 + 256 wide layers, most
// of it the 2 MB of weights through one L1; 32 rows take 28, 128 rows 70 us).
// Then 32-row blocks, two to a CU, up to one round of them (31 us for 8192
// rows; 16 rows 51, 64 rows 44).  Past that 64-row blocks, two to a CU: one
// block's GELU runs while the other's products do, which one 128-row block
// per CU cannot (65536 rows, us: 148; 32 rows 181, 128 rows 157; with row
// order weights and integer rounding 128 rows took 215).
template <int BM, int NW, int CF, int PD>
static void mlp_infer(const MlpArgs& a, int nets, hipStream_t s) {
  k_mlp_infer<BM, NW, CF, PD><<<dim3((a.M + BM - 1) / BM, nets), 64 * NW, 0, s>>>(a);
}

int launch_mlp_infer(const MlpArgs& a, int nets, void* stream) {
  if (a.M <= 0) return 0;
  const hipStream_t s = (hipStream_t)stream;
  const long long n16 = (long long)((a.M + 15) / 16) * nets, n32 = (long long)((a.M + 31) / 32) * nets;
  if (n16 <= 256)
    mlp_infer<16, 16, 2, 6>(a, nets, s);
  else if (n32 <= 512)
    mlp_infer<32, 8, 4, 3>(a, nets, s);
  else
    mlp_infer<64, 8, 4, 2>(a, nets, s);
  return last();
}

int launch_gather(const float* x, const int* rows, int m_valid, int M, int kin, uint16_t* X16, uint16_t* XT,
                  void* stream) {
  const long long work = (long long)M * 32;
  const int blocks = (int)((work + 255) / 256 < 4096 ? (work + 255) / 256 : 4096);
  k_gather<<<blocks, 256, 0, (hipStream_t)stream>>>(x, rows, m_valid, M, kin, X16, XT);
  return last();
}

int loss_parts(int M, int W) { return (W / 64) * (M / 16); }

int launch_loss(const float* y, const float* t, const int* rows, int M, int m_valid, int W, float scale, uint16_t* g16,
                uint16_t* gT, float* dz, float* part, void* stream) {
  k_loss<<<dim3(W / 64, M / 16), 256, 0, (hipStream_t)stream>>>(y, t, rows, M, m_valid, W, scale, g16, gT, dz, part);
  return last();
}

int launch_mlp_train(const TrainArgs& a, void* stream) {
  k_mlp_train<4><<<a.M / 16, 1024, 0, (hipStream_t)stream>>>(a);
  return last();
}

// Tiles of 32 x 16 a wave, 8 K steps' loads in flight: 12 us for batches of
// 256 (32 x 32 17, 16 x 16 12), 53 for 4096 (85 and 61; 32 x 16 with 4 steps 56).
constexpr int DW_KF = 2, DW_NF = 1, DW_U = 8;

int launch_dw_adam(DwArgs a, void* stream) {
  a.n_wave = a.n_col = 0;
  for (int l = 0; l < a.nl; ++l) {
    a.L[l].t0 = a.n_wave;
    a.L[l].c0 = a.n_col;
    a.n_wave += (a.L[l].n / (16 * DW_NF)) * (a.L[l].kp / (16 * DW_KF));
    a.n_col += a.L[l].n / 64;
  }
  a.n_tile = (a.n_wave + 3) / 4;
  k_dw_adam<DW_KF, DW_NF, DW_U><<<a.n_tile + a.n_col + (a.loss ? 1 : 0), 256, 0, (hipStream_t)stream>>>(a);
  return last();
}

int launch_copies(const CopyArgs& a, void* stream) {
  k_copies<<<(a.P + 255) / 256, 256, 0, (hipStream_t)stream>>>(a);
  return last();
}

int launch_route(const float* ys, int nets, int ld_net, int m, int W, const float* x, int kin, float xbound,
                 float* ymean, float* spread, void* stream) {
  if (m <= 0) return 0;
  const bool vec = nets == 4 && W % 4 == 0 && ld_net % 4 == 0 && ((uintptr_t)ys & 15) == 0 &&
                   ((uintptr_t)ymean & 15) == 0;
  if (vec)
    k_route4<<<(m + 3) / 4, 256, 0, (hipStream_t)stream>>>(ys, ld_net, m, W, x, kin, xbound, ymean, spread);
  else
    k_route<<<(m + 3) / 4, 256, 0, (hipStream_t)stream>>>(ys, nets, ld_net, m, W, x, kin, xbound, ymean, spread);
  return last();
}

int launch_compact(const float* spread, int n, float threshold, int* ids, int* count, void* stream) {
  if (((uintptr_t)spread & 15) == 0)
    k_compact_chunks<<<1, 1024, 0, (hipStream_t)stream>>>(spread, n, threshold, ids, count);
  else
    k_compact<<<1, 1024, 0, (hipStream_t)stream>>>(spread, n, threshold, ids, count);
  return last();
}

}  // namespace mi355sur
