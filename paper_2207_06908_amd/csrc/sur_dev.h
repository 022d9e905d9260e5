// sur_dev.h -- host-side view of the surrogate kernels (launchers only).
#pragma once
#include <stdint.h>

namespace mi355sur {

enum Epi {
  EPI_GELU_TRAIN = 0,  // o16 = bf16(gelu(z)), oT = its transpose, o32 = gelu'(z)
  EPI_GELU_INFER = 1,  // o16 = bf16(gelu(z))
  EPI_LINEAR = 2,      // o32 = z (rows < m_valid)
  EPI_BWD = 3,         // dz = acc * o32; o16 = bf16(dz), oT = its transpose, o32 = dz
};

// C[M x N] = A[M x K] B[N x K]^T (bfloat16; A K-contiguous, B a weight copy
// in fragment order), FP32 accumulation on the matrix cores, then the
// epilogue.  oT is in fragment order, as is o32 in training (EPI_LINEAR:
// row-major).  M and N are multiples of 16, K a multiple of 32, leading
// dimensions multiples of 8.
struct GemmArgs {
  const uint16_t* A;
  const uint16_t* B;
  int lda, M, N, K;
  const float* bias;  // [N], z = acc + bias
  uint16_t* o16;
  int ld16;
  uint16_t* oT;
  float* o32;
  int ld32;
  int m_valid;
};

struct CopyLayer {
  int off, n, k, kp;  // flat offset of W (bias follows), shape, padded K
  long long w16, wt;  // element offsets of the bfloat16 copies W [n x kp], W^T [kp x n] (fragment order)
};
struct CopyArgs {
  const float* p;
  uint16_t* bf;  // base of the bfloat16 copies of this net
  int P, nl;
  CopyLayer L[8];
};

// Forward, loss and backward in one launch (k_mlp_train): M rows (a multiple
// of 64), hidden widths <= MLP_KMAX, output width <= MLP_TOUT.
constexpr int MLP_TOUT = 256;
struct TrainLayer {
  long long w16, wt;  // element offsets of the copies W, W^T
  int bias, kp, n;    // offset of b in the parameters, padded fan-in, fan-out
  uint16_t* aT;       // transposed activations (hidden layers)
  uint16_t* gT;       // transposed dZ
  float* gz;          // GELU derivatives, then dZ
};
struct TrainArgs {
  const float* x;  // [. x kin]
  const float* t;  // [. x W]
  const int* rows; // batch rows of x and t, or null for the first m_valid
  const uint16_t* bf;
  const float* p;
  int M, m_valid, kin, L;
  float scale;     // dY = scale (y - t)
  uint16_t* XT;
  float* part;     // loss_parts(M, W) sums of squared errors
  TrainLayer lay[7];
};

// Weight and bias gradients, Adam (update != 0) and the loss (k_dw_adam).
struct DwLayer {
  const uint16_t* aT;  // transposed inputs [kp x M], fragment order
  const uint16_t* gT;  // transposed dZ [n x M]
  const float* dz;     // dZ, fragment order
  int off, n, k, kp;
  long long w16, wt;
  int t0, c0;          // first wave tile and bias block (launch_dw_adam)
};
struct DwArgs {
  float* p;
  float* m;
  float* v;
  float* g;
  uint16_t* bf;
  int M, nl, update;
  float lr, b1, b2, eps, c1, c2;
  const float* part;
  int n_part;
  float inv;           // loss = inv * sum of the parts
  float* loss;         // or null
  int n_wave, n_tile, n_col;  // (launch_dw_adam)
  DwLayer L[7];
};

// Fused inference (k_mlp_infer): all layers of `nets` consecutive nets over
// M rows of kin inputs, activations kept on chip; hidden widths <= MLP_KMAX,
// the output width <= MLP_NOUT (its FP32 rows are staged in the same LDS).
// Net q's bfloat16 weight copies start at bf + q bf_stride, its FP32
// parameters at p + q p_stride; its outputs go to out[q ld_net], dense rows
// (ld_net a multiple of 4).
constexpr int MLP_KMAX = 512, MLP_LDA = MLP_KMAX + 8, MLP_NOUT = MLP_LDA / 2;
struct MlpLayer {
  long long w16;   // element offset of W [n x kp] in a net's bfloat16 copies
  int bias;        // offset of b in a net's FP32 parameters
  int kp, n;
};
struct MlpArgs {
  const float* x;  // [M x kin]
  const uint16_t* bf;
  const float* p;
  long long bf_stride, p_stride;
  int M, L, kin;
  float* out;
  long long ld_net;
  MlpLayer lay[8];
};
int launch_mlp_infer(const MlpArgs& a, int nets, void* stream);

int launch_gemm(int epi, const GemmArgs& a, void* stream);
int launch_gather(const float* x, const int* rows, int m_valid, int M, int kin, uint16_t* X16, uint16_t* XT,
                  void* stream);
int launch_loss(const float* y, const float* t, const int* rows, int M, int m_valid, int W, float scale, uint16_t* g16,
                uint16_t* gT, float* dz, float* part, void* stream);
int launch_mlp_train(const TrainArgs& a, void* stream);
int launch_dw_adam(DwArgs a, void* stream);
int launch_copies(const CopyArgs& a, void* stream);
// Mean over nets and peak spread per row; a row with an input outside
// [-xbound, xbound] (x: m rows of kin <= 64 inputs) gets an infinite spread.
int launch_route(const float* ys, int nets, int ld_net, int m, int W, const float* x, int kin, float xbound,
                 float* ymean, float* spread, void* stream);
int launch_compact(const float* spread, int n, float threshold, int* ids, int* count, void* stream);
int loss_parts(int M, int W);

}  // namespace mi355sur
