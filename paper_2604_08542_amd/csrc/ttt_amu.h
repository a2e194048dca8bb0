// Launch-plan structs of the paper's memory unit (SwiGLU fast network,
// dot-product inner loss with token-wise step sizes; Supp. A, Sec. 4.2
// Eq. 8-10): forward step, update, operand preparation, and the reverse mode.
#pragma once
#include <stdint.h>
#ifdef __HIPCC__
#include "ttt_common.h"
#endif

namespace ttt {

// Weights of the SwiGLU fast network per head: W1 [d][h], W2 [h][d], W3 [d][h]
// at w1/w2/w3 + head * stride.
struct AmuWeights {
  const float* w1;
  const float* w2;
  const float* w3;
  int64_t stride;
};

// Operand copies per head (ttt_amu_prep), n_prep matrices of D*h elements in
// the matrix-core type: 0 W1 as [hid][d], 1 W3 as [hid][d], 2 W2 as [hid][d],
// 3 W2 as [d][hid]; with n_prep = 6 also 4 W1 as [d][hid], 5 W3 as [d][hid].
enum { AMU_W1T = 0, AMU_W3T = 1, AMU_W2N = 2, AMU_W2D = 3, AMU_W1D = 4, AMU_W3D = 5 };

// One chunk step of one sequence, every head: gradient of chunk s over a
// token shard (work-group = head * G + shard) and apply of chunk s-1.
struct AmuStepArgs {
  const void* Q;
  const void* K;
  const void* V;
  void* O;
  const float* eta_tok;  // [N][H] token-wise step sizes
  int64_t stride_tok, stride_head;
  int32_t H;
  uint32_t flags;
  int32_t G;
  const void* prep;      // [H][n_prep][D*h] operand copies (ttt_amu_prep)
  int32_t n_prep;
  float* partial;        // [H*G][3*D*h]: grad W1 | grad W2 | grad W3
  int64_t grad_start;
  int32_t grad_len;
  int64_t app_start;
  int32_t app_len;
};

struct AmuUpdArgs {
  AmuWeights src;
  const float* partial;
  int32_t G, H, h;
  float* w_dst;          // [H][3*D*h] packed W1 | W2 | W3
  float* wT1;            // final split copies, nullable
  float* wT2;
  float* wT3;
  void* prep;            // operand copies of the result as ttt_amu_prep writes them, nullable
  int32_t n_mats, prep_bf16;
  int32_t n_copies;      // how many of them (0 .. n_copies - 1 of the list above): 3, 4 or 6
};

struct AmuPrepArgs {
  AmuWeights src;
  void* prep;
  int32_t n_mats;        // 4 or 6 (see the operand-copy list above)
  int32_t H, h;
};

// Reverse mode over a token range [start, start+len) of every head, work-group
// = head * G + shard.  Apply adjoint (X = Q, Y = dO): dQ and the adjoint of
// the weights the queries were mapped with.  Update adjoint (X = K, Y = V):
// dK, dV, d eta_i and the second-order contribution -(dG/dW)^T Wh of one
// update W' = W - G(W) given the adjoint Wh of W'.
struct AmuBwdArgs {
  const void* X;
  const void* Y;
  void* dX;
  void* dY;                // update only
  const float* eta_tok;    // update only, [N][H]
  float* deta_tok;         // update only, [N][H]
  int64_t stride_tok, stride_head;
  int32_t H;
  uint32_t flags;
  int32_t G;
  const void* prep_w;      // [H][6][D*h] operand copies of the weights
  const void* prep_a;      // [H][6][D*h] operand copies of Wh (update only)
  float* partial;          // [H*G][3*D*h] contributions to the weights' adjoint
  int64_t start;
  int32_t len;
};

// dst = base + sum over the G shard partials in shard order (base nullable);
// split copies of the result when out1..3 are set.  Packed [H][3*D*h].  The
// launch that ends a chunk of the chain's reverse mode also writes the operand
// copies of the weights that the chunk before it starts from.
struct AmuPsumArgs {
  const float* partial;
  int32_t G, H, h;
  const float* base;
  float* dst;
  float* out1;
  float* out2;
  float* out3;
  void* prep;              // operand copies (six) of the result, nullable
  int32_t prep_bf16;
  AmuWeights next;         // with prep_next: weights to copy
  void* prep_next;         // their operand copies (six), nullable
};

#ifdef __HIPCC__
// Operand copies (see the list above) of four consecutive elements v at
// offset off of matrix mat (0 W1, 1 W2, 2 W3) of one head, o = the head's
// matrices of dh = 64 h elements, of which the first n_copies (3, 4 or 6) are
// written; called by all 256 threads of a work-group for 1,024 consecutive elements.  Written by the kernels that step
// the weights or sum an adjoint, so that no launch of its own has to read
// them back (7.7 us per launch at 16 heads, h = 256).
template <typename MT>
__device__ __forceinline__ void amu_put_prep(MT* o, int mat, int off, int h, int n_copies, const f32x4& v) {
  typedef MT mt4 __attribute__((ext_vector_type(4)));
  const int dh = D * h, off0 = off - 4 * (int)threadIdx.x;
  const mt4 m = {(MT)v[0], (MT)v[1], (MT)v[2], (MT)v[3]};
  if (mat == 1) {
    *reinterpret_cast<mt4*>(o + AMU_W2N * dh + off) = m;
    if (n_copies > 3) put_transposed(o + AMU_W2D * dh + off0 / D, h, D, h, v);
  } else {
    if (n_copies == 6) *reinterpret_cast<mt4*>(o + (mat ? AMU_W3D : AMU_W1D) * dh + off) = m;
    put_transposed(o + (mat ? AMU_W3T : AMU_W1T) * dh + off0 / h, D, h, h, v);
  }
}
#endif

}  // namespace ttt
