// The paper's memory unit with BF16 products on gfx950 (d = 64; the FP32 form
// and the formulas are in ttt_amu.hip).
//
// ttt_amu_step_bf: one chunk step, the gradient of chunk s over a token shard
// and the apply of chunk s-1.  Wave w owns hidden units [32w, 32w+32).  What
// bounds it is the elementwise work (two transcendentals and about twenty
// other operations per token and hidden unit) next to 24 matrix products per
// tile and wave; what it spent its time on instead was waiting for weight
// fragments read from the L2 for every tile, so here a wave keeps them in
// registers for the whole loop: W1, W3, W2 (48 registers) beside the three
// gradient accumulators (96) in the gradient loop; W1, W3 and its share of
// W2^T (64) in the apply loop, which starts after the partials are written.
// Token rows are staged once, row-major; the token-contraction operands are
// transposing reads of the same rows.
#include <hip/hip_runtime.h>

#include "ttt_amu_bf.h"
#include "ttt_common.h"
#include "ttt_internal.h"

namespace ttt {
namespace {

template <typename IOT, int NW>
__global__ __launch_bounds__(NW * 64, 2) void ttt_amu_step_bf(AmuStepArgs p) {
  constexpr int HH = NW * 32, NT = NW * 64, EPT = D * TT / NT, TPR = D / EPT, DH = D * HH;
  constexpr int AS_LD = HH + 8;
  // two copies of the row tiles, one barrier per tile: a copy is rewritten
  // two tiles later, after every wave has passed the next tile's barrier
  __shared__ __attribute__((aligned(16))) bf16 xs[2][TT * XLD];  // K or Q rows
  __shared__ __attribute__((aligned(16))) bf16 es[2][TT * XLD];  // E = -eta v rows
  __shared__ __attribute__((aligned(16))) bf16 hs[2][TT * AS_LD];  // Hq of the apply

  const Lane L;
  const int tid = threadIdx.x, row = tid / TPR, col0 = (tid % TPR) * EPT;
  const int lin = xcd_linear_block();
  const int G = p.G, head = lin / G, g = lin % G;
  const int64_t hoff = (int64_t)head * p.stride_head;
  const bool norm_q = p.flags & 1u, norm_k = p.flags & 2u, norm_v = p.flags & 4u;
  const bf16* W1t = static_cast<const bf16*>(p.prep) + (int64_t)head * p.n_prep * DH;
  bf16x8 w1[4], w3[4];
  L.weights(W1t + AMU_W1T * DH, w1);
  L.weights(W1t + AMU_W3T * DH, w3);

  // ------------------------------------------------ gradient of chunk s
  const int gl = p.grad_len;
  if (gl > 0) {
    bf16x8 w2[4];
    L.weights(W1t + AMU_W2N * DH, w2);
    f32x16 g1[2] = {}, g2[2] = {}, g3[2] = {};
    RowPart<IOT, EPT> rk, rv;
    float et = 0.f;
    auto fetch = [&](int t) {
      const int64_t tok = p.grad_start + (int64_t)t * TT + row;
      const bool valid = row < gl - t * TT;
      rk.load(static_cast<const IOT*>(p.K) + tok * p.stride_tok + hoff + col0, valid);
      rv.load(static_cast<const IOT*>(p.V) + tok * p.stride_tok + hoff + col0, valid);
      et = valid ? p.eta_tok[tok * p.H + head] : 0.f;
    };
    auto stage = [&](int b) {
      float x[EPT];
      const float sk = rk.get(norm_k, x);
      put_part<EPT>(&xs[b][row * XLD + col0], x, sk);
      const float sv = rv.get(norm_v, x);
      put_part<EPT>(&es[b][row * XLD + col0], x, sv * -et);
    };
    if (g * TT < gl) fetch(g);
    for (int t = g, b = 0; t * TT < gl; t += G, b ^= 1) {
      stage(b);
      if ((t + G) * TT < gl) fetch(t + G);
      __syncthreads();
      bf16x8 a[4];
      L.rows(xs[b], a);
      const f32x16 Z1 = dot4(a, w1), Z3 = dot4(a, w3);
      L.rows(es[b], a);
      const f32x16 dH = dot4(a, w2);
      f32x16 Hd, dZ1, dZ3;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float z = Z1[r];
        const float sg = sigmoid(z);
        const float s = z * sg;
        Hd[r] = s * Z3[r];
        dZ3[r] = dH[r] * s;
        dZ1[r] = dH[r] * Z3[r] * fmaf(s, 1.0f - sg, sg);
      }
      const Packed ph = pack32(Hd), p3 = pack32(dZ3), p1 = pack32(dZ1);
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          g2[db] = mma32(ph.f[m], L.cols(es[b], m, db), g2[db]);
          const bf16x8 k = L.cols(xs[b], m, db);
          g3[db] = mma32(k, p3.f[m], g3[db]);
          g1[db] = mma32(k, p1.f[m], g1[db]);
        }
    }
    // shard partials
    float* part = p.partial + ((int64_t)head * G + g) * (3 * DH);
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int rr = c32_row(r, L.hf);
        part[(32 * db + rr) * HH + L.hid] = g1[db][r];
        part[DH + (32 * L.w + rr) * D + 32 * db + L.l32] = g2[db][r];
        part[2 * DH + (32 * db + rr) * HH + L.hid] = g3[db][r];
      }
    __syncthreads();  // the apply reuses the tiles
  }

  // ------------------------------------------------ apply of chunk s-1
  // Transposed products (hidden units in registers, one token per lane): Hq
  // is staged with 8-byte writes.  One barrier per tile: the barrier that
  // publishes Hq of a tile also publishes the rows of the next.
  const int al = p.app_len;
  if (g * TT >= al) return;
  constexpr int NBK = 8 / NW;  // 16x16 output blocks per wave
  bf16x8 wo[NBK][HH / 32];
#pragma unroll
  for (int bi = 0; bi < NBK; ++bi) {
    const bf16* mrow = W1t + AMU_W2D * DH + (16 * ((L.w + NW * bi) >> 1) + L.l16) * HH;
#pragma unroll
    for (int u = 0; u < HH / 32; ++u)
      wo[bi][u] = *reinterpret_cast<const bf16x8*>(mrow + (HH / 4) * L.g4 + 8 * u);
  }
  RowPart<IOT, EPT> rq;
  auto fetch = [&](int t) {
    const int64_t tok = p.app_start + (int64_t)t * TT + row;
    rq.load(static_cast<const IOT*>(p.Q) + tok * p.stride_tok + hoff + col0, row < al - t * TT);
  };
  auto stage = [&](int b) {
    float x[EPT];
    const float sq = rq.get(norm_q, x);
    put_part<EPT>(&xs[b][row * XLD + col0], x, sq);
  };
  fetch(g);
  stage(0);
  if ((g + G) * TT < al) fetch(g + G);
  __syncthreads();
  for (int t = g, b = 0; t * TT < al; t += G, b ^= 1) {
    {
      bf16x8 a[4];
      L.rows(xs[b], a);
      const f32x16 Z1 = dot4(w1, a), Z3 = dot4(w3, a);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float h[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const float z = Z1[4 * j + q];
          h[q] = z * sigmoid(z) * Z3[4 * j + q];
        }
        *reinterpret_cast<u32x2*>(&hs[b][L.l32 * AS_LD + 32 * L.w + 8 * j + 4 * L.hf]) =
            (u32x2){pack_bf16x2(h[0], h[1]), pack_bf16x2(h[2], h[3])};
      }
    }
    if ((t + G) * TT < al) {
      stage(b ^ 1);
      if ((t + 2 * G) * TT < al) fetch(t + 2 * G);
    }
    __syncthreads();
    const int nv = al - t * TT;
    const int64_t t0 = p.app_start + (int64_t)t * TT;
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi) {
      const int bk = L.w + NW * bi, tb = bk & 1, db = bk >> 1;
      f32x4 o = {};
#pragma unroll
      for (int u = 0; u < HH / 32; ++u)
        o = mma16(*reinterpret_cast<const bf16x8*>(&hs[b][(16 * tb + L.l16) * AS_LD + (HH / 4) * L.g4 + 8 * u]),
                  wo[bi][u], o);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int tr = 16 * tb + 4 * L.g4 + r;
        if (tr < nv)
          static_cast<IOT*>(p.O)[(t0 + tr) * p.stride_tok + hoff + 16 * db + L.l16] = from_f<IOT>(o[r]);
      }
    }
  }
}

}  // namespace

template <typename IOT, int NW>
static hipError_t launch_step_t(const AmuStepArgs& a, int n_blocks, hipStream_t st) {
  hipLaunchKernelGGL((ttt_amu_step_bf<IOT, NW>), dim3(n_blocks), dim3(NW * 64), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_amu_step_bf(const AmuStepArgs& a, int n_blocks, int h, bool io_bf16, hipStream_t st) {
  if (h == 128) return io_bf16 ? launch_step_t<bf16, 4>(a, n_blocks, st) : launch_step_t<float, 4>(a, n_blocks, st);
  return io_bf16 ? launch_step_t<bf16, 8>(a, n_blocks, st) : launch_step_t<float, 8>(a, n_blocks, st);
}

}  // namespace ttt
