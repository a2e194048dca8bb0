// The layer around the memory unit in BF16 on the BF16 GEMM core: the
// query-key-value projection, the gated output projection, and their reverse
// mode (the FP32 form and the formulas are in ttt_gcm.hip).
//   forward   [Q | K | V] = X Wqkv (+ bqkv);  Y = alpha * (O Wo (+ bo)) + X
//   phase 0   P = X Wqkv (+ bqkv)
//   phase 1   G = O Wo (+ bo) stays in the accumulators: dG = alpha dY,
//             partials of dalpha = sum G dY and dbo = sum dG; dWo = O^T dG;
//             dO = dG Wo^T
//   phase 2   dWqkv = X^T dP; dbqkv = sum dP; dX = dY + dP Wqkv^T
// The weight gradients are a few tiles (16 of 256 x 256 for dWo at D = 1024)
// contracted over every token, so their tokens are cut into runs, one
// work-group per tile and run, and the runs' FP32 sums added in run order
// (dWo and dWqkv at 43,968 tokens and D = 1024: 449 and 447 us as one run per
// 128 x 128 tile).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "ttt_common.h"
#include "ttt_gemm_bf.h"
#include "ttt_internal.h"

namespace ttt {
namespace bfg {

// 16 consecutive floats at any 4-byte address.
__device__ __forceinline__ void load16u(const float* p, float (&x)[16]) {
  typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f4u v = reinterpret_cast<const f4u*>(p)[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
  }
}

// Product (+ bias per column) stored at a row pitch; with `third` > 0 the
// columns are split into three tensors of that width (a wave's 64 columns
// never straddle two: the width is a multiple of 128).
struct EpBias : Ep<EpBias> {
  bf16* out[3];
  const float* bias;  // nullable
  int64_t ld;
  int third;
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, In, const f32x16 (&x)[NB]) {
    uint32_t pk[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      float b[16];
      if (bias) {
        load16u(bias + st.col + 32 * n + 16 * st.hf(), b);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) b[r] = 0.f;
      }
      pack_each(pk[n], [&](int r) { return x[n][r] + b[r]; });
    }
    const int t = third > 0 ? (st.col >= third) + (st.col >= 2 * third) : 0;
    bf16* o = t == 0 ? out[0] : t == 1 ? out[1] : out[2];
    st.template rows_out<NB>(o, ld, st.col - t * third, pk);
  }
};
// Y = alpha * (value + bias) + X, one 32-column block of the wave after the
// other, so that a block's alpha, bias and all of its X rows (requested
// together) fit beside the accumulators.
struct EpGate : Ep<EpGate> {
  bf16* y;
  const bf16* x;
  const float* bias;  // nullable
  const float* alpha;
  int ld;
  template <int MB, int NB>
  __device__ __forceinline__ void tile(Strip st, int row0, f32x16 (&acc)[MB][NB]) {
    if (row0 >= st.rows) return;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int c0 = st.col + 32 * n, c = c0 + 16 * st.hf();
      Raw16<bf16> xr[MB];
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        xr[i] = {};
        if (row0 + 32 * i + st.l32() < st.rows) xr[i].load(x + (int64_t)(row0 + 32 * i + st.l32()) * ld + c);
      }
      float a[16], b[16];
      load16u(alpha + c, a);
      if (bias) {
        load16u(bias + c, b);
      } else {
#pragma unroll
        for (int r = 0; r < 16; ++r) b[r] = 0.f;
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        st.row0 = row0 + 32 * i;
        if (st.row0 >= st.rows) break;
        uint32_t pk[1][8];
        pack_each(pk[0], [&](int r) { return fmaf(a[r], acc[i][n][r] + b[r], xr[i].get(r)); });
        st.template rows_out<1>(y, ld, c0, pk);
      }
    }
  }
};
// out = add + value.
struct EpAdd : Ep<EpAdd> {
  bf16* out;
  const bf16* add;
  int ld;
  struct In {
    Raw16<bf16> x[2];
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in{};
    if (st.valid()) {
#pragma unroll
      for (int n = 0; n < NB; ++n) in.x[n].load(add + (int64_t)st.row() * ld + st.col + 32 * n + 16 * st.hf());
    }
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&v)[NB]) {
    uint32_t pk[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n) pack_each(pk[n], [&](int r) { return in.x[n].get(r) + v[n][r]; });
    st.template rows_out<NB>(out, ld, st.col, pk);
  }
};
// Gate adjoint on G = value + bias: dG = alpha dY rows, and over the wave's
// rows of the tile the column sums of G dY and of dG: part[row / 32 of the
// wave's first row][2 ld].
struct EpGateBwd : Ep<EpGateBwd> {
  bf16* dg;
  const bf16* dy;
  const float* bias;  // nullable
  const float* alpha;
  float* part;
  int ld;
  // Sums v over the 32 lanes of a half; lane l32 returns the sum of column
  // l32 / 2 (each exchange halves the columns a lane still carries).
  __device__ __forceinline__ static float columns(float (&v)[16]) {
    const int l = threadIdx.x & 31;
#pragma unroll
    for (int k = 8; k >= 1; k >>= 1) {
      const int m = 2 * k;  // lane distance 16, 8, 4, 2
      const bool hi = l & m;
#pragma unroll
      for (int i = 0; i < k; ++i) {
        const float a = v[i], b = v[i + k];  // (a choice between the elements themselves puts v in scratch)
        v[i] = (hi ? b : a) + __shfl_xor(hi ? a : b, m, 64);
      }
    }
    return v[0] + __shfl_xor(v[0], 1, 64);
  }
  template <int MB, int NB>
  __device__ __forceinline__ void tile(Strip st, int row0, f32x16 (&acc)[MB][NB]) {
    if (row0 >= st.rows) return;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int c0 = st.col + 32 * n, c = c0 + 16 * st.hf();
      float a[16], sa[16], sd[16];
      load16u(alpha + c, a);
#pragma unroll
      for (int r = 0; r < 16; ++r) sa[r] = sd[r] = 0.f;
      Raw16<bf16> nx{};
      if (row0 + st.l32() < st.rows) nx.load(dy + (int64_t)(row0 + st.l32()) * ld + c);
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        st.row0 = row0 + 32 * i;
        if (st.row0 >= st.rows) break;
        const Raw16<bf16> y = nx;
        nx = {};
        if (i + 1 < MB && st.row() + 32 < st.rows) nx.load(dy + (int64_t)(st.row() + 32) * ld + c);
        uint32_t pk[1][8];
        pack_each(pk[0], [&](int r) {
          const float d = y.get(r);
          sa[r] = fmaf(acc[i][n][r], d, sa[r]);
          sd[r] += d;
          return a[r] * d;
        });
        st.template rows_out<1>(dg, ld, c0, pk);
      }
      const float ta = columns(sa), td = columns(sd);
      if (!(threadIdx.x & 1)) {
        const int cc = c + (st.l32() >> 1);
        float* o = part + (int64_t)(row0 >> 5) * 2 * ld + cc;
        o[0] = bias ? fmaf(bias[cc], td, ta) : ta;  // sum (value + bias) dY
        o[ld] = alpha[cc] * td;
      }
    }
  }
};

// out[c] = sum over i < n of part[i * step * pitch + c]: 16 runs of
// consecutive i in order, then the runs in order.  64 columns per work-group.
__global__ __launch_bounds__(1024) void k_colsums(const float* part, int n, int64_t pitch, int cols, float* out) {
  __shared__ float run[16][64];
  const int c = blockIdx.x * 64 + (threadIdx.x & 63), g = threadIdx.x >> 6, per = (n + 15) / 16;
  float s = 0.f;
  if (c < cols)
    for (int i = g * per; i < min(n, g * per + per); ++i) s += part[(int64_t)i * pitch + c];
  run[g][threadIdx.x & 63] = s;
  __syncthreads();
  if (g == 0 && c < cols) {
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) t += run[i][threadIdx.x];
    out[c] = t;
  }
}
// Column sums of a slab of 256 rows of a [rows][ld] tensor: part[slab][cols].
// 256 columns per work-group: 32 threads of 8 columns on each of 8 runs of 32
// rows, the runs added in order.
__global__ __launch_bounds__(256) void k_slab_sums(const bf16* a, int64_t ld, int rows, int cols, float* part) {
  __shared__ float run[8][256];
  const int t = threadIdx.x & 31, g = threadIdx.x >> 5, c = blockIdx.x * 256 + 8 * t;
  const int r0 = blockIdx.y * 256 + 32 * g;
  float s[8] = {};
  if (c < cols) {
#pragma unroll 8
    for (int i = 0; i < 32; ++i) {
      if (r0 + i >= rows) break;
      const u32x4 v = *reinterpret_cast<const u32x4*>(a + (int64_t)(r0 + i) * ld + c);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[2 * e] += __uint_as_float(v[e] << 16);
        s[2 * e + 1] += __uint_as_float(v[e] & 0xffff0000u);
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) run[g][8 * t + e] = s[e];
  __syncthreads();
  const int cc = blockIdx.x * 256 + threadIdx.x;
  if (cc >= cols) return;
  float o = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) o += run[i][threadIdx.x];
  part[(int64_t)blockIdx.y * cols + cc] = o;
}
// out = part[0] + part[1] + ... + part[n-1], n4 float4 each.
__global__ __launch_bounds__(256) void k_runs(const float* part, int n, int64_t n4, float* out) {
  const int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x;
  if (i >= n4) return;
  const f32x4* p = reinterpret_cast<const f32x4*>(part) + i;
  const f32x4 s = add_shards((f32x4){0.f, 0.f, 0.f, 0.f}, p, n4, n);
  reinterpret_cast<f32x4*>(out)[i] = s;
}

// dW = A^T B over all tokens, the tokens cut into runs.
static void weight_grad(const bf16* A, int lda, const bf16* B, int ldb, int M, int N, int tokens, int runs, float* dw,
                        float* part, hipStream_t st) {
  WArgs w{};
  w.tokens = tokens;
  w.nsplit = runs;
  add_weight(w, A, lda, B, ldb, M, N, runs > 1 ? part : dw, nullptr, 1.0f, 0);
  wgrad(w, st);
  if (runs > 1) {
    const int64_t n4 = (int64_t)M * N / 4;
    hipLaunchKernelGGL(k_runs, dim3((unsigned)((n4 + 255) / 256)), dim3(256), 0, st, part, runs, n4, dw);
  }
}

}  // namespace bfg

// The rows of one launch are limited so that an operand slab stays within
// the 32-bit byte range of a buffer resource.
hipError_t launch_gcm_gemm_bf(const GcmGemmArgs& a, hipStream_t st) {
  using namespace bfg;
  const int D = a.D;
  const int64_t slab = std::max<int64_t>(128, ((int64_t(1) << 31) - 1) / ((int64_t)D * 2) / 128 * 128);
  for (int64_t r0 = 0; r0 < a.rows; r0 += slab) {
    const int rows = (int)std::min<int64_t>(slab, a.rows - r0);
    const int64_t off = r0 * D;
    const bf16* w = static_cast<const bf16*>(a.w);
    if (a.kind == 0) {
      EpBias ep{{}, {static_cast<bf16*>(a.q) + off, static_cast<bf16*>(a.k) + off, static_cast<bf16*>(a.v) + off},
                a.bias, D, D};
      gemm<MNMAJ, 1>(product(static_cast<const bf16*>(a.x) + off, D, rows, w, 3 * D, D, rows, 3 * D, D), ep, st);
    } else {
      EpGate ep{{}, static_cast<bf16*>(a.y) + off, static_cast<const bf16*>(a.x) + off, a.bias, a.alpha, D};
      gemm<MNMAJ, 1>(product(static_cast<const bf16*>(a.o) + off, D, rows, w, D, D, rows, D, D), ep, st);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_gcm_bwd_bf(const GcmBwdArgs& a, hipStream_t st) {
  using namespace bfg;
  const int D = a.D, rows = (int)a.rows, D3 = 3 * D;
  auto C = [](const void* p) { return static_cast<const bf16*>(p); };
  auto P = [](void* p) { return static_cast<bf16*>(p); };
  if (a.phase == 0) {
    EpBias ep{{}, {P(a.P), nullptr, nullptr}, a.bqkv, D3, 0};
    gemm<MNMAJ, 1>(product(C(a.X), D, rows, C(a.Wqkv), D3, D, rows, D3, D), ep, st);
  } else if (a.phase == 1) {
    const bf16* O = C(a.O);
    EpGateBwd eg{{}, P(a.dG), C(a.dY), a.bo, a.alpha, a.part, D};
    const GemmArgs g = product(O, D3, rows, C(a.Wo), D, D, rows, D, D);
    // the partials sit at the first rows of the waves' shares of the tiles
    const int step = gemm<MNMAJ, 1>(g, eg, st).blocks;
    const int n = ((rows + 31) / 32 + step - 1) / step;
    const int64_t pitch = (int64_t)step * 2 * D;
    const dim3 cs((D + 63) / 64);
    hipLaunchKernelGGL(k_colsums, cs, dim3(1024), 0, st, a.part, n, pitch, D, a.dalpha);
    if (a.dbo) hipLaunchKernelGGL(k_colsums, cs, dim3(1024), 0, st, a.part + D, n, pitch, D, a.dbo);
    weight_grad(O, D3, C(a.dG), D, D, D, rows, a.runs_o, a.dWo, a.part_o, st);
    EpBias eo{{}, {P(a.dO), nullptr, nullptr}, nullptr, D3, 0};
    gemm<KMAJ, 1>(product(C(a.dG), D, rows, C(a.Wo), D, D, rows, D, D), eo, st);
  } else {
    const bf16* dP = C(a.dP);
    weight_grad(C(a.X), D, dP, D3, D, D3, rows, a.runs_p, a.dWqkv, a.part_p, st);
    if (a.dbqkv) {
      const int ns = (rows + 255) / 256;
      hipLaunchKernelGGL(k_slab_sums, dim3((D3 + 255) / 256, ns), dim3(256), 0, st, dP, (int64_t)D3, rows, D3, a.part);
      hipLaunchKernelGGL(k_colsums, dim3((D3 + 63) / 64), dim3(1024), 0, st, a.part, ns, (int64_t)D3, D3, a.dbqkv);
    }
    EpAdd ex{{}, P(a.dX), C(a.dY), D};
    gemm<KMAJ, 1>(product(dP, D3, rows, C(a.Wqkv), D3, D, rows, D, D3), ex, st);
  }
  return hipGetLastError();
}

}  // namespace ttt
