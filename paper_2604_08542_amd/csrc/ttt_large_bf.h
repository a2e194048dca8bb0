// Pieces shared by the BF16 forward and reverse steps at large state sizes.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ttt_gemm_bf.h"
#include "ttt_internal.h"

namespace ttt {

namespace bfg {

// Row normalisation of a chunk (see k_norm); null outputs are skipped.
struct NormArgs {
  const void* K;
  const void* V;
  const void* Q;
  int64_t stride_tok;
  uint32_t flags;
  int32_t rows, d;
  void* Kn;
  void* Qn;
  float* vinv;  // [rows]: V's normalisation factor
  void* E;      // the unit's -eta_i v_i rows (with vinv)
  const float* eta;
  int64_t eta_stride;
};
hipError_t launch_norm(const NormArgs& a, bool io_bf16, hipStream_t st);

// Sum of part[0..n) by a work-group of 256 threads in a fixed order: thread t
// adds the run part[t c .. t c + c) in index order (c = ceil(n / 256)), then
// the run sums are added in a tree.  Valid in thread 0.
__device__ __forceinline__ float fixed_sum(const float* part, int n) {
  __shared__ float run[256];
  const int t = threadIdx.x, c = (n + 255) / 256;
  const int i0 = t * c, i1 = i0 + c < n ? i0 + c : n;
  float s = 0.f;
  for (int i = i0; i < i1; ++i) s += part[i];
  run[t] = s;
#pragma unroll
  for (int m = 128; m >= 1; m >>= 1) {
    __syncthreads();
    if (t < m) run[t] += run[t + m];
  }
  return run[0];
}

// x rounded to BF16.
__device__ __forceinline__ float round_bf(float x) { return __uint_as_float(pack_bf16x2(x, x) << 16); }

// A = SiLU(Z) and, for the gradient, S1 = SiLU'(Z).
template <bool GRAD>
struct EpAct : Ep<EpAct<GRAD>> {
  bf16* a;
  bf16* s1;
  int ld;
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, typename Ep<EpAct<GRAD>>::In, const f32x16 (&z)[NB]) {
    uint32_t pa[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      f32x16 sp;
#pragma unroll
      for (int r = 0; r < 16; r += 2) {
        float v[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float zz = z[n][r + e], sg = sigmoid(zz);
          v[e] = zz * sg;
          sp[r + e] = fmaf(v[e], 1.0f - sg, sg);
        }
        pa[n][r / 2] = pack_bf16x2(v[0], v[1]);
      }
      if constexpr (GRAD) {
        uint32_t ps[8];
        pack_each(ps, [&](int r) { return sp[r]; });
        nat_store(s1, nat_at(st.row0, st.col + 32 * n, ld), ps);
      }
    }
    st.template rows_out<NB>(a, ld, st.col, pa);
  }
};
// out = value * factor (D = P S1; dZq = (dO W2^T) s'(Zq)).
struct EpD : Ep<EpD> {
  bf16* d;
  const bf16* s1;
  int ld;
  struct In {
    Nat s[2];
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in;
#pragma unroll
    for (int n = 0; n < NB; ++n) in.s[n] = nat_load(s1, nat_at(st.row0, st.col + 32 * n, ld));
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&p)[NB]) {
    uint32_t pd[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n) pack_each(pd[n], [&](int r) { return p[n][r] * in.s[n].get(r); });
    st.template rows_out<NB>(d, ld, st.col, pd);
  }
};
// Z1 (block 0) and Z3 (block 1): Hd = SiLU(Z1) Z3 and, for the gradient, the
// factors of the hidden adjoint G1 = Z3 SiLU'(Z1), G3 = SiLU(Z1).  Z3 enters
// as an operand value (rounded to BF16).
template <bool GRAD>
struct EpSwi : Ep<EpSwi<GRAD>> {
  bf16* hd;
  bf16* g1;
  bf16* g3;
  int ld;
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, typename Ep<EpSwi<GRAD>>::In, const f32x16 (&z)[NB]) {
    static_assert(NB == 2, "one block per matrix");
    f32x16 h, f1, f3;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float z1 = z[0][r], z3 = round_bf(z[1][r]), sg = sigmoid(z1), s = z1 * sg;
      h[r] = s * z3;
      f1[r] = z3 * fmaf(s, 1.0f - sg, sg);
      f3[r] = s;
    }
    uint32_t pk[1][8];
    pack_each(pk[0], [&](int r) { return h[r]; });
    st.template rows_out<1>(hd, ld, st.col, pk);
    if constexpr (GRAD) {
      const int64_t at = nat_at(st.row0, st.col, ld);
      pack_each(pk[0], [&](int r) { return f1[r]; });
      nat_store(g1, at, pk[0]);
      pack_each(pk[0], [&](int r) { return f3[r]; });
      nat_store(g3, at, pk[0]);
    }
  }
};
// dH = E W2^T: D1 = dH G1, D3 = dH G3 (in the reverse mode: dZq1, dZq3).
struct EpD2 : Ep<EpD2> {
  const bf16* g1;
  const bf16* g3;
  bf16* d1;
  bf16* d3;
  int ld;
  struct In {
    Nat a[2], b[2];
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int64_t at = nat_at(st.row0, st.col + 32 * n, ld);
      in.a[n] = nat_load(g1, at);
      in.b[n] = nat_load(g3, at);
    }
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&dh)[NB]) {
    uint32_t pk[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n) pack_each(pk[n], [&](int r) { return dh[n][r] * in.a[n].get(r); });
    st.template rows_out<NB>(d1, ld, st.col, pk);
#pragma unroll
    for (int n = 0; n < NB; ++n) pack_each(pk[n], [&](int r) { return dh[n][r] * in.b[n].get(r); });
    st.template rows_out<NB>(d3, ld, st.col, pk);
  }
};

}  // namespace bfg
}  // namespace ttt
