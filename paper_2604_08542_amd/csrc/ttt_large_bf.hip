// Chunk step at large state sizes with BF16 products (the paper's state: one
// head of 1024 with hidden 4096): the same steps as the FP32 form, on the
// BF16 GEMM core.  MSE unit, per chunk:
//   norm   K, Q rows / max(||row||, eps) in BF16; 1 / max(||v||, eps) per row
//   Z      Z = K W1           -> A = SiLU(Z), S1 = SiLU'(Z)
//   Y      Y = A W2           -> R = Y - V, E = (2/M_c) R, loss partials
//   P      P = E W2^T         -> D = P * S1
//   gW     W1 -= eta K^T D, W2 -= eta A^T E   (one launch)
//   apply  Aq = SiLU(Q W1'),  O = Aq W2'
// The paper's unit (f_W(x) = (SiLU(x W1) * (x W3)) W2, E = -eta_i v_i):
//   norm   K, Q rows; E rows
//   Z      Z1 = K W1, Z3 = K W3 in one product over K
//                             -> Hd = SiLU(Z1) Z3, G1 = Z3 SiLU'(Z1), G3 = SiLU(Z1)
//   dH     dH = E W2^T        -> D1 = dH G1, D3 = dH G3
//   gW     W1 -= K^T D1, W3 -= K^T D3, W2 -= Hd^T E   (one launch)
//   apply  Hq = SiLU(Q W1') * (Q W3') in one product over Q, O = Hq W2'
// S1, G1 and G3, which only epilogues touch, are kept in the tile-native
// layout.  Every output element is summed in a fixed order.
#include <hip/hip_runtime.h>

#include "ttt_common.h"
#include "ttt_gemm_bf.h"
#include "ttt_internal.h"
#include "ttt_large_bf.h"

namespace ttt {
namespace bfg {

// R = Y - V, E = scale R; sum of R^2 into the launch's partials (a strip's
// terms in one run, the strips in another: a lane's run over all of its tiles
// would lose a rounding per element of the chunk).
template <typename IOT>
struct EpRes : Ep<EpRes<IOT>> {
  bf16* e;
  const IOT* v;        // raw rows of the chunk
  const float* vinv;   // their normalisation factors
  int64_t v_stride;
  float* loss_part;
  int ld;
  float scale;
  float acc = 0.f;
  // the rows are held as loaded until they are used (BF16: half the registers)
  struct In {
    Raw16<IOT> v[2];
    float inv;
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in{};
    if (st.valid()) {
      in.inv = vinv[st.row()];
#pragma unroll
      for (int n = 0; n < NB; ++n) in.v[n].load(v + (int64_t)st.row() * v_stride + st.col + 32 * n + 16 * st.hf());
    }
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&y)[NB]) {
    uint32_t pe[NB][8];
    const bool ok = st.valid();
    float sum = 0.f;
#pragma unroll
    for (int n = 0; n < NB; ++n)
      pack_each(pe[n], [&](int r) {
        const float R = y[n][r] - mul_rn(in.v[n].get(r), in.inv);
        if (ok) sum = fmaf(R, R, sum);
        return scale * R;
      });
    acc += sum;
    st.template rows_out<NB>(e, ld, st.col, pe);
  }
  __device__ __forceinline__ void finish() { this->put_partial(loss_part, acc); }
};
// O rows of the chunk into the strided token tensor.
template <typename IOT>
struct EpOut : Ep<EpOut<IOT>> {
  IOT* o;
  int64_t stride_tok;
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, typename Ep<EpOut<IOT>>::In, const f32x16 (&y)[NB]) {
    if constexpr (std::is_same_v<IOT, bf16>) {
      uint32_t po[NB][8];
#pragma unroll
      for (int n = 0; n < NB; ++n) pack_each(po[n], [&](int r) { return y[n][r]; });
      st.template rows_out<NB>(o, stride_tok, st.col, po);
    } else if (st.valid()) {
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        float x[16];
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = y[n][r];
        store16(o + (int64_t)st.row() * stride_tok + st.col + 32 * n + 16 * st.hf(), x);
      }
    }
  }
};
// Row normalisation of the chunk's K, V, Q rows (one wave per token; each
// lane holds runs of 4 consecutive elements, 256 elements per wave pass, at
// most 16 passes): Kn, Qn in BF16; V's factor 1 / max(||v||, eps) per row (1
// where V is not normalised), and with `e` the unit's E = -eta_i v_i rows.
// Null outputs are skipped.
template <typename IOT>
__global__ __launch_bounds__(256) void k_norm(NormArgs p) {
  typedef IOT iov4 __attribute__((ext_vector_type(4)));
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (row >= p.rows) return;
  const int passes = p.d / 256;
#pragma unroll
  for (int which = 0; which < 3; ++which) {
    bf16* dst = static_cast<bf16*>(which == 0 ? p.Kn : which == 1 ? p.E : p.Qn);
    if (which == 1 ? !p.vinv : !dst) continue;
    const IOT* src =
        static_cast<const IOT*>(which == 0 ? p.K : which == 1 ? p.V : p.Q) + (int64_t)row * p.stride_tok;
    const bool nrm = (p.flags >> (which == 0 ? 1 : which == 1 ? 2 : 0)) & 1u;
    f32x4 x[16];
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < passes) {
        const iov4 v = *reinterpret_cast<const iov4*>(src + 256 * i + 4 * l);
        x[i] = (f32x4){(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
#pragma unroll
        for (int e = 0; e < 4; ++e) ss = fmaf(x[i][e], x[i][e], ss);
      }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, 64);
    const float inv = nrm ? 1.0f / fmaxf(sqrtf(ss), NORM_EPS) : 1.0f;
    float f = 1.0f;
    if (which == 1) {
      if (l == 0) p.vinv[row] = inv;
      if (!dst) continue;
      f = -p.eta[(int64_t)row * p.eta_stride];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < passes) {
        f32x4 y = x[i] * inv;
        if (which == 1) y = y * f;
        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
        *reinterpret_cast<u32x2*>(dst + (int64_t)row * p.d + 256 * i + 4 * l) =
            (u32x2){pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])};
      }
    }
  }
}

hipError_t launch_norm(const NormArgs& a, bool io_bf16, hipStream_t st) {
  const dim3 grid((a.rows + 3) / 4);
  if (io_bf16)
    hipLaunchKernelGGL(k_norm<bf16>, grid, dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(k_norm<float>, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

// loss[c] = (sum of the wave partials, in a fixed order) / M_c; one work-group
__global__ __launch_bounds__(256) void k_loss(const float* part, int n, float inv_m, float* out) {
  const float s = fixed_sum(part, n);
  if (threadIdx.x == 0) *out = s * inv_m;
}

template <typename IOT>
static hipError_t step_bf(const LargeStepArgs& a, hipStream_t st) {
  const int M = a.rows, d = a.d, h = a.h;
  bf16* Kn = static_cast<bf16*>(a.Kn);
  bf16* Qn = static_cast<bf16*>(a.Qn);
  bf16* E = static_cast<bf16*>(a.E);
  bf16* A = static_cast<bf16*>(a.A);
  bf16* D = static_cast<bf16*>(a.D);
  bf16* Aq = static_cast<bf16*>(a.Aq);
  bf16* S1 = static_cast<bf16*>(a.S1);
  bf16* W1 = static_cast<bf16*>(a.W1op);
  bf16* W2 = static_cast<bf16*>(a.W2op);
  NormArgs na{};
  na.K = a.K; na.V = a.V; na.Q = a.Q;
  na.stride_tok = a.stride_tok; na.flags = a.flags; na.rows = M; na.d = d;
  na.Kn = a.grad ? Kn : nullptr; na.vinv = a.grad ? a.Vn : nullptr; na.Qn = a.O ? Qn : nullptr;
  const hipError_t en = launch_norm(na, std::is_same_v<IOT, bf16>, st);
  if (en != hipSuccess) return en;
  if (a.grad) {
    EpAct<true> e1{{}, A, S1, h};
    gemm<MNMAJ, 1>(product(Kn, d, M, W1, h, d, M, h, d), e1, st);
    EpRes<IOT> e2{{}, E, static_cast<const IOT*>(a.V), a.Vn, a.stride_tok, a.loss_part, d, 2.0f / (float)M};
    const int wgs = gemm<MNMAJ, 1>(product(A, h, M, W2, d, h, M, d, h), e2, st).wgs;
    if (a.loss) hipLaunchKernelGGL(k_loss, dim3(1), dim3(256), 0, st, a.loss_part, wgs * NW, 1.0f / (float)M, a.loss);
    EpD e3{{}, D, S1, h};
    gemm<KMAJ, 1>(product(E, d, M, W2, d, h, M, h, d), e3, st);
    WArgs w{};
    w.tokens = M;
    add_weight(w, Kn, d, D, h, d, h, a.W1, a.masters_only ? nullptr : W1, -a.eta, 1);
    add_weight(w, A, h, E, d, h, d, a.W2, a.masters_only ? nullptr : W2, -a.eta, 1);
    wgrad(w, st);
  }
  if (a.O) {
    EpAct<false> e6{{}, Aq, nullptr, h};
    gemm<MNMAJ, 1>(product(Qn, d, M, W1, h, d, M, h, d), e6, st);
    EpOut<IOT> e7{{}, static_cast<IOT*>(a.O), a.stride_tok};
    gemm<MNMAJ, 1>(product(Aq, h, M, W2, d, h, M, d, h), e7, st);
  }
  return hipGetLastError();
}

template <typename IOT>
static hipError_t amu_step_bf(const LargeAmuArgs& a, hipStream_t st) {
  const int M = a.rows, d = a.d, h = a.h;
  bf16* Kn = static_cast<bf16*>(a.Kn);
  bf16* Qn = static_cast<bf16*>(a.Qn);
  bf16* E = static_cast<bf16*>(a.E);
  bf16* Hd = static_cast<bf16*>(a.Hd);
  bf16* G1 = static_cast<bf16*>(a.G1);
  bf16* G3 = static_cast<bf16*>(a.G3);
  bf16* D1 = static_cast<bf16*>(a.D1);
  bf16* D3 = static_cast<bf16*>(a.D3);
  bf16* W1 = static_cast<bf16*>(a.W1op);
  bf16* W2 = static_cast<bf16*>(a.W2op);
  bf16* W3 = static_cast<bf16*>(a.W3op);
  NormArgs na{};
  na.K = a.K; na.V = a.V; na.Q = a.Q;
  na.stride_tok = a.stride_tok; na.flags = a.flags; na.rows = M; na.d = d;
  na.Kn = a.grad ? Kn : nullptr; na.vinv = a.grad ? a.Vn : nullptr; na.E = E; na.Qn = a.O ? Qn : nullptr;
  na.eta = a.eta; na.eta_stride = a.eta_stride;
  const hipError_t en = launch_norm(na, std::is_same_v<IOT, bf16>, st);
  if (en != hipSuccess) return en;
  if (a.grad) {
    GemmArgs z = product(Kn, d, M, W1, h, d, M, h, d);
    z.B[1] = W3;
    EpSwi<true> e2{{}, Hd, G1, G3, h};
    gemm<MNMAJ, 2>(z, e2, st);
    EpD2 e3{{}, G1, G3, D1, D3, h};
    gemm<KMAJ, 1>(product(E, d, M, W2, d, h, M, h, d), e3, st);
    // the step sizes are inside the loss: W <- W - grad
    WArgs w{};
    w.tokens = M;
    add_weight(w, Kn, d, D1, h, d, h, a.W1, a.write_op ? W1 : nullptr, -1.0f, 1, a.from1);
    add_weight(w, Kn, d, D3, h, d, h, a.W3, a.write_op ? W3 : nullptr, -1.0f, 1, a.from3);
    add_weight(w, Hd, h, E, d, h, d, a.W2, a.write_op ? W2 : nullptr, -1.0f, 1, a.from2);
    wgrad(w, st);
  }
  if (a.O) {
    GemmArgs z = product(Qn, d, M, W1, h, d, M, h, d);
    z.B[1] = W3;
    EpSwi<false> e7{{}, Hd, nullptr, nullptr, h};
    gemm<MNMAJ, 2>(z, e7, st);
    EpOut<IOT> e8{{}, static_cast<IOT*>(a.O), a.stride_tok};
    gemm<MNMAJ, 1>(product(Hd, h, M, W2, d, h, M, d, h), e8, st);
  }
  return hipGetLastError();
}

}  // namespace bfg

hipError_t launch_large_step_bf(const LargeStepArgs& a, bool io_bf16, hipStream_t st) {
  return io_bf16 ? bfg::step_bf<bf16>(a, st) : bfg::step_bf<float>(a, st);
}
hipError_t launch_large_amu_step_bf(const LargeAmuArgs& a, bool io_bf16, hipStream_t st) {
  return io_bf16 ? bfg::amu_step_bf<bf16>(a, st) : bfg::amu_step_bf<float>(a, st);
}

}  // namespace ttt

// Tile choice of the BF16 GEMM core, for tests that have to reach every tile:
// rows of the tiles of a product of `nmat` matrices, and rows * 1000 + columns
// of the tiles of a launch of weight terms.  Not part of the C ABI.
extern "C" int32_t ttt_internal_gemm_tile(int32_t M, int32_t N, int32_t nmat, int64_t K) {
  using namespace ttt::bfg;
  const int cfg = pick_tile(M, N, nmat, K);
  return cfg == T_L ? 256 : cfg == T_M ? 192 : 128;
}
extern "C" int32_t ttt_internal_wgrad_tile(int32_t np, const int32_t* M, const int32_t* N, const int32_t* nterm,
                                           int32_t nsplit) {
  using namespace ttt::bfg;
  if (np < 1 || np > 3) return 0;
  WArgs a{};
  a.nsplit = nsplit;
  for (int p = 0; p < np; ++p) {
    add_weight(a, nullptr, 0, nullptr, 0, M[p], N[p], nullptr, nullptr, 1.0f, 1);
    a.p[p].nterm = nterm[p];
  }
  const WTile t = pick_wgrad(a);
  return t.bm * 1000 + t.bn;
}
