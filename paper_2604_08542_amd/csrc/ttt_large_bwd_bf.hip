// Reverse steps at large state sizes with BF16 products, on the BF16 GEMM
// core.  The mathematics is that of the FP32 form (ttt_large_bwd.hip); what
// differs is how the products are grouped, so that an operand is read once
// for every weight it meets and sums of products stay in the accumulators.
//
// MSE unit, W = W_c, W' = W_{c+1}, Wh the adjoint of W':
//   apply   Zq = Q W1' -> Aq, s'(Zq);  dZq = (dO W2'^T) s'(Zq);
//           Wh2 += Aq^T dO, Wh1 += Q^T dZq (one launch);  dq = dZq W1'^T
//   update  Z = K W1 -> A, s'(Z), s''(Z)
//           [A W2 | A Wh2] = [Y | u2] -> E = (2/M)(Y - V), dE = -eta u2, deta -= <u2, E>
//           [E W2^T | E Wh2^T] = [P | EWh] -> D = P s'(Z)
//           u1 = K Wh1 -> dP = -eta u1 s'(Z), dZa = -eta u1 P s''(Z), deta -= <u1, D>
//           dP W2 -> dY = (2/M)(dE + dP W2), dv = -dY
//           dY W2^T -> dZ = dZa + (-eta EWh + dY W2^T) s'(Z)
//           dk = -eta D Wh1^T + dZ W1^T (one sum)
//           Wh2 += dP^T E, then A^T dY; Wh1 += K^T dZ (one launch)
// The paper's unit, E_i = -eta_i v_i:
//   apply   [Q W1' | Q W3'] -> Hq, F1, F3;  dZq1, dZq3 = (dO W2'^T) F1, F3;
//           Wh1 += Q^T dZq1, Wh2 += Hq^T dO, Wh3 += Q^T dZq3 (one launch);
//           dq = dZq1 W1'^T + dZq3 W3'^T (one sum)
//   update  [K W1 | K W3 | K Wh1 | K Wh3] = [Z1 | Z3 | Zd1 | Zd3] ->
//             Hd = S Z3, Hdot = Sd Z3 + S Zd3 with S = s(Z1), Sd = s'(Z1) Zd1,
//             T2 = s''(Z1) Zd1
//           [E W2^T | E Wh2^T] = [dH | dHh] ->
//             aZ1 = dH Z3 T2 + (dH Zd3 + dHh Z3) s'(Z1), aZ3 = dH Sd + dHh S,
//             aZd1 = dH Z3 s'(Z1), aZd3 = dH S
//           Ydot = Hdot W2 + Hd Wh2 (one sum) -> dv = eta Ydot, deta = <v, Ydot>
//           dk = -(aZ1 W1^T + aZ3 W3^T + aZd1 Wh1^T + aZd3 Wh3^T) (one sum)
//           W1 -= K^T aZ1, W2 -= Hdot^T E, W3 -= K^T aZ3 (one launch)
// Z, Z3, Zd1 and so on never leave the registers; the factors that a later
// epilogue needs are kept tile-native in BF16.
#include <hip/hip_runtime.h>

#include "ttt_common.h"
#include "ttt_gemm_bf.h"
#include "ttt_internal.h"
#include "ttt_large_bf.h"

namespace ttt {
namespace bfg {

// s(z), s'(z), s''(z) of SiLU.
__device__ __forceinline__ void silu3(float z, float& s, float& s1, float& s2) {
  const float sg = sigmoid(z);
  s = z * sg;
  s1 = fmaf(s, 1.0f - sg, sg);
  s2 = sg * (1.0f - sg) * fmaf(z, 1.0f - 2.0f * sg, 2.0f);
}

// Z: A rows; s'(Z), s''(Z) tile-native.
struct EpAct3 : Ep<EpAct3> {
  bf16* a;
  bf16* s1;
  bf16* s2;
  int ld;
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, In, const f32x16 (&z)[NB]) {
    uint32_t pa[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      uint32_t p1[8], p2[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        float s[2], d1[2], d2[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) silu3(z[n][2 * q + e], s[e], d1[e], d2[e]);
        pa[n][q] = pack_bf16x2(s[0], s[1]);
        p1[q] = pack_bf16x2(d1[0], d1[1]);
        p2[q] = pack_bf16x2(d2[0], d2[1]);
      }
      const int64_t at = nat_at(st.row0, st.col + 32 * n, ld);
      nat_store(s1, at, p1);
      nat_store(s2, at, p2);
    }
    st.template rows_out<NB>(a, ld, st.col, pa);
  }
};
// [Y | u2]: E rows, dE = -eta u2 (FP32); -<u2, E> into the partials.
template <typename IOT>
struct EpYU : Ep<EpYU<IOT>> {
  bf16* e;
  float* de;
  const IOT* v;
  const float* vinv;
  int64_t v_stride;
  float* part;
  int ld;
  float scale, eta;
  float acc = 0.f;
  struct In {
    Raw16<IOT> v;
    float inv;
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in{};
    if (st.valid()) {
      in.inv = vinv[st.row()];
      in.v.load(v + (int64_t)st.row() * v_stride + st.col + 16 * st.hf());
    }
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&x)[NB]) {
    uint32_t pk[1][8];
    pack_each(pk[0], [&](int r) { return scale * (x[0][r] - mul_rn(in.v.get(r), in.inv)); });
    Nat ev;
    ev.v[0] = (u32x4){pk[0][0], pk[0][1], pk[0][2], pk[0][3]};
    ev.v[1] = (u32x4){pk[0][4], pk[0][5], pk[0][6], pk[0][7]};
    if (st.valid()) {
      float dv[16], sum = 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        sum = fmaf(-x[1][r], ev.get(r), sum);
        dv[r] = -eta * x[1][r];
      }
      acc += sum;
      store16(de + (int64_t)st.row() * ld + st.col + 16 * st.hf(), dv);
    }
    st.template rows_out<1>(e, ld, st.col, pk);
  }
  __device__ __forceinline__ void finish() { this->put_partial(part, acc); }
};
// [P | EWh]: P, EWh and D tile-native, D rows (an operand).
struct EpPE : Ep<EpPE> {
  bf16* d;
  bf16* dn;
  bf16* p;
  bf16* ewh;
  const bf16* s1;
  int ld;
  typedef Nat In;
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    return nat_load(s1, nat_at(st.row0, st.col, ld));
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&x)[NB]) {
    const int64_t at = nat_at(st.row0, st.col, ld);
    uint32_t pk[1][8];
    pack_each(pk[0], [&](int r) { return x[0][r]; });
    nat_store(p, at, pk[0]);
    pack_each(pk[0], [&](int r) { return x[1][r]; });
    nat_store(ewh, at, pk[0]);
    pack_each(pk[0], [&](int r) { return x[0][r] * in.get(r); });
    nat_store(dn, at, pk[0]);
    st.template rows_out<1>(d, ld, st.col, pk);
  }
};
// u1 = K Wh1: dP = -eta u1 s'(Z) rows, dZa = -eta u1 P s''(Z) tile-native;
// -<u1, D> into the partials.  dza may be s2: a lane writes what it has read.
struct EpU1 : Ep<EpU1> {
  static constexpr bool AHEAD = false;
  bf16* dp;
  bf16* dza;
  const bf16* d;
  const bf16* s1;
  const bf16* p;
  const bf16* s2;
  float* part;
  int ld;
  float eta;
  float acc = 0.f;
  struct In {
    Nat d[2], s1[2], p[2], s2[2];
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int64_t at = nat_at(st.row0, st.col + 32 * n, ld);
      in.d[n] = nat_load(d, at);
      in.s1[n] = nat_load(s1, at);
      in.p[n] = nat_load(p, at);
      in.s2[n] = nat_load(s2, at);
    }
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&u)[NB]) {
    uint32_t pd[NB][8];
    const bool ok = st.valid();
    float sum = 0.f;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      uint32_t pz[8];
      pack_each(pz, [&](int r) {
        const float dd = -eta * u[n][r];
        if (ok) sum = fmaf(-u[n][r], in.d[n].get(r), sum);
        return dd * in.p[n].get(r) * in.s2[n].get(r);
      });
      nat_store(dza, nat_at(st.row0, st.col + 32 * n, ld), pz);
      pack_each(pd[n], [&](int r) { return (-eta * u[n][r]) * in.s1[n].get(r); });
    }
    acc += sum;
    st.template rows_out<NB>(dp, ld, st.col, pd);
  }
  __device__ __forceinline__ void finish() { this->put_partial(part, acc); }
};
// dP W2: dY = scale (dE + dP W2) rows, dv = -dY (FP32).
struct EpDY : Ep<EpDY> {
  bf16* dy;
  float* dv;
  const float* de;
  int ld;
  float scale;
  struct In {
    float de[2][16];
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in{};
    if (st.valid()) {
#pragma unroll
      for (int n = 0; n < NB; ++n) load16(de + (int64_t)st.row() * ld + st.col + 32 * n + 16 * st.hf(), in.de[n]);
    }
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&x)[NB]) {
    uint32_t pk[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      float y[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = scale * (in.de[n][r] + x[n][r]);
      pack_each(pk[n], [&](int r) { return y[r]; });
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = -y[r];
      if (st.valid()) store16(dv + (int64_t)st.row() * ld + st.col + 32 * n + 16 * st.hf(), y);
    }
    st.template rows_out<NB>(dy, ld, st.col, pk);
  }
};
// dY W2^T: dA = -eta EWh + dY W2^T, dZ = dZa + dA s'(Z) rows.
struct EpDZ : Ep<EpDZ> {
  static constexpr bool AHEAD = false;
  bf16* dz;
  const bf16* ewh;
  const bf16* dza;
  const bf16* s1;
  int ld;
  float eta;
  struct In {
    Nat e[2], z[2], s[2];
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    In in;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int64_t at = nat_at(st.row0, st.col + 32 * n, ld);
      in.e[n] = nat_load(ewh, at);
      in.z[n] = nat_load(dza, at);
      in.s[n] = nat_load(s1, at);
    }
    return in;
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&x)[NB]) {
    uint32_t pk[NB][8];
#pragma unroll
    for (int n = 0; n < NB; ++n)
      pack_each(pk[n], [&](int r) {
        return fmaf(fmaf(-eta, in.e[n].get(r), x[n][r]), in.s[n].get(r), in.z[n].get(r));
      });
    st.template rows_out<NB>(dz, ld, st.col, pk);
  }
};
// FP32 rows: out = scale * value.
struct EpF32 : Ep<EpF32> {
  float* out;
  int ld;
  float scale;
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, In, const f32x16 (&x)[NB]) {
    if (!st.valid()) return;
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      float y[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) y[r] = scale * x[n][r];
      store16(out + (int64_t)st.row() * ld + st.col + 32 * n + 16 * st.hf(), y);
    }
  }
};
// [Z1 | Z3 | Zd1 | Zd3] of the paper's unit: Hd = S Z3, Hdot = Sd Z3 + S Zd3
// rows; S = s(Z1), S1 = s'(Z1), Z3, Zd3, Sd = S1 Zd1, T2 = s''(Z1) Zd1
// tile-native.  Z3, Zd3, S1 and s'' enter the products rounded to BF16.
struct EpTan : Ep<EpTan> {
  bf16* hd;
  bf16* hdot;
  bf16* s;
  bf16* s1;
  bf16* z3;
  bf16* zd3;
  bf16* sd;
  bf16* t2;
  int ld;
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, In, const f32x16 (&x)[NB]) {
    static_assert(NB == 4, "one block per matrix");
    const int64_t at = nat_at(st.row0, st.col, ld);
    uint32_t ph[1][8], px[1][8], pk[6][8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      float a[2], b1[2], b2[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) silu3(x[0][2 * q + e], a[e], b1[e], b2[e]);
      const uint32_t ps = pack_bf16x2(a[0], a[1]), p1 = pack_bf16x2(b1[0], b1[1]), p2 = pack_bf16x2(b2[0], b2[1]);
      const uint32_t pz = pack_bf16x2(x[1][2 * q], x[1][2 * q + 1]), pe = pack_bf16x2(x[3][2 * q], x[3][2 * q + 1]);
      float h[2], hx[2], sdv[2], tv[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        auto up = [&](uint32_t w) { return __uint_as_float(e ? (w & 0xffff0000u) : (w << 16)); };
        const float zd1 = x[2][2 * q + e];
        h[e] = a[e] * up(pz);
        sdv[e] = up(p1) * zd1;
        tv[e] = up(p2) * zd1;
        hx[e] = fmaf(sdv[e], up(pz), mul_rn(up(ps), up(pe)));
      }
      ph[0][q] = pack_bf16x2(h[0], h[1]);
      px[0][q] = pack_bf16x2(hx[0], hx[1]);
      pk[0][q] = ps;
      pk[1][q] = p1;
      pk[2][q] = pz;
      pk[3][q] = pe;
      pk[4][q] = pack_bf16x2(sdv[0], sdv[1]);
      pk[5][q] = pack_bf16x2(tv[0], tv[1]);
    }
    nat_store(s, at, pk[0]);
    nat_store(s1, at, pk[1]);
    nat_store(z3, at, pk[2]);
    nat_store(zd3, at, pk[3]);
    nat_store(sd, at, pk[4]);
    nat_store(t2, at, pk[5]);
    st.template rows_out<1>(hd, ld, st.col, ph);
    st.template rows_out<1>(hdot, ld, st.col, px);
  }
};
// [dH | dHh]: the four adjoints (dHh rounded to BF16).
struct EpAdj : Ep<EpAdj> {
  static constexpr bool AHEAD = false;
  const bf16* z3;
  const bf16* sd;
  const bf16* s;
  const bf16* zd3;
  const bf16* s1;
  const bf16* t2;
  bf16* az1;
  bf16* az3;
  bf16* azd1;
  bf16* azd3;
  int ld;
  struct In {
    Nat z3, sd, s, zd3, s1, t2;
  };
  template <int NB>
  __device__ __forceinline__ In pre(const Strip& st) const {
    const int64_t at = nat_at(st.row0, st.col, ld);
    return {nat_load(z3, at), nat_load(sd, at), nat_load(s, at), nat_load(zd3, at), nat_load(s1, at), nat_load(t2, at)};
  }
  template <int NB>
  __device__ __forceinline__ void strip(const Strip& st, const In& in, const f32x16 (&x)[NB]) {
    uint32_t pk[1][8];
    pack_each(pk[0], [&](int r) {
      const float z = in.z3.get(r), dh = x[0][r];
      const float as = fmaf(dh, in.zd3.get(r), mul_rn(round_bf(x[1][r]), z));
      return fmaf(mul_rn(dh, z), in.t2.get(r), mul_rn(as, in.s1.get(r)));
    });
    st.template rows_out<1>(az1, ld, st.col, pk);
    pack_each(pk[0], [&](int r) { return fmaf(x[0][r], in.sd.get(r), mul_rn(round_bf(x[1][r]), in.s.get(r))); });
    st.template rows_out<1>(az3, ld, st.col, pk);
    pack_each(pk[0], [&](int r) { return mul_rn(x[0][r], in.z3.get(r)) * in.s1.get(r); });
    st.template rows_out<1>(azd1, ld, st.col, pk);
    pack_each(pk[0], [&](int r) { return x[0][r] * in.s.get(r); });
    st.template rows_out<1>(azd3, ld, st.col, pk);
  }
};

// dO rows of the chunk as a BF16 operand ([rows][d]; one wave per row).
template <typename IOT>
__global__ __launch_bounds__(256) void k_rows(const IOT* src, int64_t stride_tok, bf16* dst, int rows, int d) {
  typedef IOT iov4 __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (row >= rows) return;
  for (int c = 4 * l; c < d; c += 256) {
    const iov4 v = *reinterpret_cast<const iov4*>(src + (int64_t)row * stride_tok + c);
    *reinterpret_cast<u32x2*>(dst + (int64_t)row * d + c) =
        (u32x2){pack_bf16x2((float)v[0], (float)v[1]), pack_bf16x2((float)v[2], (float)v[3])};
  }
}

// Adjoint of the row normalisation x / max(||x||, eps) for the chunk's rows:
// (g - xhat <xhat, g>) / ||x|| where ||x|| > eps, g / eps where the floor is
// active, g itself for a tensor that is not normalised.  For the paper's unit
// g of V is eta_i Ydot_i and deta_i = <vhat_i, Ydot_i>.  One wave per token, 4
// consecutive elements per lane, at most 16 passes of 256.
struct RowsBwdArgs {
  const void* X[3];   // K, V, Q (null: skipped)
  const float* g[3];  // their adjoints, [rows][d] (V of the paper's unit: Ydot)
  void* dX[3];
  int64_t stride_tok;
  uint32_t nrm[3];
  int32_t rows, d;
  const float* eta;   // paper's unit (nullable)
  float* deta;
  int64_t eta_stride;
};
template <typename IOT>
__global__ __launch_bounds__(256) void k_rows_bwd(RowsBwdArgs p) {
  typedef IOT iov4 __attribute__((ext_vector_type(4)));
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
  if (row >= p.rows) return;
  const int passes = p.d / 256;
#pragma unroll
  for (int which = 0; which < 3; ++which) {
    if (!p.X[which]) continue;
    const IOT* src = static_cast<const IOT*>(p.X[which]) + (int64_t)row * p.stride_tok;
    IOT* dst = static_cast<IOT*>(p.dX[which]) + (int64_t)row * p.stride_tok;
    const float* g = p.g[which] + (int64_t)row * p.d;
    const bool nrm = p.nrm[which];
    f32x4 x[16], gv[16];
    float ss = 0.f, xg = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < passes) {
        const iov4 v = *reinterpret_cast<const iov4*>(src + 256 * i + 4 * l);
        x[i] = (f32x4){(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
        gv[i] = *reinterpret_cast<const f32x4*>(g + 256 * i + 4 * l);
#pragma unroll
        for (int e = 0; e < 4; ++e) ss = fmaf(x[i][e], x[i][e], ss);
      }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) ss += __shfl_xor(ss, m, 64);
    const float n = sqrtf(ss);
    const bool above = n > NORM_EPS;
    const float inv = nrm ? 1.0f / fmaxf(n, NORM_EPS) : 1.0f;
    const bool unit_v = which == 1 && p.eta;
    if (nrm || unit_v) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (i < passes)
#pragma unroll
          for (int e = 0; e < 4; ++e) xg = fmaf(x[i][e] * inv, gv[i][e], xg);
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) xg += __shfl_xor(xg, m, 64);
    }
    float f = 1.0f;
    if (unit_v) {
      f = p.eta[(int64_t)row * p.eta_stride];
      if (l == 0) p.deta[(int64_t)row * p.eta_stride] = xg;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i < passes) {
        f32x4 y = gv[i];
        if (nrm) {
          if (above) {
#pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = (gv[i][e] - x[i][e] * inv * xg) * inv;
          } else {
            y = gv[i] * (1.0f / NORM_EPS);
          }
        }
        y = y * f;
        *reinterpret_cast<iov4*>(dst + 256 * i + 4 * l) = (iov4){(IOT)y[0], (IOT)y[1], (IOT)y[2], (IOT)y[3]};
      }
    }
  }
}

// *deta += (the step-size partials of two launches, in a fixed order)
__global__ __launch_bounds__(256) void k_deta(const float* part, int n, float* deta) {
  const float s = fixed_sum(part, n);
  if (threadIdx.x == 0) *deta += s;
}

// The chunk's dO rows as a BF16 operand: the caller's where they are BF16 and
// within the 32-bit byte range of a buffer resource, else a packed copy.
template <typename IOT>
static const bf16* rows_operand(const void* src, int64_t stride_tok, void* copy, int rows, int d, int* ld,
                                hipStream_t st) {
  if constexpr (std::is_same_v<IOT, bf16>) {
    if ((int64_t)rows * stride_tok * 2 < (int64_t(1) << 31)) {
      *ld = (int)stride_tok;
      return static_cast<const bf16*>(src);
    }
  }
  *ld = d;
  hipLaunchKernelGGL(k_rows<IOT>, dim3((rows + 3) / 4), dim3(256), 0, st, static_cast<const IOT*>(src), stride_tok,
                     static_cast<bf16*>(copy), rows, d);
  return static_cast<const bf16*>(copy);
}
template <typename IOT, typename A>
static RowsBwdArgs rows_bwd(const A& a) {
  RowsBwdArgs r{};
  if (a.update) {
    r.X[0] = a.K; r.X[1] = a.V;
    r.g[0] = a.dk;
    r.dX[0] = a.dK; r.dX[1] = a.dV;
  }
  if (a.apply) {
    r.X[2] = a.Q; r.g[2] = a.dq; r.dX[2] = a.dQ;
  }
  r.nrm[0] = a.flags & 2u; r.nrm[1] = a.flags & 4u; r.nrm[2] = a.flags & 1u;
  r.stride_tok = a.stride_tok;
  r.rows = a.rows; r.d = a.d;
  return r;
}

template <typename IOT>
static hipError_t bwd_step_bf(const LargeBwdArgs& a, hipStream_t st) {
  const int M = a.rows, d = a.d, h = a.h;
  const float eta = a.eta, scale = 2.0f / (float)M;
  auto P = [](void* q) { return static_cast<bf16*>(q); };
  auto C = [](const void* q) { return static_cast<const bf16*>(q); };
  bf16 *Kn = P(a.Kn), *Qn = P(a.Qn), *E = P(a.E), *dY = P(a.dY), *A = P(a.A), *S1 = P(a.S1), *S2 = P(a.S2),
       *Pn = P(a.P), *D = P(a.D), *Dn = P(a.Dn), *Aq = P(a.Aq), *Sq1 = P(a.Sq1), *dZq = P(a.dZq), *dP = P(a.dP),
       *dZa = P(a.dZa), *EWh = P(a.EWh), *dZ = P(a.dZ);
  const bf16 *W1 = C(a.W1op), *W2 = C(a.W2op), *W1n = C(a.W1nop), *W2n = C(a.W2nop);
  bf16 *Wh1 = P(a.Wh1op), *Wh2 = P(a.Wh2op);
  float* vinv = a.Vn;
  NormArgs na{};
  na.K = a.K; na.V = a.V; na.Q = a.Q;
  na.stride_tok = a.stride_tok; na.flags = a.flags; na.rows = M; na.d = d;
  na.Kn = a.update ? Kn : nullptr; na.vinv = a.update ? vinv : nullptr; na.Qn = a.apply ? Qn : nullptr;
  const hipError_t en = launch_norm(na, std::is_same_v<IOT, bf16>, st);
  if (en != hipSuccess) return en;
  if (a.apply) {
    int ldo = d;
    const bf16* dO = rows_operand<IOT>(a.dO, a.stride_tok, a.dOn, M, d, &ldo, st);
    EpAct<true> e4{{}, Aq, Sq1, h};
    gemm<MNMAJ, 1>(product(Qn, d, M, W1n, h, d, M, h, d), e4, st);
    EpD e6{{}, dZq, Sq1, h};
    gemm<KMAJ, 1>(product(dO, ldo, M, W2n, d, h, M, h, d), e6, st);
    WArgs w{};
    w.tokens = M;
    add_weight(w, Aq, h, dO, ldo, h, d, a.Wh2, Wh2, 1.0f, 1);
    add_weight(w, Qn, d, dZq, h, d, h, a.Wh1, Wh1, 1.0f, 1);
    wgrad(w, st);
    EpF32 e8{{}, a.dq, d, 1.0f};
    gemm<KMAJ, 1>(product(dZq, h, M, W1n, h, d, M, d, h), e8, st);
  }
  if (a.update) {
    EpAct3 e1{{}, A, S1, S2, h};
    gemm<MNMAJ, 1>(product(Kn, d, M, W1, h, d, M, h, d), e1, st);
    GemmArgs yu = product(A, h, M, W2, d, h, M, d, h);
    yu.B[1] = Wh2;
    EpYU<IOT> e2{{}, E, a.dE, static_cast<const IOT*>(a.V), vinv, a.stride_tok, a.deta_part, d, scale, eta};
    const int n1 = gemm<MNMAJ, 2>(yu, e2, st).wgs * NW;
    GemmArgs pe = product(E, d, M, W2, d, h, M, h, d);
    pe.B[1] = Wh2;
    EpPE e3{{}, D, Dn, Pn, EWh, S1, h};
    gemm<KMAJ, 2>(pe, e3, st);
    EpU1 e9{{}, dP, dZa, Dn, S1, Pn, S2, a.deta_part + n1, h, eta};
    const int n2 = gemm<MNMAJ, 1>(product(Kn, d, M, Wh1, h, d, M, h, d), e9, st).wgs * NW;
    hipLaunchKernelGGL(k_deta, dim3(1), dim3(256), 0, st, a.deta_part, n1 + n2, a.deta);
    EpDY e11{{}, dY, a.dv, a.dE, d, scale};
    gemm<MNMAJ, 1>(product(dP, h, M, W2, d, h, M, d, h), e11, st);
    EpDZ e13{{}, dZ, EWh, dZa, S1, h, eta};
    gemm<KMAJ, 1>(product(dY, d, M, W2, d, h, M, h, d), e13, st);
    GemmArgs dk = product(D, h, M, Wh1, h, d, M, d, h);
    dk.A[1] = dZ; dk.B[1] = W1;
    dk.nseg = 2; dk.seg0_scale = -eta;
    EpF32 e14{{}, a.dk, d, 1.0f};
    gemm<KMAJ, 1>(dk, e14, st);
    // the weight terms of the update adjoint (the adjoint of W_c in the chain)
    WArgs w{};
    w.tokens = M;
    add_weight(w, dP, h, E, d, h, d, a.Acc2, P(a.Acc2op), 1.0f, 1);
    w.p[0].A[1] = A; w.p[0].B[1] = dY; w.p[0].nterm = 2;
    add_weight(w, Kn, d, dZ, h, d, h, a.Acc1, P(a.Acc1op), 1.0f, 1);
    wgrad(w, st);
  }
  RowsBwdArgs r = rows_bwd<IOT>(a);
  r.g[1] = a.dv;
  hipLaunchKernelGGL(k_rows_bwd<IOT>, dim3((M + 3) / 4), dim3(256), 0, st, r);
  return hipGetLastError();
}

template <typename IOT>
static hipError_t amu_bwd_step_bf(const LargeAmuBwdArgs& a, hipStream_t st) {
  const int M = a.rows, d = a.d, h = a.h;
  auto P = [](void* q) { return static_cast<bf16*>(q); };
  auto C = [](const void* q) { return static_cast<const bf16*>(q); };
  bf16 *Kn = P(a.Kn), *Qn = P(a.Qn), *E = P(a.E), *Z3 = P(a.Z3), *Hd = P(a.Hd), *Hdot = P(a.Hdot), *S = P(a.S),
       *S1 = P(a.S1), *Zd3 = P(a.Zd3), *Sd = P(a.Sd), *T2 = P(a.T2), *aZ1 = P(a.aZ1), *aZ3 = P(a.aZ3),
       *aZd1 = P(a.aZd1), *aZd3 = P(a.aZd3);
  const bf16 *W1 = C(a.Wop[0]), *W2 = C(a.Wop[1]), *W3 = C(a.Wop[2]);
  const bf16 *W1n = C(a.Wnop[0]), *W2n = C(a.Wnop[1]), *W3n = C(a.Wnop[2]);
  bf16 *Wh1 = P(a.Whop[0]), *Wh2 = P(a.Whop[1]), *Wh3 = P(a.Whop[2]);
  NormArgs na{};
  na.K = a.K; na.V = a.V; na.Q = a.Q;
  na.stride_tok = a.stride_tok; na.flags = a.flags; na.rows = M; na.d = d;
  na.Kn = a.update ? Kn : nullptr; na.vinv = a.update ? a.Vn : nullptr; na.E = E; na.Qn = a.apply ? Qn : nullptr;
  na.eta = a.eta; na.eta_stride = a.eta_stride;
  const hipError_t en = launch_norm(na, std::is_same_v<IOT, bf16>, st);
  if (en != hipSuccess) return en;
  if (a.apply) {
    int ldo = d;
    const bf16* dO = rows_operand<IOT>(a.dO, a.stride_tok, a.dOn, M, d, &ldo, st);
    GemmArgs z = product(Qn, d, M, W1n, h, d, M, h, d);
    z.B[1] = W3n;
    EpSwi<true> q1{{}, Hd, S1, S, h};  // Hq, F1, F3
    gemm<MNMAJ, 2>(z, q1, st);
    EpD2 q2{{}, S1, S, aZ1, aZ3, h};  // dZq1, dZq3
    gemm<KMAJ, 1>(product(dO, ldo, M, W2n, d, h, M, h, d), q2, st);
    WArgs w{};
    w.tokens = M;
    add_weight(w, Qn, d, aZ1, h, d, h, a.Wh[0], Wh1, 1.0f, 1);
    add_weight(w, Qn, d, aZ3, h, d, h, a.Wh[2], Wh3, 1.0f, 1);
    add_weight(w, Hd, h, dO, ldo, h, d, a.Wh[1], Wh2, 1.0f, 1);
    wgrad(w, st);
    GemmArgs q = product(aZ1, h, M, W1n, h, d, M, d, h);
    q.A[1] = aZ3; q.B[1] = W3n;
    q.nseg = 2;
    EpF32 g1{{}, a.dq, d, 1.0f};
    gemm<KMAJ, 1>(q, g1, st);
  }
  if (a.update) {
    GemmArgs z = product(Kn, d, M, W1, h, d, M, h, d);
    z.B[1] = W3; z.B[2] = Wh1; z.B[3] = Wh3;
    EpTan e1{{}, Hd, Hdot, S, S1, Z3, Zd3, Sd, T2, h};
    gemm<MNMAJ, 4>(z, e1, st);
    GemmArgs y = product(Hdot, h, M, W2, d, h, M, d, h);
    y.A[1] = Hd; y.B[1] = Wh2;
    y.nseg = 2;
    EpF32 ey{{}, a.Ydot, d, 1.0f};
    gemm<MNMAJ, 1>(y, ey, st);
    GemmArgs dh = product(E, d, M, W2, d, h, M, h, d);
    dh.B[1] = Wh2;
    EpAdj e9{{}, Z3, Sd, S, Zd3, S1, T2, aZ1, aZ3, aZd1, aZd3, h};
    gemm<KMAJ, 2>(dh, e9, st);
    GemmArgs k = product(aZ1, h, M, W1, h, d, M, d, h);
    k.A[1] = aZ3; k.B[1] = W3;
    k.A[2] = aZd1; k.B[2] = Wh1;
    k.A[3] = aZd3; k.B[3] = Wh3;
    k.nseg = 4;
    EpF32 ek{{}, a.dk, d, -1.0f};
    gemm<KMAJ, 1>(k, ek, st);
    // the weight terms (after the last use of Wh, which they change in the chain)
    WArgs w{};
    w.tokens = M;
    add_weight(w, Kn, d, aZ1, h, d, h, a.Acc[0], P(a.Accop[0]), -1.0f, 1);
    add_weight(w, Kn, d, aZ3, h, d, h, a.Acc[2], P(a.Accop[2]), -1.0f, 1);
    add_weight(w, Hdot, h, E, d, h, d, a.Acc[1], P(a.Accop[1]), -1.0f, 1);
    wgrad(w, st);
  }
  RowsBwdArgs r = rows_bwd<IOT>(a);
  r.g[1] = a.Ydot;
  r.eta = a.eta; r.deta = a.deta; r.eta_stride = a.eta_stride;
  hipLaunchKernelGGL(k_rows_bwd<IOT>, dim3((M + 3) / 4), dim3(256), 0, st, r);
  return hipGetLastError();
}

}  // namespace bfg

hipError_t launch_large_bwd_step_bf(const LargeBwdArgs& a, bool io_bf16, hipStream_t st) {
  return io_bf16 ? bfg::bwd_step_bf<bf16>(a, st) : bfg::bwd_step_bf<float>(a, st);
}
hipError_t launch_large_amu_bwd_step_bf(const LargeAmuBwdArgs& a, bool io_bf16, hipStream_t st) {
  return io_bf16 ? bfg::amu_bwd_step_bf<bf16>(a, st) : bfg::amu_bwd_step_bf<float>(a, st);
}

}  // namespace ttt
