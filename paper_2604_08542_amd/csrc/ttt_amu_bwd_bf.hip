// Reverse mode of the paper's memory unit with BF16 products on gfx950 (d =
// 64; the FP32 form and the formulas are in ttt_amu_bwd.hip).
//
// The update adjoint multiplies a token tile by twelve weight matrices (six
// into the hidden axis, six out of it), 384 KiB at h = 256; read from the L2
// per tile, as one kernel did, they cost 32 us per tile and work-group, of
// which the products are less than 1.  They do not fit one CU's registers
// beside the accumulators, so the work is split in two kernels that each keep
// their matrices on chip for all their tiles and repeat the cheap part (the
// six 32x32 products and the elementwise work; a row's norm is summed in one
// order by both, so that they see the same operands):
//   sums    the token sums (adjoints of W1, W2, W3): no contraction over the
//           hidden axis, one barrier per tile; 8 waves of 32 hidden units (h =
//           256), two matrices in registers, four in LDS
//   tokens  dK, dV, d(eta): 4 waves of 64 hidden units at up to 512 registers;
//           the six inner matrices and three outer ones in registers, three
//           in LDS.  The hidden products are taken transposed (hidden units
//           in registers), so the factors of the outer products are operands
//           straight from the registers; a wave's partial results over its
//           hidden units meet in LDS and are added in wave order.
// The apply adjoint needs five matrices and runs as one kernel: three in
// registers, two in LDS.
// Measured on MI355X, 5,496 tokens x 16 heads, h = 256: update adjoint 354 ->
// 138 us, apply adjoint 106 -> 51 us.
#include <hip/hip_runtime.h>

#include "ttt_amu_bf.h"
#include "ttt_common.h"
#include "ttt_internal.h"

namespace ttt {
namespace {

// Weight fragments of one wave in LDS: fragment f at 1 KiB strides, one 16-byte
// read per lane.
__device__ __forceinline__ bf16x8 lds_frag(const bf16* base, int f) {
  return *reinterpret_cast<const bf16x8*>(base + f * 512 + (threadIdx.x & 63) * 8);
}
__device__ __forceinline__ void lds_put(bf16* base, int f, const bf16x8& v) {
  *reinterpret_cast<bf16x8*>(base + f * 512 + (threadIdx.x & 63) * 8) = v;
}

// One token and hidden unit of the update adjoint.
struct UpdEl {
  float hdot, hd, az1, az3, azd1, azd3;
};
__device__ __forceinline__ UpdEl upd_el(float z, float z3, float zd1, float zd3, float dh, float dhh) {
  UpdEl o;
  const float sg = sigmoid(z);
  const float s = z * sg;
  const float s1 = fmaf(s, 1.0f - sg, sg);                              // s'(z)
  const float s2 = sg * (1.0f - sg) * fmaf(z, 1.0f - 2.0f * sg, 2.0f);  // s''(z)
  const float sd = s1 * zd1;
  o.hdot = fmaf(sd, z3, s * zd3);
  o.hd = s * z3;
  const float asd = dh * z3;
  o.az3 = fmaf(dh, sd, dhh * s);
  const float as = fmaf(dh, zd3, dhh * z3);
  o.azd3 = dh * s;
  o.azd1 = asd * s1;
  o.az1 = fmaf(asd * s2, zd1, as * s1);
  return o;
}

// Shard partials of the three weight adjoints of one 32-unit hidden block.
template <int HH>
__device__ __forceinline__ void put_partials(float* part, const f32x16 (&g1)[2], const f32x16 (&g2)[2],
                                             const f32x16 (&g3)[2], int hb, int l32, int hf, float sign) {
  constexpr int DH = D * HH;
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = c32_row(r, hf);
      part[(32 * db + rr) * HH + 32 * hb + l32] = sign * g1[db][r];
      part[DH + (32 * hb + rr) * D + 32 * db + l32] = sign * g2[db][r];
      part[2 * DH + (32 * db + rr) * HH + 32 * hb + l32] = sign * g3[db][r];
    }
}

// Adjoint of the normalisation for this thread's row part (see the FP32
// form): g becomes (g - xh (xh . g)) inv where the norm exceeds eps, else g inv.
template <int EPT>
__device__ __forceinline__ void norm_adjoint(float (&g)[EPT], const float (&xh)[EPT], bool did_norm, float inv,
                                             bool above) {
  if (!did_norm) return;
  float dot = 0.f;
#pragma unroll
  for (int i = 0; i < EPT; ++i) dot = fmaf(xh[i], g[i], dot);
  dot = lane_group_sum<D / EPT>(dot);
#pragma unroll
  for (int i = 0; i < EPT; ++i) g[i] = above ? (g[i] - xh[i] * dot) * inv : g[i] * inv;
}

// Update adjoint, token sums: X = K, Y = V.
template <typename IOT, int NW>
__global__ __launch_bounds__(NW * 64) void ttt_amu_bwd_sums_bf(AmuBwdArgs p) {
  constexpr int HH = NW * 32, NT = NW * 64, EPT = D * TT / NT, TPR = D / EPT, DH = D * HH;
  __shared__ __attribute__((aligned(16))) bf16 xs[2][TT * XLD];
  __shared__ __attribute__((aligned(16))) bf16 es[2][TT * XLD];
  __shared__ __attribute__((aligned(16))) bf16 wl[NW][16 * 512];  // each wave's fragments of four matrices

  const Lane L;
  const int tid = threadIdx.x, row = tid / TPR, col0 = (tid % TPR) * EPT;
  const int lin = xcd_linear_block();
  const int G = p.G, head = lin / G, g = lin % G;
  const int64_t hoff = (int64_t)head * p.stride_head;
  const bool norm_k = p.flags & 2u, norm_v = p.flags & 4u;
  const bf16* Wb = static_cast<const bf16*>(p.prep_w) + (int64_t)head * 6 * DH;
  const bf16* Ab = static_cast<const bf16*>(p.prep_a) + (int64_t)head * 6 * DH;
  if (p.len <= 0) return;
  bf16x8 w1[4], w3[4];
  L.weights(Wb + AMU_W1T * DH, w1);
  L.weights(Wb + AMU_W3T * DH, w3);
  bf16* wv = wl[L.w];  // read only by the wave that writes it
  {
    const bf16* src[4] = {Ab + AMU_W1T * DH, Ab + AMU_W3T * DH, Wb + AMU_W2N * DH, Ab + AMU_W2N * DH};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      bf16x8 f[4];
      L.weights(src[k], f);
#pragma unroll
      for (int m = 0; m < 4; ++m) lds_put(wv, 4 * k + m, f[m]);
    }
  }
  auto dot_l = [&](const bf16x8 (&a)[4], int k) {
    f32x16 c = {};
#pragma unroll
    for (int m = 0; m < 4; ++m) c = mma32(a[m], lds_frag(wv, 4 * k + m), c);
    return c;
  };

  f32x16 g1[2] = {}, g2[2] = {}, g3[2] = {};
  RowPart<IOT, EPT> rk, rv;
  float et = 0.f;
  auto fetch = [&](int t) {
    const int64_t tok = p.start + (int64_t)t * TT + row;
    const bool valid = row < p.len - t * TT;
    rk.load(static_cast<const IOT*>(p.X) + tok * p.stride_tok + hoff + col0, valid);
    rv.load(static_cast<const IOT*>(p.Y) + tok * p.stride_tok + hoff + col0, valid);
    et = valid ? p.eta_tok[tok * p.H + head] : 0.f;
  };
  auto stage = [&](int b) {
    float x[EPT];
    const float sk = rk.get(norm_k, x);
    put_part<EPT>(&xs[b][row * XLD + col0], x, sk);
    const float sv = rv.get(norm_v, x);
#pragma unroll
    for (int i = 0; i < EPT; ++i) x[i] = mul_rn(x[i], sv);
    put_part<EPT>(&es[b][row * XLD + col0], x, -et);
  };
  if (g * TT < p.len) fetch(g);
  for (int t = g, b = 0; t * TT < p.len; t += G, b ^= 1) {
    stage(b);
    if ((t + G) * TT < p.len) fetch(t + G);
    __syncthreads();
    bf16x8 a[4];
    L.rows(xs[b], a);
    const f32x16 Z1 = dot4(a, w1), Z3 = dot4(a, w3), Zd1 = dot_l(a, 0), Zd3 = dot_l(a, 1);
    L.rows(es[b], a);
    const f32x16 dH = dot_l(a, 2), dHh = dot_l(a, 3);
    uint32_t ph[8], p1[8], p3[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const UpdEl u = upd_el(Z1[2 * q], Z3[2 * q], Zd1[2 * q], Zd3[2 * q], dH[2 * q], dHh[2 * q]);
      const UpdEl v = upd_el(Z1[2 * q + 1], Z3[2 * q + 1], Zd1[2 * q + 1], Zd3[2 * q + 1], dH[2 * q + 1],
                             dHh[2 * q + 1]);
      ph[q] = pack_bf16x2(u.hdot, v.hdot);
      p1[q] = pack_bf16x2(u.az1, v.az1);
      p3[q] = pack_bf16x2(u.az3, v.az3);
    }
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        g2[db] = mma32(opnd(ph, m), L.cols(es[b], m, db), g2[db]);
        const bf16x8 k = L.cols(xs[b], m, db);
        g1[db] = mma32(k, opnd(p1, m), g1[db]);
        g3[db] = mma32(k, opnd(p3, m), g3[db]);
      }
  }
  put_partials<HH>(p.partial + ((int64_t)head * G + g) * (3 * DH), g1, g2, g3, L.w, L.l32, L.hf, -1.0f);
}

// Update adjoint, token side: dX = dK, dY = dV, d(eta).  NB hidden blocks per
// wave (h = 128 NB).
template <typename IOT, int NB>
__global__ __launch_bounds__(256) void ttt_amu_bwd_tokens_bf(AmuBwdArgs p) {
  constexpr int HH = 128 * NB, EPT = 8, TPR = D / EPT, DH = D * HH;
  constexpr int FLD = D + 4;
  __shared__ __attribute__((aligned(16))) bf16 xs[2][TT * XLD];
  __shared__ __attribute__((aligned(16))) bf16 es[2][TT * XLD];
  __shared__ __attribute__((aligned(16))) bf16 wl[4][NB * 12 * 512];   // each wave's fragments of three outer matrices
  __shared__ __attribute__((aligned(16))) float part[4][TT * FLD];     // the waves' partial Ydot, then dK

  const Lane L;
  const int tid = threadIdx.x, row = tid / TPR, col0 = (tid % TPR) * EPT;
  const int lin = xcd_linear_block();
  const int G = p.G, head = lin / G, g = lin % G;
  const int64_t hoff = (int64_t)head * p.stride_head;
  const bool norm_k = p.flags & 2u, norm_v = p.flags & 4u;
  const bf16* Wb = static_cast<const bf16*>(p.prep_w) + (int64_t)head * 6 * DH;
  const bf16* Ab = static_cast<const bf16*>(p.prep_a) + (int64_t)head * 6 * DH;
  if (g * TT >= p.len) return;
  // inner fragments: row 32 hb + l32 of a [hid][d] matrix
  auto inner = [&](const bf16* M, int j, bf16x8 (&f)[4]) {
    const bf16* r = M + (32 * (NB * L.w + j) + L.l32) * D + 8 * L.hf;
#pragma unroll
    for (int m = 0; m < 4; ++m) f[m] = *reinterpret_cast<const bf16x8*>(r + 16 * m);
  };
  // outer fragment (m, db): feature 32 db + l32 of a [d][hid] matrix, hidden
  // units in the register order of a 32x32 result
  auto outer = [&](const bf16* M, int j, int m, int db) {
    const bf16* r = M + (32 * db + L.l32) * HH + 32 * (NB * L.w + j) + 16 * m + 4 * L.hf;
    const u32x2 lo = *reinterpret_cast<const u32x2*>(r), hi = *reinterpret_cast<const u32x2*>(r + 8);
    return as_bf16x8(lo[0], lo[1], hi[0], hi[1]);
  };
  bf16x8 wi[6][NB][4], wo[3][NB][4];
  bf16* wv = wl[L.w];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    inner(Wb + AMU_W1T * DH, j, wi[0][j]);
    inner(Wb + AMU_W3T * DH, j, wi[1][j]);
    inner(Ab + AMU_W1T * DH, j, wi[2][j]);
    inner(Ab + AMU_W3T * DH, j, wi[3][j]);
    inner(Wb + AMU_W2N * DH, j, wi[4][j]);
    inner(Ab + AMU_W2N * DH, j, wi[5][j]);
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        const int f = 2 * db + m;
        wo[0][j][f] = outer(Wb + AMU_W1D * DH, j, m, db);
        wo[1][j][f] = outer(Wb + AMU_W3D * DH, j, m, db);
        wo[2][j][f] = outer(Ab + AMU_W1D * DH, j, m, db);
        lds_put(wv, 12 * j + f, outer(Ab + AMU_W3D * DH, j, m, db));
        lds_put(wv, 12 * j + 4 + f, outer(Wb + AMU_W2D * DH, j, m, db));
        lds_put(wv, 12 * j + 8 + f, outer(Ab + AMU_W2D * DH, j, m, db));
      }
  }

  RowPart<IOT, EPT> rk, rv;
  float etn = 0.f;
  auto fetch = [&](int t) {
    const int64_t tok = p.start + (int64_t)t * TT + row;
    const bool valid = row < p.len - t * TT;
    rk.load(static_cast<const IOT*>(p.X) + tok * p.stride_tok + hoff + col0, valid);
    rv.load(static_cast<const IOT*>(p.Y) + tok * p.stride_tok + hoff + col0, valid);
    etn = valid ? p.eta_tok[tok * p.H + head] : 0.f;
  };
  // a wave's partial results: feature 8q + 4hf + 0..3 (+ 32 db) of token l32
  auto put_part32 = [&](const f32x16 (&c)[2]) {
    float* o = part[L.w] + L.l32 * FLD + 4 * L.hf;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        *reinterpret_cast<f32x4*>(o + 32 * db + 8 * q) =
            (f32x4){c[db][4 * q], c[db][4 * q + 1], c[db][4 * q + 2], c[db][4 * q + 3]};
  };
  auto sum_parts = [&](float (&x)[EPT]) {
#pragma unroll
    for (int i = 0; i < EPT; i += 4) {
      f32x4 s = *reinterpret_cast<const f32x4*>(part[0] + row * FLD + col0 + i);
#pragma unroll
      for (int w = 1; w < 4; ++w) s += *reinterpret_cast<const f32x4*>(part[w] + row * FLD + col0 + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) x[i + e] = s[e];
    }
  };
  fetch(g);
  for (int t = g, b = 0; t * TT < p.len; t += G, b ^= 1) {
    const int nv = p.len - t * TT;
    const int64_t at = (p.start + (int64_t)t * TT + row) * p.stride_tok + hoff + col0;
    // rows: BF16 tiles for the products, FP32 parts of this thread's row kept
    float xh[EPT], vh[EPT], kn = 1.f, vn = 1.f;
    const float et = etn, kinv = rk.template get<8 / NB>(norm_k, xh, &kn), vinv = rv.template get<8 / NB>(norm_v, vh, &vn);
    {
      float e[EPT];
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        xh[i] = mul_rn(xh[i], kinv);
        vh[i] = mul_rn(vh[i], vinv);
        e[i] = vh[i];
      }
      put_part<EPT>(&xs[b][row * XLD + col0], xh, 1.0f);
      put_part<EPT>(&es[b][row * XLD + col0], e, -et);
    }
    if ((t + G) * TT < p.len) fetch(t + G);
    __syncthreads();
    f32x16 yd[2] = {}, dk[2] = {};
    {
      bf16x8 a[4], e[4];
      L.rows(xs[b], a);
      L.rows(es[b], e);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const f32x16 Z1 = dot4(wi[0][j], a), Z3 = dot4(wi[1][j], a), Zd1 = dot4(wi[2][j], a), Zd3 = dot4(wi[3][j], a),
                     dH = dot4(wi[4][j], e), dHh = dot4(wi[5][j], e);
        uint32_t ph[8], pd[8], p1[8], p3[8], q1[8], q3[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const UpdEl u = upd_el(Z1[2 * q], Z3[2 * q], Zd1[2 * q], Zd3[2 * q], dH[2 * q], dHh[2 * q]);
          const UpdEl v = upd_el(Z1[2 * q + 1], Z3[2 * q + 1], Zd1[2 * q + 1], Zd3[2 * q + 1], dH[2 * q + 1],
                                 dHh[2 * q + 1]);
          ph[q] = pack_bf16x2(u.hdot, v.hdot);
          pd[q] = pack_bf16x2(u.hd, v.hd);
          p1[q] = pack_bf16x2(u.az1, v.az1);
          p3[q] = pack_bf16x2(u.az3, v.az3);
          q1[q] = pack_bf16x2(u.azd1, v.azd1);
          q3[q] = pack_bf16x2(u.azd3, v.azd3);
        }
#pragma unroll
        for (int db = 0; db < 2; ++db)
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            const int f = 2 * db + m;
            yd[db] = mma32(lds_frag(wv, 12 * j + 4 + f), opnd(ph, m), yd[db]);
            yd[db] = mma32(lds_frag(wv, 12 * j + 8 + f), opnd(pd, m), yd[db]);
            dk[db] = mma32(wo[0][j][f], opnd(p1, m), dk[db]);
            dk[db] = mma32(wo[1][j][f], opnd(p3, m), dk[db]);
            dk[db] = mma32(wo[2][j][f], opnd(q1, m), dk[db]);
            dk[db] = mma32(lds_frag(wv, 12 * j + f), opnd(q3, m), dk[db]);
          }
      }
    }
    put_part32(yd);
    __syncthreads();
    {
      float y[EPT], de = 0.f;
      sum_parts(y);
#pragma unroll
      for (int i = 0; i < EPT; ++i) {
        de = fmaf(vh[i], y[i], de);
        y[i] *= et;
      }
      de = lane_group_sum<TPR>(de);
      norm_adjoint<EPT>(y, vh, norm_v, vinv, vn > NORM_EPS);
      if (row < nv) {
        store_vec<IOT, EPT>(static_cast<IOT*>(p.dY) + at, y);
        if (tid % TPR == 0) p.deta_tok[(p.start + (int64_t)t * TT + row) * p.H + head] = de;
      }
    }
    __syncthreads();
    put_part32(dk);
    __syncthreads();
    {
      float k[EPT];
      sum_parts(k);
#pragma unroll
      for (int i = 0; i < EPT; ++i) k[i] = -k[i];
      norm_adjoint<EPT>(k, xh, norm_k, kinv, kn > NORM_EPS);
      if (row < nv) store_vec<IOT, EPT>(static_cast<IOT*>(p.dX) + at, k);
    }
  }
}

// Apply adjoint: X = Q, Y = dO, dX = dQ.  Two waves per SIMD: at h = 128 two
// work-groups per CU (16 heads x 6,000 tokens 44 -> 37 us).
template <typename IOT, int NW>
__global__ __launch_bounds__(NW * 64, 2) void ttt_amu_bwd_apply_bf(AmuBwdArgs p) {
  constexpr int HH = NW * 32, NT = NW * 64, EPT = D * TT / NT, TPR = D / EPT, DH = D * HH;
  constexpr int AS_LD = HH + 8, FLD = D + 4, NU = HH / 32, NBK = 8 / NW;
  __shared__ __attribute__((aligned(16))) bf16 xs[2][TT * XLD];
  __shared__ __attribute__((aligned(16))) bf16 ys[2][TT * XLD];
  __shared__ __attribute__((aligned(16))) bf16 s1[TT * AS_LD];
  __shared__ __attribute__((aligned(16))) bf16 s3[TT * AS_LD];
  __shared__ __attribute__((aligned(16))) float dq[TT * FLD];
  __shared__ __attribute__((aligned(16))) bf16 wl[2][4][NU * 512];  // W1, W3 as [d][hid]: fragments per 16 features

  const Lane L;
  const int tid = threadIdx.x, row = tid / TPR, col0 = (tid % TPR) * EPT;
  const int lin = xcd_linear_block();
  const int G = p.G, head = lin / G, g = lin % G;
  const int64_t hoff = (int64_t)head * p.stride_head;
  const bool norm_q = p.flags & 1u;
  const bf16* Wb = static_cast<const bf16*>(p.prep_w) + (int64_t)head * 6 * DH;
  if (p.len <= 0) return;
  bf16x8 w1[4], w3[4], w2[4];
  L.weights(Wb + AMU_W1T * DH, w1);
  L.weights(Wb + AMU_W3T * DH, w3);
  L.weights(Wb + AMU_W2N * DH, w2);
  for (int f = L.w; f < 2 * 4 * NU; f += NW) {
    const int mat = f / (4 * NU), db = (f / NU) & 3, u = f % NU;
    const bf16* M = Wb + (mat ? AMU_W3D : AMU_W1D) * DH;
    lds_put(wl[mat][db], u, *reinterpret_cast<const bf16x8*>(M + (16 * db + L.l16) * HH + (HH / 4) * L.g4 + 8 * u));
  }

  f32x16 g1[2] = {}, g2[2] = {}, g3[2] = {};
  RowPart<IOT, EPT> rq, ro;
  float xn[EPT], invn = 1.f, nrmn = 1.f;  // the staged tile's row part
  auto fetch = [&](int t) {
    const int64_t tok = p.start + (int64_t)t * TT + row;
    const bool valid = row < p.len - t * TT;
    rq.load(static_cast<const IOT*>(p.X) + tok * p.stride_tok + hoff + col0, valid);
    ro.load(static_cast<const IOT*>(p.Y) + tok * p.stride_tok + hoff + col0, valid);
  };
  auto stage = [&](int b) {
    nrmn = 1.f;
    invn = rq.get(norm_q, xn, &nrmn);
#pragma unroll
    for (int i = 0; i < EPT; ++i) xn[i] = mul_rn(xn[i], invn);
    put_part<EPT>(&xs[b][row * XLD + col0], xn, 1.0f);
    float y[EPT];
    ro.get(false, y);
    put_part<EPT>(&ys[b][row * XLD + col0], y, 1.0f);
  };
  if (g * TT < p.len) {
    fetch(g);
    stage(0);
    if ((g + G) * TT < p.len) fetch(g + G);
  }
  __syncthreads();
  for (int t = g, b = 0; t * TT < p.len; t += G, b ^= 1) {
    const int nv = p.len - t * TT;
    float xh[EPT];
    const float inv = invn, nrm = nrmn;
#pragma unroll
    for (int i = 0; i < EPT; ++i) xh[i] = xn[i];
    {
      bf16x8 a[4];
      L.rows(xs[b], a);
      const f32x16 Z1 = dot4(a, w1), Z3 = dot4(a, w3);
      L.rows(ys[b], a);
      const f32x16 dH = dot4(a, w2);
      f32x16 Hq, d1, d3;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float z = Z1[r];
        const float sg = sigmoid(z);
        const float s = z * sg;
        Hq[r] = s * Z3[r];
        d3[r] = dH[r] * s;
        d1[r] = dH[r] * Z3[r] * fmaf(s, 1.0f - sg, sg);
      }
      const Packed ph = pack32(Hq), p1 = pack32(d1), p3 = pack32(d3);
      auto put = [&](bf16* S, const Packed& q) {
        uint16_t* c = reinterpret_cast<uint16_t*>(S) + L.hid;
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const u32x4 u = __builtin_bit_cast(u32x4, q.f[m]);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            c[c32_row(8 * m + e, L.hf) * AS_LD] = (uint16_t)(e & 1 ? u[e >> 1] >> 16 : u[e >> 1]);
        }
      };
      put(s1, p1);
      put(s3, p3);
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          g2[db] = mma32(ph.f[m], L.cols(ys[b], m, db), g2[db]);
          const bf16x8 q = L.cols(xs[b], m, db);
          g1[db] = mma32(q, p1.f[m], g1[db]);
          g3[db] = mma32(q, p3.f[m], g3[db]);
        }
    }
    __syncthreads();
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi) {
      const int bk = L.w + NW * bi, tb = bk & 1, db = bk >> 1;
      f32x4 c = {};
      auto td = [&](const bf16* S, int mat) {
#pragma unroll
        for (int u = 0; u < NU; ++u)
          c = mma16(*reinterpret_cast<const bf16x8*>(&S[(16 * tb + L.l16) * AS_LD + (HH / 4) * L.g4 + 8 * u]),
                    lds_frag(wl[mat][db], u), c);
      };
      td(s1, 0);
      td(s3, 1);
#pragma unroll
      for (int r = 0; r < 4; ++r) dq[(16 * tb + 4 * L.g4 + r) * FLD + 16 * db + L.l16] = c[r];
    }
    // the other copy was last read before the barrier above
    if ((t + G) * TT < p.len) {
      stage(b ^ 1);
      if ((t + 2 * G) * TT < p.len) fetch(t + 2 * G);
    }
    __syncthreads();
    {
      float gq[EPT];
#pragma unroll
      for (int e = 0; e < EPT; ++e) gq[e] = dq[row * FLD + col0 + e];
      norm_adjoint<EPT>(gq, xh, norm_q, inv, nrm > NORM_EPS);
      if (row < nv)
        store_vec<IOT, EPT>(static_cast<IOT*>(p.dX) + (p.start + (int64_t)t * TT + row) * p.stride_tok + hoff + col0,
                            gq);
    }
  }
  put_partials<HH>(p.partial + ((int64_t)head * G + g) * (3 * DH), g1, g2, g3, L.w, L.l32, L.hf, 1.0f);
}

}  // namespace

template <typename IOT>
static hipError_t launch_update_t(const AmuBwdArgs& a, int n_blocks, int h, hipStream_t st) {
  if (h == 128) {
    hipLaunchKernelGGL((ttt_amu_bwd_sums_bf<IOT, 4>), dim3(n_blocks), dim3(256), 0, st, a);
    hipLaunchKernelGGL((ttt_amu_bwd_tokens_bf<IOT, 1>), dim3(n_blocks), dim3(256), 0, st, a);
  } else {
    hipLaunchKernelGGL((ttt_amu_bwd_sums_bf<IOT, 8>), dim3(n_blocks), dim3(512), 0, st, a);
    hipLaunchKernelGGL((ttt_amu_bwd_tokens_bf<IOT, 2>), dim3(n_blocks), dim3(256), 0, st, a);
  }
  return hipGetLastError();
}
hipError_t launch_amu_bwd_update_bf(const AmuBwdArgs& a, int n_blocks, int h, bool io_bf16, hipStream_t st) {
  return io_bf16 ? launch_update_t<bf16>(a, n_blocks, h, st) : launch_update_t<float>(a, n_blocks, h, st);
}
template <typename IOT>
static hipError_t launch_apply_t(const AmuBwdArgs& a, int n_blocks, int h, hipStream_t st) {
  if (h == 128)
    hipLaunchKernelGGL((ttt_amu_bwd_apply_bf<IOT, 4>), dim3(n_blocks), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL((ttt_amu_bwd_apply_bf<IOT, 8>), dim3(n_blocks), dim3(512), 0, st, a);
  return hipGetLastError();
}
hipError_t launch_amu_bwd_apply_bf(const AmuBwdArgs& a, int n_blocks, int h, bool io_bf16, hipStream_t st) {
  return io_bf16 ? launch_apply_t<bf16>(a, n_blocks, h, st) : launch_apply_t<float>(a, n_blocks, h, st);
}

}  // namespace ttt
