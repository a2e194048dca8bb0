// Device machinery shared by the BF16 kernels at d = 64 (the memory unit and
// the reverse step of the MSE unit): lane layout, operand fragments of staged
// token rows, token-row parts.
#pragma once
#include <hip/hip_runtime.h>

#include "ttt_common.h"
#include "ttt_internal.h"

namespace ttt {
namespace {

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int XLD = 88;  // pitch of a [token][d] BF16 tile (16-byte rows; transposing reads of 4 rows on disjoint banks)

// Lane-dependent machinery of a kernel with NW waves of 32 hidden units.
struct Lane {
  int w, l, l32, hf, l16, g4, hid;
  __device__ __forceinline__ Lane() {
    w = threadIdx.x >> 6;
    l = threadIdx.x & 63;
    l32 = l & 31;
    hf = l >> 5;
    l16 = l & 15;
    g4 = l >> 4;
    hid = 32 * w + l32;
  }
  // Fragments (4 steps of 16 features) of row `hid` of M[hid][d].
  __device__ __forceinline__ void weights(const bf16* M, bf16x8 (&f)[4]) const {
#pragma unroll
    for (int m = 0; m < 4; ++m) f[m] = *reinterpret_cast<const bf16x8*>(M + hid * D + 16 * m + 8 * hf);
  }
  // The same for token row l32 of a staged tile.
  __device__ __forceinline__ void rows(const bf16* X, bf16x8 (&a)[4]) const {
#pragma unroll
    for (int m = 0; m < 4; ++m) a[m] = *reinterpret_cast<const bf16x8*>(&X[l32 * XLD + 16 * m + 8 * hf]);
  }
  // Token-contraction operand of a staged tile: lane (d = 32 db + l32) holds
  // tokens 16m + 4hf + 0..3 and 16m + 8 + 4hf + 0..3, the token slots of
  // result registers 8m .. 8m+7 of a 32x32 block.
  template <int LD>
  __device__ __forceinline__ bf16x8 cols_at(const bf16* X, int m, int db) const {
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    typedef __attribute__((address_space(3))) bf16 lds_bf16;
    const bf16* p = X + ((l16 >> 2) + 4 * hf + 16 * m) * LD + 4 * (l16 & 3) + 16 * ((l >> 4) & 1) + 32 * db;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)((lds_bf16*)(p)));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)((lds_bf16*)(p + 8 * LD)));
    return (bf16x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  }
  __device__ __forceinline__ bf16x8 cols(const bf16* X, int m, int db) const { return cols_at<XLD>(X, m, db); }
};
// 32x32 block: sum over the four steps of a[m] b[m].
__device__ __forceinline__ f32x16 dot4(const bf16x8 (&a)[4], const bf16x8 (&b)[4]) {
  f32x16 c = {};
#pragma unroll
  for (int m = 0; m < 4; ++m) c = mma32(a[m], b[m], c);
  return c;
}
// A 32x32 result as two operand fragments (contraction over its rows).
struct Packed {
  bf16x8 f[2];
};
__device__ __forceinline__ Packed pack32(const f32x16& y) {
  Packed p;
#pragma unroll
  for (int m = 0; m < 2; ++m)
    p.f[m] = as_bf16x8(pack_bf16x2(y[8 * m], y[8 * m + 1]), pack_bf16x2(y[8 * m + 2], y[8 * m + 3]),
                       pack_bf16x2(y[8 * m + 4], y[8 * m + 5]), pack_bf16x2(y[8 * m + 6], y[8 * m + 7]));
  return p;
}

// Fragment m of 16 packed result words.
__device__ __forceinline__ bf16x8 opnd(const uint32_t (&pk)[8], int m) {
  return as_bf16x8(pk[4 * m], pk[4 * m + 1], pk[4 * m + 2], pk[4 * m + 3]);
}

// EPT consecutive elements of a token row, as loaded.
template <typename IOT, int EPT>
struct RowPart {
  static constexpr int BYTES = EPT * (int)sizeof(IOT);
  typedef IOT vec __attribute__((ext_vector_type(EPT), aligned(BYTES < 16 ? BYTES : 16)));
  vec v;
  __device__ __forceinline__ void load(const IOT* p, bool valid) {
    v = vec{};
    if (valid) v = *reinterpret_cast<const vec*>(p);
  }
  // as floats; returns 1 / max(||row||, eps), or 1 when not normalised (the
  // row is spread over D / EPT consecutive lanes; the squares are summed in
  // runs of RUN elements and those in a tree, so a kernel whose lanes hold
  // more elements can follow the order of one whose lanes hold RUN)
  template <int RUN = EPT>
  __device__ __forceinline__ float get(bool do_norm, float (&x)[EPT], float* norm = nullptr) const {
    float sc = 1.f;
#pragma unroll
    for (int i = 0; i < EPT; ++i) x[i] = (float)v[i];
    if (do_norm) {
      static_assert(RUN == EPT || 2 * RUN == EPT, "one or two runs per lane");
      float ss = 0.f, s2 = 0.f;
#pragma unroll
      for (int i = 0; i < RUN; ++i) ss = fmaf(x[i], x[i], ss);
      if constexpr (RUN < EPT) {
#pragma unroll
        for (int i = RUN; i < EPT; ++i) s2 = fmaf(x[i], x[i], s2);
        ss += s2;
      }
      ss = lane_group_sum<D / EPT>(ss);
      const float n = sqrtf(ss);
      sc = 1.0f / fmaxf(n, NORM_EPS);
      if (norm) *norm = n;
    }
    return sc;
  }
};
template <int EPT>
__device__ __forceinline__ void put_part(bf16* p, const float (&x)[EPT], float scale) {
  uint32_t pk[EPT / 2];
#pragma unroll
  for (int i = 0; i < EPT; i += 2) pk[i / 2] = pack_bf16x2(x[i] * scale, x[i + 1] * scale);
  if constexpr (EPT == 4)
    *reinterpret_cast<u32x2*>(p) = (u32x2){pk[0], pk[1]};
  else
    *reinterpret_cast<u32x4*>(p) = (u32x4){pk[0], pk[1], pk[2], pk[3]};
}

}  // namespace
}  // namespace ttt
