// BF16 matrix-core backward step of the chunked TTT chain (h = 128 or 256).
//
// Same mathematics as ttt_bwd_step (reverse mode through the inner update of
// chunk s, second-order terms included, plus the apply adjoint of chunk s-1;
// Sec. 4.2 Eq. 8 and Sec. 3.2 Eq. 3-4), organised for BF16 operands.
//
// What bounds it: an update tile is a chain of contractions over the hidden
// axis (A W2, then dP W2, then D Wh1^T and dZ W1^T) with elementwise work
// between them, phase after phase behind barriers, and four weight matrices in
// two orders (256 KiB at h = 256) take part.  Read from the L2 per tile, their
// latency (and, loads and stores completing in order, that of the row prefetch
// and of the gradient stores before them) stood in every phase.  Here:
//  - the four matrices stay in LDS for all tiles of a work-group, once each:
//    straight reads serve the contractions over the hidden axis, transposing
//    reads those over d;
//  - 8 waves, two per SIMD, so one's elementwise work overlaps the other's
//    products.  A wave owns 32 hidden units; at h = 128 two groups of 4 waves
//    share the matrices, each with a shard of its own (one group, where the
//    shards do not fill the CUs);
//  - LDS is what is left beside them: the BF16 rows of K, E and dY (transposing
//    reads give their columns) and one staged [token][hidden] tile that A, dP,
//    D and dZ take in turn.  At h = 256 V and K enter the residual and the
//    normalisation adjoints in FP32 from the token tensors, in the layout of the
//    16x16 results, times the row's factor, and the row factors and row dots sit
//    in the padding of the row tiles;
//  - at h = 128 two FP32 row tiles fit as well (F32T): normalised V for the
//    residual, and the way of dV, dK and dQ to the threads that hold the raw
//    rows, which take the dots and store 16 bytes at a time (with one wave per
//    SIMD a step is as long as its instructions).  The rows are requested before
//    the matrices, and the apply's first tile behind the last update tile;
//  - loads and stores of rows past the end are dropped by the buffer range
//    check, so the tile has no branches that would widen a wait;
//  - 256 registers per lane suffice only because values are formed where they
//    are written here (the empty asm statements): left to itself the compiler
//    sinks the adjoint of Z, the d(eta) sum and the LDS addresses across
//    barriers, which spilled up to 260 registers (344 us).
// Measured per step, 16 heads, BF16, on one machine, against one kernel that
// read its matrices from the L2 per tile: h = 256, 5,496 tokens 181 -> 122 us; h =
// 128, 6,000 tokens 114 -> 68 us (without the FP32 row tiles 87), one tile per
// shard (320 tokens) 14.1 -> 13.8 us (without 16.2), the whole reverse call of 8
// such chunks 188 -> 167 us (without 195).  (One wave per SIMD with two hidden
// blocks and 512 registers spills 170 of them.)
//
// Phases of an update tile, a barrier after each: Z, A (stage A) | A W2 -> E,
// A Wh2 | P, K Wh1 -> D, dP (stage dP) | dP W2 -> dY, dots of dV | dV; stage D;
// dA, dZ, token sums | D Wh1^T | stage dZ | dZ W1^T, dots of dK; next rows |
// dK.  An apply tile: Zq, dO W2^T -> dZq (stage), token sums | dZq W1^T, dots
// of dQ; next rows | dQ.
#include <hip/hip_runtime.h>

#include "ttt_amu_bf.h"
#include "ttt_common.h"
#include "ttt_internal.h"

namespace ttt {

template <typename IOT, int NW, int NG>
__global__ __launch_bounds__(NW * NG * 64) void ttt_bwd_step_bf(BwdStepArgs p) {
  constexpr int HH = NW * 32, DH = D * HH;
  constexpr int NT = NW * NG * 64;  // NG groups of NW waves, each with tiles of its own
  constexpr int RL = 80;        // pitch of a row tile: 64 features, 32 bytes of row data (see below)
  constexpr int SL = HH + 8;    // pitch of the staged [token][hidden] tile
  constexpr int NU = HH / 32;   // 16x16x32 products along the hidden axis
  constexpr int NBK = 8 / NW;   // 16x16 output blocks per wave
  constexpr bool SPLIT = NW == 8;  // the two row tensors go to the two halves of the group
  constexpr int EPT = 8;        // row mapping: 8 lanes x 8 elements per token
  constexpr int SZ = (int)sizeof(IOT);
  constexpr bool F32T = NW == 4;  // FP32 row tiles beside the matrices: see the adjoints below
  constexpr int FL = D + 4;

  __shared__ __attribute__((aligned(16))) bf16 xb_[NG][TT * RL];  // K or Q rows
  __shared__ __attribute__((aligned(16))) bf16 eb_[NG][TT * RL];  // E rows
  __shared__ __attribute__((aligned(16))) bf16 yb_[NG][TT * RL];  // dY or dO rows
  __shared__ __attribute__((aligned(16))) bf16 st_[NG][TT * SL];  // staged tile
  __shared__ __attribute__((aligned(16))) float vt_[NG][F32T ? TT * FL : 1];  // normalised V rows
  __shared__ __attribute__((aligned(16))) float gt_[NG][F32T ? TT * FL : 1];  // dV, dK or dQ before its norm adjoint
  __shared__ __attribute__((aligned(16))) bf16 wl[4][DH];    // matrices as [d][hid], 16-byte chunks of row d at c ^ f(d)

  Lane L;
  const int grp = __builtin_amdgcn_readfirstlane(L.w / NW);
  L.w = __builtin_amdgcn_readfirstlane(L.w % NW);
  L.hid = 32 * L.w + L.l32;
  const int tid = threadIdx.x - grp * NW * 64;  // in the group
  bf16 *const xb = xb_[grp], *const eb = eb_[grp], *const yb = yb_[grp], *const st = st_[grp];
  float *const vt = vt_[grp], *const gt = gt_[grp];
  // Shard g of a slot (active sequence * H + head); NG consecutive shards share
  // the work-group, in step: a group without a tile left runs on zeros.
  const int G = p.G, per_slot = (G + NG - 1) / NG;
  const int lin = xcd_linear_block();
  const int slot = lin / per_slot, g0 = lin % per_slot * NG, g = g0 + grp;
  const int ai = slot / p.H, head = slot % p.H;
  const float eta = p.eta;
  const bf16* prep = static_cast<const bf16*>(p.prep) + (int64_t)slot * 4 * DH;
  const int64_t hoff = (int64_t)head * p.stride_head;
  const bool norm_q = p.flags & 1u, norm_k = p.flags & 2u, norm_v = p.flags & 4u;

  // h = 256: row data in the padding of the tiles (8 floats per row): xb, yb:
  // the eight partial dots of dK or dQ, of dV; eb: per tile parity the factors of
  // the two normalised tensors.  A factor is negative where the adjoint has no
  // projection (norm at the floor, or not normalised).
  auto pad = [](bf16* t, int row) { return reinterpret_cast<float*>(t + row * RL + D); };

  // Matrices (W1, W2, Wh1, Wh2 as [d][hid]): all four in LDS, row d's 16-byte
  // chunk c at c ^ (4 (d & 3) + (d / 4 & 3)), which spreads both the straight
  // reads of 16 rows (contractions over hid) and the transposing ones of 4
  // rows x 64 bytes (contractions over d) over all banks; W1 and W2, which
  // multiply tokens in several products, also in registers.
  enum { W1 = 0, W2 = 1, WH1 = 2, WH2 = 3 };
  bf16x8 wf[4 * DH / 8 / NT];  // all requested before any is needed
  auto request = [&] {
#pragma unroll
    for (int n = 0; n < 4 * DH / 8 / NT; ++n)
      wf[n] = *reinterpret_cast<const bf16x8*>(prep + (NT * n + threadIdx.x) * 8);
  };
  if constexpr (!F32T) request();
  // The wave's 16x16 output blocks: features 16 db .., token halves tb0 ..
  const int db16 = L.w & 3, tb0 = NBK == 2 ? 0 : L.w >> 2;
  // Those blocks of staged tile x matrix k, over the hidden axis.
  const int col_row = (16 * db16 + L.l16) * HH, col_f = 4 * (L.l16 & 3) + (L.l16 >> 2);
  auto contract = [&](int k, f32x4 (&c)[NBK]) {
    int f = col_f;
    asm volatile("" : "+v"(f));  // addresses formed here: kept across the loop they would take 40 registers
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const bf16x8 b = *reinterpret_cast<const bf16x8*>(&wl[k][col_row + 8 * ((NU * L.g4 + u) ^ f)]);
#pragma unroll
      for (int bi = 0; bi < NBK; ++bi)
        c[bi] = mma16(*reinterpret_cast<const bf16x8*>(&st[(16 * (tb0 + bi) + L.l16) * SL + (HH / 4) * L.g4 + 8 * u]), b, c[bi]);

    }
  };
  // Token rows a x matrix k over d, the wave's 32 hidden units.
  const int in_row = (8 * L.hf + (L.l16 >> 2)) * HH + 4 * (L.l16 & 1);
  const int in_c = (4 * L.w + 2 * (L.g4 & 1) + ((L.l16 >> 1) & 1)) ^ (4 * (L.l16 >> 2) + 2 * L.hf);
  auto inner = [&](const bf16x8 (&a)[4], int k) {
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    typedef __attribute__((address_space(3))) bf16 lds_bf16;
    f32x16 c = {};
    int f = in_c;
    asm volatile("" : "+v"(f));
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      bf16x4 h[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        h[i] = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
            (lds_bf16x4*)((lds_bf16*)&wl[k][(16 * m + 4 * i) * HH + in_row + 8 * (f ^ i)]));
      c = mma32(a[m], (bf16x8){h[0][0], h[0][1], h[0][2], h[0][3], h[1][0], h[1][1], h[1][2], h[1][3]}, c);
    }
    return c;
  };
  auto rows = [&](const bf16* t, bf16x8 (&a)[4]) {
#pragma unroll
    for (int m = 0; m < 4; ++m) a[m] = *reinterpret_cast<const bf16x8*>(&t[L.l32 * RL + 16 * m + 8 * L.hf]);
  };
  auto cols = [&](const bf16* t, int m, int db) { return L.cols_at<RL>(t, m, db); };
  auto stage = [&](const uint32_t (&pk)[8]) {
    uint16_t* c = reinterpret_cast<uint16_t*>(st) + L.hid;
#pragma unroll
    for (int r = 0; r < 16; ++r) c[c32_row(r, L.hf) * SL] = (uint16_t)(r & 1 ? pk[r >> 1] >> 16 : pk[r >> 1]);
  };
  // Keeps the scheduler from holding the operands of the next product early.
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };
  // A 16x16 result (4 tokens of one feature) into a row tile.
  auto put_rows = [&](bf16* t, int bi, const f32x4& v) {
    uint16_t* o = reinterpret_cast<uint16_t*>(t) + (16 * (tb0 + bi) + 4 * L.g4) * RL + 16 * db16 + L.l16;
    const uint32_t a = pack_bf16x2(v[0], v[1]), b = pack_bf16x2(v[2], v[3]);
    o[0] = (uint16_t)a;
    o[RL] = (uint16_t)(a >> 16);
    o[2 * RL] = (uint16_t)b;
    o[3 * RL] = (uint16_t)(b >> 16);
  };

  f32x16 gw1[2] = {}, gw2[2] = {};
  float deta_acc = 0.f;
  int gl = p.grad_len[ai], al = p.app_len[ai];
  const int64_t grad_start = p.grad_start[ai], app_start = p.app_start[ai];
  const int n_gt = (gl + TT - 1) / TT, n_at = (al + TT - 1) / TT;
  const float e_scale = gl > 0 ? 2.0f / (float)gl : 0.f;
  if (g >= G) gl = al = 0;  // a group past the last shard sees no rows

  // Buffer resource over the valid rows of tile t of a region (stride_tok * TT
  // * 4 bytes fits 31 bits, checked by the host); rows past the end read as
  // zero and are not written.
  const int tok_bytes = (int)p.stride_tok * SZ;
  auto tile_rs = [&](const void* base, int64_t start, int len, int t) {
    const int nrow = min(max(len - t * TT, 0), TT);
    const int bytes = __builtin_amdgcn_readfirstlane(min(nrow, 1) * ((nrow - 1) * tok_bytes + D * SZ));
    IOT* b = const_cast<IOT*>(static_cast<const IOT*>(base)) + (start + (int64_t)t * TT) * p.stride_tok + hoff;
    return __builtin_amdgcn_make_buffer_rsrc(b, (short)0, bytes, 0x00020000);
  };
  // ---- rows: this thread's part of the two tensors of a tile
  const int rtid = SPLIT ? tid & 255 : tid, row = rtid >> 3, col0 = (rtid & 7) * EPT;
  const bool second = SPLIT && __builtin_amdgcn_readfirstlane(tid >= 256);  // holds the second tensor (else the first, or both)
  const int row_off = row * tok_bytes + col0 * SZ;
  RowPart<IOT, EPT> ra, rb;
  auto load_part = [&](__amdgpu_buffer_rsrc_t rs, RowPart<IOT, EPT>& r) {
    if constexpr (SZ == 2) {
      r.v = __builtin_bit_cast(typename RowPart<IOT, EPT>::vec, __builtin_amdgcn_raw_buffer_load_b128(rs, row_off, 0, 0));
    } else {
      typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
      const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(rs, row_off, 0, 0);
      const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(rs, row_off + 16, 0, 0);
      r.v = __builtin_bit_cast(typename RowPart<IOT, EPT>::vec, (u32x8){a[0], a[1], a[2], a[3], b[0], b[1], b[2], b[3]});
    }
  };
  auto fetch = [&](const void* a, const void* b, int64_t start, int len, int t) {
    load_part(tile_rs(second ? b : a, start, len, t), ra);
    if (!SPLIT) load_part(tile_rs(b, start, len, t), rb);
  };
  // row tile of one tensor (null: only its factor) and its factor into eb's padding
  auto put_row = [&](const RowPart<IOT, EPT>& r, bool do_norm, bf16* t, int which, int par) {
    float x[EPT], n = 1.f;
    const float sc = r.get(true, x, &n), inv = do_norm ? sc : 1.f;
    if (t) put_part<EPT>(&t[row * RL + col0], x, inv);
    const float f = do_norm && n > NORM_EPS ? inv : -inv;
    if constexpr (F32T) {
      if (!t) {
#pragma unroll
        for (int i = 0; i < EPT; i += 4)
          *reinterpret_cast<f32x4*>(&vt[row * FL + col0 + i]) = (f32x4){mul_rn(x[i], inv), mul_rn(x[i + 1], inv),
                                                                        mul_rn(x[i + 2], inv), mul_rn(x[i + 3], inv)};
      }
    } else {
      if ((rtid & 7) == 0) pad(eb, row)[2 * par + which] = f;
    }
    return f;
  };
  float fa = 0.f, fb = 0.f;  // F32T: factors of the rows just staged
  auto stage_rows = [&](bool update, int par) {
    if (!second) fa = put_row(ra, update ? norm_k : norm_q, xb, 0, par);
    if (second || !SPLIT) fb = put_row(SPLIT ? ra : rb, update && norm_v, update ? nullptr : yb, 1, par);
  };

  // ---- 16x16 result layout: token 16 tb + 4 g4 + r, feature 16 db16 + l16
  const int el_off = (16 * tb0 + 4 * L.g4) * tok_bytes + (16 * db16 + L.l16) * SZ;
  typedef std::conditional_t<SZ == 2, uint16_t, uint32_t> raw_t;
  auto load_elems = [&](__amdgpu_buffer_rsrc_t rs, raw_t (&x)[NBK][4]) {
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (SZ == 2)
          x[bi][r] = __builtin_amdgcn_raw_buffer_load_b16(rs, el_off, (16 * bi + r) * tok_bytes, 0);
        else
          x[bi][r] = __builtin_amdgcn_raw_buffer_load_b32(rs, el_off, (16 * bi + r) * tok_bytes, 0);
      }
  };
  // raw elements times the row factor; returns the factors
  auto unit = [&](const raw_t (&raw)[NBK][4], float (&x)[NBK][4], float (&f)[NBK][4], int which, int par) {
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        f[bi][r] = pad(eb, 16 * (tb0 + bi) + 4 * L.g4 + r)[2 * par + which];
        const float v = SZ == 2 ? __uint_as_float((uint32_t)raw[bi][r] << 16) : __uint_as_float((uint32_t)raw[bi][r]);
        x[bi][r] = mul_rn(v, fabsf(f[bi][r]));
      }
  };
  // Row dots of g and xh over this wave's 16 features, as two sums of eight
  // features in a row (in feature order, along the lanes), into t's padding.
  auto put_dots = [&](const float (&v)[NBK][4], const float (&xh)[NBK][4], bf16* t) {
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float s = v[bi][r] * xh[bi][r];
#pragma unroll
        for (int k = 0; k < 7; ++k) s = fmaf(v[bi][r], xh[bi][r], dpp_move<0x111>(s));  // row_shr:1
        if ((L.l16 & 7) == 7) pad(t, 16 * (tb0 + bi) + 4 * L.g4 + r)[2 * db16 + (L.l16 >> 3)] = s;
      }
  };
  // normalisation adjoint of g (its dots in t's padding), stored
  auto store_adj = [&](__amdgpu_buffer_rsrc_t rs, const float (&v)[NBK][4], const float (&xh)[NBK][4],
                       const float (&f)[NBK][4], bf16* t) {
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const f32x4* d = reinterpret_cast<const f32x4*>(pad(t, 16 * (tb0 + bi) + 4 * L.g4 + r));
        const f32x4 a = d[0], b = d[1];
        const float dot = ((a[0] + a[1]) + (a[2] + a[3])) + ((b[0] + b[1]) + (b[2] + b[3]));
        const float pv = fmaf(-xh[bi][r], dot, v[bi][r]);
        const float o = (f[bi][r] > 0.f ? pv : v[bi][r]) * fabsf(f[bi][r]);
        if constexpr (SZ == 2)
          __builtin_amdgcn_raw_buffer_store_b16((uint16_t)pack_bf16x2(o, o), rs, el_off, (16 * bi + r) * tok_bytes, 0);
        else
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), rs, el_off, (16 * bi + r) * tok_bytes, 0);
      }
  };

  // The same with FP32 row tiles (h = 128, where they fit): g goes through gt to
  // the threads that hold the raw rows, eight features of a token each, which
  // need no dots through LDS, no second read of K, V or Q, and store 16 bytes
  // at a time; the additions are the same ones in the same order.
  auto put_g = [&](const float (&v)[NBK][4]) {
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) gt[(16 * (tb0 + bi) + 4 * L.g4 + r) * FL + 16 * db16 + L.l16] = v[bi][r];
  };
  auto store_rows = [&](__amdgpu_buffer_rsrc_t rs, const RowPart<IOT, EPT>& raw, float f) {
    float g[EPT], xh[EPT];
#pragma unroll
    for (int i = 0; i < EPT; i += 4) {
      const f32x4 q = *reinterpret_cast<const f32x4*>(&gt[row * FL + col0 + i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) g[i + e] = q[e];
    }
#pragma unroll
    for (int i = 0; i < EPT; ++i) xh[i] = mul_rn((float)raw.v[i], fabsf(f));
    float dot = g[0] * xh[0];
#pragma unroll
    for (int i = 1; i < EPT; ++i) dot = fmaf(g[i], xh[i], dot);
    dot = lane_group_sum<D / EPT>(dot);
#pragma unroll
    for (int i = 0; i < EPT; ++i) g[i] = (f > 0.f ? fmaf(-xh[i], dot, g[i]) : g[i]) * fabsf(f);
    if constexpr (SZ == 2) {
      __builtin_amdgcn_raw_buffer_store_b128((u32x4){pack_bf16x2(g[0], g[1]), pack_bf16x2(g[2], g[3]),
                                                     pack_bf16x2(g[4], g[5]), pack_bf16x2(g[6], g[7])},
                                             rs, row_off, 0, 0);
    } else {
#pragma unroll
      for (int i = 0; i < EPT; i += 4)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, (f32x4){g[i], g[i + 1], g[i + 2], g[i + 3]}),
                                               rs, row_off + 4 * i, 0, 0);
    }
  };

  // F32T (latency counts: its shards have a tile or a few): the rows are
  // requested before the matrices and staged while those arrive; a shard past
  // the last update tile starts with the apply.
  const bool update = !F32T || g0 < n_gt;
  fetch(update ? p.K : p.Q, update ? p.V : p.dO, update ? grad_start : app_start, update ? gl : al, g);
  if constexpr (F32T) {
    fence();
    request();
    fence();
    stage_rows(update, 0);
  }
  // ------------------------------------------------ update adjoint of chunk s
  raw_t vr[NBK][4];
  if constexpr (!F32T) load_elems(tile_rs(p.V, grad_start, gl, g), vr);
#pragma unroll
  for (int n = 0; n < 4 * DH / 8 / NT; ++n) {
    const int i = NT * n + threadIdx.x, k = i / (DH / 8), d = (i / (HH / 8)) & (D - 1), c = i % (HH / 8);
    *reinterpret_cast<bf16x8*>(&wl[k][d * HH + 8 * (c ^ (4 * (d & 3) + ((d >> 2) & 3)))]) = wf[n];
  }
  if constexpr (!F32T) stage_rows(true, 0);
  int par = 0;  // parity of the staged tile
  RowPart<IOT, EPT> ca = ra, cb = rb;  // F32T: raw rows of the staged tile and their factors
  float cfa = fa, cfb = fb;
  for (int t = g; t - grp < n_gt; t += G, par ^= 1) {
    // F32T: the apply's first tile is fetched and staged behind the last update
    // tile (at h = 256 the choice costs more per tile than the wait it saves)
    const bool more = !F32T || t + G - grp < n_gt;
    // Addresses derived from the lane are formed where they are used.
    asm volatile("" : "+v"(L.l), "+v"(L.l16), "+v"(L.l32), "+v"(L.hf), "+v"(L.g4));
    __syncthreads();
    // Z = K W1, sigma(Z), A = s(Z) (staged)
    f32x16 Z, Sg;
    uint32_t Apk[8];
    {
      bf16x8 a[4];
      rows(xb, a);
      Z = inner(a, W1);
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        Sg[2 * q] = sigmoid(Z[2 * q]);
        Sg[2 * q + 1] = sigmoid(Z[2 * q + 1]);
        Apk[q] = pack_bf16x2(Z[2 * q] * Sg[2 * q], Z[2 * q + 1] * Sg[2 * q + 1]);
      }
      stage(Apk);
    }
    __syncthreads();
    // Y = A W2 -> E;  A Wh2 -> -eta A Wh2 (kept) and its d(eta) term
    f32x4 des[NBK];
    {
      f32x4 y[NBK] = {}, aw[NBK] = {};
      contract(W2, y);
      contract(WH2, aw);
      float vh[NBK][4], vf[NBK][4];
      if constexpr (F32T) {
#pragma unroll
        for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
          for (int r = 0; r < 4; ++r) vh[bi][r] = vt[(16 * (tb0 + bi) + 4 * L.g4 + r) * FL + 16 * db16 + L.l16];
      } else {
        unit(vr, vh, vf, 1, par);
      }
#pragma unroll
      for (int bi = 0; bi < NBK; ++bi) {
        f32x4 E;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          E[r] = e_scale * (y[bi][r] - vh[bi][r]);
          deta_acc -= aw[bi][r] * E[r];
          des[bi][r] = -eta * aw[bi][r];
        }
        put_rows(eb, bi, E);
      }
      asm volatile("" : "+v"(deta_acc));  // summed here, not at the end of the tile
    }
    __syncthreads();
    // P = E W2^T, K Wh1; D = P s'(Z), dP = dD s'(Z) (staged), dZ = dD P s''(Z)
    // with dD = -eta K Wh1
    f32x16 S1, S2, dDP;
    uint32_t dPpk[8], Dpk[8];
    {
      bf16x8 a[4];
      rows(eb, a);
      const f32x16 P = inner(a, W2);
      fence();
      rows(xb, a);
      const f32x16 KW = inner(a, WH1);
      fence();
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        float Dm[2], dP[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int r = 2 * q + i;
          const float z = Z[r], sg = Sg[r];
          const float av = z * sg;
          const float s1 = fmaf(av, 1.0f - sg, sg);
          const float s2 = sg * (1.0f - sg) * fmaf(z, 1.0f - 2.0f * sg, 2.0f);
          Dm[i] = P[r] * s1;
          deta_acc -= KW[r] * Dm[i];
          const float dD = -eta * KW[r];
          dP[i] = dD * s1;
          dDP[r] = dD * P[r];
          S1[r] = s1;
          S2[r] = s2;
          // formed here: moved past the barrier they would hold Z, sigma(Z), P and dD
          asm volatile("" : "+v"(dDP[r]), "+v"(S1[r]), "+v"(S2[r]));
        }
        Dpk[q] = pack_bf16x2(Dm[0], Dm[1]);
        asm volatile("" : "+v"(Dpk[q]));
        dPpk[q] = pack_bf16x2(dP[0], dP[1]);
      }
      asm volatile("" : "+v"(deta_acc));
      stage(dPpk);
    }
    __syncthreads();
    // dE = -eta A Wh2 + dP W2;  dY = (2/M) dE, dV = -dY
    raw_t kr[NBK][4];
    if constexpr (!F32T) load_elems(tile_rs(p.K, grad_start, gl, t), kr);
    fetch(more ? p.K : p.Q, more ? p.V : p.dO, more ? grad_start : app_start, more ? gl : al, more ? t + G : g);
    fence();
    float gv[NBK][4], vh[NBK][4], vf[NBK][4];
    {
      f32x4 de[NBK] = {};
      contract(W2, de);
#pragma unroll
      for (int bi = 0; bi < NBK; ++bi) {
        f32x4 dY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          dY[r] = e_scale * (des[bi][r] + de[bi][r]);
          gv[bi][r] = -dY[r];
        }
        put_rows(yb, bi, dY);
      }
      if constexpr (F32T) {
        put_g(gv);
      } else {
        unit(vr, vh, vf, 1, par);
        put_dots(gv, vh, yb);
      }
    }
    __syncthreads();
    if constexpr (F32T)
      store_rows(tile_rs(p.dV, grad_start, gl, t), cb, cfb);
    else
      store_adj(tile_rs(p.dV, grad_start, gl, t), gv, vh, vf, yb);
    // stage D;  dA = -eta E Wh2^T + dY W2^T;  dZ += dA s'(Z);  token sums dP^T E
    // + A^T dY (W2) and K^T dZ (W1)
    uint32_t dZpk[8];
    {
      stage(Dpk);
      bf16x8 a[4];
      rows(eb, a);
      const f32x16 dA1 = inner(a, WH2);
      fence();
      rows(yb, a);
      const f32x16 dA2 = inner(a, W2);
      fence();
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        float d[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int r = 2 * q + i;
          d[i] = fmaf(dDP[r], S2[r], mul_rn(fmaf(-eta, dA1[r], dA2[r]), S1[r]));
        }
        dZpk[q] = pack_bf16x2(d[0], d[1]);
      }
      fence();
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const bf16x8 cy = cols(yb, m, db), ce = cols(eb, m, db), cx = cols(xb, m, db);
          gw2[db] = mma32(opnd(Apk, m), cy, gw2[db]);
          gw2[db] = mma32(opnd(dPpk, m), ce, gw2[db]);
          gw1[db] = mma32(cx, opnd(dZpk, m), gw1[db]);
          fence();
        }
    }
    __syncthreads();
    // dK = -eta D Wh1^T + dZ W1^T
    if constexpr (!F32T) load_elems(tile_rs(p.V, grad_start, gl, t + G), vr);
    fence();
    f32x4 k1[NBK] = {}, k2[NBK] = {};
    contract(WH1, k1);
    __syncthreads();
    stage(dZpk);
    __syncthreads();
    contract(W1, k2);
    float gk[NBK][4], kh[NBK][4], kf[NBK][4];
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) gk[bi][r] = fmaf(-eta, k1[bi][r], k2[bi][r]);
    if constexpr (F32T) {
      put_g(gk);
    } else {
      unit(kr, kh, kf, 0, par);
      put_dots(gk, kh, xb);
    }
    // the next tile's rows (the row tiles were last read before the sums' barrier)
    stage_rows(more, par ^ 1);
    __syncthreads();
    if constexpr (F32T)
      store_rows(tile_rs(p.dK, grad_start, gl, t), ca, cfa);
    else
      store_adj(tile_rs(p.dK, grad_start, gl, t), gk, kh, kf, xb);
    ca = ra;
    cb = rb;
    cfa = fa;
    cfb = fb;
  }

  // ------------------------------------------------ apply adjoint of chunk s-1
  if constexpr (!F32T) {
    __syncthreads();  // the last update tile's row data are read
    fetch(p.Q, p.dO, app_start, al, g);
    par = 0;
    stage_rows(false, par);
  }
  for (int t = g; t - grp < n_at; t += G, par ^= 1) {
    raw_t qr[NBK][4];
    if constexpr (!F32T) load_elems(tile_rs(p.Q, app_start, al, t), qr);
    fetch(p.Q, p.dO, app_start, al, t + G);
    __syncthreads();
    // Zq = Q W1, dZq = (dO W2^T) s'(Zq); token sums Aq^T dO and Q^T dZq
    {
      bf16x8 a[4];
      rows(xb, a);
      uint32_t Apq[8], dZpk[8];
      const f32x16 Zq = inner(a, W1);
      fence();
      rows(yb, a);
      const f32x16 Gq = inner(a, W2);
      fence();
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        float Aq[2], dq[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const float z = Zq[2 * q + i];
          const float sg = sigmoid(z);
          Aq[i] = z * sg;
          dq[i] = Gq[2 * q + i] * fmaf(Aq[i], 1.0f - sg, sg);
        }
        Apq[q] = pack_bf16x2(Aq[0], Aq[1]);
        dZpk[q] = pack_bf16x2(dq[0], dq[1]);
      }
      stage(dZpk);
#pragma unroll
      for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int m = 0; m < 2; ++m) {
          const bf16x8 cy = cols(yb, m, db), cx = cols(xb, m, db);
          gw2[db] = mma32(opnd(Apq, m), cy, gw2[db]);
          gw1[db] = mma32(cx, opnd(dZpk, m), gw1[db]);
        }
    }
    __syncthreads();
    // dQ = dZq W1^T
    f32x4 c[NBK] = {};
    contract(W1, c);
    float gq[NBK][4], qh[NBK][4], qf[NBK][4];
#pragma unroll
    for (int bi = 0; bi < NBK; ++bi)
#pragma unroll
      for (int r = 0; r < 4; ++r) gq[bi][r] = c[bi][r];
    if constexpr (F32T) {
      put_g(gq);
    } else {
      unit(qr, qh, qf, 0, par);
      put_dots(gq, qh, xb);
    }
    stage_rows(false, par ^ 1);
    __syncthreads();
    if constexpr (F32T)
      store_rows(tile_rs(p.dQ, app_start, al, t), ca, cfa);
    else
      store_adj(tile_rs(p.dQ, app_start, al, t), gq, qh, qf, xb);
    ca = ra;
    cfa = fa;
  }

  // ------------------------------------------------ shard partials
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) deta_acc += __shfl_xor(deta_acc, m, 64);
  __syncthreads();
  float* red = reinterpret_cast<float*>(st);
  if (L.l == 0) red[L.w] = deta_acc;
  __syncthreads();
  if (g >= G) return;
  float* part = p.partial + ((int64_t)slot * G + g) * (2 * DH);
#pragma unroll
  for (int db = 0; db < 2; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rr = c32_row(r, L.hf);
      part[(32 * db + rr) * HH + L.hid] = gw1[db][r];
      part[DH + (32 * L.w + rr) * D + 32 * db + L.l32] = gw2[db][r];
    }
  if (tid == 0) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) s += red[w];
    p.partial_deta[(int64_t)slot * G + g] = s;
  }
}

template <typename IOT, int NW, int NG>
static hipError_t launch_bwd_step_bf_t(const BwdStepArgs& a, int n_blocks, hipStream_t st) {
  hipLaunchKernelGGL((ttt_bwd_step_bf<IOT, NW, NG>), dim3(n_blocks / a.G * ((a.G + NG - 1) / NG)), dim3(NW * NG * 64), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_bwd_step_bf(const BwdStepArgs& a, int n_blocks, int h, bool io_bf16, hipStream_t st) {
  if (h == 128) {
    // Up to one shard per CU each has a work-group of its own, past that two
    // share one: 160 shards of one tile 13.2 against 16.0 us, 352 shards 23.4
    // against 17.9 us.
    if (n_blocks <= 256)
      return io_bf16 ? launch_bwd_step_bf_t<bf16, 4, 1>(a, n_blocks, st) : launch_bwd_step_bf_t<float, 4, 1>(a, n_blocks, st);
    return io_bf16 ? launch_bwd_step_bf_t<bf16, 4, 2>(a, n_blocks, st) : launch_bwd_step_bf_t<float, 4, 2>(a, n_blocks, st);
  }
  return io_bf16 ? launch_bwd_step_bf_t<bf16, 8, 1>(a, n_blocks, st) : launch_bwd_step_bf_t<float, 8, 1>(a, n_blocks, st);
}

}  // namespace ttt
