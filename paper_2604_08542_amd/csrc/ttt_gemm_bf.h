// BF16 matrix-core GEMM core of the large-state steps and of the surrounding
// layer's projections on gfx950: C[m][n] = sum_k A(m, k) B(k, n), FP32
// accumulation, the caller's elementwise work fused into an epilogue functor.
//
// What bounds it, and the shape that follows:
//  - LDS traffic.  A wave that owns 128 x 64 of C reads 6 KiB of operand
//    fragments per eight 32x32x16 products (64 x 64: 8 KiB), and a 256 x 256
//    work-group tile stages 32 KiB per 32-wide contraction slice; together
//    128 B per clock and CU at the full matrix rate, which the LDS sustains.
//    Hence 8 waves (2 x 4) on one 256 x 256 tile, one work-group per CU.
//  - Load latency.  Slices go from global memory straight into an LDS ring of
//    four slices (buffer loads with the LDS destination, no registers), three
//    slices ahead.  One barrier per slice; the first fragments of a slice are
//    read before the barrier that precedes its products, so the products
//    start right behind the barrier.
//  - Tile starts.  The kernel is persistent (at most one work-group per CU);
//    the ring runs on into the next tile while the epilogue of the last one
//    executes.
// Measured on MI355X at 10,992 rows, against the register-staged 128 x 128
// core it replaces, epilogues included: Z = K W1 (to 4096 columns) 131 -> 111
// us, Y = A W2 (over 4096) 136 -> 104 us, the two weight terms 238 -> 197 us,
// the paper unit's three 336 -> 254 us; the paper-state forward 7.53 -> 5.69
// ms, the paper unit's training step 14.7 -> 11.2 ms.  At full occupancy the
// products alone run near 1.3 PFLOP/s (a square 8192 library product: 1.37);
// what is left is the epilogue, during which the matrix cores idle.
//
// Results sit transposed in the registers (the B fragment is the first
// operand of the product) with the columns read in an order that gives a lane
// 16 consecutive columns of one row per 32x32 block.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "ttt_common.h"
#include "ttt_internal.h"

namespace ttt {
namespace bfg {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Operand layouts: KMAJ [m or n][k], MNMAJ [k][m or n].
enum { KMAJ = 0, MNMAJ = 1 };
constexpr int KS = 32;      // contraction slice (64 bytes of a k-major row)
constexpr int NST = 4;      // slices in the LDS ring
constexpr int NW = 8;       // waves per work-group
constexpr int NTHR = NW * 64;
constexpr int MAX_WG = 256;  // one work-group per CU
constexpr int STAGE_BYTES = 4096;  // per wave: 32 rows x 64 BF16 columns on their way to row-major memory

// WM x WN waves, each MB x NB blocks of 32x32.
template <int MB_, int NB_, int WM_, int WN_>
struct Tile {
  static constexpr int MB = MB_, NB = NB_, WM = WM_, WN = WN_;
  static constexpr int BM = WM * MB * 32, BN = WN * NB * 32;
  static_assert(WM * WN == NW, "8 waves");
};
using TileL = Tile<4, 2, 2, 4>;   // 256 x 256
using TileM = Tile<3, 2, 2, 4>;   // 192 x 256
using TileH = Tile<2, 2, 2, 4>;   // 128 x 256
using TileS = Tile<1, 2, 4, 2>;   // 128 x 128
using TileL4 = Tile<2, 4, 4, 2>;  // 256 x 4 matrices of 64 columns
using TileS4 = Tile<1, 4, 4, 2>;  // 128 x 4 matrices of 64 columns

// A product (or a sum of up to four: segments) over the same operand shapes.
// With NMAT > 1 matrices, B[0..NMAT-1] are multiplied by the same A and a
// wave's block n of 32 columns belongs to matrix n.
struct GemmArgs {
  const bf16* A[4];
  const bf16* B[4];
  int lda, ldb, a_rows, b_rows;  // rows as stored (bounds of the loads)
  int K;                         // contraction length of one segment
  int nseg;
  float seg0_scale;              // factor of segment 0 (when nseg > 1)
  int M, N;                      // result rows, columns of one matrix
};

typedef __attribute__((address_space(3))) char lds_char;

// 64 lanes x 16 bytes from global memory to LDS at byte address lds +
// 16 * lane; reads past the resource's end deliver zeros.  The compiler does
// not count these loads; the waits below do.  (It warns that m0 is a reserved
// register: the clobber is what keeps it from holding a value of its own there.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(u32x4 rs, int vo, int so, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(vo), "s"(rs),
               "s"(so)
               : "memory", "m0");
}
#pragma clang diagnostic pop
// All but the newest N of this wave's memory operations are complete, then
// the work-group's barrier.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(N) : "memory");
}
__device__ __forceinline__ u32x4 make_rs(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  return (u32x4){(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu)),
                 (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), 0x00020000u};
}

// LDS image of an operand tile of ROWS x KS: k-major [ROWS][KS] (64-byte
// rows, 16-byte chunks XORed with bits 2-3 of the row), mn-major [KS][ROWS]
// (32-byte column runs XORed with the low bits of the row), so that both the
// 16-byte fragment reads and the transposing reads cover the banks once.
template <int LAYOUT, int ROWS>
struct Img {
  static constexpr int BYTES = ROWS * KS * 2;
  static constexpr int INSTR = BYTES / 1024;
  __device__ __forceinline__ static int swz(int row) {
    if constexpr (LAYOUT == KMAJ) return (row >> 2) & 3;
    if constexpr (ROWS == 64) return ((row >> 1) & 1) << 2;
    return (row & 3) << 2;
  }
  // Byte offset in the operand of the chunk that lane l of load q delivers.
  __device__ __forceinline__ static int voff(int q, int ld, int mn0) {
    const int l = threadIdx.x & 63;
    if constexpr (LAYOUT == KMAJ) {
      const int row = 16 * q + (l >> 2), c = (l & 3) ^ swz(row);
      return (int)(((uint32_t)(mn0 + row) * (uint32_t)ld + 8u * c) * 2u);  // past the end: beyond the resource
    } else {
      constexpr int CPR = ROWS / 8;
      const int row = q * (64 / CPR) + l / CPR, c = (l % CPR) ^ swz(row);
      return (row * ld + mn0 + 8 * c) * 2;
    }
  }
  // This lane's byte address of the fragment of 32 rows/columns from mn on,
  // contraction step 0.  PERM: the result's column order (see the top).
  template <bool PERM>
  __device__ __forceinline__ static int fbase(int mn) {
    const int l = threadIdx.x & 63, l32 = l & 31, hf = l >> 5;
    if constexpr (LAYOUT == KMAJ) {
      const int row = mn + (PERM ? 16 * ((l32 >> 2) & 1) + 4 * (l32 >> 3) + (l32 & 3) : l32);
      return row * 64 + ((hf ^ swz(row)) << 4);
    } else {
      const int l16 = l & 15, g = (l >> 4) & 1, u = l16 & 3;
      const int run = PERM ? 4 * (u & 1) + 2 * g + (u >> 1) : 4 * g + u;  // 8-byte run of 4 columns
      const int kr = 8 * hf + (l16 >> 2), bc = 2 * (mn + 4 * run);
      return kr * (ROWS * 2) + (((bc >> 4) ^ swz(kr)) << 4) + (bc & 15);
    }
  }
  // Fragment of contraction step j (16 wide) of the slice image at t.
  __device__ __forceinline__ static bf16x8 frag(const char* t, int fb, int j) {
    if constexpr (LAYOUT == KMAJ) {
      return *reinterpret_cast<const bf16x8*>(t + (fb ^ (j << 5)));
    } else {
      typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
      const char* p0 = t + fb + j * 16 * ROWS * 2;
      const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)((lds_char*)(p0)));
      const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)((lds_char*)(p0 + 4 * ROWS * 2)));
      return (bf16x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    }
  }
};

// ------------------------------------------------------------- epilogue io
// A lane's 16 values of one 32x32 block of an intermediate [rows][ld] that
// only epilogues touch, in the tile-native layout: blocks of 1,024 elements
// in row-major block order, each as two runs of 8 elements per lane, so that
// a wave's accesses are contiguous.
struct Nat {
  u32x4 v[2];
  __device__ __forceinline__ float get(int i) const {
    const uint32_t w = v[i >> 3][(i >> 1) & 3];
    return __uint_as_float((i & 1) ? (w & 0xffff0000u) : (w << 16));
  }
};
__device__ __forceinline__ int64_t nat_at(int row0, int col, int ld) {
  return ((int64_t)(row0 >> 5) * (ld >> 5) + (col >> 5)) * 1024 + (threadIdx.x & 63) * 8;
}
__device__ __forceinline__ Nat nat_load(const bf16* p, int64_t at) {
  Nat n;
  n.v[0] = *reinterpret_cast<const u32x4*>(p + at);
  n.v[1] = *reinterpret_cast<const u32x4*>(p + at + 512);
  return n;
}
__device__ __forceinline__ void nat_store(bf16* p, int64_t at, const uint32_t (&pk)[8]) {
  *reinterpret_cast<u32x4*>(p + at) = (u32x4){pk[0], pk[1], pk[2], pk[3]};
  *reinterpret_cast<u32x4*>(p + at + 512) = (u32x4){pk[4], pk[5], pk[6], pk[7]};
}
template <typename F>
__device__ __forceinline__ void pack_each(uint32_t (&pk)[8], F&& f) {
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const float a = f(2 * q), b = f(2 * q + 1);
    pk[q] = pack_bf16x2(a, b);
  }
}

// What an epilogue gets for one strip (32 rows x NB blocks of a wave).
struct Strip {
  char* stage;  // this wave's staging bytes
  int row0, rows;  // first row of the strip; result rows
  int col;         // first column of block 0
  __device__ __forceinline__ int l32() const { return threadIdx.x & 31; }
  __device__ __forceinline__ int hf() const { return (threadIdx.x >> 5) & 1; }
  __device__ __forceinline__ int row() const { return row0 + l32(); }
  __device__ __forceinline__ bool valid() const { return row() < rows; }
  // Packed BF16 blocks (NBLK adjacent ones, each lane 16 columns of its row)
  // to row-major memory, through the staging bytes so that a store covers
  // whole rows (direct 16-byte stores to 64 rows each took 18 of 97 us per
  // product at 10,992 x 4096).
  template <int NBLK>
  __device__ __forceinline__ void rows_out(bf16* dst, int64_t ld, int c0, const uint32_t (&pk)[NBLK][8]) const {
    constexpr int CPR = 4 * NBLK;  // 16-byte chunks per row
    const int l = threadIdx.x & 63, r = l & 31, h = l >> 5;
    auto sw = [](int q) { return NBLK == 2 ? (q & 7) : ((q >> 1) & 3); };
    auto fence = [] {
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    };
    fence();  // the reads of an earlier call stay before these writes
#pragma unroll
    for (int n = 0; n < NBLK; ++n)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        *reinterpret_cast<u32x4*>(stage + (r * CPR + ((4 * n + 2 * h + u) ^ sw(r))) * 16) =
            (u32x4){pk[n][4 * u], pk[n][4 * u + 1], pk[n][4 * u + 2], pk[n][4 * u + 3]};
    fence();
#pragma unroll
    for (int k = 0; k < CPR / 2; ++k) {
      const int rr = (k * 64 + l) / CPR, c = (k * 64 + l) % CPR;
      const u32x4 v = *reinterpret_cast<const u32x4*>(stage + (rr * CPR + (c ^ sw(rr))) * 16);
      if (row0 + rr < rows) *reinterpret_cast<u32x4*>(dst + (int64_t)(row0 + rr) * ld + c0 + 8 * c) = v;
    }
  }
};
// 16 consecutive floats of a row.
__device__ __forceinline__ void load16(const float* p, float (&x)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = reinterpret_cast<const f32x4*>(p)[q];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[4 * q + e] = v[e];
  }
}
// 16 consecutive io values of a row, as loaded.
template <typename T>
struct Raw16 {
  f32x4 v[4];
  __device__ __forceinline__ void load(const float* p) {
#pragma unroll
    for (int q = 0; q < 4; ++q) v[q] = reinterpret_cast<const f32x4*>(p)[q];
  }
  __device__ __forceinline__ float get(int i) const { return v[i >> 2][i & 3]; }
};
template <>
struct Raw16<bf16> : Nat {
  __device__ __forceinline__ void load(const bf16* p) {
    v[0] = reinterpret_cast<const u32x4*>(p)[0];
    v[1] = reinterpret_cast<const u32x4*>(p)[1];
  }
};
__device__ __forceinline__ void store16(float* p, const float (&x)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) reinterpret_cast<f32x4*>(p)[q] = (f32x4){x[4 * q], x[4 * q + 1], x[4 * q + 2], x[4 * q + 3]};
}

// ------------------------------------------------------------- the machine
// Per-wave state of the slice ring: where the next slice to be loaded comes
// from, the fragments in registers, the accumulators.
template <class TL, int LA, int LB, int NMAT>
struct Machine {
  static constexpr int MB = TL::MB, NB = TL::NB;
  static constexpr int RB = TL::BN / NMAT;  // B rows (columns of C) per matrix
  using IA = Img<LA, TL::BM>;
  using IB = Img<LB, RB>;
  static constexpr int SB = IA::BYTES + NMAT * IB::BYTES;  // one slice
  static constexpr int PA = (IA::INSTR + NW - 1) / NW;
  static constexpr int PB = (NMAT * IB::INSTR + NW - 1) / NW;
  static constexpr int PER = PA + PB;  // loads per wave and slice
  static constexpr int LDS = NST * SB + NW * STAGE_BYTES;
  static_assert(LDS <= 163840, "160 KiB");

  char* sm;
  uint32_t lds0;
  int w, wm, wn;
  int va[PA], vb[PB];
  int fa0[MB], fb0[NB];
  bf16x8 fa[2][MB], fb[2][NB];
  f32x16 acc[MB][NB];

  __device__ __forceinline__ void init(char* smem) {
    sm = smem;
    lds0 = (uint32_t)(uintptr_t)(lds_char*)smem;
    w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    wm = (w / TL::WN) * MB * 32;
    wn = (w % TL::WN) * (NMAT > 1 ? 32 : NB * 32);
#pragma unroll
    for (int i = 0; i < MB; ++i) fa0[i] = IA::template fbase<false>(wm + 32 * i);
#pragma unroll
    for (int n = 0; n < NB; ++n)
      fb0[n] = IA::BYTES + (NMAT > 1 ? n * IB::BYTES + IB::template fbase<true>(wn) : IB::template fbase<true>(wn + 32 * n));
  }
  // Load q of this wave's A share (a 192-row tile's twelve loads wrap around,
  // four of them repeated with the same bytes, so every wave counts alike).
  __device__ __forceinline__ int qa(int i) const { return IA::INSTR % NW == 0 ? w * PA + i : (w + NW * i) % IA::INSTR; }
  __device__ __forceinline__ int qb(int i) const { return w * PB + i; }
  __device__ __forceinline__ void tile(int lda, int ldb, int m0, int n0) {
#pragma unroll
    for (int i = 0; i < PA; ++i) va[i] = IA::voff(qa(i), lda, m0);
#pragma unroll
    for (int i = 0; i < PB; ++i) vb[i] = IB::voff(qb(i) % IB::INSTR, ldb, n0);
  }
  __device__ __forceinline__ int matrix(int i) const { return NMAT > 1 ? qb(i) / IB::INSTR : 0; }
  __device__ __forceinline__ void load(u32x4 ra, const u32x4 (&rb)[PB], int ka, int kb, int slot) {
#pragma unroll
    for (int i = 0; i < PA; ++i) dma16(ra, va[i], ka, lds0 + slot * SB + qa(i) * 1024);
#pragma unroll
    for (int i = 0; i < PB; ++i) dma16(rb[i], vb[i], kb, lds0 + slot * SB + IA::BYTES + qb(i) * 1024);
  }
  __device__ __forceinline__ void read(int slot, int j) {
    const char* t = sm + slot * SB;
#pragma unroll
    for (int n = 0; n < NB; ++n) fb[j][n] = IB::frag(t, fb0[n], j);
#pragma unroll
    for (int i = 0; i < MB; ++i) fa[j][i] = IA::frag(t, fa0[i], j);
  }
  __device__ __forceinline__ void mul(int j) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[i][n] = mma32(fb[j][n], fa[j][i], acc[i][n]);
  }
  // One slice: the ring slot s holds it; returns the next slot.  On entry
  // the fragments of its first step are in registers.
  template <typename L>
  __device__ __forceinline__ int slice(int s, L&& load_next) {
    const int sl = (s + NST - 1) & (NST - 1), s1 = (s + 1) & (NST - 1);
    // the next slice has landed for every wave, the previous one is read by none
    wait_barrier<PER*(NST - 3)>();
    load_next(sl);
    read(s, 1);
    mul(0);
    __builtin_amdgcn_sched_barrier(0);
    read(s1, 0);
    mul(1);
    return s1;
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int n = 0; n < NB; ++n) acc[i][n] = f32x16{};
  }
  __device__ __forceinline__ static constexpr int kbytes(int layout, int ld) { return (layout == KMAJ ? 1 : ld) * KS * 2; }
  __device__ __forceinline__ char* stage() const { return sm + NST * SB + w * STAGE_BYTES; }
};

// Tile t of an mt x nt grid: groups of 8 tile rows, rows fastest, so that the
// work-groups of an XCD (a run of consecutive tiles) share operand slices in
// its L2.
__device__ __forceinline__ void tile_at(int t, int mt, int nt, int& im, int& in) {
  const int per = 8 * nt, g = t / per, r = t - g * per, gm = min(8, mt - 8 * g);
  in = r / gm;
  im = 8 * g + r - in * gm;
}
// This work-group's index with the work-groups of one XCD consecutive.
__device__ __forceinline__ int xcd_index(int& first, int& count, int total) {
  const int x = blockIdx.x & 7;
  // XCD x owns items [first, first + count) of total
  const int q = total >> 3, r = total & 7;
  first = x * q + min(x, r);
  count = q + (x < r);
  return blockIdx.x >> 3;
}

template <class TL, int LB, int NMAT, class EP>
__global__ __launch_bounds__(NTHR) void k_gemm(GemmArgs g, EP ep) {
  using MC = Machine<TL, KMAJ, LB, NMAT>;
  constexpr int CN = TL::BN / NMAT;  // columns per tile (of each matrix)
  __shared__ __attribute__((aligned(1024))) char sm[MC::LDS];
  MC mc;
  mc.init(sm);
  const int mt = (g.M + TL::BM - 1) / TL::BM, nt = g.N / CN;
  int first, count;
  const int j0 = xcd_index(first, count, mt * nt), stride = (gridDim.x + 7 - (blockIdx.x & 7)) >> 3;
  const int nks = (g.K + KS - 1) / KS, nk = nks * g.nseg;
  const int ka = MC::kbytes(KMAJ, g.lda), kb = MC::kbytes(LB, g.ldb);
  // the load cursor: tile index, segment, slice of the segment
  u32x4 ra, rb[MC::PB];
  int lt = j0, lseg = 0, lk = 0;
  auto sources = [&]() {
    ra = make_rs(g.A[lseg], (uint32_t)g.a_rows * (uint32_t)g.lda * 2u);
#pragma unroll
    for (int i = 0; i < MC::PB; ++i)
      rb[i] = make_rs(g.B[NMAT > 1 ? mc.matrix(i) : lseg], (uint32_t)g.b_rows * (uint32_t)g.ldb * 2u);
  };
  auto at_tile = [&]() {
    int im, in;
    tile_at(first + lt, mt, nt, im, in);
    mc.tile(g.lda, g.ldb, im * TL::BM, in * CN);
  };
  auto load_next = [&](int slot) {  // past the last slice: the last tile's first slices again, never used
    mc.load(ra, rb, lk * ka, lk * kb, slot);
    if (++lk == nks) {
      lk = 0;
      if (++lseg == g.nseg) {
        lseg = 0;
        if (lt + stride < count) {
          lt += stride;
          at_tile();
        }
      }
      if (g.nseg > 1) sources();
    }
  };
  if (j0 < count) {
    sources();
    at_tile();
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) load_next(s);
    wait_barrier<MC::PER*(NST - 2)>();
    mc.read(0, 0);
    int s = 0;
    for (int t = j0; t < count; t += stride) {
      mc.clear();
      for (int kt = 0; kt < nk; ++kt) {
        if (g.nseg > 1 && kt == nks) {
#pragma unroll
          for (int i = 0; i < MC::MB; ++i)
#pragma unroll
            for (int n = 0; n < MC::NB; ++n) mc.acc[i][n] *= g.seg0_scale;
        }
        s = mc.slice(s, load_next);
      }
      int im, in;
      tile_at(first + t, mt, nt, im, in);
      Strip st{mc.stage(), 0, g.M, in * CN + mc.wn};
      ep.template tile<MC::MB, MC::NB>(st, im * TL::BM + mc.wm, mc.acc);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  ep.finish();
}

// Base of the epilogues.  pre(strip) loads a strip's inputs (requested one
// strip ahead of their use, or with AHEAD = false, for inputs too large to be
// held twice beside the accumulators, when the strip begins); strip(strip,
// inputs, block results) does the work.
template <class D>
struct Ep {
  static constexpr bool AHEAD = true;
  struct In {};
  template <int NB>
  __device__ __forceinline__ In pre(const Strip&) const {
    return {};
  }
  __device__ __forceinline__ void finish() {}
  template <int MB, int NB>
  __device__ __forceinline__ void tile(Strip st, int row0, f32x16 (&acc)[MB][NB]) {
    D& d = static_cast<D&>(*this);
    if (row0 >= st.rows) return;
    st.row0 = row0;
    auto in = d.template pre<NB>(st);
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      st.row0 = row0 + 32 * i;
      if (st.row0 >= st.rows) return;
      if (!D::AHEAD && i > 0) in = d.template pre<NB>(st);
      auto cur = in;
      if (D::AHEAD && i + 1 < MB && st.row0 + 32 < st.rows) {
        Strip nx = st;
        nx.row0 += 32;
        in = d.template pre<NB>(nx);
      }
      d.template strip<NB>(st, cur, acc[i]);
    }
  }
  // Sum over a wave's lanes of one value, in a fixed order, in every lane.
  __device__ __forceinline__ static float wave_sum(float v) {
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
    return v;
  }
  // One value per wave of the launch (a scalar sum's partials).
  __device__ __forceinline__ static void put_partial(float* part, float v) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) part[blockIdx.x * NW + (threadIdx.x >> 6)] = v;
  }
};

// Tile choice.  The whole of a launch takes the rounds of its largest share;
// a round costs its matrix work at the tile's rate plus a fixed part (ring
// fill, epilogue).  Rates per CU measured on MI355X at full occupancy: 256 x
// 256 about 5.2 TFLOP/s, 192 x 256 about 5.0, 128 x 128 about 2.9.  The
// smaller tiles win where the larger ones leave CUs idle: 10,992 x 1024 over
// 4096 is 172 tiles of 256 x 256 (87 us) but 232 of 192 x 256 (80 us).
enum { T_L = 0, T_M = 1, T_S = 2 };
// A launched product: its work-groups (the waves that write partials are 8
// times as many) and the 32-row blocks of a wave.
struct Launched {
  int wgs, blocks;
};
inline int64_t gemm_tiles(int cfg, int M, int N, int nmat) {
  const int bm = cfg == T_L ? 256 : cfg == T_M ? 192 : 128;
  const int cn = nmat == 4 ? 64 : (cfg == T_S ? 128 : 256) / nmat;
  return (int64_t)((M + bm - 1) / bm) * (N / cn);
}
inline int pick_tile(int M, int N, int nmat, int64_t K) {
  int best = T_S;
  double bc = 1e30;
  for (int cfg : {T_L, T_M, T_S}) {
    if (cfg == T_M && nmat == 4) continue;
    if (nmat < 4 && N % ((cfg == T_S ? 128 : 256) / nmat)) continue;
    const int bm = cfg == T_L ? 256 : cfg == T_M ? 192 : 128, bn = cfg == T_S && nmat < 4 ? 128 : 256;
    const double rate = cfg == T_L ? 5.2e6 : cfg == T_M ? 5.0e6 : (nmat == 4 ? 4.0e6 : 2.9e6);
    const double rounds = (double)((gemm_tiles(cfg, M, N, nmat) + MAX_WG - 1) / MAX_WG);
    const double c = rounds * (2.0 * bm * bn * (double)K / rate + (cfg == T_S ? 3.0 : 6.0));
    if (c < bc) {
      bc = c;
      best = cfg;
    }
  }
  return best;
}

template <class TL, int LB, int NMAT, class EP>
inline Launched launch_tile(const GemmArgs& g, const EP& ep, int64_t tiles, hipStream_t st) {
  const int grid = (int)std::min<int64_t>(tiles, MAX_WG);
  hipLaunchKernelGGL((k_gemm<TL, LB, NMAT, EP>), dim3(grid), dim3(NTHR), 0, st, g, ep);
  return {grid, TL::MB};
}
// Launches one product (A k-major, B in layout LB).
template <int LB, int NMAT, class EP>
inline Launched gemm(const GemmArgs& g, const EP& ep, hipStream_t st) {
  const int cfg = pick_tile(g.M, g.N, NMAT, (int64_t)g.K * g.nseg);
  const int64_t tiles = gemm_tiles(cfg, g.M, g.N, NMAT);
  if constexpr (NMAT == 4) {
    if (cfg == T_L) return launch_tile<TileL4, LB, NMAT>(g, ep, tiles, st);
    return launch_tile<TileS4, LB, NMAT>(g, ep, tiles, st);
  } else {
    if (cfg == T_L) return launch_tile<TileL, LB, NMAT>(g, ep, tiles, st);
    if (cfg == T_M) return launch_tile<TileM, LB, NMAT>(g, ep, tiles, st);
    return launch_tile<TileS, LB, NMAT>(g, ep, tiles, st);
  }
}
static_assert(MAX_WG == 256 && NW == 8, "sum_parts counts the waves of a launch");
inline GemmArgs product(const bf16* A, int lda, int a_rows, const bf16* B, int ldb, int b_rows, int M, int N, int K) {
  GemmArgs g{};
  g.A[0] = A; g.B[0] = B;
  g.lda = lda; g.ldb = ldb; g.a_rows = a_rows; g.b_rows = b_rows;
  g.K = K; g.nseg = 1; g.seg0_scale = 1.f;
  g.M = M; g.N = N;
  return g;
}

// ------------------------------------------------------------- weight terms
// W (+)= coef * sum over tokens A^T B for up to three weights in one launch
// (both operands [tokens][...]), each result element summed by one work-group
// over its tokens in order.  One weight alone is 64 tiles of 256 x 256 at the
// paper's state, a quarter of the chip, so the weights of a step share a
// launch: the paper unit's three are 192 tiles of 256 x 256, the MSE unit's
// two 256 tiles of 128 x 256.  A weight may have a second term: its tile is
// then updated twice, by the same work-group, one term after the other.
// nsplit > 1 cuts the tokens into that many runs whose sums go to separate
// [M][N] outputs (w + run * M * N; the caller adds them in run order).
struct WProb {
  const bf16* A[2];
  const bf16* B[2];
  int lda, ldb, M, N, nterm;
  float* w;        // FP32 [M][N]
  const float* from;  // the W added to (w itself, or the masters of the step before)
  bf16* op;        // operand copy of the result, nullable
  float coef;      // w = (add ? from : 0) + coef * sum
  int add;
};
struct WArgs {
  WProb p[3];
  int np, tokens, nsplit;
};

template <class TL>
__global__ __launch_bounds__(NTHR) void k_wgrad(WArgs a) {
  using MC = Machine<TL, MNMAJ, MNMAJ, 1>;
  __shared__ __attribute__((aligned(1024))) char sm[MC::LDS];
  MC mc;
  mc.init(sm);
  const int nks = (a.tokens + KS - 1) / KS;
  // a tile of the launch: weight p, run r of tokens (nk slices from k0 on), tile of the weight
  struct Pos {
    int p, r, im, in, k0, nk;
  };
  auto tiles_of = [&](int p) { return (a.p[p].M / TL::BM) * (a.p[p].N / TL::BN); };
  auto locate = [&](int t) {
    int p = 0;
    while (p + 1 < a.np && t >= tiles_of(p) * a.nsplit) t -= tiles_of(p++) * a.nsplit;
    const int n = tiles_of(p);
    Pos o;
    o.p = p;
    o.r = t / n;
    tile_at(t - o.r * n, a.p[p].M / TL::BM, a.p[p].N / TL::BN, o.im, o.in);
    o.k0 = __builtin_amdgcn_readfirstlane(o.r * nks / a.nsplit);
    o.nk = __builtin_amdgcn_readfirstlane((o.r + 1) * nks / a.nsplit) - o.k0;
    return o;
  };
  int total = 0, first, count;
  for (int p = 0; p < a.np; ++p) total += tiles_of(p) * a.nsplit;
  const int j0 = xcd_index(first, count, total), stride = (gridDim.x + 7 - (blockIdx.x & 7)) >> 3;
  if (j0 >= count) return;
  // the load cursor: tile, term, slice
  u32x4 ra, rb[MC::PB];
  int lt = j0, lterm = 0, lk = 0, ka = 0, kb = 0;
  Pos lp = locate(first + lt);
  auto sources = [&]() {
    const WProb& w = a.p[lp.p];
    ra = make_rs(w.A[lterm], (uint32_t)a.tokens * (uint32_t)w.lda * 2u);
    const u32x4 r = make_rs(w.B[lterm], (uint32_t)a.tokens * (uint32_t)w.ldb * 2u);
#pragma unroll
    for (int i = 0; i < MC::PB; ++i) rb[i] = r;
    ka = MC::kbytes(MNMAJ, w.lda);
    kb = MC::kbytes(MNMAJ, w.ldb);
    mc.tile(w.lda, w.ldb, lp.im * TL::BM, lp.in * TL::BN);
  };
  auto load_next = [&](int slot) {  // past the last slice: the last tile's first slices again, never used
    const int k = lp.k0 + lk;
    mc.load(ra, rb, k * ka, k * kb, slot);
    if (++lk == lp.nk) {
      lk = 0;
      if (++lterm == a.p[lp.p].nterm) {
        lterm = 0;
        if (lt + stride < count) {
          lt += stride;
          lp = locate(first + lt);
        }
      }
      sources();
    }
  };
  sources();
#pragma unroll
  for (int s = 0; s < NST - 1; ++s) load_next(s);
  wait_barrier<MC::PER*(NST - 2)>();
  mc.read(0, 0);
  int s = 0;
  const int l32 = threadIdx.x & 31, hf = (threadIdx.x >> 5) & 1;
  for (int t = j0; t < count; t += stride) {
    const Pos o = locate(first + t);
    const WProb& w = a.p[o.p];
    for (int term = 0; term < w.nterm; ++term) {
      mc.clear();
      for (int k = 0; k < o.nk; ++k) s = mc.slice(s, load_next);
      float* wr = w.w + (int64_t)o.r * w.M * w.N;
      bf16* op = term + 1 == w.nterm ? w.op : nullptr;
#pragma unroll
      for (int i = 0; i < MC::MB; ++i)
#pragma unroll
        for (int n = 0; n < MC::NB; ++n) {
          const int64_t at =
              (int64_t)(o.im * TL::BM + mc.wm + 32 * i + l32) * w.N + o.in * TL::BN + mc.wn + 32 * n + 16 * hf;
          float wv[16], nv[16];
          if (w.add) {
            load16((term == 0 ? w.from : wr) + at, wv);
          } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) wv[r] = 0.f;
          }
#pragma unroll
          for (int r = 0; r < 16; ++r) nv[r] = fmaf(w.coef, mc.acc[i][n][r], wv[r]);
          store16(wr + at, nv);
          if (op) {
            uint32_t pk[8];
            pack_each(pk, [&](int r) { return nv[r]; });
            *reinterpret_cast<u32x4*>(op + at) = (u32x4){pk[0], pk[1], pk[2], pk[3]};
            *reinterpret_cast<u32x4*>(op + at + 8) = (u32x4){pk[4], pk[5], pk[6], pk[7]};
          }
        }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// Adds a weight term to a launch.
inline void add_weight(WArgs& a, const bf16* A, int lda, const bf16* B, int ldb, int M, int N, float* w, bf16* op,
                       float coef, int add, const float* from = nullptr) {
  WProb& p = a.p[a.np++];
  p.A[0] = A; p.B[0] = B;
  p.lda = lda; p.ldb = ldb; p.M = M; p.N = N; p.nterm = 1;
  p.w = w; p.from = from ? from : w; p.op = op; p.coef = coef; p.add = add;
}
// Tiles by the rounds of the launch and the measured rate of a work-group
// (per CU, 256 x 256: 5.2 TFLOP/s, 128 x 256: 4.2, 128 x 128: 2.9).
struct WTile {
  int bm, bn;
  int64_t tiles;
};
inline WTile pick_wgrad(const WArgs& a) {
  struct {
    int bm, bn;
    double rate;
  } const kind[3] = {{256, 256, 5.2}, {128, 256, 4.2}, {128, 128, 2.9}};
  WTile best{128, 128, 0};
  double bc = 1e30;
  for (const auto& k : kind) {
    int64_t tiles = 0, longest = 1;
    bool fits = true;
    for (int p = 0; p < a.np; ++p) {
      fits = fits && a.p[p].M % k.bm == 0 && a.p[p].N % k.bn == 0;
      tiles += (int64_t)(a.p[p].M / k.bm) * (a.p[p].N / k.bn) * a.nsplit;
      longest = std::max<int64_t>(longest, a.p[p].nterm);
    }
    const double cost = (double)((tiles + MAX_WG - 1) / MAX_WG * longest) * k.bm * k.bn / k.rate;
    if (fits && cost < bc) {
      bc = cost;
      best = {k.bm, k.bn, tiles};
    }
  }
  return best;
}
inline void wgrad(WArgs a, hipStream_t st) {
  a.nsplit = std::max(1, std::min(a.nsplit, (a.tokens + KS - 1) / KS));
  const WTile t = pick_wgrad(a);
  const dim3 g((unsigned)std::min<int64_t>(t.tiles, MAX_WG)), nt(NTHR);
  if (t.bm == 256)
    hipLaunchKernelGGL(k_wgrad<TileL>, g, nt, 0, st, a);
  else if (t.bn == 256)
    hipLaunchKernelGGL(k_wgrad<TileH>, g, nt, 0, st, a);
  else
    hipLaunchKernelGGL(k_wgrad<TileS>, g, nt, 0, st, a);
}

}  // namespace bfg
}  // namespace ttt
