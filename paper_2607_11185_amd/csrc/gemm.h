// Shared GEMM of the libseg translation units (gfx950, bf16 MFMA):
//   C(m, n) = sum_k A(m, k) B(n, k)
// with each operand k-contiguous or row-major over K, read in place; one
// kernel (k_gemm) with one epilogue interface: a functor called by every
// thread with its accumulators and a Tile that says where they sit.
#pragma once

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace seg {
namespace gemm {

typedef int gemm_i32x4 __attribute__((ext_vector_type(4)));
typedef short gemm_v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) gemm_v4i16 gemm_lds_v4i16;
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// Where a wave's accumulators sit.  (wr, wc) is the wave tile's corner inside
// the block at (m0, n0).  Register r of acc[i][j] holds, in the lane with
// col = lane % 16 and grp = lane / 16,
//   row wr + 16 i + 4 grp + r, column wc + 16 j + col
// or, for an epilogue with kSwap (the products' operands swapped, so that a
// lane holds runs of a row),
//   row wr + 16 i + col, column wc + 16 j + 4 grp + r.
// lds: at least 16 KB that belong to the wave alone.  split: which part of K.
struct Tile {
  int m0, n0, M, N, wr, wc, col, grp, split;
  char *lds;
};

__device__ __forceinline__ unsigned pack2(float a, float b) {
  return (unsigned)f2bf_bits(a) | ((unsigned)f2bf_bits(b) << 16);
}

// Output of a product: 32 rows at a time go through the wave's LDS so that a
// lane ends with 8 consecutive columns of a row and stores (and, for the
// accumulating kinds, loads) them with 16-byte accesses, 8 lanes to a
// 128-byte (bf16) or 256-byte (fp32) piece of a row.  The reads of the next
// 32 rows are issued before the stores of the current ones.
//   ST    C = scale A B^T            (TO bf16 or fp32)
//   RESID C = R + scale A B^T        (bf16, a residual connection; R may be C)
//   ACC   C = first ? scale A B^T : C + scale A B^T  (fp32: gradients summed
//         over row chunks, in chunk order)
// vec: C (and R) rows start on 16-byte boundaries; otherwise, and in a ragged
// last column group, elements are handled one by one.
enum OutMode { ST, RESID, ACC };

template <class TO, OutMode MODE>
struct EpiOut {
  static constexpr bool kSwap = true;
  TO *c;
  long ldc;
  const unsigned short *r;
  long ldr;
  float scale;
  int vec, first;
  long split_stride;  // elements between the partial sums of the parts of K

  static EpiOut make(TO *c, long ldc, float scale = 1.f, const unsigned short *r = nullptr,
                     long ldr = 0, bool first = true, long split_stride = 0) {
    EpiOut e{c, ldc, r, ldr, scale, 0, first ? 1 : 0, split_stride};
    const bool cv = (reinterpret_cast<uintptr_t>(c) & 15) == 0 && ldc * sizeof(TO) % 16 == 0;
    const bool rv = MODE != RESID || ((reinterpret_cast<uintptr_t>(r) & 15) == 0 && ldr % 8 == 0);
    e.vec = cv && rv ? 1 : 0;
    return e;
  }

  struct Pre {
    u16x8 r;
    f32x4 a, b;
  };
  __device__ __forceinline__ Pre load(const TO *cc, int m, int n, const Tile &t) const {
    Pre p{};
    if (m >= t.M || n >= t.N) return p;
    const bool whole = vec && n + 8 <= t.N;
    if constexpr (MODE == RESID) {
      const unsigned short *s = r + (long)m * ldr + n;
      if (whole) p.r = *reinterpret_cast<const u16x8 *>(s);
      else
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (n + j < t.N) p.r[j] = s[j];
    } else if constexpr (MODE == ACC) {
      if (first) return p;
      const float *s = reinterpret_cast<const float *>(cc) + (long)m * ldc + n;
      if (whole) {
        p.a = *reinterpret_cast<const f32x4 *>(s);
        p.b = *reinterpret_cast<const f32x4 *>(s + 4);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (n + j < t.N) p.a[j] = s[j];
          if (n + 4 + j < t.N) p.b[j] = s[4 + j];
        }
      }
    }
    return p;
  }

  template <int NI, int NJ>
  __device__ __forceinline__ void operator()(const f32x4 (&acc)[NI][NJ], const Tile &t) const {
    static_assert(NJ == 4, "64-column wave tiles");
    constexpr int TM = NI / 2;
    const int lane = t.grp * 16 + t.col, lr = lane >> 3, q = lane & 7;
    const int m_base = t.m0 + t.wr + lr, n = t.n0 + t.wc + q * 8;
    TO *const cc = c + (long)t.split * split_stride;
    f32x4 *w = reinterpret_cast<f32x4 *>(t.lds);
    Pre pre[2][4];
    if constexpr (MODE != ST) {
#pragma unroll
      for (int p = 0; p < 4; ++p) pre[0][p] = load(cc, m_base + p * 8, n, t);
    }
#pragma unroll
    for (int bm = 0; bm < TM; ++bm) {
      if constexpr (MODE != ST) {
        if (bm + 1 < TM) {
#pragma unroll
          for (int p = 0; p < 4; ++p)
            pre[(bm + 1) & 1][p] = load(cc, m_base + (bm + 1) * 32 + p * 8, n, t);
        }
      }
      // [32 rows][16 chunks of 4 columns], chunk c of row m in slot c ^ (m & 15)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          w[(i * 16 + t.col) * 16 + ((j * 4 + t.grp) ^ t.col)] = acc[bm * 2 + i][j] * scale;
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int row = p * 8 + lr, m = m_base + bm * 32 + p * 8;
        f32x4 a = w[row * 16 + ((2 * q) ^ (row & 15))];
        f32x4 b = w[row * 16 + ((2 * q + 1) ^ (row & 15))];
        if (m >= t.M || n >= t.N) continue;
        const Pre &pr = pre[bm & 1][p];
        if constexpr (MODE == RESID) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            a[j] += bf_bits2f(pr.r[j]);
            b[j] += bf_bits2f(pr.r[4 + j]);
          }
        } else if constexpr (MODE == ACC) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            a[j] += pr.a[j];
            b[j] += pr.b[j];
          }
        }
        TO *d = cc + (long)m * ldc + n;
        if (vec && n + 8 <= t.N) {
          if constexpr (sizeof(TO) == 2) {
            typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
            *reinterpret_cast<u32x4 *>(d) =
                u32x4{pack2(a[0], a[1]), pack2(a[2], a[3]), pack2(b[0], b[1]), pack2(b[2], b[3])};
          } else {
            *reinterpret_cast<f32x4 *>(d) = a;
            *reinterpret_cast<f32x4 *>(d + 4) = b;
          }
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            if (n + j < t.N) store_val(d, j, a[j]);
            if (n + 4 + j < t.N) store_val(d, 4 + j, b[j]);
          }
        }
      }
      __builtin_amdgcn_wave_barrier();
    }
  }
};

// ------------------------------------------------------------------ kernel
//
// One block of 8 waves computes 64 TM x 256, each wave 32 TM x 64 (TM = 4:
// 128 accumulator registers).  The schedule keeps one wave of every SIMD on
// products all the time: the waves form two groups of four (one wave of each
// group per SIMD) that run half a step apart.  In a phase one group issues the
// 16 TM products of a K step of 64 (1,024 cycles of its SIMD's matrix core at
// TM = 4) while the other reads its 4 TM + 8 fragments of the next step from
// LDS and issues its share of the direct global->LDS loads; a barrier ends the
// phase and the groups change places.  Group 0 loads A (two ring slots, two
// phases ahead of use), group 1 loads B (three slots, three phases ahead): 160
// KB of LDS at TM = 4.
//
// What bounds it is power: at 8192^3 with random operands the matrix cores are
// 84% busy at 1.65 GHz (the card's 2.4 GHz needs less switching).  Hence
// 16x16x32 products (they move half the accumulator bits of 32x32x16 ones: N
// operands 1,360 -> 1,500 TFLOP/s) and an order in which one operand changes
// from product to product.  Measured rates at 8192^3, TFLOP/s, both operands
// k-contiguous / one / none: one-barrier-per-step kernels with 32x32x16
// products 1,160-1,240; this schedule with steps of 32 (64-byte row pieces,
// half a cache line) 1,240 / 1,230 / 1,150; steps of 64 1,370 / 1,360 / 1,330;
// 16x16x32 1,500 / 1,460 / 1,310; loads issued between the fragment reads
// instead of after them 1,470 / 1,470 / 1,450 (kept).  TM = 2: 1,190 / 1,130 /
// 1,150.
//
// LDS tiles.  N: [rows][64 k], 128 B per row, 16-byte chunk c of row r in slot
// c ^ ((r >> 1) & 7): a 16-lane fragment read of 16 rows hits 16 distinct
// 16-byte slots of the 64 banks.  T: [64 k][columns], chunk c of row r in slot
// c ^ t_swizzle(r): a 32-lane transpose read (rows 0-3 and 8-11 of a slice x
// 32 bytes) hits 16 distinct slots.  SQ_LDS_BANK_CONFLICT reads 0 for both.
constexpr int BN = 256, BK = 64, THREADS = 512, SLOTS_A = 2, SLOTS_B = 3;
constexpr int bm_of(int TM) { return 64 * TM; }

// Raw buffer descriptor over [base, base + bytes): loads at or past the end
// return zeros.
__device__ __forceinline__ gemm_i32x4 gemm_desc(const void *base, long bytes) {
  const unsigned long p = (unsigned long)base;
  const long lim = bytes < 0x7fffffffL ? bytes : 0x7fffffffL;
  return gemm_i32x4{(int)(unsigned)p, (int)((unsigned)(p >> 32) & 0xffffu), (int)lim, 0x00020000};
}

// 64 lanes x 16 bytes from rs (byte offset voff per lane) to LDS at byte
// address dst (scalar).  Written as an instruction so that the compiler does
// not wait for it before LDS reads of other slots; it has no register
// result, and the phases below wait for it by count before its slot is read.
__device__ __forceinline__ void dma16(unsigned dst, int voff, gemm_i32x4 rs) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %1, %2, 0 offen lds"
      :
      : "s"(dst), "v"(voff), "s"(rs)
      : "memory", "m0");
#endif
}

// chunk swizzle of k row r of a T tile
__device__ __forceinline__ int t_swizzle(int r) { return 4 * (r & 3) ^ 2 * ((r >> 3) & 1); }

// The direct loads of one operand (R rows of it per block): R / 32 loads of
// 1 KB per step by each of the four waves (w = 0..3) of the group that loads
// it.  prep() sets up a step, load() issues its j-th load.
struct Loader {
  const unsigned short *x;  // T: column c0 of row 0
  long ld;
  int width;                // T: columns of the last row, whole 16-byte chunks
  gemm_i32x4 rs;
  int voff[2], kchunk, stride, add;

  template <bool T, int R>
  __device__ __forceinline__ void init(const unsigned short *X, long ld_, int row0, int rows, int w,
                                       int lane) {
    ld = ld_;
    if constexpr (T) {
      constexpr int CPR = R / 8, RPL = 64 / CPR;  // chunks per row, rows per load
      x = X + row0;
      // the last row stops at the operand's last row rounded up to a 16-byte
      // chunk: ld is a multiple of 8 and every k row holds ld elements, so
      // that end stays inside the matrix
      width = (rows - row0 + 7) & ~7;
      stride = (int)(4 * RPL * ld * 2);
#pragma unroll
      for (int j = 0; j < 2; ++j) {  // load j: k rows RPL (w + 4 j) ..; the swizzle repeats with j + 2
        const int r = RPL * (w + 4 * j) + lane / CPR;
        voff[j] = (int)(r * ld * 2) + ((lane % CPR) ^ t_swizzle(r)) * 16;
      }
    } else {
      // the descriptor covers the block's own rows only (< 2^30 bytes)
      rs = gemm_desc(X + (long)row0 * ld, (long)(rows - row0 < R ? rows - row0 : R) * ld * 2);
      const int r = w * 8 + (lane >> 3);  // load j: rows 8 (w + 4 j) .. + 7
      kchunk = (lane & 7) ^ ((r >> 1) & 7);
      stride = (int)(32 * ld * 2);
      voff[0] = (int)(r * ld * 2) + kchunk * 16;
      voff[1] = voff[0] + stride;
    }
  }
  // step at k0 of K: what lies at or past K (the whole step where k0 >= K)
  // reads as zero
  template <bool T>
  __device__ __forceinline__ void prep(int k0, int K) {
    if constexpr (T) {
      const int rows = K - k0 < BK ? K - k0 : BK;
      rs = gemm_desc(x + (long)k0 * ld, rows > 0 ? ((long)(rows - 1) * ld + width) * 2 : 0);
      add = 0;
    } else {
      add = k0 + kchunk * 8 < K ? k0 * 2 : 0x40000000;
    }
  }
  __device__ __forceinline__ void load(unsigned dst, int j, int w) const {
    dma16(dst + (w + 4 * j) * 1024, voff[j & 1] + add + (j >> 1) * 2 * stride, rs);
  }
};

// Fragment reads of NB 16-row blocks from the tile corner `c0` (rows of the
// operand): lane l holds row l % 16, k = 8 (l / 16) .. + 7 of 32-wide slice kk.
template <bool T, int R, int NB>
struct Frag;

template <int R, int NB>
struct Frag<false, R, NB> {
  int off[2];
  __device__ __forceinline__ void init(int ring, int c0, int lane) {
    const int col = lane & 15, grp = lane >> 4;
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
      off[kk] = ring + (c0 + col) * 128 + (((4 * kk + grp) ^ (col >> 1)) << 4);
  }
  __device__ __forceinline__ bf16x8 read(const char *lds, int slot, int kk, int i) const {
    return *reinterpret_cast<const bf16x8 *>(lds + (off[kk] + slot) + i * 2048);
  }
};

template <int R, int NB>
struct Frag<true, R, NB> {
  static constexpr int ROW = R * 2;  // bytes of one k row
  int off[NB];
  __device__ __forceinline__ void init(int ring, int c0, int lane) {
    const int l16 = lane & 15, r = 8 * (lane >> 4) + (l16 >> 2);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int c = c0 + 16 * i + 4 * (l16 & 3);
      off[i] = ring + r * ROW + (((c >> 3) ^ t_swizzle(r)) << 4) + (c & 7) * 2;
    }
  }
  __device__ __forceinline__ bf16x8 read(const char *lds, int slot, int kk, int i) const {
    const char *p = lds + (off[i] + slot) + kk * 32 * ROW;
    const gemm_v4i16 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((gemm_lds_v4i16 *)p);
    const gemm_v4i16 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((gemm_lds_v4i16 *)(p + 4 * ROW));
    const bf16x4 a4 = __builtin_bit_cast(bf16x4, a), b4 = __builtin_bit_cast(bf16x4, b);
    bf16x8 r;
    r[0] = a4[0]; r[1] = a4[1]; r[2] = a4[2]; r[3] = a4[3];
    r[4] = b4[0]; r[5] = b4[1]; r[6] = b4[2]; r[7] = b4[3];
    return r;
  }
};

// Tile order: a 1-D grid of 8 * ceil(T / 8) blocks for T tiles.  Block b runs
// on XCD b % 8; XCD x takes the contiguous tile range [x*C, (x+1)*C) so its
// concurrent blocks share an L2, and tiles are ordered in groups of 8 M-tiles
// (column by column inside a group) so those blocks reuse A and B rows.
__device__ __forceinline__ int xcd_index(int total) {
  const int per = (total + 7) / 8;
  return (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
}

__device__ __forceinline__ void tile_of(int idx, int nM, int nN, int &mt, int &nt) {
  const int G = 8;
  const int group = idx / (G * nN);
  const int first = group * G;
  const int gs = nM - first < G ? nM - first : G;
  const int in = idx - group * G * nN;
  mt = first + in % gs;
  nt = in / gs;
}

// NP problems run by one launch (their tiles in sequence, so a short last
// wave of one is filled by the next); each sums NS products over their own K:
//   C_p = sum_s A_ps B_ps^T
// lda, ldb multiples of 8 (and at least the operand's width); N operands need
// K a multiple of 8; 256 * ld * 2 < 2^30 (N), 64 * ld * 2 < 2^31 (T).  The
// steps of 64 of the K ranges, in order, may be cut into `splits` parts of
// `part` steps, each a set of tiles of its own: the epilogue then gets partial
// sums.
template <class Epi, int NP, int NS>
struct Problems {
  const unsigned short *A[NP][NS], *B[NP][NS];
  long lda[NP][NS], ldb[NP][NS];
  int K[NS];
  int M[NP], N[NP];
  Epi ep[NP];
  int start[NP + 1];  // first tile of each problem; start[NP] = all tiles
  int splits, part;
};

#define GEMM_FENCE() asm volatile("" ::: "memory")

// Grid: 8 * ceil(tiles * splits / 8) x 512.
template <bool TA, bool TB, int TM, class Epi, int NP, int NS>
__global__ void __launch_bounds__(THREADS, 1) k_gemm(const Problems<Epi, NP, NS> g) {
  constexpr int BM = bm_of(TM), SA = BM * BK * 2, SB = BN * BK * 2;  // bytes of a slot
  constexpr int LDS_B = SA * SLOTS_A;                                // the B ring follows the A ring
  __shared__ __attribute__((aligned(1024))) char lds[LDS_B + SB * SLOTS_B];
  int idx = xcd_index(g.start[NP] * g.splits);
  if (idx >= g.start[NP] * g.splits) return;
  const int split = idx / g.start[NP];
  idx -= split * g.start[NP];
  // the problem's fields by unrolled selects (no dynamic indexing of the
  // kernel argument, which would copy it to scratch)
  int M = g.M[0], N = g.N[0], first = 0;
  const unsigned short *pA[NS], *pB[NS];
  long la[NS], lb[NS];
  Epi ep = g.ep[0];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    pA[s] = g.A[0][s];
    pB[s] = g.B[0][s];
    la[s] = g.lda[0][s];
    lb[s] = g.ldb[0][s];
  }
#pragma unroll
  for (int q = 1; q < NP; ++q)
    if (idx >= g.start[q]) {
      M = g.M[q];
      N = g.N[q];
      first = g.start[q];
      ep = g.ep[q];
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        pA[s] = g.A[q][s];
        pB[s] = g.B[q][s];
        la[s] = g.lda[q][s];
        lb[s] = g.ldb[q][s];
      }
    }
  int mt, nt;
  tile_of(idx - first, (M + BM - 1) / BM, (N + BN - 1) / BN, mt, nt);
  const int m0 = mt * BM, n0 = nt * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int grp = wave >> 2;  // waves w and w + 4 share a SIMD
  const int wm = grp, wn = wave & 3, w4 = wave & 3;

  Loader ldr;
  auto open = [&](int s) __attribute__((always_inline)) {  // the group's operand of product s
    if (grp == 0) ldr.init<TA, BM>(pA[s], la[s], m0, M, w4, lane);
    else ldr.init<TB, BN>(pB[s], lb[s], n0, N, w4, lane);
  };
  Frag<TA, BM, 2 * TM> fA;
  Frag<TB, BN, 4> fB;
  fA.init(0, wm * 32 * TM, lane);
  fB.init(LDS_B, wn * 64, lane);

  f32x4 acc[2 * TM][4];
#pragma unroll
  for (int i = 0; i < 2 * TM; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{};

  // the part's first step and its number of steps
  int nk = 0, seg = 0, k_next = split * g.part * BK, K_seg = g.K[0];
#pragma unroll
  for (int s = 0; s < NS; ++s) nk += (g.K[s] + BK - 1) / BK;
  nk = min(g.part, nk - split * g.part);
#pragma unroll
  for (int s = 0; s + 1 < NS; ++s)
    if (seg == s && k_next >= g.K[s]) {
      k_next -= (g.K[s] + BK - 1) / BK * BK;
      K_seg = g.K[s + 1];
      seg = s + 1;
    }
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s == seg) open(s);
  const unsigned base = (unsigned)(unsigned long)(__attribute__((address_space(3))) char *)lds;
  // sets up the group's next step of loads
  auto prep = [&]() __attribute__((always_inline)) {
    if constexpr (NS > 1) {
      if (k_next >= K_seg && seg + 1 < NS) {
        ++seg;
        k_next = 0;
#pragma unroll
        for (int s = 1; s < NS; ++s)
          if (s == seg) {
            K_seg = g.K[s];
            open(s);
          }
      }
    }
    if (TA == TB || grp == 0) ldr.prep<TA>(k_next, K_seg);
    else ldr.prep<TB>(k_next, K_seg);
    if constexpr (NS > 1) {
      // carried through the change of products in vector registers
#pragma unroll
      for (int i = 0; i < 4; ++i) ldr.rs[i] = __builtin_amdgcn_readfirstlane(ldr.rs[i]);
    }
    k_next += BK;
  };
  constexpr int LA = BM / 32, LB = BN / 32;  // loads per wave of an A and of a B step
  const unsigned ring = base + (grp == 0 ? 0 : LDS_B);
  auto load = [&](int slot, int j) __attribute__((always_inline)) {
    if (LA == LB || j < LA || grp == 1) ldr.load(ring + slot, j, w4);
  };
  prep();
#pragma unroll
  for (int j = 0; j < LB; ++j) load(0, j);
  if (grp == 0) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  } else {
    prep();
#pragma unroll
    for (int j = 0; j < LB; ++j) load(SB, j);
    if (nk > 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LB) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  __builtin_amdgcn_s_barrier();
  GEMM_FENCE();
  if (grp == 1 && nk > 0) __builtin_amdgcn_s_barrier();  // half a step behind group 0
  GEMM_FENCE();

  // Both groups pass the same number of barriers (group 1 one more before the
  // loop and none after its last products).  Before the barrier that opens
  // group 0's reads of step t + 1, group 0 has waited for its A loads of that
  // step (issued with step t) and group 1 for its B loads of it (issued with
  // step t - 1; those of t + 2 stay in flight).  A slot is overwritten by
  // loads issued behind a barrier that both groups reach with their reads of
  // it complete.  One loop body for every slot: unrolled with an exit in each
  // copy, the accumulators went through memory at the exits.
  int slot_b = 0, slot_b2 = 2 * SB;  // of steps t and t + 2
#pragma unroll 1
  for (int t = 0; t < nk; ++t) {
    const int slot_a = (t & 1) * SA;
    const int slot_n = grp == 0 ? SA - slot_a : slot_b2;
    bf16x8 a[2][2 * TM], b[2][4];
    // the loads (of A for step t + 1, of B for t + 2; past the end they read
    // zeros into a free slot) go out between the fragment reads, so that the
    // two queues work side by side
    prep();
    constexpr int NR = 2 * TM + 4, PER = LB / 2;  // reads and loads per slice
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
      for (int f = 0; f < NR; ++f) {
#pragma unroll
        for (int j = f * PER / NR; j < PER; ++j)
          if (j * NR / PER == f) load(slot_n, kk * PER + j);
        if (f < 4) b[kk][f] = fB.read(lds, slot_b, kk, f);
        else a[kk][f - 4] = fA.read(lds, slot_a, kk, f - 4);
      }
    }
    if (grp == 0)
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    else if (t + 2 < nk)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(LB) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    GEMM_FENCE();
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 2 * TM; ++i)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int j = (i & 1) ? 3 - jj : jj;  // one operand changes at a time
          acc[i][j] = Epi::kSwap ? mfma16(b[kk][j], a[kk][i], acc[i][j])
                                 : mfma16(a[kk][i], b[kk][j], acc[i][j]);
        }
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
    slot_b = slot_b == 2 * SB ? 0 : slot_b + SB;
    slot_b2 = slot_b2 == 2 * SB ? 0 : slot_b2 + SB;
    if (grp == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (grp == 0 || t + 1 < nk) __builtin_amdgcn_s_barrier();
    GEMM_FENCE();
  }
  // every load has landed and every slot has been read: a wave may use its
  // own eighth of the LDS in the epilogue
  ep(acc, Tile{m0, n0, M, N, wm * 32 * TM, wn * 64, lane & 15, lane >> 4, split,
               lds + wave * (int)(sizeof(lds) / 8)});
}

inline long tiles_of(long M, long N, int TM) {
  return M <= 0 || N <= 0 ? 0 : ((M + bm_of(TM) - 1) / bm_of(TM)) * ((N + BN - 1) / BN);
}

template <bool TA, bool TB, int TM, class Epi, int NP, int NS>
inline void launch_tm(Problems<Epi, NP, NS> &g, hipStream_t st) {
  g.start[0] = 0;
  for (int q = 0; q < NP; ++q) g.start[q + 1] = g.start[q] + (int)tiles_of(g.M[q], g.N[q], TM);
  const long total = (long)g.start[NP] * g.splits;
  if (total == 0) return;
  k_gemm<TA, TB, TM, Epi, NP, NS><<<(unsigned)((total + 7) / 8 * 8), THREADS, 0, st>>>(g);
  SEG_LAUNCH_CHECK();
}

constexpr int NUM_CU = 256;

// Sums the parts of split products and finishes them as their epilogues say:
// 8 columns of a row a thread, parts in order.  Rows of N elements (a multiple
// of 8), problem after problem, in each part.
template <class TO, OutMode MODE, int NP>
struct Finish {
  EpiOut<TO, MODE> ep[NP];
  int n8[NP];         // chunks of a row
  long end[NP];       // chunks, running over the problems
  const float *part;
  int parts;
};

template <class TO, OutMode MODE, int NP>
__global__ void __launch_bounds__(256) k_finish(const Finish<TO, MODE, NP> f) {
  const long total = f.end[NP - 1];
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
    EpiOut<TO, MODE> e = f.ep[0];
    int n8 = f.n8[0];
    long first = 0;
#pragma unroll
    for (int q = 1; q < NP; ++q)
      if (i >= f.end[q - 1]) {
        e = f.ep[q];
        n8 = f.n8[q];
        first = f.end[q - 1];
      }
    const long m = (i - first) / n8, n = (i - first - m * n8) * 8;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int k = 0; k < f.parts; ++k) {
      const f32x4 *p = reinterpret_cast<const f32x4 *>(f.part + (k * total + i) * 8);
      const f32x4 a = p[0], b = p[1];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[j] += a[j];
        v[4 + j] += b[j];
      }
    }
    TO *d = e.c + m * e.ldc + n;
    const unsigned short *r = MODE == RESID ? e.r + m * e.ldr + n : nullptr;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] *= e.scale;
      if constexpr (MODE == RESID) v[j] += bf_bits2f(r[j]);
      if constexpr (MODE == ACC)
        if (!e.first) v[j] += (float)d[j];
    }
    if constexpr (sizeof(TO) == 2) {
      if (e.vec) {
        u16x8 o;
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = f2bf_bits(v[j]);
        *reinterpret_cast<u16x8 *>(d) = o;
        continue;
      }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) store_val(d, j, v[j]);
  }
}

// Workspace for partial sums.
struct Scratch {
  float *p;
  long elems;
};

// How a group of products is launched: rows of a tile and parts of K, by the
// time that each choice is expected to take: whole waves of blocks over the
// chip (one block per CU), a step of 64 at 1.5 us (the rate of the full chip;
// a 128-row tile takes 0.62 of it: 1,190 against 1,470 TFLOP/s at 8192^3) and
// 4 us to start and end a block; the partial sums written and read at 4 TB/s
// and a launch to finish them.  So 128-row tiles serve grids whose last wave of
// 256-row ones would be nearly empty, and long sums over few tiles are cut.
// Measured: 1,024 x 2,048 over K = 32,000 (32 tiles) 783 us in one part, 105 +
// 15 us in eight.
struct Choice {
  int tm, parts, part;  // part: steps of 64
};

inline Choice choose(long t4, long t2, long steps, double elems, long scratch) {
  Choice best{4, 1, (int)steps};
  double best_us = 0;
  for (int s = 1; s <= 16; ++s) {
    const long per = (steps + s - 1) / s;
    if (s > 1 && (per < 8 || s * elems > (double)scratch || (s - 1) * per >= steps)) continue;
    for (int tm = 4; tm >= 2; tm -= 2) {
      const double waves = (double)(((tm == 4 ? t4 : t2) * s + NUM_CU - 1) / NUM_CU);
      const double us = waves * ((tm == 4 ? 1.5 : 0.93) * per + 4) + (s > 1 ? s * elems / 5e5 + 5 : 0);
      if ((s == 1 && tm == 4) || us < best_us) {
        best = Choice{tm, s, (int)per};
        best_us = us;
      }
    }
  }
  return best;
}

// The choice for a group of np products (rows M, or `rows` where not 0, and
// columns N) that each sum over the ns ranges K.
inline Choice choose_group(int np, const int *M, const int *N, int ns, const int *K, long scratch,
                           long rows) {
  long t4 = 0, t2 = 0, steps = 0;
  double elems = 0;
  bool whole = true;  // rows of whole 8-element chunks
  for (int q = 0; q < np; ++q) {
    const long m = rows ? rows : M[q];
    t4 += tiles_of(m, N[q], 4);
    t2 += tiles_of(m, N[q], 2);
    elems += (double)m * N[q];
    whole = whole && N[q] % 8 == 0;
  }
  for (int s = 0; s < ns; ++s) steps += (K[s] + BK - 1) / BK;
  return choose(t4, t2, steps, elems, whole ? scratch : 0);
}

template <class Epi, int NP, int NS>
inline Choice choose_for(const Problems<Epi, NP, NS> &g, long scratch, long rows = 0) {
  return choose_group(NP, g.M, g.N, NS, g.K, scratch, rows);
}

// All products of the group with one launch.
template <bool TA, bool TB, class Epi, int NP, int NS>
inline void launch(Problems<Epi, NP, NS> g, hipStream_t st) {
  const Choice c = choose_for(g, 0);
  g.splits = 1;
  g.part = c.part;
  if (c.tm == 2) launch_tm<TA, TB, 2>(g, st);
  else launch_tm<TA, TB, 4>(g, st);
}

// The same, cut into parts of K where that is faster and `sc` holds them.
// rows > 0: the parts are chosen as for products of that many rows (a whole
// batch whose chunks of rows are multiplied one by one: a row's sum must not
// depend on the chunking); M must not be larger.
template <bool TA, bool TB, class TO, OutMode MODE, int NP, int NS>
inline void launch(const Problems<EpiOut<TO, MODE>, NP, NS> &g, const Scratch &sc, long rows,
                   hipStream_t st) {
  const Choice c = choose_for(g, sc.elems, rows);
  if (c.parts == 1) {
    launch<TA, TB>(g, st);
    return;
  }
  typedef EpiOut<float, ST> Part;
  Problems<Part, NP, NS> h{};
  Finish<TO, MODE, NP> f{};
  long total = 0;
  for (int q = 0; q < NP; ++q) total += (long)g.M[q] * g.N[q];
  long at = 0;
  for (int q = 0; q < NP; ++q) {
    for (int s = 0; s < NS; ++s) {
      h.A[q][s] = g.A[q][s];
      h.B[q][s] = g.B[q][s];
      h.lda[q][s] = g.lda[q][s];
      h.ldb[q][s] = g.ldb[q][s];
    }
    h.M[q] = g.M[q];
    h.N[q] = g.N[q];
    h.ep[q] = Part::make(sc.p + at, g.N[q], 1.f, nullptr, 0, true, total);
    at += (long)g.M[q] * g.N[q];
    f.ep[q] = g.ep[q];
    f.n8[q] = g.N[q] / 8;
    f.end[q] = at / 8;
  }
  for (int s = 0; s < NS; ++s) h.K[s] = g.K[s];
  h.splits = c.parts;
  h.part = c.part;
  if (c.tm == 2) launch_tm<TA, TB, 2>(h, st);
  else launch_tm<TA, TB, 4>(h, st);
  f.part = sc.p;
  f.parts = c.parts;
  k_finish<TO, MODE, NP><<<(unsigned)std::min<long>(8192, (total / 8 + 255) / 256), 256, 0, st>>>(f);
  SEG_LAUNCH_CHECK();
}

// One product.
template <bool TA, bool TB, class Epi>
inline Problems<Epi, 1, 1> one(const unsigned short *A, long lda, const unsigned short *B, long ldb,
                               int M, int N, int K, const Epi &ep) {
  return Problems<Epi, 1, 1>{{{A}}, {{B}}, {{lda}}, {{ldb}}, {K}, {M}, {N}, {ep}, {}, 1, 0};
}
template <bool TA, bool TB, class Epi>
inline void launch_one(const unsigned short *A, long lda, const unsigned short *B, long ldb, int M,
                       int N, int K, const Epi &ep, hipStream_t st) {
  launch<TA, TB>(one<TA, TB>(A, lda, B, ldb, M, N, K, ep), st);
}
template <bool TA, bool TB, class Epi>
inline void launch_one(const unsigned short *A, long lda, const unsigned short *B, long ldb, int M,
                       int N, int K, const Epi &ep, const Scratch &sc, long rows, hipStream_t st) {
  launch<TA, TB>(one<TA, TB>(A, lda, B, ldb, M, N, K, ep), sc, rows, st);
}

}  // namespace gemm
}  // namespace seg
