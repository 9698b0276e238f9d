// Masked GQA attention over packed VCS segments, forward and backward
// (the policy-update attention of Sec. 3.3 training items), bf16 MFMA on gfx950.
//
// Every segment is an independent attention unit.  A query row sees the keys of
// its segment that are not after it, except screenshot tokens more than W-1
// turns older than its own turn.  The layout's tile map lists, per 128-row
// q-tile, the k-tiles that hold at least one visible pair (CSR) and marks them
// FULL (every pair visible: no predicate) or PARTIAL (per-element predicate).
//
// MFMA v_mfma_f32_16x16x32_bf16 lane layout used throughout (lane l, c = l%16,
// g = l/16):  A[i][k]: i = c, k = 8g + 0..7;  B[k][j]: j = c, k = 8g + 0..7;
// D[i][j] (4 regs r): j = c, i = 4g + r.
// This shape moves half the accumulator bits of 32x32x16 products: on the
// benchmark batch the clock under load rose from 1.82 / 1.81 / 1.97 to 2.03 /
// 2.02 / 2.21 GHz (forward, dQ, dK/dV) and the kernels took 132.5 -> 128.5,
// 179.2 -> 168.5 and 265.5 -> 257.0 ms.
// Products that contract over 32 rows held in the accumulators of two 16-row
// blocks take rows {4g..4g+3, 16+4g..16+4g+3} as a lane's eight k (any order
// serves as long as both operands use it); their other operand comes from LDS
// through transpose reads in the same row order.
#include <climits>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "common.h"

namespace seg {
namespace {

constexpr int TQ = 128;  // tile edge
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

struct TileRows {
  int start, len, qbase, i, row0, nrows;  // row0 is segment-relative
};

__device__ __forceinline__ TileRows tile_rows(const int32_t *seg_info, const int32_t *tile_seg,
                                              int g) {
  TileRows t;
  const int s = tile_seg[g];
  const int32_t *si = seg_info + (long)s * SEG_INFO_FIELDS;
  t.start = si[SEG_INFO_START];
  t.len = si[SEG_INFO_LEN];
  t.qbase = si[SEG_INFO_QTILE_BASE];
  t.i = g - t.qbase;
  t.row0 = t.i * TQ;
  t.nrows = min(TQ, t.len - t.row0);
  return t;
}

__device__ __forceinline__ int key_expiry(int meta, int W) {
  return ((meta & 3) == SEG_KIND_IMAGE) ? (meta >> 2) + W : INT_MAX;
}

// The window test of a key's turn/kind word (turn << 2 | kind) in one
// unsigned compare: with the kind bits xored with IMAGE and rotated to the
// top, an image key reads as its turn tau and any other kind as >= 2^30.  A
// query of turn t sees an image key iff t < tau + W, i.e. iff the rotated
// word is >= max(t - W + 1, 0).
__device__ __forceinline__ unsigned window_word(int meta) {
  return __builtin_rotateright32((unsigned)meta ^ SEG_KIND_IMAGE, 2);
}
__device__ __forceinline__ unsigned window_floor(int qstep, int W) {
  return (unsigned)max(qstep - W + 1, 0);
}

__device__ __forceinline__ bf16x8 lds8(const unsigned short *p) {
  return *reinterpret_cast<const bf16x8 *>(p);
}

// a lane's rows of two 16-row accumulator blocks as one operand fragment
__device__ __forceinline__ bf16x8 pack8(const f32x4 &lo, const f32x4 &hi) {
  bf16x8 r;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    r[j] = (__bf16)lo[j];
    r[4 + j] = (__bf16)hi[j];
  }
  return r;
}

// a row's value summed or maximised over the four lanes that share it
__device__ __forceinline__ float row_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  return x + __shfl_xor(x, 32, 64);
}
__device__ __forceinline__ float row_max(float x) {
  x = fmaxf(x, __shfl_xor(x, 16, 64));
  return fmaxf(x, __shfl_xor(x, 32, 64));
}

__device__ __forceinline__ u16x8 load8_bf(const unsigned short *p) {
  return *reinterpret_cast<const u16x8 *>(p);
}
__device__ __forceinline__ u16x8 load8_bf(const float *p) {
  const f32x4 a = *reinterpret_cast<const f32x4 *>(p);
  const f32x4 b = *reinterpret_cast<const f32x4 *>(p + 4);
  u16x8 r;
  r[0] = f2bf_bits(a[0]); r[1] = f2bf_bits(a[1]); r[2] = f2bf_bits(a[2]); r[3] = f2bf_bits(a[3]);
  r[4] = f2bf_bits(b[0]); r[5] = f2bf_bits(b[1]); r[6] = f2bf_bits(b[2]); r[7] = f2bf_bits(b[3]);
  return r;
}

// ------------------------------------------------------------- prep kernels

// bf16 copies of a call's fp32 tensors, all in one launch (a launch of its own
// for each of seven tensors was a fifth of a small call's time), 8 elements a
// thread (every size is a multiple of d; 16-byte loads need only the 4-byte
// alignment a float has); and zeros in `zero`.
struct ToBf16 {
  const float *x[4];
  unsigned short *y[4];
  long end[4];  // in 8-element chunks, running over the tensors
};
__global__ void __launch_bounds__(256) k_f32_to_bf16(const ToBf16 t, unsigned *__restrict__ zero,
                                                     long nzero) {
  const long at = (long)blockIdx.x * 256 + threadIdx.x, step = (long)gridDim.x * 256;
  for (long i = at; i < nzero; i += step) zero[i] = 0;
  for (long i = at; i < t.end[3]; i += step) {
    const float *x = t.x[0];
    unsigned short *y = t.y[0];
    long first = 0;
#pragma unroll
    for (int k = 1; k < 4; ++k)
      if (i >= t.end[k - 1]) {
        x = t.x[k];
        y = t.y[k];
        first = t.end[k - 1];
      }
    *reinterpret_cast<u16x8 *>(y + (i - first) * 8) = load8_bf(x + (i - first) * 8);
  }
}

// Delta[h][row] = sum_d dO[row][h][d] * O[row][h][d]  (D/8 lanes per (row, head)),
// stored negated (the backward kernels start their dP accumulators from
// -Delta, so dP - Delta costs no instruction), and the row's log-sum-exp in
// log2 units for the backward kernels.
template <class TI, int D>
__global__ void __launch_bounds__(256) k_delta(const TI *__restrict__ o, const TI *__restrict__ dout,
                                               const float *__restrict__ lse, int hq, long P,
                                               float *__restrict__ delta, float *__restrict__ lse2) {
  constexpr int LPR = D / 8;  // lanes per (row, head)
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  const long pair = gid / LPR;
  const int part = (int)(gid % LPR);
  const bool ok = pair < P * hq;
  float acc = 0.f;
  if (ok) {
    const long base = pair * D + part * 8;  // pair = row * hq + h
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float a, b;
      if constexpr (sizeof(TI) == 2) {
        a = bf_bits2f(((const unsigned short *)o)[base + j]);
        b = bf_bits2f(((const unsigned short *)dout)[base + j]);
      } else {
        a = ((const float *)o)[base + j];
        b = ((const float *)dout)[base + j];
      }
      acc += a * b;
    }
  }
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (ok && part == 0) {
    const long row = pair / hq;
    const int h = (int)(pair % hq);
    delta[(long)h * P + row] = -acc;
    lse2[(long)h * P + row] = lse[(long)h * P + row] * LOG2E;
  }
}

// Largest squared key norm of each (segment, kv head), a bound on the
// forward's scores: |q . k| <= |q| |k|.  One block per (k-tile, kv head), two
// lanes per row; squared norms are >= 0, so their float bits order as
// unsigned integers and the maximum is an integer atomic (any order gives
// the same result).  The targets start at 0.
template <int D>
__global__ void __launch_bounds__(256) k_key_norm(const unsigned short *__restrict__ k,
                                                  const int32_t *__restrict__ seg_info,
                                                  const int32_t *__restrict__ tile_seg, int hkv,
                                                  unsigned *__restrict__ kn2) {
  constexpr int LPR = 256 / TQ, PER = D / LPR;
  const int g = blockIdx.x, hk = blockIdx.y;
  const TileRows tr = tile_rows(seg_info, tile_seg, g);
  const int r = threadIdx.x / LPR, part = threadIdx.x % LPR;
  float n2 = 0.f;
  if (r < tr.nrows) {
    const unsigned short *src = k + ((long)(tr.start + tr.row0 + r) * hkv + hk) * D + part * PER;
#pragma unroll
    for (int i = 0; i < PER; i += 8) {
      const bf16x8 x = lds8(src + i);
#pragma unroll
      for (int j = 0; j < 8; ++j) n2 = fmaf((float)x[j], (float)x[j], n2);
    }
  }
  n2 += __shfl_xor(n2, 1, 64);
#pragma unroll
  for (int off = 2; off < 64; off <<= 1) n2 = fmaxf(n2, __shfl_xor(n2, off, 64));
  __shared__ float wmax[4];
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = n2;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(kn2 + (long)tile_seg[g] * hkv + hk,
              __float_as_uint(fmaxf(fmaxf(wmax[0], wmax[1]), fmaxf(wmax[2], wmax[3]))));
}

// Order of a block of products whose operand fragments come from LDS: `ahead`
// reads first, then PROD products and READ reads in turn, so that a product
// finds its fragments read `ahead` reads before.  The compiler alone issues a
// read one or two products ahead and waits on it.
template <int READS, int AHEAD, int PROD, int READ>
__device__ __forceinline__ void read_ahead() {
  static_assert(AHEAD <= READS && AHEAD % READ == 0 && READS % READ == 0, "whole groups");
  __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);  // LDS reads
#pragma unroll
  for (int i = 0; i < (READS - AHEAD) / READ; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, PROD, 0);  // products
    __builtin_amdgcn_sched_group_barrier(0x100, READ, 0);
  }
  __builtin_amdgcn_sched_group_barrier(0x008, AHEAD / READ * PROD, 0);
}

// ------------------------------------------------------------- pipelined kernels
//
// Tiles of 64 rows x d (row-major, bf16) are multi-buffered in LDS: the
// loads of the next unit are in flight while the current one is computed.
// Every kernel fills them with direct 16-byte buffer->LDS loads.  All tile
// loads go through buffer resources that start at the segment's first row, so a lane's offset inside a tile is
// fixed for the kernel and a unit adds one scalar; rows past the segment read
// as zeros.  Rows are stored with a 16-byte-chunk swizzle that keeps both
// 16-byte row reads (MFMA operands contracting over d; 16 lanes per LDS
// cycle) and transpose reads (ds_read_b64_tr_b16: operands contracting over
// the rows; 32 lanes per cycle) free of bank conflicts on 64 four-byte banks,
// so no transposed copy of any tensor is needed.  Every lane's swizzled
// offsets are computed once; inside the loops a read is a register offset plus an immediate.

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// 16-byte chunk swizzle of row `row`.  Two properties make both kinds of read
// conflict-free.  Rows 8m..8m+7 differ in bits 1-3: a 32-lane transpose read
// of 8 rows x 2 chunks hits 16 distinct chunks.  And a 16-byte read, which
// takes 16 lanes at a time as {0-3, 12-15, 20-27} and the rest (rows 0-3 and
// 12-15 of one chunk with rows 4-11 of the next), hits 16 distinct chunks:
// rows of equal bits 1-3 (r and 8 + (r ^ 4)) fall on the same side of that
// split and differ in bit 0.  (With the plain rotation (row & 7) << 1 | row >>
// 3 half of a row read conflicts: dQ 175 against 169 ms on the benchmark batch.)  For d = 64 two rows
// share one 256-byte bank line, so the same properties are built from row / 2.
template <int D>
__device__ __forceinline__ int swz(int row) {
  constexpr int H = D == 128 ? 8 : 4;  // rows, or row pairs, of half a pattern
  const int r = (D == 128 ? row : row >> 1) & (2 * H - 1), hi = r / H;
  return (((r & (H - 1)) ^ (hi * (H / 2))) << 1) | hi;
}

// element offset of (row, col) in a swizzled row-major tile of d columns
template <int D>
__device__ __forceinline__ int toff(int row, int col) {
  return row * D + (((col >> 3) ^ swz<D>(row)) << 3) + (col & 7);
}

// Per-lane byte offsets into a 64-row tile, valid for any row block R that is
// a multiple of 16 (the swizzle depends on row % 16 only).
template <int D>
struct LaneOffsets {
  static constexpr int KK = D / 32, DB = D / 16;
  int row[KK];  // 16-byte read of row R + lane%16, chunk 4*kk + lane/16
  int tr[DB];   // transpose reads: rows R + 4g + (lane%16)/4 (and 16 below), columns
                // 16*db + 4*(lane%4)
  __device__ __forceinline__ void init(int lane) {
    const int c = lane & 15, g = lane >> 4;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) row[kk] = toff<D>(c, (kk * 4 + g) * 8) * 2;
#pragma unroll
    for (int db = 0; db < DB; ++db) tr[db] = toff<D>(4 * g + (c >> 2), db * 16 + 4 * (c & 3)) * 2;
  }
};

template <int D>
__device__ __forceinline__ bf16x8 frag_row(const char *tile, int R, int off) {
  return *reinterpret_cast<const bf16x8 *>(tile + R * D * 2 + off);
}

// Operand fragment contracting over tile rows: lane l receives column c(l) of
// rows R + 4g + 0..3 and R + 16 + 4g + 0..3 (g = l/16), the k order of
// accumulator-held operands.
// `bias` is a constant already added to off (see the dK/dV kernel).
template <int D>
__device__ __forceinline__ bf16x8 frag_tr(const char *tile, int R, int off, int bias = 0) {
  const v4i16 a =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(tile + (R * D * 2 - bias + off)));
  const v4i16 b =
      __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16 *)(tile + ((R + 16) * D * 2 - bias + off)));
  const bf16x4 a4 = __builtin_bit_cast(bf16x4, a), b4 = __builtin_bit_cast(bf16x4, b);
  bf16x8 r;
  r[0] = a4[0]; r[1] = a4[1]; r[2] = a4[2]; r[3] = a4[3];
  r[4] = b4[0]; r[5] = b4[1]; r[6] = b4[2]; r[7] = b4[3];
  return r;
}

// four consecutive output values (as a whole where `vec`: the tensor starts
// on an 8-byte, for fp32 a 16-byte boundary)
__device__ __forceinline__ void store4(unsigned short *p, const f32x4 &v, bool vec) {
  const u16x4 b = {f2bf_bits(v[0]), f2bf_bits(v[1]), f2bf_bits(v[2]), f2bf_bits(v[3])};
  if (vec) *reinterpret_cast<u16x4 *>(p) = b;
  else
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = b[j];
}
__device__ __forceinline__ void store4(float *p, const f32x4 &v, bool vec) {
  if (vec) *reinterpret_cast<f32x4 *>(p) = v;
  else
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = v[j];
}
template <class T>
__device__ __forceinline__ bool aligned4(const T *p) {
  return (reinterpret_cast<uintptr_t>(p) & (4 * sizeof(T) - 1)) == 0;
}

// Raw buffer resource over [base, base + bytes): loads past the end return
// zeros, so a tile fill needs no clamping of its rows.
__device__ __forceinline__ i32x4 make_rsrc(const void *base, unsigned bytes) {
  const unsigned long p = (unsigned long)base;
  return i32x4{(int)(unsigned)p, (int)((unsigned)(p >> 32) & 0xffffu), (int)bytes, 0x00020000};
}

__device__ __forceinline__ unsigned lds_addr(const void *p) {
  return (unsigned)(unsigned long)(__attribute__((address_space(3))) const char *)p;
}

// Direct loads of 64 lanes x 16 (or 4) bytes from rs (byte offset voff per lane
// plus the scalar soff) to LDS at byte address dst.  Written as instructions:
// with the builtin the compiler makes every LDS wait drain the LDS queue while
// such a load is in flight.  They have no register result; the end of a step
// waits for them (wait_loads_and_sync).  No memory clobber: LDS is only read
// again behind that barrier (see common.h), and a clobber would turn the scalar
// loads of the walking order into vector loads, whose waits drain these loads.
__device__ __forceinline__ void dma16(unsigned dst, int voff, i32x4 rs, int soff) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
               :: "s"(dst), "v"(voff), "s"(rs), "s"(soff) : "m0");
#endif
}
__device__ __forceinline__ void dma4(unsigned dst, int voff, i32x4 rs, int soff) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
               :: "s"(dst), "v"(voff), "s"(rs), "s"(soff) : "m0");
#endif
}

// Direct buffer->LDS fill of a 64-row tile by NW waves: per-lane byte offsets
// are fixed for the kernel (tile row * row stride + swizzled chunk); a unit
// only adds its first row's byte offset (a scalar).
template <int D, int NW>
struct BufFill {
  static constexpr int CPR = D / 8, PW = 64 * CPR / (64 * NW);
  int voff[PW];
  __device__ __forceinline__ void init(int wave, int lane, int row_bytes) {
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const int s = (wave * PW + i) * 64 + lane;
      const int row = s / CPR;
      voff[i] = row * row_bytes + ((s % CPR) ^ swz<D>(row)) * 16;
    }
  }
  __device__ __forceinline__ void issue(unsigned short *tile, i32x4 rs, int soff, int wave) const {
#pragma unroll
    for (int i = 0; i < PW; ++i) dma16(lds_addr(tile) + (wave * PW + i) * 1024, voff[i], rs, soff);
  }
};

// one dword per lane (lane l: byte l*4 + soff) into 64 consecutive dwords of LDS
__device__ __forceinline__ void buf64_dw(void *dst, i32x4 rs, int lane, int soff) {
  dma4(lds_addr(dst), lane * 4, rs, soff);
}

// Software pipelining over units.  The loads of unit n+1 are issued, then unit
// n is computed from the other buffer, then a barrier behind the loads ends the
// step.  Both happen inside one always-inline step whose LDS buffers are
// distinct __restrict__ parameters.

// the direct loads in flight have landed, for every wave
__device__ __forceinline__ void wait_loads_and_sync() {
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  __syncthreads();
}

// sum of 8 bf16 values (fp32 accumulation)
__device__ __forceinline__ float sum8(const bf16x8 &v, float acc) {
  const bf16x2 one = {(__bf16)1.f, (__bf16)1.f};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    acc = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{v[2 * i], v[2 * i + 1]}, one, acc, false);
  return acc;
}

// XCD-aware block mapping.  Blocks are dispatched round-robin over the 8
// XCDs (block b runs on XCD b % 8), each with its own L2.  XCD x takes the
// contiguous tile range [r.b[x], r.b[x+1]) chosen by the layout so that the
// ranges hold about equal work (the kernel ends with the slowest XCD), and
// runs it kv head by kv head, with the grp query heads of one tile back to
// back: those heads read the same key/value tiles, and neighbouring tiles of
// a segment read mostly the same ones, so the blocks resident on one XCD
// share one kv head's tiles in its L2 (the whole range of one kv head before
// the next measured 1.5-2% faster for the forward and dQ than all nh heads
// of a tile back to back).  `reverse` walks the range from its end (the
// longest rows of each segment first).  The grid is 8 * max range * nh
// blocks; blocks past their XCD's range exit at once.
struct XcdRanges {
  int32_t b[9];
};

__device__ __forceinline__ bool xcd_block(const XcdRanges &r, int nh, int grp, bool reverse,
                                          int &tile, int &head) {
  const int bx = blockIdx.x, x = bx & 7, i = bx >> 3;
  const int lo = r.b[x], C = r.b[x + 1] - lo;
  const int per = C * grp;  // blocks of one kv head's query heads over the range
  if (per == 0) return false;
  const int hk = i / per;
  if (hk >= nh / grp) return false;
  const int rem = i - hk * per;
  const int t = rem / grp;
  head = hk * grp + (rem - t * grp);
  tile = lo + (reverse ? C - 1 - t : t);
  return true;
}

// Longest first, in classes.  The idx-th block of an XCD's C tiles (lo ..) x
// hkv kv heads, with the tiles sorted into eight classes of their number of
// listed partners (ptr), the longest class first; inside a class kv head by kv
// head and in tile order, so neighbouring blocks still share their tiles in
// L2.  The ranges hold equal work, but a range run in tile order can meet a
// long tile near its end: that costs the dK/dV kernel 20% on the 16-segment
// small batch, 130% on one trajectory of it (1.7 blocks per CU) and 14% on one
// trajectory of the 7B-class batch (list scheduling over its tile lists); in
// classes 4%, 58% and 3%.  C <= MAX_CLASSED, blocks of 512
// threads; scratch: 128 ints of LDS.  The result is the same for every thread.
constexpr int MAX_CLASSED = 512;

__device__ __forceinline__ void classed_block(const int32_t *ptr, int lo, int C, int hkv, int idx,
                                              int *scratch, int &tile, int &hk) {
  constexpr int NC = 8, WAVES = MAX_CLASSED / 64;
  int *cnt = scratch, *wmax = scratch + NC * WAVES, *pick = wmax + WAVES;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int len = t < C ? ptr[lo + t + 1] - ptr[lo + t] : 0;
  int m = len;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
  if (lane == 0) wmax[wave] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) m = max(m, wmax[w]);
  const int cls = t < C ? (int)((long)len * NC / (m + 1)) : NC;
  unsigned long long mine = 0;  // lanes of the thread's class
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const unsigned long long b = __ballot(cls == c);
    if (cls == c) mine = b;
    if (lane == 0) cnt[c * WAVES + wave] = __popcll(b);
  }
  __syncthreads();
  // the class, kv head and place of the block (the same in every thread)
  int c = NC - 1, n = 0, rest = idx;
  for (;; --c) {
    n = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) n += cnt[c * WAVES + w];
    if (c == 0 || rest < n * hkv) break;
    rest -= n * hkv;
  }
  hk = rest / n;
  int before = 0;  // tiles of the class in the waves before
#pragma unroll
  for (int w = 0; w < WAVES; ++w) before += w < wave ? cnt[c * WAVES + w] : 0;
  if (cls == c && before + __popcll(mine & ((1ull << lane) - 1)) == rest - hk * n) *pick = t;
  __syncthreads();
  tile = lo + *pick;
}

inline XcdRanges xcd_ranges(const int32_t (&b)[9]) {
  XcdRanges r;
  for (int i = 0; i < 9; ++i) r.b[i] = b[i];
  return r;
}

inline int xcd_grid(const XcdRanges &r, int nh) {
  int c = 0;
  for (int x = 0; x < 8; ++x) c = std::max(c, r.b[x + 1] - r.b[x]);
  return std::max(1, 8 * c * nh);
}

// A unit of work: 64 rows (half of a 128-row tile) of the tile listed at CSR
// entry e.
struct Unit {
  int e, half;
  int r0;       // segment-relative first row of the unit
  int vrows;    // valid rows (1..64)
  int partial;  // PARTIAL tile (an int: a struct without padding bytes is
                // copied field by field, never through private memory)
};

// Unit (e, half) of a q-tile's walking order (`qt_ord`: the global k-tile
// index, bit 31 set for PARTIAL), read as a uniform load through the scalar
// cache (which measured faster than staging the entries in LDS).
__device__ __forceinline__ Unit make_unit(const int32_t *ord, int e, int half, int qbase,
                                          int seg_len) {
  Unit u;
  u.e = e;
  u.half = half;
  const unsigned x = (unsigned)ord[e];
  const int t0 = ((int)(x & 0x7fffffffu) - qbase) * TQ;
  u.r0 = t0 + half * 64;
  u.vrows = min(64, seg_len - u.r0);
  u.partial = (int)(x >> 31);
  return u;
}

// next unit: the second half of the same tile when it has rows, else the next entry
__device__ __forceinline__ bool next_unit(const Unit &u, int e1, const int32_t *ord, int qbase,
                                          int seg_len, Unit &nu) {
  if (u.half == 0 && u.r0 + 64 < seg_len) {
    nu = make_unit(ord, u.e, 1, qbase, seg_len);
    return true;
  }
  if (u.e + 1 < e1) {
    nu = make_unit(ord, u.e + 1, 0, qbase, seg_len);
    return true;
  }
  return false;
}

// The q-tile-stationary kernels walk a q-tile's units in the order of
// `qt_ord`, every FULL unit first and the PARTIAL ones after (measured about
// 3% faster for dQ and 1.5% for the forward than ascending k-tiles, where
// the PARTIAL units of expired turns' text sit between FULL ones; running
// the FULL units in a loop of their own, without the masking branch, gained
// nothing more).  Units alternate between two LDS buffers; `step(u, more,
// nu, current..., next...)` issues the loads of `nu` and computes `u`.
template <class Step, class Issue, class Next>
__device__ __forceinline__ void walk_units(Unit u, const Step &step, const Issue &issue,
                                           const Next &next, unsigned short *__restrict__ k0,
                                           unsigned short *__restrict__ v0, int *__restrict__ m0,
                                           unsigned short *__restrict__ k1,
                                           unsigned short *__restrict__ v1, int *__restrict__ m1) {
  Unit nu;
  issue(u, k0, v0, m0);
  wait_loads_and_sync();
  for (;;) {
    bool more = next(u, nu);
    step(u, more, nu, k0, v0, m0, k1, v1, m1);
    wait_loads_and_sync();
    if (!more) return;
    u = nu;
    more = next(u, nu);
    step(u, more, nu, k1, v1, m1, k0, v0, m0);
    wait_loads_and_sync();
    if (!more) return;
    u = nu;
  }
}

// Forward: one block = one q-tile x one query head, 4 waves of 32 query rows;
// units are 64-key halves of the listed k-tiles.  S^T = K Q^T keeps a lane on
// two queries (rows c and 16 + c of the wave), so the online softmax is
// in-lane (plus two exchanges between the lanes of a row); O^T += V^T P^T with
// V^T by transpose reads.
template <int D, class TO>
__global__ void __launch_bounds__(256, 2) k_attn_fwd(
    const unsigned short *__restrict__ q, const unsigned short *__restrict__ k,
    const unsigned short *__restrict__ v, const int32_t *__restrict__ seg_info,
    const int32_t *__restrict__ tile_seg, const int32_t *__restrict__ tok_meta,
    const int32_t *__restrict__ qt_ptr, const int32_t *__restrict__ qt_ord,
    const float *__restrict__ kn2, const XcdRanges xr, int hq, int hkv, int W, float scale_log2,
    long P, TO *__restrict__ o, float *__restrict__ lse) {
  constexpr int KK = D / 32, DB = D / 16, T64 = 64 * D;
  __shared__ __attribute__((aligned(16))) unsigned short sK0[T64], sK1[T64], sV0[T64], sV1[T64];
  __shared__ __attribute__((aligned(16))) int sM0[64], sM1[64];

  int g, h;
  if (!xcd_block(xr, hq, hq / hkv, true, g, h)) return;
  const int hk = h / (hq / hkv);
  const TileRows tr = tile_rows(seg_info, tile_seg, g);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  bool qvalid[2];
  int qr[2], qstep[2];
  bf16x8 qf[2][KK];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int qloc = wave * 32 + qb * 16 + col;
    qvalid[qb] = qloc < tr.nrows;
    qr[qb] = tr.row0 + (qvalid[qb] ? qloc : 0);
    qstep[qb] = tok_meta[tr.start + qr[qb]] >> 2;
    const unsigned short *qrow = q + ((long)(tr.start + qr[qb]) * hq + h) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[qb][kk] = lds8(qrow + kk * 32 + grp * 8);
  }
  // Fixed offset: when |q| max|k| * scale * log2(e) <= 64 for every row of
  // the wave (max over the segment's keys), every score in log2 units lies
  // in [-64, 64], so P = exp2(S) needs no running max (P and its sums stay
  // within fp32 and bf16 range, and relative precision does not depend on
  // the offset).  Other waves keep the lazily rescaled running max.
  bool zoff;
  {
    const float kmax2 = kn2[(long)tile_seg[g] * hkv + hk];
    bool small = true;
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      float qn2 = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int j = 0; j < 8; ++j) qn2 = fmaf((float)qf[qb][kk][j], (float)qf[qb][kk][j], qn2);
      qn2 = row_sum(qn2);
      small = small && (!qvalid[qb] || qn2 * kmax2 * (scale_log2 * scale_log2) <= 4096.f);
    }
    zoff = __all(small);
  }
  f32x4 oacc[DB][2];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) oacc[db][qb] = f32x4{};
  float m_run[2], l_run[2];
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    m_run[qb] = zoff ? 0.f : -INFINITY;
    l_run[qb] = 0.f;
  }

  LaneOffsets<D> lo;
  lo.init(lane);
  const long kv_stride = (long)hkv * D;
  const int row_bytes = (int)(kv_stride * 2);
  BufFill<D, 4> fp;
  fp.init(wave, lane, row_bytes);
  // the segment's rows of this kv head; rows past the segment read as zeros
  const i32x4 rK =
      make_rsrc(k + (long)hk * D + (long)tr.start * kv_stride, (unsigned)tr.len * row_bytes);
  const i32x4 rV =
      make_rsrc(v + (long)hk * D + (long)tr.start * kv_stride, (unsigned)tr.len * row_bytes);
  const i32x4 rM = make_rsrc(tok_meta + tr.start, (unsigned)tr.len * 4);

  const int swave = __builtin_amdgcn_readfirstlane(wave);  // LDS addresses in scalar registers
  auto issue = [&](const Unit &u, unsigned short *__restrict__ nK, unsigned short *__restrict__ nV,
                   int *__restrict__ nM) __attribute__((always_inline)) {
    fp.issue(nK, rK, u.r0 * row_bytes, swave);
    fp.issue(nV, rV, u.r0 * row_bytes, swave);
    if (swave == 0) buf64_dw(nM, rM, lane, u.r0 * 4);
  };
  auto compute = [&](const Unit &u, const char *__restrict__ sK, const char *__restrict__ sV,
                     const int *__restrict__ sM) __attribute__((always_inline)) {
    f32x4 sacc[4][2];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      bf16x8 ak[KK];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) ak[kk] = frag_row<D>(sK, kb * 16, lo.row[kk]);
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) sacc[kb][qb] = f32x4{};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) sacc[kb][qb] = mfma16(ak[kk], qf[qb][kk], sacc[kb][qb]);
    }
    // 128.0 -> 125.0 ms on the benchmark batch (4 and 6 ahead: 125.5, 125.2)
    read_ahead<4 * KK, 8, 2, 1>();
    // raw scores; masked entries -inf (scale > 0 keeps the order)
    if (__builtin_expect(u.partial, 0)) {
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        const int kb0 = kb * 16 + 4 * grp;
        const i32x4 M4 = *reinterpret_cast<const i32x4 *>(sM + kb0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          // bitwise, not short-circuit: no branch per element
          const int key = kb0 + j, ex = key_expiry(M4[j], W);
#pragma unroll
          for (int qb = 0; qb < 2; ++qb) {
            const bool vis = qvalid[qb] & (key < u.vrows) & (u.r0 + key <= qr[qb]) & (qstep[qb] < ex);
            sacc[kb][qb][j] = vis ? sacc[kb][qb][j] : -INFINITY;
          }
        }
      }
    }
    if (!zoff) {
      float mloc[2];
      bool grow[2];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) {
        mloc[qb] = -INFINITY;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r) mloc[qb] = fmaxf(mloc[qb], sacc[kb][qb][r]);
        mloc[qb] = row_max(mloc[qb]) * scale_log2;
        // Lazy rescaling: the running max (log2 units) only moves when a row's
        // tile max exceeds it by more than 8, so unnormalised P stays below 2^8.
        grow[qb] = mloc[qb] > m_run[qb] + 8.f;
      }
      if (__any(grow[0] | grow[1])) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          // lanes that keep their max keep alpha = 1: with an unset (-inf)
          // max, exp2(m_run - m_new) would be exp2(NaN)
          const float m_new = grow[qb] ? mloc[qb] : m_run[qb];
          const float alpha = grow[qb] ? __builtin_amdgcn_exp2f(m_run[qb] - m_new) : 1.f;
          l_run[qb] *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db) oacc[db][qb] *= alpha;
          m_run[qb] = m_new;
        }
      }
    }
    bf16x8 pf[2][2];
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      const float m_use = (m_run[qb] == -INFINITY) ? 0.f : m_run[qb];
      float rsum = 0.f;
#pragma unroll
      for (int p = 0; p < 2; ++p) {
#pragma unroll
        for (int kb = 2 * p; kb < 2 * p + 2; ++kb)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            sacc[kb][qb][r] = __builtin_amdgcn_exp2f(fmaf(sacc[kb][qb][r], scale_log2, -m_use));
        pf[p][qb] = pack8(sacc[2 * p][qb], sacc[2 * p + 1][qb]);
        rsum = sum8(pf[p][qb], rsum);
      }
      // l_run holds the sum over this lane's keys only: the four lanes of a
      // row share its max and rescale factors, so their sums are combined
      // once at the end
      l_run[qb] += rsum;
    }
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const bf16x8 av = frag_tr<D>(sV, p * 32, lo.tr[db]);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) oacc[db][qb] = mfma16(av, pf[p][qb], oacc[db][qb]);
      }
  };
  auto step = [&](const Unit &u, const bool more, const Unit &nu,
                  const unsigned short *__restrict__ cK, const unsigned short *__restrict__ cV,
                  const int *__restrict__ cM, unsigned short *__restrict__ nK,
                  unsigned short *__restrict__ nV, int *__restrict__ nM)
                  __attribute__((always_inline)) {
    if (more) issue(nu, nK, nV, nM);
    compute(u, reinterpret_cast<const char *>(cK), reinterpret_cast<const char *>(cV), cM);
  };

  const int e0 = qt_ptr[g], e1 = qt_ptr[g + 1];
  auto next = [&](const Unit &u, Unit &n) __attribute__((always_inline)) -> bool {
    return next_unit(u, e1, qt_ord, tr.qbase, tr.len, n);
  };
  walk_units(make_unit(qt_ord, e0, 0, tr.qbase, tr.len), step, issue, next, sK0, sV0, sM0,
             sK1, sV1, sM1);

  const bool vec = aligned4(o);
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const float l = row_sum(l_run[qb]);
    if (!qvalid[qb]) continue;
    const float inv = l > 0.f ? 1.f / l : 0.f;
    const long row = tr.start + qr[qb];
    TO *orow = o + (row * hq + h) * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) store4(orow + db * 16 + 4 * grp, oacc[db][qb] * inv, vec);
    if (grp == 0) lse[(long)h * P + row] = (m_run[qb] + log2f(l)) * LN2;
  }
}

// dK/dV: one block = one k-tile x one kv head, 8 waves, two per SIMD.  Waves
// 0-3 (the P side) each hold K of 32 keys and their dV accumulator; waves
// 4-7 (the dS side) hold V of the same 32 keys and their dK accumulator.  A
// unit is 64 rows of one query head; per 32-row block:
//   P side:  S = Q K^T, P = exp2(S * scale - lse) (masked pairs give 0),
//            P -> LDS, dV += P^T dO
//   dS side: dP = dO V^T, P <- LDS, dS = P (dP - Delta), dK += dS^T Q
// The dS side works one unit behind the P side, so the P of a unit crosses
// the barrier that ends a step; Q/dO tiles therefore live in three buffers
// (the P side's unit, the dS side's unit, and the next unit being loaded;
// the step is unrolled three ways so that each is a compile-time buffer).
// Units are 64-row halves of the listed q-tiles, for every query head of the
// group, in the order of `kt_ord` (FULL q-tiles first, then the PARTIAL
// ones, each from the segment's last q-tile down).  No atomics.  parts > 1: a
// block takes one of `parts` shares of the group's query heads and writes its
// sums (fp32) to that part's array; k_sum_parts adds the parts.
template <int D, class TO>
__global__ void __launch_bounds__(512, 1) k_attn_bwd_dkdv(
    const unsigned short *__restrict__ q, const unsigned short *__restrict__ k,
    const unsigned short *__restrict__ v, const unsigned short *__restrict__ dout,
    const float *__restrict__ lse2, const float *__restrict__ delta,
    const int32_t *__restrict__ seg_info, const int32_t *__restrict__ tile_seg,
    const int32_t *__restrict__ tok_meta, const int32_t *__restrict__ kt_ptr,
    const int32_t *__restrict__ kt_ord, const XcdRanges xr,
    int hq, int hkv, int W,
    float scale_log2, float scale, long P, TO *__restrict__ dk, TO *__restrict__ dv, int parts,
    long part_stride, int classed) {
  constexpr int KK = D / 32, T64 = 64 * D, DB = D / 16, NB = 3;
  // three Q/dO buffers (and their per-row values) as distinct objects: Q/dO
  // tiles first (LDS is laid out by decreasing alignment), buffers 0
  // and 1 in the low 64 KB and buffer 2 above it
  __shared__ __attribute__((aligned(1024))) unsigned short sQ0[T64], sQ1[T64], sD0[T64], sD1[T64];
  __shared__ __attribute__((aligned(512))) unsigned short sQ2[T64], sD2[T64];
  __shared__ __attribute__((aligned(16))) unsigned short sP[2][64 * TQ];
  __shared__ __attribute__((aligned(16))) float sL0[64], sL1[64], sL2[64];
  __shared__ __attribute__((aligned(16))) float sE0[64], sE1[64], sE2[64];
  __shared__ __attribute__((aligned(16))) int sM0[64], sM1[64], sM2[64];

  int g, hk, part;
  {
    // XCD x takes the tiles of its range kv head by kv head, so the blocks
    // resident on one XCD are neighbouring k-tiles of one kv head: they walk
    // the same q-tiles of a segment and share their Q/dO tiles in L2.  A range
    // with more tiles than the classes take runs in tile order (its many
    // blocks even out: 1% on the benchmark batch, where a full sort, which
    // mixes segments, was 7% slower); so does one whose blocks all run at once
    // and a batch of short walks (`classed`, see bwd_impl).
    const int bx = blockIdx.x, x = bx & 7, i = bx >> 3;
    const int lo = xr.b[x], C = xr.b[x + 1] - lo;
    const int nh = hkv * parts;  // a kv head's parts count as heads of their own
    if (i >= C * nh) return;
    int hp;
    if (classed && C <= MAX_CLASSED && C * nh > 32) {
      int *scratch = reinterpret_cast<int *>(sP);
      classed_block(kt_ptr, lo, C, nh, i, scratch, g, hp);
      g = __builtin_amdgcn_readfirstlane(g);
      hp = __builtin_amdgcn_readfirstlane(hp);
    } else {
      hp = i / C;
      g = lo + (i - hp * C);
    }
    hk = hp / parts;
    part = hp - hk * parts;
  }
  const int grp = hq / hkv;
  // the block's query heads of the group
  const int h0 = part * grp / parts, h1 = (part + 1) * grp / parts;
  const TileRows tr = tile_rows(seg_info, tile_seg, g);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int side = wave >> 2, kg = wave & 3;  // side 0: P, dV; side 1: dS, dK
  const int col = lane & 15, grp4 = lane >> 4;
  // the lane's two keys, c and 16 + c of the wave's 32.  A query row sees a
  // key only if its turn/kind word is below kexp4 = 4 x (the key's expiry
  // turn), INT_MAX for keys that never expire
  bool kvalid[2];
  int kr[2], kexp4[2];
  bf16x8 xf[2][KK];  // K fragments (P side) or V fragments (dS side) of the wave's 32 keys
#pragma unroll
  for (int jb = 0; jb < 2; ++jb) {
    const int kloc = kg * 32 + jb * 16 + col;
    kvalid[jb] = kloc < tr.nrows;
    kr[jb] = tr.row0 + (kvalid[jb] ? kloc : 0);
    const int kexp = key_expiry(tok_meta[tr.start + kr[jb]], W);
    kexp4[jb] = kexp >= (1 << 29) ? INT_MAX : kexp << 2;
    const long row = tr.start + kr[jb];
    const unsigned short *src = (side == 0 ? k : v) + (row * hkv + hk) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) xf[jb][kk] = lds8(src + kk * 32 + grp4 * 8);
  }
  f32x4 acc[2][DB];  // dV (P side) or dK (dS side): D[i = key][j = d]
#pragma unroll
  for (int jb = 0; jb < 2; ++jb)
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[jb][db] = f32x4{};

  LaneOffsets<D> lo;
  lo.init(lane);
  // Transposed-read offsets with 64 KB added, hidden from the compiler: for
  // d = 128 a tile of buffer 2 lies above the 64 KB that an LDS
  // instruction's offset field reaches, and with these its reads carry the
  // tile's address in that field instead of adding it to the lane offset per
  // read.
  constexpr int HIBUF = 2, HIBIAS = 65536;
  constexpr bool HIGH2 = 4 * T64 * 2 >= HIBIAS;  // buffers 0 and 1 fill the low 64 KB
  int trh[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) {
    trh[db] = lo.tr[db] + HIBIAS;
    asm volatile("" : "+v"(trh[db]));
  }
  const long q_stride = (long)hq * D;
  const int e0 = kt_ptr[g], e1 = kt_ptr[g + 1];

  // Fill of one unit by all 8 waves with direct buffer->LDS loads: Q and dO
  // rows, and one per-row value by waves 0-2 (log2-sum-exp, Delta, turn).
  // The Q/dO resources start at the segment's first row of the group's first
  // head and a unit adds a scalar byte offset; the per-row resources cover
  // one head's rows of the segment, so rows past the segment (the next
  // segment's, or buffer padding whose log-sum-exp and Delta were never
  // computed) read as zeros and no non-finite value can reach dS = P (dP -
  // Delta) through a masked P = 0.
  const int qrow_bytes = (int)(q_stride * 2);
  BufFill<D, 8> fq;
  fq.init(wave, lane, qrow_bytes);
  const long hbase = (long)hk * grp * D + (long)tr.start * q_stride;
  const unsigned qbytes = (unsigned)(tr.len * (long)qrow_bytes);
  const i32x4 rQ = make_rsrc(q + hbase, qbytes);
  const i32x4 rO = make_rsrc(dout + hbase, qbytes);
  // the wave index as a scalar: the resources and the direct loads' LDS
  // addresses are then built in scalar registers (a resource held in vector
  // registers needs a waterfall loop around every load)
  const int swave = __builtin_amdgcn_readfirstlane(wave);
  const unsigned rbytes = (unsigned)tr.len * 4;
  auto issue = [&](int r0, int hi, unsigned short *__restrict__ nQ, unsigned short *__restrict__ nD,
                   float *__restrict__ nL, float *__restrict__ nE, int *__restrict__ nM)
                   __attribute__((always_inline)) {
    const int so = r0 * qrow_bytes + hi * D * 2;
    fq.issue(nQ, rQ, so, swave);
    fq.issue(nD, rO, so, swave);
    if (swave < 3) {
      const long hrow = (long)(hk * grp + hi) * P + tr.start;
      const i32x4 rS =
          make_rsrc(swave == 0 ? (const void *)(lse2 + hrow)
                    : swave == 1 ? (const void *)(delta + hrow)
                                 : (const void *)(tok_meta + tr.start),
                    rbytes);
      buf64_dw(swave == 0 ? (void *)nL : swave == 1 ? (void *)nE : (void *)nM, rS, lane, r0 * 4);
    }
  };

  // P side: one unit (rows r0 .. r0 + vrows - 1, PARTIAL or ragged if masked)
  auto p_side = [&](auto hi_tag, const int r0, const int vrows, const bool masked,
                    const unsigned short *__restrict__ bQ, const unsigned short *__restrict__ bD,
                    const float *__restrict__ bL, const int *__restrict__ bM,
                    unsigned short *__restrict__ bP) __attribute__((always_inline)) {
    const char *cQ = reinterpret_cast<const char *>(bQ);
    const char *cD = reinterpret_cast<const char *>(bD);
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      // 32 query rows (two 16-row blocks ib) x 32 keys (jb)
      f32x4 s[2][2];
#pragma unroll
      for (int ib = 0; ib < 2; ++ib) {
        bf16x8 aq[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) aq[kk] = frag_row<D>(cQ, qb * 32 + ib * 16, lo.row[kk]);
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) s[ib][jb] = f32x4{};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
          for (int jb = 0; jb < 2; ++jb) s[ib][jb] = mfma16(aq[kk], xf[jb][kk], s[ib][jb]);
      }
#pragma unroll
      for (int ib = 0; ib < 2; ++ib) {
        const f32x4 L4 = *reinterpret_cast<const f32x4 *>(&bL[qb * 32 + ib * 16 + 4 * grp4]);
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[ib][jb][r] = fmaf(s[ib][jb][r], scale_log2, -L4[r]);
      }
      if (masked) {  // uniform branch: only the exponents change
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
          // the lane's query rows qc + 4 grp4 in [qlo, qhi) are inside the
          // unit and not before its key
          const int qhi = vrows - 4 * grp4;
          const int qlo = kvalid[jb] ? kr[jb] - r0 - 4 * grp4 : qhi;
#pragma unroll
          for (int ib = 0; ib < 2; ++ib) {
            const int qc0 = qb * 32 + ib * 16;
            const i32x4 M4 = *reinterpret_cast<const i32x4 *>(&bM[qc0 + 4 * grp4]);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int qc = qc0 + r;
              const bool vis = (qc >= qlo) & (qc < qhi) & (M4[r] < kexp4[jb]);
              s[ib][jb][r] = vis ? s[ib][jb][r] : -INFINITY;
            }
          }
        }
      }
      bf16x8 pa[2];
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) {
#pragma unroll
        for (int ib = 0; ib < 2; ++ib)
#pragma unroll
          for (int r = 0; r < 4; ++r) s[ib][jb][r] = __builtin_amdgcn_exp2f(s[ib][jb][r]);
        pa[jb] = pack8(s[0][jb], s[1][jb]);
      }
      // P in the accumulator's lane order, read back by the dS wave of the same keys
      bf16x8 *pdst = reinterpret_cast<bf16x8 *>(bP) + ((qb * 4 + kg) * 2) * 64 + lane;
      pdst[0] = pa[0];
      pdst[64] = pa[1];
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const bf16x8 bo = decltype(hi_tag)::value ? frag_tr<D>(cD, qb * 32, trh[db], HIBIAS)
                                                  : frag_tr<D>(cD, qb * 32, lo.tr[db]);
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) acc[jb][db] = mfma16(pa[jb], bo, acc[jb][db]);
      }
    }
  };
  // dS side: one unit, whose P was written in the previous step
  auto ds_side = [&](auto hi_tag, const unsigned short *__restrict__ bQ,
                     const unsigned short *__restrict__ bD,
                     const float *__restrict__ bE, const unsigned short *__restrict__ bP)
                     __attribute__((always_inline)) {
    const char *cQ = reinterpret_cast<const char *>(bQ);
    const char *cD = reinterpret_cast<const char *>(bD);
    f32x4 dp[4][2];  // [16-row block][key block]
#pragma unroll
    for (int ib = 0; ib < 4; ++ib) {
      bf16x8 ad[KK];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) ad[kk] = frag_row<D>(cD, ib * 16, lo.row[kk]);
      // dP - Delta: the chain starts from the rows' -Delta
      const f32x4 N4 = *reinterpret_cast<const f32x4 *>(&bE[ib * 16 + 4 * grp4]);
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) dp[ib][jb] = N4;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) dp[ib][jb] = mfma16(ad[kk], xf[jb][kk], dp[ib][jb]);
    }
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) {
      const bf16x8 *psrc = reinterpret_cast<const bf16x8 *>(bP) + ((qb * 4 + kg) * 2) * 64 + lane;
      bf16x8 dsa[2];
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) {
        const bf16x8 pj = psrc[64 * jb];
        f32x4 lo4 = dp[qb * 2][jb], hi4 = dp[qb * 2 + 1][jb];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          lo4[r] *= (float)pj[r];
          hi4[r] *= (float)pj[4 + r];
        }
        dsa[jb] = pack8(lo4, hi4);
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const bf16x8 bq = decltype(hi_tag)::value ? frag_tr<D>(cQ, qb * 32, trh[db], HIBIAS)
                                                  : frag_tr<D>(cQ, qb * 32, lo.tr[db]);
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) acc[jb][db] = mfma16(dsa[jb], bq, acc[jb][db]);
      }
    }
  };

  if (e0 < e1) {
    // Unit state as scalars: walking-order entry, half, query head, first row.
    int ce = e0, chalf = 0, chi = h0;
    int cr0 = (((int)((unsigned)kt_ord[ce] & 0x7fffffffu)) - tr.qbase) * TQ;
    int cpart = (int)((unsigned)kt_ord[ce] >> 31);
    issue(cr0, h0, sQ0, sD0, sL0, sE0, sM0);
    wait_loads_and_sync();
    bool have_cur = true;  // the P side has a unit this step
    int pb = 0;            // P buffer of the P side's unit (the dS side uses the other)
    bool first = true;
    // The work of one step: the direct loads into the next unit's buffers
    // (n*), the P side (c*), the dS side (p*) and the P exchange (wP, rP).
    auto body = [&](auto cur_hi, auto prev_hi, const bool more, const int nr0, const int nhi,
                    unsigned short *__restrict__ nQ,
                    unsigned short *__restrict__ nD, float *__restrict__ nL,
                    float *__restrict__ nE, int *__restrict__ nM,
                    const unsigned short *__restrict__ cQ, const unsigned short *__restrict__ cD,
                    const float *__restrict__ cL, const int *__restrict__ cM,
                    const unsigned short *__restrict__ pQ, const unsigned short *__restrict__ pD,
                    const float *__restrict__ pE, unsigned short *__restrict__ wP,
                    const unsigned short *__restrict__ rP) __attribute__((always_inline)) {
      if (more) issue(nr0, nhi, nQ, nD, nL, nE, nM);
      if (side == 0) {
        if (have_cur) {
          const int vrows = min(64, tr.len - cr0);
          p_side(cur_hi, cr0, vrows, (cpart | (vrows < 64)) != 0, cQ, cD, cL, cM, wP);
        }
      } else if (!first) {
        ds_side(prev_hi, pQ, pD, pE, rP);
      }
    };
    // One step on Q/dO buffer B (the P side's unit; the dS side's is the
    // previous buffer, the next unit's loads go to the following one), with
    // the buffers as compile-time indices, so that their addresses fit the
    // instructions' offset fields.
    auto step = [&](auto bc) __attribute__((always_inline)) -> bool {
      constexpr int B = decltype(bc)::value, NBUF = (B + 1) % NB, PBUF = (B + NB - 1) % NB;
      // next unit: other half of this tile, else next head, else next entry
      int ne = ce, nhalf = 0, nhi = chi, nr0 = 0, npart = cpart;
      bool more = false;
      if (have_cur) {
        const bool second = chalf == 0 && cr0 + 64 < tr.len;
        const bool head = !second && chi + 1 < h1;
        const bool entry = !second && !head && ce + 1 < e1;
        more = second || head || entry;
        if (second) {
          nhalf = 1;
          nr0 = cr0 + 64;
        } else if (head) {
          nr0 = cr0 - chalf * 64;
          nhi = chi + 1;
        } else if (entry) {
          ne = ce + 1;
          const unsigned x = (unsigned)kt_ord[ne];
          nr0 = ((int)(x & 0x7fffffffu) - tr.qbase) * TQ;
          npart = (int)(x >> 31);
          nhi = h0;
        }
      }
      unsigned short *const Q[NB] = {sQ0, sQ1, sQ2}, *const Dd[NB] = {sD0, sD1, sD2};
      float *const Lr[NB] = {sL0, sL1, sL2}, *const Er[NB] = {sE0, sE1, sE2};
      int *const Mr[NB] = {sM0, sM1, sM2};
      body(std::integral_constant<bool, HIGH2 && B == HIBUF>{},
           std::integral_constant<bool, HIGH2 && PBUF == HIBUF>{},
           more, nr0, nhi, Q[NBUF], Dd[NBUF], Lr[NBUF], Er[NBUF], Mr[NBUF], Q[B], Dd[B], Lr[B],
           Mr[B], Q[PBUF], Dd[PBUF], Er[PBUF], sP[pb], sP[pb ^ 1]);
      wait_loads_and_sync();
      if (!have_cur) return false;
      have_cur = more;
      ce = ne;
      chalf = nhalf;
      chi = nhi;
      cr0 = nr0;
      cpart = npart;
      pb ^= 1;
      first = false;
      return true;
    };
    for (;;) {
      if (!step(std::integral_constant<int, 0>{})) break;
      if (!step(std::integral_constant<int, 1>{})) break;
      if (!step(std::integral_constant<int, 2>{})) break;
    }
  }

  // stage through LDS (RP key rows per pass) for coalesced stores;
  // accumulator D[i = key][j = d]
  wait_loads_and_sync();
  TO *st = reinterpret_cast<TO *>(sQ0);
  constexpr int CH = 16 / sizeof(TO);   // elements per 16-byte chunk
  constexpr int RP = 128 / sizeof(TO);  // key rows per pass (16 KB)
  const float mul = side == 0 ? 1.f : scale;
#pragma unroll
  for (int which = 0; which < 2; ++which) {
    TO *dst = (which == 0 ? dv : dk) + part * part_stride;
#pragma unroll
    for (int pass = 0; pass < TQ / RP; ++pass) {
      if (side == which && kg * 32 >= pass * RP && kg * 32 < (pass + 1) * RP) {
#pragma unroll
        for (int jb = 0; jb < 2; ++jb)
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const int kl = kg * 32 + jb * 16 + 4 * grp4 + r - pass * RP;
              store_val(st, kl * D + db * 16 + col, acc[jb][db][r] * mul);
            }
      }
      __syncthreads();
      for (int c = threadIdx.x; c < RP * D / CH; c += 512) {
        const int kl = c / (D / CH), ch = c % (D / CH);
        const int key = pass * RP + kl;
        if (key < tr.nrows) {
          const long row = tr.start + tr.row0 + key;
          *reinterpret_cast<u16x8 *>(dst + (row * hkv + hk) * D + ch * CH) =
              *reinterpret_cast<const u16x8 *>(st + kl * D + ch * CH);
        }
      }
      __syncthreads();
    }
  }
}

// dk and dv [P, hkv, D] from `parts` fp32 arrays (dk then dv in each), summed in
// order, 8 elements a thread; padding rows are not written.
template <class TO>
__global__ void __launch_bounds__(256) k_sum_parts(const float *__restrict__ part, int parts, long P,
                                                   int width, const int32_t *__restrict__ tok_meta,
                                                   TO *__restrict__ dk, TO *__restrict__ dv) {
  const long n = P * width, n8 = n / 8;
  for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < 2 * n8; i += (long)gridDim.x * 256) {
    const bool second = i >= n8;
    const long at = (second ? i - n8 : i) * 8;
    if ((tok_meta[at / width] & 3) == SEG_KIND_PAD) continue;
    f32x4 a = f32x4{}, b = f32x4{};
    for (int k = 0; k < parts; ++k) {
      const f32x4 *p = reinterpret_cast<const f32x4 *>(part + k * 2 * n + i * 8);
      a += p[0];
      b += p[1];
    }
    TO *d = (second ? dv : dk) + at;
    store4(d, a, true);
    store4(d + 4, b, true);
  }
}

// dQ: one block = one q-tile x one query head, 4 waves of 32 query rows;
// units are 64-key halves of the listed k-tiles.  Recomputes S^T and dP^T per
// unit; dQ^T += K^T dS^T with K^T by transpose reads.  With FUSE (bf16
// inputs) the kernel also forms each of its rows' -Delta = -(dO . O) and
// log2-sum-exp from O and the natural-log LSE, uses them, and writes them for
// the dK/dV kernel that runs after it (no separate pre-pass); without FUSE it
// reads what the pre-pass wrote.
template <int D, class TO, bool FUSE>
__global__ void __launch_bounds__(256, 2) k_attn_bwd_dq(
    const unsigned short *__restrict__ q, const unsigned short *__restrict__ k,
    const unsigned short *__restrict__ v, const unsigned short *__restrict__ dout,
    const unsigned short *__restrict__ o, const float *__restrict__ lse,
    float *__restrict__ lse2, float *__restrict__ delta,
    const int32_t *__restrict__ seg_info, const int32_t *__restrict__ tile_seg,
    const int32_t *__restrict__ tok_meta, const int32_t *__restrict__ qt_ptr,
    const int32_t *__restrict__ qt_ord, const XcdRanges xr, int hq, int hkv, int W,
    float scale_log2, float scale, long P, TO *__restrict__ dq) {
  constexpr int KK = D / 32, DB = D / 16, T64 = 64 * D;
  __shared__ __attribute__((aligned(16))) unsigned short sK0[T64], sK1[T64], sV0[T64], sV1[T64];
  __shared__ __attribute__((aligned(16))) int sM0[64], sM1[64];

  int g, h;
  if (!xcd_block(xr, hq, hq / hkv, true, g, h)) return;
  const int hk = h / (hq / hkv);
  const TileRows tr = tile_rows(seg_info, tile_seg, g);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int col = lane & 15, grp = lane >> 4;
  // the lane's two queries, rows c and 16 + c of the wave's 32
  bool qvalid[2];
  int qr[2], qstep[2];
  bf16x8 qf[2][KK], df[2][KK];
  float l2[2], ndlt[2];  // log2-sum-exp and -Delta
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    const int qloc = wave * 32 + qb * 16 + col;
    qvalid[qb] = qloc < tr.nrows;
    qr[qb] = tr.row0 + (qvalid[qb] ? qloc : 0);
    const long qrow_abs = tr.start + qr[qb];
    qstep[qb] = tok_meta[qrow_abs] >> 2;
    const unsigned short *qp = q + (qrow_abs * hq + h) * D;
    const unsigned short *dp = dout + (qrow_abs * hq + h) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      qf[qb][kk] = lds8(qp + kk * 32 + grp * 8);
      df[qb][kk] = lds8(dp + kk * 32 + grp * 8);
    }
    const long rv = (long)h * P + qrow_abs;
    if constexpr (FUSE) {
      // the lane holds a quarter of the row's d (the other lanes of the row
      // the rest): bf16 products are exact in fp32, summed in a fixed order
      const unsigned short *op = o + (qrow_abs * hq + h) * D;
      float acc = 0.f;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 of = lds8(op + kk * 32 + grp * 8);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          acc = __builtin_amdgcn_fdot2_f32_bf16(bf16x2{df[qb][kk][2 * i], df[qb][kk][2 * i + 1]},
                                                bf16x2{of[2 * i], of[2 * i + 1]}, acc, false);
      }
      ndlt[qb] = -row_sum(acc);
      l2[qb] = lse[rv] * LOG2E;
      if (qvalid[qb] && grp == 0) {
        delta[rv] = ndlt[qb];
        lse2[rv] = l2[qb];
      }
    } else {
      l2[qb] = lse2[rv];
      ndlt[qb] = delta[rv];
    }
  }
  f32x4 dqacc[DB][2];
#pragma unroll
  for (int db = 0; db < DB; ++db)
#pragma unroll
    for (int qb = 0; qb < 2; ++qb) dqacc[db][qb] = f32x4{};

  LaneOffsets<D> lo;
  lo.init(lane);
  const long kv_stride = (long)hkv * D;
  const int row_bytes = (int)(kv_stride * 2);
  BufFill<D, 4> fp;
  fp.init(wave, lane, row_bytes);
  // the segment's rows of this kv head; rows past the segment read as zeros
  const i32x4 rK =
      make_rsrc(k + (long)hk * D + (long)tr.start * kv_stride, (unsigned)tr.len * row_bytes);
  const i32x4 rV =
      make_rsrc(v + (long)hk * D + (long)tr.start * kv_stride, (unsigned)tr.len * row_bytes);
  const i32x4 rM = make_rsrc(tok_meta + tr.start, (unsigned)tr.len * 4);

  // the wave index as a scalar: the direct loads' LDS addresses are then
  // formed in scalar registers (no readfirstlane per load)
  const int swave = __builtin_amdgcn_readfirstlane(wave);
  auto issue = [&](const Unit &u, unsigned short *__restrict__ nK, unsigned short *__restrict__ nV,
                   int *__restrict__ nM) __attribute__((always_inline)) {
    fp.issue(nK, rK, u.r0 * row_bytes, swave);
    fp.issue(nV, rV, u.r0 * row_bytes, swave);
    if (swave == 0) buf64_dw(nM, rM, lane, u.r0 * 4);
  };
  auto compute = [&](const Unit &u, const char *__restrict__ sK, const char *__restrict__ sV,
                     const int *__restrict__ sM) __attribute__((always_inline)) {
#pragma unroll
    for (int kh = 0; kh < 2; ++kh) {  // 32-key halves, two 16-key blocks kb each
      if (kh * 32 >= u.vrows) break;
      f32x4 s[2][2], dp[2][2];
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        bf16x8 ak[KK], av[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          ak[kk] = frag_row<D>(sK, kh * 32 + kb * 16, lo.row[kk]);
          av[kk] = frag_row<D>(sV, kh * 32 + kb * 16, lo.row[kk]);
        }
        // dP^T - Delta: the chain starts from -Delta (one value per query)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          s[kb][qb] = f32x4{};
          dp[kb][qb] = f32x4{ndlt[qb], ndlt[qb], ndlt[qb], ndlt[qb]};
        }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
#pragma unroll
          for (int qb = 0; qb < 2; ++qb) {
            s[kb][qb] = mfma16(ak[kk], qf[qb][kk], s[kb][qb]);
            dp[kb][qb] = mfma16(av[kk], df[qb][kk], dp[kb][qb]);
          }
      }
      // with the order below 172.1 -> 168.0 ms on the benchmark batch (this
      // one alone 169.0; 6 or 8 ahead 169.3, 169.8).  The dK/dV kernel's
      // products in such orders: 259.5 -> 261-266 ms, so it has none
      read_ahead<4 * KK, 4, 2, 1>();
      // dS^T = P^T (dP^T - Delta); a masked pair gets exponent -inf (P = 0).
      // One uniform branch; inside, the predicate is bitwise (no branch per
      // element).
      if (__builtin_expect(u.partial, 0)) {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) {
          // the lane's keys kc + 4 grp < lim are inside the unit and not
          // after its query
          const int lim = (qvalid[qb] ? min(u.vrows, qr[qb] - u.r0 + 1) : 0) - 4 * grp;
          const unsigned wfloor = window_floor(qstep[qb], W);
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            const int kc0 = kh * 32 + kb * 16;
            const i32x4 M4 = *reinterpret_cast<const i32x4 *>(sM + kc0 + 4 * grp);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              const bool vis = (kc0 + j < lim) & (window_word(M4[j]) >= wfloor);
              const float x = vis ? fmaf(s[kb][qb][j], scale_log2, -l2[qb]) : -INFINITY;
              s[kb][qb][j] = __builtin_amdgcn_exp2f(x) * dp[kb][qb][j];
            }
          }
        }
      } else {
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
#pragma unroll
            for (int j = 0; j < 4; ++j)
              s[kb][qb][j] = __builtin_amdgcn_exp2f(fmaf(s[kb][qb][j], scale_log2, -l2[qb])) *
                             dp[kb][qb][j];
      }
      bf16x8 dsb[2];
#pragma unroll
      for (int qb = 0; qb < 2; ++qb) dsb[qb] = pack8(s[0][qb], s[1][qb]);
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        const bf16x8 kt = frag_tr<D>(sK, kh * 32, lo.tr[db]);
#pragma unroll
        for (int qb = 0; qb < 2; ++qb) dqacc[db][qb] = mfma16(kt, dsb[qb], dqacc[db][qb]);
      }
      read_ahead<2 * DB, DB == 8 ? 6 : 4, 2, 2>();
    }
  };
  auto step = [&](const Unit &u, const bool more, const Unit &nu,
                  const unsigned short *__restrict__ cK, const unsigned short *__restrict__ cV,
                  const int *__restrict__ cM, unsigned short *__restrict__ nK,
                  unsigned short *__restrict__ nV, int *__restrict__ nM)
                  __attribute__((always_inline)) {
    if (more) issue(nu, nK, nV, nM);
    compute(u, reinterpret_cast<const char *>(cK), reinterpret_cast<const char *>(cV), cM);
  };

  const int e0 = qt_ptr[g], e1 = qt_ptr[g + 1];
  auto next = [&](const Unit &u, Unit &n) __attribute__((always_inline)) -> bool {
    return next_unit(u, e1, qt_ord, tr.qbase, tr.len, n);
  };
  walk_units(make_unit(qt_ord, e0, 0, tr.qbase, tr.len), step, issue, next, sK0, sV0, sM0,
             sK1, sV1, sM1);

  const bool vec = aligned4(dq);
#pragma unroll
  for (int qb = 0; qb < 2; ++qb) {
    if (!qvalid[qb]) continue;
    TO *qrowp = dq + ((long)(tr.start + qr[qb]) * hq + h) * D;
#pragma unroll
    for (int db = 0; db < DB; ++db) store4(qrowp + db * 16 + 4 * grp, dqacc[db][qb] * scale, vec);
  }
}

// ------------------------------------------------------------- host side

struct AttnWs {
  size_t kn2, delta, lse2, qb, kb, vb, dob, part, base, total;  // base: without the dK/dV parts
  int parts;
};

// Shares of a kv head's query heads that dK/dV blocks take.  With fewer blocks
// (tiles x kv heads) than CUs a block's walk over all heads of the group is the
// kernel's time, so the heads are shared out: 4q/1kv, 1,088 rows: 55 us in one
// part, 19 in four and 4 for the sums.  A block owns its CU, so
//  - more blocks than CUs run in two rounds, and two rounds of half a walk win
//    nothing where both hold walks of about the same length: where every segment
//    is one tile (12q/4kv, 60 of 128 rows: backward 53 us in one part, 83 in two),
//    or where an eighth of the work lies in the first columns of one segment and
//    its blocks exceed an XCD's 32 CUs (16q/4kv d = 64, 8,000 rows: 783 and 825;
//    7,100 rows, 32 blocks: 1,092 and 959).  Where an eighth holds whole segments
//    the second round is their short walks (16q/2kv, 20 of 700: 267 and 241);
//  - only the longest share counts: a group of 7 in five parts waits for two
//    heads as in four;
//  - a walk must get shorter by more than the sums cost: 1.6 us (d = 64: 1.1) for
//    64 rows of a head against a launch of 4.4 us or, if longer, the parts written
//    and read at 2.7 TB/s (16q/8kv, one of 100 rows: 27.0 us in one part, 29.4 in
//    two; one of 200: 37.7 and 36.5; three of 1,000: 117 and 123).
// The parts' fp32 sums stay within the fixed scratch of seg_attn_bwd_noalloc, so
// that both entry points take the same path.
int dkdv_parts(const seg_sizes &sz, size_t base, size_t part_bytes, int hq, int hkv, int d) {
  const long blocks = (long)sz.num_qtiles * hkv, grp = hq / hkv;
  if (blocks <= 0) return 1;
  long n = std::min<long>(grp, (256 + blocks - 1) / blocks);
  if (n > 1 && blocks * n > 256) {
    // columns of an eighth of the lower triangles that starts with a longest segment
    const long tiles = ((long)sz.max_seg_len + TQ - 1) / TQ;
    long c = 0;
    for (long work = 0; c < tiles && 8 * work < sz.tile_nnz_max; ++c) work += tiles - c;
    if (tiles == 1 || (n == 2 && c < tiles && c * hkv * n > 32)) n = 256 / blocks;
  }
  while (n > 1 && base + n * part_bytes > SEG_ATTN_BWD_SCRATCH_BYTES) --n;
  if (n <= 1) return 1;
  const long share = (grp + n - 1) / n;
  n = (grp + share - 1) / share;
  const double saved = (double)(grp - share) * (((long)sz.max_seg_len + 63) / 64) * (d == 128 ? 1.6 : 1.1);
  return saved < std::max(4.4, n * 2.0 * part_bytes / 2.7e6) ? 1 : (int)n;
}

AttnWs attn_ws(const seg_sizes &sz, seg_dtype dt, int hq, int hkv, int d, int bwd) {
  AttnWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  const size_t P = (size_t)std::max<int64_t>(1, sz.packed_tokens);
  if (!bwd) w.kn2 = take((size_t)std::max(1, sz.num_segments) * hkv * sizeof(float));
  if (bwd) {
    w.delta = take(P * hq * sizeof(float));
    w.lse2 = take(P * hq * sizeof(float));
  }
  if (dt == SEG_F32) {
    w.qb = take(P * hq * d * 2);
    w.kb = take(P * hkv * d * 2);
    w.vb = take(P * hkv * d * 2);
    if (bwd) w.dob = take(P * hq * d * 2);
  }
  w.base = std::max<size_t>(off, 256);
  w.parts = 1;
  if (bwd) {
    const size_t bytes = P * hkv * d * 2 * sizeof(float);
    w.parts = dkdv_parts(sz, off, bytes, hq, hkv, d);
    if (w.parts > 1) w.part = take(w.parts * bytes);
  }
  w.total = std::max<size_t>(off, 256);
  return w;
}

void check_common(const seg_layout *L, const seg_sizes *sz, seg_dtype dt, int hq, int hkv, int d) {
  SEG_CHECK(L && sz, SEG_ERR_ARG, "layout or sizes is NULL");
  SEG_CHECK(dt == SEG_BF16 || dt == SEG_F32, SEG_ERR_ARG, "unknown dtype %d", (int)dt);
  SEG_CHECK(hq >= 1 && hkv >= 1 && hq % hkv == 0, SEG_ERR_UNSUPPORTED,
            "need hq %% hkv == 0 (hq=%d, hkv=%d)", hq, hkv);
  SEG_CHECK(d == 64 || d == 128, SEG_ERR_UNSUPPORTED, "head_dim %d not in {64, 128}", d);
  SEG_CHECK(L->tile == TQ, SEG_ERR_UNSUPPORTED, "attention needs a layout with tile 128 (got %d)",
            L->tile);
  SEG_CHECK(L->window >= 1, SEG_ERR_ARG, "layout window not set (build the layout first)");
  // the launch schedule: eight ranges covering every tile once
  for (const int32_t *b : {L->xcd_rows, L->xcd_cols}) {
    bool ok = b[0] == 0 && b[8] == sz->num_qtiles;
    for (int x = 0; x < 8; ++x) ok = ok && b[x] <= b[x + 1];
    SEG_CHECK(ok, SEG_ERR_ARG, "layout schedule ranges not set (build the layout first)");
  }
  SEG_CHECK((long)sz->packed_tokens * hq * d < (1L << 40), SEG_ERR_CAPACITY, "tensor too large");
  // tile loads address a segment's rows, and the per-row values of a head
  // group, with 32-bit byte offsets from one buffer resource
  SEG_CHECK((long)sz->max_seg_len * hq * d * 2 <= INT32_MAX, SEG_ERR_CAPACITY,
            "a segment of %d rows exceeds the 2 GiB addressable per tile stream", sz->max_seg_len);
  SEG_CHECK((long)sz->packed_tokens * hq * 4 <= INT32_MAX, SEG_ERR_CAPACITY,
            "%lld packed rows x %d heads of fp32 row values exceed 2 GiB",
            (long long)sz->packed_tokens, hq);
}

// q, k, v and (backward) dO as bf16 in the workspace
void to_bf16(const void *q, const void *k, const void *v, const void *d_o, unsigned short *q2,
             unsigned short *k2, unsigned short *v2, unsigned short *do2, long nq, long nkv,
             unsigned *zero, long nzero, hipStream_t st) {
  ToBf16 t{{static_cast<const float *>(q), static_cast<const float *>(k), static_cast<const float *>(v),
            static_cast<const float *>(d_o)},
           {q2, k2, v2, do2},
           {}};
  t.end[0] = nq / 8;
  t.end[1] = t.end[0] + nkv / 8;
  t.end[2] = t.end[1] + nkv / 8;
  t.end[3] = t.end[2] + (d_o ? nq / 8 : 0);
  ProfScope prof("attn_prep", st);
  k_f32_to_bf16<<<(int)std::max<long>(1, std::min<long>(16384, (t.end[3] + 255) / 256)), 256, 0, st>>>(
      t, zero, nzero);
  SEG_LAUNCH_CHECK();
}

template <int D, class TO>
void fwd_impl(const seg_layout *L, const seg_sizes *sz, int hq, int hkv, float scale,
              const unsigned short *q, const unsigned short *k, const unsigned short *v, void *o,
              float *lse, unsigned *kn2, hipStream_t st) {
  const int G = sz->num_qtiles;
  ProfScope prof("attn_fwd", st);
  if (sizeof(TO) == 2) fill32(kn2, (long)sz->num_segments * hkv, 0u, st);  // else cleared by to_bf16
  k_key_norm<D><<<dim3(G, hkv), 256, 0, st>>>(k, L->seg_info, L->tile_seg, hkv, kn2);
  SEG_LAUNCH_CHECK();
  const XcdRanges xr = xcd_ranges(L->xcd_rows);
  k_attn_fwd<D, TO><<<xcd_grid(xr, hq), 256, 0, st>>>(
      q, k, v, L->seg_info, L->tile_seg, L->tok_meta, L->qt_ptr, L->qt_ord,
      reinterpret_cast<const float *>(kn2), xr, hq, hkv, L->window, scale * LOG2E,
      sz->packed_tokens, static_cast<TO *>(o), lse);
  SEG_LAUNCH_CHECK();
}

template <int D, class TO, class TI>
void bwd_impl(const seg_layout *L, const seg_sizes *sz, int hq, int hkv, float scale,
              const unsigned short *q, const unsigned short *k, const unsigned short *v,
              const unsigned short *dout, const TI *o_raw, const TI *dout_raw,
              const float *lse, float *delta, float *lse2, void *dq, void *dk, void *dv,
              int parts, float *part, hipStream_t st) {
  const int G = sz->num_qtiles;
  const long P = sz->packed_tokens;
  // bf16 inputs: the dQ kernel forms -Delta and the log2-sum-exp of its rows
  // and runs first; fp32 inputs: the pre-pass forms them from the unrounded
  // O and dO
  constexpr bool FUSE = sizeof(TI) == 2;
  if constexpr (!FUSE) {
    const long threads = P * hq * (D / 8);
    ProfScope prof("attn_delta", st);
    k_delta<TI, D><<<(int)((threads + 255) / 256), 256, 0, st>>>(o_raw, dout_raw, lse, hq, P, delta,
                                                                 lse2);
    SEG_LAUNCH_CHECK();
  }
  {
    ProfScope prof("attn_bwd_dq", st);
    const XcdRanges xr = xcd_ranges(L->xcd_rows);
    k_attn_bwd_dq<D, TO, FUSE><<<xcd_grid(xr, hq), 256, 0, st>>>(
        q, k, v, dout, reinterpret_cast<const unsigned short *>(o_raw), lse, lse2, delta,
        L->seg_info, L->tile_seg, L->tok_meta, L->qt_ptr, L->qt_ord, xr, hq, hkv, L->window,
        scale * LOG2E, scale, P, static_cast<TO *>(dq));
    SEG_LAUNCH_CHECK();
  }
  {
    ProfScope prof("attn_bwd_dkdv", st);
    const XcdRanges xc = xcd_ranges(L->xcd_cols);
    // Sorting its range into classes costs a block about 2 us.  Where every
    // segment is one tile all walks are equal and nothing is won (8q/8kv, 300
    // segments: 240 us sorted, 224 in order); where the longest walk is below
    // four tiles x heads, less than the sort (8q/8kv, 100 segments of 3 tiles:
    // 295 against 283); from four on, more (8q/4kv, 50 of 2: 82 against 87).
    const int lmax = (int)((sz->max_seg_len + (long)TQ - 1) / TQ), share = (hq / hkv + parts - 1) / parts;
    const int classed = lmax >= 2 && (long)lmax * share >= 4;
    if (parts > 1) {
      const long n = P * hkv * D;
      k_attn_bwd_dkdv<D, float><<<xcd_grid(xc, hkv * parts), 512, 0, st>>>(
          q, k, v, dout, lse2, delta, L->seg_info, L->tile_seg, L->tok_meta, L->kt_ptr, L->kt_ord,
          xc, hq, hkv, L->window, scale * LOG2E, scale, P, part, part + n, parts, 2 * n, classed);
      SEG_LAUNCH_CHECK();
      k_sum_parts<TO><<<(int)std::max<long>(1, std::min<long>(4096, (n / 4 + 255) / 256)), 256, 0, st>>>(
          part, parts, P, hkv * D, L->tok_meta, static_cast<TO *>(dk), static_cast<TO *>(dv));
    } else {
      k_attn_bwd_dkdv<D, TO><<<xcd_grid(xc, hkv), 512, 0, st>>>(
          q, k, v, dout, lse2, delta, L->seg_info, L->tile_seg, L->tok_meta, L->kt_ptr, L->kt_ord,
          xc, hq, hkv, L->window, scale * LOG2E, scale, P, static_cast<TO *>(dk),
          static_cast<TO *>(dv), 1, 0, classed);
    }
    SEG_LAUNCH_CHECK();
  }
}

}  // namespace
}  // namespace seg

using namespace seg;

extern "C" size_t seg_attn_workspace_bytes(const seg_sizes *sz, seg_dtype dt, int32_t hq,
                                           int32_t hkv, int32_t d, int32_t bwd) {
  if (!sz || hq < 1 || hkv < 1) return 0;
  return attn_ws(*sz, dt, hq, hkv, d, bwd).total;
}

extern "C" seg_status seg_attn_fwd(const seg_layout *L, const seg_sizes *sz, seg_dtype dt,
                                   int32_t hq, int32_t hkv, int32_t d, float softmax_scale,
                                   const void *q, const void *k, const void *v, void *o,
                                   float *lse, void *ws, size_t ws_bytes, hipStream_t stream) {
  return guarded([&] {
    check_common(L, sz, dt, hq, hkv, d);
    const AttnWs w = attn_ws(*sz, dt, hq, hkv, d, 0);
    SEG_CHECK(ws_bytes >= w.total, SEG_ERR_WORKSPACE, "workspace of %zu bytes < required %zu",
              ws_bytes, w.total);
    if (sz->num_qtiles == 0) return;
    SEG_CHECK(q && k && v && o && lse && ws, SEG_ERR_ARG, "a tensor pointer is NULL");
    SEG_CHECK(std::isfinite(softmax_scale), SEG_ERR_ARG, "softmax_scale is not finite");
    char *base = static_cast<char *>(ws);
    const long P = sz->packed_tokens;
    unsigned *kn2 = reinterpret_cast<unsigned *>(base + w.kn2);
    const unsigned short *qb, *kb, *vb;
    if (dt == SEG_F32) {
      unsigned short *q2 = reinterpret_cast<unsigned short *>(base + w.qb);
      unsigned short *k2 = reinterpret_cast<unsigned short *>(base + w.kb);
      unsigned short *v2 = reinterpret_cast<unsigned short *>(base + w.vb);
      to_bf16(q, k, v, nullptr, q2, k2, v2, nullptr, P * hq * d, P * hkv * d, kn2,
              (long)sz->num_segments * hkv, stream);
      qb = q2;
      kb = k2;
      vb = v2;
    } else {
      qb = static_cast<const unsigned short *>(q);
      kb = static_cast<const unsigned short *>(k);
      vb = static_cast<const unsigned short *>(v);
    }
    if (d == 128) {
      if (dt == SEG_F32) fwd_impl<128, float>(L, sz, hq, hkv, softmax_scale, qb, kb, vb, o, lse, kn2, stream);
      else fwd_impl<128, unsigned short>(L, sz, hq, hkv, softmax_scale, qb, kb, vb, o, lse, kn2, stream);
    } else {
      if (dt == SEG_F32) fwd_impl<64, float>(L, sz, hq, hkv, softmax_scale, qb, kb, vb, o, lse, kn2, stream);
      else fwd_impl<64, unsigned short>(L, sz, hq, hkv, softmax_scale, qb, kb, vb, o, lse, kn2, stream);
    }
  });
}

extern "C" seg_status seg_attn_bwd(const seg_layout *L, const seg_sizes *sz, seg_dtype dt,
                                   int32_t hq, int32_t hkv, int32_t d, float softmax_scale,
                                   const void *q, const void *k, const void *v, const void *o,
                                   const float *lse, const void *d_o, void *dq, void *dk, void *dv,
                                   void *ws, size_t ws_bytes, hipStream_t stream) {
  return guarded([&] {
    check_common(L, sz, dt, hq, hkv, d);
    const AttnWs w = attn_ws(*sz, dt, hq, hkv, d, 1);
    SEG_CHECK(ws_bytes >= w.base, SEG_ERR_WORKSPACE, "workspace of %zu bytes < required %zu",
              ws_bytes, w.base);
    // (a workspace without room for the parts of dK/dV serves in one part)
    const int parts = ws_bytes >= w.total ? w.parts : 1;
    if (sz->num_qtiles == 0) return;
    SEG_CHECK(q && k && v && o && lse && d_o && dq && dk && dv && ws, SEG_ERR_ARG,
              "a tensor pointer is NULL");
    SEG_CHECK(std::isfinite(softmax_scale), SEG_ERR_ARG, "softmax_scale is not finite");
    char *base = static_cast<char *>(ws);
    const long P = sz->packed_tokens;
    float *delta = reinterpret_cast<float *>(base + w.delta);
    float *lse2 = reinterpret_cast<float *>(base + w.lse2);
    float *part = reinterpret_cast<float *>(base + w.part);
    if (dt == SEG_F32) {
      unsigned short *q2 = reinterpret_cast<unsigned short *>(base + w.qb);
      unsigned short *k2 = reinterpret_cast<unsigned short *>(base + w.kb);
      unsigned short *v2 = reinterpret_cast<unsigned short *>(base + w.vb);
      unsigned short *do2 = reinterpret_cast<unsigned short *>(base + w.dob);
      to_bf16(q, k, v, d_o, q2, k2, v2, do2, P * hq * d, P * hkv * d, nullptr, 0, stream);
      const float *o32 = static_cast<const float *>(o), *do32 = static_cast<const float *>(d_o);
      if (d == 128)
        bwd_impl<128, float, float>(L, sz, hq, hkv, softmax_scale, q2, k2, v2, do2, o32, do32,
                                    lse, delta, lse2, dq, dk, dv, parts, part, stream);
      else
        bwd_impl<64, float, float>(L, sz, hq, hkv, softmax_scale, q2, k2, v2, do2, o32, do32, lse,
                                   delta, lse2, dq, dk, dv, parts, part, stream);
    } else {
      const unsigned short *qb = static_cast<const unsigned short *>(q);
      const unsigned short *kb = static_cast<const unsigned short *>(k);
      const unsigned short *vb = static_cast<const unsigned short *>(v);
      const unsigned short *dob = static_cast<const unsigned short *>(d_o);
      const unsigned short *o16 = static_cast<const unsigned short *>(o);
      if (d == 128)
        bwd_impl<128, unsigned short, unsigned short>(L, sz, hq, hkv, softmax_scale, qb, kb, vb,
                                                      dob, o16, dob, lse, delta, lse2, dq, dk,
                                                      dv, parts, part, stream);
      else
        bwd_impl<64, unsigned short, unsigned short>(L, sz, hq, hkv, softmax_scale, qb, kb, vb,
                                                     dob, o16, dob, lse, delta, lse2, dq, dk,
                                                     dv, parts, part, stream);
    }
  });
}

// Workspace of seg_attn_bwd_noalloc: one copy of this array per GPU, held
// until the process ends.  Host code never uses the name itself (on the host
// it is a stand-in, not a device address): the device address comes from
// hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[SEG_ATTN_BWD_SCRATCH_BYTES];

namespace seg {
namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device.
void *scratch_on_current_device() {
  int dev = -1;
  SEG_HIP(hipGetDevice(&dev));
  SEG_CHECK(dev >= 0 && dev < kMaxDevices, SEG_ERR_UNSUPPORTED, "device %d above %d", dev,
            kMaxDevices - 1);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *ptr = nullptr;
    SEG_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    SEG_CHECK(ptr != nullptr, SEG_ERR_HIP, "no device address for the scratch array");
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}

}  // namespace
}  // namespace seg

extern "C" seg_status seg_attn_bwd_noalloc(const seg_layout *L, const seg_sizes *sz, seg_dtype dt,
                                           int32_t hq, int32_t hkv, int32_t d,
                                           float softmax_scale, const void *q, const void *k,
                                           const void *v, const void *o, const float *lse,
                                           const void *d_o, void *dq, void *dk, void *dv,
                                           hipStream_t stream) {
  void *ptr = nullptr;
  const seg_status st = guarded([&] {
    check_common(L, sz, dt, hq, hkv, d);
    const size_t need = attn_ws(*sz, dt, hq, hkv, d, 1).base;
    SEG_CHECK(need <= SEG_ATTN_BWD_SCRATCH_BYTES, SEG_ERR_WORKSPACE,
              "the backward needs %zu bytes of workspace, above the %zu-byte fixed scratch of "
              "seg_attn_bwd_noalloc (use seg_attn_bwd with a workspace)",
              need, (size_t)SEG_ATTN_BWD_SCRATCH_BYTES);
    if (sz->num_qtiles == 0) return;
    ptr = scratch_on_current_device();
  });
  if (st != SEG_OK) return st;
  return seg_attn_bwd(L, sz, dt, hq, hkv, d, softmax_scale, q, k, v, o, lse, d_o, dq, dk, dv, ptr,
                      SEG_ATTN_BWD_SCRATCH_BYTES, stream);
}
