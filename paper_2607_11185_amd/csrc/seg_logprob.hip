// Fused action-token log-prob and clipped policy-ratio loss with gradients
// (Eq. (loss) of App. E: min(rho A, clip(rho, 1 - eps_l, 1 + eps_h) A) over the
// trained action tokens, rho = pi_theta / pi_rollout), bf16 MFMA on gfx950.
//
// Only the R action rows are projected onto the vocabulary.  Pipeline:
//   1. zT[v][r] = s * W[v] . h[r] (MFMA, fp32 out) with a fused epilogue that
//      writes per-(row, 128-vocab tile) max / sum-exp partials and captures the
//      target logit;
//   2. per row: LSE from the partials (fixed order), logp, rho, loss, the
//      clipped flag and g = d loss_sum / d logp;
//   3. dzT = g * (onehot(target) - softmax(z))^T as bf16 (one pass over zT);
//   4. dH = s * dz W and dW = s * dz^T h (MFMA).
// All products use the shared kernel of gemm.h, which reads each operand in
// the orientation it has: dzT [V][R] serves dH (contracting over its rows)
// and dW (contracting along them), W and h serve as they are.
#include <climits>
#include <cmath>

#include "common.h"
#include "gemm.h"

namespace seg {
namespace {

using gemm::EpiOut;
using gemm::ST;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// Epilogue of the logits GEMM (M = vocab, N = rows): writes zT, captures the
// target logit and the per-(row, vocab tile) max / sum-exp partials.
struct EpiLogits {
  float *zt;        // [M][ldz] fp32, or NULL (a forward-only call needs the statistics alone)
  long ldz;
  float2 *stats;    // [ceil(M/128) slabs][N]: (max, sum exp(z - max)) in log2 units
  int nrows;        // N
  const int32_t *target;  // [N]
  float *ztgt;      // [N]
  float scale;
  // zT is larger than the 256 MB last-level cache: its stores go past the
  // caches (a smaller one's stay, for the pass over it that follows: 1,024 x
  // 32,000, 46 us with them in the cache, 52 without)
  bool stream;
  static constexpr bool kSwap = false;
  // A lane holds 32 of the 128 vocabulary rows of one column n (three other
  // lanes the rest), so maximum, exponentials and sum mostly stay in the lane;
  // a wave covers one 128-row slab.  Only the slab that the vocabulary ends in
  // tests its rows, and only waves that hold a target look for it.  The
  // exponents come from the logits as they are stored, scaled and rounded first:
  // scale * log2(e) as one rounded factor moved every exponent of a row the same
  // way, up to 6e-8 of the logit (log-probs up to 1.7 times further off).
  template <int NI, int NJ>
  __device__ __forceinline__ void operator()(const f32x4 (&acc)[NI][NJ],
                                             const gemm::Tile &t) const {
    static_assert(NI == 8, "logits epilogue expects 128-row wave tiles");
    const int slab_row = t.m0 + t.wr;
    if (slab_row >= t.M) return;
    if (zt) {
      // 16 rows x 64 columns at a time through the wave's LDS: column c of row
      // r in place c ^ 16 (r / 4), stored 16 bytes a lane, 256 to a row (4
      // bytes a lane, 64 to a row: 7.3 ms for 7,680 rows x 3,584 x 151,936; so
      // 6.8, past the caches 6.6)
      float *w = reinterpret_cast<float *>(t.lds);
      const int lane = t.grp * 16 + t.col, n = t.n0 + t.wc + t.col * 4;
      float *zp = zt + (long)slab_row * ldz + n;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            w[(4 * t.grp + r) * 64 + ((16 * j + t.col) ^ (16 * t.grp))] = acc[i][j][r] * scale;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          const int rr = p * 4 + t.grp, row = 16 * i + rr;
          const f32x4 v = *reinterpret_cast<const f32x4 *>(w + rr * 64 + ((4 * t.col) ^ (16 * p)));
          if (n < ldz && slab_row + row < t.M) {
            f32x4 *d = reinterpret_cast<f32x4 *>(zp + (long)row * ldz);
            if (stream) __builtin_nontemporal_store(v, d);
            else *d = v;
          }
        }
        __builtin_amdgcn_wave_barrier();
      }
    }
    if (slab_row + 128 <= t.M) slab<true>(acc, t, slab_row);
    else slab<false>(acc, t, slab_row);
  }
  template <bool WHOLE, int NI, int NJ>
  __device__ __forceinline__ void slab(const f32x4 (&acc)[NI][NJ], const gemm::Tile &t,
                                       int slab_row) const {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = t.n0 + t.wc + j * 16 + t.col;
      const bool nok = n < t.N;
      // the lane's rows are base + k, k = 16 i + r
      const int base = slab_row + 4 * t.grp, left = t.M - base;
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int k = 16 * i + r;
          const float z = acc[i][j][r] * scale;
          if (WHOLE || k < left) mx = fmaxf(mx, z);
        }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      const float mx2 = mx * LOG2E;
      float sm = 0.f;
      if (mx != -INFINITY) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (WHOLE || 16 * i + r < left)
              sm += __builtin_amdgcn_exp2f(fmaf(acc[i][j][r] * scale, LOG2E, -mx2));
      }
      sm += __shfl_xor(sm, 16, 64);
      sm += __shfl_xor(sm, 32, 64);
      if (t.grp == 0 && nok) stats[(long)(slab_row / 128) * nrows + n] = make_float2(mx2, sm);
      const int at = (nok ? target[n] : -1) - base;  // the target as a k of the lane
      const bool mine = at >= 0 && at < min(116, left) && !(at & 12);
      if (__any(mine)) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (mine && at == 16 * i + r) ztgt[n] = acc[i][j][r] * scale;
      }
    }
  }
};

// The row statistics and the loss of LOSS_ROWS rows per block.  16 threads
// share a row, each taking every 16th slab, so a block reads 128-byte pieces
// of the slab-major statistics (one block per row read 8 of every 64 bytes: 89
// us for 7,680 rows x 1,187 slabs, now 26); their results are combined
// in a fixed order.
constexpr int LOSS_ROWS = 16;

__global__ void __launch_bounds__(256) k_row_loss(
    const float2 *__restrict__ stats, int ntiles, int rows, const float *__restrict__ ztgt,
    const float *__restrict__ old_logp, const float *__restrict__ ref_logp,
    const float *__restrict__ adv, const int32_t *__restrict__ row_traj, int num_traj,
    seg_loss_cfg cfg, float *__restrict__ logp, float *__restrict__ loss_tok,
    uint8_t *__restrict__ clipped, float *__restrict__ kl_tok, float *__restrict__ lse_out,
    float *__restrict__ g_out) {
  constexpr int SL = 256 / LOSS_ROWS;
  __shared__ float2 red[SL][LOSS_ROWS];
  const int t = threadIdx.x % LOSS_ROWS, part = threadIdx.x / LOSS_ROWS;
  const int r = blockIdx.x * LOSS_ROWS + t;
  float mx = -INFINITY, sm = 0.f;
  if (r < rows) {
#pragma unroll 4
    for (int i = part; i < ntiles; i += SL) {
      const float2 p = stats[(long)i * rows + r];
      const float m2 = fmaxf(mx, p.x);
      // (an all -inf slab, or no slab yet, adds nothing)
      sm = (mx == -INFINITY ? 0.f : sm * exp2f(mx - m2)) + (p.x == -INFINITY ? 0.f : p.y * exp2f(p.x - m2));
      mx = m2;
    }
  }
  red[part][t] = make_float2(mx, sm);
  __syncthreads();
  if (part == 0 && r < rows) {
    for (int k = 1; k < SL; ++k) {
      const float2 p = red[k][t];
      const float m2 = fmaxf(mx, p.x);
      sm = (mx == -INFINITY ? 0.f : sm * exp2f(mx - m2)) + (p.x == -INFINITY ? 0.f : p.y * exp2f(p.x - m2));
      mx = m2;
    }
    const float lse = (mx + log2f(sm)) * LN2;
    const float lp = ztgt[r] - lse;
    // an out-of-range trajectory index yields NaN rather than a stray read
    const int tj = row_traj[r];
    const float A = (tj >= 0 && tj < num_traj) ? adv[tj] : __builtin_nanf("");
    const float rho = expf(lp - old_logp[r]);
    const float lo = 1.f - cfg.eps_low, hi = 1.f + cfg.eps_high;
    const float unc = rho * A;
    const float clp = fminf(fmaxf(rho, lo), hi) * A;
    float obj = fminf(unc, clp);
    bool cl = (A > 0.f && rho > hi) || (A < 0.f && rho < lo);
    if (cfg.dual_clip_c > 0.f && A < 0.f) {
      obj = fmaxf(obj, cfg.dual_clip_c * A);
      cl = cl || rho > cfg.dual_clip_c;
    }
    // KL(pi_theta || pi_ref) per token: e^x - x - 1 with x = ref - logp,
    // written expm1(x) - x (no cancellation for small x); its logp
    // derivative is 1 - e^x = -expm1(x)
    float kl = 0.f, dkl = 0.f;
    if (ref_logp) {
      const float x = ref_logp[r] - lp, em1 = expm1f(x);
      kl = em1 - x;
      dkl = -em1;
    }
    logp[r] = lp;
    loss_tok[r] = -obj + cfg.kl_coef * kl;
    clipped[r] = cl ? 1 : 0;
    if (kl_tok) kl_tok[r] = kl;
    lse_out[r] = lse;
    g_out[r] = (cl ? 0.f : -cfg.loss_scale * rho * A) + cfg.loss_scale * cfg.kl_coef * dkl;
  }
}

// loss_sum = loss_scale * sum(loss_tok), fixed-order reduction by one block of
// 256 threads.
__device__ __forceinline__ void loss_sum_block(const float *__restrict__ loss_tok, int rows,
                                               float scale, float *__restrict__ out) {
  __shared__ double red[256];
  const int t = threadIdx.x;
  double s = 0.0;
#pragma unroll 8
  for (int i = t; i < rows; i += 256) s += (double)loss_tok[i];
  red[t] = s;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (t < o) red[t] += red[t + o];
    __syncthreads();
  }
  if (t == 0) *out = (float)(red[0] * (double)scale);
}

__global__ void __launch_bounds__(256) k_loss_sum(const float *__restrict__ loss_tok, int rows,
                                                  float scale, float *__restrict__ out) {
  loss_sum_block(loss_tok, rows, scale, out);
}

// dzT = g[r] * (onehot(target[r]) - exp(z - lse[r])) from zT [V][Rp] to bf16
// [V][Rp], zero in the padded columns.  Bound by HBM (6 bytes an element):
// a thread keeps lse, g and target of its 8 columns in registers and walks
// down the vocabulary rows of its block with 16-byte accesses.  One more row of
// the grid's blocks has its first block form loss_sum.
constexpr int DZ_COLS = 256;  // of a block of 256 threads

// Vocabulary rows per block: about 1,024 blocks, and no longer ones than
// hide the loads of lse, g and target (7,680 rows x 151,936: 1.86 ms with 32
// rows, 1.34 with 64, 1.31 with 256; 1,024 x 32,000: 70 us with 24, 45 with
// 64).
inline int dz_rows(int V, int Rp) {
  const long r = (long)V * ((Rp + DZ_COLS - 1) / DZ_COLS) / 1024 / 8 * 8;
  return (int)std::min<long>(128, std::max<long>(8, r));
}

__global__ void __launch_bounds__(256) k_dz(const float *__restrict__ zt, int V, int R, int Rp, int vrows,
                                            const float *__restrict__ lse,
                                            const float *__restrict__ g,
                                            const int32_t *__restrict__ target,
                                            unsigned short *__restrict__ dzt,
                                            const float *__restrict__ loss_tok, float loss_scale,
                                            float *__restrict__ loss_sum) {
  if (blockIdx.y == gridDim.y - 1) {
    if (blockIdx.x == 0) loss_sum_block(loss_tok, R, loss_scale, loss_sum);
    return;
  }
  const int r0 = blockIdx.x * DZ_COLS + (threadIdx.x & 31) * 8;
  if (r0 >= Rp) return;  // Rp is a multiple of 32
  float l[8], gr[8];
  int tg[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const bool ok = r0 + j < R;
    l[j] = ok ? lse[r0 + j] : 0.f;
    gr[j] = ok ? g[r0 + j] : 0.f;
    tg[j] = ok ? target[r0 + j] : -1;
  }
  const int v1 = min(V, (int)(blockIdx.y + 1) * vrows);
#pragma unroll 4
  for (int v = blockIdx.y * vrows + (threadIdx.x >> 5); v < v1; v += 8) {
    const f32x4 *src = reinterpret_cast<const f32x4 *>(zt + (long)v * Rp + r0);
    const f32x4 a = src[0], b = src[1];
    u16x8 o;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float z = j < 4 ? a[j] : b[j - 4];
      // (x log2(e) rounded once in front of the hardware exponential is 16
      // times further from e^x at x = -12 and no faster at 7,680 rows x 151,936:
      // 1.30 against 1.31 ms; 49 against 51 us at 1,024 x 32,000)
      const float p = expf(z - l[j]);
      o[j] = r0 + j < R ? f2bf_bits(gr[j] * ((v == tg[j] ? 1.f : 0.f) - p)) : 0;
    }
    *reinterpret_cast<u16x8 *>(dzt + (long)v * Rp + r0) = o;
  }
}

// Preparation of a call in one launch: the gathered action rows as bf16
// (y[r] = h[rowmap[r]], zero from `rows` to rows_pad), for fp32 inputs the
// projection as bf16 (wb), and NaN in the target logits (a target outside the
// vocabulary keeps it).  8 elements a thread where `vec` (the tensors start on
// 16-byte boundaries; cols is a multiple of 8), else one by one.
template <class TI>
__device__ __forceinline__ u16x8 load8(const TI *p, bool vec) {
  u16x8 r;
  if (vec && sizeof(TI) == 2) return *reinterpret_cast<const u16x8 *>(p);
  if (vec) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(p), b = *reinterpret_cast<const f32x4 *>(p + 4);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      r[j] = f2bf_bits(a[j]);
      r[4 + j] = f2bf_bits(b[j]);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) r[j] = load_bf(p, j);
  }
  return r;
}

template <class TI>
__global__ void __launch_bounds__(256) k_lp_prep(const TI *__restrict__ h,
                                                 const int32_t *__restrict__ rowmap, int rows,
                                                 int rows_pad, int cols, bool hvec,
                                                 unsigned short *__restrict__ y,
                                                 const TI *__restrict__ w, long w8, bool wvec,
                                                 unsigned short *__restrict__ wb,
                                                 float *__restrict__ ztgt) {
  const unsigned c8 = cols / 8;
  const long n = (long)rows_pad * c8, step = (long)gridDim.x * 256;
  const long at = (long)blockIdx.x * 256 + threadIdx.x;
  for (long i = at; i < rows_pad; i += step) ztgt[i] = __builtin_nanf("");
  for (long i = at; i < n; i += step) {
    const int r = n >> 32 ? (int)(i / c8) : (int)((unsigned)i / c8);
    const long c = i - (long)r * c8;
    u16x8 v = u16x8{0, 0, 0, 0, 0, 0, 0, 0};
    if (r < rows) v = load8(h + (long)(rowmap ? rowmap[r] : r) * cols + c * 8, hvec);
    *reinterpret_cast<u16x8 *>(y + i * 8) = v;
  }
  if constexpr (sizeof(TI) == 4) {
    for (long i = at; i < w8; i += step)
      *reinterpret_cast<u16x8 *>(wb + i * 8) = load8(w + i * 8, wvec);
  }
}

struct LpWs {
  size_t hb, wb, zt, stats, ztgt, lse, g, dzt, total;
  int Rp, ntiles;
};

LpWs lp_ws(int rows, int hidden, int vocab, seg_dtype dt) {
  LpWs w{};
  w.Rp = (rows + 31) / 32 * 32;
  w.ntiles = (vocab + 127) / 128;  // 128-row slabs of the logits epilogue
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + std::max<size_t>(bytes, 1));
    return o;
  };
  const size_t Rp = w.Rp, H = hidden;
  w.hb = take(Rp * H * 2);
  w.wb = dt == SEG_F32 ? take((size_t)vocab * H * 2) : 0;
  w.zt = take((size_t)vocab * Rp * 4);
  w.stats = take((size_t)w.ntiles * std::max(rows, 1) * sizeof(float2));
  w.ztgt = take(Rp * 4);
  w.lse = take(Rp * 4);
  w.g = take(Rp * 4);
  w.dzt = take((size_t)vocab * Rp * 2);
  w.total = off;
  return w;
}

template <class TI, class TO>
void logprob_impl(int rows, int H, int V, const TI *h, const int32_t *row_index, const TI *w,
                  const int32_t *target, const float *old_logp, const float *ref_logp,
                  const float *adv, const int32_t *row_traj, int num_traj,
                  const seg_loss_cfg &cfg, float *logp, float *loss_tok, uint8_t *clipped,
                  float *kl_tok, float *loss_sum, void *dh, float *dw, char *base,
                  const LpWs &L, hipStream_t st) {
  const int Rp = L.Rp;
  unsigned short *hb = reinterpret_cast<unsigned short *>(base + L.hb);
  float *zt = reinterpret_cast<float *>(base + L.zt);
  float2 *stats = reinterpret_cast<float2 *>(base + L.stats);
  float *ztgt = reinterpret_cast<float *>(base + L.ztgt);
  float *lse = reinterpret_cast<float *>(base + L.lse);
  float *g = reinterpret_cast<float *>(base + L.g);
  unsigned short *dzt = reinterpret_cast<unsigned short *>(base + L.dzt);

  const unsigned short *wb;
  {
    unsigned short *w2 = sizeof(TI) == 4 ? reinterpret_cast<unsigned short *>(base + L.wb) : nullptr;
    const long n8 = (long)Rp * (H / 8), w8 = sizeof(TI) == 4 ? (long)V * (H / 8) : 0;
    auto vec = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
    ProfScope prof("lp_prep", st);
    k_lp_prep<TI><<<(int)std::min<long>(16384, (std::max(n8, w8) + 255) / 256), 256, 0, st>>>(
        h, row_index, rows, Rp, H, vec(h), hb, w, w8, vec(w), w2, ztgt);
    SEG_LAUNCH_CHECK();
    wb = w2 ? w2 : reinterpret_cast<const unsigned short *>(w);
  }
  // 1. logits zT = s * W h^T with partial softmax stats; the target logit
  //    stays NaN for a target outside [0, vocab)
  {
    EpiLogits e{cfg.want_grad ? zt : nullptr, Rp, stats, rows, target, ztgt, cfg.logit_scale,
                (long)V * Rp * 4 > (256L << 20)};
    ProfScope prof("logits", st);
    gemm::Problems<EpiLogits, 1, 1> g{{{wb}}, {{hb}}, {{H}}, {{H}}, {H}, {V}, {rows}, {e}, {}, 1,
                                      (H + gemm::BK - 1) / gemm::BK};
    gemm::launch_tm<false, false, 4>(g, st);
  }
  // 2. per-row loss
  {
  ProfScope prof("row_loss", st);
  k_row_loss<<<(rows + LOSS_ROWS - 1) / LOSS_ROWS, 256, 0, st>>>(stats, L.ntiles, rows, ztgt, old_logp, ref_logp, adv, row_traj,
                                   num_traj, cfg, logp, loss_tok, clipped, kl_tok, lse, g);
  SEG_LAUNCH_CHECK();
  if (!cfg.want_grad) {
    k_loss_sum<<<1, 256, 0, st>>>(loss_tok, rows, cfg.loss_scale, loss_sum);
    SEG_LAUNCH_CHECK();
    return;
  }
  }
  // 3. dz
  {
    ProfScope prof("dz", st);
    const int vr = dz_rows(V, Rp);
    k_dz<<<dim3((Rp + DZ_COLS - 1) / DZ_COLS, (V + vr - 1) / vr + 1), 256, 0, st>>>(
        zt, V, rows, Rp, vr, lse, g, target, dzt, loss_tok, cfg.loss_scale, loss_sum);
    SEG_LAUNCH_CHECK();
  }
  // 4. dH = s * dz W: A = dz^T [V][Rp], B = W [V][H], contracting over the
  //    vocabulary rows of both
  {
    ProfScope prof("dh", st);
    // zT has served: its place holds partial sums when the vocabulary is cut
    gemm::launch_one<true, true>(dzt, Rp, wb, H, rows, H, V,
                                 EpiOut<TO, ST>::make(static_cast<TO *>(dh), H, cfg.logit_scale),
                                 gemm::Scratch{zt, (long)V * Rp}, 0, st);
  }
  //    dW = s * dz^T h: A = dz^T along its rows (zero in the padded columns),
  //    B = h [Rp][H] (zero in the padded rows)
  {
    ProfScope prof("dw", st);
    gemm::launch_one<false, true>(dzt, Rp, hb, H, V, H, Rp,
                                  EpiOut<float, ST>::make(dw, H, cfg.logit_scale), st);
  }
}

}  // namespace
}  // namespace seg

using namespace seg;

extern "C" size_t seg_logprob_workspace_bytes(int32_t rows, int32_t hidden, int32_t vocab,
                                              seg_dtype dt) {
  if (rows < 0 || hidden < 1 || vocab < 1) return 0;
  return lp_ws(rows, hidden, vocab, dt).total;
}

extern "C" seg_status seg_logprob_loss(int32_t rows, int32_t hidden, int32_t vocab, seg_dtype dt,
                                       const void *h, const int32_t *row_index, const void *w,
                                       const int32_t *target, const float *old_logp,
                                       const float *ref_logp, const float *adv,
                                       const int32_t *row_traj, int32_t num_traj,
                                       const seg_loss_cfg *cfg, float *logp, float *loss_tok,
                                       uint8_t *clipped, float *kl_tok, float *loss_sum,
                                       void *dh, float *dw, void *ws, size_t ws_bytes,
                                       hipStream_t stream) {
  return guarded([&] {
    SEG_CHECK(cfg != nullptr, SEG_ERR_ARG, "cfg is NULL");
    SEG_CHECK(dt == SEG_BF16 || dt == SEG_F32, SEG_ERR_ARG, "unknown dtype %d", (int)dt);
    SEG_CHECK(rows >= 0 && hidden >= 1 && vocab >= 1 && num_traj >= 0, SEG_ERR_ARG,
              "bad sizes rows=%d hidden=%d vocab=%d num_traj=%d", rows, hidden, vocab, num_traj);
    SEG_CHECK(hidden % 8 == 0, SEG_ERR_UNSUPPORTED, "hidden %d must be a multiple of 8", hidden);
    // GEMM operand rows (hidden, padded vocab, padded rows) are addressed with
    // 32-bit offsets inside a 256-row block
    SEG_CHECK(hidden <= (1 << 20) && vocab <= (1 << 20) - 256 && rows <= (1 << 20) - 256,
              SEG_ERR_CAPACITY, "rows %d, hidden %d or vocab %d above 2^20", rows, hidden, vocab);
    SEG_CHECK(std::isfinite(cfg->eps_low) && std::isfinite(cfg->eps_high) &&
                  std::isfinite(cfg->loss_scale) && std::isfinite(cfg->logit_scale) &&
                  std::isfinite(cfg->dual_clip_c) && std::isfinite(cfg->kl_coef),
              SEG_ERR_ARG, "non-finite loss setting");
    SEG_CHECK(cfg->eps_low >= 0.f && cfg->eps_high >= 0.f, SEG_ERR_ARG, "negative clip range");
    SEG_CHECK(cfg->kl_coef >= 0.f, SEG_ERR_ARG, "negative kl_coef");
    SEG_CHECK(cfg->kl_coef == 0.f || ref_logp != nullptr, SEG_ERR_ARG,
              "kl_coef > 0 needs ref_logp");
    const LpWs L = lp_ws(rows, hidden, vocab, dt);
    SEG_CHECK(ws_bytes >= L.total, SEG_ERR_WORKSPACE, "workspace of %zu bytes < required %zu",
              ws_bytes, L.total);
    SEG_CHECK(loss_sum != nullptr, SEG_ERR_ARG, "loss_sum is NULL");
    if (rows == 0) {
      fill32(loss_sum, 1, 0u, stream);
      if (cfg->want_grad && dw) fill32(dw, (long)vocab * hidden, 0u, stream);
      return;
    }
    SEG_CHECK(h && w && target && old_logp && adv && row_traj && logp && loss_tok && clipped && ws,
              SEG_ERR_ARG, "a tensor pointer is NULL");
    SEG_CHECK(num_traj >= 1, SEG_ERR_ARG, "num_traj must be >= 1 when rows > 0");
    if (cfg->want_grad) SEG_CHECK(dh && dw, SEG_ERR_ARG, "dh/dw is NULL with want_grad");
    char *base = static_cast<char *>(ws);
    if (dt == SEG_F32)
      logprob_impl<float, float>(rows, hidden, vocab, static_cast<const float *>(h), row_index,
                                 static_cast<const float *>(w), target, old_logp, ref_logp, adv,
                                 row_traj, num_traj, *cfg, logp, loss_tok, clipped, kl_tok,
                                 loss_sum, dh, dw, base, L, stream);
    else
      logprob_impl<unsigned short, unsigned short>(
          rows, hidden, vocab, static_cast<const unsigned short *>(h), row_index,
          static_cast<const unsigned short *>(w), target, old_logp, ref_logp, adv, row_traj,
          num_traj, *cfg, logp, loss_tok, clipped, kl_tok, loss_sum, dh, dw, base, L, stream);
  });
}
