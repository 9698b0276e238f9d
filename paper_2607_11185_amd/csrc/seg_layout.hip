// Segmentation and packed layout of Visual Context Segmentation training items
// (Sec. 3.3; App. D, Alg. "Sliding-window trajectory processing with token-ID
// stream"), read with a sliding window of W screenshots and L-turn segments.
//
// Host part (seg_layout_query and the first half of seg_build_layout): cut each
// trajectory's turns into segments and pack them, O(turns) arithmetic on the
// span lists; for a build also four numbers per tile (its first and last turn,
// its keys' earliest and latest expiry), the CSR pointers and visible-pair
// counts that follow from them, and the attention kernels' launch schedule.
// Device part, one kernel: expand these tables into per-token descriptors, the
// loss rows, and the 128x128 block-sparse tile map with its transposed CSR.
#include <algorithm>
#include <climits>
#include <cstring>
#include <string>
#include <vector>

#include "common.h"

namespace seg {

static thread_local std::string g_err;
void set_error(const std::string &m) { g_err = m; }
void clear_error() { g_err.clear(); }

namespace {

// One contiguous run of tokens of a segment (a prompt, screenshot or text block).
struct Piece {
  int32_t off;    // segment-relative position of its first token
  int32_t canon;  // canonical index of its first token
  int32_t len;
  int32_t meta;   // turn << 2 | kind
};

// A run of trained action tokens (the tail of one turn's text block).
struct LossPiece {
  int32_t row_base;  // first loss row
  int32_t pos;       // packed row of the first action token
  int32_t canon;     // canonical index of the first action token
  int32_t traj;
};

// Per-segment record used by the kernels (device copy lives in the workspace).
struct DevSeg {
  int32_t start, len, qbase;
  int32_t piece_base, piece_count;
};

// What decides the class of a tile pair (see tile_class): turns of the tile's
// first and last row, earliest and latest turn at which one of its keys
// expires (INT32_MAX: never).
struct TileSpan {
  int32_t first_turn, last_turn, min_exp, max_exp;
};

struct Plan {
  seg_sizes sz{};
  std::vector<int32_t> seg_info;  // [S*8]
  std::vector<DevSeg> dsegs;
  std::vector<Piece> pieces;
  std::vector<LossPiece> lpieces;
  // of a build only (plan_tiles)
  std::vector<TileSpan> spans;          // [G]
  std::vector<int32_t> qt_ptr, kt_ptr;  // [G+1]
  std::vector<int64_t> seg_pairs;       // [S]
  // launch schedule of the attention kernels (see seg_layout)
  int32_t xcd_rows[9] = {}, xcd_cols[9] = {};
};

// Spans of every tile of one segment and its listed partners, from its token
// runs.  Turns never decrease along a segment, so a q-tile's most permissive
// row is its first one; a k-tile's most permissive key is the one that expires
// last (text and prompt never do, a screenshot of turn s at turn s + Wv).  An
// off-diagonal pair (q-tile i > k-tile j) holds a visible pair iff the first
// row's turn of i is below the latest expiry in j, so k-tile j is listed by the
// contiguous q-tiles j .. r_j - 1 (the diagonal always).
void tile_work(const Piece *pc, int npc, int len, int tile, int Wv, TileSpan *sp, int32_t *row_w,
               int32_t *col_w) {
  // 64-bit: any tile edge up to 2^31 - 1 is taken, so len + tile may pass it
  const int n = (int)(((int64_t)len + tile - 1) / tile);
  int k = 0;
  for (int t = 0; t < n; ++t) {
    const int64_t r0 = (int64_t)t * tile, r1 = std::min<int64_t>(len, r0 + tile);
    while (k + 1 < npc && pc[k + 1].off <= r0) ++k;
    TileSpan d{pc[k].meta >> 2, 0, INT32_MAX, INT32_MIN};
    for (int i = k; i < npc && pc[i].off < r1; ++i) {
      if (pc[i].len == 0 || pc[i].off + pc[i].len <= r0) continue;
      const int kind = pc[i].meta & 3;
      const int64_t e = kind == SEG_KIND_IMAGE ? (int64_t)(pc[i].meta >> 2) + Wv : INT32_MAX;
      d.min_exp = (int32_t)std::min<int64_t>(d.min_exp, e);
      d.max_exp = (int32_t)std::max<int64_t>(d.max_exp, std::min<int64_t>(e, INT32_MAX));
      d.last_turn = pc[i].meta >> 2;
    }
    sp[t] = d;
  }
  std::fill(row_w, row_w + n, 0);
  for (int j = 0; j < n; ++j) {
    // first q-tile after j whose first row's turn has reached the expiry
    const int r = (int)(std::lower_bound(sp + j + 1, sp + n, sp[j].max_exp,
                                         [](const TileSpan &x, int32_t e) { return x.first_turn < e; }) -
                        sp);
    col_w[j] = r - j;
    if (j + 1 < n) ++row_w[j + 1];
    if (r < n) --row_w[r];
  }
  int run = 0;
  for (int i = 0; i < n; ++i) {
    run += row_w[i];
    row_w[i] = 1 + run;
  }
}

// Visible pairs of one segment: every row sees the rows up to itself, except
// the screenshots of turns more than Wv - 1 before its own.
int64_t count_pairs(const Piece *pc, int npc, int64_t len, int Wv) {
  int64_t n = len * (len + 1) / 2;
  int f = 0;  // first run of a turn that no longer sees run i
  for (int i = 0; i < npc; ++i) {
    if ((pc[i].meta & 3) != SEG_KIND_IMAGE) continue;
    while (f < npc && (pc[f].meta >> 2) < (int64_t)(pc[i].meta >> 2) + Wv) ++f;
    if (f < npc) n -= (int64_t)pc[i].len * (len - pc[f].off);
  }
  return n;
}

// Boundaries of eight consecutive tile ranges with about equal total work.
void balance8(const std::vector<int32_t> &w, int32_t *b) {
  const int G = (int)w.size();
  std::vector<int64_t> pre(G + 1, 0);
  for (int g = 0; g < G; ++g) pre[g + 1] = pre[g] + w[g];
  b[0] = 0;
  for (int x = 1; x < 8; ++x) {
    const int64_t target = (pre[G] * x + 7) / 8;
    b[x] = (int32_t)(std::lower_bound(pre.begin(), pre.end(), target) - pre.begin());
    b[x] = std::max(b[x], b[x - 1]);
  }
  b[8] = G;
}

// Byte offsets of the build workspace: the host tables, the token runs last.
struct BuildWs {
  size_t dseg, lpiece, info, span, qptr, kptr, pairs, piece, total;
};

// token runs larger than this are uploaded from where they were made (4 x 1,000 turns,
// 4.2 MB of runs: 1.49 ms a build gathered, 1.38 apart; 0.7 MB: 242 us either way; 0.25
// MB: 110 against 116)
constexpr size_t PIECES_APART = 1 << 20;

BuildWs build_ws_layout(const seg_sizes &sz, size_t npieces, size_t nlpieces) {
  BuildWs w{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  const size_t S = sz.num_segments, G = sz.num_qtiles;
  w.dseg = take(sizeof(DevSeg) * std::max<size_t>(1, S));
  w.lpiece = take(sizeof(LossPiece) * std::max<size_t>(1, nlpieces));
  w.info = take(sizeof(int32_t) * SEG_INFO_FIELDS * std::max<size_t>(1, S));
  w.span = take(sizeof(TileSpan) * std::max<size_t>(1, G));
  w.qptr = take(sizeof(int32_t) * (G + 1));
  w.kptr = take(sizeof(int32_t) * (G + 1));
  w.pairs = take(sizeof(int64_t) * std::max<size_t>(1, S));
  w.piece = take(sizeof(Piece) * std::max<size_t>(1, npieces));
  w.total = off;
  return w;
}

// Tokens of segment [a, b) of a trajectory: prompt + text of turns < b +
// screenshots of turns j with max(1, a - W + 1) <= j < b (turns 1-based).
int64_t seg_len(const int32_t *img, const int32_t *text, int64_t p, int W, int a, int b) {
  int64_t n = p;
  int lo = std::max(1, a - W + 1);
  for (int j = 1; j < b; ++j) {
    n += text[j - 1];
    if (j >= lo) n += img[j - 1];
  }
  return n;
}

void validate(const seg_problem *p) {
  SEG_CHECK(p != nullptr, SEG_ERR_ARG, "problem is NULL");
  SEG_CHECK(p->num_traj >= 0, SEG_ERR_ARG, "num_traj < 0");
  SEG_CHECK(p->window >= 1, SEG_ERR_ARG, "window must be >= 1 (got %d)", p->window);
  SEG_CHECK(p->seg_steps >= 1, SEG_ERR_ARG, "seg_steps must be >= 1 (got %d)", p->seg_steps);
  SEG_CHECK(p->max_seg_tokens >= 0, SEG_ERR_ARG, "max_seg_tokens < 0");
  SEG_CHECK(p->buffer_tokens >= 0, SEG_ERR_ARG, "buffer_tokens < 0");
  SEG_CHECK(p->tile >= 1, SEG_ERR_ARG, "tile must be >= 1 (got %d)", p->tile);
  SEG_CHECK(p->mode == SEG_MODE_SLIDING || p->mode == SEG_MODE_ANCHORED, SEG_ERR_ARG,
            "unknown mode %d", p->mode);
  SEG_CHECK(p->mode == SEG_MODE_SLIDING || p->max_seg_tokens == 0, SEG_ERR_UNSUPPORTED,
            "the anchored mode has no token cap (max_seg_tokens must be 0)");
  SEG_CHECK(p->mode == SEG_MODE_SLIDING || p->window < (SEG_WINDOW_ANCHORED >> 1), SEG_ERR_ARG,
            "window too large");
  if (p->num_traj == 0) return;
  SEG_CHECK(p->step_offsets && p->prompt_len, SEG_ERR_ARG, "step_offsets/prompt_len is NULL");
  SEG_CHECK(p->step_offsets[0] == 0, SEG_ERR_ARG, "step_offsets[0] must be 0");
  for (int t = 0; t < p->num_traj; ++t) {
    SEG_CHECK(p->step_offsets[t + 1] >= p->step_offsets[t], SEG_ERR_ARG,
              "step_offsets must be non-decreasing (trajectory %d)", t);
    SEG_CHECK(p->prompt_len[t] >= 0, SEG_ERR_ARG, "prompt_len[%d] < 0", t);
  }
  int32_t ns = p->step_offsets[p->num_traj];
  if (ns > 0)
    SEG_CHECK(p->img_len && p->text_len && p->action_len, SEG_ERR_ARG,
              "img_len/text_len/action_len is NULL");
  for (int s = 0; s < ns; ++s) {
    SEG_CHECK(p->img_len[s] >= 0, SEG_ERR_ARG, "img_len[%d] < 0", s);
    SEG_CHECK(p->text_len[s] >= 0, SEG_ERR_ARG, "text_len[%d] < 0", s);
    SEG_CHECK(p->action_len[s] >= 0 && p->action_len[s] <= p->text_len[s], SEG_ERR_ARG,
              "action_len[%d] must be in [0, text_len]", s);
  }
}

Plan make_plan(const seg_problem *p) {
  validate(p);
  Plan pl;
  seg_sizes &sz = pl.sz;
  // Anchored mode: a segment keeps the K = window screenshots before its
  // first turn (K + 1 with its own), the first segment runs K + Delta turns
  // and later ones Delta = seg_steps (the count of the algorithm's trigger).
  const bool anchored = p->mode == SEG_MODE_ANCHORED;
  const int W = anchored ? p->window + 1 : p->window, L = p->seg_steps, tile = p->tile;
  const int L0 = anchored ? p->window + p->seg_steps : L;  // turns of a trajectory's first segment
  const int64_t cap = p->max_seg_tokens, B = p->buffer_tokens;
  sz.num_steps = p->num_traj ? p->step_offsets[p->num_traj] : 0;

  struct S0 {
    int traj, a, b;
    int64_t len;
  };
  std::vector<S0> segs;
  std::vector<int64_t> canon0(p->num_traj + 1, 0);
  for (int t = 0; t < p->num_traj; ++t) {
    const int s0 = p->step_offsets[t], T = p->step_offsets[t + 1] - s0;
    const int32_t *img = p->img_len + s0, *text = p->text_len + s0;
    const int64_t pr = p->prompt_len[t];
    int64_t tot = pr;
    for (int j = 0; j < T; ++j) tot += (int64_t)img[j] + text[j];
    canon0[t + 1] = canon0[t] + tot;
    int a = 1;
    while (a <= T) {
      int64_t one = seg_len(img, text, pr, W, a, a + 1);
      SEG_CHECK(!cap || one <= cap, SEG_ERR_CAPACITY,
                "trajectory %d turn %d alone needs %lld tokens > max_seg_tokens %lld", t, a,
                (long long)one, (long long)cap);
      int b = a + 1;
      const int La = a == 1 ? L0 : L;
      while (b - a < La && b <= T && (!cap || seg_len(img, text, pr, W, a, b + 1) <= cap)) ++b;
      int64_t n = seg_len(img, text, pr, W, a, b);
      SEG_CHECK(n >= 1, SEG_ERR_ARG, "segment of trajectory %d, turns %d..%d holds no token", t, a,
                b - 1);
      SEG_CHECK(!B || n <= B, SEG_ERR_CAPACITY,
                "segment of %lld tokens (trajectory %d, turns %d..%d) exceeds buffer_tokens %lld",
                (long long)n, t, a, b - 1, (long long)B);
      segs.push_back({t, a, b, n});
      a = b;
    }
  }
  sz.traj_tokens = canon0[p->num_traj];
  SEG_CHECK(sz.traj_tokens <= INT32_MAX, SEG_ERR_CAPACITY, "more than 2^31-1 canonical tokens");
  SEG_CHECK(segs.size() <= (size_t)INT32_MAX / SEG_INFO_FIELDS, SEG_ERR_CAPACITY, "too many segments");

  // packing
  int64_t pos = 0, fill = 0;
  int nbuf = 0;
  std::vector<int64_t> starts(segs.size());
  for (size_t i = 0; i < segs.size(); ++i) {
    if (B) {
      if (nbuf == 0 || fill + segs[i].len > B) {
        pos = (int64_t)nbuf * B;
        ++nbuf;
        fill = 0;
      }
      fill += segs[i].len;
    }
    starts[i] = pos;
    pos += segs[i].len;
  }
  int64_t packed = B ? (int64_t)nbuf * B : pos;
  if (!B) nbuf = segs.empty() ? 0 : 1;
  SEG_CHECK(packed <= INT32_MAX, SEG_ERR_CAPACITY, "packed buffer exceeds 2^31-1 rows");
  sz.packed_tokens = packed;
  sz.num_buffers = nbuf;
  sz.num_segments = (int32_t)segs.size();
  sz.max_seg_len = 0;
  for (const S0 &sg : segs) sz.max_seg_len = std::max(sz.max_seg_len, (int32_t)sg.len);

  // per-segment tables
  int64_t qbase = 0, tri = 0, rows = 0;
  for (size_t i = 0; i < segs.size(); ++i) {
    const S0 &sg = segs[i];
    const int s0 = p->step_offsets[sg.traj];
    const int32_t *img = p->img_len + s0, *text = p->text_len + s0, *act = p->action_len + s0;
    const int64_t nt = (sg.len + tile - 1) / tile;
    DevSeg d{};
    d.start = (int32_t)starts[i];
    d.len = (int32_t)sg.len;
    d.qbase = (int32_t)qbase;
    d.piece_base = (int32_t)pl.pieces.size();
    // pieces: prompt, then per turn j < b: screenshot if j > a - W, text
    int32_t off = 0, c = (int32_t)canon0[sg.traj];
    int32_t pr = p->prompt_len[sg.traj];
    pl.pieces.push_back({off, c, pr, SEG_KIND_PROMPT});
    off += pr;
    c += pr;
    int64_t loss_base = rows;
    for (int j = 1; j < sg.b; ++j) {
      int32_t m = img[j - 1], x = text[j - 1];
      if (j > sg.a - W && m > 0) {
        pl.pieces.push_back({off, c, m, (j << 2) | SEG_KIND_IMAGE});
        off += m;
      }
      c += m;
      if (x > 0) {
        if (j >= sg.a && act[j - 1] > 0) {
          int32_t na = act[j - 1];
          // the ratio of a token uses the row before it (Eq. loss): a trained
          // token cannot open its segment
          SEG_CHECK(off + x - na > 0, SEG_ERR_ARG,
                    "trajectory %d turn %d: a trained token is the first token of its segment "
                    "(no row predicts it)", sg.traj, j);
          pl.lpieces.push_back({(int32_t)rows, d.start + off + x - na, c + x - na, sg.traj});
          rows += na;
        }
        pl.pieces.push_back({off, c, x, (j << 2) | SEG_KIND_TEXT});
        off += x;
      }
      c += x;
    }
    d.piece_count = (int32_t)pl.pieces.size() - d.piece_base;
    pl.dsegs.push_back(d);
    int32_t info[SEG_INFO_FIELDS] = {sg.traj, sg.a, sg.b, d.start, d.len, d.qbase,
                                     (int32_t)loss_base, (int32_t)(rows - loss_base)};
    pl.seg_info.insert(pl.seg_info.end(), info, info + SEG_INFO_FIELDS);
    qbase += nt;
    tri += nt * (nt + 1) / 2;
    SEG_CHECK(qbase <= INT32_MAX && tri <= INT32_MAX && rows <= INT32_MAX, SEG_ERR_CAPACITY,
              "tile or loss-row count exceeds 2^31-1");
  }
  sz.num_qtiles = (int32_t)qbase;
  sz.tile_nnz_max = tri;
  sz.loss_rows = (int32_t)rows;
  sz.workspace_bytes = build_ws_layout(sz, pl.pieces.size(), pl.lpieces.size()).total;
  return pl;
}

// The per-tile part of a build: tile spans, CSR pointers, pair counts and the
// launch schedule (eight balanced tile ranges per pass).
void plan_tiles(const seg_problem *p, Plan &pl) {
  const int Wv = p->mode == SEG_MODE_ANCHORED ? SEG_WINDOW_ANCHORED : p->window;
  const size_t G = pl.sz.num_qtiles;
  std::vector<int32_t> row_work(G), col_work(G);
  pl.spans.resize(G);
  for (const DevSeg &d : pl.dsegs) {
    const Piece *pc = pl.pieces.data() + d.piece_base;
    tile_work(pc, d.piece_count, d.len, p->tile, Wv, pl.spans.data() + d.qbase,
              row_work.data() + d.qbase, col_work.data() + d.qbase);
    pl.seg_pairs.push_back(count_pairs(pc, d.piece_count, d.len, Wv));
  }
  auto scan = [](const std::vector<int32_t> &w, std::vector<int32_t> &ptr) {
    ptr.resize(w.size() + 1);
    ptr[0] = 0;
    for (size_t i = 0; i < w.size(); ++i) ptr[i + 1] = ptr[i] + w[i];
  };
  scan(row_work, pl.qt_ptr);
  scan(col_work, pl.kt_ptr);
  balance8(row_work, pl.xcd_rows);
  balance8(col_work, pl.xcd_cols);
}

// ------------------------------------------------------------------ kernels

// last index i in [0, n) with key(i) <= x (keys ascending); -1 if none
template <class F>
__device__ __forceinline__ int upper_index(int n, int x, F key) {
  int lo = 0, hi = n;  // answer in [lo-1, hi-1]
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (key(mid) <= x) lo = mid + 1;
    else hi = mid;
  }
  return lo - 1;
}

// Class of the pair (q-tile i, k-tile j <= i) of a segment; 0: no visible pair.
// Every row of a later tile is after every key, so the pair holds a visible
// one iff i's first row is before j's latest expiry, and is FULL iff i's last
// row is before j's earliest and i has all its rows.  A diagonal tile of more
// than one row holds pairs in both orders.
__device__ __forceinline__ int tile_class(const TileSpan &q, const TileSpan &k, bool diagonal,
                                          bool whole, int tile) {
  if (diagonal) return tile == 1 ? SEG_TILE_FULL : SEG_TILE_PARTIAL;
  if (q.first_turn >= k.max_exp) return 0;
  return whole && q.last_turn < k.min_exp ? SEG_TILE_FULL : SEG_TILE_PARTIAL;
}

struct BuildArgs {
  const DevSeg *segs;
  const Piece *pieces;
  const LossPiece *lp;
  const int32_t *info, *qptr, *kptr;
  const TileSpan *span;
  const int64_t *pairs;
  seg_layout out;
  int S, P, R, G, nlp, tile;
  int tok_blocks, loss_blocks, tile_blocks, copy_blocks;
};

constexpr int TOK_BLOCK = 1024;  // rows of a token block

// The whole layout in one launch; blocks of 256 threads take, in turn, runs of
// packed rows, runs of loss rows, four q-tiles (CSR rows), four k-tiles
// (transposed CSR) and runs of the tables that are copied.  Everything is a
// few MB at most, so latency bounds it: no pass over the result of another,
// and the class of a tile pair is two compares of its tiles' spans (tested key
// by key against the token descriptors it took 312 us of the 390 us that the
// 7B-class batch's build spent in nine kernels; this one takes 24 us).
__global__ void __launch_bounds__(256) k_build(const BuildArgs a) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int b = blockIdx.x;
  if (b < a.tok_blocks) {
    // the rows of a block mostly lie in one segment: search from there (the
    // end of the last block may lie past 2^31 - 1, so rows count from its first)
    const int first = b * TOK_BLOCK, n = min(TOK_BLOCK, a.P - first);
    const int s0 = max(0, upper_index(a.S, first, [&](int i) { return a.segs[i].start; }));
    for (int o = tid; o < n; o += 256) {
      const int r = first + o;
      int s = s0;
      while (s + 1 < a.S && a.segs[s + 1].start <= r) ++s;
      const DevSeg d = a.segs[s];
      int src = -1, meta = SEG_KIND_PAD;
      const int pos = r - d.start;
      if (pos >= 0 && pos < d.len) {
        const Piece *pc = a.pieces + d.piece_base;
        const Piece p = pc[upper_index(d.piece_count, pos, [&](int k) { return pc[k].off; })];
        src = p.canon + (pos - p.off);
        meta = p.meta;
      }
      a.out.tok_src[r] = src;
      a.out.tok_meta[r] = meta;
    }
    return;
  }
  b -= a.tok_blocks;
  if (b < a.loss_blocks) {
    const int r = b * 256 + tid;
    if (r < a.R) {
      const LossPiece l = a.lp[upper_index(a.nlp, r, [&](int k) { return a.lp[k].row_base; })];
      const int o = r - l.row_base;
      a.out.loss_pred_row[r] = l.pos + o - 1;
      a.out.loss_tgt_src[r] = l.canon + o;
      a.out.loss_traj[r] = l.traj;
    }
    return;
  }
  b -= a.loss_blocks;
  if (b < 2 * a.tile_blocks) {
    const bool cols = b >= a.tile_blocks;
    const int g = (cols ? b - a.tile_blocks : b) * 4 + wave;
    if (g >= a.G) return;
    const int s = upper_index(a.S, g, [&](int i) { return a.segs[i].qbase; });
    const DevSeg d = a.segs[s];
    const TileSpan *sp = a.span + d.qbase;
    const int me = g - d.qbase;
    const TileSpan mine = sp[me];
    const unsigned long long below = (1ull << lane) - 1;
    if (!cols) {
      // CSR row of q-tile `me`: k-tiles ascending; then the walking order of
      // the q-tile-stationary kernels: FULL tiles first and PARTIAL ones
      // after (each ascending), with bit 31 marking PARTIAL
      const bool whole = (long)(me + 1) * a.tile <= d.len;
      const int e0 = a.qptr[g];
      if (lane == 0) a.out.tile_seg[g] = s;
      int out = e0, nfull = 0;
      for (int j0 = 0; j0 <= me; j0 += 64) {
        const int j = j0 + lane;
        const int c = j <= me ? tile_class(mine, sp[j], j == me, whole, a.tile) : 0;
        const unsigned long long m = __ballot(c != 0);
        if (c) {
          const int at = out + __popcll(m & below);
          a.out.qt_col[at] = d.qbase + j;
          a.out.qt_cls[at] = (uint8_t)c;
        }
        out += __popcll(m);
        nfull += __popcll(__ballot(c == SEG_TILE_FULL));
      }
      int rf = 0, rp = 0;  // ranks so far within each class
      for (int j0 = 0; j0 <= me; j0 += 64) {
        const int j = j0 + lane;
        const int c = j <= me ? tile_class(mine, sp[j], j == me, whole, a.tile) : 0;
        const unsigned long long mf = __ballot(c == SEG_TILE_FULL), mp = __ballot(c == SEG_TILE_PARTIAL);
        if (c == SEG_TILE_FULL) a.out.qt_ord[e0 + rf + __popcll(mf & below)] = d.qbase + j;
        if (c == SEG_TILE_PARTIAL)
          a.out.qt_ord[e0 + nfull + rp + __popcll(mp & below)] =
              (int32_t)((unsigned)(d.qbase + j) | 0x80000000u);
        rf += __popcll(mf);
        rp += __popcll(mp);
      }
    } else {
      // transposed CSR of k-tile `me`: its listed q-tiles me .. me + n - 1,
      // ascending; then the walking order of the k-tile-stationary kernel:
      // FULL q-tiles first, then PARTIAL ones, each descending, with bit 31
      // marking PARTIAL
      const int e0 = a.kptr[g], n = a.kptr[g + 1] - e0;
      auto cls = [&](int k) {
        const int i = me + k;
        return k < n ? tile_class(sp[i], mine, k == 0, (long)(i + 1) * a.tile <= d.len, a.tile) : 0;
      };
      int nfull = 0;
      for (int k0 = 0; k0 < n; k0 += 64) {
        const int c = cls(k0 + lane);
        if (c) {
          a.out.kt_row[e0 + k0 + lane] = g + k0 + lane;
          a.out.kt_cls[e0 + k0 + lane] = (uint8_t)c;
        }
        nfull += __popcll(__ballot(c == SEG_TILE_FULL));
      }
      int rf = 0, rp = 0;  // ascending ranks so far within each class
      for (int k0 = 0; k0 < n; k0 += 64) {
        const int c = cls(k0 + lane);
        const unsigned long long mf = __ballot(c == SEG_TILE_FULL), mp = __ballot(c == SEG_TILE_PARTIAL);
        if (c == SEG_TILE_FULL) a.out.kt_ord[e0 + nfull - 1 - (rf + __popcll(mf & below))] = g + k0 + lane;
        if (c == SEG_TILE_PARTIAL)
          a.out.kt_ord[e0 + n - 1 - (rp + __popcll(mp & below))] =
              (int32_t)((unsigned)(g + k0 + lane) | 0x80000000u);
        rf += __popcll(mf);
        rp += __popcll(mp);
      }
    }
    return;
  }
  b -= 2 * a.tile_blocks;
  // (64-bit: an index steps past tables of up to 2^31 - 1 entries)
  for (long i = b * 256 + tid; i <= a.G; i += a.copy_blocks * 256) {
    a.out.qt_ptr[i] = a.qptr[i];
    a.out.kt_ptr[i] = a.kptr[i];
  }
  for (long i = b * 256 + tid; i < a.S * SEG_INFO_FIELDS; i += a.copy_blocks * 256)
    a.out.seg_info[i] = a.info[i];
  for (long i = b * 256 + tid; i < a.S; i += a.copy_blocks * 256) a.out.seg_pairs[i] = a.pairs[i];
  if (b == 0 && tid == 0) *a.out.tile_nnz = a.qptr[a.G];
}

}  // namespace
}  // namespace seg

using namespace seg;

extern "C" const char *seg_last_error(void) { return g_err.c_str(); }

extern "C" seg_status seg_layout_query(const seg_problem *p, seg_sizes *out) {
  return guarded([&] {
    SEG_CHECK(out != nullptr, SEG_ERR_ARG, "sizes output is NULL");
    Plan pl = make_plan(p);
    *out = pl.sz;
  });
}

extern "C" seg_status seg_build_layout(const seg_problem *p, const seg_sizes *sz, seg_layout *out,
                                       void *ws, size_t ws_bytes, hipStream_t stream) {
  return guarded([&] {
    SEG_CHECK(sz != nullptr && out != nullptr, SEG_ERR_ARG, "sizes or layout is NULL");
    Plan pl = make_plan(p);
    plan_tiles(p, pl);
    SEG_CHECK(std::memcmp(&pl.sz, sz, sizeof(seg_sizes)) == 0, SEG_ERR_ARG,
              "sizes do not match seg_layout_query of this problem");
    SEG_CHECK(ws_bytes >= sz->workspace_bytes, SEG_ERR_WORKSPACE,
              "workspace of %zu bytes < required %zu", ws_bytes, sz->workspace_bytes);
    // visibility window of the kernels: none inside an anchored segment
    const int Wv = p->mode == SEG_MODE_ANCHORED ? SEG_WINDOW_ANCHORED : p->window;
    out->window = Wv;
    out->tile = p->tile;
    std::memcpy(out->xcd_rows, pl.xcd_rows, sizeof(pl.xcd_rows));
    std::memcpy(out->xcd_cols, pl.xcd_cols, sizeof(pl.xcd_cols));
    const int S = sz->num_segments, G = sz->num_qtiles, R = sz->loss_rows;
    const int P = (int)sz->packed_tokens;
    if (S > 0) {
      SEG_CHECK(ws && out->seg_info && out->tok_src && out->tok_meta && out->tile_seg &&
                    out->qt_ptr && out->qt_col && out->qt_cls && out->qt_ord && out->kt_ptr &&
                    out->kt_row && out->kt_ord &&
                    out->kt_cls && out->seg_pairs && out->tile_nnz,
                SEG_ERR_ARG, "a layout array is NULL");
      SEG_CHECK(R == 0 || (out->loss_pred_row && out->loss_tgt_src && out->loss_traj),
                SEG_ERR_ARG, "a loss-row array is NULL");
    }
    if (S == 0) {
      if (P > 0 || out->tile_nnz) {
        // nothing to compute; still define the scalar outputs
      }
      if (out->qt_ptr) SEG_HIP(hipMemsetAsync(out->qt_ptr, 0, sizeof(int32_t), stream));
      if (out->kt_ptr) SEG_HIP(hipMemsetAsync(out->kt_ptr, 0, sizeof(int32_t), stream));
      if (out->tile_nnz) SEG_HIP(hipMemsetAsync(out->tile_nnz, 0, sizeof(int64_t), stream));
      if (P > 0 && out->tok_src) {
        SEG_HIP(hipMemsetAsync(out->tok_src, 0xff, sizeof(int32_t) * P, stream));
      }
      return;
    }
    const BuildWs w = build_ws_layout(*sz, pl.pieces.size(), pl.lpieces.size());
    // One upload of all tables, gathered on the host.  Every segment holds the
    // text runs of all turns before it, so the runs grow with the square of a
    // trajectory's turns, and gathering many costs more than an upload of their own.
    const size_t piece_bytes = pl.pieces.size() * sizeof(Piece);
    const bool apart = piece_bytes > PIECES_APART;
    const size_t gathered = apart ? w.piece : w.total;
    std::vector<char> tab(gathered);
    auto put = [&](size_t off, const auto &v) {
      if (!v.empty()) std::memcpy(tab.data() + off, v.data(), v.size() * sizeof(v[0]));
    };
    put(w.dseg, pl.dsegs);
    if (!apart) put(w.piece, pl.pieces);
    put(w.lpiece, pl.lpieces);
    put(w.info, pl.seg_info);
    put(w.span, pl.spans);
    put(w.qptr, pl.qt_ptr);
    put(w.kptr, pl.kt_ptr);
    put(w.pairs, pl.seg_pairs);
    SEG_HIP(hipMemcpyAsync(ws, tab.data(), gathered, hipMemcpyHostToDevice, stream));
    if (apart)
      SEG_HIP(hipMemcpyAsync(static_cast<char *>(ws) + w.piece, pl.pieces.data(), piece_bytes,
                             hipMemcpyHostToDevice, stream));
    // the host tables are locals of this call: wait until they have been read
    SEG_HIP(hipStreamSynchronize(stream));

    ProfScope prof("layout", stream);
    const char *base = static_cast<const char *>(ws);
    BuildArgs a{};
    a.segs = reinterpret_cast<const DevSeg *>(base + w.dseg);
    a.pieces = reinterpret_cast<const Piece *>(base + w.piece);
    a.lp = reinterpret_cast<const LossPiece *>(base + w.lpiece);
    a.info = reinterpret_cast<const int32_t *>(base + w.info);
    a.qptr = reinterpret_cast<const int32_t *>(base + w.qptr);
    a.kptr = reinterpret_cast<const int32_t *>(base + w.kptr);
    a.span = reinterpret_cast<const TileSpan *>(base + w.span);
    a.pairs = reinterpret_cast<const int64_t *>(base + w.pairs);
    a.out = *out;
    a.S = S;
    a.P = P;
    a.R = R;
    a.G = G;
    a.nlp = (int)pl.lpieces.size();
    a.tile = p->tile;
    a.tok_blocks = (int)((P + (int64_t)TOK_BLOCK - 1) / TOK_BLOCK);
    a.loss_blocks = (int)((R + 255LL) / 256);
    a.tile_blocks = (int)((G + 3LL) / 4);
    a.copy_blocks = (int)std::min<int64_t>(64, (G + 256LL) / 256);
    const int64_t blocks = (int64_t)a.tok_blocks + a.loss_blocks + 2LL * a.tile_blocks + a.copy_blocks;
    SEG_CHECK(blocks <= INT_MAX, SEG_ERR_CAPACITY, "layout too large");
    k_build<<<(unsigned)blocks, 256, 0, stream>>>(a);
    SEG_LAUNCH_CHECK();
  });
}
