// Acceptance walk with the LM head applied at the visited nodes only
// (MFMA, gfx950).
//
// Method: the lossless acceptance walk of Sections 1 and 3 (descend while
// the policy's own next token -- greedy arg-max, or Gumbel-max for sampling
// at temperature T -- is a child's token, then emit it as the bonus token),
// where the policy's logits at tree node u are its LM head applied to the
// node's final hidden state, logit_j = <hidden[b,u], w_head[j]>.  The walk
// needs the arg-max at the nodes it visits and nothing else, so the
// [B, N, V] logits tensor and the head's products for most unvisited nodes
// are never formed.
//
// GPU design.  The batch advances in passes; a pass reads the head once.
//   * Rows of a pass: every sequence still walking brings its current node
//     and, as long as the pass has room (look_for), the next nodes of that
//     node's subtree in tree order, the same number for everybody (draft
//     rank order: likely descendants first).  Each of these rows may spare
//     the walk a pass of its own.
//   * A product kernel multiplies the rows with the whole head and reduces
//     each to one (score, token) candidate per tile of the vocabulary.
//   * A walk kernel (one workgroup per walking sequence) follows the walk
//     through the nodes of the pass; where it leaves them it lists the new
//     current node's subtree for the next pass.
// A walk that leaves a pass with quota q stands at least q places further in
// its tree, so ceil(N / q) passes always suffice, or one more than leave every
// tree with so few nodes that they are the last pass; no more are enqueued.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"

using namespace srt;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// 16-byte loads of noise rows, which start at any multiple of 4 bytes (the
// hardware's requirement) when V is not a multiple of 4.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kUnit = 16;                // head rows are shared out in units of 16
constexpr int kKC = 64;                  // d_model elements per step (one 128-byte line of a row)
constexpr int kRowBytes = kKC * 2 + 16;  // padded LDS row (conflict-free operand reads)
// Rows that a pass is filled up to, at most.  One pass over a 152064 x 3584 head takes
// 221 us for 64 rows, 260 for 128 and 380 for 256 (sampled; reading the head
// alone takes 190); see look_for for what they save.
constexpr int kLook = 256;
constexpr int kMaxLevels = 64;           // Dmax + 1 <= 64
constexpr int kGrid = 256;               // workgroups of a pass over a large head: one per CU
constexpr int kXcds = 8;
constexpr int kWalkThreads = 256;
constexpr int kParents = 1024;           // nodes of a tree whose parents are staged in LDS
constexpr int kUncovered = 0x7FFFFFFF;   // place of a subtree node beyond every pass

struct HeadArgs {
  const uint16_t* hidden;   // [B, N, dm]
  const uint16_t* w_head;   // [V, dm]
  const float* gumbel;      // [B, Dmax+1, V] or null
  const int32_t* tree_tokens;
  const int32_t* tree_parent;
  const int32_t* n_nodes;
  int32_t* n_accepted;
  int32_t* out_tokens;
  int32_t* out_nodes;
  int32_t* n_emitted;
  int32_t* n_act;           // [kMaxLevels + 1] walking sequences per pass
  int32_t* act;             // [2, B] walking sequences, by pass parity
  int32_t* listed;          // [2, B] their listed nodes, or null (one each)
  int2* span;               // [kLook] first row and row count of each walker of the pass
  int2* list;               // [B, L] (node, depth) of each sequence's next subtree
  int32_t* place;           // [B, N] place of a node in its list, or null (L = 1)
  unsigned long long* cand; // [max(B, kLook), n_cand] packed candidates of the pass
  int B, N, L, dm, V, Dmax, n_cand;
  int look, finish;         // rows that a pass is filled up to; nodes that make it the last
  int units, tiles;         // see Split
  float invT;
};

// How a pass divides the head.  Large heads (wide): 16-row units shared out
// evenly over kGrid workgroups, one per CU, each of which reads its share (at
// least 128 rows) in tiles of up to 256 rows.  Small ones: 128-row tiles, a
// workgroup for each and 64 or 128 rows of the pass.
struct Split {
  bool wide, tall;
  int units, grid, tiles;  // wide: units, workgroups, tiles per workgroup; else tiles in all
};

// The line lies where the small tiles need more than one round of the CUs.
// Small and wide tiles, us, d 1536: V 32768, 256 sequences of 32 nodes, Dmax 8 222
// and 256, of 64, Dmax 1 82 and 97, 8 of 32, Dmax 8 42 and 46; V 36000, the same 297
// and 269, 110 and 102, 55 and 49; V 65536, d 512 (64 MB) 228 and 187, 83 and 77, 43
// and 38.  The head's bytes make no difference: what decides is how many CUs
// have a tile, and how full theirs are.
constexpr int kSmallTiles = kGrid;
// Passes of more than 64 rows over small heads: workgroups of 128 rows read the
// head half as often, but up to here those of 64 are done with 256 rows in one
// round of two a CU (us with 64 and with 128 rows, d 3072, 256 sequences of 64
// nodes, Dmax 1: V 8192 66 and 87, 16384 81 and 89, 24576 114 and 109).
constexpr int kFlatTiles = kGrid / 2;

inline Split split_for(int64_t V) {
  Split s;
  s.units = s.grid = 0;
  s.tiles = static_cast<int>((V + 127) / 128);
  s.wide = s.tiles > kSmallTiles;
  s.tall = !s.wide && s.tiles > kFlatTiles;
  if (!s.wide) return s;
  static_assert(kSmallTiles * 128 / kUnit >= 8 * kGrid, "units for every workgroup");
  s.units = static_cast<int>((V + kUnit - 1) / kUnit);
  s.grid = kGrid;
  const int per = s.grid * (256 / kUnit);
  s.tiles = (s.units + per - 1) / per;
  return s;
}

// Rows that passes are filled up to, unless the nodes that the walks can still
// reach are kLook or fewer: a pass then takes them all and is the last, as it
// costs less than two smaller ones (us; V 151936, d 1536, 32 sequences of 64
// nodes, Dmax 6, greedy: 434 without, 300 with it; 8 of 64, Dmax 1: 200 and 162;
// up to 7% more than two passes for narrow heads, whose rows' noise weighs most:
// d 896, 16 of 32, Dmax 2, sampled: 133 and 140).
// Rows after the first 64 cost products and noise (kLook) and are lost on walks
// that end before them; what they save are the later passes of deep walks.
// Time of a call with 64, 128 and 256 rows to that of a pass per level, over
// 2912 batches (1 to 256 sequences of up to 128 nodes, Dmax 1 to 12, eight heads of
// 8192 x 1024 to 151936 x 3584; geometric mean, and the worst):
// - Dmax <= 2, which two or three passes end anyhow: 0.91 (1.25), 0.93 (1.34),
//   1.02 (1.77);
// - room for at most 512 tree nodes (drafted trees fill half of it as a rule: the
//   first pass is the last): 0.64 (1.11), 0.63 (1.08), 0.62 (1.04);
// - light heads, whose rows cost less than a pass's launches: 0.78, 0.75, 0.70;
// - more than 128 sequences of small or deep trees, which fill several passes
//   in any case: 0.86, 0.79, 0.77 (trees of over 64 nodes: 0.90, 0.84, 0.90);
// - shallow walks of up to 64 sequences: 0.91 (1.13), 0.96 (1.26), 1.09 (1.58),
//   of more: 0.87, 0.85, 0.93 (1.34) (us: 16 sequences of 64, Dmax 3, sampled, V
//   151936, d 2560: 335, 359, 439, with a pass per level 334);
// - deep ones over large heads: 0.78, 0.75 (1.11), 0.81 (1.33); over those in
//   between 0.81, 0.75, 0.75, and 256 rows are fewer passes.
constexpr int64_t kLightHead = int64_t(20) << 20;  // elements
constexpr int64_t kLargeHead = int64_t(48) << 20;

inline int look_for(int64_t B, int64_t N, int64_t V, int64_t d_model, int Dmax) {
  if (Dmax <= 2) return 64;
  const int64_t head = V * d_model;
  if (B * N <= 2 * kLook || head <= kLightHead) return kLook;
  if (B > 128 && (N <= 16 || (Dmax > 6 && N <= 64))) return kLook;
  if (Dmax <= 6) return B <= 64 ? 64 : 128;
  return head <= kLargeHead ? kLook : 128;
}

// Scratch layout: counters, lists, node places, candidates of passes of up to
// `rows` rows (or a row for each sequence).  rows = 1: the walking sequences'
// own nodes only.
struct ScratchLayout {
  int rows, L;
  size_t off_act, off_listed, off_span, off_list, off_place, off_cand, total;
};

inline size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

inline ScratchLayout scratch_layout(int64_t B, int64_t N, int rows, int64_t n_cand) {
  ScratchLayout s;
  const size_t b = static_cast<size_t>(B), n = static_cast<size_t>(N);
  s.rows = rows;
  s.L = static_cast<int>(std::min<int64_t>(N, rows));
  s.off_act = up256(sizeof(int32_t) * (kMaxLevels + 1));
  s.off_listed = s.off_act + up256(sizeof(int32_t) * 2 * b);
  s.off_span = s.off_listed + (rows > 1 ? up256(sizeof(int32_t) * 2 * b) : 0);
  s.off_list = s.off_span + up256(sizeof(int2) * kLook);
  s.off_place = s.off_list + up256(sizeof(int2) * b * s.L);
  s.off_cand = s.off_place + (rows > 1 ? up256(sizeof(int32_t) * b * n) : 0);
  s.total = s.off_cand +
            up256(sizeof(unsigned long long) * std::max<size_t>(b, rows) * static_cast<size_t>(n_cand));
  return s;
}

// The scratch that callers are asked for: room for full passes, and one
// candidate per row and 128 head rows (the wide division has no more: kGrid per
// 256 kGrid rows or part of them, from 128 kGrid rows on).
inline size_t full_scratch(int64_t B, int64_t N, int64_t V) {
  return scratch_layout(B, N, kLook, (V + 127) / 128).total;
}

// What callers were asked for while a pass took the sequences' own nodes, or
// the last 128 in all.  Sizes from there on are accepted still, if they are
// whole 256 bytes as every size is that callers were ever told: anything else
// below the full size is a mistake.
inline size_t least_scratch(int64_t B, int64_t N, int64_t V) {
  const size_t b = static_cast<size_t>(B), n = static_cast<size_t>(N);
  return 1024 + up256(8 * b) + 3072 + up256(4 * b) + up256(4 * b * n) +
         up256(8 * std::max<size_t>(b, 128) * ((static_cast<size_t>(V) + 127) / 128));
}

// The layout of the fullest passes that a scratch of `bytes` has room for.
// (rows = 1 fits the least one: 512 + 2048 + 2 up256(8 B) is no more than 4096 +
// up256(8 B) + up256(4 B) + up256(4 B N), and a pass has B rows.)
inline ScratchLayout layout_for(int64_t B, int64_t N, int64_t n_cand, size_t bytes) {
  for (int rows = kLook; rows >= 64; rows -= 64) {
    const ScratchLayout s = scratch_layout(B, N, rows, n_cand);
    if (s.total <= bytes) return s;
  }
  return scratch_layout(B, N, 1, n_cand);
}

// Total order key of a (score, token) candidate: larger score first, then
// the lower token.  +0 and -0 compare equal, as fp32 comparisons do.
__device__ inline unsigned long long pack_key(float x, int tok) {
  uint32_t u = __float_as_uint(x == 0.f ? 0.f : x);
  u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  return (static_cast<unsigned long long>(u) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(tok));
}

__device__ inline int key_token(unsigned long long k) {
  return static_cast<int>(~static_cast<uint32_t>(k & 0xFFFFFFFFull));
}

__device__ inline void take(float& bv, int& bi, float v, int i) {
  if (v > bv || (v == bv && i < bi)) {
    bv = v;
    bi = i;
  }
}

// One wave lists the subtree of node u of sequence b (u at depth du, nodes of
// depth <= Dmax, in tree order): the first a.L nodes go to the list, every
// node learns its place; returns the number listed.  Descendants have larger indices; a
// node's ancestry is followed up through parents with smaller indices only,
// so malformed parent links end the search.  `par`: the tree's parents in
// LDS (staged), or null.
__device__ inline int list_subtree(const HeadArgs& a, int b, int u, int du, int n, const int32_t* par) {
  const int lane = threadIdx.x % SRT_WAVE;
  const int64_t tr = static_cast<int64_t>(b) * a.N;
  int base = 0;
  for (int c0 = u; c0 < n; c0 += SRT_WAVE) {
    const int c = c0 + lane;
    int depth = -1;
    if (c < n) {
      int x = c, steps = 0;
      while (x > u && steps <= a.Dmax - du) {
        const int p = par ? par[x] : a.tree_parent[tr + x];
        if (p < 0 || p >= x) break;
        x = p;
        ++steps;
      }
      if (x == u && du + steps <= a.Dmax) depth = du + steps;
    }
    const unsigned long long m = __ballot(depth >= 0);
    if (depth >= 0) {
      const int j = base + __popcll(m & ((1ull << lane) - 1));
      if (j < a.L) a.list[static_cast<int64_t>(b) * a.L + j] = make_int2(c, depth);
      if (a.place) a.place[tr + c] = j < a.L ? j : kUncovered;
    }
    base += __popcll(m);
  }
  return min(base, a.L);
}

// One wave per sequence: outputs to -1, walking from the root with its whole
// tree listed; the first one also sets the counters (n_act[0] = B, the rest 0).
__global__ __launch_bounds__(SRT_WAVE) void head_init_kernel(HeadArgs a) {
  __shared__ int32_t s_par[kParents];
  const int b = blockIdx.x;
  const int lane = threadIdx.x;
  if (b == 0)
    for (int i = lane; i <= kMaxLevels; i += SRT_WAVE) a.n_act[i] = i == 0 ? a.B : 0;
  const int64_t row = static_cast<int64_t>(b) * (a.Dmax + 1);
  for (int k = lane; k <= a.Dmax; k += SRT_WAVE) {
    a.out_tokens[row + k] = -1;
    a.out_nodes[row + k] = -1;
  }
  const int n = min(max(a.n_nodes[b], 1), a.N);
  if (n <= kParents)
    for (int c = lane; c < n; c += SRT_WAVE) s_par[c] = a.tree_parent[static_cast<int64_t>(b) * a.N + c];
  __syncthreads();
  const int listed = list_subtree(a, b, 0, 0, n, n <= kParents ? s_par : nullptr);
  if (lane == 0) {
    a.act[b] = b;
    if (a.listed) a.listed[b] = listed;
  }
}

// LDS of a product kernel: TV head rows and TM hidden rows a tile.
template <int TV, int TM>
struct PassShared {
  union {
    struct {
      uint8_t w[2][TV * kRowBytes];              // head rows of two steps
      uint8_t h[2][TM * kRowBytes];              // hidden rows of two steps
    };
    unsigned long long key[8][TM];               // after the steps, by wave
  };
  int64_t hoff[TM], goff[TM];                    // a row's hidden and noise offsets
  int base[kLook];                               // first row of each walker
  alignas(16) int cnt[kLook];                    // its listed nodes
  int seq[kLook];                                // its sequence
};

// A pass of this many walkers or more brings their current nodes only: rows are
// neither left to fill, nor can the nodes be few enough to end every walk
// (unless there are no others).
__device__ inline int lone_from(const HeadArgs& a) { return max(a.look, a.finish); }

// A thread's walker of the pass: its sequence and listed nodes (loaded beside
// the number of walkers, unused past it).
__device__ inline int2 load_walker(const HeadArgs& a, int pass) {
  const int tid = threadIdx.x;
  if (tid >= kLook || tid >= a.B) return make_int2(0, 0);
  const int64_t at = static_cast<int64_t>(pass & 1) * a.B + tid;
  return make_int2(a.act[at], a.listed ? a.listed[at] : 1);
}

// Rows of the pass: fills s.base (for fewer than lone_from walkers) and returns their
// number.  Where all listed nodes are few they are the pass.  Else each walker
// takes the first min(q, listed) nodes of its list, q the largest number for
// which the rows fit, and the first walkers with more listed one more each
// while rows are left.  Every workgroup works this out for itself (every wave
// the number, from the counts in its lanes); the first records it for the walk
// kernel.  A thread for each q, summing over the counts in LDS, took 12 us for
// 256 walkers: V 32000, d 1024, a pass over 256 sequences' roots 44 us, 32 so.
template <typename Shared>
__device__ inline int pass_rows(const HeadArgs& a, int2 walker, int W, Shared& s) {
  static_assert(kLook == 256 && kLook % SRT_WAVE == 0, "a thread per walker (workgroups have 256 or more)");
  const int tid = threadIdx.x, lane = tid % SRT_WAVE;
  if (tid < kLook) {
    s.seq[tid] = min(max(walker.x, 0), a.B - 1);
    s.cnt[tid] = tid < W ? min(max(walker.y, 1), a.L) : 0;
  }
  __syncthreads();
  constexpr int kPer = kLook / SRT_WAVE;
  int c[kPer];  // (counts past W are 0)
#pragma unroll
  for (int k = 0; k < kPer; ++k) c[k] = s.cnt[lane * kPer + k];
  auto lane_rows = [&](int q) __attribute__((always_inline)) {
    int x = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) x += min(c[k], q);
    return x;
  };
  const int look = wave_sum(lane_rows(kLook)) <= a.finish ? kLook : max(a.look, W);
  int q = 0, rows = 0;  // (the rows grow with q; 1 always fits)
#pragma unroll 1
  for (int step = kLook; step >= 1; step >>= 1) {
    if (q + step > kLook) continue;
    const int x = wave_sum(lane_rows(q + step));
    if (x <= look) {
      q += step;
      rows = x;
    }
  }
  int more = 0;  // walkers of this lane that have more than q listed
#pragma unroll
  for (int k = 0; k < kPer; ++k) more += c[k] > q;
  const int left = look - rows, total = rows + min(left, wave_sum(more));
  if (tid < SRT_WAVE) {
    // those ahead of this lane, and the rows of the walkers ahead
    const int mine = lane_rows(q);
    int im = more, ir = mine;
#pragma unroll
    for (int off = 1; off < SRT_WAVE; off <<= 1) {
      const int x = __shfl_up(im, off, SRT_WAVE), y = __shfl_up(ir, off, SRT_WAVE);
      if (lane >= off) {
        im += x;
        ir += y;
      }
    }
    int ahead = im - more, first = ir - mine;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int i = lane * kPer + k;
      s.base[i] = first + min(ahead, left);
      const int n = min(c[k], q) + (c[k] > q && ahead < left);
      if (blockIdx.x == 0 && i < W) a.span[i] = make_int2(s.base[i], n);
      first += min(c[k], q);
      ahead += c[k] > q;
    }
  }
  __syncthreads();
  return total;
}

// Offsets of rows m0 .. m0 + TM - 1 of the pass (a thread per row).
template <int TM, typename Shared>
__device__ inline void row_offsets(const HeadArgs& a, int pass, int W, int n_rows, int m0, Shared& s) {
  const int r = m0 + static_cast<int>(threadIdx.x);
  if (threadIdx.x >= TM) return;
  int64_t ho = 0, go = 0;
  if (r < n_rows) {
    int b, j = 0;
    if (W < lone_from(a)) {  // the walker whose rows hold r
      int lo = 0, hi = W - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (s.base[mid] <= r) lo = mid;
        else hi = mid - 1;
      }
      b = s.seq[lo];
      j = r - s.base[lo];
    } else {
      b = min(max(a.act[static_cast<int64_t>(pass & 1) * a.B + r], 0), a.B - 1);
    }
    const int2 x = a.list[static_cast<int64_t>(b) * a.L + j];
    ho = (static_cast<int64_t>(b) * a.N + min(max(x.x, 0), a.N - 1)) * a.dm;
    go = (static_cast<int64_t>(b) * (a.Dmax + 1) + min(max(x.y, 0), a.Dmax)) * a.V;
  }
  s.hoff[threadIdx.x] = ho;
  s.goff[threadIdx.x] = go;
}

// Wave layouts of a tile: the WV x WS waves split its TV = 32 WV VT head rows
// and its TM = 32 WS ST hidden rows; a wave multiplies its head rows with its
// hidden rows (VT x ST products a step of 16).  kRing, kRingH: steps of head
// and hidden loads in registers (256 rows leave room for two and one, and the
// hidden rows come from the L2).
struct Rows64 {
  static constexpr int WV = 8, VT = 1, WS = 1, ST = 2, kRing = 4, kRingH = 4;
};
struct Rows128 {
  static constexpr int WV = 4, VT = 2, WS = 2, ST = 2, kRing = 4, kRingH = 4;
};
struct Rows256 {
  static constexpr int WV = 4, VT = 2, WS = 2, ST = 4, kRing = 2, kRingH = 1;
};
struct Small64 {
  static constexpr int WV = 4, VT = 1, WS = 1, ST = 2, kRing = 4, kRingH = 4;
};
struct Small128 {
  static constexpr int WV = 2, VT = 2, WS = 2, ST = 2, kRing = 4, kRingH = 4;
};

// One tile: head rows v0 .. v_end-1 (at most TV) times the TM rows of the pass
// from m0 on (m_end: the end of this workgroup's rows).  Both operands are staged in padded, double-buffered
// LDS.  Up to 128 rows a pass is bound by streaming the head (4.2 TB/s at 128
// rows, 5.1 at 64), above by the products (0.75 PFLOP/s at 256 rows; large
// matrix products reach 1.2 on this card).  256 x 256 tiles read 0.75 KB of
// LDS a product and stage each head row once for all rows (385 us -> 355 for
// 256 greedy rows against 128 x 128 tiles, two workgroups a CU).  Head operands
// loaded straight into registers (16 rows of 64 bytes an instruction) took
// 510: 64 separate 16-byte accesses an instruction keep the L1 busy.  Issuing a
// tile's first loads before the epilogue of the one before it cost 14-23 us at
// 128 rows (loads retire in order, so the noise waits for them).
template <bool kNoise, typename Lay, typename Shared>
__device__ inline void head_tile(const HeadArgs& a, Shared& s, int v0, int v_end, int m0, int m_end, int col) {
  constexpr int VT = Lay::VT, ST = Lay::ST, R = Lay::kRing, RH = Lay::kRingH;
  constexpr int TV = 32 * Lay::WV * VT, TM = 32 * Lay::WS * ST;
  constexpr int kStageRows = Lay::WV * Lay::WS * SRT_WAVE / 8;  // rows staged by one load of every thread
  constexpr int WJ = TV / kStageRows, HJ = TM / kStageRows;
  // (values of its own for each layout: addresses that the compiler would
  // otherwise work out once for all three take registers in every loop)
  int tid = threadIdx.x;
  v0 = __builtin_amdgcn_readfirstlane(v0);
  v_end = __builtin_amdgcn_readfirstlane(v_end);
  asm volatile("" : "+v"(tid), "+s"(v0));
  const int lane = tid % SRT_WAVE;
  const int wave = __builtin_amdgcn_readfirstlane(tid / SRT_WAVE);
  const int l32 = lane % 32, hf = lane / 32;
  const int wv = wave % Lay::WV, ws = wave / Lay::WV;

  // Loads: 8 threads read one row's 128-byte line, so every load instruction
  // reads whole lines.  Rows past the tile read its last row (never used).
  const int lc = tid % 8, r0 = tid / 8;
  const char* wbase = reinterpret_cast<const char*>(a.w_head + static_cast<int64_t>(v0) * a.dm);
  uint32_t woff[WJ];
#pragma unroll
  for (int j = 0; j < WJ; ++j)
    woff[j] = static_cast<uint32_t>(min(r0 + kStageRows * j, v_end - v0 - 1)) * static_cast<uint32_t>(a.dm * 2) +
              static_cast<uint32_t>(lc * 16);
  const uint16_t* hp[HJ];
#pragma unroll
  for (int j = 0; j < HJ; ++j) hp[j] = a.hidden + s.hoff[r0 + kStageRows * j] + lc * 8;

  const int n_steps = a.dm / kKC;
  u32x4 wr[R][WJ], hr[RH][HJ];
  auto hload = [&](int slot, int c) __attribute__((always_inline)) {
    c = min(c, n_steps - 1);
#pragma unroll
    for (int j = 0; j < HJ; ++j) hr[slot][j] = *reinterpret_cast<const u32x4*>(hp[j] + c * kKC);
  };
  auto wload = [&](int slot, int c) __attribute__((always_inline)) {
    const char* p = wbase + static_cast<int64_t>(min(c, n_steps - 1)) * (kKC * 2);
#pragma unroll
    for (int j = 0; j < WJ; ++j) wr[slot][j] = *reinterpret_cast<const u32x4*>(p + woff[j]);
  };
  // Quarter `part` of the staging stores of step c (4: all of them).  With one
  // step of hidden rows in registers these come last, as late as they can.
  constexpr bool kLateH = RH < R;
  auto stage = [&](int c, int part) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < WJ; ++j)
      if (part == 4 || j * (kLateH ? 2 : 4) / WJ == part)
        *reinterpret_cast<u32x4*>(&s.w[c % 2][(r0 + kStageRows * j) * kRowBytes + lc * 16]) = wr[c % R][j];
#pragma unroll
    for (int j = 0; j < HJ; ++j)
      if (part == 4 || (kLateH ? 2 + j * 2 / HJ : j * 4 / HJ) == part)
        *reinterpret_cast<u32x4*>(&s.h[c % 2][(r0 + kStageRows * j) * kRowBytes + lc * 16]) = hr[c % RH][j];
  };

  const int a_rd = (32 * VT * wv + l32) * kRowBytes + 16 * hf;
  const int b_rd = (32 * ST * ws + l32) * kRowBytes + 16 * hf;
  const bool active = __builtin_amdgcn_readfirstlane(v0 + 32 * VT * wv < v_end && m0 + 32 * ST * ws < m_end);
  f32x16 acc[VT][ST];
#pragma unroll
  for (int x = 0; x < VT; ++x)
#pragma unroll
    for (int y = 0; y < ST; ++y)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[x][y][r] = 0.f;

  // Step c: loads of step c + R are issued (its slot was staged a step ago),
  // step c is multiplied, step c + 1 is staged.  Loads retire in order, so
  // each wait leaves the newer ones in flight.
  auto step = [&](auto s_c, int c) __attribute__((always_inline)) {
    constexpr int S = decltype(s_c)::value;
    if (!kLateH) hload(S % RH, c + RH);
    wload(S % R, c + R);
    if (active) {
      // Operands are read one group of products ahead: a group is the whole of
      // a 16-wide step, or half its hidden rows where four of them would
      // leave too few registers.
      constexpr int YH = ST > 2 ? 2 : 1, SY = ST / YH;
      bf16x8 af[2][VT], bf[2][SY];
      auto read = [&](int i) __attribute__((always_inline)) {
        const int ks = i / YH;
        if (i % YH == 0) {
#pragma unroll
          for (int x = 0; x < VT; ++x)
            af[ks % 2][x] = *reinterpret_cast<const bf16x8*>(&s.w[S % 2][a_rd + 32 * x * kRowBytes + ks * 32]);
        }
#pragma unroll
        for (int y = 0; y < SY; ++y)
          bf[i % 2][y] =
              *reinterpret_cast<const bf16x8*>(&s.h[S % 2][b_rd + 32 * (i % YH * SY + y) * kRowBytes + ks * 32]);
      };
      read(0);
#pragma unroll
      for (int i = 0; i < 4 * YH; ++i) {
        const int ks = i / YH;
        if (i + 1 < 4 * YH) read(i + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int y = 0; y < SY; ++y)
#pragma unroll
          for (int x = 0; x < VT; ++x)
            acc[x][i % YH * SY + y] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[ks % 2][x], bf[i % 2][y],
                                                                              acc[x][i % YH * SY + y], 0, 0, 0);
        if (i % YH == YH - 1) stage(S + 1, ks);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      stage(S + 1, 4);
    }
    if (kLateH) hload((S + 1) % RH, c + 1 + RH);
    __syncthreads();
  };
  // (in the steady state's order, so that the waits inside the loop count the
  // same loads on entry)
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if (i < RH) hload(i, i);
    wload(i, i);
  }
  stage(0, 4);
  if (kLateH) hload(0, RH);
  __syncthreads();
  constexpr int U = R < 2 ? 2 : R;
  int c = 0;
  for (; c + U <= n_steps; c += U) {
    step(std::integral_constant<int, 0>(), c);
    step(std::integral_constant<int, 1>(), c + 1);
    if constexpr (U > 2) {
      step(std::integral_constant<int, 2>(), c + 2);
      step(std::integral_constant<int, 3>(), c + 3);
    }
  }
  if (c < n_steps) step(std::integral_constant<int, 0>(), c);
  if constexpr (U > 2) {
    if (c + 1 < n_steps) step(std::integral_constant<int, 1>(), c + 1);
    if (c + 2 < n_steps) step(std::integral_constant<int, 2>(), c + 2);
  }

  // Epilogue: lane column l32 of tile y is row m0 + 32 ST ws + 32 y + l32 of the
  // pass; element r of tile x is head row v0 + 32 VT wv + 32 x + 8 (r / 4) +
  // 4 hf + r % 4.  (The keys take the staging buffers' place: every wave is
  // past the last step's barrier.)
#pragma unroll
  for (int y = 0; y < ST; ++y) {
    const int sl = 32 * ST * ws + 32 * y + l32;
    float bv = -INFINITY;
    int bi = 0x7FFFFFFF;
    if (active && m0 + sl < m_end) {
      const float* gr = kNoise ? a.gumbel + s.goff[sl] : nullptr;
#pragma unroll
      for (int x = 0; x < VT; ++x)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int vb = v0 + 32 * VT * wv + 32 * x + 8 * q + 4 * hf;
          float gv[4] = {0.f, 0.f, 0.f, 0.f};
          if (kNoise) {
            if (vb + 4 <= v_end) {
              const f32x4 g = *reinterpret_cast<const f32x4u*>(gr + vb);
              gv[0] = g.x; gv[1] = g.y; gv[2] = g.z; gv[3] = g.w;
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) gv[e] = vb + e < v_end ? gr[vb + e] : 0.f;
            }
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (vb + e < v_end) {
              float sc = acc[x][y][4 * q + e];
              if (kNoise) sc = __fadd_rn(__fmul_rn(sc, a.invT), gv[e]);
              take(bv, bi, sc, vb + e);
            }
          }
        }
    }
    const float ov = __shfl_xor(bv, 32, SRT_WAVE);
    const int oi = __shfl_xor(bi, 32, SRT_WAVE);
    take(bv, bi, ov, oi);
    if (hf == 0) s.key[wv][sl] = pack_key(bv, bi);
  }
  __syncthreads();
  if (tid < TM && m0 + tid < m_end) {
    unsigned long long k = s.key[0][tid];
#pragma unroll
    for (int w = 1; w < Lay::WV; ++w) k = s.key[w][tid] > k ? s.key[w][tid] : k;
    a.cand[static_cast<int64_t>(m0 + tid) * a.n_cand + col] = k;
  }
  __syncthreads();  // the keys' memory is the next tile's staging buffers
}

// One pass's products and per-tile arg-max candidates over a large head.  The
// workgroups share the head's units out evenly (so that no CU is left with a
// tile more than the others), the shares of one tile next to each other.
template <bool kNoise>
__global__ __launch_bounds__(512, 1) void head_pass_kernel(HeadArgs a, int pass) {
  using Shared = PassShared<256, 256>;  // 151 of the CU's 160 KB
  __shared__ __attribute__((aligned(16))) Shared s;
  const int2 walker = load_walker(a, pass);
  const int W = a.n_act[pass];
  if (W <= 0) return;
  const int n_rows = W < lone_from(a) ? pass_rows(a, walker, W, s) : W;
  const int g = blockIdx.x, shares = gridDim.x;
  for (int m0 = 0; m0 < n_rows; m0 += 256) {
    row_offsets<256>(a, pass, W, n_rows, m0, s);
    __syncthreads();
    for (int t = 0; t < a.tiles; ++t) {
      const int u0 = static_cast<int>(static_cast<int64_t>(t) * a.units / a.tiles);
      const int nu = static_cast<int>(static_cast<int64_t>(t + 1) * a.units / a.tiles) - u0;
      const int v0 = (u0 + static_cast<int>(static_cast<int64_t>(g) * nu / shares)) * kUnit;
      const int v1 = min((u0 + static_cast<int>(static_cast<int64_t>(g + 1) * nu / shares)) * kUnit, a.V);
      const int col = t * shares + g, m = n_rows - m0;
      // (a tile has 2048 units or more, so every share has at least 8: v0 < v1)
      if (m <= 64) {
        head_tile<kNoise, Rows64>(a, s, v0, v1, m0, n_rows, col);
      } else if (m <= 128) {
        head_tile<kNoise, Rows128>(a, s, v0, v1, m0, n_rows, col);
      } else {
        head_tile<kNoise, Rows256>(a, s, v0, v1, m0, n_rows, col);
      }
    }
  }
}

// The same over a small head: a workgroup takes 128 head rows and 64 rows of
// the pass (kTall: 128 of a pass of more than 64), working ones first in
// dispatch order; those of one tile are on one XCD, whose L2 serves the head
// rows they share.
template <bool kNoise, bool kTall>
__global__ __launch_bounds__(256, 2) void head_small_kernel(HeadArgs a, int pass) {
  constexpr int TM = kTall ? 128 : 64;
  using Shared = PassShared<128, TM>;  // 79 KB or less, two workgroups a CU
  __shared__ __attribute__((aligned(16))) Shared s;
  const int2 walker = load_walker(a, pass);
  const int W = a.n_act[pass];
  if (W <= 0) return;
  const int n_rows = W < lone_from(a) ? pass_rows(a, walker, W, s) : W;
  const int tm = n_rows > 64 ? TM : 64;
  const int n_mb = (n_rows + tm - 1) / tm;
  const int i = blockIdx.x / kXcds;
  const int vt = i / n_mb * kXcds + blockIdx.x % kXcds;
  if (vt >= a.tiles) return;
  const int m0 = i % n_mb * tm;
  row_offsets<TM>(a, pass, W, n_rows, m0, s);
  __syncthreads();
  const int v0 = vt * 128, v1 = min(v0 + 128, a.V), m1 = min(n_rows, m0 + tm);
  if constexpr (kTall) {
    if (tm == TM) {
      head_tile<kNoise, Small128>(a, s, v0, v1, m0, m1, vt);
      return;
    }
  }
  head_tile<kNoise, Small64>(a, s, v0, v1, m0, m1, vt);
}

// Best candidate of one row over the tiles: every thread of the workgroup
// takes a few, then a block reduction; the result is in every thread.
__device__ inline unsigned long long row_best(const HeadArgs& a, int r, unsigned long long* s_best) {
  const int tid = threadIdx.x, lane = tid % SRT_WAVE, wave = tid / SRT_WAVE;
  const unsigned long long* c = a.cand + static_cast<int64_t>(r) * a.n_cand;
  unsigned long long best = 0;
  for (int t = tid; t < a.n_cand; t += kWalkThreads) best = c[t] > best ? c[t] : best;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long o = shfl_xor_u64(best, off);
    best = o > best ? o : best;
  }
  __syncthreads();  // s_best is free (previous readers done)
  if (lane == 0) s_best[wave] = best;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWalkThreads / SRT_WAVE; ++w) best = s_best[w] > best ? s_best[w] : best;
  return best;
}

// Child of u carrying tok (wave-wide search), or -1.  par, ptok: the tree's
// parents and tokens, in LDS where they fit.
__device__ inline int find_child(const int32_t* par, const int32_t* ptok, int u, int n, int tok) {
  const int lane = threadIdx.x % SRT_WAVE;
  int child = -1;
  for (int c0 = u + 1; c0 < n && child < 0; c0 += SRT_WAVE) {
    const int cc = c0 + lane;
    const bool hit = cc < n && par[cc] == u && ptok[cc] == tok;
    const unsigned long long m = __ballot(hit);
    if (m) child = c0 + __ffsll(static_cast<long long>(m)) - 1;
  }
  return child;
}

// One workgroup per walking sequence: the walk goes on through the nodes of
// the pass; a sequence that leaves them for a node further down joins the
// next pass with that node's subtree listed.
__global__ __launch_bounds__(kWalkThreads) void head_walk_kernel(HeadArgs a, int pass) {
  __shared__ unsigned long long s_best[kWalkThreads / SRT_WAVE];
  __shared__ int s_next;
  __shared__ int32_t s_par[kParents], s_tok[kParents];
  const int slot = blockIdx.x;
  const int W = a.n_act[pass];
  if (slot >= W) return;
  const int tid = threadIdx.x, lane = tid % SRT_WAVE, wave = tid / SRT_WAVE;
  const int b = min(max(a.act[static_cast<int64_t>(pass & 1) * a.B + slot], 0), a.B - 1);
  const int n = min(max(a.n_nodes[b], 1), a.N);
  const int64_t tr = static_cast<int64_t>(b) * a.N;
  const int64_t orow = static_cast<int64_t>(b) * (a.Dmax + 1);
  const bool staged = n <= kParents;  // beside the first row's candidates
  if (staged)
    for (int c = tid; c < n; c += kWalkThreads) {
      s_par[c] = a.tree_parent[tr + c];
      s_tok[c] = a.tree_tokens[tr + c];
    }
  const int2 span = W < lone_from(a) ? a.span[slot] : make_int2(slot, 1);
  const int2 first = a.list[static_cast<int64_t>(b) * a.L];
  int u = min(max(first.x, 0), a.N - 1);
  int at = 0;                               // u's place in the list
  int k = min(max(first.y, 0), a.Dmax);     // its depth = the walk's step
  for (;;) {
    const int tok = key_token(row_best(a, span.x + at, s_best));
    if (wave == 0) {
      int child = -1;
      if (k < a.Dmax)
        child = staged ? find_child(s_par, s_tok, u, n, tok)
                       : find_child(a.tree_parent + tr, a.tree_tokens + tr, u, n, tok);
      if (lane == 0) {
        a.out_tokens[orow + k] = tok;
        if (child >= 0) {
          a.out_nodes[orow + k] = child;
        } else {
          a.n_accepted[b] = k;
          if (a.n_emitted) a.n_emitted[b] = k + 1;
        }
        s_next = child;
      }
    }
    __syncthreads();
    if (s_next < 0) return;
    u = s_next;
    ++k;
    at = a.place ? a.place[tr + u] : kUncovered;
    if (at >= span.y) break;
  }
  __syncthreads();  // every wave has read the places that are rewritten now
  if (wave > 0) return;
  const int listed = list_subtree(a, b, u, k, n, staged ? s_par : nullptr);
  if (lane == 0) {
    const int pos = atomicAdd(&a.n_act[pass + 1], 1);
    const int64_t to = static_cast<int64_t>((pass + 1) & 1) * a.B + pos;
    a.act[to] = b;
    if (a.listed) a.listed[to] = listed;
  }
}

}  // namespace

extern "C" size_t srt_accept_lmhead_scratch_bytes(int32_t B, int32_t N, int32_t V) {
  if (B < 0 || N < 1 || V < 1) return 0;
  return full_scratch(std::max(B, 1), N, V);
}

extern "C" int srt_accept_lmhead(int32_t B, int32_t N, int32_t d_model, int32_t V, int32_t Dmax,
                                 const uint16_t* hidden, const uint16_t* w_head, const float* gumbel,
                                 float inv_temperature, const int32_t* tree_tokens, const int32_t* tree_parent,
                                 const int32_t* n_nodes, int32_t* n_accepted, int32_t* out_tokens,
                                 int32_t* out_nodes, int32_t* n_emitted, void* scratch, size_t scratch_bytes,
                                 void* stream) {
  if (B < 0 || N < 1 || V < 1 || d_model < 1 || Dmax < 0 || Dmax >= kMaxLevels) return SRT_ERR_INVALID;
  if (gumbel && !std::isfinite(inv_temperature)) return SRT_ERR_INVALID;
  if (d_model % kKC != 0) return SRT_ERR_UNSUPPORTED;
  if (B == 0) return SRT_OK;
  if (!hidden || !w_head || !tree_tokens || !tree_parent || !n_nodes || !n_accepted || !out_tokens || !out_nodes ||
      !scratch)
    return SRT_ERR_INVALID;
  if ((reinterpret_cast<uintptr_t>(hidden) | reinterpret_cast<uintptr_t>(w_head)) & 15) return SRT_ERR_INVALID;
  if (reinterpret_cast<uintptr_t>(scratch) & 255) return SRT_ERR_INVALID;
  if (scratch_bytes < full_scratch(B, N, V) && (scratch_bytes < least_scratch(B, N, V) || scratch_bytes % 256 != 0))
    return SRT_ERR_CAPACITY;
  const Split sp = split_for(V);
  const int n_cand = sp.wide ? sp.grid * sp.tiles : sp.tiles;
  const ScratchLayout L = layout_for(B, N, n_cand, scratch_bytes);
  const int64_t small_grid = static_cast<int64_t>((sp.tiles + kXcds - 1) / kXcds * kXcds) *
                             ((std::max<int64_t>(B, kLook) + 63) / 64);
  if (small_grid > 0x7FFFFFFF) return SRT_ERR_UNSUPPORTED;

  char* base = static_cast<char*>(scratch);
  HeadArgs a;
  a.hidden = hidden;
  a.w_head = w_head;
  a.gumbel = gumbel;
  a.tree_tokens = tree_tokens;
  a.tree_parent = tree_parent;
  a.n_nodes = n_nodes;
  a.n_accepted = n_accepted;
  a.out_tokens = out_tokens;
  a.out_nodes = out_nodes;
  a.n_emitted = n_emitted;
  a.n_act = reinterpret_cast<int32_t*>(base);
  a.act = reinterpret_cast<int32_t*>(base + L.off_act);
  a.listed = L.rows > 1 ? reinterpret_cast<int32_t*>(base + L.off_listed) : nullptr;
  a.span = reinterpret_cast<int2*>(base + L.off_span);
  a.list = reinterpret_cast<int2*>(base + L.off_list);
  a.place = L.rows > 1 ? reinterpret_cast<int32_t*>(base + L.off_place) : nullptr;
  a.cand = reinterpret_cast<unsigned long long*>(base + L.off_cand);
  a.B = B;
  a.N = N;
  a.dm = d_model;
  a.V = V;
  a.Dmax = Dmax;
  a.L = L.L;
  a.look = std::min(look_for(B, N, V, d_model, Dmax), L.rows);
  a.finish = L.rows;
  a.n_cand = n_cand;
  a.units = sp.units;
  a.tiles = sp.tiles;
  a.invT = inv_temperature;

  hipStream_t s = as_stream(stream);
  head_init_kernel<<<B, SRT_WAVE, 0, s>>>(a);
  int st = launch_status();
  // A walker's quota is at least look / B (see pass_rows), and a walk that
  // leaves a pass has moved that many places on in its tree.
  const int quota = std::max(1, std::min(a.L, a.look / B));
  // Once every tree has at most finish / B nodes left, the pass is the last.
  const int moves = (std::max(0, N - a.finish / B) + quota - 1) / quota;
  const int passes = std::min({Dmax + 1, (N - 1) / quota + 1, moves + 1});
  for (int pass = 0; pass < passes && st == SRT_OK; ++pass) {
    if (sp.wide) {
      if (gumbel) head_pass_kernel<true><<<sp.grid, 512, 0, s>>>(a, pass);
      else head_pass_kernel<false><<<sp.grid, 512, 0, s>>>(a, pass);
    } else {
      const unsigned grid = static_cast<unsigned>(small_grid);
      if (sp.tall) {
        if (gumbel) head_small_kernel<true, true><<<grid, 256, 0, s>>>(a, pass);
        else head_small_kernel<false, true><<<grid, 256, 0, s>>>(a, pass);
      } else {
        if (gumbel) head_small_kernel<true, false><<<grid, 256, 0, s>>>(a, pass);
        else head_small_kernel<false, false><<<grid, 256, 0, s>>>(a, pass);
      }
    }
    st = launch_status();
    if (st != SRT_OK) break;
    head_walk_kernel<<<static_cast<unsigned>(B), kWalkThreads, 0, s>>>(a, pass);
    st = launch_status();
  }
  return st;
}
