// Stage 2: dual-branch block selection (Sec. 3.2; Algorithm 1, selection loop)
// and the supporting selectors of the paper's selector comparison.
//
// A wave scores the key blocks of one row (query head h, query block i) for 32,
// 64 or 128 of its tokens (row_tokens): a whole row, or two or four waves share
// it.  The wave's Q rows are read from HBM once and held in
// registers as f16 (bf16 -> f16 is exact in the normal range).  Candidate key
// blocks 0..i are scored in tiles of 32 centroids that the workgroup's waves --
// rows of one KV head, next to each other in the work order -- stage through
// LDS together (double buffered, one barrier per tile):
//
//   S = Q_i C'^T on the f16 MFMA (32x32x16), where C' = c_b log2(e)/sqrt(d)
//   is the select-ready centroid written by the statistics stage, so S holds
//   base logits / sqrt(d) in log2 units.  Rescue logits add |q_t| u_b with the
//   per-block uplift u_b = r_b beta_b log2(e)/sqrt(d) (Eq. rescue_score).
//
// Per centroid, each group of 32 tokens gives a (shift, sum of exp2) pair per
// branch; the groups' pairs are merged into the block score L_b = log2 S_b (the
// local log-sum-exp form allowed by Eq. block_aggregation).  Then: row maxima,
// relative thresholds in log2 space (L_b >= max L + log2 tau, Eq.
// branch_thresholds), union with the forced blocks, and compaction of the mask
// to an ascending index list with wave ballots.
//
// What bounds it: per 32 centroids and 32 tokens 8 matrix ops (256 cycles of a
// SIMD) and vector work of nearly that length (16 exponentials, their sums), which
// one SIMD overlaps only in part, and the read of Q, which no tile's work covers
// (0.8 GB at 48K tokens, 64 heads).  A wave of 128 tokens takes all 256 VGPRs and
// spills 13 to 16 more, written as Q is read and read back on the way to the tile
// loop: some 30 accesses per row, none in a loop.  A row in one wave needs no
// barrier after the base pass, and one staged operand read serves up to 4
// matrix ops.  Against one workgroup of B / 32 waves per row (32 tokens a
// wave, every step behind a barrier), selection alone, 32 / 4 heads: B = 128
// 32K 104 -> 82 us, 128K 880 -> 696; 48K with 64 / 8 heads 384 -> 303; B = 64
// 128K 1693 -> 1259; B = 256 32K 97 -> 64, 128K 606 -> 500; box selector 32K
// 251 -> 144.  Lists are bit-identical.
#include <type_traits>

#include "rbs_device.hpp"
#include "rbs_launch.hpp"

namespace rbs {

constexpr int kTile = 32;  // centroids per tile
constexpr int kTileBytes = kTile * kHeadDim * 2;
// |exponent| bound for unshifted exp2 sums.  A block's sum adds at most 256
// terms, each below 2^(112 (1 + 2^-10)) -- the bound is tested with the fp32
// centroid norm, and the f16-rounded centroid the MFMA uses is at most 2^-11
// relatively longer -- so a sum stays below 2^121, inside fp32's range, and
// every term above fp32's normal minimum 2^-126.
constexpr float kPlainBound = 112.0f;
constexpr float kCandSlack = 1e-2f;  // log2 units: rounding allowance of the rescue-candidate test
constexpr int kCandRing = 128;       // pending rescue candidates of a wave: at most 31 + 64

// Selection policies: the method's dual-branch selector and the three
// supporting selectors of the paper's selector comparison (Table
// selector_ablation), each a single branch united with the forced blocks.
enum SelectMode {
  kSelectDual = 0,      // base + rescue branches (Sec. 3.2)
  kSelectCentroid = 1,  // base branch alone, relative threshold
  kSelectFullL2 = 2,    // rescue branch with beta = 1 (Eq. full_l2_bound), relative threshold
  kSelectBox = 3,       // Quest-style box bound (Eq. quest_box), fixed budget
};

struct SelectCore {
  const uint16_t* Q;
  int64_t q_head, q_tok;  // element strides of Q between heads and between tokens
  int N, M, group, n_kv;
  int ldm;  // blocks between consecutive heads of the block arrays and counts (M, or the batch's total)
  const _Float16* cent16;     // dual, centroid, full-L2: scaled centroids; box: scaled box centres
  const _Float16* half16;     // box: scaled box half-widths
  const float* uplift;        // dual: r beta log2(e)/sqrt(d)
  const float* cnorm;         // norms of the scaled centroids (not the box's)
  const float* radii;         // full-L2: r (scaled here)
  float log2_tau_base, log2_tau_rescue;  // centroid / full-L2: the one threshold in both
  float budget;               // box: budget fraction rho
  int base_all, rescue_all, n_sink, n_local, n_recent;
  int32_t* counts;
  int32_t* indices;
  int64_t capacity;
};

// A row's split over waves: T tokens per wave in G groups of 32, WPR waves per
// row; W waves per workgroup.
template <int BS, int T, int W>
struct RowSplit {
  static constexpr int TOK = T;
  static constexpr int G = TOK / 32;
  static constexpr int WPR = BS / TOK;
  static constexpr int RPW = W / WPR;  // rows per workgroup
  static_assert(W % WPR == 0 && (WPR == 1 || RPW == 1), "a shared row has the workgroup to itself");
};

// LDS layout (byte offsets): centroid tiles (and half-width tiles, box), two of
// each | |q| of every wave's tokens | per wave, the ring of pending rescue
// candidates (dual) | the groups' pairs of two tiles (a shared row) | L
// (block scores) of every row.
template <int BS, int MODE, int T, int W>
struct SelectLds {
  using S = RowSplit<BS, T, W>;
  static constexpr size_t nq = (MODE == kSelectBox ? 4 : 2) * (size_t)kTileBytes;
  static constexpr size_t ring = nq + W * S::TOK * 4;
  static constexpr size_t stage = ring + (MODE == kSelectDual ? W * kCandRing * 4 : 0);
  static constexpr size_t L = stage + (S::WPR > 1 ? 2 * W * S::G * kTile * 8 : 0);
  static constexpr size_t bytes(int M) { return L + (size_t)S::RPW * M * 4; }
};

// Physical 16-byte chunk of logical chunk c in staged row r (conflict-free
// 16-byte reads of one chunk of 32 rows).
__device__ __forceinline__ int tile_chunk(int r, int c) { return c ^ (r & 15); }

// LDS written by other lanes of this wave is read after this point (a wave's
// LDS operations execute in order; the compiler must keep them so).
__device__ __forceinline__ void wave_lds_fence() { asm volatile("" ::: "memory"); }

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>).
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unroll(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unroll<N, I + 1>(f);
  }
}

// Rows chunk * RPW .. of KV head g, in the order of row numbers descending, the
// group's query heads adjacent; smem: SelectLds bytes.  Writes counts and lists.
template <int BS, int MODE, int T, int W>
__device__ __forceinline__ void select_rows(const SelectCore& c, int g, int chunk, unsigned char* smem) {
  using S = RowSplit<BS, T, W>;
  using Lds = SelectLds<BS, MODE, T, W>;
  constexpr int G = S::G, WPR = S::WPR, TG = G * WPR;
  constexpr bool kDual = MODE == kSelectDual;
  constexpr bool kBound = MODE != kSelectBox;  // the centroids' norms bound the logits
  const int M = c.M;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int slot = chunk * S::RPW + wave / WPR;
  const bool live = slot < c.group * M;  // past the last row: the wave only helps staging
  const int i = live ? M - 1 - slot / c.group : -1;
  const int h = g * c.group + slot % c.group;
  const int n_cand = i + 1;
  const int n_tiles = (M - 1 - chunk * S::RPW / c.group) / kTile + 1;  // of the workgroup's first, longest row
  const int row0 = i * BS;
  const int nb = live ? min(BS, c.N - row0) : 0;  // tokens of the query block
  const int part = WPR > 1 ? wave % WPR : 0;      // this wave's tokens start at part * TOK

  const _Float16* cg = c.cent16 + (size_t)g * c.ldm * kHeadDim;
  const _Float16* hg = MODE == kSelectBox ? c.half16 + (size_t)g * c.ldm * kHeadDim : nullptr;
  const float* ug = MODE == kSelectFullL2 ? c.radii + (size_t)g * c.ldm : c.uplift + (size_t)g * c.ldm;
  const float* cng = kBound ? c.cnorm + (size_t)g * c.ldm : nullptr;
  const float u_scale = MODE == kSelectFullL2 ? kLog2e / sqrtf((float)kHeadDim) : 1.0f;

  float* nq_s = reinterpret_cast<float*>(smem + Lds::nq) + wave * S::TOK;
  int* ring = reinterpret_cast<int*>(smem + Lds::ring) + wave * kCandRing;
  float2* stage = reinterpret_cast<float2*>(smem + Lds::stage);  // [2][TG][kTile]
  // Block scores: the base branch's (centroid, box), the rescue branch's
  // (full-L2); dual: the base scores, and after the rescue pass each rescue
  // candidate's exact rescue score in place of its base score.
  float* L = reinterpret_cast<float*>(smem + Lds::L) + (size_t)(wave / WPR) * M;

  // ---- Tile staging: the waves copy 32 / W rows of a tile each.
  const uint32_t lds0 = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) unsigned char*)smem;
  auto issue_tile = [&](int tile) __attribute__((always_inline)) {
    constexpr int kRows = kTile / W;
#pragma unroll
    for (int j = 0; j < kRows / 4; ++j) {
      const int r = kRows * wave + 4 * j + (lane >> 4);
      const uint32_t voff = (uint32_t)min(tile * kTile + r, M - 1) * (kHeadDim * 2) + 16 * tile_chunk(r, lane & 15);
      const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + (tile & 1) * kTileBytes + (kRows * wave + 4 * j) * 256);
      lds_dma16(cg, voff, dst);
      if constexpr (MODE == kSelectBox) lds_dma16(hg, voff, dst + 2 * kTileBytes);
    }
  };
  issue_tile(0);

  // ---- Q rows of this wave as MFMA A operands (group gr: row 32 gr + l32).
  f16x8 qa[G][8];
  float nq_row = 0.f, nq_min = INFINITY;  // largest and smallest |q| of the query block
  {
    // Tokens past nb read the block's last row (their results are left out):
    // loads under a condition would be issued group by group, each group's
    // after the one before it has arrived.
    const uint16_t* qrow = c.Q + h * c.q_head + (int64_t)max(row0, 0) * c.q_tok + 8 * half;
    uint4 raw[G][8];
#pragma unroll
    for (int gr = 0; gr < G; ++gr) {
      const int t = max(min(part * S::TOK + 32 * gr + l32, nb - 1), 0);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) raw[gr][ks] = *reinterpret_cast<const uint4*>(qrow + t * c.q_tok + 16 * ks);
    }
#pragma unroll
    for (int gr = 0; gr < G; ++gr) {
      float sq = 0.f;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        float f[8];
        unpack8(raw[gr][ks], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          qa[gr][ks][e] = (_Float16)f[e];
          sq = fmaf(f[e], f[e], sq);
        }
      }
      const bool ok = part * S::TOK + 32 * gr + l32 < nb;
      const float nq = sqrtf(half_sum(sq));
      if (half == 0) nq_s[32 * gr + l32] = nq;
      nq_row = fmaxf(nq_row, ok ? nq : 0.f);
      nq_min = fminf(nq_min, ok ? nq : INFINITY);
    }
  }
  nq_row = wave_max(nq_row);
  nq_min = wave_min(nq_min);
  if constexpr (WPR > 1) {
    if (lane == 0) stage[wave] = make_float2(nq_row, nq_min);
    __syncthreads();
#pragma unroll
    for (int w = 0; w < WPR; ++w) {
      nq_row = fmaxf(nq_row, stage[w].x);
      nq_min = fminf(nq_min, stage[w].y);
    }
    // (Read by the row's waves before the tile loop's first barrier, written after it.)
  }

  // ---- Scores of one tile of 32 key blocks, centroid rows in op (lane: block
  // row l32): one branch's (shift, sum) pairs of the wave's token groups.
  // SHIFTED: sums relative to the group's largest exponent; otherwise
  // unshifted (base) or relative to nq_row u (rescue), for tiles whose every
  // exponent is bounded by kPlainBound.  PARTIAL: tokens past nb are left out.
  // A group's exponentials are placed between the next group's matrix ops: left
  // to itself the compiler issues each chain of eight and waits for it before
  // the sums, and two waves per SIMD do not cover that.
  f16x8 op[8];
  const unsigned char* tile_row = nullptr;  // lane's row of the staged tile
  float gm[G], gs[G];
  auto score_groups = [&](auto rescue, auto shifted, auto partial, float u) __attribute__((always_inline)) {
    constexpr bool RES = decltype(rescue)::value, SHIFTED = decltype(shifted)::value;
    constexpr bool PARTIAL = decltype(partial)::value;
    f32x16 acc[2];
    float e[16], m = 0.f, ms = 0.f, sum = 0.f;
    // Part k of 8 of group gr's sums (its products are in acc[gr & 1]).
    auto sums_part = [&](auto group, auto part_of_8) __attribute__((always_inline)) {
      constexpr int gr = decltype(group)::value, k = decltype(part_of_8)::value;
      f32x16& v = acc[gr & 1];
      if constexpr (k == 0) {
        const int t0 = part * S::TOK + 32 * gr;  // the group's first token
        int lim = nb - t0 - 4 * half;            // tokens left, from the lane's first on
        if constexpr (PARTIAL) asm volatile("" : "+v"(lim));  // compared at each use: 16 masks kept for the loop would spill
        if constexpr (RES) {
          // Rescue logit of token t: acc + |q_t| u = nq_row u + (acc + (|q_t| - nq_row) u).
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const float4 nq4 = *reinterpret_cast<const float4*>(nq_s + 32 * gr + 8 * q4 + 4 * half);
            v[4 * q4 + 0] = fmaf(nq4.x - nq_row, u, v[4 * q4 + 0]);
            v[4 * q4 + 1] = fmaf(nq4.y - nq_row, u, v[4 * q4 + 1]);
            v[4 * q4 + 2] = fmaf(nq4.z - nq_row, u, v[4 * q4 + 2]);
            v[4 * q4 + 3] = fmaf(nq4.w - nq_row, u, v[4 * q4 + 3]);
          }
        }
        if constexpr (PARTIAL) {
#pragma unroll
          for (int r = 0; r < 16; ++r) v[r] = 8 * (r >> 2) + (r & 3) >= lim ? -INFINITY : v[r];
        }
        if constexpr (SHIFTED) {
          m = v[0];
#pragma unroll
          for (int r = 1; r < 16; ++r) m = fmaxf(m, v[r]);
          m = half_max(m);
          ms = PARTIAL && m == -INFINITY ? 0.f : m;  // no token in the group
        }
      }
      // (Sums start from their first term: an added 0 is an instruction the
      // compiler must keep, since 0 + -0 is not -0.)
      e[2 * k] = fast_exp2(SHIFTED ? v[2 * k] - ms : v[2 * k]);
      e[2 * k + 1] = fast_exp2(SHIFTED ? v[2 * k + 1] - ms : v[2 * k + 1]);
      if constexpr (k == 1) sum = e[0] + e[1];
      if constexpr (k > 1) sum = (sum + e[2 * k - 2]) + e[2 * k - 1];
      if constexpr (k == 7) {
        sum = (sum + e[14]) + e[15];
        gs[gr] = half_sum(sum);
        gm[gr] = RES ? m + nq_row * u : m;
      }
    };
    auto chain = [&](auto group) __attribute__((always_inline)) {
      constexpr int gr = decltype(group)::value;
      f32x16 a = {};
      // (Opaque: |q| of every operand, kept for the loop, would spill.)
      uint32_t sign_off = 0x7fff7fffu;
      if constexpr (MODE == kSelectBox) asm volatile("" : "+s"(sign_off));
      unroll<8>([&](auto ks_t) __attribute__((always_inline)) {
        constexpr int ks = decltype(ks_t)::value;
        a = mfma_f16(qa[gr][ks], op[ks], a);
        if constexpr (MODE == kSelectBox) {
          // + |q| . h_b: Eq. quest_box written as q . v_b + |q|^T h_b.
          uint32_t w[4];
          __builtin_memcpy(w, &qa[gr][ks], 16);
#pragma unroll
          for (int x = 0; x < 4; ++x) w[x] &= sign_off;
          f16x8 qabs;
          __builtin_memcpy(&qabs, w, 16);
          const f16x8 hop = *reinterpret_cast<const f16x8*>(tile_row + 2 * kTileBytes +
                                                            16 * tile_chunk(l32, 2 * ks + half));
          a = mfma_f16(qabs, hop, a);
        }
        if constexpr (gr > 0) {
          sums_part(std::integral_constant<int, gr - 1>{}, ks_t);
          __builtin_amdgcn_sched_barrier(0);
        }
      });
      acc[gr & 1] = a;
    };
    unroll<G>(chain);
    unroll<8>([&](auto k) __attribute__((always_inline)) { sums_part(std::integral_constant<int, G - 1>{}, k); });
  };
  // The block score of lane row l32 from all groups' pairs, in group order.
  auto merge = [&](bool plain, auto m_of, auto s_of) __attribute__((always_inline)) {
    if (plain) {  // one shift for all groups
      float sum = s_of(0);
#pragma unroll
      for (int k = 1; k < TG; ++k) sum += s_of(k);
      return m_of(0) + log2f(sum);
    }
    float top = m_of(0);
#pragma unroll
    for (int k = 1; k < TG; ++k) top = fmaxf(top, m_of(k));
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < TG; ++k) {
      const float s = s_of(k);
      if (s > 0.f) sum += s * fast_exp2(m_of(k) - top);
    }
    return top + log2f(sum);
  };
  auto merge_own = [&](bool plain) __attribute__((always_inline)) {
    return merge(plain, [&](int k) { return gm[k]; }, [&](int k) { return gs[k]; });
  };
  // A shared row: the wave's pairs to the stage, and the merge from it
  // (after a barrier).
  auto put_stage = [&](int buf) __attribute__((always_inline)) {
    if (half == 0) {
#pragma unroll
      for (int gr = 0; gr < G; ++gr)
        stage[(buf * TG + part * G + gr) * kTile + l32] = make_float2(gm[gr], gs[gr]);
    }
  };
  auto merge_stage = [&](int buf, bool plain) __attribute__((always_inline)) {
    return merge(plain, [&](int k) { return stage[(buf * TG + k) * kTile + l32].x; },
                 [&](int k) { return stage[(buf * TG + k) * kTile + l32].y; });
  };
  constexpr std::true_type yes{};
  constexpr std::false_type no{};
  // (Each form is compiled where it is common; the rest take the general one.)
  auto score = [&](auto rescue, bool plain, float u) __attribute__((always_inline)) {
    if constexpr (kBound) {
      if (plain && nb == BS) score_groups(rescue, no, no, u);
      else if (plain) score_groups(rescue, no, yes, u);
      else score_groups(rescue, yes, yes, u);
    } else {
      if (nb == BS) score_groups(rescue, yes, no, u);
      else score_groups(rescue, yes, yes, u);
    }
  };

  // ---- Base pass: every candidate's score (full-L2: rescue scores with beta = 1).
  constexpr bool kBaseIsRescue = MODE == kSelectFullL2;
  constexpr bool kUplift = kDual || MODE == kSelectFullL2;
  float u_cur = 0.f, cn_cur = 0.f, u_prev = 0.f;
  auto fetch_u = [&](int tile) __attribute__((always_inline)) {
    const int b = min(tile * kTile + l32, M - 1);
    if constexpr (kUplift) u_cur = ug[b];
    if constexpr (kBound) cn_cur = cng[b];
  };
  fetch_u(0);
  // Row maxima (per lane until the end): of the scores, and, dual, of the lower
  // bounds L_b + nq_min u_b of the rescue scores.
  float mb = -INFINITY, lbv = -INFINITY;
  auto settle = [&](int tile, float score_b, float u) __attribute__((always_inline)) {
    const int b = tile * kTile + l32;
    if (b < n_cand) {
      if (half == 0 && part == 0) L[b] = score_b;
      mb = fmaxf(mb, score_b);
      if constexpr (kDual) lbv = fmaxf(lbv, score_b + nq_min * u);
    }
  };
  bool plain_prev = false;
  for (int tile = 0; tile < n_tiles; ++tile) {
    // This wave's part of the tile, its uplifts and norms (vmcnt 0), and its pairs
    // and scores in LDS (lgkmcnt 0: left to the barrier, the compiler drops that
    // wait on the way round the loop, because another one stands right before it).
    __builtin_amdgcn_s_waitcnt(0x0070);
    __syncthreads();                     // the tile is complete, and the other buffer free
    const float u = u_cur, cn = cn_cur;
    if (tile + 1 < n_tiles) {
      issue_tile(tile + 1);
      fetch_u(tile + 1);
    }
    if constexpr (WPR > 1) {
      if (tile > 0) settle(tile - 1, merge_stage((tile - 1) & 1, plain_prev), u_prev);
    }
    if (tile * kTile < n_cand) {
      tile_row = smem + (tile & 1) * kTileBytes + l32 * 256;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
        op[ks] = *reinterpret_cast<const f16x8*>(tile_row + 16 * tile_chunk(l32, 2 * ks + half));
      // Unshifted sums where the tile's exponents are bounded: |q_t . c'_b| <=
      // |q_t| |c'_b| (Cauchy-Schwarz), and rescue logits relative to nq_row u
      // lie in [-nq_row (|c'_b| + u), nq_row |c'_b|].  The waves of a shared row
      // read the same values and take the same path.
      const float up = kBaseIsRescue ? u * u_scale : 0.f;
      bool plain = false;
      if constexpr (kBound) plain = __all(tile * kTile + l32 >= n_cand || nq_row * (cn + up) <= kPlainBound);
      if constexpr (kBaseIsRescue) score(yes, plain, up);
      else score(no, plain, 0.f);
      if constexpr (WPR > 1) {
        put_stage(tile & 1);
        plain_prev = plain;
        u_prev = u;
      } else {
        settle(tile, merge_own(plain), u);
      }
    }
  }
  if constexpr (WPR > 1) {
    __syncthreads();
    settle(n_tiles - 1, merge_stage((n_tiles - 1) & 1, plain_prev), u_prev);
    __syncthreads();  // L is complete
  } else {
    wave_lds_fence();
  }
  if (!live) return;  // (a shared row is always live; no barrier follows otherwise)
  mb = wave_max(mb);

  // ---- Thresholds.  Dual: the rescue branch scores only the blocks that can
  // reach its threshold: every token's rescue logit lies between its base logit
  // plus nq_min u_b and plus nq_row u_b, so L_res(b) <= U(b) = L_base(b) + nq_row
  // u_b, and the row's largest rescue score is at least LB = max_b L_base(b) +
  // nq_min u_b.  A block with U(b) < LB + log2 tau_rescue can be neither
  // selected by the rescue branch nor its maximum; a block with u_b = 0 has
  // L_res(b) = L_base(b).  The remaining blocks (a few percent) get their exact
  // rescue scores, 32 at a time as the listing finds them.
  float thr_base = mb + c.log2_tau_base, thr_res = -INFINITY;
  static_assert(kMaxBlocks <= 64 * kWave, "one mask of 64 blocks per lane");
  // Per 64 blocks (lane k: blocks 64 k ..), bit b % 64: selected by
  // the base branch; L[b] is the rescue score (no uplift, or a candidate).
  uint64_t in_base = 0, res_in_l = 0;
  if constexpr (MODE == kSelectFullL2) thr_res = mb + c.log2_tau_rescue;
  if constexpr (kDual) {
    if (!c.rescue_all) {
      const float cut = wave_max(lbv) + c.log2_tau_rescue - kCandSlack;
      float mres = -INFINITY;  // over the blocks whose L[b] is already their rescue score
      int head = 0, pending = 0;
      float u_next = ug[min(lane, n_cand - 1)];
      for (int base = 0; base < n_cand; base += kWave) {
        const int b = base + lane;
        const float u = u_next;
        u_next = ug[min(b + kWave, n_cand - 1)];
        bool is_cand = false, sel = false, in_l = false;
        if (b < n_cand) {
          const float lb = L[b];
          is_cand = u > 0.f && lb + nq_row * u >= cut;
          sel = lb >= thr_base;
          in_l = !(u > 0.f) || is_cand;
          if (!(u > 0.f)) mres = fmaxf(mres, lb);
        }
        const uint64_t m_base = __ballot(sel), m_res = __ballot(in_l), m_cand = __ballot(is_cand);
        if (lane == base >> 6) {
          in_base = m_base;
          res_in_l = m_res;
        }
        if (is_cand) {
          const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m_cand >> 32),
                                                       __builtin_amdgcn_mbcnt_lo((uint32_t)m_cand, 0u));
          ring[(head + pending + before) & (kCandRing - 1)] = b;
        }
        pending += __popcll(m_cand);
        wave_lds_fence();
        const bool last = base + kWave >= n_cand;
        while (pending >= kTile || (last && pending > 0)) {
          const bool have = l32 < pending;
          const int rb = have ? ring[(head + l32) & (kCandRing - 1)] : 0;
          const _Float16* crow = cg + (size_t)rb * kHeadDim + 8 * half;
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) op[ks] = *reinterpret_cast<const f16x8*>(crow + 16 * ks);
          const float ru = have ? ug[rb] : 0.f, rcn = cng[rb];
          const bool plain = __all(!have || nq_row * (rcn + ru) <= kPlainBound);
          score(yes, plain, ru);
          float lres;
          if constexpr (WPR > 1) {
            __syncthreads();  // the previous round's pairs are read
            put_stage(0);
            __syncthreads();
            lres = merge_stage(0, plain);
          } else {
            lres = merge_own(plain);
          }
          if (have) {
            if (half == 0 && part == 0) L[rb] = lres;
            mres = fmaxf(mres, lres);
          }
          head += kTile;
          pending = max(pending - kTile, 0);
        }
      }
      thr_res = wave_max(mres) + c.log2_tau_rescue;
    }
  }
  if (WPR > 1 && part != 0) return;  // the row's first wave writes its list
  wave_lds_fence();
  const bool recent_row = i >= M - c.n_recent;

  // ---- Box: fixed budget, the k = max(1, ceil(rho |C_i|)) highest scores
  // (ties with the k-th kept).  The k-th largest is found by a bitwise
  // bisection on order-preserving integer keys of the scores: it is the
  // largest key v with #{key >= v} >= k; a v met by exactly k keys on the way
  // keeps the same blocks.
  auto okey = [](float f) __attribute__((always_inline)) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
  };
  uint32_t kth_key = 0u;
  if constexpr (MODE == kSelectBox) {
    const int k = max(1, min(n_cand, (int)ceil((double)c.budget * (double)n_cand - 1e-12)));
    auto search = [&](auto count_from) __attribute__((always_inline)) {
      for (int bit = 31; bit >= 0; --bit) {
        const uint32_t cand_key = kth_key | (1u << bit);
        const int total = count_from(cand_key);
        if (total >= k) kth_key = cand_key;
        if (total == k) break;
      }
    };
    // Four scores a lane at a time: one at a time, each of a row's 32 x n_cand / 64
    // steps waits for its LDS read (131072 tokens, 1 head, B = 128: 94 us, now 70).
    // (No searched key is 0: a slot past the row is never counted.)
    uint32_t key[4];
    auto load4 = [&](int base) __attribute__((always_inline)) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int b = base + j * kWave + lane;
        key[j] = b < n_cand ? okey(L[b]) : 0u;
      }
    };
    auto count4 = [&](uint32_t cand_key) __attribute__((always_inline)) {
      int total = 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) total += __popcll(__ballot(key[j] >= cand_key));
      return total;
    };
    if (n_cand <= 4 * kWave) {
      load4(0);
      search(count4);
    } else {
      search([&](uint32_t cand_key) __attribute__((always_inline)) {
        int total = 0, base = 0;
        for (; base + 4 * kWave <= n_cand; base += 4 * kWave) {
#pragma unroll
          for (int j = 0; j < 4; ++j) key[j] = okey(L[base + j * kWave + lane]);
          total += count4(cand_key);
        }
        load4(base);
        return total + count4(cand_key);
      });
    }
  }

  // ---- Union with forced blocks and compaction to an ascending list.
  int32_t* out = c.indices + (int64_t)h * c.capacity + (int64_t)i * (i + 1) / 2;
  int total = 0;
  for (int base = 0; base < n_cand; base += kWave) {
    const int b = base + lane;
    const float lb = L[min(b, n_cand - 1)];
    bool sel = recent_row || b < c.n_sink || b > i - c.n_local;
    if constexpr (kDual) {
      // (The masks are filled only when the rescue threshold is in use.)
      const int w = base >> 6;
      auto word = [&](uint64_t m) __attribute__((always_inline)) {
        return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, w) |
               (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(m >> 32), w) << 32;
      };
      sel |= c.base_all || c.rescue_all || ((word(in_base) >> lane) & 1) ||
             (((word(res_in_l) >> lane) & 1) && lb >= thr_res);
    } else if constexpr (MODE == kSelectCentroid) {
      sel |= c.base_all || lb >= thr_base;
    } else if constexpr (MODE == kSelectFullL2) {
      sel |= c.rescue_all || lb >= thr_res;
    } else {
      sel |= okey(lb) >= kth_key;
    }
    sel = sel && b < n_cand;
    const uint64_t ballot = __ballot(sel);
    const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32),
                                                 __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
    if (sel) out[total + before] = b;
    total += __popcll(ballot);
  }
  if (lane == 0) c.counts[(size_t)h * c.ldm + i] = total;
}

// Waves per SIMD that the register budget is set for: the wave's Q takes one
// VGPR per token.
template <int T>
constexpr int kWavesPerEu = T == 32 ? 4 : T == 64 ? 3 : 2;

// Workgroup j takes chunk j / n_kv of KV head j % n_kv: late (long) rows first
// over all heads, and with 1, 2, 4 or 8 KV heads each XCD (workgroup j runs on
// XCD j % 8) reads one head's centroids.
template <int BS, int MODE, int T, int W>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(kWavesPerEu<T>))) void select_kernel(
    SelectCore c) {
  extern __shared__ __align__(1024) unsigned char smem[];
  select_rows<BS, MODE, T, W>(c, blockIdx.x % c.n_kv, blockIdx.x / c.n_kv, smem);
}

// Every sequence of a batch in one launch, sequence-major: workgroups wg.at[s] ..
// wg.at[s + 1] - 1 (per KV head) are sequence s's.  The core is narrowed to the
// sequence: its tokens, blocks, counts and list slots (the head strides stay
// the batch's).
struct SeqChunks {
  int at[kMaxSeqs + 1];
};

template <int BS, int T, int W>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(kWavesPerEu<T>))) void select_varlen_kernel(
    SelectCore c, const SeqTable t, const SeqChunks wg) {
  extern __shared__ __align__(1024) unsigned char smem[];
  const int chunk = blockIdx.x / c.n_kv;
  const int sq = seq_of(wg.at, t.n, chunk);
  c.N = t.tok[sq + 1] - t.tok[sq];
  c.M = t.blk[sq + 1] - t.blk[sq];
  c.Q += t.tok[sq] * c.q_tok;
  c.cent16 += (size_t)t.blk[sq] * kHeadDim;
  c.uplift += t.blk[sq];
  c.cnorm += t.blk[sq];
  c.counts += t.blk[sq];
  c.indices += t.cap[sq];
  select_rows<BS, kSelectDual, T, W>(c, blockIdx.x % c.n_kv, chunk - wg.at[sq], smem);
}

static SelectCore make_select_core(const SelectArgs& a) {
  SelectCore c;
  c.Q = a.Q;
  c.q_head = a.q_head;
  c.q_tok = a.q_tok;
  c.N = a.n_tokens;
  c.M = a.n_blocks;
  c.group = a.n_q_heads / a.n_kv_heads;
  c.n_kv = a.n_kv_heads;
  c.ldm = a.n_blocks;
  c.cent16 = a.cent16;
  c.half16 = a.half16;
  c.uplift = a.uplift;
  c.cnorm = a.cnorm;
  c.radii = a.radii;
  c.budget = a.budget;
  c.log2_tau_base = a.tau_base > 0.f ? log2f(a.tau_base) : -INFINITY;
  c.log2_tau_rescue = a.tau_rescue > 0.f ? log2f(a.tau_rescue) : -INFINITY;
  c.base_all = a.tau_base <= 0.f;
  c.rescue_all = a.tau_rescue <= 0.f;
  c.n_sink = a.n_sink;
  c.n_local = a.n_local;
  c.n_recent = a.n_recent;
  c.counts = a.counts;
  c.indices = a.indices;
  c.capacity = a.capacity;
  return c;
}

// Workgroups that n_blocks rows of `group` heads take per KV head.
template <int BS, int T, int W>
static int chunks_of(int n_blocks, int group) {
  constexpr int rpw = RowSplit<BS, T, W>::RPW;
  return (int)(((int64_t)n_blocks * group + rpw - 1) / rpw);
}

template <int BS, int MODE, int T, int W>
static hipError_t launch_select_w(const SelectCore& c, hipStream_t s) {
  const size_t smem = SelectLds<BS, MODE, T, W>::bytes(c.M);
  hipError_t e = hipFuncSetAttribute((const void*)select_kernel<BS, MODE, T, W>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((select_kernel<BS, MODE, T, W>), dim3(chunks_of<BS, T, W>(c.M, c.group) * c.n_kv), dim3(W * 64), smem,
                     s, c);
  return hipGetLastError();
}

template <int BS, int T, int W>
static hipError_t launch_select_mode(const SelectCore& c, int mode, hipStream_t s) {
  switch (mode) {
    case kSelectDual: return launch_select_w<BS, kSelectDual, T, W>(c, s);
    case kSelectCentroid: return launch_select_w<BS, kSelectCentroid, T, W>(c, s);
    case kSelectFullL2: return launch_select_w<BS, kSelectFullL2, T, W>(c, s);
    case kSelectBox: return launch_select_w<BS, kSelectBox, T, W>(c, s);
    default: return hipErrorInvalidValue;
  }
}

// f(integral_constant<int, T>, integral_constant<int, W>) with the split of
// `rows` rows of up to M blocks.
template <int BS, typename F>
static hipError_t with_split(int M, int rows, F f) {
  const int tokens = row_tokens(BS, M, rows);
  constexpr std::integral_constant<int, 64> t64{};
  constexpr std::integral_constant<int, 2> w2{};
  constexpr std::integral_constant<int, 4> w4{};
  if constexpr (BS == 256) {
    return f(t64, w4);
  } else {
    if (tokens == 32) return f(std::integral_constant<int, 32>{}, std::integral_constant<int, BS / 32>{});
    if constexpr (BS == 128) {
      if (tokens == 64) return f(t64, w2);
      return f(std::integral_constant<int, 128>{}, w4);
    } else {
      // Four rows per workgroup (128K: 1253 us, two rows 1500, eight 1490), until
      // their score rows leave a compute unit's 160 KB of LDS to one workgroup
      // (256K: 7670 us, two rows 6530).
      if (2 * SelectLds<BS, kSelectDual, 64, 4>::bytes(M) > 160 * 1024) return f(t64, w2);
      return f(t64, w4);
    }
  }
}

template <int BS>
static hipError_t launch_select_bs(const SelectCore& c, int mode, hipStream_t s) {
  return with_split<BS>(c.M, c.M * c.group * c.n_kv, [&](auto t, auto w) {
    return launch_select_mode<BS, decltype(t)::value, decltype(w)::value>(c, mode, s);
  });
}

template <int BS, int T, int W>
static hipError_t launch_select_varlen_w(const SelectCore& c, const SeqTable& t, int m_max, hipStream_t s) {
  SeqChunks wg{};
  for (int q = 0; q < t.n; ++q) wg.at[q + 1] = wg.at[q] + chunks_of<BS, T, W>(t.blk[q + 1] - t.blk[q], c.group);
  const size_t smem = SelectLds<BS, kSelectDual, T, W>::bytes(m_max);
  hipError_t e = hipFuncSetAttribute((const void*)select_varlen_kernel<BS, T, W>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((select_varlen_kernel<BS, T, W>), dim3(wg.at[t.n] * c.n_kv), dim3(W * 64), smem, s, c, t, wg);
  return hipGetLastError();
}

template <int BS>
static hipError_t launch_select_varlen_bs(const SelectCore& c, const SeqTable& t, hipStream_t s) {
  int m_max = 0;
  for (int q = 0; q < t.n; ++q) m_max = t.blk[q + 1] - t.blk[q] > m_max ? t.blk[q + 1] - t.blk[q] : m_max;
  return with_split<BS>(m_max, t.blk[t.n] * c.group * c.n_kv, [&](auto tok, auto w) {
    return launch_select_varlen_w<BS, decltype(tok)::value, decltype(w)::value>(c, t, m_max, s);
  });
}

hipError_t launch_select_varlen(const SelectArgs& a, const SeqTable& t, hipStream_t s) {
  const SelectCore c = make_select_core(a);
  switch (a.block_size) {
    case 64: return launch_select_varlen_bs<64>(c, t, s);
    case 128: return launch_select_varlen_bs<128>(c, t, s);
    case 256: return launch_select_varlen_bs<256>(c, t, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_select(const SelectArgs& a, hipStream_t s) {
  const SelectCore c = make_select_core(a);
  switch (a.block_size) {
    case 64: return launch_select_bs<64>(c, a.mode, s);
    case 128: return launch_select_bs<128>(c, a.mode, s);
    case 256: return launch_select_bs<256>(c, a.mode, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace rbs
