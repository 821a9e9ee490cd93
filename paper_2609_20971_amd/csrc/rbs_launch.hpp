// Host-side launchers of the RBS kernels (internal to librbs; the public
// surface is include/rbs.h).  Arguments are assumed validated by api.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <limits.h>
#include <stdint.h>

namespace rbs {

// Element strides of the bf16 tensors between heads and between tokens (the
// head dimension is contiguous): Q and O share q_*, K and V share kv_*.
struct Strides {
  int64_t q_head, q_tok, kv_head, kv_tok;
};

struct StatsArgs {
  const uint16_t* K;
  int64_t kv_head, kv_tok;  // K strides
  int n_tokens, n_kv_heads, block_size, n_blocks;
  float* centroids;
  float* radii;
  float* beta;
  float* quantiles;
  _Float16* cent16;  // select-ready centroids [H_kv][M][d]
  float* uplift;     // select-ready rescue uplift [H_kv][M]
  float* cnorm;      // norm of each select-ready centroid [H_kv][M]
};

struct BoxArgs {
  const uint16_t* K;
  int64_t kv_head, kv_tok;  // K strides
  int n_tokens, n_kv_heads, block_size, n_blocks;
  float* center;
  float* half;
  _Float16* center16;  // select-ready copies [H_kv][M][d]
  _Float16* half16;
};

struct SelectArgs {
  const uint16_t* Q;
  int64_t q_head, q_tok;  // Q strides
  int n_tokens, n_q_heads, n_kv_heads, block_size, n_blocks;
  int mode = 0;                       // SelectMode (select.hip)
  const _Float16* cent16;             // box: scaled box centres
  const _Float16* half16 = nullptr;   // box: scaled box half-widths
  const float* uplift;
  const float* cnorm = nullptr;       // select-ready centroid norms (not the box's)
  const float* radii = nullptr;       // full-L2
  float budget = 0.f;                 // box: budget fraction
  float tau_base, tau_rescue;
  int n_sink, n_local, n_recent;
  int32_t* counts;
  int32_t* indices;
  int64_t capacity;
};

struct AttnArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  Strides st;  // Q and O; K and V
  int n_tokens, n_q_heads, n_kv_heads, block_size, n_blocks;
  const int32_t* counts;
  const int32_t* indices;
  int64_t capacity;
  float scale;
  uint16_t* O;
  float* lse;
  int* queue = nullptr;  // persistent launch's work queues (kQueueInts ints), or one workgroup per item
  bool selected = false;  // the lists are this call's own selection (work_order, queue_line)
};

// Select-ready summary, each part 256-byte aligned: f16 centroids scaled by
// log2(e)/sqrt(d) [H_kv][M][d] | fp32 uplift [H_kv][M] | fp32 norms of the
// scaled centroids [H_kv][M].
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
inline size_t summary_uplift_offset(int n_kv_heads, int n_blocks) {
  return align256((size_t)n_kv_heads * n_blocks * 128 * sizeof(_Float16));
}
inline size_t summary_cnorm_offset(int n_kv_heads, int n_blocks) {
  return align256(summary_uplift_offset(n_kv_heads, n_blocks) + (size_t)n_kv_heads * n_blocks * sizeof(float));
}
inline size_t summary_bytes(int n_kv_heads, int n_blocks) {
  return summary_cnorm_offset(n_kv_heads, n_blocks) + (size_t)n_kv_heads * n_blocks * sizeof(float);
}

// A batch of independent sequences packed along the token axis (the varlen
// entry points).  Sequence s holds tokens tok[s] .. tok[s+1]-1 of every head,
// blocks blk[s] .. blk[s+1]-1 of the block arrays and index-list slots
// cap[s] .. cap[s+1]-1 of every query head; a single sequence is {n = 1}.
constexpr int kMaxSeqs = 64;
constexpr int kMaxBlocks = 4096;  // key blocks of a sequence (api.hip refuses more)
constexpr int kMaxDevices = 64;  // devices whose resident-grid size the launchers cache
constexpr int kQueues = 8;       // work queues of a persistent attention launch, one per XCD
constexpr int kQueueInts = 64;   // its workspace: 256 bytes, the eight counters spread over it
constexpr int kQueueStride = kQueueInts / kQueues;
struct SeqTable {
  int n;
  int tok[kMaxSeqs + 1];
  int blk[kMaxSeqs + 1];
  int64_t cap[kMaxSeqs + 1];
};

// The sequence holding position x of an offset array off[0..n] (off[0] = 0,
// ascending): the largest s < n with off[s] <= x.
__host__ __device__ inline int seq_of(const int* off, int n, int x) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= x) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The rows (query blocks) of all sequences of a batch by descending row number
// i within their sequence, so that a launch's longest rows come first whatever
// sequence they belong to.  Sequences sorted by descending block count:
// seq[0], seq[1], ...; level k (1 <= k <= n) holds the row numbers that exactly
// the first k of them have, the k rows of one number next to each other:
// row r of level k (start[k] <= r < start[k + 1]) is number
// blocks[k - 1] - 1 - (r - start[k]) / k of sequence seq[(r - start[k]) % k].
struct RowOrder {
  int n;
  int seq[kMaxSeqs];
  int blocks[kMaxSeqs];     // block count of seq[k]
  int start[kMaxSeqs + 2];  // index by level; start[0] = start[1] = 0, start[n + 1] = all rows
};

inline RowOrder rows_by_length(const SeqTable& t) {
  RowOrder o{};
  o.n = t.n;
  for (int q = 0; q < t.n; ++q) {  // insertion sort, stable
    const int m = t.blk[q + 1] - t.blk[q];
    int p = q;
    for (; p > 0 && o.blocks[p - 1] < m; --p) {
      o.blocks[p] = o.blocks[p - 1];
      o.seq[p] = o.seq[p - 1];
    }
    o.blocks[p] = m;
    o.seq[p] = q;
  }
  for (int k = 1; k <= t.n; ++k)
    o.start[k + 1] = o.start[k] + k * (o.blocks[k - 1] - (k < t.n ? o.blocks[k] : 0));
  return o;
}

// Row r of the order: its sequence and row number.
__host__ __device__ inline void row_at(const RowOrder& o, int r, int* seq, int* i) {
  int lo = 1, hi = o.n;  // the largest level with start <= r; empty levels share a start with the next one
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (o.start[mid] <= r) lo = mid;
    else hi = mid - 1;
  }
  const int off = r - o.start[lo];
  *seq = o.seq[off % lo];
  *i = o.blocks[lo - 1] - 1 - off / lo;
}

// Workgroup id -> logical work item, so that groups of 8 consecutive items (of a
// group of 8: the query heads of one KV head, same query block) run on the same
// XCD (workgroups are dealt to the 8 XCDs round-robin by id) and share its L2.
__host__ __device__ inline int xcd_remap(int id, int total) {
  const int full = total & ~63;
  if (id >= full) return id;
  const int x = id & 7, s = id >> 3;
  return ((s >> 3) << 6) + (x << 3) + (s & 7);
}

// The order of a launch's work slots (query head, query block), late (long)
// rows first in each.
enum WorkOrder {
  kByGroup = 0,  // all rows of one KV head's group, then the next group's: every XCD works on the same KV head
  kByRow = 1,    // one query block of every head, then the block before it; 8 consecutive heads to an XCD
  kByXcdRow = 2, // the same, each XCD on KV heads of its own
};

// Whether each XCD can have KV heads of its own: one head that 8 / n_kv XCDs
// share, or n_kv / 8 heads.
__host__ __device__ inline bool kv_heads_tile_xcds(int n_kv) { return n_kv <= 8 ? 8 % n_kv == 0 : n_kv % 8 == 0; }

// Work slot id (of total = M hq) -> (query head h, query block i).
__host__ __device__ inline void work_of(int id, int total, int M, int hq, int group, int order, int& h, int& i) {
  if (order == kByXcdRow) {
    // XCD id % 8 takes the rows of its own KV heads in order; the 8 / n_kv XCDs
    // of one head every 8 / n_kv-th row each, up to the last full set of rows.
    const int n_kv = hq / group;
    const int sharing = n_kv < 8 ? 8 / n_kv : 1, own = n_kv < 8 ? 1 : n_kv / 8, heads = 8 / sharing;
    const int rows = M - M % sharing;
    if (id < rows * hq) {
      const int x = id & 7, unit = (id >> 3) / group;  // unit: one row of one KV head
      i = M - 1 - (unit / own * sharing + x / heads);
      h = (x % heads + 8 * (unit % own)) * group + (id >> 3) % group;
      return;
    }
  }
  const int work = order == kByXcdRow ? id : xcd_remap(id, total);
  if (order != kByGroup) {
    i = M - 1 - work / hq;
    h = work % hq;
    return;
  }
  const int per_group = M * group;
  const int g = work / per_group;
  const int rem = work - g * per_group;
  i = M - 1 - rem / group;
  h = g * group + rem % group;
}

// Whether a launch over n_kv_heads heads of n_tokens K and V rows (row_bytes for
// the two together) goes by rows.  That starts the longest rows of every head
// first, where the order by groups starts the last group's longest rows last and
// ends on them alone; but it keeps all KV heads in use at once.  The line is
// where they still fit the 256 MiB Infinity Cache (half of it at B = 64, whose
// tiles are used for half as many queries).  Attention, by group against by row:
// 3001 dense tokens, 32 / 4 heads 128 / 102 us, 8192 565 / 518, 16384 1966 / 1928,
// 16384 with 8 / 8 heads 640 / 555, 64K with 64 / 8 heads 8.47 / 8.39 ms; past the
// line 128K with 64 / 8 heads 18.6 / 18.8 ms, 256K with 32 / 4 heads 23.3 / 23.6,
// 128K at B = 64 15.3 / 15.45 ms.
inline bool row_major_work(int n_tokens, int n_kv_heads, int row_bytes, int block_size) {
  return (int64_t)n_tokens * n_kv_heads * row_bytes <= (block_size >= 128 ? 256 : 128) * (int64_t(1) << 20);
}

// The order of a launch over one sequence.  Eight consecutive heads per XCD are
// one KV head for groups of 8 (both orders by rows are then the same); for other
// groups every XCD reads up to all KV heads, whose K and V its 4 MB L2 does not
// hold once many rows are in flight.  A KV head per XCD costs balance instead
// (heads differ in density), so it takes launches of many items: sparse lists,
// by row / by XCD's rows: 28 / 4 heads, B = 64, 16384 tokens (7168 items) 1374 /
// 976 us (by group 1060), 40 / 8 8100 tokens (5080) 700 / 513 (580), 12 / 2 40000
// tokens (7500) 1084 / 898 (920), 40 / 8, B = 128, 16384 (5120) 1181 / 1129
// (1175); the other way at 16384 tokens, 8 / 8 heads, B = 64 (2048 items) 325 /
// 390, B = 128 at 40000 tokens (2504) 584 / 616, and at B = 256 at every size (643
// / 722 with 1256 items).  FP8 tiles are half the size: B = 64, 28 / 4, 8100
// tokens (3556) 239 / 257, 16 / 16 16384 (4096) 326 / 344, 8 / 8 40000 (5000) 512
// / 454.  KV heads that do not tile the XCDs, by row / by group: B = 64, 20 / 5,
// 8100 tokens (2540) 264 / 324, 16384 (5120) 910 / 765; FP8 16384 423 / 467,
// 40000 (12500) 1329 / 1152.
//
// B = 64 and a whole number of KV heads per XCD (own_head_rows): from 1900 items
// on by XCD's rows, and through the queues, which level the heads' densities.  By
// row against that, 8 / 8 heads 16000 tokens (2000 items): selected lists 304 /
// 250 us, random ones 254 / 236, dense 669 / 562; 20000 328 / 275, 334 / 303, 1100 /
// 851; 16 / 16 10000 (2512) 242 / 213, 321 / 298, 513 / 443; fewer items 16 / 16
// 6000 (1504) 127 / 125, 150 / 166, 179 / 185; rows of 50 and 63 blocks, 40 / 8,
// 86 / 124 and 116 / 141.  Past the cache line an XCD's own heads still pay, by
// group against by XCD's rows: 8 / 8 49145 (192 MiB) 874 / 617, 699 / 686, 5841 /
// 4770; not on random lists with two heads per XCD or much more memory: 16 / 16
// 32000 (250 MiB) 912 / 787 selected but 1139 / 1204 random, 64000 1574 / 1405 and
// 2393 / 2786; 8 / 8 128000 (500 MiB) random 2084 / 2154.  selected: the lists are
// known to be a selection's.
constexpr int kOwnHeadItems = 1900, kOwnHeadBlocks = 96;
inline bool own_head_rows(int n_tokens, int n_q_heads, int n_kv_heads, int row_bytes, int block_size, int n_blocks,
                          bool selected) {
  return block_size == 64 && row_bytes > 256 && n_kv_heads % 8 == 0 && n_q_heads / n_kv_heads % 8 != 0 &&
         n_blocks > kOwnHeadBlocks && n_blocks * n_q_heads > kOwnHeadItems &&
         (int64_t)n_tokens * n_kv_heads * row_bytes <= (selected ? 512 : n_kv_heads == 8 ? 256 : 128) * (int64_t(1) << 20);
}

inline WorkOrder work_order(int n_tokens, int n_q_heads, int n_kv_heads, int row_bytes, int block_size, int n_blocks,
                            bool selected = false) {
  if (own_head_rows(n_tokens, n_q_heads, n_kv_heads, row_bytes, block_size, n_blocks, selected)) return kByXcdRow;
  if (!row_major_work(n_tokens, n_kv_heads, row_bytes, block_size)) return kByGroup;
  const bool tiles = kv_heads_tile_xcds(n_kv_heads);
  const int few = row_bytes > 256 ? 3072 : tiles ? 4096 : 8192;
  if (block_size > 128 || n_blocks * n_q_heads <= few) return kByRow;
  return tiles ? kByXcdRow : kByGroup;
}

// Items past which a launch goes through the queues (launch_slots), where the
// GPU holds `resident` workgroups at once, at B = 128 and 256.  At B = 256 one
// workgroup fills a compute unit and an item is long, so that the queues' own time
// (some 10 us a launch) is won back earlier.  Queues / per slot at twice and at
// three times the resident items: B = 256, 32 / 4 heads bf16 random lists 0.95 and
// 0.85, selected 0.99 and 1.01, dense 1.00 and 1.01; FP8 0.91 and 0.82, dense 1.01
// and 1.00; 8 / 1 bf16 0.97 and 0.94, 0.99 and 0.98, 0.93 and 0.99; at one and a
// half times 1.05, 1.03, 1.03; B = 128 32 / 4 1.03 and 0.92, 1.03 and 0.99, 1.03 and
// 1.03.
inline int general_line(int block_size, int resident) { return (block_size > 128 ? 2 : 3) * resident; }

// Items past which a bf16 launch over one sequence goes through the queues
// (general_line past B = 64).  At B = 64 the queues cost some 20 us a launch and 1
// us an item, which short rows do not
// win back.  Queues against per slot: 64 / 8 heads 3593 tokens (57 blocks, 3648
// items) selected lists 178 / 159, random ones 224 / 212, dense 257 / 247; 5000 (79)
// 254 / 234, 381 / 379, 464 / 458; 6137 (96) 294 / 323, 504 / 522, 654 / 621.  With
// one KV head every XCD has the same mix of rows and the queues only level their
// ends: selected lists, 8 / 1 heads 27026 tokens 267 / 238, 49145 290 / 266, 114681
// 443 / 425; random lists, 4 / 1 51200 481 / 525, 16 / 1 48000 1891 / 2023.
inline int queue_line(int n_tokens, int n_q_heads, int n_kv_heads, int block_size, int n_blocks, int resident,
                      bool selected) {
  if (block_size != 64) return general_line(block_size, resident);
  if (own_head_rows(n_tokens, n_q_heads, n_kv_heads, 512, block_size, n_blocks, selected)) return kOwnHeadItems;
  if (selected && n_kv_heads == 1) return INT_MAX;
  return n_blocks <= 80 ? 6 * resident : 3 * resident;
}

// The order of a launch over a batch: the longest rows of all sequences first
// (kByRow), or the sequences one after another (kByGroup).  The rows of a large
// batch keep the balance by themselves, and one sequence after another uses each
// one's K and V while they are near.  By sequence against by row, 32 / 4 heads,
// B = 128: 4 sequences of 150 to 4000 tokens 165 / 136 us, 40 of 500 tokens 209 /
// 174; 16 of 1 to 7001 (30 K tokens) 951 / 952 us and at B = 64 687 / 704; three
// of 30 K to 64 K 27.8 / 28.1 ms.  At B = 64 and groups other than 8 as for one
// sequence (work_order): two sequences, 28 / 4 heads (27 K tokens) 742 / 886 us,
// 40 / 8 (19 K) 802 / 1031, 20 / 5 (38 K) 1109 / 1518; B = 128 1859 / 1866, 1514 /
// 1515, 2502 / 2480.
inline WorkOrder batch_order(int n_tokens, int n_q_heads, int n_kv_heads, int block_size, int n_blocks) {
  if (!row_major_work(n_tokens, n_kv_heads, 512, block_size)) return kByGroup;
  if ((int64_t)n_tokens * n_q_heads > 3 << 18) return kByGroup;
  const bool eighths = n_q_heads / n_kv_heads % 8 == 0;  // eight consecutive heads share a KV head
  return block_size > 64 || eighths || n_blocks * n_q_heads <= 3072 ? kByRow : kByGroup;
}

// Tokens that one wave of a selection launch scores: a row (query block) of B
// tokens takes B / row_tokens waves.  rows: query heads x query blocks of the
// launch; n_blocks: of its longest sequence.
// Long rows (past kSharedRowBlocks blocks) are the launch's time by themselves
// where there are few: 32 tokens a wave, so that a row's tiles are scored side by
// side.  32 / 64 / 128 tokens a wave, B = 128, selection alone: 41200 tokens, 2
// heads (644 rows) 19.0 / 21.6 / 28.0 us, 70000 (1094) 27.2 / 31.4 / 43.0, 100000
// (1564) 44.8 / 43.6 / 54.5; 4 heads 41200 (1288) 25.9 / 24.9 / 33.2; box selector
// 70000, 2 heads 60 / 64 / 84; B = 64 30000, 2 heads (938) 20.9 / 23.6, box 44 /
// 52, 4 heads (1876) 23.4 / 25.2, 64000 tokens 65.5 / 56.8.
// B = 128, more rows: shared by two waves a row holds 64 VGPRs of Q in each and
// runs at three waves per SIMD instead of two, which covers short rows' latencies
// better; long rows are bound by their tiles, where one wave per row reads each
// staged operand half as often.  64 / 128 tokens a wave, 32 / 4 heads: 16K (128
// blocks) 36.9 / 41.4 us, 32K 82 / 88, 45K (352) 146 / 141, 64K 255 / 241, 128K
// 770 / 696; fewer rows: 8 heads 52000 (3256) 46.6 / 52.5, 6 heads 100000 (4692)
// 91.9 / 90.0, 4 heads 128K (4096) 99.4 / 94.4.
// B = 256: 64 against 128 32K 64 / 87 us, 128K 500 / 505, 256K 1575 / 1538.
constexpr int kSharedRowBlocks = 320;
constexpr int kFewRows = 1200, kSharedRows = 4000;
inline int row_tokens(int block_size, int n_blocks, int rows) {
  const bool long_rows = n_blocks > kSharedRowBlocks;
  if (block_size <= 128 && long_rows && rows <= kFewRows) return 32;
  return block_size == 128 && long_rows && rows > kSharedRows ? 128 : 64;
}

inline SeqTable single_sequence(int n_tokens, int n_blocks) {
  SeqTable t{};
  t.n = 1;
  t.tok[1] = n_tokens;
  t.blk[1] = n_blocks;
  t.cap[1] = (int64_t)n_blocks * (n_blocks + 1) / 2;
  return t;
}

hipError_t launch_stats(const StatsArgs& a, hipStream_t s);
// The select-ready summary from fp32 centroids, radii and beta [H_kv][M].
hipError_t launch_summarize(const float* centroids, const float* radii, const float* beta, int n_kv_heads,
                            int n_blocks, _Float16* cent16, float* uplift, float* cnorm, hipStream_t s);
hipError_t launch_box(const BoxArgs& a, hipStream_t s);
hipError_t launch_select(const SelectArgs& a, hipStream_t s);
hipError_t launch_attention(const AttnArgs& a, hipStream_t s);
// The persistent attention launch with its queue counters in the library's
// per-device static scratch (a.queue is ignored): allocates nothing.
hipError_t launch_attention_noalloc(AttnArgs a, hipStream_t s);
hipError_t launch_dense_indices(int n_q_heads, int n_blocks, int64_t capacity, int32_t* counts,
                                int32_t* indices, hipStream_t s);

// FP8 attention inputs (fp8.hip).  The bf16 inputs have the strides st; the
// FP8 copies are dense; O is written with Q's strides.
hipError_t launch_fp8_amax(const uint16_t* Q, const uint16_t* K, const uint16_t* V, const Strides& st, int n_tokens,
                           int n_q_heads, int n_kv_heads, float* amax, hipStream_t s);
hipError_t launch_fp8_pack(const uint16_t* Q, const uint16_t* K, const uint16_t* V, const Strides& st, int n_tokens,
                           int n_q_heads, int n_kv_heads, int block_size, int n_blocks, const float* amax, uint8_t* Q8,
                           uint8_t* K8, uint8_t* V8t, hipStream_t s);
hipError_t launch_attention_fp8(const uint8_t* Q8, const uint8_t* K8, const uint8_t* V8t, const float* amax,
                                int n_tokens, int n_q_heads, int n_kv_heads, int block_size, int n_blocks,
                                const int32_t* counts, const int32_t* indices, int64_t capacity, float scale,
                                uint16_t* O, int64_t o_head, int64_t o_tok, float* lse, int* queue, hipStream_t s);

// Varlen launchers: the Args hold the batch totals (n_tokens = T, n_blocks and
// capacity = the table's last offsets); every sequence runs in the same launch.
hipError_t launch_stats_varlen(const StatsArgs& a, const SeqTable& t, hipStream_t s);
hipError_t launch_select_varlen(const SelectArgs& a, const SeqTable& t, hipStream_t s);
hipError_t launch_attention_varlen(const AttnArgs& a, const SeqTable& t, hipStream_t s);
hipError_t launch_dense_indices_varlen(int n_q_heads, const SeqTable& t, int32_t* counts, int32_t* indices,
                                       hipStream_t s);

}  // namespace rbs
