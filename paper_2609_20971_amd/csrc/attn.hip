// Stage 3: causal GQA block-sparse attention (Sec. 3.3; Algorithm 1, last
// step).  The work of one (query head, query block) is attend_block
// (attend_block.hpp).  Two launches of the same work: one workgroup per
// (query head, query block), or a persistent grid that takes them from the
// per-XCD queues of next_slot (the same slots on the same XCDs in the same
// order, apart from the tail that other XCDs take over; bit-identical
// results; fewer idle workgroup slots when the rows' lengths differ a lot,
// as a sparse selection's do).
#include "attend_block.hpp"
#include "rbs_launch.hpp"

namespace rbs {

template <int BS, typename LastBlock>
__device__ __forceinline__ void attend_slot(const AttnCore& c, const int32_t* __restrict__ counts,
                                            const int32_t* __restrict__ indices, int64_t capacity, int slot,
                                            int total, unsigned char* k_lds, unsigned char* v_lds, LastBlock last_block) {
  int h, i;
  work_of(slot, total, c.M, total / c.M, c.group, c.order, h, i);
  const int count = min(max(counts[(size_t)h * c.M + i], 0), i + 1);
  const int32_t* list = indices + (int64_t)h * capacity + (int64_t)i * (i + 1) / 2;
  attend_block<BS>(c, h, i, count, [&](int n) __attribute__((always_inline)) { return list[n]; }, k_lds, v_lds,
                   last_block);
}

template <int BS>
__global__ __launch_bounds__(BS * 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_kernel(
    AttnCore c, const int32_t* __restrict__ counts, const int32_t* __restrict__ indices, int64_t capacity) {
  __shared__ __align__(1024) unsigned char k_lds[BS * 256];
  __shared__ __align__(1024) unsigned char v_lds[BS * 256];
  attend_slot<BS>(c, counts, indices, capacity, blockIdx.x, gridDim.x, k_lds, v_lds, [] {});
}

// Persistent form: total = M * H_q work slots, queue as reset_queues leaves it.
// (B = 256 takes all 256 VGPRs; two are spilled for an item's length and read back
// once per item, none in the block loop.)
template <int BS>
__global__ __launch_bounds__(BS * 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_queue_kernel(
    AttnCore c, const int32_t* __restrict__ counts, const int32_t* __restrict__ indices, int64_t capacity,
    int total, int* __restrict__ queue) {
  __shared__ __align__(1024) unsigned char k_lds[BS * 256];
  __shared__ __align__(1024) unsigned char v_lds[BS * 256];
  __shared__ int lds_slot;
  QueueTicket ticket(queue);
  for (int slot = blockIdx.x; slot >= 0; slot = next_slot(ticket, total, &lds_slot)) {
    attend_slot<BS>(c, counts, indices, capacity, slot, total, k_lds, v_lds,
                    [&]() __attribute__((always_inline)) { ticket.take(); });
    __syncthreads();  // tiles and lds_slot free for the next item
  }
}

// Every sequence of a batch in one launch: in row-major order the longest rows
// of all sequences first (RowOrder), otherwise sequence-major and, inside a
// sequence, ordered as work_of orders them.
template <int BS, typename LastBlock>
__device__ __forceinline__ void attend_slot_varlen(AttnCore c, const int32_t* __restrict__ counts,
                                                   const int32_t* __restrict__ indices, const SeqTable& t,
                                                   const RowOrder& rows, int slot,
                                                   int total, unsigned char* k_lds, unsigned char* v_lds, LastBlock last_block) {
  const int hq = total / t.blk[t.n];  // query heads
  const int work = xcd_remap(slot, total);
  int sq, i, h;
  if (c.order != kByGroup) {
    row_at(rows, work / hq, &sq, &i);
    h = work % hq;
  } else {
    sq = seq_of(t.blk, t.n, work / hq);
    const int local = work - hq * t.blk[sq];
    const int m = t.blk[sq + 1] - t.blk[sq];
    const int per_group = m * c.group;
    const int g = local / per_group;
    const int rem = local - g * per_group;
    i = m - 1 - rem / c.group;
    h = g * c.group + rem % c.group;
  }
  c.N = t.tok[sq + 1] - t.tok[sq];
  c.M = t.blk[sq + 1] - t.blk[sq];
  const int64_t tok0 = t.tok[sq];
  c.Q += tok0 * c.q_tok;
  c.K += tok0 * c.kv_tok;
  c.V += tok0 * c.kv_tok;
  c.O += tok0 * c.q_tok;
  if (c.lse != nullptr) c.lse += t.tok[sq];
  const int count = min(max(counts[(size_t)h * t.blk[t.n] + t.blk[sq] + i], 0), i + 1);
  const int32_t* list = indices + (int64_t)h * t.cap[t.n] + t.cap[sq] + (int64_t)i * (i + 1) / 2;
  attend_block<BS, true>(c, h, i, count, [&](int n) __attribute__((always_inline)) { return list[n]; }, k_lds,
                         v_lds, last_block);
}

template <int BS>
__global__ __launch_bounds__(BS * 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_varlen_kernel(
    AttnCore c, const int32_t* __restrict__ counts, const int32_t* __restrict__ indices, const SeqTable t,
    const RowOrder rows) {
  __shared__ __align__(1024) unsigned char k_lds[BS * 256];
  __shared__ __align__(1024) unsigned char v_lds[BS * 256];
  attend_slot_varlen<BS>(c, counts, indices, t, rows, blockIdx.x, gridDim.x, k_lds, v_lds, [] {});
}

template <int BS>
__global__ __launch_bounds__(BS * 2) __attribute__((amdgpu_waves_per_eu(2, 2))) void attn_varlen_queue_kernel(
    AttnCore c, const int32_t* __restrict__ counts, const int32_t* __restrict__ indices, const SeqTable t,
    const RowOrder rows, int total, int* __restrict__ queue) {
  __shared__ __align__(1024) unsigned char k_lds[BS * 256];
  __shared__ __align__(1024) unsigned char v_lds[BS * 256];
  __shared__ int lds_slot;
  QueueTicket ticket(queue);
  for (int slot = blockIdx.x; slot >= 0; slot = next_slot(ticket, total, &lds_slot)) {
    attend_slot_varlen<BS>(c, counts, indices, t, rows, slot, total, k_lds, v_lds,
                    [&]() __attribute__((always_inline)) { ticket.take(); });
    __syncthreads();
  }
}

// Scratch of the allocation-free entry point (rbs_sparse_prefill_noalloc):
// the kQueueInts queue counters of its persistent launch.  Each device holds
// its own copy until the process ends; host code must use the address that
// hipGetSymbolAddress returns for the current device, never the name.
static __device__ __align__(256) int scratch[kQueueInts];

namespace {
int* g_scratch_of_device[kMaxDevices] = {};
}  // namespace

// The device address of this device's scratch, looked up once per device.
hipError_t noalloc_scratch(int** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  int* p = __atomic_load_n(&g_scratch_of_device[dev], __ATOMIC_ACQUIRE);
  if (p == nullptr) {
    e = hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    __atomic_store_n(&g_scratch_of_device[dev], p, __ATOMIC_RELEASE);  // concurrent first calls store the same value
  }
  *out = p;
  return hipSuccess;
}

hipError_t launch_attention_noalloc(AttnArgs a, hipStream_t s) {
  hipError_t e = noalloc_scratch(&a.queue);
  if (e != hipSuccess) return e;
  return launch_attention(a, s);
}

__global__ void reset_queues_kernel(int* __restrict__ queue, int taken) {
  if (threadIdx.x < kQueueInts) queue[threadIdx.x] = taken;  // one in kQueueStride is a counter
}

hipError_t reset_queues(int* queue, int grid, hipStream_t s) {
  hipLaunchKernelGGL(reset_queues_kernel, dim3(1), dim3(kQueueInts), 0, s, queue, grid / kQueues);
  return hipGetLastError();
}


__global__ void dense_indices_kernel(int M, int64_t capacity, int32_t* __restrict__ counts,
                                     int32_t* __restrict__ indices) {
  const int i = blockIdx.x, h = blockIdx.y;
  int32_t* out = indices + (int64_t)h * capacity + (int64_t)i * (i + 1) / 2;
  for (int b = threadIdx.x; b <= i; b += blockDim.x) out[b] = b;
  if (threadIdx.x == 0) counts[(size_t)h * M + i] = i + 1;
}

template <int BS>
static hipError_t launch_attention_bs(const AttnCore& c, const AttnArgs& a, hipStream_t s) {
  const int total = a.n_blocks * a.n_q_heads;
  return launch_slots<attn_queue_kernel<BS>>(
      BS * 2, total, a.queue, s,
      [&](int resident) { return queue_line(a.n_tokens, a.n_q_heads, a.n_kv_heads, BS, a.n_blocks, resident, a.selected); },
      [&](int grid) {
        hipLaunchKernelGGL(attn_kernel<BS>, dim3(grid), dim3(BS * 2), 0, s, c, a.counts, a.indices, a.capacity);
      },
      [&](int grid) {
        hipLaunchKernelGGL(attn_queue_kernel<BS>, dim3(grid), dim3(BS * 2), 0, s, c, a.counts, a.indices, a.capacity,
                           total, a.queue);
      });
}

hipError_t launch_attention(const AttnArgs& a, hipStream_t s) {
  const AttnCore c = make_attn_core(a);
  switch (a.block_size) {
    case 64: return launch_attention_bs<64>(c, a, s);
    case 128: return launch_attention_bs<128>(c, a, s);
    case 256: return launch_attention_bs<256>(c, a, s);
    default: return hipErrorInvalidValue;
  }
}

__global__ void dense_indices_varlen_kernel(const SeqTable t, int32_t* __restrict__ counts,
                                            int32_t* __restrict__ indices) {
  const int bg = blockIdx.x, h = blockIdx.y;
  const int sq = seq_of(t.blk, t.n, bg);
  const int i = bg - t.blk[sq];
  int32_t* out = indices + (int64_t)h * t.cap[t.n] + t.cap[sq] + (int64_t)i * (i + 1) / 2;
  for (int b = threadIdx.x; b <= i; b += blockDim.x) out[b] = b;
  if (threadIdx.x == 0) counts[(size_t)h * t.blk[t.n] + bg] = i + 1;
}

template <int BS>
static hipError_t launch_attention_varlen_bs(const AttnCore& c, const AttnArgs& a, const SeqTable& t, hipStream_t s) {
  const int total = t.blk[t.n] * a.n_q_heads;
  const RowOrder rows = rows_by_length(t);
  // (At B = 256 too, where one sequence takes the queues from twice the resident
  // items on: a batch's rows are shorter, per slot / queues at 2.2 times, 28 / 4
  // heads, three sequences 94 / 98 us, 64 / 8 four of 1 K tokens 46 / 48.)
  return launch_slots<attn_varlen_queue_kernel<BS>>(
      BS * 2, total, a.queue, s, [](int resident) { return 3 * resident; },
      [&](int grid) {
        hipLaunchKernelGGL(attn_varlen_kernel<BS>, dim3(grid), dim3(BS * 2), 0, s, c, a.counts, a.indices, t, rows);
      },
      [&](int grid) {
        hipLaunchKernelGGL(attn_varlen_queue_kernel<BS>, dim3(grid), dim3(BS * 2), 0, s, c, a.counts, a.indices, t,
                           rows, total, a.queue);
      });
}

hipError_t launch_attention_varlen(const AttnArgs& a, const SeqTable& t, hipStream_t s) {
  AttnCore c = make_attn_core(a);
  c.order = batch_order(a.n_tokens, a.n_q_heads, a.n_kv_heads, a.block_size, a.n_blocks);
  switch (a.block_size) {
    case 64: return launch_attention_varlen_bs<64>(c, a, t, s);
    case 128: return launch_attention_varlen_bs<128>(c, a, t, s);
    case 256: return launch_attention_varlen_bs<256>(c, a, t, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_dense_indices_varlen(int n_q_heads, const SeqTable& t, int32_t* counts, int32_t* indices,
                                       hipStream_t s) {
  hipLaunchKernelGGL(dense_indices_varlen_kernel, dim3(t.blk[t.n], n_q_heads), dim3(256), 0, s, t, counts,
                     indices);
  return hipGetLastError();
}

hipError_t launch_dense_indices(int n_q_heads, int n_blocks, int64_t capacity, int32_t* counts,
                                int32_t* indices, hipStream_t s) {
  hipLaunchKernelGGL(dense_indices_kernel, dim3(n_blocks, n_q_heads), dim3(256), 0, s, n_blocks, capacity, counts,
                     indices);
  return hipGetLastError();
}

}  // namespace rbs
