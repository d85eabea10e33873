// The serving step around the verification path: the greedy target token of
// every verify slot (argmax of its vocabulary logits) feeding acceptance, and
// the commit of each request's accepted path into a paged KV cache.
//
//   target_argmax   one workgroup per slot row: streams the row's bfloat16
//                   logits with 16-byte loads, two batches in flight per thread
//                   (HBM-bound: Nq * V * 2 bytes), as 16-bit integers: a thread
//                   keeps its largest value and the first group of blocks of eight
//                   that holds it; the threads that have the row's largest then find
//                   its first element.  Then the acceptance kernel.
//   commit_kv       one workgroup per request: copies the root slot's and the
//                   accepted slots' K and V rows into their pages, then advances
//                   the request's cached length.
#include "echo_device.h"
#include "echo_internal.h"

namespace echo {
namespace {

constexpr int kCommitThreads = 256;
typedef uint32_t uint32x4 __attribute__((ext_vector_type(4)));
typedef short short2v __attribute__((ext_vector_type(2)));

typedef unsigned short ushort2v __attribute__((ext_vector_type(2)));

// Two bfloat16 as signed 16-bit integers in the order of the argmax: numbers as they
// compare (-0 and +0 are both kOrdZero), NaN of either sign below -inf.  Two's
// complement magnitudes, moved up by kOrdZero: the positive NaN, above +inf, wrap
// around to the bottom, where the negative ones are.
constexpr short kOrdZero = 0x7F;
constexpr int kOrdNegInf = kOrdZero - 0x7F80;
__device__ __forceinline__ short2v ordered(uint32_t w) {
  const short2v neg = __builtin_bit_cast(short2v, w) >> short2v{15, 15};  // 0 or -1
  const short2v mag = __builtin_bit_cast(short2v, w & 0x7FFF7FFFu);
  return __builtin_bit_cast(  // (in unsigned arithmetic, which wraps)
      short2v, __builtin_bit_cast(ushort2v, mag ^ neg) +
                   __builtin_bit_cast(ushort2v, short2v{kOrdZero, kOrdZero} - neg));
}

// The largest of a block's eight elements, in that order.
__device__ __forceinline__ int block_max(const uint4& x) {
  const short2v m = __builtin_elementwise_max(
      __builtin_elementwise_max(ordered(x.x), ordered(x.y)),
      __builtin_elementwise_max(ordered(x.z), ordered(x.w)));
  return max(int(m[0]), int(m[1]));
}

// The same over N blocks, with two instructions per two elements instead of five: the
// largest bit pattern as signed (a positive one wins, in its order) and the smallest as
// unsigned (without positive ones, the negative one nearest to zero).  A positive NaN
// takes the plain order.
template <int N>
__device__ __forceinline__ int group_max(const uint4* x) {
  short2v hi = __builtin_bit_cast(short2v, x[0].x);
  ushort2v lo = __builtin_bit_cast(ushort2v, x[0].x);
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const uint32_t w[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      hi = __builtin_elementwise_max(hi, __builtin_bit_cast(short2v, w[k]));
      lo = __builtin_elementwise_min(lo, __builtin_bit_cast(ushort2v, w[k]));
    }
  }
  const int p = max(int(hi[0]), int(hi[1]));
  const int n = min(int(lo[0]), int(lo[1]));
  if (p > 0x7F80) {
    int o = block_max(x[0]);
#pragma unroll
    for (int u = 1; u < N; ++u) o = max(o, block_max(x[u]));
    return o;
  }
  return p >= 0 ? p + kOrdZero : kOrdZero - (n & 0x7FFF);
}

// One workgroup of NT threads per slot row, kArgBatch 16-byte loads per batch.
// * At most one row per CU: 1024 threads keep the most bytes in flight.  160 rows of
//   128,256 (41 MB): 11.9 -> 10.4 us.
// * More rows: 512 threads, two or more workgroups of which share a CU, longer
//   batches, and loads with the non-temporal hint, as the logits no longer stay in
//   the caches.  384 rows of 151,936 (117 MB): 26.4 -> 22.0 us, 5.3 TB/s (24.0
//   without the hint, 25.5 with batches of 12; the 128 CUs with two rows set the
//   end).  For the smaller case the hint is slower (12.0).
// (Before: one batch of eight loads at a time, compared as floats element by
// element, four instructions each, and a remainder of single loads.)
// NaN and zeros of either sign cost nothing: rows that hold them once took a second,
// element-by-element pass, and one such row 14.5 -> 64 us (160 x 151,936), 24 -> 79 (384).
//
// A thread keeps its largest value and the first group of kArgGroup blocks that holds
// it; once the row's largest is known, those that have it look the element up.
constexpr int kArgGroup = 5;
template <int NT, int kArgBatch, bool kStream>
__global__ __launch_bounds__(NT) void target_argmax_kernel(
    const uint16_t* __restrict__ logits, long long vocab, const int32_t* __restrict__ q_offsets,
    int R, int32_t* __restrict__ target) {
  static_assert(kArgBatch % kArgGroup == 0, "whole groups");
  __shared__ uint32_t s_wave[NT / kWave];
  __shared__ uint32_t s_first;
  const int s = blockIdx.x;
  const uint16_t* row = logits + size_t(s) * size_t(vocab);
  const int tid = threadIdx.x;
  // scalar head up to 16-byte alignment, blocks of 8, scalar tail
  const long long head =
      min<long long>(vocab, ((16 - (reinterpret_cast<uintptr_t>(row) & 15)) & 15) / 2);
  const long long nvec = (vocab - head) / 8;
  const long long tail0 = head + nvec * 8;
  const uint4* body = reinterpret_cast<const uint4*>(row + head);
  if (s >= q_offsets[R]) return;  // uniform over the workgroup
  int best = -0x8000 - 1;  // below every ordered value
  uint32_t at = 0u;        // its element (head, tail) or its group's first block
  bool group = false;
  // the head precedes the blocks in index order: taken first
  for (long long v = tid; v < head; v += NT) {
    const int o = int(ordered(row[v])[0]);
    if (o > best) {
      best = o;
      at = uint32_t(v);
    }
  }
  constexpr long long kStep = (long long)kArgBatch * NT;
  // rows of at most one batch: their blocks one by one and nothing beyond them.  160 and
  // 384 rows of 1000: 5.8 and 6.1 us, of 16,000: 6.3 and 7.0 (through the loop, whose
  // three batches of whole groups mostly repeat the last block, 7.5, 9.8, 7.7 and 10.0)
  const bool one = nvec <= kStep;  // uniform
  if (one) {
    uint4 x[kArgBatch];
#pragma unroll
    for (int u = 0; u < kArgBatch; ++u)
      if ((long long)u * NT < nvec)
        x[u] = body[min<long long>(tid + (long long)u * NT, nvec - 1)];
#pragma unroll
    for (int u = 0; u < kArgBatch; ++u) {
      if ((long long)u * NT < nvec) {
        const int o = group_max<1>(&x[u]);
        if (o > best) {
          best = o;
          at = uint32_t(tid + u * NT);
          group = true;
        }
      }
    }
  } else {
    // blocks past the last one repeat it (no effect: same value, same place)
    const auto load = [&](uint4 (&x)[kArgBatch], long long c) {
#pragma unroll
      for (int u = 0; u < kArgBatch; ++u) {
        const long long i = c + (long long)u * NT;
        const uint4* p = body + (i < nvec ? i : nvec - 1);
        if (kStream) {
          const uint32x4 q = __builtin_nontemporal_load(reinterpret_cast<const uint32x4*>(p));
          x[u] = make_uint4(q[0], q[1], q[2], q[3]);
        } else {
          x[u] = *p;
        }
      }
    };
    const auto take = [&](const uint4 (&x)[kArgBatch], long long c) {
#pragma unroll
      for (int g = 0; g < kArgBatch; g += kArgGroup) {
        const int o = group_max<kArgGroup>(&x[g]);
        if (o > best) {
          best = o;
          at = uint32_t(c + (long long)g * NT);
          group = true;
        }
      }
    };
    uint4 x0[kArgBatch], x1[kArgBatch];
    load(x0, tid);
    for (long long c = tid; c - tid < nvec; c += 2 * kStep) {
      load(x1, c + kStep);
      take(x0, c);
      load(x0, c + 2 * kStep);
      take(x1, c + kStep);
    }
  }
  for (long long v = tail0 + tid; v < vocab; v += NT) {
    const int o = int(ordered(row[v])[0]);
    if (o > best) {
      best = o;
      at = uint32_t(v);
      group = false;
    }
  }
  const uint32_t wmax = wave_max(uint32_t(best + 0x8001));
  if ((tid & (kWave - 1)) == 0) s_wave[tid / kWave] = wmax;
  if (tid == 0) s_first = 0xFFFFFFFFu;
  __syncthreads();
  uint32_t w = s_wave[0];
#pragma unroll
  for (int k = 1; k < NT / kWave; ++k) w = max(w, s_wave[k]);
  const int top = int(w) - 0x8001;
  uint32_t idx = 0xFFFFFFFFu;
  if (best == top) {
    idx = at;
    if (group) {
      // the group's first block with that value, then its first element
      uint4 x[kArgGroup];
      uint32_t blk[kArgGroup];
#pragma unroll
      for (int u = 0; u < kArgGroup; ++u) {
        const long long i = (long long)at + (one ? 0 : (long long)u * NT);
        blk[u] = uint32_t(i < nvec ? i : nvec - 1);
        x[u] = body[blk[u]];
      }
      uint4 y = x[0];
      uint32_t in = blk[0];
      if (!one && block_max(y) != top) {
        y = x[kArgGroup - 1];
        in = blk[kArgGroup - 1];
#pragma unroll
        for (int u = kArgGroup - 2; u >= 1; --u) {
          if (block_max(x[u]) == top) {
            y = x[u];
            in = blk[u];
          }
        }
      }
      const short2v o[4] = {ordered(y.x), ordered(y.y), ordered(y.z), ordered(y.w)};
      uint32_t e = 7u;
#pragma unroll
      for (int k = 6; k >= 0; --k)
        if (int(o[k >> 1][k & 1]) == top) e = uint32_t(k);
      idx = uint32_t(head) + in * 8u + e;
    }
  }
  // (one atomic per wave: in a row of equal logits every thread is here)
  const uint32_t first = ~wave_max(~idx);
  if ((tid & (kWave - 1)) == 0 && first != 0xFFFFFFFFu) atomicMin(&s_first, first);
  __syncthreads();
  if (tid == 0) target[s] = top < kOrdNegInf ? 0 : int32_t(s_first);  // (only NaN: 0)
}

__global__ __launch_bounds__(kCommitThreads) void commit_kv_kernel(
    const int32_t* __restrict__ q_offsets, const int32_t* __restrict__ accept_len,
    const int32_t* __restrict__ accept_slots, int max_depth, const uint16_t* __restrict__ k_new,
    const uint16_t* __restrict__ v_new, int max_rows, int hkv, uint16_t* __restrict__ k_pages,
    uint16_t* __restrict__ v_pages, long long num_pages, int page_size,
    const int32_t* __restrict__ block_table, int max_pages, int32_t* __restrict__ prefix_len,
    int32_t* status) {
  __shared__ int s_slot[ECHO_MAX_DEPTH + 1];
  __shared__ long long s_dst[ECHO_MAX_DEPTH + 1];  // destination row (page * page_size + offset)
  __shared__ int s_bad;
  const int r = blockIdx.x;
  const int tid = threadIdx.x;
  const int q0 = q_offsets[r], q1 = q_offsets[r + 1];
  const int L = accept_len[r];
  const int P = prefix_len[r];
  bool ok = true;
  int n = 0;
  if (q1 > q0) {  // a request without slots verified nothing and commits nothing
    ok = q0 >= 0 && q1 <= max_rows && L >= 0 && L <= max_depth && P >= 0;
    n = ok ? 1 + L : 0;
  }
  if (tid == 0) s_bad = ok ? 0 : 1;
  __syncthreads();
  // thread j resolves committed row j: its slot and its place in the pages
  if (tid < n) {
    const int j = tid;
    const int s = j == 0 ? q0 : accept_slots[size_t(r) * max_depth + (j - 1)];
    const long long pos = (long long)P + j;
    const long long e = pos / page_size;
    const int page = e < max_pages ? block_table[size_t(r) * max_pages + size_t(e)] : -1;
    if (s < 0 || s >= max_rows || page < 0 || page >= num_pages) atomicOr(&s_bad, 1);
    s_slot[j] = s;
    s_dst[j] = (long long)page * page_size + (pos % page_size);
  }
  __syncthreads();
  if (s_bad) n = 0;  // nothing of the request is written
  // each row is hkv * 128 bf16 = hkv * 16 chunks of 16 bytes, for K and for V
  const int chunks = hkv * (ECHO_HEAD_DIM * 2 / 16);
  for (int i = tid; i < n * chunks; i += kCommitThreads) {
    const int j = i / chunks, c = i % chunks;
    const size_t src = size_t(s_slot[j]) * size_t(chunks) + size_t(c);
    const size_t dst = size_t(s_dst[j]) * size_t(chunks) + size_t(c);
    reinterpret_cast<uint4*>(k_pages)[dst] = reinterpret_cast<const uint4*>(k_new)[src];
    reinterpret_cast<uint4*>(v_pages)[dst] = reinterpret_cast<const uint4*>(v_new)[src];
  }
  if (tid == 0) {
    if (s_bad) status_or(status, ECHO_DATA_BAD_OFFSETS);
    else if (n > 0) prefix_len[r] = P + n;
  }
}

}  // namespace

int32_t launch_accept_logits(const int32_t* q_offsets, const int32_t* slot_parent,
                             const int32_t* slot_token, const uint16_t* logits, int64_t vocab,
                             int32_t R, int32_t max_rows, int32_t max_depth, int32_t* target,
                             int32_t* accept_len, int32_t* accept_slots, int32_t* bonus_token,
                             int32_t* status, hipStream_t stream) {
  (void)hipGetLastError();
  if (max_rows > 0) {
    const bool few = max_rows <= device_cu_count();
    auto kern = few ? target_argmax_kernel<1024, 5, false> : target_argmax_kernel<512, 10, true>;
    hipLaunchKernelGGL(kern, dim3(max_rows), dim3(few ? 1024 : 512), 0, stream, logits,
                       static_cast<long long>(vocab), q_offsets, R, target);
  }
  if (hipGetLastError() != hipSuccess) return ECHO_ERR_HIP;
  return launch_accept(q_offsets, slot_parent, slot_token, target, R, max_rows, max_depth,
                       accept_len, accept_slots, bonus_token, status, stream);
}

int32_t launch_commit_kv(const int32_t* q_offsets, const int32_t* accept_len,
                         const int32_t* accept_slots, int32_t max_depth, const uint16_t* k_new,
                         const uint16_t* v_new, int32_t R, int32_t max_rows, int32_t hkv,
                         uint16_t* k_pages, uint16_t* v_pages, int64_t num_pages,
                         int32_t page_size, const int32_t* block_table, int32_t max_pages,
                         int32_t* prefix_len, int32_t* status, hipStream_t stream) {
  (void)hipGetLastError();
  hipLaunchKernelGGL(commit_kv_kernel, dim3(R), dim3(kCommitThreads), 0, stream, q_offsets,
                     accept_len, accept_slots, max_depth, k_new, v_new, max_rows, hkv, k_pages,
                     v_pages, static_cast<long long>(num_pages), page_size, block_table,
                     max_pages, prefix_len, status);
  return hipGetLastError() == hipSuccess ? ECHO_OK : ECHO_ERR_HIP;
}

}  // namespace echo
