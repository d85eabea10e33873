// The serving step around the verification path: the greedy target token of
// every verify slot (argmax of its vocabulary logits) feeding acceptance, and
// the commit of each request's accepted path into a paged KV cache.
//
//   target_argmax   one workgroup per slot row: streams the row's bfloat16
//                   logits with 16-byte loads, two batches in flight per thread
//                   (HBM-bound: Nq * V * 2 bytes), as ordered 16-bit integers: the
//                   maximum of eight at a time, and the first block of eight that
//                   holds the thread's largest; a workgroup reduction picks the
//                   row's block and its first largest element.  Then the acceptance
//                   kernel.
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

// Two bfloat16 as signed 16-bit integers in their numeric order (-0 below +0;
// negative NaN below -inf, positive NaN above +inf).
__device__ __forceinline__ short2v ordered(uint32_t w) {
  const short2v x = __builtin_bit_cast(short2v, w);
  return x ^ ((x >> short2v{15, 15}) & short2v{0x7FFF, 0x7FFF});
}
constexpr int kOrdInf = 0x7F80;        // +inf
constexpr int kOrdNegInf = -0x7F80 - 1;  // -inf

// The row's argmax element by element, for the rows whose order as integers is not
// the order asked for: NaN (never wins over a number), a maximum of zero (-0 and +0
// are equal) or nothing above -inf (then the first -inf; only NaN: 0).  Every thread
// of the workgroup calls it; the result is in s_best (value above, ~index below).
template <int NT>
__device__ __forceinline__ uint32_t argmax_plain(const uint16_t* row, long long vocab,
                                                 unsigned long long* s_best) {
  __syncthreads();
  if (threadIdx.x == 0) *s_best = 0ull;
  __syncthreads();
  unsigned long long best = 0ull;
  for (long long v = threadIdx.x; v < vocab; v += NT) {
    const uint32_t u = uint32_t(row[v]);
    if ((u & 0x7FFFu) > 0x7F80u) continue;  // NaN
    const uint32_t b = u == 0x8000u ? 0u : u;  // -0 -> +0
    const uint32_t k = (b & 0x8000u) ? (~b & 0xFFFFu) : (b | 0x8000u);
    const unsigned long long w =
        ((unsigned long long)(k + 1u) << 32) | (0xFFFFFFFFu - uint32_t(v));
    best = w > best ? w : best;
  }
  if (best != 0ull) atomicMax(s_best, best);
  __syncthreads();
  return *s_best == 0ull ? 0u : 0xFFFFFFFFu - uint32_t(*s_best);
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
template <int NT, int kArgBatch, bool kStream>
__global__ __launch_bounds__(NT) void target_argmax_kernel(
    const uint16_t* __restrict__ logits, long long vocab, const int32_t* __restrict__ q_offsets,
    int R, int32_t* __restrict__ target) {
  __shared__ unsigned long long s_wave[NT / kWave];
  __shared__ unsigned long long s_best;
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
  uint32_t at = 0u;        // its element (head, tail) or the first one of its block
  // the head precedes the blocks in index order: taken first
  for (long long v = tid; v < head; v += NT) {
    const int o = int(ordered(row[v])[0]);
    if (o > best) {
      best = o;
      at = uint32_t(v);
    }
  }
  if (nvec > 0) {
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
      for (int u = 0; u < kArgBatch; ++u) {
        const long long i = c + (long long)u * NT;
        const short2v m = __builtin_elementwise_max(
            __builtin_elementwise_max(ordered(x[u].x), ordered(x[u].y)),
            __builtin_elementwise_max(ordered(x[u].z), ordered(x[u].w)));
        const int o = max(int(m[0]), int(m[1]));
        if (o > best) {
          best = o;
          at = uint32_t(head + (i < nvec ? i : nvec - 1) * 8);
        }
      }
    };
    constexpr long long kStep = (long long)kArgBatch * NT;
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
    }
  }
  // largest value, then the smallest place
  unsigned long long w =
      ((unsigned long long)(uint32_t(best + 0x8001)) << 32) | (0xFFFFFFFFu - at);
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const unsigned long long o = __shfl_xor(w, off, kWave);
    w = o > w ? o : w;
  }
  if ((tid & (kWave - 1)) == 0) s_wave[tid / kWave] = w;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NT / kWave; ++k) w = s_wave[k] > w ? s_wave[k] : w;
  const int top = int(uint32_t(w >> 32)) - 0x8001;
  uint32_t idx = 0xFFFFFFFFu - uint32_t(w);
  if (top > kOrdInf || top == 0 || top <= kOrdNegInf) {  // uniform, rare
    idx = argmax_plain<NT>(row, vocab, &s_best);
  } else if (idx >= head && (long long)idx < tail0) {
    // the first of the block's eight elements with that value
    const uint4 x = *reinterpret_cast<const uint4*>(row + idx);
    const short2v o[4] = {ordered(x.x), ordered(x.y), ordered(x.z), ordered(x.w)};
    uint32_t e = 7u;
#pragma unroll
    for (int k = 6; k >= 0; --k)
      if (int(o[k >> 1][k & 1]) == top) e = uint32_t(k);
    idx += e;
  }
  if (tid == 0) target[s] = int32_t(idx);
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
