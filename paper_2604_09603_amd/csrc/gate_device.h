// Gate state shared by the gate launches and the fused step's front kernel:
// the workspace layout, the radix selection and the last phase of the global
// top-B selection (eq. 4).
#pragma once

#include "echo_device.h"
#include "echo_internal.h"

namespace echo {
namespace {

constexpr int kGateThreads = 1024;
constexpr int kHistBins = 2048;   // top 11 bits of the key
constexpr int kHistShift = 21;
constexpr int kSortCap = 8192;    // candidates gate_finish gathers into LDS
constexpr int kWinBack = 3072;    // nodes before a score block kept in its LDS window
constexpr int kWin = kWinBack + kGateThreads;
constexpr int kDepths = ECHO_MAX_DEPTH + 1;  // per-request depth slots (0 = root, unused)
constexpr int kTabReq = 64;                  // requests per score block with an LDS max table

struct GateMeta {
  int32_t num_selected;  // m
  uint32_t bin;          // histogram bin of the m-th largest key
  uint32_t bin_need;     // how many keys of that bin are selected
  uint32_t bin_cnt;      // keys in that bin
  uint32_t thr_key;      // selected iff key > thr_key || (key == thr_key && g <= thr_g)
  int32_t thr_g;
};

struct GateWs {
  GateMeta* meta;
  uint32_t* keys;    // [N] orderable key, 0 = never selected
  int32_t* pglob;    // [N] clamped parent, global index (-1: child of the root)
  uint32_t* bhist;   // [nblocks][2048] per-block histograms
  uint32_t* ccount;  // [nblocks] candidates found by each select block
  uint2* bsum;       // [nblocks] (finite keys, highest occupied bin + 1) of each score block
  uint2* cand;       // [nblocks * 1024] (key, index) candidates, block slices
  uint32_t* lmax;    // [R][kDepths] max key per (request, depth), checkpoint depths only
  uint8_t* depth;    // [N] node depth (1 = child of the root), capped at ECHO_MAX_DEPTH + 1
};

// Checkpoint table of sparse gating: request r passes depth d iff the largest
// path score among its depth-d nodes is above lt[d] (eq. 7 in the log domain).
struct SparseArgs {
  int enabled;
  uint32_t mask;     // bit d set iff depth d is a checkpoint
  float lt[kDepths]; // ln tau of each checkpoint depth (the largest if repeated)
  int32_t* trunc_out;  // nullable [R]: first failed checkpoint, ECHO_MAX_DEPTH + 1 if none
};

__host__ __device__ inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

__host__ __device__ inline int gate_blocks(int32_t N) {
  return N > 0 ? (N + kGateThreads - 1) / kGateThreads : 1;
}

__host__ __device__ inline GateWs gate_ws_layout(void* base, int32_t N, int32_t R) {
  const size_t nb = size_t(gate_blocks(N));
  char* p = static_cast<char*>(base);
  GateWs w;
  w.meta = reinterpret_cast<GateMeta*>(p);
  p += 256;
  w.keys = reinterpret_cast<uint32_t*>(p);
  p += align_up(size_t(N) * 4, 256);
  w.pglob = reinterpret_cast<int32_t*>(p);
  p += align_up(size_t(N) * 4, 256);
  w.bhist = reinterpret_cast<uint32_t*>(p);
  p += align_up(nb * kHistBins * 4, 256);
  w.ccount = reinterpret_cast<uint32_t*>(p);
  p += align_up(nb * 4, 256);
  w.bsum = reinterpret_cast<uint2*>(p);
  p += align_up(nb * 8, 256);
  w.cand = reinterpret_cast<uint2*>(p);
  p += align_up(nb * kGateThreads * 8, 256);
  w.lmax = reinterpret_cast<uint32_t*>(p);
  p += align_up(size_t(R) * kDepths * 4, 256);
  w.depth = reinterpret_cast<uint8_t*>(p);
  return w;
}

// ---------------------------------------------------------------- score ----
struct NodeScore {
  float score;   // S after the clamps, -inf below ECHO_MAX_DEPTH
  uint32_t key;  // its orderable key
  int parent;    // clamped parent, global index (-1: child of the root)
  int depth;     // 1 = child of the root; exact up to ECHO_MAX_DEPTH + 1
  int bits;      // status bits
};

// Path score of candidate g, whose request's candidates start at lo: the root ->
// leaf binary32 fold of eq. 5 with the clamps.  par_at(x) and lq_at(x) give the
// parent (request-local) and log q of candidate x.
template <typename ParAt, typename LqAt>
__device__ __forceinline__ NodeScore node_score(int g, int lo, ParAt par_at, LqAt lq_at) {
  NodeScore r;
  r.bits = 0;
  const int n = g - lo;
  int p = par_at(g);
  if (p < -1 || p >= n) { r.bits |= ECHO_DATA_BAD_PARENT; p = -1; }
  r.parent = p < 0 ? -1 : lo + p;
  float own = lq_at(g);
  if (own != own) { r.bits |= ECHO_DATA_NAN_LOGQ; own = -__builtin_inff(); }
  else if (own > 0.0f) { r.bits |= ECHO_DATA_POS_LOGQ; own = 0.0f; }
  // collect log q along the path, leaf first: vals[0] = own, vals[i] = i-th ancestor
  float vals[ECHO_MAX_DEPTH + 1];
  vals[0] = own;
  int depth = 1;
#pragma unroll
  for (int i = 1; i <= ECHO_MAX_DEPTH; ++i) {
    vals[i] = 0.0f;
    if (p >= 0) {
      const int a = lo + p;
      float v = lq_at(a);
      if (v != v) v = -__builtin_inff();
      else if (v > 0.0f) v = 0.0f;
      int pp = par_at(a);
      if (pp < -1 || pp >= p) pp = -1;
      vals[i] = v;
      depth = i + 1;
      p = pp;
    }
  }
  r.score = -__builtin_inff();
  if (depth > ECHO_MAX_DEPTH) {
    r.bits |= ECHO_DATA_TOO_DEEP;
  } else {
    // root -> leaf: S = ((0 + lq[top]) + ...) + lq[own], one binary32 add per level
    r.score = 0.0f;
#pragma unroll
    for (int i = ECHO_MAX_DEPTH; i >= 0; --i)
      if (i < depth) r.score = r.score + vals[i];
  }
  r.key = score_key(r.score);
  r.depth = depth;
  return r;
}

// --------------------------------------------------------------- finish ----
// Radix selection: among the entries i < n with match(i), each carrying an
// unsigned value val(i), find the value of the need-th largest, 8 bits at a
// time from the top.  A step counts the entries whose value has the known high
// bits into a 256-bin LDS histogram and one wave finds the bin where the count
// from the top reaches need.  Once every entry matching the known bits is
// selected (need == cnt) the lower bits no longer matter and the walk stops.
struct RadixSel {
  uint32_t prefix;  // known high bits of the value (value >> shift)
  int shift;        // number of still unknown low bits
  uint32_t need;    // rank of the sought entry among those matching the prefix (1..cnt)
  uint32_t cnt;     // entries matching the prefix
};

struct RadixLds {
  uint32_t h[2][256];  // histograms, used alternately
  int d[2][2];         // (bin, count above the bin) of each step
};

// One wave: the bin of h whose cumulative count from bin 255 downwards first
// reaches need, and the count of the bins above it.
__device__ __forceinline__ void digit_search(const uint32_t* h, uint32_t need, int* out) {
  const int lane = threadIdx.x & (kWave - 1);
  uint32_t c[4];
  uint32_t sum = 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) {  // lane l holds bins 255-4l .. 252-4l, highest first
    c[j] = h[255 - 4 * lane - j];
    sum += c[j];
  }
  const uint32_t incl = wave_scan(sum, 0u, AddOp{});
  const unsigned long long hit = __ballot(incl >= need);
  const int l0 = hit != 0ull ? __builtin_ctzll(hit) : 0;
  if (lane == l0) {
    uint32_t above = incl - sum;
    int j = 0;
    for (; j < 3; ++j) {
      if (above + c[j] >= need) break;
      above += c[j];
    }
    out[0] = 255 - 4 * lane - j;
    out[1] = int(above);
  }
}

// The histograms of both buffers must be zero on entry; they are on return.
template <typename Val, typename Match>
__device__ void radix_select(RadixSel& st, int n, Val val, Match match, RadixLds& L) {
  int cur = 0;
  while (st.shift > 0 && st.need < st.cnt) {
    const int bits = st.shift >= 8 ? 8 : st.shift;
    const int nsh = st.shift - bits;
    const uint32_t pre = st.prefix, sh = uint32_t(st.shift);
    if (sh >= 32u) {
      // no bit is known yet: all keys fall into a few bins (their leading bits are
      // the sign and most of the exponent), so a wave adds once per distinct bin
      for (int i0 = 0; i0 < n; i0 += blockDim.x) {
        const int i = i0 + int(threadIdx.x);
        const bool on = i < n && match(i);
        const int d = on ? int(val(i) >> nsh) : 0;
        uint64_t rem = __ballot(on);
        while (rem != 0ull) {
          const int lead = __builtin_ctzll(rem);
          const int dl = __builtin_amdgcn_readlane(d, lead);
          const uint64_t bal = __ballot(on && d == dl);
          if (int(threadIdx.x & (kWave - 1)) == lead) atomicAdd(&L.h[cur][dl], uint32_t(__popcll(bal)));
          rem &= ~bal;
        }
      }
    } else {
      for (int i = threadIdx.x; i < n; i += blockDim.x) {
        if (match(i)) {
          const uint32_t v = val(i);
          if ((v >> sh) == pre) atomicAdd(&L.h[cur][(v >> nsh) & ((1u << bits) - 1u)], 1u);
        }
      }
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
      digit_search(L.h[cur], st.need, L.d[cur]);
    } else {  // the other buffer was read before the barrier above
      for (int i = threadIdx.x - kWave; i < 256; i += blockDim.x - kWave) L.h[cur ^ 1][i] = 0u;
    }
    __syncthreads();
    const int d = L.d[cur][0];
    st.need -= uint32_t(L.d[cur][1]);
    st.cnt = L.h[cur][d];
    st.prefix = (pre << bits) | uint32_t(d);
    st.shift = nsh;
    cur ^= 1;
  }
  __syncthreads();  // every thread has read the last histogram
  for (int i = threadIdx.x; i < 512; i += blockDim.x) (&L.h[0][0])[i] = 0u;
  __syncthreads();
}

// Threshold (thr_key, thr_g) of the selection: the st.need-th largest of the st.cnt
// (> 0) keys with the known high bits st.prefix, under (key descending, index
// ascending).  keyv(i) and idx(i) describe the n entries searched; every such key
// must be among them.
template <typename KeyV, typename Idx>
__device__ void find_threshold(RadixSel st, int n, int N, KeyV keyv, Idx idx, RadixLds& L,
                               uint32_t* thr_key, int32_t* thr_g) {
  radix_select(st, n, keyv, [&](int i) { return keyv(i) != 0u; }, L);
  const uint32_t K = st.shift >= 32 ? 0u : st.prefix << st.shift;  // 0: every key is selected
  int32_t tg = 0x7FFFFFFF;
  if (st.need < st.cnt) {
    // st.shift == 0: cnt keys equal K, the need-th smallest index among them
    // is the need-th largest of (N - 1 - index)
    const uint32_t top = uint32_t(N - 1);
    RadixSel si;
    si.prefix = 0u;
    si.shift = top == 0u ? 0 : 32 - __builtin_clz(top);
    si.need = st.need;
    si.cnt = st.cnt;
    radix_select(si, n, [&](int i) { return top - uint32_t(idx(i)); },
                 [&](int i) { return keyv(i) == K; }, L);
    tg = int32_t(top - (si.prefix << si.shift));
  }
  *thr_key = K;
  *thr_g = tg;
}

// The same for the bin_need-th largest of the bin_cnt keys of bin b*.
template <typename KeyV, typename Idx>
__device__ void find_threshold(const GateMeta& mt, int n, int N, KeyV keyv, Idx idx, RadixLds& L,
                               uint32_t* thr_key, int32_t* thr_g) {
  find_threshold(RadixSel{mt.bin, kHistShift, mt.bin_need, mt.bin_cnt}, n, N, keyv, idx, L, thr_key,
                 thr_g);
}

// LDS of the last phase that may come from a larger buffer: the gathered
// candidates' keys and indices (kSortCap each) and the candidate offsets of
// the select blocks (kGateThreads + 1).
struct FinishLds {
  uint32_t* s_k;
  int32_t* s_g;
  int* s_base;
};

// Ordered compaction of n <= kSortCap entries, entry i = k kGateThreads + tid on
// thread tid: comp[0 ..) receives value(i) of those with sel(i), in the order of i,
// at most cap of them.  Returns their number.  s_cnt: 8 x 16 words.  Contains one
// barrier; s_cnt may be reused after another.
template <typename Sel, typename Value>
__device__ __forceinline__ int compact_entries(int n, Sel sel, Value value, int32_t* comp, int cap,
                                               uint32_t* s_cnt) {
  constexpr int kPer = kSortCap / kGateThreads, kW = kGateThreads / kWave;
  static_assert(kPer * kW == 2 * kWave, "two counts per lane");
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
  uint32_t on = 0u;
  int below[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int i = k * kGateThreads + int(threadIdx.x);
    below[k] = 0;
    uint32_t c = 0u;
    if (k * kGateThreads < n) {  // uniform
      const bool s = i < n && sel(i);
      const uint64_t bal = __ballot(s);
      c = uint32_t(__popcll(bal));
      below[k] = lanes_below(bal);
      on |= uint32_t(s) << k;
    }
    if (lane == 0) s_cnt[k * kW + wid] = c;
  }
  __syncthreads();
  const uint32_t c0 = s_cnt[2 * lane], c1 = s_cnt[2 * lane + 1];
  const uint32_t inc = wave_scan(c0 + c1, 0u, AddOp{});
  const uint32_t excl = inc - c0 - c1;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    if (k * kGateThreads >= n) break;
    const int e = k * kW + wid;
    int pos = __builtin_amdgcn_readlane(int(excl), e >> 1) + below[k];
    if (e & 1) pos += __builtin_amdgcn_readlane(int(c0), e >> 1);
    if (((on >> k) & 1u) && pos < cap) comp[pos] = value(k * kGateThreads + int(threadIdx.x));
  }
  return __builtin_amdgcn_readlane(int(inc), kWave - 1);
}

// The last phase of the top-B selection, one workgroup of kGateThreads: gathers
// the candidates of the threshold bin, finds the threshold (key descending,
// index ascending) by radix selection and writes their selection flags.  If the
// bin holds more keys than LDS takes, the same selection runs over all keys in
// place.
[[maybe_unused]] __device__ void gate_finish_body(int N, int nblocks, const GateWs& ws,
                                 uint8_t* __restrict__ selected, int32_t* status,
                                 const FinishLds& lds) {
  uint32_t* s_k = lds.s_k;
  int32_t* s_g = lds.s_g;
  int* s_base = lds.s_base;
  __shared__ int s_scan[kGateThreads / kWave + 1];
  __shared__ RadixLds s_rl;
  // the first kGateThreads block counts are loaded with the selection's size
  const int c_first = int(threadIdx.x) < nblocks ? int(ws.ccount[threadIdx.x]) : 0;
  const GateMeta mt = *ws.meta;
  const uint32_t m = uint32_t(mt.num_selected);
  if (m == 0u) return;
  for (int i = threadIdx.x; i < 512; i += kGateThreads) (&s_rl.h[0][0])[i] = 0u;
  // exclusive scan of the per-block candidate counts
  int run = 0;
  for (int b0 = 0; b0 < nblocks; b0 += kGateThreads) {
    const int b = b0 + threadIdx.x;
    const int c = b0 == 0 ? c_first : (b < nblocks ? int(ws.ccount[b]) : 0);
    int tot;
    const int ex = block_exclusive_sum<kGateThreads>(c, s_scan, &tot);
    if (b < nblocks && b < kGateThreads) s_base[b] = run + ex;
    run += tot;
  }
  const int nc = run;
  uint32_t tk;
  int32_t tg;
  // No ancestor-closure check is needed: a child's score is its parent's plus a
  // clamped log q <= 0 in one binary32 add, so the parent's key is at least the
  // child's, and its global index is smaller; under (key descending, index
  // ascending) the parent of a selected node is always selected.
  (void)status;
  if (nc <= kSortCap && nblocks <= kGateThreads) {
    if (threadIdx.x == 0) s_base[nblocks] = nc;
    __syncthreads();
    for (int i = threadIdx.x; i < nc; i += kGateThreads) {
      const int b = upper_bound_idx(s_base, nblocks + 1, i);
      const uint2 c = ws.cand[size_t(b) * kGateThreads + (i - s_base[b])];
      s_k[i] = c.x;
      s_g[i] = int32_t(c.y);
    }
    __syncthreads();
    find_threshold(mt, nc, N, [&](int i) { return s_k[i]; }, [&](int i) { return s_g[i]; }, s_rl,
                   &tk, &tg);
    for (int i = threadIdx.x; i < nc; i += kGateThreads) {
      const uint32_t k = s_k[i];
      const int32_t g = s_g[i];
      const bool sel = k > tk || (k == tk && g <= tg);
      selected[g] = sel ? 1 : 0;
    }
  } else {
    __syncthreads();
    const uint32_t* keys = ws.keys;
    find_threshold(mt, N, N, [&](int i) { return keys[i]; }, [](int i) { return int32_t(i); },
                   s_rl, &tk, &tg);
    for (int b = 0; b < nblocks; ++b) {
      const int c = int(ws.ccount[b]);
      for (int i = threadIdx.x; i < c; i += kGateThreads) {
        const uint2 e = ws.cand[size_t(b) * kGateThreads + i];
        const bool sel = e.x > tk || (e.x == tk && int32_t(e.y) <= tg);
        selected[e.y] = sel ? 1 : 0;
      }
    }
  }
  if (threadIdx.x == 0) {
    ws.meta->thr_key = tk;
    ws.meta->thr_g = tg;
  }
}


// ---------------------------------------------------------- small pools ----
// Candidates of a small pool, kSmallPer per thread: its whole top-B gate runs on one
// workgroup, in LDS.  Whole fused steps over N candidates
// (8 / 8 heads, 64 keys), lists -> small pool: 28.5 -> 23.3 us at 208, 32.1 -> 28.6
// at 2080, 36.6 -> 34.7 at 3120, 38.7 -> 38.4 at 4160, 42.0 -> 44.7 at 6136 (one
// workgroup's searches and histogram rounds grow with N).  A round of the scores was two
// barriers then; with one, steps over 208, 2400 and 3072 candidates take 23.4 -> 22.1,
// 34.5 -> 31.2 and 38.8 -> 35.2 us, the last two with chains of 16 levels.
constexpr int kSmallPer = 3;
constexpr int kSmallPool = kSmallPer * kGateThreads;

// What a small pool's gate reads and writes.
struct SmallGate {
  int N, R, budget;
  const int32_t* parent;
  const float* logq;
  float* path_score;  // nullable
  uint8_t* selected;
  int32_t* num_selected;
};

// A small pool's candidates in registers, loaded before anything waits.
struct SmallPool {
  int32_t par[kSmallPer];
  float lq[kSmallPer];
};

__device__ __forceinline__ SmallPool load_small(const SmallGate& a) {
  SmallPool p;
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k) {
    const int g = k * kGateThreads + int(threadIdx.x);
    p.par[k] = g < a.N ? a.parent[g] : -1;
    p.lq[k] = g < a.N ? a.logq[g] : 0.0f;
  }
  return p;
}

// The whole top-B gate of a small pool; finish(sel): the caller's pass over the
// candidates, sel(i) says whether candidate i is selected and, if `first`, writes its
// flag.  offs: the candidate offsets in LDS, ok: they are well formed; smem: 8 bytes
// per candidate.
template <typename Finish>
__device__ __forceinline__ auto select_small(const SmallGate& a, const SmallPool& in,
                                             const int32_t* offs, bool ok, bool first,
                                             int32_t* smem, int* bits, Finish finish) {
  __shared__ RadixLds s_rl;
  __shared__ uint32_t s_fin[kGateThreads / kWave];
  __shared__ uint32_t s_more[3];  // round r, entry r % 3: a node is still open
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  if (tid < 3) s_more[tid] = 0u;
  // Scores top-down, all nodes of a depth in one round: (score, depth) of every node
  // whose score is known, a NaN score where it is not.  A node folds the same
  // binary32 adds in the same order as a walk from the root.  (Short code: with the
  // instruction cache cold, an unrolled walk per node cost more than the launches
  // it saved.)
  uint64_t* s_node = reinterpret_cast<uint64_t*>(smem);  // depth above, score below
  uint32_t* s_key = reinterpret_cast<uint32_t*>(smem);  // replaces them
  constexpr uint32_t kUnknown = 0x7FFFFFFFu;
  const int n = a.N;
  int par[kSmallPer];
  float lq[kSmallPer], sc[kSmallPer];
  uint32_t open = 0u;  // bit k: the thread's node k has no score yet
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k) {
    const int g = k * kGateThreads + tid;
    sc[k] = -__builtin_inff();
    lq[k] = in.lq[k];
    par[k] = -1;
    if (!ok || g >= n) continue;
    const int lo = offs[upper_bound_idx(offs, a.R + 1, g)];
    int p = in.par[k];
    if (p < -1 || p >= g - lo) { *bits |= ECHO_DATA_BAD_PARENT; p = -1; }
    if (lq[k] != lq[k]) { *bits |= ECHO_DATA_NAN_LOGQ; lq[k] = -__builtin_inff(); }
    else if (lq[k] > 0.0f) { *bits |= ECHO_DATA_POS_LOGQ; lq[k] = 0.0f; }
    if (p < 0) {
      sc[k] = 0.0f + lq[k];
      s_node[g] = (uint64_t(1) << 32) | __float_as_uint(sc[k]);
    } else {
      par[k] = lo + p;
      open |= 1u << k;
      s_node[g] = kUnknown;
    }
  }
  for (int i = tid; i < 512; i += kGateThreads) (&s_rl.h[0][0])[i] = 0u;
  // after ECHO_MAX_DEPTH - 1 rounds every node of depth <= ECHO_MAX_DEPTH is known
  // (one barrier per round: a round's entry is cleared two rounds before it is set again,
  // when everyone has read it)
  int now = 0;
  for (int round = 1; round < ECHO_MAX_DEPTH; ++round) {
    if (round == 1) {
      if (!__syncthreads_or(open != 0u)) break;
    } else {
      if (__ballot(open != 0u) != 0ull && lane == 0) s_more[now] = 1u;
      __syncthreads();
      if (s_more[now] == 0u) break;
      const int last = now == 0 ? 2 : now - 1;
      if (tid == 0) s_more[last] = 0u;
      now = now == 2 ? 0 : now + 1;
    }
#pragma unroll
    for (int k = 0; k < kSmallPer; ++k) {
      if (!((open >> k) & 1u)) continue;
      // (a parent may be scored in this very round: either word will do)
      const uint64_t v =
          __hip_atomic_load(&s_node[par[k]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (uint32_t(v) == kUnknown || uint32_t(v >> 32) >= ECHO_MAX_DEPTH) continue;
      sc[k] = __uint_as_float(uint32_t(v)) + lq[k];
      __hip_atomic_store(&s_node[k * kGateThreads + tid],
                         (((v >> 32) + 1) << 32) | uint64_t(__float_as_uint(sc[k])),
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      open &= ~(1u << k);
    }
  }
  if (open != 0u) *bits |= ECHO_DATA_TOO_DEEP;  // deeper: their scores stay -inf
  uint32_t key[kSmallPer];
  uint32_t fin = 0u;
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k) {
    const int g = k * kGateThreads + tid;
    key[k] = score_key(sc[k]);
    if (first && g < n && a.path_score != nullptr) a.path_score[g] = sc[k];
    fin += uint32_t(__popcll(__ballot(key[k] != 0u)));
  }
  if (lane == 0) s_fin[tid / kWave] = fin;
  __syncthreads();  // every score has been read
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k) {
    const int g = k * kGateThreads + tid;
    if (g < n) s_key[g] = key[k];
  }
  fin = 0u;
#pragma unroll
  for (int w = 0; w < kGateThreads / kWave; ++w) fin += s_fin[w];
  const uint32_t m = min(uint32_t(a.budget), fin);
  if (first && tid == 0) *a.num_selected = int32_t(m);
  __syncthreads();
  uint32_t tk = 0xFFFFFFFFu;
  int32_t tg = -1;
  if (m != 0u)
    find_threshold(RadixSel{0u, 32, m, fin}, n, n, [&](int i) { return s_key[i]; },
                   [](int i) { return int32_t(i); }, s_rl, &tk, &tg);
  const auto sel = [&](int i) {
    const uint32_t k = s_key[i];
    const bool on = m != 0u && k != 0u && (k > tk || (k == tk && i <= tg));
    if (first) a.selected[i] = on ? 1 : 0;
    return on;
  };
  return finish(sel);
}

}  // namespace
}  // namespace echo
