// The fused step's front kernel: the end of the top-B gate (eq. 4), flatten & pack
// (Fig. 3, stage 3) and the attention plan in one launch of two workgroups.  All
// three are chains of one workgroup's round trips and barriers, and the plan needs
// of flatten & pack only the slot offsets: both workgroups find the selection and
// the slot offsets for themselves (the same values, from the same inputs), then
// workgroup 0 packs the slots and masks while workgroup 1 makes the plan.  Only
// workgroup 0 writes what is not also computed by the other; the slot offsets are
// written by both, with the same values.  At 90,880 candidates and 128 requests the
// kernel went from 21.3 to 15.3 us, at 208 and 4 requests this kernel and the two
// gate launches before it from 20.4 (and two launch gaps) to 14.0.
//
// The selection comes in one of three ways (see front_mode):
//   small pool   no gate launch at all: the path scores, the threshold and the
//                selection in LDS;
//   lists        gate_select left the candidates of the threshold bin and above in
//                index order: gathered, decided and compacted in LDS, where reading
//                the flags of all N candidates back had cost two phases of their own
//                (4.8 of 20 us at 90,880 candidates);
//   flags        (a budget too large for that LDS, or more such candidates than it
//                takes) the gate's last phase, then the flags.
#include "attn_device.h"
#include "echo_device.h"
#include "echo_internal.h"
#include "gate_device.h"
#include "mask_device.h"

namespace echo {
namespace {

constexpr int kFrontThreads = 1024;
static_assert(kGateThreads == kFrontThreads && kMaskThreads == kFrontThreads,
              "the gate's last phase and the mask run on one workgroup of the same size");

// LDS of the gate's last phase: keys and indices of kSortCap candidates and the
// kGateThreads + 1 offsets of the select blocks.
constexpr size_t kFinishLds = size_t(2 * kSortCap + kGateThreads + 1) * sizeof(int32_t);

constexpr int kModeFlags = 0, kModeLists = 1, kModeSmall = 2;
struct FrontArgs {
  // gate
  int N, nblocks;
  GateWs gws;
  uint8_t* selected;
  const float* logq;      // small pool
  float* path_score;      // small pool (nullable)
  int32_t* num_selected;  // small pool
  // flatten & pack
  const int32_t* cand_offsets;
  const int32_t* parent;
  const int32_t* token;
  const int32_t* root_token;
  const int32_t* prefix_len;
  int R, budget, W;
  int32_t* q_offsets;
  int32_t* slot_cand;
  int32_t* slot_parent;
  int32_t* slot_token;
  int32_t* position_ids;
  uint32_t* tree_mask;
  // attention plan
  KvSource kv;
  int hkv, G, max_rows, nb;
  int plan;  // 0: no rows (the attention call does nothing either)
  long long ucap;
  AttnWs aws;
  int32_t* status;
};

__host__ __device__ inline size_t mask_region(int32_t R, int32_t budget) {
  return (mask_words_bytes(R, budget) + 15) / 16 * 16;
}

// The selection from gate_select's lists into comp; its size, or -1 if the lists
// do not fit (nothing is written then).
__device__ int select_from_lists(const FrontArgs& a, bool first, int32_t* smem, int32_t* comp,
                                 uint32_t* s_cnt) {
  __shared__ int s_scan[kGateThreads / kWave + 1];
  __shared__ RadixLds s_rl;
  uint32_t* s_k = reinterpret_cast<uint32_t*>(smem);
  int32_t* s_g = smem + kSortCap;
  int* s_base = smem + 2 * kSortCap;
  const int tid = threadIdx.x;
  const int c = tid < a.nblocks ? int(a.gws.ccount[tid]) : 0;
  const GateMeta mt = *a.gws.meta;
  if (mt.num_selected == 0) return 0;
  if (a.nblocks > kGateThreads) return -1;
  for (int i = tid; i < 512; i += kGateThreads) (&s_rl.h[0][0])[i] = 0u;
  int n;
  const int ex = block_exclusive_sum<kGateThreads>(c, s_scan, &n);
  if (n > kSortCap) return -1;
  if (tid < a.nblocks) s_base[tid] = ex;
  if (tid == 0) s_base[a.nblocks] = n;
  __syncthreads();
  for (int i = tid; i < n; i += kGateThreads) {
    const int b = upper_bound_idx(s_base, a.nblocks + 1, i);
    const uint2 e = a.gws.cand[size_t(b) * kGateThreads + (i - s_base[b])];
    s_k[i] = e.x;
    s_g[i] = int32_t(e.y);
  }
  __syncthreads();
  uint32_t tk;
  int32_t tg;
  find_threshold(mt, n, a.N, [&](int i) { return s_k[i]; }, [&](int i) { return s_g[i]; }, s_rl,
                 &tk, &tg);
  const auto sel = [&](int i) {
    const uint32_t k = s_k[i];
    const bool in = k > tk || (k == tk && s_g[i] <= tg);
    // (gate_select wrote the flags of the bins above)
    if (first && (k >> kHistShift) == mt.bin) a.selected[s_g[i]] = in ? 1 : 0;
    return in;
  };
  return compact_entries(n, sel, [&](int i) { return s_g[i]; }, comp, a.budget, s_cnt);
}

template <bool kAligned, bool kWide, int kMode>
__global__ __launch_bounds__(kFrontThreads) void front_kernel(FrontArgs a) {
  extern __shared__ __attribute__((aligned(16))) int32_t smem[];
  __shared__ uint32_t s_cnt[2 * kWave];
  // The request tables of flatten & pack are loaded first, into registers, so
  // that their memory latency passes with that of the gate's first loads.
  const MaskTables tab = load_mask_tables(a.cand_offsets, a.root_token, a.prefix_len, a.R);
  // and the plan's KV offsets (one request per thread), which no phase before
  // it writes
  const int tid = threadIdx.x;
  const bool first = blockIdx.x == 0;  // packs; the other one plans
  const bool pre = !first && a.R <= kFrontThreads;
  long long k0 = 0, k1 = 0;
  if (pre && tid < a.R) {
    k0 = a.kv.kv_offsets[tid];
    k1 = a.kv.kv_offsets[tid + 1];
  }
  const MaskLds lds(smem, a.R, a.budget);
  int32_t* scratch = smem + mask_region(a.R, a.budget) / sizeof(int32_t);
  if (kMode == kModeFlags) {
    if (a.N > 0)  // as the gate call, which skips its last phase without candidates
      gate_finish_body(a.N, a.nblocks, a.gws, a.selected, a.status,
                       FinishLds{reinterpret_cast<uint32_t*>(smem), smem + kSortCap,
                                 smem + 2 * kSortCap});
    __syncthreads();
    mask_body<kAligned>(tab, a.parent, a.token, a.selected, a.R, a.N, a.budget, a.q_offsets,
                        a.slot_cand, a.slot_parent, a.slot_token, a.position_ids, a.tree_mask, a.W,
                        first, a.status, smem);
  } else {
    SmallPool pool;
    const SmallGate small{a.N, a.R, a.budget, a.parent, a.logq, a.path_score, a.selected,
                          a.num_selected};
    if (kMode == kModeSmall) pool = load_small(small);
    const bool ok = mask_tables(tab, a.R, a.N, lds);
    int bits = 0;
    if (tid == 0 && !ok) bits |= ECHO_DATA_BAD_OFFSETS;
    int count;
    if (kMode == kModeSmall) {
      count = select_small(small, pool, lds.offs, ok, first, scratch, &bits, [&](auto sel) {
        return compact_entries(a.N, sel, [](int i) { return int32_t(i); }, lds.comp, a.budget,
                               s_cnt);
      });
    } else {
      // (a malformed CSR leaves nothing selected)
      count = select_from_lists(a, first, scratch, lds.comp, s_cnt);
      if (count < 0) {  // uniform
        gate_finish_body(a.N, a.nblocks, a.gws, a.selected, a.status,
                         FinishLds{reinterpret_cast<uint32_t*>(scratch), scratch + kSortCap,
                                   scratch + 2 * kSortCap});
        __syncthreads();
        uint32_t m0[kChunksPerLane];
        load_round<kAligned>(a.selected, 0, a.N, m0);
        count = mask_compact<kAligned>(a.selected, a.N, a.budget, m0, lds);
      }
    }
    __syncthreads();
    mask_slots(a.R, count, first, a.q_offsets, a.slot_cand, a.slot_parent, a.slot_token,
               a.position_ids, lds);
    if (first) {
      __syncthreads();
      bits |= mask_rows(a.parent, a.token, a.R, count, a.slot_cand, a.slot_parent, a.slot_token,
                        a.position_ids, a.tree_mask, a.W, lds);
      wave_status_or(a.status, bits);
    }
  }
  if (first) return;
  __syncthreads();
  // the slot offsets just found are still in LDS
  const int32_t* s_qoff = lds.qoff;
  RequestIn in;
  in.q0 = tid < a.R ? s_qoff[tid] : 0;
  in.q1 = tid < a.R ? s_qoff[tid + 1] : 0;
  in.k0 = k0;
  in.k1 = k1;
  in.P = k1 - k0;
  // (the tables reuse the LDS of the phases before; every thread has read its
  // slot offsets before the plan's first barrier)
  plan_body<kFrontThreads, kWide>(a.q_offsets, a.kv, a.R, a.hkv, a.G, a.max_rows, a.nb, a.ucap,
                                  a.aws, a.status, smem, pre ? &in : nullptr);
}

size_t plan_lds(int32_t R) {
  return plan_table_words(R < kFrontThreads ? R : kFrontThreads) * sizeof(int32_t);
}

size_t mode_lds(int mode, int32_t N, int32_t R, int32_t budget) {
  const size_t m = mask_lds_bytes(R, budget);
  if (mode == kModeSmall) return mask_region(R, budget) + size_t(N) * 8;
  if (mode == kModeLists) return mask_region(R, budget) + kFinishLds;
  return m > kFinishLds ? m : kFinishLds;
}

template <bool kAligned, bool kWide>
void (*front_of(int mode))(FrontArgs) {
  // (a small pool's flags are only written, byte by byte, aligned or not)
  if (mode == kModeSmall) return front_kernel<true, kWide, kModeSmall>;
  if (mode == kModeLists) return front_kernel<kAligned, kWide, kModeLists>;
  return front_kernel<kAligned, kWide, kModeFlags>;
}

int front_mode(int32_t N, int32_t R, int32_t budget) {
  constexpr size_t kMost = 150 * 1024;  // beside the phases' static LDS
  if (N <= kSmallPool && mode_lds(kModeSmall, N, R, budget) <= kMost) return kModeSmall;
  return mode_lds(kModeLists, N, R, budget) <= kMost ? kModeLists : kModeFlags;
}

}  // namespace

int front_gate_list(int32_t N, int32_t R, int32_t budget) {
  const int mode = front_mode(N, R, budget);
  return mode == kModeSmall ? -1 : mode == kModeLists ? 1 : 0;
}

int32_t launch_front(const FrontLaunch& f, hipStream_t stream) {
  (void)hipGetLastError();  // clear errors left by unrelated runtime calls
  const int mode = front_mode(f.N, f.R, f.budget);
  FrontArgs a;
  a.N = f.N;
  a.nblocks = gate_blocks(f.N);
  a.gws = gate_ws_layout(f.gate_workspace, f.N, f.R);
  a.selected = f.selected;
  a.logq = f.logq;
  a.path_score = f.path_score;
  a.num_selected = f.num_selected;
  a.cand_offsets = f.cand_offsets;
  a.parent = f.parent;
  a.token = f.token;
  a.root_token = f.root_token;
  a.prefix_len = f.prefix_len;
  a.R = f.R;
  a.budget = f.budget;
  a.W = f.mask_words;
  a.q_offsets = f.q_offsets;
  a.slot_cand = f.slot_cand;
  a.slot_parent = f.slot_parent;
  a.slot_token = f.slot_token;
  a.position_ids = f.position_ids;
  a.tree_mask = f.tree_mask;
  a.kv.kv_offsets = f.kv_offsets;
  a.kv.kv_rows = static_cast<long long>(f.kv_rows);
  a.kv.block_table = nullptr;
  a.kv.prefix_len = nullptr;
  a.kv.page_size = 0;
  a.kv.max_pages = 0;
  a.kv.num_pages = 0;
  a.kv.page_bad = nullptr;
  a.kv.page_chunks = 0;
  a.hkv = f.hkv;
  a.G = f.hq / f.hkv;
  a.max_rows = f.max_rows;
  a.plan = f.max_rows > 0 ? 1 : 0;
  a.nb = device_cu_count();
  a.ucap = static_cast<long long>(unit_capacity(f.R, f.max_rows, f.hq, f.hkv));
  a.aws = attn_layout(f.attn_workspace, size_t(a.ucap), a.nb);
  a.status = f.status;
  size_t lds = mode_lds(mode, f.N, f.R, f.budget);
  if (lds < plan_lds(f.R)) lds = plan_lds(f.R);
  const bool aligned = (reinterpret_cast<uintptr_t>(f.selected) & 15u) == 0;
  const bool wide = attn_is_wide(f.R, f.max_rows, f.hq, f.hkv, a.kv.kv_rows, a.kv.kv_rows, a.nb);
  const auto kern = aligned ? (wide ? front_of<true, true>(mode) : front_of<true, false>(mode))
                            : (wide ? front_of<false, true>(mode) : front_of<false, false>(mode));
  if (lds > 64 * 1024 &&
      hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                          hipFuncAttributeMaxDynamicSharedMemorySize, int(lds)) != hipSuccess)
    return ECHO_ERR_HIP;
  hipLaunchKernelGGL(kern, dim3(a.plan ? 2 : 1), dim3(kFrontThreads), lds, stream, a);
  return hipGetLastError() == hipSuccess ? ECHO_OK : ECHO_ERR_HIP;
}

}  // namespace echo
