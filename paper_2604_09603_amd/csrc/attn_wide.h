// The main attention kernel for wide units: one KV head of one request with up
// to 256 of its rows (verify slots x query heads of the GQA group).
//
// A persistent workgroup of eight waves per CU, two waves per SIMD, streams the
// tiles of its range through one ring in LDS, two tiles between barriers: each wave
// copies an eighth of every 32-key tile.  Above 128 rows wave w multiplies all tiles
// with rows 32 w .. 32 w + 31 of the unit; up to 128 rows two waves share each 32
// rows, one on the even and one on the odd tiles, and merge their sums at the end.
// A head's tile is so copied once for all of its rows, where an ordinary unit
// copies it once per wave.  S^T = K Q^T and O^T = V^T P^T on v_mfma_f32_32x32x16_bf16:
// a lane holds 16 of a tile's 32 keys of one row, so that a row needs one exchange
// between two lanes, and only where its maximum or sum is used.  The order of the
// keys within a product of P V is the one in which S^T leaves them in the lanes (V
// is read in the same order).
//
// What bounds it (16 requests of 16384-32768 keys, 64 / 4 heads, 208 rows per head; from
// builds that skip work and from short probes, neither of them kept): copies alone 144-155 us (805 MB), arithmetic alone 191-210,
// both 230-275 (the ordinary kernel: 289-326; the first figure of each pair is the
// best launch, the second the median of launches back to back, at a lower clock).
// With one KV head (128 requests of 1024-8192 keys, 48 rows): 50-52, 45-49 and 62-66
// us (84-90).  The arithmetic is bound by instruction issue: on a SIMD a 32x32x16
// product keeps other vector instructions out for about 20 of its 32 cycles, also
// those of the other wave, so products and softmax add up; a vector instruction
// takes 4.5 cycles, an exponential 8.5.  Per 64 keys and 32 rows these are 32
// products, 32 exponentials and about 170 others.  Hence: the copies' sources come
// from a table in LDS (per-tile address arithmetic in every wave cost 13 us), LDS
// addresses need one instruction per fragment, and a step's maxima and sums run in
// independent chains (a dependent instruction waits 9 cycles).  Alternating the two
// waves of a SIMD between K and V phases, with one or two barriers per step, was
// slower (282 against 271 us; 358 against 295).
#pragma once

#include <type_traits>

#include "attn_core.h"

namespace echo {
namespace {

constexpr int kWideWaves = 8;
constexpr int kWideStages = 8;  // ring: 32-key K+V tiles
constexpr int kWideStep = 2;    // tiles between two barriers
constexpr int kWideTileBytes = kTileKeys * kD * 2;      // 8 KB per tensor
constexpr int kWideStageBytes = 2 * kWideTileBytes;     // K then V
constexpr int kWideTable = kWideWaves * kWave;  // ring positions whose sources are in LDS
constexpr int kWideXchg = 20 * 1024;  // exchange of the key halves' sums (see wide_merge)
constexpr int kWideLds = kWideStages * kWideStageBytes + kWideTable * 16 + kWideXchg;
static_assert(kWideLds <= 160 * 1024, "gfx950 LDS per workgroup");
constexpr int kWideCopies = 2;  // copy instructions per wave and tile (1 KB of K, 1 KB of V)

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) const bf16x8 lds_bf16x8_t;
typedef __attribute__((address_space(3))) char lds_char_t;

// The LDS byte address x as a pointer (constant offsets go into the instructions).
__device__ __forceinline__ lds_char_t* lds_at(uint32_t x) {
  return (lds_char_t*)(uintptr_t(x));
}

// The running softmax of the lane's row (see RowTile of the ordinary kernel).
struct WideRow {
  float m, l, lq;
  float mgrow;  // a max above it raises the reference
  float negm;
  float thr;    // screen of the residual split: m + log2(row sum) - 5, when last taken
};

// Maximum and sum over the two lanes of a row.
__device__ __forceinline__ float pair_max(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// Step a unit forward: the next stream of the same request, or the first one of
// the next request that has any (rec: its record).
__device__ __forceinline__ void wide_next_unit(Unit& u, int& rec, const Unit* units, int nrec,
                                               int hkv) {
  if (u.group + 1 < hkv * u.passes) {
    const int n = u.tile_end - u.tile_start;
    u.group += 1;
    u.tile_start = u.tile_end;
    u.tile_end += n;
    return;
  }
  while (rec + 1 < nrec) {
    rec = __builtin_amdgcn_readfirstlane(rec + 1);
    u = load_unit(units, rec);
    if (u.passes > 0) return;
  }
}

// The source of one ring position's tile, as the copies need it: the addresses of
// its first key row in K and in V (the unit's head) and the last of its valid rows,
// in the bits of V's address from 48 on.
struct WideTile {
  uint64_t k, v;
};

// Where the table of ring positions continues: tile t of unit u (record rec) is
// position pos, the first one of its segment.
struct WideWalk {
  Unit u;
  int rec, t, pos;
};

// Fill the table with positions base .. base + kWideTable - 1 (thread tid writes
// entry tid), as far as the range [.., hi) goes; every segment takes an even number
// of positions, the last one of an odd segment repeating its tile.  Returns the end
// of the positions known so far.  Every thread of the workgroup calls it.
__device__ __forceinline__ int wide_fill(WideTile* table, int base, WideWalk& w, const MainArgs& a,
                                         const AttnWs& ws, int nrec, int hi) {
  const int my = base + int(threadIdx.x);
  const uint32_t row_bytes = uint32_t(a.hkv) * kD * 2;
  int end = w.pos;
  while (w.t < hi && w.pos < base + kWideTable) {
    const int seg_hi = min(hi, w.u.tile_end);
    const int len = seg_hi - w.t;
    end = w.pos + ((len + 1) & ~1);
    if (my >= w.pos && my < end) {
      const int lt = w.t + min(my - w.pos, len - 1) - w.u.tile_start;
      const uint64_t head = uint64_t(w.u.group / w.u.passes) * kD * 2;
      uint64_t off;
      uint64_t kb = reinterpret_cast<uint64_t>(a.k_cache), vb = reinterpret_cast<uint64_t>(a.v_cache);
      uint32_t rows;
      if (lt < w.u.ntail) {
        off = uint64_t(w.u.q0 + lt * kTileKeys) * row_bytes;
        rows = uint32_t(min(kTileKeys, w.u.nslots - lt * kTileKeys));
        kb = reinterpret_cast<uint64_t>(a.k_new);
        vb = reinterpret_cast<uint64_t>(a.v_new);
      } else {
        const int key = (lt - w.u.ntail) * kTileKeys;
        if (a.block_table == nullptr) {
          off = uint64_t(w.u.kb + key) * row_bytes;
        } else {
          const int page = a.block_table[size_t(w.u.kb) * size_t(a.max_pages) + (key >> a.page_shift)];
          off = ((uint64_t(page) << a.page_shift) + uint64_t(key & ((1 << a.page_shift) - 1))) *
                row_bytes;
        }
        rows = uint32_t(min(kTileKeys, w.u.P - key));
      }
      off += head;
      table[my - base] = WideTile{kb + off, (vb + off) | (uint64_t(rows - 1) << 48)};
    }
    if (end > base + kWideTable) return base + kWideTable;  // the segment goes on in the next fill
    w.pos = end;
    w.t = seg_hi;
    if (w.t < hi) wide_next_unit(w.u, w.rec, ws.units, nrec, a.hkv);
  }
  return end;
}

// This wave's share of two tiles: rows 4 wid .. 4 wid + 3 of K and of V, one 1 KB
// direct-to-LDS load each, at lds, + 8 KB, + 16 KB and + 24 KB (the reasons for the
// assembly are those of dma_tile_full).  Every lane gives its own address, so that
// the table's entries need no trip through scalar registers.  Non-temporal: a
// head's tiles are read once, or by another workgroup much later.
__device__ __forceinline__ void wide_dma(uint32_t lds, uint64_t k0, uint64_t v0, uint64_t k1,
                                         uint64_t v1) {
  uint32_t saved;
  asm volatile(
      "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off nt\n\t"
      "s_add_u32 m0, m0, 0x2000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %3, off nt\n\t"
      "s_add_u32 m0, m0, 0x2000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %4, off nt\n\t"
      "s_add_u32 m0, m0, 0x2000\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %5, off nt\n\t"
      "s_mov_b32 m0, %0"
      : "=&s"(saved)
      : "s"(lds), "v"(k0), "v"(v0), "v"(k1), "v"(v1)
      : "memory", "scc");
}

// Copy the tiles of two table entries (the same in every lane) into the stages from
// lds on.  Rows past a tile's last valid one read that one again (masked in the
// softmax).
__device__ __forceinline__ void wide_copy(const WideTile (&e)[2], uint32_t lds, uint32_t row,
                                          uint32_t row_bytes, uint32_t chunk16) {
  uint64_t k[2], v[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const uint32_t last = uint32_t(e[j].v >> 48);
    const uint64_t off = __umul24(min(row, last), row_bytes) + chunk16;
    k[j] = e[j].k + off;
    v[j] = (e[j].v & 0xFFFFFFFFFFFFull) + off;
  }
  wide_dma(__builtin_amdgcn_readfirstlane(lds), k[0], v[0], k[1], v[1]);
}

#define ECHO_FENCE() __builtin_amdgcn_sched_barrier(0)
// S^T = K Q^T of NT tiles (32 keys each) in consecutive stages from LDS address stg
// and the wave's 32 rows.
template <int NT>
__device__ __forceinline__ void wide_scores(uint32_t stg, uint32_t ka, const bf16x8 (&qf)[8],
                                            floatx16 (&s)[NT]) {
  // (opaque: the fragments' addresses are formed per step, not kept in registers;
  // the ring starts at a multiple of 1 KB, so the swizzle's exclusive-or, of bits below
  // 256, may follow the sum)
  ka += stg;
  asm volatile("" : "+v"(ka));
  bf16x8 kf[NT][8];
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      kf[j][kk] = *(lds_bf16x8_t*)(lds_at(ka ^ uint32_t(kk << 5)) + kWideStageBytes * j);
  ECHO_FENCE();
#pragma unroll
  for (int j = 0; j < NT; ++j)
#pragma unroll
    for (int kk = 0; kk < 8; ++kk)
      s[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j][kk], qf[kk],
                                                     kk == 0 ? floatx16{} : s[j], 0, 0, 0);
  ECHO_FENCE();
}

// The softmax of those scores and O^T += V^T P^T.  masked: key k of tile j is visible
// to the lane's row iff bit k of word[j].  one (NT == 2): the second tile is the
// repeated one of an odd segment, with no visible key; its products are left out, as 0
// times an infinite value is NaN.  A wave's vector instructions overlap with
// only the last third of a matrix product, and a result is ready two issue slots
// after its instruction: the products of P V are spread between the exponentials of
// the next 16 keys, and maxima and sums run in independent chains.  Fences
// (sched_barrier) hold that order, and keep the LDS reads ahead of the products
// that use them (left alone the scheduler saves registers by waiting for each read).
template <int NT>
__device__ __forceinline__ void wide_values(uint32_t stg, uint32_t va, floatx16 (&s)[NT],
                                            floatx16 (&o)[4], WideRow& rs, bool masked,
                                            bool one, float scale2,
                                            const uint32_t (&word)[NT]) {
  const int h = (threadIdx.x & (kWave - 1)) >> 5;
  constexpr int NG = 2 * NT;  // groups of 16 keys
  va += stg;
  asm volatile("" : "+v"(va));
  // V fragments of group g: keys 16 (g & 1) .. + 15 of tile g / 2, in the order in
  // which S^T holds them
  const auto load_v = [&](int g, bf16x8 (&vf)[4]) {
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      const int at = kWideStageBytes * (g >> 1) + 4096 * (g & 1);
      const shortx4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_shortx4_t*)(lds_at(va ^ uint32_t(dt << 6)) + at));
      const shortx4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
          (lds_shortx4_t*)(lds_at(va ^ uint32_t(dt << 6) ^ 32u) + at + 2048));
      vf[dt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
    }
  };
  bf16x8 vf[2][4];
  load_v(0, vf[0]);
  load_v(1, vf[1]);
  ECHO_FENCE();
  if (masked) {
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      const uint32_t w = word[j] >> (4 * h);
#pragma unroll
      for (int r = 0; r < 16; ++r)  // key 8 (r >> 2) + 4 h + (r & 3)
        s[j][r] = ((w >> (8 * (r >> 2) + (r & 3))) & 1u) ? s[j][r] : -__builtin_inff();
    }
  }
  float mx[4] = {s[0][0], s[0][1], s[0][2], s[0][3]};
#pragma unroll
  for (int e = 4; e < 16 * NT; e += 2)
    mx[(e >> 1) & 3] = fmaxf(mx[(e >> 1) & 3], fmaxf(s[e >> 4][e & 15], s[e >> 4][(e & 15) + 1]));
  // the lane's keys of its row; -inf stays -inf
  const float lmt = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3])) * scale2;
  if (__ballot(lmt > rs.mgrow) != 0ull) {
    const float mt = pair_max(lmt);
    const bool grow = mt > rs.mgrow;
    const float alpha = grow ? __builtin_amdgcn_exp2f(rs.m - mt) : 1.0f;  // 0 from -inf
    rs.l *= alpha;
    rs.lq *= alpha;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
    rs.m = grow ? mt : rs.m;
    rs.mgrow = rs.m + kRescaleSlack;
    rs.negm = rs.m == -__builtin_inff() ? 0.0f : -rs.m;
  }
  const float neg_m = rs.negm;
  float ps[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  float lq[2] = {rs.lq, 0.0f};
  uint32_t pk[NG][4];
  // probabilities 2 i and 2 i + 1 of group g (i = 0 .. 3)
  const auto two = [&](int g, int i) {
    const int e = 8 * (g & 1) + 2 * i;
    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[g >> 1][e], scale2, neg_m));
    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[g >> 1][e + 1], scale2, neg_m));
    s[g >> 1][e] = p0;
    s[g >> 1][e + 1] = p1;
    ps[2 * (i & 1)] += p0;
    ps[2 * (i & 1) + 1] += p1;
    pk[g][i] = pack_bf16x2(p0, p1);
    lq[i & 1] = add_bf16x2(pk[g][i], lq[i & 1]);
  };
#pragma unroll
  for (int i = 0; i < 4; ++i) two(0, i);
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    if (g == 2 && one) break;  // uniform
    const bf16x8 pf = as_bf16x8(make_uint4(pk[g][0], pk[g][1], pk[g][2], pk[g][3]));
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      ECHO_FENCE();
      o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[g & 1][dt], pf, o[dt], 0, 0, 0);
      ECHO_FENCE();
      if (g + 1 < NG) two(g + 1, dt);
    }
    if (g + 2 < NG) load_v(g + 2, vf[g & 1]);
  }
  ECHO_FENCE();
  rs.lq = lq[0] + lq[1];
  rs.l += (ps[0] + ps[1]) + (ps[2] + ps[3]);
  // the residual split, as in the ordinary kernel (compute_tile): tested only where
  // the screen lets a step through; V is read again
  if (__ballot(lmt > rs.thr) != 0ull) {
    const float mt = pair_max(lmt);
    const float sum = pair_sum(rs.l);
    rs.thr = rs.m + __builtin_amdgcn_logf(sum) - 5.0f;
    if (__ballot(__builtin_amdgcn_exp2f(mt - rs.m) > kSplitFrac * sum) != 0ull) {
      const auto res = [](float p, uint32_t w, int half) {
        return p - __uint_as_float(half ? (w & 0xFFFF0000u) : (w << 16));
      };
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g == 2 && one) break;
        uint32_t pl[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int e = 8 * (g & 1) + 2 * i;
          pl[i] = pack_bf16x2(res(s[g >> 1][e], pk[g][i], 0), res(s[g >> 1][e + 1], pk[g][i], 1));
          rs.lq = add_bf16x2(pl[i], rs.lq);
        }
        bf16x8 vr[4];
        load_v(g, vr);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              vr[dt], as_bf16x8(make_uint4(pl[0], pl[1], pl[2], pl[3])), o[dt], 0, 0, 0);
      }
    }
  }
}
#undef ECHO_FENCE

// The waves of the odd tiles (half 1) hand their sums to those of the even tiles,
// which hold the same rows (rblock of nrb, 2 or 4): the maxima and sums with the
// first part of O, through 20 KB of LDS, a quarter or a half of O at a time.  Every
// wave of the workgroup calls it (barriers).
__device__ __forceinline__ void wide_merge(char* xchg, int rblock, int nrb, int half, bool active,
                                           floatx16 (&o)[4], WideRow& rs) {
  const int lane = threadIdx.x & (kWave - 1);
  const int per = 4 / nrb;  // 32-dim blocks of O per round
  floatx4* x = reinterpret_cast<floatx4*>(xchg) + size_t(rblock) * (per * 5 * kWave) + lane;
  const bool give = active && half == 1, take = active && half == 0;
  const auto sync = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  float wa = 1.0f, wb = 0.0f;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt) {
    const int in = dt & (per - 1);  // place within the round
    if (dt > 0 && in == 0) sync();  // the round before has been read
    if (give) {
      if (dt == 0) x[4 * per * kWave] = floatx4{rs.m, rs.l, rs.lq, 0.0f};
#pragma unroll
      for (int k = 0; k < 4; ++k)
        x[(4 * in + k) * kWave] =
            floatx4{o[dt][4 * k], o[dt][4 * k + 1], o[dt][4 * k + 2], o[dt][4 * k + 3]};
    }
    if (in != per - 1) continue;
    sync();
    if (!take) continue;
    if (dt == per - 1) {
      const floatx4 y = x[4 * per * kWave];
      const float M = fmaxf(rs.m, y[0]);
      if (M != -__builtin_inff()) {
        wa = __builtin_amdgcn_exp2f(rs.m - M);
        wb = __builtin_amdgcn_exp2f(y[0] - M);
      }
      rs.m = M;
      rs.l = __builtin_fmaf(wb, y[1], wa * rs.l);
      rs.lq = __builtin_fmaf(wb, y[2], wa * rs.lq);
    }
    const auto merge = [&](floatx16& v, int at) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const floatx4 y = x[(4 * at + k) * kWave];
#pragma unroll
        for (int c = 0; c < 4; ++c) v[4 * k + c] = __builtin_fmaf(wb, y[c], wa * v[4 * k + c]);
      }
    };
    if (per == 2) merge(o[dt - 1 < 0 ? 0 : dt - 1], 0);
    merge(o[dt], in);
  }
}

// All but the copies of the `later` youngest positions of this wave have landed.
// (Stores in flight can only make the wait longer: loads return in order.)
__device__ __forceinline__ void wide_wait(int later) {  // uniform
  if (later >= 6) wait_vm<6 * kWideCopies>();  // a range's first step: all eight were sent
  // the steady state: this step's two are sent after the wait, so that four stages of the
  // eight are in flight at it and six after it
  else if (later >= 4) wait_vm<4 * kWideCopies>();
  else if (later >= 2) wait_vm<2 * kWideCopies>();
  else wait_vm<0>();
}

__global__ __launch_bounds__(kWideWaves * kWave) __attribute__((amdgpu_waves_per_eu(2, 2))) void
attn_wide_kernel(MainArgs a, AttnWs ws) {
  __shared__ __attribute__((aligned(1024))) char smem[kWideLds];
  WideTile* table = reinterpret_cast<WideTile*>(smem + kWideStages * kWideStageBytes);
  char* xchg = smem + kWideStages * kWideStageBytes + kWideTable * sizeof(WideTile);
  const int b = blockIdx.x;
  const WgStart st = load_wg_start(ws.wg_start, b);
  const int lo = st.lo, hi = st.hi;
  if (lo >= hi) return;  // uniform over the workgroup
  const int lane = threadIdx.x & (kWave - 1);
  const int wid = wave_id();
  const int nrec = st.nunits;
  const int G = a.G;
  // copies: this lane's row of a tile and its 16-byte chunk (the LDS position is
  // the lane's, the source chunk the one the swizzle puts there)
  const int crow = 4 * wid + (lane >> 4);
  const uint32_t cchunk = uint32_t(((lane & 15) ^ swz_pattern(crow)) << 4);
  const uint32_t row_bytes = uint32_t(a.hkv) * kD * 2;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(
      uint32_t(reinterpret_cast<uintptr_t>((lds_void_t*)smem)));
  const uint32_t ring_lds = lds0 + uint32_t(wid) * 1024u;
  // reads: K row lane % 32, chunk 2 kk + lane / 32; V keys 4 (lane / 32) + (lr >> 2),
  // dims 16 ((lane / 16) & 1) + 4 (lr & 3) of a 32-dim block (transposed reads)
  const int h = lane >> 5, lr = lane & 15, krow = lane & 31;
  const uint32_t ka = uint32_t(krow * 256 + ((h ^ swz_pattern(krow)) << 4));
  const int vrow = 4 * h + (lr >> 2);
  const uint32_t va =
      uint32_t(kWideTileBytes + vrow * 256 +
               (((2 * ((lane >> 4) & 1) + ((lr & 3) >> 1)) ^ swz_pattern(vrow)) << 4) +
               ((lr & 1) << 3));

  // copy side: positions [.., known) are in the table, which starts at `base`;
  // positions below `sent` have been copied; `nx` holds the next two entries
  WideWalk walk;
  walk.u = st.u;
  walk.rec = st.first_unit;
  walk.t = lo;
  walk.pos = 0;
  int base = 0, sent = 0;
  const auto sync = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  int known = wide_fill(table, 0, walk, a, ws, nrec, hi);
  sync();
  WideTile nx[2] = {table[0], table[1]};
  // copy the next two positions (segments have an even number of them)
  const auto send = [&] {
    wide_copy(nx, ring_lds + uint32_t((sent & (kWideStages - 1)) * kWideStageBytes), uint32_t(crow),
              row_bytes, cchunk);
    sent += 2;
    if (sent >= base + kWideTable) {  // the table is used up: the next part of it
      sync();
      base = sent;
      known = wide_fill(table, base, walk, a, ws, nrec, hi);
      sync();
    }
    nx[0] = table[sent - base];
    nx[1] = table[sent - base + 1];
  };
  while (sent < known && sent < kWideStages) send();

  Unit ud = st.u;
  int rec = st.first_unit;
  int pos = 0;  // ring position of the next tile to multiply
  while (true) {
    const int seg_lo = max(lo, ud.tile_start);
    const int seg_hi = min(hi, ud.tile_end);
    const int kvh = ud.group / ud.passes;
    const int row0 = (ud.group % ud.passes) * ud.rpp;
    const int rows = min(ud.rpp, ud.nslots * G - row0);
    // up to 128 rows: two waves for each 32 rows, which take every other tile each;
    // up to 64 rows: on SIMDs of their own (waves 4-7 only copy)
    const bool by_key = rows <= kWideRows / 2;
    const int nrb = rows <= 2 * 32 ? 2 : 4;
    const int rblock = by_key ? wid & (nrb - 1) : wid;
    const int half = by_key ? wid / nrb : 0;  // which of a step's tiles
    const bool active = 32 * rblock < rows && half < 2;  // wave-uniform
    const int rho = 32 * rblock + (lane & 31);
    const int lt0 = seg_lo - ud.tile_start;
    bf16x8 qf[8];
    uint32_t mw[kMaskWords];
    floatx16 o[4];
    WideRow rs;
    {
      const bool row_ok = rho < rows;
      const int ra = row0 + rho;
      const int slot = ud.q0 + ra / G;
      const uint16_t* qrow = a.q + (size_t(slot) * a.hq + size_t(kvh) * G + ra % G) * kD;
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row_ok) v = *reinterpret_cast<const uint4*>(qrow + 16 * kk + 8 * h);
        qf[kk] = as_bf16x8(v);
      }
#pragma unroll
      for (int k = 0; k < kMaskWords; ++k) mw[k] = mask_word(a, ud, row_ok, slot, lt0 + k);
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) o[dt] = floatx16{};
      rs.m = -__builtin_inff();
      rs.l = 0.0f;
      rs.lq = 0.0f;
      rs.mgrow = -__builtin_inff();
      rs.negm = 0.0f;
      rs.thr = -__builtin_inff();
    }
    wait_vm<0>();  // no compiler-visible load is in flight in the tile loop

    // visible keys of tile t for the lane's row
    const auto tile_word = [&](int t) -> uint32_t {
      if (t >= seg_hi) return 0u;  // the repeated tile of an odd segment
      const int lt = t - ud.tile_start;
      uint32_t w = 0xFFFFFFFFu;
      int tn;
      if (lt < ud.ntail) {
        tn = min(kTileKeys, ud.nslots - lt * kTileKeys);
        if (lt - lt0 < kMaskWords) {
          w = lt == lt0 ? mw[0] : mw[1];
        } else {  // more than 64 verify slots in the segment's tail: fetch the word now
          int rv = rho;
          asm volatile("" : "+v"(rv));
          w = mask_word(a, ud, rv < rows, ud.q0 + (row0 + rv) / G, lt);
          wait_vm<0>();
        }
      } else {
        tn = min(kTileKeys, ud.P - (lt - ud.ntail) * kTileKeys);
      }
      return tn >= kTileKeys ? w : (w & ((1u << tn) - 1u));
    };
    // tiles [full_lo, full_hi) are full prefix tiles: nothing to mask
    const int full_lo = ud.tile_start + ud.ntail;
    const int full_hi = min(seg_hi, full_lo + ud.P / kTileKeys);
    const auto steps = [&](auto nt) {
      constexpr int NT = decltype(nt)::value;
      const int mine = NT == 1 ? half : 0;
      for (int t = seg_lo; t < seg_hi; t += kWideStep, pos += kWideStep) {
        wide_wait(sent - pos - kWideStep);
        // every wave's share of these tiles has landed, and every wave is done with
        // the ones before
        sync();
        if (sent < known && sent < pos + kWideStages) send();
        if (!active || t + mine >= seg_hi) continue;
        const uint32_t stg = lds0 + uint32_t(((pos + mine) & (kWideStages - 1)) * kWideStageBytes);
        floatx16 s[NT];
        wide_scores<NT>(stg, ka, qf, s);
        const int tt = t + mine;
        uint32_t word[NT];
        const bool masked = tt < full_lo || tt + NT > full_hi;
#pragma unroll
        for (int j = 0; j < NT; ++j) word[j] = masked ? tile_word(tt + j) : 0u;
        wide_values<NT>(stg, va, s, o, rs, masked, t + 1 == seg_hi, a.scale2, word);
      }
    };
    if (by_key) {
      steps(std::integral_constant<int, 1>{});
      wide_merge(xchg, rblock, nrb, half, active, o, rs);
    } else {
      steps(std::integral_constant<int, 2>{});
    }

    // ---- output of the segment ----
    if (active && half == 0) {
      int rv = rho;  // (opaque: the output's addresses are formed here, not kept in registers)
      asm volatile("" : "+v"(rv));
      const bool row_ok = rv < rows;
      const int slot = ud.q0 + (row0 + rv) / G;
      const int hd = (row0 + rv) % G;
      const float L = pair_sum(rs.l);
      const float Lq = pair_sum(rs.lq);
      if (ud.tile_start >= lo && ud.tile_end <= hi) {
        if (row_ok) {
          const size_t orow = size_t(slot) * a.hq + size_t(kvh) * G + hd;
          const float inv = Lq > 0.0f ? 1.0f / Lq : 0.0f;
          float* po = a.out + orow * kD + 4 * h;
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
              const floatx4 v = {o[dt][4 * r4] * inv, o[dt][4 * r4 + 1] * inv,
                                 o[dt][4 * r4 + 2] * inv, o[dt][4 * r4 + 3] * inv};
              // (32 bytes of a row per store: left to the caches to join.  64 / 8 heads,
              // 128 requests of 33 keys with 17 and 32 slots: 79.5 and 177.6 us
              // non-temporal, 54.8 and 76.4 now; the ordinary kernel, whose stores
              // cover 64 bytes of a row, 53.3 and 89.9)
              *reinterpret_cast<floatx4*>(po + 32 * dt + 8 * r4) = v;
            }
          if (a.lse != nullptr && h == 0)
            a.lse[orow] = L > 0.0f ? (rs.m + log2f(L)) * kLn2 : -__builtin_inff();
        }
      } else {
        // a partial in fp16, each row scaled by 2^-e (see the ordinary kernel)
        float mx = 0.0f;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) mx = fmaxf(mx, fabsf(o[dt][r]));
        mx = pair_max(mx);
        const int e = mx > 0.0f ? __builtin_amdgcn_frexp_expf(mx) - 15 : 0;
        if (row_ok) {
          const float sc = __builtin_amdgcn_ldexpf(1.0f, -e);
          const int slot_id = lo < ud.tile_start ? 1 : 0;
          const size_t prow = part_row(b, slot_id, 0, 0) + size_t(rv);
#pragma unroll
          for (int dt = 0; dt < 4; ++dt)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              // dims 32 dt + 8 j + 4 h + [0, 4) and the same + 16: 8 halves in the
              // partial's order (part_dim)
              const floatx4 f0 = {o[dt][4 * j], o[dt][4 * j + 1], o[dt][4 * j + 2], o[dt][4 * j + 3]};
              const floatx4 f1 = {o[dt][4 * j + 8], o[dt][4 * j + 9], o[dt][4 * j + 10],
                                  o[dt][4 * j + 11]};
              const halfx4 a0 = __builtin_convertvector(f0 * sc, halfx4);
              const halfx4 a1 = __builtin_convertvector(f1 * sc, halfx4);
              *reinterpret_cast<halfx8*>(ws.part_o + prow * kD + 32 * dt + (2 * j + h) * 8) =
                  halfx8{a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
            }
          if (h == 0)
            *reinterpret_cast<floatx4*>(ws.part_ml + prow * 4) = floatx4{rs.m, L, Lq, float(e)};
        }
      }
    }
    if (seg_hi >= hi) break;
    wide_next_unit(ud, rec, ws.units, nrec, a.hkv);
  }
}

}  // namespace
}  // namespace echo
