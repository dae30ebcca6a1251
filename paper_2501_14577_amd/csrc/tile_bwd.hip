// Gradients of the bfloat16 one-pass attention over the windows of
// zeta_select_attend_fwd (Appendix E.2, summary of gradient computations), on
// the matrix cores.  With S_ij = 1 / delta_ij, delta_ij = |q_i - k_j|^2 + eps,
// Z_i = sum_j S_ij, A_ij = S_ij / Z_i, p_ij = dout_i . v_j,
// c_i = dout_i . o_i = sum_j A_ij p_ij and w_ij = (p_ij - c_i) S_ij^2 / Z_i:
//   dv_j = sum_i A_ij dout_i,        dk_j = 2 sum_i w_ij (q_i - k_j),
//   dq_i = -2 sum_j w_ij (q_i - k_j), deps = -sum_ij w_ij.
//
// A tile is 16 consecutive slots of one segment's processing order.
//  1. Query pass, one wavefront per tile, walking the union of its windows in
//     16-entry chunks as the forward tile kernel does.  Per chunk the 16 x 16
//     dot products p_ij are one matrix-core product per 32 value columns (V
//     rows times dout^T).  Each lane sums over its 4 entries
//       Z = sum S, P = sum S p, X = sum S^2 p, Y = sum S^2,
//       U = sum S^2 p (q - k), R = sum S^2 (q - k),
//     so one walk gives c = P / Z, dq = -(2 / Z)(U - c R) and the query's
//     part of deps, -(X - c Y) / Z.  Per slot it stores a 32-byte record (q,
//     list, 1/Z, c, window, pool limit, position) for the key pass; per list
//     it stores the first and last list index of the tile's windows.
//  2. Envelopes, per segment and level: the running maximum (from the first
//     tile) of the tiles' last indices and the running minimum (from the last
//     tile) of their first indices.  Both are non-decreasing, so the tiles
//     whose windows meet a chunk lie between two positions, found by binary
//     search per chunk.
//  3. Key pass, one launch per list (the full sorted list first, then each
//     prefix list), one wavefront per two 16-entry chunks.  Over the candidate
//     tiles (64 tiles' ranges tested at once) a lane takes one entry and 4 of
//     the tile's queries: S_ij, the dot
//     products (dout x V^T, one product per 32 columns), w_ij and A_ij.  dv^T
//     accumulates as dout^T (columns x queries) times A (queries x entries),
//     with the high and low bfloat16 parts of A in one 16x16x32 product per 16
//     columns; dk accumulates in float32 on the vector ALUs.  The full list's
//     launch writes the rows of every key (each key is in it once); a prefix
//     list's launch adds to the rows of its keys.
// Launches run in a fixed order and a chunk visits its tiles in processing
// order: no atomics, and the outputs are the same from run to run for a given
// processing order.  Any processing order is correct; the one from
// zeta_query_order keeps each chunk's candidate tiles few.
//
// With the history-mean candidate (Section 3.4, last paragraph) the query pass
// adds the pair (mean_k[i], mean_v[i]) to its sums once per query (float32,
// its dot product dout_i . mean_v[i] from the lanes' dout slices) and writes
// the gradients reaching the means, divided by the history's length; after
// the key passes a reverse scan adds them to the rows of every history.
#include "attend_device.h"
#include "device_common.h"
#include "kernels.h"
#include "layout.h"
#include "select_device.h"
#include "tile_device.h"

#include <type_traits>

namespace zeta {
namespace {

constexpr int kBtWaves = 4;          // wavefronts per block
constexpr int kBtChunk = kChunk;      // list entries per product step
constexpr int kRedThreads = 1024;
constexpr uint32_t kNoList = 0xFFFFu;  // record of a slot whose query has no window

// What the key pass needs of a slot's query, in 32 bytes: q as bfloat16 bits,
// the list index (kNoList: no window), 1/Z, c, the window as its first list
// index a and its last less a (no window: a = INT32_MIN, span = 0, which no
// entry meets), the pool limit and the query's position.
struct alignas(16) SlotRec {
  uint32_t q01;     // q[0] | q[1] << 16
  uint32_t q2_list;  // q[2] | list index << 16
  float zinv, c;
  int32_t a;
  uint32_t span, lim;
  int32_t row;
};

// The list of a level: the full sorted list, or prefix list `lvl`.
struct LevelList {
  const int32_t* pos;
  const uint2* key;
  int32_t n;
};

__device__ __forceinline__ LevelList level_list(const int32_t* sorted_pos, const int32_t* list_pos,
                                                const uint2* keys_full, const uint2* keys_list, int64_t seg,
                                                int64_t N, int causal, int lvl, int t0, int t_hi, int64_t cap) {
  LevelList L;
  L.pos = sorted_pos + seg * N;
  L.key = keys_full + seg * N;
  L.n = int32_t(N);
  if (causal && lvl <= t_hi) {
    const int64_t off = seg * cap + ((int64_t(1) << lvl) - (int64_t(1) << t0));
    L.pos = list_pos + off;
    L.key = keys_list + off;
    L.n = int32_t(1) << lvl;
  }
  return L;
}

// Key row (d_k = 3) from its list-order copy: x | y << 16, z.
__device__ __forceinline__ void key_row(uint2 w, float (&kv)[3]) {
  kv[0] = __uint_as_float(w.x << 16);
  kv[1] = __uint_as_float(w.x & 0xFFFF0000u);
  kv[2] = __uint_as_float(w.y << 16);
}

// Eight bfloat16 values (16 bytes) at a 16-byte aligned address.
__device__ __forceinline__ void load8(const uint16_t* p, uint32_t (&o)[4]) {
  const uint4 x = *reinterpret_cast<const uint4*>(p);
  o[0] = x.x;
  o[1] = x.y;
  o[2] = x.z;
  o[3] = x.w;
}

__device__ __forceinline__ Frag8 frag8(const uint32_t (&w)[4]) {
  Frag8 f;
  f.w[0] = w[0];
  f.w[1] = w[1];
  f.w[2] = w[2];
  f.w[3] = w[3];
  return f;
}

// Four weights as bfloat16 high parts (first K half of a product) and low parts
// (second half).
__device__ __forceinline__ Frag8 split_weights(const float (&aw)[4]) {
  Frag8 b;
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const bf16x2_t h = {(__bf16)aw[2 * t], (__bf16)aw[2 * t + 1]};
    uint32_t hw = __builtin_bit_cast(uint32_t, h);
    asm("" : "+v"(hw));  // the packed pair, reused as is (one conversion)
    const bf16x2_t l = {(__bf16)(aw[2 * t] - __uint_as_float(hw << 16)),
                        (__bf16)(aw[2 * t + 1] - __uint_as_float(hw & 0xFFFF0000u))};
    b.w[t] = hw;
    b.w[t + 2] = __builtin_bit_cast(uint32_t, l);
  }
  return b;
}

// Sum over the 4 lanes of a column of the product layout (lanes l, l^16,
// l^32, l^48).
__device__ __forceinline__ float kg_sum(float x) {
  x += __shfl_xor(x, 16, 64);
  x += __shfl_xor(x, 32, 64);
  return x;
}

// The index of a list among a call's lists: prefix list lvl is lvl - t0, the
// full sorted list (lvl > t_hi) comes after the `levels` prefix lists; 0 when
// not causal (the full list only).
__device__ __forceinline__ int level_index(int lvl, int causal, int t0, int t_hi, int levels) {
  return causal ? (lvl > t_hi ? levels : lvl - t0) : 0;
}

// ---- 1. query pass ----------------------------------------------------------
// Bound: vector issue (about 130 instructions per chunk: distances, tests, the
// ten sums), with the value rows' latency behind it.  The rows are copied
// straight into LDS a chunk ahead, as in the forward, instead of gathered into
// registers, and no copy of the dout rows is kept for the key pass (it gathers
// them itself).  16 x 65536, k 128, d_v 128: 616 -> 400 us; 96 x 8192, k 64, d_v
// 64: 207 -> 153 us (161 since its first lists are merged).
template <int DV, bool kOff32, bool kHist>
__global__ void __launch_bounds__(kBtWaves * 64) __attribute__((amdgpu_waves_per_eu(DV <= 128 ? 3 : 1)))
    bwd_tile_query_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ v,
                          const uint16_t* __restrict__ dout, const int32_t* __restrict__ sorted_pos,
                          const int32_t* __restrict__ list_pos, const int32_t* __restrict__ order,
                          const int2* __restrict__ bounds, const uint2* __restrict__ keys_full,
                          const uint2* __restrict__ keys_list, int64_t S, int64_t N, int64_t ct, int causal,
                          int chunk, int t0, int t_hi, int levels, int nl, int64_t cap, float eps, float* __restrict__ dq,
                          SlotRec* __restrict__ rec, float* __restrict__ deps_part,
                          int2* __restrict__ env, const float* __restrict__ mk, const float* __restrict__ mv,
                          float* __restrict__ hk, float* __restrict__ hv) {
  constexpr int NS = DV / 32;  // 32-column slices of a row: one product each
  static_assert(DV % 32 == 0, "d_v must be a multiple of 32");
  using VS = VStage<DV>;
  using Off = typename RowOff<kOff32>::type;
  // List entries staged at once (x, y, z, position), and two chunks of value
  // rows copied straight into LDS (even chunks, odd chunks).
  constexpr int kBtStage = DV <= 128 ? 320 : 128;
  constexpr int kBtStageChunks = kBtStage / kBtChunk;
  static_assert(kBtStage % 64 == 0, "staging fills rounds of 64 entries");
  __shared__ __align__(16) float s_ent[kBtWaves][kBtStage][4];
  __shared__ __align__(16) unsigned char s_v[kBtWaves][2 * VS::kBytes];

  const int lane = threadIdx.x & 63;
  // Wave-uniform (the LDS destination of a copy instruction must be).
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int qn = lane & 15;  // this lane's query (B column) and entry (A row)
  const int kg = lane >> 4;  // this lane's entries 4kg..4kg+3 and column slice 8kg..8kg+7
  const int64_t tiles = S * ct;
  const int64_t nb = gridDim.x;

  // Copy instruction j: this lane's piece of the value row of chunk entry
  // entry_of_row(j kR + vq); the row fragments it reads back (entry qn, columns
  // 32s + 8kg .. + 7) lie at row_addr[s] of the even buffer.
  const int vq = lane / VS::kP, vp = lane % VS::kP;
  uint32_t copy_off[VS::kLoads];
  int copy_ent[VS::kLoads];
#pragma unroll
  for (int j = 0; j < VS::kLoads; ++j) {
    copy_off[j] = uint32_t(16 * (vp ^ VS::sw(j * VS::kR + vq)));
    copy_ent[j] = VS::entry_of_row(j * VS::kR + vq);
  }
  uint32_t row_addr[NS];
  {
    const int rho = VS::row_of_entry(qn);
    const uint32_t base = uint32_t(reinterpret_cast<uintptr_t>(
        (const __attribute__((address_space(3))) unsigned char*)(&s_v[wave][0])));
#pragma unroll
    for (int s = 0; s < NS; ++s) row_addr[s] = base + uint32_t(rho * VS::kRowBytes + 16 * ((4 * s + kg) ^ VS::sw(rho)));
  }

  for (int64_t blk = xcd_contiguous_block(blockIdx.x, nb); blk * kBtWaves < tiles; blk += nb) {
    const int64_t tile = blk * kBtWaves + wave;
    if (tile >= tiles) continue;
    const int64_t seg = tile / ct;
    const int64_t tau = tile - seg * ct;
    const int64_t xs = tau * 16 + qn;  // slot within the segment
    const int64_t slot = seg * N + xs;
    int32_t my_i = -1, my_a = 0, my_b = -1;
    int my_lvl = 0;
    if (xs < N) {
      const int64_t ii = order != nullptr ? int64_t(order[slot]) : xs;
      if (ii >= 0 && ii < N) {
        my_i = int32_t(ii);
        my_lvl = causal ? pool_level(pool_limit(my_i, chunk), t0, t_hi) : 0;
        const int2 bb = bounds[slot];
        my_a = bb.x;
        my_b = bb.y;
      }
    }
    // Slots without a query still hold a defined record.
    if (xs < N && my_i < 0 && kg == 0) {
      SlotRec r = {};
      r.q2_list = kNoList << 16;
      r.a = INT32_MIN;
      rec[slot] = r;
    }
    // Lane l: the tile's window range in list l (empty so far), and this
    // lane's query's part of deps.
    int2 my_env = make_int2(INT32_MAX, INT32_MIN);
    float my_deps = 0.0f;
    uint32_t pending = uint32_t(wave_ballot(my_i >= 0)) & 0xFFFFu;

    // Queries that search one list form a group (nearly always the whole tile).
    while (pending != 0u) {
      const int leader = __ffs(int(pending)) - 1;
      const int g_lvl = __builtin_amdgcn_readlane(my_lvl, leader);
      const uint32_t gmask = uint32_t(wave_ballot(my_i >= 0 && my_lvl == g_lvl)) & pending;
      pending &= ~gmask;
      const LevelList L = level_list(sorted_pos, list_pos, keys_full, keys_list, seg, N, causal, g_lvl, t0, t_hi, cap);
      const bool in_grp = ((gmask >> qn) & 1u) != 0u;
      const bool mine = in_grp && 0 <= my_a && my_a <= my_b && my_b < L.n;
      const int32_t my_lim = causal ? pool_limit(my_i, chunk) : int32_t(N - 1);

      // The group's window range in this list, for the key pass.
      {
        const int lo = wave_min_int(mine ? my_a : INT32_MAX);
        const int hi = wave_max_int(mine ? my_b : INT32_MIN);
        if (lane == level_index(g_lvl, causal, t0, t_hi, levels)) my_env = make_int2(lo, hi);
      }

      float qv[3] = {0.0f, 0.0f, 0.0f};
      uint32_t dfr[NS][4];  // dout of query qn, columns 32s + 8kg .. 32s + 8kg + 7
#pragma unroll
      for (int s = 0; s < NS; ++s) dfr[s][0] = dfr[s][1] = dfr[s][2] = dfr[s][3] = 0u;
      // With the history-mean candidate every query has a candidate.
      if (kHist ? in_grp : mine) {
        const int64_t gq = seg * N + my_i;
        Row3<uint16_t>::load(q, gq, S * N, qv);
#pragma unroll
        for (int s = 0; s < NS; ++s) load8(dout + gq * DV + 32 * s + 8 * kg, dfr[s]);
      }
      float z, pz, xz, yz, u[3], rr[3];

      // Window and pool tests as single unsigned compares (as in the forward).
      const uint32_t span = mine ? uint32_t(my_b - my_a) : 0u;
      const int32_t a_eff = mine ? my_a : INT32_MIN;
      const uint32_t lim_u = uint32_t(my_lim);
      const unsigned char* vbytes = reinterpret_cast<const unsigned char*>(v + seg * N * DV);

      // Copy the value rows of staged chunk ch into LDS buffer `buf` (a missing
      // entry reads row 0 and has weight 0).
      auto copy_rows = [&](int ch, unsigned char* buf) {
#pragma unroll
        for (int j = 0; j < VS::kLoads; ++j) {
          const int32_t pv = __float_as_int(s_ent[wave][ch * kBtChunk + copy_ent[j]][3]);
          const Off boff = Off(pv) * Off(VS::kRowBytes) + Off(copy_off[j]);
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(vbytes + boff),
                                           (__attribute__((address_space(3))) void*)(buf + 1024 * j), 16, 0, 0);
        }
      };
      // Sums over this lane's 4 entries of chunk ch, whose rows' fragments are vf.
      // `masked`: entries outside the window add nothing, whatever their rows hold.
      auto accumulate = [&](int cb, int ch, const u32x4_t(&vf)[NS], auto masked) {
        f32x4_t d = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < NS; ++s)
          d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, vf[s]), frag8(dfr[s]).v, d, 0, 0, 0);
        const int32_t r0 = (cb + ch) * kBtChunk + kg * 4;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const float4 kr = *reinterpret_cast<const float4*>(&s_ent[wave][ch * kBtChunk + kg * 4 + kk][0]);
          float df[3] = {qv[0] - kr.x, qv[1] - kr.y, qv[2] - kr.z};
          const float d2 = fmaf(df[2], df[2], fmaf(df[1], df[1], fmaf(df[0], df[0], eps)));
          const bool in = uint32_t(r0 + kk) - uint32_t(a_eff) <= span && uint32_t(__float_as_int(kr.w)) <= lim_u;
          const float sc = in ? __builtin_amdgcn_rcpf(d2) : 0.0f;
          float p = d[kk];
          if constexpr (masked) {
            p = in ? p : 0.0f;
#pragma unroll
            for (int a = 0; a < 3; ++a) df[a] = in ? df[a] : 0.0f;
          }
          const float s2 = sc * sc;
          z += sc;
          pz = fmaf(sc, p, pz);
          yz += s2;
          const float s2p = s2 * p;
          xz += s2p;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            u[a] = fmaf(s2p, df[a], u[a]);
            rr[a] = fmaf(s2, df[a], rr[a]);
          }
        }
      };

      // The chunks that meet some window, run by run, kBtStageChunks at a time.
      const int a_ch = mine ? my_a / kBtChunk : INT32_MAX;
      const int b_ch = mine ? my_b / kBtChunk : INT32_MIN;
      auto walk = [&](auto masked) {
        z = pz = xz = yz = 0.0f;
#pragma unroll
        for (int a = 0; a < 3; ++a) u[a] = rr[a] = 0.0f;
        for (int c = wave_min_int(a_ch); c != INT32_MAX;) {
          int e = c - 1;
          for (;;) {
            const int e2 = wave_max_int(a_ch <= e + 1 ? b_ch : e);
            if (e2 == e) break;
            e = e2;
          }
          for (int cb = c; cb <= e; cb += kBtStageChunks) {
            const int nch = e - cb + 1 < kBtStageChunks ? e - cb + 1 : kBtStageChunks;
            {
              const int32_t base = cb * kBtChunk;
              int32_t pv[kBtStage / 64];
              uint2 kw[kBtStage / 64];
#pragma unroll
              for (int t = 0; t < kBtStage / 64; ++t) {
                const int e_ = t * 64 + lane;
                const int32_t r = base + e_;
                pv[t] = 0;  // an entry past the list's end: outside every window
                kw[t] = make_uint2(0u, 0u);
                if (e_ < nch * kBtChunk && r < L.n) {
                  pv[t] = L.pos[r];
                  kw[t] = L.key[r];
                }
              }
#pragma unroll
              for (int t = 0; t < kBtStage / 64; ++t) {
                const int e_ = t * 64 + lane;
                if (e_ < nch * kBtChunk) {
                  float kv[3];
                  key_row(kw[t], kv);
                  *reinterpret_cast<float4*>(&s_ent[wave][e_][0]) = make_float4(kv[0], kv[1], kv[2], __int_as_float(pv[t]));
                }
              }
            }
            wave_lds_sync();
            // Chunk ch+1's value rows are copied while chunk ch is summed (past
            // the last chunk the other buffer receives that chunk again, so that
            // one chunk's copies are always in flight behind the one being read).
            unsigned char* const v0 = s_v[wave];
            unsigned char* const v1 = s_v[wave] + VS::kBytes;
            u32x4_t vf[NS];
            copy_rows(0, v0);
            for (int ch = 0; ch < nch; ch += 2) {
              copy_rows(ch + 1 < nch ? ch + 1 : ch, v1);
              read_rows16<0, VS::kLoads>(row_addr, vf);
              accumulate(cb, ch, vf, masked);
              if (ch + 1 >= nch) break;
              copy_rows(ch + 2 < nch ? ch + 2 : ch + 1, v0);
              read_rows16<VS::kBytes, VS::kLoads>(row_addr, vf);
              accumulate(cb, ch + 1, vf, masked);
            }
            // Every copy has landed before the buffers are refilled.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            wave_lds_sync();
          }
          c = wave_min_int(a_ch > e ? a_ch : INT32_MAX);
        }
      };
      walk(std::false_type{});
      // Weight 0 times a term that is not finite is NaN: a value or key row that
      // some query's window leaves out shows in these sums, and only then are
      // they formed again with such terms masked.
      if (wave_ballot(!__builtin_isfinite(pz + rr[0] + rr[1] + rr[2])) != 0ull) walk(std::true_type{});

      z = kg_sum(z);
      pz = kg_sum(pz);
      xz = kg_sum(xz);
      yz = kg_sum(yz);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        u[a] = kg_sum(u[a]);
        rr[a] = kg_sum(rr[a]);
      }
      // The history-mean candidate's terms, once per query (every lane of the
      // query adds them to its totals).
      float s_m = 0.0f, p_m = 0.0f, dm[3] = {0.0f, 0.0f, 0.0f};
      if constexpr (kHist) {
        if (in_grp) {
          const int64_t gq = seg * N + my_i;
          const float4* mrow = reinterpret_cast<const float4*>(mv + gq * DV);
          float part = 0.0f;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            const float4 m0 = mrow[(32 * s + 8 * kg) / 4], m1 = mrow[(32 * s + 8 * kg) / 4 + 1];
            const float mvv[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              part = fmaf(__uint_as_float(dfr[s][t] << 16), mvv[2 * t], part);
              part = fmaf(__uint_as_float(dfr[s][t] & 0xFFFF0000u), mvv[2 * t + 1], part);
            }
          }
          p_m = kg_sum(part);
#pragma unroll
          for (int a = 0; a < 3; ++a) dm[a] = qv[a] - mk[gq * 3 + a];
          s_m = __builtin_amdgcn_rcpf(fmaf(dm[2], dm[2], fmaf(dm[1], dm[1], fmaf(dm[0], dm[0], eps))));
          const float s2 = s_m * s_m;
          z += s_m;
          pz = fmaf(s_m, p_m, pz);
          yz += s2;
          xz = fmaf(s2, p_m, xz);
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            u[a] = fmaf(s2 * p_m, dm[a], u[a]);
            rr[a] = fmaf(s2, dm[a], rr[a]);
          }
        }
      }
      if constexpr (kHist) {
        if (in_grp) {
          // The gradients reaching mean_k[i] and mean_v[i], divided by the
          // history's length.
          const float inv = z > 0.0f ? 1.0f / z : 0.0f;
          const float cc = pz * inv;
          const float inv_cnt = 1.0f / float(causal ? my_i + 1 : N);
          const int64_t gq = seg * N + my_i;
          const float w_m = (p_m - cc) * s_m * s_m * inv;
          if (kg == 0) {
#pragma unroll
            for (int a = 0; a < 3; ++a) hk[gq * 3 + a] = 2.0f * w_m * dm[a] * inv_cnt;
          }
          const float am = s_m * inv * inv_cnt;
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            float4* dst = reinterpret_cast<float4*>(hv + gq * DV + 32 * s + 8 * kg);
            dst[0] = make_float4(am * __uint_as_float(dfr[s][0] << 16), am * __uint_as_float(dfr[s][0] & 0xFFFF0000u),
                                 am * __uint_as_float(dfr[s][1] << 16), am * __uint_as_float(dfr[s][1] & 0xFFFF0000u));
            dst[1] = make_float4(am * __uint_as_float(dfr[s][2] << 16), am * __uint_as_float(dfr[s][2] & 0xFFFF0000u),
                                 am * __uint_as_float(dfr[s][3] << 16), am * __uint_as_float(dfr[s][3] & 0xFFFF0000u));
          }
        }
      }
      if (in_grp && kg == 0) {
        const float inv = z > 0.0f ? 1.0f / z : 0.0f;
        const float cc = pz * inv;
        const int64_t gq = seg * N + my_i;
#pragma unroll
        for (int a = 0; a < 3; ++a) dq[gq * 3 + a] = -2.0f * inv * (u[a] - cc * rr[a]);
        my_deps = -inv * (xz - cc * yz);
        SlotRec r;
        r.q01 = (__float_as_uint(qv[0]) >> 16) | (__float_as_uint(qv[1]) & 0xFFFF0000u);
        const uint32_t list = mine ? uint32_t(level_index(g_lvl, causal, t0, t_hi, levels)) : kNoList;
        r.q2_list = (__float_as_uint(qv[2]) >> 16) | (list << 16);
        r.zinv = inv;
        r.c = cc;
        r.a = mine ? my_a : INT32_MIN;
        r.span = span;
        r.lim = lim_u;
        r.row = my_i;
        rec[slot] = r;
      }
    }
    if (lane < nl) env[(int64_t(lane) * S + seg) * ct + tau] = my_env;
    // The tile's part of deps: lanes 0..15 hold the queries', summed as a tree.
    double tile_deps = my_deps;
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) tile_deps += __shfl_xor(tile_deps, off, 64);
    if (lane == 0) deps_part[tile] = float(tile_deps);
  }
}

// ---- 2. envelopes ---------------------------------------------------------------
// One block per (list, segment): out[t] = (min over t' >= t of the first
// index, max over t' <= t of the last index).  Each thread scans a stretch of
// consecutive tiles; the stretches' totals are scanned in LDS.
constexpr int kEnvThreads = 256;

__global__ void __launch_bounds__(kEnvThreads)
    bwd_envelope_kernel(const int2* __restrict__ env, int64_t ct, int2* __restrict__ env2) {
  __shared__ int s_mx[kEnvThreads];
  __shared__ int s_mn[kEnvThreads];
  const int tid = threadIdx.x;
  const int2* in = env + int64_t(blockIdx.x) * ct;
  int2* out = env2 + int64_t(blockIdx.x) * ct;
  const int64_t per = (ct + kEnvThreads - 1) / kEnvThreads;
  const int64_t b0 = int64_t(tid) * per < ct ? int64_t(tid) * per : ct;
  const int64_t b1 = b0 + per < ct ? b0 + per : ct;
  int mx = INT32_MIN, mn = INT32_MAX;
  for (int64_t t = b0; t < b1; ++t) {
    const int2 r = in[t];
    mx = r.y > mx ? r.y : mx;
    mn = r.x < mn ? r.x : mn;
  }
  s_mx[tid] = mx;
  s_mn[tid] = mn;
  __syncthreads();
  // Inclusive scans: maximum from the first stretch, minimum from the last.
  for (int off = 1; off < kEnvThreads; off <<= 1) {
    const int a = tid >= off ? s_mx[tid - off] : INT32_MIN;
    const int b = tid + off < kEnvThreads ? s_mn[tid + off] : INT32_MAX;
    __syncthreads();
    s_mx[tid] = a > s_mx[tid] ? a : s_mx[tid];
    s_mn[tid] = b < s_mn[tid] ? b : s_mn[tid];
    __syncthreads();
  }
  int carry = tid > 0 ? s_mx[tid - 1] : INT32_MIN;
  for (int64_t t = b0; t < b1; ++t) {
    const int y = in[t].y;
    carry = y > carry ? y : carry;
    out[t].y = carry;
  }
  carry = tid + 1 < kEnvThreads ? s_mn[tid + 1] : INT32_MAX;
  for (int64_t t = b1 - 1; t >= b0; --t) {
    const int x = in[t].x;
    carry = x < carry ? x : carry;
    out[t].x = carry;
  }
}

// First tile t in [0, ct) with key(t) >= want for a non-decreasing key
// (ct when none): the running maximum of last indices (kHi) or the running
// minimum of first indices.
template <bool kHi>
__device__ __forceinline__ int64_t first_at_least(const int2* p, int64_t ct, int want) {
  int64_t lo = 0, hi = ct;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    const int2 r = p[mid];
    if ((kHi ? r.y : r.x) >= want)
      hi = mid;
    else
      lo = mid + 1;
  }
  return lo;
}

// Per list, segment and chunk: the candidate tiles [ta, tb).  Tiles before ta
// end before the chunk; tiles from tb on start after it.  One thread per
// (list, segment, chunk), in the envelopes' layout.
__global__ void __launch_bounds__(256)
    bwd_ranges_kernel(const int2* __restrict__ env2, int64_t S, int64_t N, int64_t ct, int causal, int t0, int t_hi,
                      int levels, int nl, int2* __restrict__ ranges) {
  const int64_t t = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
  if (t >= int64_t(nl) * S * ct) return;
  const int64_t row = t / ct;
  const int64_t c = t - row * ct;
  const int li = int(row / S);
  const int lvl = !causal ? 0 : (li == levels ? t_hi + 1 : t0 + li);
  const int64_t ln = (causal && lvl <= t_hi) ? (int64_t(1) << lvl) : N;
  if (c * 16 >= ln) return;
  const int lo_c = int(c * 16);
  const int hi_c = int(c * 16 + 15 < ln - 1 ? c * 16 + 15 : ln - 1);
  const int2* ev2 = env2 + row * ct;
  ranges[t] = make_int2(int(first_at_least<true>(ev2, ct, lo_c)), int(first_at_least<false>(ev2, ct, hi_c + 1)));
}

// Envelopes and candidate ranges of a (list, segment) in one workgroup, for
// segments of up to kEnvLdsTiles tiles: the envelopes stay in LDS (a thread
// scans PER consecutive tiles in registers, wavefronts and the block are joined
// by shuffles), where both binary searches of a chunk then run, instead of
// through memory in two launches (16 x 65536: 17.5 + 12.5 -> 13.8 us).
constexpr int64_t kEnvLdsTiles = 8192;

template <int THREADS, int PER>
__global__ void __launch_bounds__(THREADS)
    bwd_envelope_ranges_kernel(const int2* __restrict__ env, int64_t S, int64_t N, int ct, int causal, int t0, int t_hi,
                               int levels, int2* __restrict__ ranges) {
  constexpr int kWaves = THREADS / 64;
  __shared__ int s_mx[THREADS * PER];  // running maximum of the tiles' last indices
  __shared__ int s_mn[THREADS * PER];  // running minimum, from the last tile, of their first indices
  __shared__ int s_wmx[kWaves], s_wmn[kWaves];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int64_t row = blockIdx.x;  // list * S + segment
  const int li = int(row / S);
  const int lvl = !causal ? 0 : (li == levels ? t_hi + 1 : t0 + li);
  const int ln = (causal && lvl <= t_hi) ? (1 << lvl) : int(N);
  const int2* in = env + row * ct;
  int2 r[PER];
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const int t = tid * PER + j;
    const int2 x = in[t < ct ? t : ct - 1];
    r[j] = t < ct ? x : make_int2(INT32_MAX, INT32_MIN);
  }
  int mx = INT32_MIN, mn = INT32_MAX;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    mx = r[j].y > mx ? r[j].y : mx;
    mn = r[j].x < mn ? r[j].x : mn;
  }
  // Inclusive scans over the threads: maximum upwards, minimum downwards.
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int a = __shfl_up(mx, off, 64), b = __shfl_down(mn, off, 64);
    if (lane >= off) mx = a > mx ? a : mx;
    if (lane + off < 64) mn = b < mn ? b : mn;
  }
  if (lane == 63) s_wmx[wave] = mx;
  if (lane == 0) s_wmn[wave] = mn;
  int before = __shfl_up(mx, 1, 64), after = __shfl_down(mn, 1, 64);
  if (lane == 0) before = INT32_MIN;
  if (lane == 63) after = INT32_MAX;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    if (w < wave) before = s_wmx[w] > before ? s_wmx[w] : before;
    if (w > wave) after = s_wmn[w] < after ? s_wmn[w] : after;
  }
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    before = r[j].y > before ? r[j].y : before;
    s_mx[tid * PER + j] = before;
  }
#pragma unroll
  for (int j = PER - 1; j >= 0; --j) {
    after = r[j].x < after ? r[j].x : after;
    s_mn[tid * PER + j] = after;
  }
  __syncthreads();
  const int chunks = (ln + 15) / 16;
  for (int c = tid; c < chunks; c += THREADS) {
    const int lo_c = c * 16;
    const int hi_c = c * 16 + 15 < ln - 1 ? c * 16 + 15 : ln - 1;
    // First tiles with maximum >= lo_c and with minimum >= hi_c + 1, halving
    // both at once (the tiles past ct hold the neutral ends).
    int a0 = 0, a1 = ct, b0 = 0, b1 = ct;
    while (a0 < a1 || b0 < b1) {
      const int am = (a0 + a1) >> 1, bm = (b0 + b1) >> 1;
      const int av = s_mx[am < ct ? am : ct - 1], bv = s_mn[bm < ct ? bm : ct - 1];
      if (a0 < a1) {
        if (av >= lo_c)
          a1 = am;
        else
          a0 = am + 1;
      }
      if (b0 < b1) {
        if (bv >= hi_c + 1)
          b1 = bm;
        else
          b0 = bm + 1;
      }
    }
    ranges[row * ct + c] = make_int2(a0, b0);
  }
}

// ---- 3. key pass ------------------------------------------------------------------
// A wavefront takes SUB consecutive 16-entry chunks of one list (two; one for
// d_v = 256, whose sums fill the registers, and for short lists) and walks the tiles whose
// windows meet them, so that a tile's dout rows, copied into LDS, serve both
// chunks.  Wavefronts share nothing, so no barrier holds the fast ones up: while
// a tile is summed the next tile's rows are copied straight into LDS and the
// records of the one after it load into registers.  The rows are read back
// twice: as they lie (dot products, A operand: the tile's queries x 32 columns)
// and transposed (dv, A operand: 16 columns x queries).
// Two chunks, not one: the dout rows, their two reads and the records are then
// shared, and the longer visits outweigh the third wavefront per SIMD that one
// chunk leaves room for (16 x 65536, k 128, d_v 128: 886 against 935 us; with the
// barrier-coupled blocks of four chunks before, 1144 us; 96 x 8192, k 64, d_v 64:
// 340 against 355, before 431 us; 861 and 318 us now that the first lists are
// merged).  A wavefront spends about a quarter of its time
// on its first dependent loads and a third on the sums; the prefix lists' adds
// (dv read and written again) take a quarter of the call.  Persistent wavefronts
// that prefetch the next unit were slower (1004 us: they wait for their own
// stores).
constexpr int kKeyWaves = 4;  // wavefronts per block
constexpr int kKeyThreads = kKeyWaves * 64;

template <int DV, int SUB, bool kOff32>
__global__ void __launch_bounds__(kKeyThreads) __attribute__((amdgpu_waves_per_eu(DV <= 32 ? 4 : (DV <= 64 ? 3 : 2))))
    bwd_tile_key_kernel(const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout,
                        const int32_t* __restrict__ sorted_pos, const int32_t* __restrict__ list_pos,
                        const uint2* __restrict__ keys_full, const uint2* __restrict__ keys_list,
                        const SlotRec* __restrict__ rec, const int2* __restrict__ env,
                        const int2* __restrict__ ranges, int64_t S, int64_t N, int64_t ct, int causal, int t0,
                        int t_hi, int levels, int64_t cap, int lvl, int first, float eps, float* __restrict__ dk,
                        float* __restrict__ dv) {
  using VS = VStage<DV>;
  constexpr int NS = DV / 32;
  constexpr int E = VS::kBlocks;  // 16-column blocks of a row: one dv product each
  // Byte offsets into a segment's dout rows: 32-bit when they span under 4 GiB.
  using Off = typename RowOff<kOff32>::type;
  __shared__ __align__(16) uint32_t s_rec[kKeyWaves][2][16][8];
  __shared__ __align__(512) unsigned char s_d[kKeyWaves][2 * VS::kBytes];
  const int lane = threadIdx.x & 63;
  // Wave-uniform (the LDS destination of a copy instruction must be).
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int ent = lane & 15;  // this lane's entry of each chunk (B column)
  const int kg = lane >> 4;   // this lane's queries 4kg..4kg+3 of a tile
  const uint32_t li = uint32_t(level_index(lvl, causal, t0, t_hi, levels));
  const int64_t ln = (causal && lvl <= t_hi) ? (int64_t(1) << lvl) : N;
  const int64_t cl = (ln + kBtChunk - 1) / kBtChunk;  // chunks per segment
  const int64_t cw = (cl + SUB - 1) / SUB;            // wavefronts' worth of them
  const int64_t total = S * cw;
  const int64_t nb = gridDim.x;
  const int32_t n32 = int32_t(N);

  // Copy instruction j: this lane's piece of the dout row of tile query
  // entry_of_row(j kR + vq), whose position lane copy_src + j copy_step holds;
  // row fragments (query ent) and transposed fragments of a buffer (see VStage).
  const int vq = lane / VS::kP, vp = lane % VS::kP;
  uint32_t copy_off[VS::kLoads];
#pragma unroll
  for (int j = 0; j < VS::kLoads; ++j) copy_off[j] = uint32_t(16 * (vp ^ VS::sw(j * VS::kR + vq)));
  const int copy_src = 2 * VS::entry_of_row(vq) + 1;
  constexpr int copy_step = 2 * (VS::entry_of_row(VS::kR % kChunk) - VS::entry_of_row(0));
  uint32_t row_off[NS], tr_off[E];
  {
    const int rho = VS::row_of_entry(ent);
#pragma unroll
    for (int s = 0; s < NS; ++s) row_off[s] = uint32_t(rho * VS::kRowBytes + 16 * ((4 * s + kg) ^ VS::sw(rho)));
    const int rt = VS::row_of_entry(4 * kg + ent / 4);
    const int x = (ent % 4) / 2, half = ent % 2;
#pragma unroll
    for (int j = 0; j < E; ++j) tr_off[j] = uint32_t(rt * VS::kRowBytes + 16 * ((2 * j + x) ^ VS::sw(rt)) + 8 * half);
  }

  for (int64_t blk = xcd_contiguous_block(blockIdx.x, nb); blk * kKeyWaves < total; blk += nb) {
    const int64_t unit = blk * kKeyWaves + wave;
    if (unit >= total) continue;
    const int64_t seg = unit / cw;
    const int64_t c = (unit - seg * cw) * SUB;  // this wavefront's first chunk
    const LevelList L = level_list(sorted_pos, list_pos, keys_full, keys_list, seg, N, causal, lvl, t0, t_hi, cap);
    const uint16_t* vseg = v + seg * N * DV;
    int32_t e[SUB], pos_e[SUB];
    float kv[SUB][3];
    uint32_t vfr[SUB][NS][4];  // value slices of this lane's entries: columns 32s + 8kg .. + 7
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      // An entry past the list's end lies outside every window.
      e[u] = int32_t((c + u) * kBtChunk + ent);
      pos_e[u] = e[u] < L.n ? L.pos[e[u]] : 0;
      const uint2 kw = e[u] < L.n ? L.key[e[u]] : make_uint2(0u, 0u);
      key_row(kw, kv[u]);
    }
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
#pragma unroll
      for (int s = 0; s < NS; ++s) load8(vseg + int64_t(pos_e[u]) * DV + 32 * s + 8 * kg, vfr[u][s]);
    }

    f32x4_t acc[SUB][E];
    float gk[SUB][3];
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
#pragma unroll
      for (int j = 0; j < E; ++j) acc[u][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int a = 0; a < 3; ++a) gk[u][a] = 0.0f;
    }

    const int lo_c = int(c * kBtChunk);
    const int hi_c = int((c + SUB) * kBtChunk < ln ? (c + SUB) * kBtChunk : ln) - 1;
    const int2* ev = env + (int64_t(li) * S + seg) * ct;
    const int2* rgs = ranges + (int64_t(li) * S + seg) * ct;
    // The candidate ranges grow with the chunk.
    const int ta = rgs[c].x, tb = rgs[c + SUB - 1 < cl ? c + SUB - 1 : cl - 1].y;
    const SlotRec* rseg = rec + seg * N;
    const unsigned char* dbytes = reinterpret_cast<const unsigned char*>(dout + seg * N * DV);

    // The tiles whose windows meet the chunks, 64 candidates tested at once.
    int blk_base = ta, cur_base = ta;
    uint64_t pend = 0ull;
    auto next_tile = [&]() -> int32_t {
      while (pend == 0ull && blk_base < tb) {
        const int tl = blk_base + lane;
        const int2 rg = tl < tb ? ev[tl] : make_int2(INT32_MAX, INT32_MIN);
        pend = wave_ballot((rg.x <= hi_c) & (rg.y >= lo_c));
        cur_base = blk_base;
        blk_base += 64;
      }
      if (pend == 0ull) return -1;
      const int b = __ffsll((unsigned long long)pend) - 1;
      pend &= pend - 1ull;
      return cur_base + b;
    };
    // Half a record per lane (lanes 0..31; the others repeat them): q, list,
    // 1/Z, c on even lanes, window, pool limit and position on odd ones.  (The
    // slots past the segment's end of its last tile read what follows its
    // records in the workspace; their records are replaced before use.)
    uint4 st = make_uint4(0u, 0u, 0u, 0u);
    auto load_rec = [&](int32_t tau) { st = reinterpret_cast<const uint4*>(rseg + tau * 16)[lane & 31]; };
    // The loaded records into buffer `buf` (a query of another list, or past
    // the segment's end, gets the empty window), and their dout rows' copies
    // issued.  A query of weight 0 still enters the products and sums, where an
    // infinity or NaN would not vanish: one without a window here has q, 1/Z and
    // c zero and takes the row of the tile's first query with one.
    auto stage = [&](int32_t tau, int buf) {
      uint4 r = st;
      const uint32_t pair = uint32_t(__builtin_amdgcn_update_dpp(int(r.y), int(r.y), 0xB1, 0xF, 0xF, false));
      const uint32_t list = ((lane & 1) != 0 ? pair : r.y) >> 16;  // held by the even lane
      const bool past = tau * 16 + ((lane & 31) >> 1) >= n32;
      if (past) r = make_uint4(0u, 0u, 0u, 0u);
      const bool other = past || list != li;
      // A visited tile has a window in this list, so such a lane exists.
      const uint64_t own = wave_ballot((lane & 1) != 0 && !other);
      const uint32_t own_row = uint32_t(
          __builtin_amdgcn_readlane(int(r.w), own != 0ull ? __ffsll((unsigned long long)own) - 1 : 0));
      if (other) {
        const bool odd = (lane & 1) != 0;
        r.x = odd ? uint32_t(INT32_MIN) : 0u;
        r.y = 0u;
        r.z = odd ? r.z : 0u;
        r.w = odd && own != 0ull ? own_row : 0u;
      }
      if (lane < 32) *reinterpret_cast<uint4*>(&s_rec[wave][buf][lane >> 1][(lane & 1) * 4]) = r;
#pragma unroll
      for (int j = 0; j < VS::kLoads; ++j) {
        const int32_t row = __shfl(int(r.w), copy_src + j * copy_step, 64);
        const Off boff = Off(row) * Off(VS::kRowBytes) + Off(copy_off[j]);
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(dbytes + boff),
                                         (__attribute__((address_space(3))) void*)(s_d[wave] + buf * VS::kBytes + 1024 * j),
                                         16, 0, 0);
      }
    };
    // The rows' fragments of buffer `buf`, as they lie and transposed (read
    // twice, once per K half of the products).
    u32x4_t dr[NS];
    s16x4_t tr[2 * E];
    auto read_tile = [&](int buf) {
      const unsigned char* rows = s_d[wave] + buf * VS::kBytes;
#pragma unroll
      for (int s = 0; s < NS; ++s) dr[s] = *reinterpret_cast<const u32x4_t*>(rows + row_off[s]);
#pragma unroll
      for (int j = 0; j < E; ++j) {
        auto* at = (__attribute__((address_space(3))) s16x4_t*)(rows + tr_off[j]);
        tr[2 * j] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(at);
        tr[2 * j + 1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(at);
      }
    };
    auto sum_tile = [&](int buf) {
      // Dot products: lane holds p for queries 4kg..4kg+3 and entry ent of each
      // chunk (A rows: dout of the tile's query ent).
      f32x4_t d[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        d[u] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < NS; ++s)
          d[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, dr[s]), frag8(vfr[u][s]).v, d[u], 0, 0, 0);
      }
      float aw[SUB][4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const uint4 h0 = *reinterpret_cast<const uint4*>(&s_rec[wave][buf][kg * 4 + r][0]);
        const uint4 h1 = *reinterpret_cast<const uint4*>(&s_rec[wave][buf][kg * 4 + r][4]);
        const float qx = __uint_as_float(h0.x << 16);
        const float qy = __uint_as_float(h0.x & 0xFFFF0000u);
        const float qz = __uint_as_float(h0.y << 16);
        const float zinv = __uint_as_float(h0.z), cc = __uint_as_float(h0.w);
#pragma unroll
        for (int u = 0; u < SUB; ++u) {
          const float df[3] = {qx - kv[u][0], qy - kv[u][1], qz - kv[u][2]};
          const float d2 = fmaf(df[2], df[2], fmaf(df[1], df[1], fmaf(df[0], df[0], eps)));
          const bool in = (uint32_t(e[u]) - h1.x <= h1.y) & (uint32_t(pos_e[u]) <= h1.z);
          const float sc = in ? __builtin_amdgcn_rcpf(d2) : 0.0f;
          aw[u][r] = sc * zinv;
          const float w = (d[u][r] - cc) * sc * aw[u][r];
#pragma unroll
          for (int a = 0; a < 3; ++a) gk[u][a] = fmaf(w, df[a], gk[u][a]);
        }
      }
      // dv^T += dout^T (columns x queries) * A (queries x entries), high and
      // low parts of A in one product per 16 columns (the K halves hold the
      // same dout fragment).
      Frag8 b[SUB];
#pragma unroll
      for (int u = 0; u < SUB; ++u) b[u] = split_weights(aw[u]);
#pragma unroll
      for (int j = 0; j < E; ++j) {
        const bf16x8_t a8 = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(tr[2 * j], tr[2 * j + 1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
        for (int u = 0; u < SUB; ++u) acc[u][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a8, b[u].v, acc[u][j], 0, 0, 0);
      }
    };
    const int32_t head = next_tile();
    const bool touched = head >= 0;
    if (touched) {
      load_rec(head);
      stage(head, 0);
      int32_t nxt = next_tile();
      load_rec(nxt >= 0 ? nxt : head);
      // The tile in buffer `buf` is read whole first; then the next tile's
      // copies into the other buffer are issued and the records of the one
      // after it loaded (reads issued after the copies would wait for them),
      // and the tile is summed meanwhile.
      for (int buf = 0;; buf ^= 1) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this tile's rows (and the next one's records) have landed
        read_tile(buf);
        const bool more = nxt >= 0;
        if (more) {
          stage(nxt, buf ^ 1);
          nxt = next_tile();
          // Loaded without a branch, which could cost a register copy and with it a
          // wait for the load.
          load_rec(nxt >= 0 ? nxt : head);
        }
        wave_lds_sync();
        sum_tile(buf);
        if (!more) break;
      }
    }
    // Weight 0 times a term that is not finite is NaN: an infinite or NaN row of
    // q, dout, k or v would spoil sums of keys (or, for k and v, of the key) in no
    // window that holds it.  Each leaves its NaN in dk, and only then are the
    // sums formed again, query by query on the vector units, pairs outside a
    // window left out.  (Records and rows come straight from memory: this path
    // must not take registers from the one above.  16 x 65536, k 128, d_v 128: finite
    // 1.32 ms a call, one infinite dout row a segment 1.44, dout all NaN 6.9.)
    float all = 0.0f;  // infinite or NaN when one of them is
#pragma unroll
    for (int u = 0; u < SUB; ++u) all += gk[u][0] + gk[u][1] + gk[u][2];
    if (wave_ballot(!__builtin_isfinite(all)) != 0ull) {
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
#pragma unroll
        for (int j = 0; j < E; ++j) acc[u][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int a = 0; a < 3; ++a) gk[u][a] = 0.0f;
      }
      blk_base = ta;
      for (int32_t t = next_tile(); t >= 0; t = next_tile()) {
        // Lane i: query i of the tile; those whose windows meet the chunks.
        const int32_t xs = t * 16 + ent;
        const SlotRec mine = rseg[xs < n32 ? xs : n32 - 1];
        const bool meets = xs < n32 && (mine.q2_list >> 16) == li && mine.a <= hi_c && mine.a + int32_t(mine.span) >= lo_c;
        for (uint32_t m = uint32_t(wave_ballot(meets)) & 0xFFFFu; m != 0u; m &= m - 1u) {
          const int i = __ffs(int(m)) - 1;
          auto bits = [&](uint32_t x) { return uint32_t(__builtin_amdgcn_readlane(int(x), i)); };
          SlotRec r;
          r.q01 = bits(mine.q01);
          r.q2_list = bits(mine.q2_list);
          r.zinv = __uint_as_float(bits(__float_as_uint(mine.zinv)));
          r.c = __uint_as_float(bits(__float_as_uint(mine.c)));
          r.a = int32_t(bits(uint32_t(mine.a)));
          r.span = bits(mine.span);
          r.lim = bits(mine.lim);
          r.row = int32_t(bits(uint32_t(mine.row)));
          const uint16_t* drow = dout + (seg * N + r.row) * DV;
#pragma unroll
          for (int u = 0; u < SUB; ++u) {
            float p = 0.0f;
#pragma unroll
            for (int s = 0; s < NS; ++s) {
              uint32_t x[4];
              load8(drow + 32 * s + 8 * kg, x);
#pragma unroll
              for (int c2 = 0; c2 < 4; ++c2) {
                p = fmaf(__uint_as_float(x[c2] << 16), __uint_as_float(vfr[u][s][c2] << 16), p);
                p = fmaf(__uint_as_float(x[c2] & 0xFFFF0000u), __uint_as_float(vfr[u][s][c2] & 0xFFFF0000u), p);
              }
            }
            p = kg_sum(p);
            const float df[3] = {__uint_as_float(r.q01 << 16) - kv[u][0], __uint_as_float(r.q01 & 0xFFFF0000u) - kv[u][1],
                                 __uint_as_float(r.q2_list << 16) - kv[u][2]};
            const float sc = __builtin_amdgcn_rcpf(fmaf(df[2], df[2], fmaf(df[1], df[1], fmaf(df[0], df[0], eps))));
            const float aw = sc * r.zinv;
            const float w = (p - r.c) * sc * aw;
            if ((uint32_t(e[u]) - uint32_t(r.a) <= r.span) & (uint32_t(pos_e[u]) <= r.lim)) {
              if (kg == 0) {  // summed over the 4 lanes of an entry below
#pragma unroll
                for (int a = 0; a < 3; ++a) gk[u][a] = fmaf(w, df[a], gk[u][a]);
              }
#pragma unroll
              for (int j = 0; j < E; ++j) {
                asm volatile("" ::: "memory");  // one block's loads at a time
#pragma unroll
                for (int c4 = 0; c4 < 4; ++c4)
                  acc[u][j][c4] = fmaf(aw, bf16_bits_to_float(drow[16 * j + 4 * kg + c4]), acc[u][j][c4]);
              }
            }
          }
        }
      }
    }

    // Write (full list) or add (prefix lists) these chunks' rows: lane holds
    // columns 16j + 4kg .. + 3 of entry ent's dv row for every block j.
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
#pragma unroll
      for (int a = 0; a < 3; ++a) gk[u][a] = 2.0f * kg_sum(gk[u][a]);
      if (e[u] < L.n && (first || touched)) {
        float* drow = dv + (seg * N + pos_e[u]) * int64_t(DV) + kg * 4;
        if (!first) {
          float4 old[E];
#pragma unroll
          for (int j = 0; j < E; ++j) old[j] = *reinterpret_cast<const float4*>(drow + 16 * j);
#pragma unroll
          for (int j = 0; j < E; ++j)
            acc[u][j] += f32x4_t{old[j].x, old[j].y, old[j].z, old[j].w};
        }
#pragma unroll
        for (int j = 0; j < E; ++j)
          *reinterpret_cast<float4*>(drow + 16 * j) = make_float4(acc[u][j][0], acc[u][j][1], acc[u][j][2], acc[u][j][3]);
        if (kg == 0) {
          float* krow = dk + (seg * N + pos_e[u]) * 3;
#pragma unroll
          for (int a = 0; a < 3; ++a) krow[a] = first ? gk[u][a] : krow[a] + gk[u][a];
        }
      }
    }
    // The next chunks' copies reuse the buffers once every read is done.
    wave_lds_sync();
  }
}

// ---- deps -----------------------------------------------------------------------
// Fixed-order sum of the tiles' parts: one block when there are at most
// kRedOne of them, else block sums first and then one block over those.  Sums
// are kept in 64 bits: the parts' signs differ, so the sum is smaller than what
// it adds up and would show every rounding of 32 bits (the loads bound the
// kernel either way).
constexpr int64_t kRedOne = int64_t(1) << 17;

template <typename In, typename Out>
__global__ void __launch_bounds__(kRedThreads)
    bwd_tile_reduce_kernel(const In* __restrict__ part, int64_t n, int64_t per_block, Out* __restrict__ sums) {
  __shared__ double s_red[kRedThreads];
  const int64_t b0 = int64_t(blockIdx.x) * per_block;
  const int64_t b1 = b0 + per_block < n ? b0 + per_block : n;
  // Independent loads in batches, so their latencies overlap.
  constexpr int kBatch = 16;
  double acc = 0.0;
  for (int64_t t = b0 + threadIdx.x; t < b1; t += kBatch * kRedThreads) {
    In x[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) {
      const int64_t e = t + j * kRedThreads;
      x[j] = part[e < b1 ? e : t];
    }
#pragma unroll
    for (int j = 0; j < kBatch; ++j) acc += t + j * kRedThreads < b1 ? double(x[j]) : 0.0;
  }
  s_red[threadIdx.x] = acc;
  __syncthreads();
  for (int w = kRedThreads / 2; w > 0; w >>= 1) {
    if (int(threadIdx.x) < w) s_red[threadIdx.x] += s_red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = Out(s_red[0]);
}

template <int DV>
hipError_t launch_tile_bwd_t(const uint16_t* q, const uint16_t* v, const uint16_t* dout, int64_t S, int64_t N,
                             int topk, bool causal, int chunk, const int32_t* perm, const int32_t* list_pos,
                             const int32_t* q_order, const int2* bounds, const uint2* keys_full,
                             const uint2* keys_list, float eps, HistMean hm, float* dq, float* dk, float* dv,
                             float* deps, const TileBwdWs& ws, char* wsb, hipStream_t stream) {
  const ListPlan lp = list_plan(N, tile_bwd_list_topk(N, topk));
  const int64_t ct = ceil_div(N, int64_t(16));
  const int nl = tile_bwd_levels(N, topk, causal);
  const bool off32 = N * int64_t(DV) * 2 <= int64_t(0xFFFFFFFF);
  SlotRec* rec = reinterpret_cast<SlotRec*>(wsb + ws.rec_off);
  float* part = reinterpret_cast<float*>(wsb + ws.part_off);
  int2* env = reinterpret_cast<int2*>(wsb + ws.env_off);
  int2* env2 = reinterpret_cast<int2*>(wsb + ws.env2_off);
  int2* ranges = reinterpret_cast<int2*>(wsb + ws.ranges_off);
  float* hk = reinterpret_cast<float*>(wsb + ws.hist_k_off);
  float* hv = reinterpret_cast<float*>(wsb + ws.hist_v_off);
  double* sums = reinterpret_cast<double*>(wsb + ws.sums_off);
  const int64_t nenv = int64_t(nl) * S * ct;
  const int cz = causal ? 1 : 0;
  {
    const int64_t tiles = S * ct;
    const int64_t want = ceil_div(tiles, int64_t(kBtWaves));
    const unsigned blocks = unsigned(want < (int64_t(1) << 20) ? want : (int64_t(1) << 20));
#define ZETA_BT_QUERY(OFF, HIST)                                                                                  \
  hipLaunchKernelGGL((bwd_tile_query_kernel<DV, OFF, HIST>), dim3(blocks), dim3(kBtWaves * 64), 0, stream, q, v, dout, \
                     perm, list_pos, q_order, bounds, keys_full, keys_list, S, N, ct, cz, chunk, lp.t0, lp.t_hi,        \
                     lp.levels, nl, lp.cap, eps, dq, rec, part, env, hm.k, hm.v, hk, hv)
    if (off32) {
      if (hm.k != nullptr)
        ZETA_BT_QUERY(true, true);
      else
        ZETA_BT_QUERY(true, false);
    } else {
      if (hm.k != nullptr)
        ZETA_BT_QUERY(false, true);
      else
        ZETA_BT_QUERY(false, false);
    }
#undef ZETA_BT_QUERY
  }
  if (ct <= kEnvLdsTiles) {
    const dim3 grid(unsigned(int64_t(nl) * S));
#define ZETA_BT_ENV(THREADS, PER)                                                                                \
  hipLaunchKernelGGL((bwd_envelope_ranges_kernel<THREADS, PER>), grid, dim3(THREADS), 0, stream, env, S, N, int(ct), \
                     cz, lp.t0, lp.t_hi, lp.levels, ranges)
    if (ct <= 256)
      ZETA_BT_ENV(256, 1);
    else if (ct <= 1024)
      ZETA_BT_ENV(256, 4);
    else if (ct <= 4096)
      ZETA_BT_ENV(1024, 4);
    else
      ZETA_BT_ENV(1024, 8);
#undef ZETA_BT_ENV
  } else {
    hipLaunchKernelGGL(bwd_envelope_kernel, dim3(unsigned(int64_t(nl) * S)), dim3(kEnvThreads), 0, stream, env, ct,
                       env2);
    hipLaunchKernelGGL(bwd_ranges_kernel, dim3(unsigned(ceil_div(nenv, int64_t(256)))), dim3(256), 0, stream, env2, S,
                       N, ct, cz, lp.t0, lp.t_hi, lp.levels, nl, ranges);
  }
  // The full list first (its launch writes every key's rows), then the prefix
  // lists from the longest down.
  for (int li = nl - 1; li >= 0; --li) {
    const int lvl = !causal ? 0 : (li == lp.levels ? lp.t_hi + 1 : lp.t0 + li);
    const int64_t ln = (causal && lvl <= lp.t_hi) ? (int64_t(1) << lvl) : N;
    const int64_t chunks = ceil_div(ln, int64_t(16));
    // One chunk a wavefront where two leave SIMDs without a wavefront: the
    // launch then lasts as long as one wavefront's visits (a list of 1024 entries
    // in 16 segments, d_v 128: 21.9 -> 15.9 us).
    const bool pairs = DV <= 128 && S * ceil_div(chunks, int64_t(2)) > 1024;
    const int64_t want = ceil_div(S * (pairs ? ceil_div(chunks, int64_t(2)) : chunks), int64_t(kKeyWaves));
    const unsigned blocks = unsigned(want < (int64_t(1) << 20) ? want : (int64_t(1) << 20));
#define ZETA_BT_KEY(SUB, OFF)                                                                                       \
  hipLaunchKernelGGL((bwd_tile_key_kernel<DV, SUB, OFF>), dim3(blocks), dim3(kKeyThreads), 0, stream, v, dout, perm,     \
                     list_pos, keys_full, keys_list, rec, env, ranges, S, N, ct, cz, lp.t0, lp.t_hi, lp.levels, lp.cap, \
                     lvl, li == nl - 1 ? 1 : 0, eps, dk, dv)
    constexpr int kPair = DV <= 128 ? 2 : 1;
    if (pairs) {
      if (off32)
        ZETA_BT_KEY(kPair, true);
      else
        ZETA_BT_KEY(kPair, false);
    } else {
      if (off32)
        ZETA_BT_KEY(1, true);
      else
        ZETA_BT_KEY(1, false);
    }
#undef ZETA_BT_KEY
  }
  if (hm.k != nullptr) {
    // The gradients reaching the means pass to the rows of every history.
    const hipError_t e = launch_history_spread(hv, dv, DV, hk, dk, 3, S, N, causal, wsb + ws.hist_scan_off, stream);
    if (e != hipSuccess) return e;
  }
  const int64_t total = S * ct;
  if (total <= kRedOne) {
    hipLaunchKernelGGL((bwd_tile_reduce_kernel<float, float>), dim3(1), dim3(kRedThreads), 0, stream, part, total, total,
                       deps);
    return hipGetLastError();
  }
  const int64_t nred = ceil_div(total, kTileBwdRedPer) < kTileBwdRedMax ? ceil_div(total, kTileBwdRedPer)
                                                                        : kTileBwdRedMax;
  const int64_t per = ceil_div(total, nred);
  hipLaunchKernelGGL((bwd_tile_reduce_kernel<float, double>), dim3(unsigned(nred)), dim3(kRedThreads), 0, stream, part,
                     total, per, sums);
  hipLaunchKernelGGL((bwd_tile_reduce_kernel<double, float>), dim3(1), dim3(kRedThreads), 0, stream, sums, nred, nred,
                     deps);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_select_attend_bwd(const void* q, const void* k, const void* v, const void* dout, int64_t S,
                                    int64_t N, int dk_, int dv_, int topk, bool causal, int chunk,
                                    const uint32_t* q_codes, const uint32_t* sorted_codes, const int32_t* perm,
                                    const int32_t* q_order, float eps, HistMean hm, float* dq, float* dk,
                                    float* dv, float* deps, void* workspace, hipStream_t stream) {
  const uint32_t* list_codes = nullptr;
  const int32_t* list_pos = nullptr;
  const TileBwdWs ws = tile_bwd_ws(S, N, dv_, topk, causal ? 1 : 0, hm.k != nullptr);
  char* wsb = static_cast<char*>(workspace);
  int2* bounds = reinterpret_cast<int2*>(wsb + ws.fused.bounds_off);
  uint2* keys_full = reinterpret_cast<uint2*>(wsb + ws.fused.keys_full_off);
  uint2* keys_list = reinterpret_cast<uint2*>(wsb + ws.fused.keys_list_off);
  if (causal) {
    // The key rows in list order come with the prefix lists.
    const hipError_t e = launch_prefix_lists(sorted_codes, perm, S, N, tile_bwd_list_topk(N, topk), workspace, stream, &list_codes,
                                             &list_pos, static_cast<const uint16_t*>(k), keys_full, keys_list);
    if (e != hipSuccess) return e;
  }
  hipError_t e = launch_tile_windows(k, S, N, dk_, topk, causal, chunk, q_codes, sorted_codes, perm, list_codes,
                                     list_pos, q_order, nullptr, bounds, keys_full, keys_list, list_codes != nullptr,
                                     stream, tile_bwd_list_topk(N, topk));
  if (e != hipSuccess) return e;
  const uint16_t* qq = static_cast<const uint16_t*>(q);
  const uint16_t* vv = static_cast<const uint16_t*>(v);
  const uint16_t* dd = static_cast<const uint16_t*>(dout);
#define ZETA_TILE_BWD_CASE(DVV)                                                                                      \
  case DVV:                                                                                                          \
    return launch_tile_bwd_t<DVV>(qq, vv, dd, S, N, topk, causal, chunk, perm, list_pos, q_order, bounds, keys_full, \
                                  keys_list, eps, hm, dq, dk, dv, deps, ws, wsb, stream);
  switch (dv_) {
    ZETA_TILE_BWD_CASE(32)
    ZETA_TILE_BWD_CASE(64)
    ZETA_TILE_BWD_CASE(128)
    ZETA_TILE_BWD_CASE(256)
    default:
      return hipErrorInvalidValue;
  }
#undef ZETA_TILE_BWD_CASE
}

}  // namespace zeta
