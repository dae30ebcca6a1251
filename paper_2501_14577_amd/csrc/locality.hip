// The locality experiment of Section 4.4: how many of a query's kn nearest
// keys in Euclidean distance its Z-order window of kn keys also holds.
//
//   The squared distance to every key of the query's pool is computed in
//     float32 (one rounding per subtraction, product and sum, axes in order:
//     no fused multiply-add, so that ties and near-ties are decided as a plain
//     float32 evaluation decides them); non-negative floats order as their
//     bits.  The answer is ordered by (distance, position); a pool smaller
//     than kn is padded with -1.
//   knn_wave (kn <= 64): one wavefront per query, a lane holding the distances
//     of keys lane, lane + 64, ... in registers.  The largest of the lanes'
//     smallest distances bounds the kn-th smallest (64 lanes hold at least 64
//     distances up to it), which leaves about 15% of 2048 keys; those are
//     compacted into LDS, the kn-th smallest is found by bisection on the bits
//     (about 10 counts: it ends as soon as exactly kn distances lie below),
//     and one 64-lane bitonic sort orders them.
//   exact_knn (kn > 64, where that bound does not hold, and a few hundred
//     queries over at most 256 keys): one workgroup per query packs (distance,
//     position) into 64-bit words and sorts up to 4096 of them in LDS by a
//     bitonic network.
//   index_overlap: one wavefront per row marks row b's entries in an LDS
//     bit set of the segment's positions, counts row a's marked entries, and
//     clears its marks again.
// Both are small experiments (N up to 4096 keys per query for the exact
// search), not part of the attention's hot path.
#include "attend_device.h"
#include "device_common.h"
#include "kernels.h"
#include "layout.h"
#include "tile_device.h"

namespace zeta {
namespace {

constexpr int kKnnThreads = 256;
constexpr int kOvWaves = 4;

// Squared distance of a query to key row kr, in float32 with one rounding
// per subtraction, product and sum, axes in order (no contraction into
// fused multiply-adds).
template <typename T, int KD>
__device__ __forceinline__ float plain_d2(const float* qv, const T* __restrict__ kr, int dk) {
#pragma clang fp contract(off)
  float d2 = 0.0f;
#pragma unroll
  for (int a = 0; a < KD; ++a) {
    if (a < dk) {
      const float diff = qv[a] - Elem<T>::load(kr + a);
      d2 = d2 + diff * diff;
    }
  }
  return d2;
}

template <typename T, int DK>
__global__ void __launch_bounds__(kKnnThreads)
    exact_knn_kernel(const T* __restrict__ q, const T* __restrict__ k, int64_t N, int dk_rt, int kn, int causal,
                     int P, int32_t* __restrict__ out) {
  constexpr int KD = DK > 0 ? DK : kMaxDk;
  const int dk = DK > 0 ? DK : dk_rt;
  __shared__ uint64_t s_key[kKnnMaxN];
  const int64_t row = blockIdx.x;  // segment * N + query position
  const int64_t seg = row / N;
  const int64_t i = row - seg * N;
  const int64_t end = causal ? i + 1 : N;  // pool: keys 0 .. end - 1
  float qv[KD];
#pragma unroll
  for (int a = 0; a < KD; ++a) qv[a] = a < dk ? Elem<T>::load(q + row * dk + a) : 0.0f;
  const T* kseg = k + seg * N * dk;
  for (int j = threadIdx.x; j < P; j += kKnnThreads) {
    uint64_t key = ~uint64_t(0);
    if (j < end) {
      const float d2 = plain_d2<T, KD>(qv, kseg + int64_t(j) * dk, dk);
      key = (uint64_t(__float_as_uint(d2)) << 32) | uint32_t(j);
    }
    s_key[j] = key;
  }
  __syncthreads();
  // Bitonic sort of the P words, ascending.
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      for (int t = threadIdx.x; t < P; t += kKnnThreads) {
        const int u = t ^ stride;
        if (u > t) {
          const uint64_t x = s_key[t], y = s_key[u];
          const bool up = (t & size) == 0;
          if ((x > y) == up) {
            s_key[t] = y;
            s_key[u] = x;
          }
        }
      }
      __syncthreads();
    }
  }
  const int64_t m = end < kn ? end : kn;
  for (int c = threadIdx.x; c < kn; c += kKnnThreads)
    out[row * kn + c] = c < m ? int32_t(uint32_t(s_key[c] & 0xFFFFFFFFu)) : -1;
}

// ---- kn <= 64: one wavefront per query ------------------------------------------
constexpr int kKnnWaves = 4;       // queries per block
constexpr int kKnnCand = 512;      // candidates kept in LDS
constexpr int kKnnMaxWave = 64;    // largest kn
constexpr int kKnnNone = 0x7FFFFFFF;  // no key (above every distance's bits)

// The first `take` of the NR x 64 values (d[r] of lane l is element 64 r + l;
// kKnnNone where there is none) in (value, element) order, element order kept:
// calls put(slot, r) on the lanes that hold them.  At least `take` values are
// <= hi and none is below lo.
template <int NR, typename Put>
__device__ __forceinline__ void knn_select(const int (&d)[NR], int take, int lo, int hi, Put&& put) {
  auto count = [&](int t) -> int {  // values <= t
    int c = 0;
#pragma unroll
    for (int r = 0; r < NR; ++r) c += __popcll(wave_ballot(d[r] <= t));
    return c;
  };
  bool whole = false;  // exactly `take` values are <= hi
  while (lo < hi) {
    const int mid = lo + ((hi - lo) >> 1);
    const int c = count(mid);
    if (c < take) {
      lo = mid + 1;
    } else {
      hi = mid;
      if (c == take) {
        whole = true;
        break;
      }
    }
  }
  // Below hi all are taken, of those at hi the first ones.
  int ties = whole ? take : take - (hi > 0 ? count(hi - 1) : 0);
  int at = 0;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const uint64_t eq = wave_ballot(d[r] == hi);
    const bool sel = d[r] < hi || (d[r] == hi && int(lanes_below(eq)) < ties);
    const uint64_t m = wave_ballot(sel);
    if (sel) put(at + int(lanes_below(m)), r);
    ties -= __popcll(eq);
    at += __popcll(m);
  }
}

// Bound: half vector issue (per query and 64 keys about 10 instructions for the
// distances, 6 for the bound and the compaction, then about 500: 54 us of the 110
// below), half the key loads' latency at the 3 wavefronts per SIMD that the
// registers of 32 keys a lane leave.  2048 keys, kn 64, 16 segments: 110 us, against
// 2340 us with the workgroup sort above.
template <typename T, int DK, int M>
__global__ void __launch_bounds__(kKnnWaves * 64)
    knn_wave_kernel(const T* __restrict__ q, const T* __restrict__ k, int64_t rows, int64_t N, int dk_rt, int kn,
                    int causal, int32_t* __restrict__ out) {
  constexpr int KD = DK > 0 ? DK : kMaxDk;
  const int dk = DK > 0 ? DK : dk_rt;
  __shared__ int s_d[kKnnWaves][kKnnCand];
  __shared__ int s_j[kKnnWaves][kKnnCand];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
  const int64_t row = int64_t(blockIdx.x) * kKnnWaves + wave;  // segment * N + query position
  if (row >= rows) return;
  const int64_t seg = row / N;
  const int end = causal ? int(row - seg * N) + 1 : int(N);  // pool: keys 0 .. end - 1
  float qv[KD];
#pragma unroll
  for (int a = 0; a < KD; ++a) qv[a] = a < dk ? Elem<T>::load(q + row * dk + a) : 0.0f;
  const T* kseg = k + seg * N * dk;
  int d[M];
  int least = kKnnNone;
#pragma unroll
  for (int r = 0; r < M; ++r) {
    const int j = r * 64 + lane;
    const int jc = j < end ? j : end - 1;
    // A NaN, of either sign, is above infinity and below "no key".
    const uint32_t bits = __float_as_uint(plain_d2<T, KD>(qv, kseg + int64_t(jc) * dk, dk));
    d[r] = int(bits < uint32_t(kKnnNone) ? bits : uint32_t(kKnnNone) - 1u);
  }
#pragma unroll
  for (int r = 0; r < M; ++r) {
    d[r] = r * 64 + lane < end ? d[r] : kKnnNone;
    least = d[r] < least ? d[r] : least;
  }
  const int take = end < kn ? end : kn;
  const int lo = wave_min_int(least);
  int hi = wave_max_int(least);
  if (hi == kKnnNone) hi = kKnnNone - 1;  // a lane without keys: every key is a candidate
  int n = 0;
#pragma unroll
  for (int r = 0; r < M; ++r) n += __popcll(wave_ballot(d[r] <= hi));
  int my_d = kKnnNone, my_j = -1;  // the lane's key among those taken
  if (n <= kKnnCand) {
    int at = 0;
#pragma unroll
    for (int r = 0; r < M; ++r) {
      const bool in = d[r] <= hi;
      const uint64_t m = wave_ballot(in);
      if (in) {
        const int slot = at + int(lanes_below(m));
        s_d[wave][slot] = d[r];
        s_j[wave][slot] = r * 64 + lane;
      }
      at += __popcll(m);
    }
    wave_lds_sync();
    constexpr int NC = kKnnCand / 64;
    int cd[NC], cj[NC];
#pragma unroll
    for (int r = 0; r < NC; ++r) {
      const bool in = r * 64 + lane < n;
      cd[r] = in ? s_d[wave][r * 64 + lane] : kKnnNone;
      cj[r] = in ? s_j[wave][r * 64 + lane] : -1;
    }
    wave_lds_sync();
    knn_select<NC>(cd, take, lo, hi, [&](int slot, int r) {
      s_d[wave][slot] = cd[r];
      s_j[wave][slot] = cj[r];
    });
  } else {
    knn_select<M>(d, take, lo, hi, [&](int slot, int r) {
      s_d[wave][slot] = d[r];
      s_j[wave][slot] = r * 64 + lane;
    });
  }
  wave_lds_sync();
  if (lane < take) {
    my_d = s_d[wave][lane];
    my_j = s_j[wave][lane];
  }
  // Bitonic sort of the 64 lanes' (distance, position), ascending; lanes
  // without a key (kKnnNone) end last.
#pragma unroll
  for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const int od = __shfl_xor(my_d, stride, 64), oj = __shfl_xor(my_j, stride, 64);
      const bool less = od < my_d || (od == my_d && uint32_t(oj) < uint32_t(my_j));
      const bool lower = (lane & stride) == 0, up = (lane & size) == 0;
      const bool other = less == (lower == up) && (od != my_d || oj != my_j);
      my_d = other ? od : my_d;
      my_j = other ? oj : my_j;
    }
  }
  if (lane < kn) out[row * kn + lane] = my_j;
}

__global__ void __launch_bounds__(kOvWaves * 64)
    index_overlap_kernel(const int32_t* __restrict__ a, int ka, const int32_t* __restrict__ b, int kb, int64_t rows,
                         int64_t N, int32_t* __restrict__ counts) {
  __shared__ uint32_t s_bits[kOvWaves][kOverlapMaxN / 32];
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int words = int((N + 31) / 32);
  for (int w = lane; w < words; w += 64) s_bits[wave][w] = 0u;
  wave_lds_sync();
  for (int64_t r = int64_t(blockIdx.x) * kOvWaves + wave; r < rows; r += int64_t(gridDim.x) * kOvWaves) {
    const int32_t* br = b + r * kb;
    const int32_t* ar = a + r * ka;
    for (int c = lane; c < kb; c += 64) {
      const int32_t j = br[c];
      if (j >= 0 && j < N) atomicOr(&s_bits[wave][j >> 5], 1u << (j & 31));
    }
    wave_lds_sync();
    int cnt = 0;
    for (int c = lane; c < ka; c += 64) {
      const int32_t j = ar[c];
      if (j >= 0 && j < N && ((s_bits[wave][j >> 5] >> (j & 31)) & 1u) != 0u) ++cnt;
    }
    cnt = int(wave_sum(float(cnt)));
    if (lane == 0) counts[r] = cnt;
    wave_lds_sync();
    for (int c = lane; c < kb; c += 64) {
      const int32_t j = br[c];
      if (j >= 0 && j < N) atomicAnd(&s_bits[wave][j >> 5], ~(1u << (j & 31)));
    }
    wave_lds_sync();
  }
}

template <typename T, int DK>
hipError_t knn_wave_t(const T* q, const T* k, int64_t S, int64_t N, int dk, int kn, int causal, int32_t* out,
                      hipStream_t stream) {
  const int64_t rows = S * N;
  const dim3 grid(unsigned(ceil_div(rows, int64_t(kKnnWaves)))), block(kKnnWaves * 64);
#define ZETA_KNN_WAVE(M) \
  hipLaunchKernelGGL((knn_wave_kernel<T, DK, M>), grid, block, 0, stream, q, k, rows, N, dk, kn, causal, out)
  // Every lane loads M keys, whether it holds them or not (a segment of 64 keys, d_k
  // 8: 12.6 us with M = 8, 8.0 with 1).
  if (N <= 64)
    ZETA_KNN_WAVE(1);
  else if (N <= 256)
    ZETA_KNN_WAVE(4);
  else if (N <= 512)
    ZETA_KNN_WAVE(8);
  else if (N <= 1024)
    ZETA_KNN_WAVE(16);
  else if (N <= 2048)
    ZETA_KNN_WAVE(32);
  else
    ZETA_KNN_WAVE(64);
#undef ZETA_KNN_WAVE
  return hipGetLastError();
}

template <typename T>
hipError_t knn_t(const void* q, const void* k, int64_t S, int64_t N, int dk, int kn, bool causal, int32_t* out,
                 hipStream_t stream) {
  static_assert(kKnnMaxN <= 64 * 64, "a lane of knn_wave holds up to 64 distances");
  const T* qq = static_cast<const T*>(q);
  const T* kk = static_cast<const T*>(k);
  // Few queries over few keys leave the chip idle, and a workgroup has its query
  // done sooner: 8.0 us against 8.7-9.8 for 4 segments of 100 keys, 8.6 against up to
  // 9.5 for 5 of 128; 3 of 256 take 9.7-12.5 against 8.3-9.6.
  const bool idle = N <= 256 && S * N <= 640;
  if (kn <= kKnnMaxWave && !idle) {
    if (dk == 3) return knn_wave_t<T, 3>(qq, kk, S, N, dk, kn, causal ? 1 : 0, out, stream);
    return knn_wave_t<T, 0>(qq, kk, S, N, dk, kn, causal ? 1 : 0, out, stream);
  }
  int P = 1;
  while (P < N) P <<= 1;
  const dim3 grid(unsigned(S * N)), block(kKnnThreads);
  if (dk == 3)
    hipLaunchKernelGGL((exact_knn_kernel<T, 3>), grid, block, 0, stream, qq, kk, N, dk, kn, causal ? 1 : 0, P, out);
  else
    hipLaunchKernelGGL((exact_knn_kernel<T, 0>), grid, block, 0, stream, qq, kk, N, dk, kn, causal ? 1 : 0, P, out);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_exact_knn(const void* q, const void* k, bool is_bf16, int64_t S, int64_t N, int dk, int kn,
                            bool causal, int32_t* out, hipStream_t stream) {
  if (is_bf16) return knn_t<uint16_t>(q, k, S, N, dk, kn, causal, out, stream);
  return knn_t<float>(q, k, S, N, dk, kn, causal, out, stream);
}

hipError_t launch_index_overlap(const int32_t* a, int ka, const int32_t* b, int kb, int64_t rows, int64_t N,
                                int32_t* counts, hipStream_t stream) {
  const int64_t want = ceil_div(rows, kOvWaves);
  const unsigned blocks = unsigned(want < 4096 ? want : 4096);
  hipLaunchKernelGGL(index_overlap_kernel, dim3(blocks), dim3(kOvWaves * 64), 0, stream, a, ka, b, kb, rows, N,
                     counts);
  return hipGetLastError();
}

}  // namespace zeta
