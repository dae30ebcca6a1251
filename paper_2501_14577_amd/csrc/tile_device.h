// Matrix-core operand types and wavefront helpers shared by the bfloat16
// tile kernels (the one-pass attention and its gradients).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace zeta {

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

union Frag {  // four bfloat16 values
  uint32_t w[2];
  s16x4_t v;
};

union Frag8 {  // eight bfloat16 values
  uint32_t w[4];
  bf16x8_t v;
};

// Minimum / maximum over the wavefront, read by every lane: within each row
// of 16 lanes by four DPP exchanges (swap neighbours, swap pairs, mirror the
// half row, mirror the row), then rows 1 and 3 take row 0's and row 2's
// result (row_bcast:15) and rows 2 and 3 take lane 31's (row_bcast:31), so
// lane 63 holds the wavefront's result.  No LDS round trip (unlike a
// shuffle through ds_bpermute).
template <bool kMax>
__device__ __forceinline__ int wave_reduce_minmax(int x) {
  auto op = [](int a, int b) { return kMax ? (a > b ? a : b) : (a < b ? a : b); };
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x140, 0xF, 0xF, false));  // row_mirror
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x142, 0xA, 0xF, false));  // row_bcast:15 into rows 1, 3
  x = op(x, __builtin_amdgcn_update_dpp(x, x, 0x143, 0xC, 0xF, false));  // row_bcast:31 into rows 2, 3
  return __builtin_amdgcn_readlane(x, 63);
}

__device__ __forceinline__ int wave_min_int(int x) { return wave_reduce_minmax<false>(x); }

__device__ __forceinline__ int wave_max_int(int x) { return wave_reduce_minmax<true>(x); }

// Lane `src`'s value of a pointer, read by every lane.  Each 32-bit half goes
// through uint32_t: widening a negative int32 would sign-extend into the
// high half.
template <typename T>
__device__ __forceinline__ T* readlane_ptr(T* p, int src) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int32_t(uint32_t(v)), src));
  const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int32_t(uint32_t(v >> 32)), src));
  // Rebuilt as a global-memory pointer, so that loads through it are global
  // loads rather than flat ones.
  using G = __attribute__((address_space(1))) T;
  G* g = (G*)((uint64_t(hi) << 32) | uint64_t(lo));
  return (T*)g;
}

constexpr int kChunk = 16;  // rows (list entries, or a tile's queries) per product step

// Value rows reach the matrix cores through LDS.  Per chunk of 16 entries the
// wavefront copies the 16 value rows straight from global memory into LDS
// (global_load_lds_dwordx4: lane L's 16 bytes land at byte 16 L of the
// instruction's 1 KiB), then reads each product's A operand with one
// transposing LDS read (ds_read_b64_tr_b16: within each group of 16 lanes,
// output lane i receives element i % 4 of the 8-byte reads of lanes
// 4j + i / 4, j = 0..3).  With lane (g, s) of a group pointing at entry row
// 4g + s / 4, columns 16 blk + 4 (s % 4) .. + 3, output lane i holds column
// 16 blk + i of entries 4g .. 4g + 3: the A operand (value columns x
// entries) of a 16 x 16 x 16 product, with no register shuffling (the kernel
// repeats it in the upper K half of a 16 x 16 x 32 product, against the low
// score parts).
//
// LDS row order.  One copy instruction fills R = 512 / d_v consecutive LDS
// rows (P = d_v / 8 pieces of 16 bytes each).  For d_v <= 128 the lanes that
// fill one LDS row share a tile-entry group kg, so each lane copies one of its
// own 4 entries (whose position it already holds): LDS row
// rho = j R + q (instruction j, q = lane / P) holds entry
// 4 kg + j (16 / P) + q % (16 / P).  For d_v = 256 row rho holds entry rho.
// Pieces are XOR-swizzled by row (sw below): physical piece p of row rho
// holds logical piece p ^ sw(rho), so that the transposing reads are free of
// bank conflicts.
// Transposing LDS reads (ds_read_b64_tr_b16) at addr[j] + kOff, kCopies of
// each (into a[kCopies j] .. a[kCopies j + kCopies - 1]), issued once the
// copies into LDS made before the last kPending copy instructions have landed
// (kPending -1: no wait here); read_tr_wait then waits for the results.
// Written as inline assembly, with the waits, because the compiler would
// otherwise wait for every copy still in flight (including the next chunk's,
// which must keep loading meanwhile) before any such read.  LDS operations of
// one wavefront complete in order, so the compiler's own waits on its later
// LDS reads stay correct with these older ones in flight.
template <int E, int kCopies, uint32_t kOff, int kPending>
__device__ __forceinline__ void read_tr_issue(const uint32_t (&addr)[E], s16x4_t (&a)[E * kCopies]) {
  static_assert(kPending >= -1 && kPending < 16, "vmcnt immediate (-1: no wait)");
  if constexpr (kPending >= 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPending) : "memory");
#pragma unroll
  for (int j = 0; j < E; ++j)
#pragma unroll
    for (int c = 0; c < kCopies; ++c)
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2"
                   : "=v"(a[kCopies * j + c])
                   : "v"(addr[j]), "n"(kOff)
                   : "memory");
}

// Waits for every LDS read of this wavefront; the reads' results are then
// used only after the wait (each passes through an ordered empty statement).
template <int N>
__device__ __forceinline__ void read_tr_wait(s16x4_t (&a)[N]) {
  asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a[0])::"memory");
#pragma unroll
  for (int j = 1; j < N; ++j) asm volatile("" : "+v"(a[j]));
}

template <int DV>
struct VStage {
  static constexpr int kRowBytes = 2 * DV;
  static constexpr int kP = DV / 8;                   // 16-byte pieces per row
  static constexpr int kR = 64 / kP;                  // LDS rows per copy instruction
  static constexpr int kLoads = kChunk / kR;          // copy instructions per chunk
  static constexpr int kOwn = kP <= 16 ? 16 / kP : 0; // rows of one entry group per instruction
  static constexpr int kBlocks = DV / 16;             // products (16 value columns each) per chunk
  static constexpr int kBytes = kChunk * kRowBytes;   // one chunk's rows
  static_assert(kR >= 2 && kChunk % kR == 0, "d_v must be 32, 64, 128 or 256");
  // Piece swizzle of LDS row rho.  A transposing read is served in two
  // halves of 32 lanes (entry groups kg = 0, 1 and kg = 2, 3), each reading
  // 256 bytes: the 16 (row, piece) pairs of one half must fall in 16
  // different 16-byte bank groups.  Row rho's bank group is set by the row's
  // offset within 256 bytes and the physical piece; the swizzle puts the
  // row bits that the offset does not separate into the piece bits that the
  // block index leaves free.
  __device__ static constexpr int sw(int rho) {
    if constexpr (kP == 16) {  // rho = 4u + kg: u into piece bits 2-3, kg's low bit into bit 1
      return (rho & 12) | ((rho & 1) << 1);
    } else if constexpr (kP == 8) {  // rho = 8(u >> 1) + 2kg + (u & 1)
      return (((rho >> 1) & 1) << 1) | (((rho >> 3) & 1) << 2);
    } else if constexpr (kP == 4) {  // rho = 4kg + u
      return ((rho >> 2) & 1) << 1;
    } else {  // kP == 32, rho = 4kg + u
      return ((rho & 3) << 1) | (((rho >> 2) & 1) << 3);
    }
  }
  // Chunk entry held by LDS row rho.
  __device__ static constexpr int entry_of_row(int rho) {
    if constexpr (kP > 16) {
      return rho;
    } else {
      const int j = rho / kR, q = rho % kR;
      return 4 * (q / kOwn) + j * kOwn + q % kOwn;
    }
  }
  // LDS row holding chunk entry e.
  __device__ static constexpr int row_of_entry(int e) {
    if constexpr (kP > 16) {
      return e;
    } else {
      const int kg = e / 4, u = e % 4;
      return (u / kOwn) * kR + kg * kOwn + u % kOwn;
    }
  }
};

// N pieces of 16 bytes from LDS at addr[i] + kOff, waited for in the same
// statement (after the vector-memory wait, when kPending >= 0: all but the last
// kPending copy instructions have landed).  Inline assembly for the same reason
// as read_tr_issue: the compiler would wait for every copy still in flight.
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

template <uint32_t kOff, int kPending>
__device__ __forceinline__ void read_rows16(const uint32_t (&addr)[1], u32x4_t (&o)[1]) {
  if constexpr (kPending >= 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPending) : "memory");
  asm volatile(
      "ds_read_b128 %0, %1 offset:%2\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(o[0])
      : "v"(addr[0]), "n"(kOff)
      : "memory");
}

template <uint32_t kOff, int kPending>
__device__ __forceinline__ void read_rows16(const uint32_t (&addr)[2], u32x4_t (&o)[2]) {
  if constexpr (kPending >= 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPending) : "memory");
  asm volatile(
      "ds_read_b128 %0, %2 offset:%4\n\t"
      "ds_read_b128 %1, %3 offset:%4\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(o[0]), "=&v"(o[1])
      : "v"(addr[0]), "v"(addr[1]), "n"(kOff)
      : "memory");
}

template <uint32_t kOff, int kPending>
__device__ __forceinline__ void read_rows16(const uint32_t (&addr)[4], u32x4_t (&o)[4]) {
  if constexpr (kPending >= 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kPending) : "memory");
  asm volatile(
      "ds_read_b128 %0, %4 offset:%8\n\t"
      "ds_read_b128 %1, %5 offset:%8\n\t"
      "ds_read_b128 %2, %6 offset:%8\n\t"
      "ds_read_b128 %3, %7 offset:%8\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3])
      : "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3]), "n"(kOff)
      : "memory");
}

template <uint32_t kOff, int kPending>
__device__ __forceinline__ void read_rows16(const uint32_t (&addr)[8], u32x4_t (&o)[8]) {
  const uint32_t a0[4] = {addr[0], addr[1], addr[2], addr[3]}, a1[4] = {addr[4], addr[5], addr[6], addr[7]};
  u32x4_t o0[4], o1[4];
  read_rows16<kOff, kPending>(a0, o0);
  read_rows16<kOff, -1>(a1, o1);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    o[i] = o0[i];
    o[4 + i] = o1[i];
  }
}

}  // namespace zeta
