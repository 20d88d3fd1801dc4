// Device helpers of the SpGEMM kernels: where an output column's products
// come from, and lane-group primitives of the one-wave paths.
#pragma once

#include "common.h"
#include "operand.h"

namespace spx {

// Semiring for the boolean (pattern only) case; values are never touched.
template <typename T>
struct Semiring<SPX_OR_AND, T> {
  static constexpr bool kUsesA = false, kUsesB = false;
  __device__ static T mul(T a, T) { return a; }
  __device__ static T add(T acc, T) { return acc; }
  __device__ static T ident() { return T(0); }
  __device__ static void lds_acc(T*, T) {}
};

__device__ __forceinline__ int floor_log2_u64(uint64_t x) { return 63 - __clzll(x); }
__device__ __forceinline__ int ceil_log2_u64(uint64_t x) { return x <= 1 ? 0 : 64 - __clzll(x - 1); }

// Where the products of one output column come from.  For every stored
// B(k,j) (index q): the start and length of A(:,k), and for long columns of
// A a row of the split table, whose entry b is the first position in A(:,k)
// with row >= b * 2^rbshift (b = 0..nblk; the last entry is the length).
// Parts of the row space start and end on those block boundaries, so a
// part's range inside a long column costs two loads; short columns are
// filtered entry by entry.
struct ProdSrc {
  const int32_t* air;
  const int64_t* a0;
  const int32_t* alen;
  const int32_t* split;
  const int32_t* splits;
  int32_t sstride;
  int32_t rbshift;
  int32_t m;
  int32_t off32;   // 1: positions in A fit 29 bits, loads take 32-bit byte offsets
  int32_t qchunk;  // B entries per set-up round of the block-cooperative iteration
};

// A value known to be the same in every lane, moved to scalar registers (values
// read from LDS or memory otherwise stay in vector registers).
__device__ __forceinline__ int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uniform(int64_t v) {
  return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(v >> 32)) << 32) |
                   (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)v));
}

__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Group-wide helpers over G lanes: the whole wave (G = 64) or one of its
// aligned halves (G = 32); exchanges stay inside the group.
// Inclusive scan with op by DPP: shifts by 1, 2, 4, 8 inside each 16-lane
// row, then the last lane of row 0 (2) is added into row 1 (3), and for
// G = 64 lane 31 into rows 2 and 3.  Lanes without a source receive ident.
template <int G, class Op>
__device__ __forceinline__ int group_scan(int v, int ident, Op op) {
  static_assert(G == 32 || G == 64, "groups of 32 or 64 lanes");
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x111, 0xF, 0xF, false));  // row_shr:1
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x112, 0xF, 0xF, false));  // row_shr:2
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x114, 0xF, 0xF, false));  // row_shr:4
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x118, 0xF, 0xF, false));  // row_shr:8
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
  if constexpr (G == 64) v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return v;
}

// Value of the next lane (lane + 1; 0 in lane 63) by a DPP wave shift.
template <typename T>
__device__ __forceinline__ T lane_next(T v) {
  if constexpr (sizeof(T) == 4) {
    const int u = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(0, u, 0x130, 0xF, 0xF, false));  // wave_shl:1
  } else {
    static_assert(sizeof(T) == 8, "32- or 64-bit values");
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, 0x130, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), 0x130, 0xF, 0xF, false);
    return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
  }
}

// Ascending bitonic sort of 64 * R keys, key lane * R + r in register r.
// Exchanges at distances below R stay in the lane.  Phases whose direction
// depends on the lane complement the keys of descending lanes instead of
// selecting, so every in-lane exchange is one minimum and one maximum.
template <int R, typename K>
__device__ __forceinline__ void sort_regs(K (&key)[R], int lane) {
#pragma unroll
  for (int k = 2; k <= kWave * R; k <<= 1) {
    const K flip = k >= R && k < kWave * R && (lane & (k / R)) ? ~K(0) : K(0);
    if (k >= R) {
#pragma unroll
      for (int r = 0; r < R; ++r) key[r] ^= flip;
    }
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j < R) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if (r & j) continue;
          const bool up = k >= R || (r & k) == 0;
          const K x = key[r], y = key[r | j];
          const K mn = x < y ? x : y, mx = x < y ? y : x;
          key[r] = up ? mn : mx;
          key[r | j] = up ? mx : mn;
        }
      } else {
        const bool lower = (lane & (j / R)) == 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const K x = key[r], y = xor_lane(x, j / R);
          const K mn = x < y ? x : y, mx = x < y ? y : x;
          key[r] = lower ? mn : mx;
        }
      }
    }
    if (k >= R) {
#pragma unroll
      for (int r = 0; r < R; ++r) key[r] ^= flip;
    }
  }
}

}  // namespace spx
