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
  __device__ static T fold(T acc, T) { return acc; }
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

// Group-wide helpers over G lanes: the whole wave (G = 64), one of its
// aligned halves (G = 32) or rows (G = 16); exchanges stay inside the group.
// Inclusive scan with op by DPP: shifts by 1, 2, 4, 8 inside each 16-lane
// row, then the last lane of row 0 (2) is added into row 1 (3), and for
// G = 64 lane 31 into rows 2 and 3.  Lanes without a source receive ident.
template <int G, class Op>
__device__ __forceinline__ int group_scan(int v, int ident, Op op) {
  static_assert(G == 16 || G == 32 || G == 64, "groups of 16, 32 or 64 lanes");
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x111, 0xF, 0xF, false));  // row_shr:1
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x112, 0xF, 0xF, false));  // row_shr:2
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x114, 0xF, 0xF, false));  // row_shr:4
  v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x118, 0xF, 0xF, false));  // row_shr:8
  if constexpr (G >= 32) v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x142, 0xA, 0xF, false));  // row_bcast:15
  if constexpr (G == 64) v = op(v, __builtin_amdgcn_update_dpp(ident, v, 0x143, 0xC, 0xF, false));  // row_bcast:31
  return v;
}

// Merge steps of a sort over G lanes, one key per lane.  side[i] is all ones
// in lanes with bit i set: such a lane keeps the larger key of its pair, the
// others the smaller, which is the median of the pair and side[i] (one
// instruction for 32-bit keys).
struct LaneSides {
  uint32_t side[6];
  __device__ __forceinline__ LaneSides() {
    const int lane = lane_id();
#pragma unroll
    for (int i = 0; i < 6; ++i) side[i] = (lane >> i) & 1 ? ~0u : 0u;
  }
};
__device__ __forceinline__ uint32_t pair_key(uint32_t a, uint32_t b, uint32_t side) {
  const uint32_t mn = a < b ? a : b, mx = a < b ? b : a;
  const uint32_t c = mx < side ? mx : side;
  return mn > c ? mn : c;
}
__device__ __forceinline__ uint64_t pair_key(uint64_t a, uint64_t b, uint32_t side) {
  return (a < b) == (side == 0) ? a : b;
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint32_t dpp_key(uint32_t v) {
  if constexpr (ROWS == 0xF) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS = 0xF>
__device__ __forceinline__ uint64_t dpp_key(uint64_t v) {
  return ((uint64_t)dpp_key<CTRL, ROWS>((uint32_t)(v >> 32)) << 32) | dpp_key<CTRL, ROWS>((uint32_t)v);
}
// Step at distance 16 (32): after the swap of a key with itself both lanes of a
// pair hold the two keys, in the same order.
template <int J>
__device__ __forceinline__ uint32_t far_step(uint32_t v, uint32_t side) {
  if constexpr (J == 16) {
    const auto s = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return pair_key((uint32_t)s[0], (uint32_t)s[1], side);
  } else {
    const auto s = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return pair_key((uint32_t)s[0], (uint32_t)s[1], side);
  }
}
template <int J>
__device__ __forceinline__ uint64_t far_step(uint64_t v, uint32_t side) {
  return pair_key(v, xor_lane(v, J), side);
}
template <int TOP, typename K>  // steps at distances TOP, .., 2, 1 (TOP <= 8)
__device__ __forceinline__ K near_steps(K key, const LaneSides& L) {
  if constexpr (TOP >= 8) key = pair_key(key, dpp_key<0x128>(key), L.side[3]);               // row_ror:8
  if constexpr (TOP >= 4) key = pair_key(key, dpp_key<0x1B>(dpp_key<0x141>(key)), L.side[2]);  // xor 7, xor 3
  if constexpr (TOP >= 2) key = pair_key(key, dpp_key<0x4E>(key), L.side[1]);
  return pair_key(key, dpp_key<0xB1>(key), L.side[0]);
}

// Ascending sort of G keys, one per lane, of which every aligned run of
// `sorted` lanes (a power of two, the same in every lane) is ascending already.
// Two ascending runs are merged by pairing lane i with lane k - 1 - i of their
// 2^x = k lanes, then at distances k/4, .., 1: up to 16 lanes that pairing is
// one DPP mirror.  For 32 lanes the odd row is mirrored and left so (its half of the
// merge is bitonic either way); for 64 the upper half is sorted descending
// (complemented) instead.
template <int G, typename K>
__device__ __forceinline__ K sort_runs(K key, int sorted, const LaneSides& L) {
  if (sorted < 2) key = near_steps<1>(key, L);
  if (sorted < 4) {
    key = pair_key(key, dpp_key<0x1B>(key), L.side[1]);
    key = near_steps<1>(key, L);
  }
  if (sorted < 8) {
    key = pair_key(key, dpp_key<0x141>(key), L.side[2]);
    key = near_steps<2>(key, L);
  }
  if (sorted < 16) {
    key = pair_key(key, dpp_key<0x140>(key), L.side[3]);
    key = near_steps<4>(key, L);
  }
  if constexpr (G >= 32) {
    if (sorted < G) {
      const K flip = (K)(int64_t)(int32_t)L.side[5];
      if constexpr (G == 64) key ^= flip;
      key = far_step<16>(dpp_key<0x140, 0xA>(key), L.side[4]);
      key = near_steps<8>(key, L);
      if constexpr (G == 64) {
        key ^= flip;
        key = far_step<32>(key, L.side[5]);
        key = far_step<16>(key, L.side[4]);
        key = near_steps<8>(key, L);
      }
    }
  }
  return key;
}

// Whether this lane's bit is set in a mask that is the same in every lane.
__device__ __forceinline__ bool lane_of_mask(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

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
