// SpGEMM C = A*B over a semiring on one gfx950 GPU.
//
// What is computed is the column-wise product of Section 3 (Algorithm 1):
// column j of C is the semiring sum, over the nonzeros B(k,j), of
// A(:,k) "times" B(k,j).  The paper's local kernel (HyperSparseGEMM, an
// outer product merged through a priority queue, Section 3.1) is prior art
// for a serial CPU; here every output column is formed independently by a
// wave or a workgroup, and the only property kept from the paper's kernel
// is that no pass is proportional to a matrix dimension when the operands
// are hypersparse (DCSC operands are iterated over their nonempty columns;
// the column lookup into a DCSC A uses the AUX index of Section 3.2).
//
// Two phases.
//   plan (symbolic): per-entry lookup of A's columns, per-column number of
//     multiplications, binning of the columns by that count, exact output
//     counts (a sort in registers for tiny columns (lane groups), an LDS hash
//     for mid ones (a wave's table) and medium ones (a workgroup's), an LDS
//     bitmap over the row space for heavy ones, which also yields per-row-block
//     counts), int64 scan into column pointers, and a list of row-range "parts"
//     (each fits one workgroup's LDS) for the numeric phase.
//   exec (numeric): tiny and mid columns are sorted with their values and
//     written; every part is accumulated in LDS either through a bitmap
//     over its row range (rank of a row = popcount prefix, which also yields
//     sorted output) or through a hash table, whose rows a two-level bitmap
//     ranks (above 2^20 rows an LDS sort orders them).
#include <algorithm>
#include <cstring>
#include <memory>
#include <type_traits>

#include "common.h"
#include "mid.h"
#include "operand.h"
#include "plan.h"
#include "scan.h"
#include "wave.h"

namespace spx {

// ------------------------------------------------------------------ bins
// Columns (slots of B) are binned by their number of multiplications mu.
// The bin id is also the processing order: heavy columns first.
//   0 .. 40   bitmap-counted columns, id = 40 - floor(log2 mu)
//   41 .. 48  hash-counted columns, table of 2^(15 - (id - 41)) keys; the last
//             three (at most kMidMax products) are mid columns, one wave each
//   49        tiny columns (mu <= tiny_max, at most 64): groups of 16 to 64 lanes
//   50        columns without products
constexpr int kBinHash0 = 41;
constexpr int kBinTiny = 49;
constexpr int kBinEmpty = 50;
constexpr int kNumBins = 51;
constexpr int kHashLog2Max = 15;
constexpr int kHashLog2Min = 8;
constexpr int kBinMid = kBinHash0 + kHashLog2Max - kMidHashLog2;
constexpr int kBitmapChunkLog2 = 20;                          // rows per bitmap-count chunk
constexpr int32_t kSplitMin = 32;  // A columns longer than this get a split-table row

struct BinCfg {
  int64_t tiny_max, hash_max;
};

__device__ __forceinline__ int bin_of(int64_t mu, const BinCfg& c) {
  if (mu <= 0) return kBinEmpty;
  if (mu <= c.tiny_max) return kBinTiny;
  if (mu <= c.hash_max) {
    int s = ceil_log2_u64((uint64_t)mu) + 1;
    if (s < kHashLog2Min) s = kHashLog2Min;
    return kBinHash0 + (kHashLog2Max - s);
  }
  int id = 40 - floor_log2_u64((uint64_t)mu);
  return id < 0 ? 0 : id;
}

// ------------------------------------------------------------------ kernels: setup
// For every stored B(k,j): where column k of A starts and how long it is.
__global__ void k_rowinfo(Operand A, Operand B, const int64_t* aux, int64_t chunk, int64_t* bq_a0, int32_t* bq_alen,
                          unsigned* err) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < B.nnz; q += stride) {
    const int32_t k = B.ir[q];
    int64_t a0 = 0, a1 = 0;
    if (k < 0 || k >= A.n) {
      atomicOr(err, 1u);
    } else {
      const int64_t slot = column_slot(A, aux, chunk, k);
      if (slot >= 0) {
        a0 = load_ptr(A.cp, A.ptr_t, slot);
        a1 = load_ptr(A.cp, A.ptr_t, slot + 1);
      }
    }
    bq_a0[q] = a0;
    bq_alen[q] = (int32_t)(a1 - a0);
  }
}

// Split table (see ProdSrc): rows are made only for the long columns of A that
// some column with row-block counts names, since only parts and row chunks read
// them.  A product without such columns makes no table (a restriction of R-MAT
// scale 23 wrote 1 GB of rows for all its long columns in 0.81 ms, and reads few
// of them).
//   k_split_mark:    flags the columns of A named by the B entries of those
//                    columns.  Groups of 16 lanes take one column each; columns
//                    with more than kLongSlot B entries (the list longs, made by
//                    k_slot_mults) are shared by kLongShare workgroups each.
//   k_split_rows:    after a scan of the flags, numbers the flagged columns
//                    (flag[k] becomes row + 1, 0: none) and lists them.
//   k_split_assign:  notes the row at every B entry of those columns, or at all
//                    entries of B (flat) where such columns are not rare: a flat
//                    pass has no chain of list, pointer and entry loads.
constexpr int64_t kLongSlot = 256;
constexpr int kLongShare = 16;

// Calls f(q) for the B entries of the columns list[multi_begin, multi_end)
// with at most kLongSlot entries, and of all columns in longs (the first
// long_blocks workgroups, a multiple of kLongShare).
template <class F>
__device__ __forceinline__ void for_multi_entries(const Operand& B, const int32_t* list, int64_t multi_begin,
                                                  int64_t multi_end, const int32_t* longs, int64_t nlong,
                                                  unsigned long_blocks, F&& f) {
  if (blockIdx.x >= long_blocks) {
    constexpr int G = 16;
    const int gl = lane_id() & (G - 1);
    const int64_t grp = ((int64_t)(blockIdx.x - long_blocks) * blockDim.x + threadIdx.x) / G;
    const int64_t ngrp = (int64_t)(gridDim.x - long_blocks) * blockDim.x / G;
    for (int64_t pos = multi_begin + grp; pos < multi_end; pos += ngrp) {
      const int32_t t = list[pos];
      const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
      if (b1 - b0 > kLongSlot) continue;
      for (int64_t q = b0 + gl; q < b1; q += 4 * G) f(q, G, b1);
    }
  } else {
    const unsigned lb = blockIdx.x, nlb = long_blocks;
    for (int64_t i = lb / kLongShare; i < nlong; i += nlb / kLongShare) {
      const int32_t t = longs[i];
      const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
      const int64_t step = (int64_t)kLongShare * blockDim.x;
      for (int64_t q = b0 + (int64_t)(lb % kLongShare) * blockDim.x + threadIdx.x; q < b1; q += 4 * step) f(q, step, b1);
    }
  }
}

__global__ void __launch_bounds__(256) k_split_mark(Operand A, Operand B, const int64_t* aux, int64_t chunk,
                                                    const int32_t* list, int64_t multi_begin, int64_t multi_end,
                                                    const int32_t* longs, const unsigned long long* nlong,
                                                    unsigned long_blocks, const int32_t* bq_alen, int32_t* flag) {
  for_multi_entries(B, list, multi_begin, multi_end, longs, (int64_t)*nlong, long_blocks,
                    [&](int64_t q, int64_t step, int64_t end) {  // four entries in flight
    int32_t al[4], k[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t x = q + u * step;
      al[u] = x < end ? bq_alen[x] : 0;
      k[u] = x < end ? B.ir[x] : 0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (al[u] > kSplitMin) flag[column_slot(A, aux, chunk, k[u])] = 1;  // longer than zero, so it is stored
  });
}

struct LoadFlag {
  const int32_t* p;
  __device__ int64_t operator()(int64_t i) const { return (int64_t)p[i]; }
};

__global__ void k_split_rows(int64_t nslots, const int64_t* sid_off, int32_t* flag, int32_t* slot_of_split) {
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < nslots; k += (int64_t)gridDim.x * blockDim.x)
    if (flag[k]) {
      const int32_t sid = (int32_t)sid_off[k];
      slot_of_split[sid] = (int32_t)k;
      flag[k] = sid + 1;
    }
}

__global__ void __launch_bounds__(256) k_split_assign(Operand A, Operand B, const int64_t* aux, int64_t chunk,
                                                      const int32_t* list, int64_t multi_begin, int64_t multi_end,
                                                      const int32_t* longs, const unsigned long long* nlong,
                                                      unsigned long_blocks, int flat, const int32_t* bq_alen,
                                                      const int32_t* flag, int32_t* bq_split) {
  auto four = [&](int64_t q, int64_t step, int64_t end) {
    int32_t al[4], k[4], sid[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t x = q + u * step;
      al[u] = x < end ? bq_alen[x] : 0;
      k[u] = x < end ? B.ir[x] : 0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) sid[u] = al[u] > kSplitMin ? flag[column_slot(A, aux, chunk, k[u])] - 1 : -1;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (q + u * step < end) bq_split[q + u * step] = sid[u];
  };
  if (flat) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < B.nnz; q += 4 * stride) four(q, stride, B.nnz);
  } else {
    for_multi_entries(B, list, multi_begin, multi_end, longs, (int64_t)*nlong, long_blocks, four);
  }
}

// Row of the split table of one long column: entry b (< sstride - 1) is the
// first position whose row lies in row block b or later, the last entry the
// column length.  One wave per column walks its rows once: the entry at
// position e fills the blocks after its predecessor's block up to its own.
// Very long columns are searched instead, a lane per block: the walk of R-MAT
// scale 23's longest column (1600 rounds of a wave) took 0.58 ms.
__global__ void k_split_fill(Operand A, const int64_t* nsplit_d, const int32_t* slot_of_split,
                             int32_t* splits, int32_t sstride, int32_t rbshift) {
  const int64_t nsplit = *nsplit_d;
  const int lane = lane_id();
  const int64_t w0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = (int64_t)gridDim.x * blockDim.x / kWave;
  for (int64_t sidx = w0; sidx < nsplit; sidx += nw) {
    const int32_t k = slot_of_split[sidx];
    const int64_t a0 = slot_begin(A, k);
    const int32_t al = (int32_t)(slot_begin(A, k + 1) - a0);
    const int32_t* col = A.ir + a0;
    int32_t* out = splits + sidx * sstride;
    // rounds of the walk against dependent loads of the searches.  Product whose A has
    // columns of this length, walked | searched: 10^4 entries over 2^20 rows (156 rounds, 42
    // loads) 289 | 241 us, over 2^25 rows (156, 910) 591 | 722; 10^5 over 2^25 (1562, 1105) 1110
    // | 780; 10^6 over 2^20 (15625, 60) 6896 | 3517; 10^3 over 2^23 (15, 170) 355 | 396.
    const int32_t searches = (sstride + kWave - 1) / kWave * (floor_log2_u64((uint64_t)al) + 1);
    if (al / kWave > searches) {
      for (int32_t b = lane; b < sstride; b += kWave) {
        int32_t lo = 0, hi = al;
        if (b == sstride - 1) lo = al;
        while (lo < hi) {
          const int32_t mid = (int32_t)(((uint32_t)lo + (uint32_t)hi) >> 1);
          if ((col[mid] >> rbshift) < b)
            lo = mid + 1;
          else
            hi = mid;
        }
        out[b] = lo;
      }
      continue;
    }
    for (int32_t e = lane; e < al; e += kWave) {
      const int32_t cur = col[e] >> rbshift;
      const int32_t prev = e == 0 ? -1 : (col[e - 1] >> rbshift);
      for (int32_t b = prev + 1; b <= cur; ++b) out[b] = e;
    }
    const int32_t last = al > 0 ? (col[al - 1] >> rbshift) : -1;
    for (int32_t b = last + 1 + lane; b < sstride; b += kWave) out[b] = al;
  }
}

// mults[t] = number of multiplications of output column (slot) t.  Groups
// of 8 lanes take one slot each (most columns hold a few B entries); slots
// with more than kLongSlot entries are listed and take a workgroup each
// (k_slot_mults_long), so a long column holds up no group.  The total goes
// to *total with one atomic per workgroup.
// Device totals spread over kSpread counters, one per 128-byte line: a single
// counter serialises the workgroups' atomics at about 10 ns each (31 us for
// 3126 workgroups).  k_cnt_apply adds them up.
constexpr int kSpread = 16;
constexpr int kSpreadWords = kSpread * 16;
__device__ __forceinline__ unsigned long long* spread(unsigned long long* total) {
  return total + (blockIdx.x % kSpread) * 16;
}

__device__ __forceinline__ void add_total(int64_t acc, bool mine, unsigned long long* total) {
  __shared__ unsigned long long s_acc;
  if (threadIdx.x == 0) s_acc = 0;
  __syncthreads();
  if (mine && acc) atomicAdd(&s_acc, (unsigned long long)acc);
  __syncthreads();
  if (threadIdx.x == 0 && s_acc) atomicAdd(spread(total), s_acc);
}

__global__ void __launch_bounds__(256) k_slot_mults(Operand B, const int32_t* bq_alen, int64_t nslots, int64_t* mults,
                                                    unsigned long long* total, int32_t* longs,
                                                    unsigned long long* nlong) {
  constexpr int G = 8;
  const int gl = lane_id() & (G - 1);
  const int64_t grp = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / G;
  const int64_t ngrp = (int64_t)gridDim.x * blockDim.x / G;
  int64_t acc = 0;
  for (int64_t t = grp; t < nslots; t += ngrp) {
    const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
    if (b1 - b0 > kLongSlot) {
      if (gl == 0) longs[atomicAdd(nlong, 1ull)] = (int32_t)t;
      continue;
    }
    int64_t s = 0;
    for (int64_t q = b0 + gl; q < b1; q += 4 * G) {
      int32_t v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = q + k * G < b1 ? bq_alen[q + k * G] : 0;
      s += (int64_t)v[0] + v[1] + v[2] + v[3];
    }
#pragma unroll
    for (int d = 1; d < G; d <<= 1) s += __shfl_xor(s, d, G);
    if (gl == 0) {
      mults[t] = s;
      acc += s;
    }
  }
  add_total(acc, gl == 0, total);
}

// Four loads in flight per thread: the longest column of R-MAT scale 20 (23,516
// entries) took 89 us on one wave.
__global__ void __launch_bounds__(256) k_slot_mults_long(Operand B, const int32_t* bq_alen, const int32_t* longs,
                                                         const unsigned long long* nlong, int64_t* mults,
                                                         unsigned long long* total) {
  __shared__ int64_t red[4];
  const int64_t n = (int64_t)*nlong;
  int64_t acc = 0;
  for (int64_t i = blockIdx.x; i < n; i += gridDim.x) {
    const int32_t t = longs[i];
    const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
    int64_t s = 0;
    for (int64_t q = b0 + threadIdx.x; q < b1; q += 4 * 256) {
      int32_t v[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) v[k] = q + k * 256 < b1 ? bq_alen[q + k * 256] : 0;
      s += (int64_t)v[0] + v[1] + v[2] + v[3];
    }
    s = wave_sum(s);
    if (lane_id() == 0) red[threadIdx.x / kWave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
      s = red[0] + red[1] + red[2] + red[3];
      mults[t] = s;
      acc += s;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0 && acc) atomicAdd(spread(total), (unsigned long long)acc);
}

// Up to kSmallSlots slots: launches and their gaps bound the plan (4096 columns of 8
// entries: 13 launches of 2 to 6 us, 106 us a pass, 76 with 9), so three launches take
// the place of seven: one finds the ranges and the products, a wave for each slot, and
// one workgroup each bins the columns and scans their counts.  The line lies where
// one workgroup's work passes the launches it saves: 2^14 columns of an R-MAT graph took
// 308 us this way, 271 by the separate launches.
constexpr int kSmallSlots = 8192;
constexpr int kSmallPer = kSmallSlots / 1024;

// k_rowinfo and k_slot_mults of a small plan.  Columns are at most kSmallSlots
// long here, 32 rounds of a wave with four loads in flight a lane; the ones above
// kLongSlot are listed as by k_slot_mults.
__global__ void __launch_bounds__(256) k_slots_small(Operand A, Operand B, const int64_t* aux, int64_t chunk,
                                                     int64_t* bq_a0, int32_t* bq_alen, int nslots, int64_t* mults,
                                                     unsigned long long* total, int32_t* longs,
                                                     unsigned long long* nlong, unsigned* err) {
  constexpr int U = 4;
  const int lane = lane_id();
  const int t = (int)((blockIdx.x * blockDim.x + threadIdx.x) / kWave);
  int64_t sum = 0;
  if (t < nslots) {
    const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
    for (int64_t q = b0 + lane; q < b1; q += U * kWave) {
      int32_t k[U];
      int64_t a0[U], a1[U];
#pragma unroll
      for (int u = 0; u < U; ++u) k[u] = q + u * kWave < b1 ? B.ir[q + u * kWave] : -1;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        a0[u] = a1[u] = 0;
        if (k[u] >= 0 && k[u] < A.n) {
          const int64_t slot = column_slot(A, aux, chunk, k[u]);
          if (slot >= 0) {
            a0[u] = load_ptr(A.cp, A.ptr_t, slot);
            a1[u] = load_ptr(A.cp, A.ptr_t, slot + 1);
          }
        } else if (q + u * kWave < b1) {
          atomicOr(err, 1u);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (q + u * kWave < b1) {
          bq_a0[q + u * kWave] = a0[u];
          bq_alen[q + u * kWave] = (int32_t)(a1[u] - a0[u]);
          sum += (int32_t)(a1[u] - a0[u]);
        }
    }
    sum = wave_sum(sum);
    if (lane == 0) {
      mults[t] = sum;
      if (b1 - b0 > kLongSlot) longs[atomicAdd(nlong, 1ull)] = t;
    }
  }
  add_total(sum, lane == 0, total);
}

// Bins, offsets and list (as k_bin_count and k_bin_fill) by one workgroup of 1024.
__global__ void __launch_bounds__(1024) k_bin_small(const int64_t* mults, int nslots, BinCfg cfg, int64_t* binoff,
                                                    int32_t* list) {
  static_assert(kNumBins < kWave, "a wave scans the bins");
  __shared__ int hist[kWave];
  const int lane = lane_id();
  if (threadIdx.x < kWave) hist[threadIdx.x] = 0;
  int b[kSmallPer], rank[kSmallPer];
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k) {
    const int t = k * 1024 + threadIdx.x;
    b[k] = t < nslots ? bin_of(mults[t], cfg) : -1;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k) {
    uint64_t rest = __ballot(b[k] >= 0);
    rank[k] = 0;
    while (rest) {  // one atomic for the lanes of a bin
      const int first = __ffsll((unsigned long long)rest) - 1;
      const int bin = __builtin_amdgcn_readlane(b[k], first);
      const uint64_t same = __ballot(b[k] == bin);
      int base = 0;
      if (lane == first) base = atomicAdd(&hist[bin], __popcll(same));
      base = __builtin_amdgcn_readlane(base, first);
      if (b[k] == bin) rank[k] = base + __popcll(same & lanemask_lt());
      rest &= ~same;
    }
  }
  __syncthreads();
  if (threadIdx.x < kWave) {
    const int n = hist[lane];
    const int off = group_scan<kWave>(n, 0, [](int x, int y) { return x + y; }) - n;
    hist[lane] = off;
    if (lane <= kNumBins) binoff[lane] = off;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k)
    if (b[k] >= 0) list[hist[b[k]] + rank[k]] = k * 1024 + threadIdx.x;
}

// Counting sort of slots into bins: histogram, offsets, fill.
__global__ void k_bin_count(const int64_t* mults, int64_t nslots, BinCfg cfg, unsigned long long* counts) {
  __shared__ unsigned hist[kNumBins];
  for (int i = threadIdx.x; i < kNumBins; i += blockDim.x) hist[i] = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < nslots; t += stride)
    atomicAdd(&hist[bin_of(mults[t], cfg)], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < kNumBins; i += blockDim.x)
    if (hist[i]) atomicAdd(&counts[i], (unsigned long long)hist[i]);
}

// Each thread ranks kFillPer slots per round in LDS, so a workgroup reserves
// its ranges of the bins once per blockDim * kFillPer slots.  Every
// workgroup derives the bin offsets from the counts itself; the first one
// also stores them (binoff, kNumBins + 1 entries).  fill must be zero.
constexpr int kFillPer = 8;
__global__ void k_bin_fill(const int64_t* mults, int64_t nslots, BinCfg cfg, const unsigned long long* counts,
                           int64_t* binoff, unsigned long long* fill, int32_t* list) {
  __shared__ unsigned hist[kNumBins];
  __shared__ int64_t base[kNumBins];
  __shared__ int64_t off[kNumBins + 1];
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int i = 0; i < kNumBins; ++i) {
      off[i] = run;
      run += (int64_t)counts[i];
    }
    off[kNumBins] = run;
  }
  __syncthreads();
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i <= kNumBins; i += blockDim.x) binoff[i] = off[i];
  const int64_t span = (int64_t)blockDim.x * kFillPer;
  for (int64_t t0 = (int64_t)blockIdx.x * span; t0 < nslots; t0 += (int64_t)gridDim.x * span) {
    for (int i = threadIdx.x; i < kNumBins; i += blockDim.x) hist[i] = 0;
    __syncthreads();
    int b[kFillPer];
    unsigned rank[kFillPer];
#pragma unroll
    for (int k = 0; k < kFillPer; ++k) {
      const int64_t t = t0 + (int64_t)k * blockDim.x + threadIdx.x;
      b[k] = t < nslots ? bin_of(mults[t], cfg) : -1;
      rank[k] = b[k] >= 0 ? atomicAdd(&hist[b[k]], 1u) : 0u;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kNumBins; i += blockDim.x)
      if (hist[i]) base[i] = off[i] + (int64_t)atomicAdd(&fill[i], (unsigned long long)hist[i]);
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kFillPer; ++k)
      if (b[k] >= 0) list[base[b[k]] + rank[k]] = (int32_t)(t0 + (int64_t)k * blockDim.x + threadIdx.x);
    __syncthreads();
  }
}

// ------------------------------------------------------------------ product iteration
// A's row and value at position o through a 32-bit byte offset from the base
// (valid when o < 2^29, so o * 8 does not wrap).
__device__ __forceinline__ int32_t load_row32(const int32_t* air, uint32_t o) {
  return *reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(air) + (o << 2));
}
template <typename T>
__device__ __forceinline__ T load_val32(const T* an, uint32_t o) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(an) + o * (uint32_t)sizeof(T));
}


// Block-cooperative iteration over the products of one output column.
// The column's stored B entries are taken in chunks of at most QC, one per
// thread: all threads load, in parallel, their entry's range in A (start,
// length -- from the split table for long columns of A -- and B's value), and
// a scan numbers the chunk's products 0..total-1 and the nonempty ranges.
// Products are taken in windows of 64 (one per lane of a wave), U windows per
// wave and round, all loads of a round in flight together; a chunk with more
// than WIN windows is taken in tiles of WIN.
// Which range a lane's product lies in comes from a bit per product: wst[k] is
// the (nonempty) range holding the first product of window k, and bits[k] has
// bit i - 1 set when a range starts at product i >= 1 of the window, so lane i
// lies in range wst[k] + (bits set below bit i).  That is two instructions per
// window and no search (a binary search over range starts bounded by ballots
// cost about 35 vector and 35 scalar instructions per window, and issuing them
// is what bounds the callers).  base[] holds each range's start in A less its
// first product's number, so a product's position is base + number.
// qidx (if given) lists the B entries to visit: qidx[b0, b1) instead of
// b0 .. b1-1.
// f receives the U products of a lane at once: rows r[u] (-1: past the end),
// A's values a[u] and B's values b[u].  Ranges of unsplit columns of A reach
// outside [r0, r1), so unless `full` f has to check the rows: a row r is
// inside if (uint32_t)(r - r0) < r1 - r0, which -1 never is.
// Must be called by every thread of the workgroup (it contains barriers).
// Positions are 32 bits with OFF32 (A has fewer than 2^29 entries), then A is
// loaded through 32-bit byte offsets; else 64 bits.
constexpr int kQChunk = 256;
constexpr int kQChunkWide = 512;
constexpr int kCountWin = 256;   // windows per tile in the counts
constexpr int kNumWin = 128;     // and in the numeric phase, whose LDS is dear

template <int QC, int WIN, bool OFF32, bool BV>
struct RangeLdsT {
  using Off = std::conditional_t<OFF32, uint32_t, int64_t>;
  static constexpr int kQ = QC, kWin = WIN;
  static constexpr bool kOff32 = OFF32;
  uint64_t bits[WIN];
  double bval[BV ? QC : 1];  // B's value, stored in the first bytes of each slot
  Off base[QC];
  uint16_t wst[WIN];
};

// Range in A of B entry q restricted to rows [r0, r1) (the whole column unless
// it is split): its start and length, and B's value.
template <typename T, bool LOADB>
__device__ __forceinline__ void load_range(const ProdSrc& S, const T* bn, int64_t q, int32_t r0, int32_t r1, bool full,
                                           int64_t& at, int32_t& len, T& bq) {
  const int64_t a0 = S.a0[q];
  int32_t e0 = 0, e1 = S.alen[q];
  const int32_t sid = !full && S.splits ? S.split[q] : -1;
  if constexpr (LOADB) bq = bn[q];
  if (sid >= 0) {
    const int32_t* sp = S.splits + (int64_t)sid * S.sstride;
    e0 = sp[r0 >> S.rbshift];
    e1 = sp[r1 >= S.m ? S.sstride - 1 : (r1 >> S.rbshift)];
  }
  at = a0 + e0;
  len = e1 - e0;
}

// Products of a chunk in the low bits of a scan value, nonempty ranges above.
constexpr int kRangeBits = 50;
__device__ __forceinline__ int64_t range_word(int32_t len) {
  return (int64_t)len | (len > 0 ? (int64_t)1 << kRangeBits : (int64_t)0);
}

// The rounds of one chunk of `total` products.  The thread's range holds
// products [ex, ex + len) and is nonempty range rk of the chunk (len 0: none);
// R.base and R.bval hold the ranges (this thread's written by the caller), and
// R.bits is zero, both as of the caller's last barrier or this thread's own
// writes.  With set false bits and wst are as the previous call left them.
// Ends with a barrier.
template <int U, typename T, bool LOADA, bool LOADB, class RL, class F>
__device__ __forceinline__ void product_tiles(const ProdSrc& S, const T* an, bool set, int64_t total, int64_t ex,
                                              int32_t len, int32_t rk, RL& R, F&& f) {
  using Off = typename RL::Off;
  constexpr int kWin = RL::kWin, kTile = kWin * kWave;
  const int lane = lane_id();
  const int tid = (int)threadIdx.x;
  const int32_t wid = __builtin_amdgcn_readfirstlane(tid / kWave), nw = (int32_t)blockDim.x / kWave;
  for (int64_t tb = 0; tb < total; tb += kTile) {
    if (set) {
      if (tb > 0) {
        __syncthreads();  // the last tile's rounds are done
        for (int k = tid; k < kWin; k += (int)blockDim.x) R.bits[k] = 0;
        __syncthreads();
      }
      if (len > 0 && ex < tb + kTile && ex + len > tb) {
        const int32_t st = (int32_t)(ex - tb > 0 ? ex - tb : 0);
        const int32_t en = (int32_t)(ex + len - tb < kTile ? ex + len - tb : kTile);
        if (ex >= tb && (st & (kWave - 1)))
          atomicOr((unsigned long long*)&R.bits[st / kWave], 1ull << ((st & (kWave - 1)) - 1));
        for (int32_t k = (st + kWave - 1) / kWave; k * kWave < en; ++k) R.wst[k] = (uint16_t)rk;
      }
      __syncthreads();
    }
    const int32_t tt = __builtin_amdgcn_readfirstlane((int32_t)(total - tb < kTile ? total - tb : kTile));
    const int32_t nwin = (tt + kWave - 1) / kWave;
    const Off tbo = (Off)tb;
    for (int32_t base = 0; base < nwin; base += U * nw) {
      // a full round gives each wave U consecutive windows (which share lines of A),
      // the last one deals the windows round robin, so that all waves have as many
      const bool whole = (base + U * nw) * kWave <= tt;
      const int32_t k0 = whole ? base + wid * U : base + wid, step = whole ? 1 : nw;
      if (k0 >= nwin) break;
      int32_t r[U], p[U];
      T a[U], bv[U];
      uint64_t w[U];
      uint32_t own[U];
      Off o[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int32_t k = k0 + u * step < nwin ? k0 + u * step : nwin - 1;
        w[u] = R.bits[k];
        own[u] = R.wst[k];
        p[u] = k * kWave + lane;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        own[u] = __builtin_amdgcn_mbcnt_hi((uint32_t)(w[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)w[u], own[u]));
        o[u] = R.base[own[u]] + (Off)(p[u] < tt ? p[u] : tt - 1) + tbo;
        bv[u] = LOADB ? reinterpret_cast<const T*>(&R.bval[own[u]])[0] : T(0);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        r[u] = -1;
        a[u] = T(0);
        if (k0 + u * step < nwin) {  // uniform
          if constexpr (RL::kOff32) {
            r[u] = load_row32(S.air, o[u]);
            if constexpr (LOADA) a[u] = load_val32(an, o[u]);
          } else {
            r[u] = S.air[o[u]];
            if constexpr (LOADA) a[u] = an[o[u]];
          }
        }
      }
      if (!whole) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (p[u] >= tt) r[u] = -1;
      }
      f(r, a, bv);
    }
  }
  __syncthreads();
}

// `first`, if given, receives the first chunk's total products and whether it
// is the only one and of one tile, so that its ranges stay in R.
struct FirstChunk {
  int32_t total;
  bool all;
};

template <int U, typename T, bool LOADA, bool LOADB, class RL, class F>
__device__ __forceinline__ void block_products(const ProdSrc& S, const T* an, const T* bn, int64_t b0, int64_t b1,
                                               int32_t r0, int32_t r1, bool full, RL& R, int64_t* red,
                                               const int32_t* qidx, FirstChunk* first, F&& f) {
  using Off = typename RL::Off;
  const int qchunk = (int)blockDim.x < S.qchunk ? (int)blockDim.x : S.qchunk;
  const int tid = (int)threadIdx.x;
  for (int64_t qc = b0; qc < b1; qc += qchunk) {
    const int nq = (int)(b1 - qc < qchunk ? b1 - qc : qchunk);
    for (int k = tid; k < RL::kWin; k += (int)blockDim.x) R.bits[k] = 0;
    int64_t at = 0;
    int32_t len = 0;
    T bq = T(0);
    if (tid < nq) load_range<T, LOADB>(S, bn, qidx ? (int64_t)qidx[qc + tid] : qc + tid, r0, r1, full, at, len, bq);
    int64_t sum;
    const int64_t pre = block_excl_scan1(range_word(len), red, &sum);
    const int64_t ex = pre & (((int64_t)1 << kRangeBits) - 1), total = sum & (((int64_t)1 << kRangeBits) - 1);
    const int32_t rk = (int32_t)(pre >> kRangeBits);
    if (len > 0) {
      R.base[rk] = (Off)(at - ex);
      if constexpr (LOADB) reinterpret_cast<T*>(&R.bval[rk])[0] = bq;
    }
    if (first && qc == b0) {
      first->all = b1 - b0 <= qchunk && total <= RL::kWin * kWave;
      first->total = (int32_t)total;
    }
    product_tiles<U, T, LOADA, LOADB>(S, an, true, total, ex, len, rk, R, f);
  }
}

__device__ __forceinline__ uint32_t hash_row(int32_t r, int log2s) {
  return ((uint32_t)r * 0x9E3779B1u) >> (32 - log2s);
}

// ------------------------------------------------------------------ tiny columns (lane groups)
struct TinyCol {
  int64_t b0, b1, o;  // B range and output offset
  int32_t t, m;       // column (slot of B), -1: none; products
};

template <typename T>
struct TinyLds {  // of one wave
  TinyCol col[kWave];
  int32_t row[kWave];
  int32_t aux[kWave];
  T val[kWave];
};

// The products of a column, one per lane of its group, when they don't fit the
// block layout: lane gl takes product gl of the column's list.  Returns its
// row, -1 past the end.
template <int G, int SR, typename T, bool VAL>
__device__ __forceinline__ int32_t tiny_listed(const Operand& A, const Operand& B, const int64_t* bq_a0,
                                               const int32_t* bq_alen, int64_t b0, int64_t b1, TinyLds<T>& L, T& val) {
  using S = Semiring<SR, T>;
  const int lane = lane_id(), gl = lane & (G - 1), gb = lane & ~(G - 1);
  int32_t *const s_row = L.row + gb, *const s_aux = L.aux + gb;
  T* const s_val = L.val + gb;
  const T* an = (const T*)A.num;
  const T* bn = (const T*)B.num;
  int total = 0;
  // groups of one wave go on until the longest is done (a group past its end has no products)
  for (int64_t qc = b0; __any(qc < b1); qc += G) {
    const int64_t q = qc + gl;
    const bool inq = q < b1;
    const int al = inq ? bq_alen[q] : 0;
    const int64_t qa0 = inq ? bq_a0[q] : 0;
    T qb = T(0);
    if constexpr (VAL && S::kUsesB) qb = inq ? bn[q] : T(0);
    const int incl = group_scan<G>(al, 0, [](int x, int y) { return x + y; });
    const int excl = incl - al;
    const int ctot = __shfl(incl, G - 1, G);
    s_aux[gl] = -1;
    wave_sync();
    if (al > 0 && excl < G) s_aux[excl] = gl;
    wave_sync();
    const int o = group_scan<G>(s_aux[gl], -1, [](int x, int y) { return x > y ? x : y; });
    const int src = o < 0 ? 0 : o;
    const int ostart = __shfl(excl, src, G);
    const int64_t ea0 = __shfl(qa0, src, G);
    T bv = T(0);
    if constexpr (VAL && S::kUsesB) bv = __shfl(qb, src, G);
    if (gl < ctot && total + gl < G) {
      const int64_t e = ea0 + (gl - ostart);
      s_row[total + gl] = A.ir[e];
      if constexpr (VAL) s_val[total + gl] = S::mul(S::kUsesA ? an[e] : T(0), bv);
    }
    total += ctot;
    wave_sync();
  }
  if constexpr (VAL) val = gl < total ? s_val[gl] : T(0);
  return gl < total ? s_row[gl] : -1;
}

// Columns k .. k + 64/G - 1 of the wave's table (at most G products each), one
// per group of G lanes.  Lanes take the products of the column's B entries in
// blocks: W = the largest power of two for which the entries of every group fit;
// lane p of block i takes product p of entry i, so a lane finds its product by
// its own number and every block is ascending before the sort.  (Columns with an
// A column longer than W list their products first.)  The numeric pass sorts
// (row, lane) keys and sums each run of equal rows in product order -- the order
// of Algorithm 1 --, the count sorts the rows and counts the first of each run.
template <int G, int SR, typename T, bool COUNT>
__device__ __forceinline__ void tiny_group(const Operand& A, const Operand& B, const int64_t* bq_a0,
                                           const int32_t* bq_alen, int k, int kend, int64_t* cnt, int32_t* cir,
                                           T* cnum, TinyLds<T>& L, const LaneSides& sides) {
  using S = Semiring<SR, T>;
  constexpr bool kVal = SR != SPX_OR_AND && !COUNT;
  const int lane = lane_id(), gl = lane & (G - 1), gb = lane & ~(G - 1);
  const int mine = k + lane / G;
  int64_t b0 = 0, b1 = 0, obase = 0;
  int32_t t = -1;
  if (mine < kend) {
    const TinyCol& c = L.col[mine];
    b0 = c.b0;
    b1 = c.b1;
    t = c.t;
    if constexpr (!COUNT) obase = c.o;
  }
  const int nb = b1 - b0 > G ? G + 1 : (int)(b1 - b0);
  int most = __builtin_amdgcn_readfirstlane(nb);
#pragma unroll
  for (int g = G; g < kWave; g += G) most = max(most, __builtin_amdgcn_readlane(nb, g));
  int32_t row = -1;
  T val = T(0);
  int sorted = 1;
  bool blocks = false;
  if (most <= G) {  // uniform
    const int lw = (G == 64 ? 6 : (G == 32 ? 5 : 4)) - (most <= 1 ? 0 : 32 - __builtin_clz((unsigned)most - 1));
    const int64_t q = b0 + (gl >> lw);
    const bool inq = q < b1;
    const int al = inq ? bq_alen[q] : 0;
    int64_t e = inq ? bq_a0[q] : 0;
    T bv = T(0);
    if constexpr (kVal && S::kUsesB) bv = inq ? ((const T*)B.num)[q] : T(0);
    blocks = __ballot(al > 1 << lw) == 0;
    if (blocks) {  // uniform
      sorted = 1 << lw;
      const int p = gl & (sorted - 1);
      e += p;
      if (p < al) {
        row = A.ir[e];
        if constexpr (kVal) val = S::mul(S::kUsesA ? ((const T*)A.num)[e] : T(0), bv);
      }
    }
  }
  if (!blocks) row = tiny_listed<G, SR, T, kVal>(A, B, bq_a0, bq_alen, b0, b1, L, val);
  // sorted rows; idx: the lane (of the group) whose product this is
  bool valid;
  int idx = 0;
  if (COUNT) {
    row = (int32_t)sort_runs<G>((uint32_t)row, sorted, sides);  // -1, the largest key, past the end
    valid = row >= 0;
  } else if (A.m <= (1ll << 25)) {  // 32-bit keys while the rows leave 6 bits for the lane
    const uint32_t key = sort_runs<G>(row < 0 ? ~0u : ((uint32_t)row << 6) | (uint32_t)gl, sorted, sides);
    valid = key != ~0u;
    row = (int32_t)(key >> 6);
    idx = (int)(key & 63u);
  } else {
    const uint64_t key = sort_runs<G>(row < 0 ? ~(uint64_t)0 : ((uint64_t)(uint32_t)row << 32) | (uint32_t)gl, sorted, sides);
    valid = key != ~(uint64_t)0;
    row = (int32_t)(key >> 32);
    idx = (int)((uint32_t)key & 63u);
  }
  // the previous lane's row (DPP wave shift; lane 0 of a group never uses it)
  const int32_t prev = __builtin_amdgcn_update_dpp(0, row, 0x138, 0xF, 0xF, false);  // wave_shr:1
  const bool head = valid && (gl == 0 || prev != row);
  const uint64_t hm = __ballot(head);
  // heads of this lane's group, and those before the lane
  uint32_t below;
  if constexpr (G == 64) {
    below = __builtin_amdgcn_mbcnt_hi((uint32_t)(hm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hm, 0));
    if (COUNT) {
      if (gl == 0 && t >= 0) cnt[t] = __popcll(hm);
      return;
    }
  } else {
    const uint32_t hg = (lane < 32 ? (uint32_t)hm : (uint32_t)(hm >> 32)) >> (gb & 31);
    if (COUNT) {
      if (gl == 0 && t >= 0) cnt[t] = __popc(G == 16 ? hg & 0xffffu : hg);
      return;
    }
    below = __popc(hg & ((1u << gl) - 1u));
  }
  if constexpr (kVal) {
    // every lane holds its sorted product's value; step d adds the value of lane
    // + d while that lane goes on with this lane's run
    T x = __shfl(val, gb + idx);
    val = x;
    const uint64_t cont = __ballot(valid && !head);
    for (uint64_t later = cont >> 1, more = later; more; later >>= 1, more &= later) {
      x = lane_next(x);
      const T sum = S::add(val, x);
      if (lane_of_mask(more)) val = sum;
    }
  }
  if (head) {
    const int64_t o = obase + below;
    cir[o] = row;
    if constexpr (kVal) cnum[o] = val;
  }
}

// Tiny columns (at most 64 products).  A wave takes up to 64 columns at a time
// (fewer when the bin is too small to give every wave 64): lane k loads column
// k's id, products, B range and output offset (two load levels for all of
// them) into the wave's LDS table, ordered by products: columns of at most 16
// are then done four at a time, of at most 32 two at a time, the others one by
// one, and a column waits only on its B entries' A ranges and then A's rows and
// values.  Half the time is instruction issue, the rest those two waits.  512
// Galerkin levels (A P with 56 products a column, then P^T (A P) with 32): numeric
// 7.36 + 4.16 -> 4.44 + 2.80 ms, count 2.57 + 1.55 -> 2.01 + 1.33 ms against a sort of
// all 64 lanes after a scan for the lanes' products (the count: a table of rows).
// Loading the next columns' ranges early took more registers than it hid: 4.37 +
// 2.58 and 2.95 + 1.73 ms.  The grid is as long as there are columns, up to 64
// workgroups a CU: with 16 the last of three rounds was mostly empty.
template <int SR, typename T, bool COUNT>
__global__ void __launch_bounds__(256) k_tiny(Operand A, Operand B, const int64_t* bq_a0, const int32_t* bq_alen,
                                              const int64_t* mults, const int32_t* list, const int64_t* binoff,
                                              int64_t* cnt, const int64_t* off, int32_t* cir, T* cnum) {
  __shared__ TinyLds<T> s_lds[4];
  const int lane = lane_id();
  TinyLds<T>& L = s_lds[threadIdx.x / kWave];
  const LaneSides sides;
  const int64_t beg = binoff[kBinTiny], ncols = binoff[kBinTiny + 1] - beg;
  constexpr int kWaves = 4;
  const int w = threadIdx.x / kWave;
  // the waves of a block take every fourth column of its share each, so that
  // neighbouring columns, which often share lines of A and always those of C, are done together
  const int64_t nwaves = (int64_t)gridDim.x * kWaves;
  const int64_t per = std::min<int64_t>(kWave, std::max<int64_t>(2, (ncols + nwaves - 1) / nwaves));
  for (int64_t c0 = blockIdx.x * kWaves * per; c0 < ncols; c0 += nwaves * per) {
    const int64_t left = ncols - c0 - w;
    const int n = left <= 0 ? 0 : (int)std::min<int64_t>(per, (left + kWaves - 1) / kWaves);
    TinyCol c{};
    c.m = kWave;
    if (lane < n) {
      c.t = list[beg + c0 + kWaves * lane + w];
      c.m = (int32_t)mults[c.t];
      c.b0 = slot_begin(B, c.t);
      c.b1 = slot_begin(B, c.t + 1);
      c.o = COUNT ? 0 : off[c.t];
    }
    const uint64_t m16 = __ballot(lane < n && c.m <= 16), m32 = __ballot(lane < n && c.m > 16 && c.m <= 32);
    const uint64_t m64 = __ballot(lane < n && c.m > 32);
    const int n16 = __popcll(m16), n32 = n16 + __popcll(m32);
    const uint64_t same = c.m <= 16 ? m16 : (c.m <= 32 ? m32 : m64);
    if (lane < n) L.col[(c.m <= 16 ? 0 : (c.m <= 32 ? n16 : n32)) + __popcll(same & lanemask_lt())] = c;
    wave_sync();
    for (int k = 0; k < n16; k += 4)
      tiny_group<16, SR, T, COUNT>(A, B, bq_a0, bq_alen, k, n16, cnt, cir, cnum, L, sides);
    for (int k = n16; k < n32; k += 2)
      tiny_group<32, SR, T, COUNT>(A, B, bq_a0, bq_alen, k, n32, cnt, cir, cnum, L, sides);
    for (int k = n32; k < n; ++k)
      tiny_group<64, SR, T, COUNT>(A, B, bq_a0, bq_alen, k, n, cnt, cir, cnum, L, sides);
    wave_sync();  // the table is rewritten for the next columns
  }
}

// ------------------------------------------------------------------ count: hash
// One workgroup per column; key-only open-addressing table of 2^log2s
// slots (at least twice the number of products).  Columns listed before
// position `multi_end` also get their distinct rows counted per row block, as
// they are inserted.  (A pass over the table for these counts, and clearing it
// word by word, took longer than the insertions: at 8192 products each thread
// handles 16 products but 32 slots.)
template <bool OFF32>
using HashRanges = RangeLdsT<kQChunk, kCountWin, OFF32, false>;

template <bool OFF32>
__global__ void __launch_bounds__(1024, 8) k_count_hash(Operand B, ProdSrc S, const int64_t* mults,
                             const int32_t* list, int64_t beg, int64_t end, int64_t multi_begin, int64_t multi_end,
                             int rbshift, int64_t nblk, uint32_t* blkcnt, int64_t* cnt, unsigned* err) {
  extern __shared__ __align__(16) unsigned char lds[];
  uint32_t* keys = (uint32_t*)lds;
  __shared__ int64_t red[1024 / kWave + 1];
  __shared__ HashRanges<OFF32> s_rng;
  for (int64_t pos = beg + blockIdx.x; pos < end; pos += gridDim.x) {
    const int32_t t = list[pos];
    const int log2s = std::max(ceil_log2_u64((uint64_t)mults[t]) + 1, kHashLog2Min);  // as bin_of
    const uint32_t TS = 1u << log2s;
    uint32_t* lblk = keys + TS;  // per-block counters when they fit
    const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
    const bool want_blk = pos < multi_end;
    const bool lds_blk = nblk <= 1024;
    uint32_t* dst = blkcnt + (pos - multi_begin) * nblk;  // zero (used with want_blk only)
    uint32_t* blk = lds_blk ? lblk : dst;
    for (uint32_t i = threadIdx.x; i < TS / 4; i += blockDim.x)
      reinterpret_cast<uint4*>(keys)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    if (want_blk && lds_blk)
      for (int64_t i = threadIdx.x; i < nblk; i += blockDim.x) lblk[i] = 0;
    __syncthreads();
    int64_t mine = 0;
    block_products<4, int, false, false>(
        S, nullptr, nullptr, b0, b1, 0, 0, true, s_rng, red, nullptr, nullptr,
        [&](const int32_t(&r)[4], const int(&)[4], const int(&)[4]) {
          // first probes of the four windows together
          uint32_t h[4], old[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            h[u] = hash_row(r[u], log2s);
            old[u] = r[u] >= 0 ? atomicCAS(&keys[h[u]], ~0u, (uint32_t)r[u]) : (uint32_t)r[u];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            for (uint32_t probe = 1; old[u] != ~0u && old[u] != (uint32_t)r[u]; ++probe) {
              if (probe >= TS) {
                atomicOr(err, 2u);
                break;
              }
              h[u] = (h[u] + 1) & (TS - 1);
              old[u] = atomicCAS(&keys[h[u]], ~0u, (uint32_t)r[u]);
            }
            if (r[u] >= 0 && old[u] == ~0u) {
              ++mine;
              if (want_blk) atomicAdd(&blk[r[u] >> rbshift], 1u);
            }
          }
        });
    __syncthreads();
    int64_t total;
    block_excl_scan1(mine, red, &total);
    if (threadIdx.x == 0) cnt[t] = total;
    if (want_blk && lds_blk)
      for (int64_t i = threadIdx.x; i < nblk; i += blockDim.x) dst[i] = lblk[i];
    __syncthreads();
  }
}

// ------------------------------------------------------------------ count: bitmap
// One workgroup per heavy column; an LDS bitmap over (a chunk of) the row
// space marks every row that receives a product.  Popcounts give the exact
// column count and the per-row-block counts used to cut parts; the bitmap is
// kept in HBM for the numeric phase.  One pass does all of that and clears the
// bitmap for the next column: a lane takes 16 bytes, a wave 8192 rows, which
// lie in one row block (rbshift >= 13 for every value type at the default part
// budget), so a wave adds up once per 8192 rows.  (Separate passes of 4-byte
// words with a wave sum per 2048 rows issued a third of the kernel's
// instructions, and issuing them is what bounds it.)
template <bool OFF32>
using BitmapRanges = RangeLdsT<kQChunkWide, kCountWin, OFF32, false>;  // heavy columns have many B entries
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <bool OFF32>
__global__ void __launch_bounds__(1024, 8) k_count_bitmap(Operand B, ProdSrc S, const int32_t* list,
                                                       const int64_t* binoff, int64_t m, int chunk_log2, int rbshift,
                                                       int64_t nblk, uint32_t* blkcnt, unsigned long long* cnt,
                                                       uint32_t* gbm, int64_t gwords, unsigned long long* qctr) {
  extern __shared__ __align__(16) unsigned char lds[];
  uint32_t* bm = (uint32_t*)lds;
  u32x4* bm4 = (u32x4*)lds;
  // a multiple of the row block and of the 128 rows of one 16-byte store: a chunk's
  // last store would else reach into the next chunk's rows, or the next column's bitmap
  const int64_t chunk_rows = 1ll << chunk_log2;
  const int64_t nchunks = (m + chunk_rows - 1) >> chunk_log2;
  const int blk_per_chunk = (int)(chunk_rows >> rbshift);
  const int all4 = (int)((chunk_rows + 127) >> 7);
  uint32_t* lblk = bm + 4 * all4;
  __shared__ int64_t red[1024 / kWave + 1];
  __shared__ BitmapRanges<OFF32> s_rng;
  __shared__ unsigned s_tot;
  const int64_t beg = binoff[0], end = binoff[kBinHash0];
  const int64_t ncols = end - beg;
  // workgroup w works on row chunk w mod nchunks (the grid is a multiple of
  // nchunks): workgroups are placed on the XCDs round robin, so each XCD's L2
  // serves one slice of A's rows.  The chunk's columns are handed out one at
  // a time by its counter qctr[chunk] (zero at launch), in list order, which
  // puts the heaviest columns first.
  const int64_t chunk = blockIdx.x % nchunks;
  const int64_t c0 = chunk * chunk_rows;
  const int64_t c1 = c0 + chunk_rows < m ? c0 + chunk_rows : m;
  const uint32_t span = (uint32_t)(c1 - c0);
  const int words4 = (int)((span + 127) >> 7);
  const int64_t bfirst = c0 >> rbshift;
  __shared__ int64_t s_ci;
  for (int i = threadIdx.x; i < all4; i += blockDim.x) bm4[i] = u32x4{0u, 0u, 0u, 0u};
  for (int i = threadIdx.x; i < blk_per_chunk; i += blockDim.x) lblk[i] = 0;
  for (;;) {
    if (threadIdx.x == 0) {
      s_ci = (int64_t)atomicAdd(&qctr[chunk], 1ull);
      s_tot = 0;
    }
    __syncthreads();
    const int64_t ci = s_ci;
    if (ci >= ncols) break;
    const int64_t pos = beg + ci;
    const int32_t t = list[pos];
    const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
    uint32_t* dst = blkcnt + (pos - beg) * nblk;
    block_products<4, int, false, false>(
        S, nullptr, nullptr, b0, b1, (int32_t)c0, (int32_t)c1, nchunks == 1, s_rng, red, nullptr, nullptr,
        [&](const int32_t(&r)[4], const int(&)[4], const int(&)[4]) {
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const uint32_t d = (uint32_t)(r[u] - (int32_t)c0);
            if (d < span) atomicOr(&bm[d >> 5], 1u << (d & 31));
          }
        });
    // (block_products ends with a barrier)
    // rows of gbm are 16-byte aligned: gwords and c0 / 32 are multiples of 4
    u32x4* g = gbm ? (u32x4*)(gbm + ci * gwords + (c0 >> 5)) : nullptr;
    const int lane = lane_id();
    for (int i0 = (int)threadIdx.x - lane; i0 < words4; i0 += blockDim.x) {
      const int i = i0 + lane;
      u32x4 v{0u, 0u, 0u, 0u};
      if (i < words4) {
        v = bm4[i];
        bm4[i] = u32x4{0u, 0u, 0u, 0u};
        // streaming (non-temporal) stores: the bitmaps are read back only by the
        // numeric phase, so they need not displace A's gathered entries from L2
        if (g) __builtin_nontemporal_store(v, g + i);
      }
      if (rbshift >= 13) {
        const int pc = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
        const int sum = __builtin_amdgcn_readlane(wave_incl_scan(pc), 63);
        if (lane == 0 && sum) {
          atomicAdd(&lblk[((int64_t)i0 * 128) >> rbshift], (uint32_t)sum);
          atomicAdd(&s_tot, (unsigned)sum);
        }
      } else if (rbshift >= 7) {
        // row blocks of 2^(rbshift - 7) lanes: the last lane of each adds its block's sum
        const int pc = __popc(v.x) + __popc(v.y) + __popc(v.z) + __popc(v.w);
        const int g = 1 << (rbshift - 7);
        const int incl = wave_incl_scan(pc);
        const int before = __shfl(incl, (lane - g) & (kWave - 1));
        const int sum = lane >= g ? incl - before : incl;
        if ((lane & (g - 1)) == g - 1 && sum) {
          atomicAdd(&lblk[((int64_t)i * 128) >> rbshift], (uint32_t)sum);
          atomicAdd(&s_tot, (unsigned)sum);
        }
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (const int pc = __popc(v[k])) {
            atomicAdd(&lblk[((int64_t)i * 128 + k * 32) >> rbshift], (uint32_t)pc);
            atomicAdd(&s_tot, (unsigned)pc);
          }
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < blk_per_chunk; i += blockDim.x) {
      if (bfirst + i < nblk) dst[bfirst + i] = lblk[i];
      lblk[i] = 0;
    }
    if (threadIdx.x == 0 && s_tot) atomicAdd(&cnt[t], (unsigned long long)s_tot);
  }
}

// ------------------------------------------------------------------ parts
struct Part {
  int64_t off;   // first output position of the part in C
  int32_t t;     // slot of B / output column
  int32_t c;     // outputs in the part
  int32_t r0, r1;  // row range [r0, r1)
  int32_t mode;  // bit 0: 0 = bitmap, 1 = hash; bit 1: [b0, b0 + nb) indexes the bucket list; bit 2: notes rows
  int32_t slice; // row slice of the part (work queue), nslice = any
  int32_t bmi;   // index of the column's stored row bitmap, -1 if none
  int32_t nb;    // B entries of the column: [b0, b0 + nb) (or the part's bucket)
  int64_t b0;
};

struct PartCfg {
  int64_t L;       // LDS bytes per part
  int64_t m;
  int32_t sz;      // value bytes (0: pattern only)
  int32_t rbshift;
  int64_t nblk;
  int64_t slice_blocks;  // row blocks per slice (parts never straddle slices); 0: one slice
  int32_t nslice;
  int32_t hash_max;  // most outputs of a hash-mode part that fits L (0: none)
  int64_t hash_span; // most rows it may span (set per cut column, see span_limit)
  int32_t note;      // bytes per output that parts leave for noted rows
  int32_t pad;
};

__device__ __forceinline__ int64_t bitmap_bytes(const PartCfg& p, int64_t span, int64_t c) {
  const int32_t w = (int32_t)((span + 63) >> 6);  // below 2^25
  return (int64_t)w * 8 + ((w * 2 + 7) & ~7) + c * (p.sz > 4 ? p.sz : 4) + 64;
}
__device__ __forceinline__ bool bitmap_ok(const PartCfg& p, int64_t span, int64_t c) {
  return c < 65536 && bitmap_bytes(p, span, c) <= p.L;
}
// Bitmap mode with the products' rows noted beside the values: 2 more bytes per
// output (see k_numeric_parts).
__device__ __forceinline__ bool noted_ok(const PartCfg& p, int64_t span, int64_t c) {
  return c < 65536 && bitmap_bytes(p, span, c) + p.note * c <= p.L;
}
// Rows a hash-mode part may span for the two-level rank (longer: sorted).
constexpr int64_t kRankSpan = 1ll << 20;

__host__ __device__ inline int64_t hash_bytes(int64_t p2, int64_t sz) {  // p2: a power of two, at least 64
  const int64_t S = 2 * p2;
  return S * 4 + ((S * sz + 7) & ~7ll) + p2 * 10 + (kRankSpan >> 9) + (kRankSpan >> 11) + 64;
}
__device__ __forceinline__ bool hash_ok(const PartCfg& p, int64_t span, int64_t c) {
  return c <= p.hash_max && span <= p.hash_span;
}

// Most rows of the hash parts of a column with c outputs.  Parts of more than kRankSpan
// rows sort their rows, so the column is rather cut there, unless that makes more than
// three times the parts that its outputs need.  Cut | sorted: 100,000 columns of 2000
// outputs (one part's worth) over 2^21 rows 6.6 | 9.3 ms, 2^21.5 (three spans) 7.9 | 9.3,
// 2^22 (four) 9.8 | 9.3, 2^23 16.8 | 9.4; 300 of 30,000 (15 parts) over 2^24 rows, 16 spans,
// 0.52 | 0.74, 2^25 0.81 | 0.94; R-MAT scale 23 with 2 edges a vertex squared 232 | 243,
// by this rule 209.
__device__ __forceinline__ int64_t span_limit(const PartCfg& p, int64_t c) {
  const int64_t spans = (p.m + kRankSpan - 1) / kRankSpan;
  const int64_t need = p.hash_max > 0 ? ((uint32_t)c + (uint32_t)p.hash_max - 1) / (uint32_t)p.hash_max : 0;
  return spans <= 3 * need ? kRankSpan : p.m;
}

__device__ __forceinline__ int choose_mode(const PartCfg& p, int64_t span, int64_t c) {
  const bool bok = bitmap_ok(p, span, c), hok = hash_ok(p, span, c);
  if (bok && hok) {
    const int64_t lg = c > 1 ? ceil_log2_u64((uint64_t)c) : 1;
    const int64_t bitmap_cost = ((span + 63) >> 6) * 3;
    const int64_t hash_cost = c * lg * (lg + 1) / 2;
    return bitmap_cost <= hash_cost ? 0 : 1;
  }
  return bok ? 0 : 1;
}

// Whether the parts of a column note a row with every product (see k_numeric_parts):
// a store per product, against a walk of the bitmap per output.  4096 columns of d
// products from each of d columns of A over 4096 rows, f64, with notes | without: 4
// products an output (d = 128) 377 | 395 us, 9 563 | 575, 16 807 | 796, 36 1568 | 1506,
// 64 2517 | 2393 (f32 7779 | 6405).
constexpr int64_t kNoteMost = 16;
__device__ __forceinline__ int note_mode(int64_t mults, int64_t c) { return mults <= kNoteMost * c ? 4 : 0; }

// Cuts one column into parts, greedily over its row blocks: a part grows while
// it still fits the LDS budget in one of the two modes (in bitmap mode with the
// noted rows; a single row block may go without).  One wave: its lanes
// test 64 ends of the part at once (whether a part fits only changes from yes
// to no as it grows).  blk: the column's row-block counts, in LDS or global
// memory; with PREF, their inclusive prefix sums.  Returns the number of parts;
// writes them if out is given.
template <bool PREF>
__device__ int64_t cut_parts(const PartCfg& p, const uint32_t* blk, int32_t t, int64_t base_off, Part* out, int note,
                             int32_t bmi, int64_t b0, int32_t nb, unsigned* err) {
  const int64_t RB = 1ll << p.rbshift;
  const int lane = lane_id();
  const int32_t nblk = (int32_t)p.nblk, sb = (int32_t)p.slice_blocks;
  int64_t np = 0, run = 0;
  uint32_t before = 0;  // outputs of row blocks [0, b)
  for (int32_t b = 0; b < nblk;) {
    uint32_t c = 0;  // outputs of row blocks [b, e)
    int32_t e = b;
    for (int f = kWave; f == kWave;) {
      const int32_t i = e + lane;
      const uint32_t x = i < nblk ? blk[i] : 0;
      const uint32_t ci = PREF ? x - before : c + (uint32_t)wave_incl_scan((int32_t)x);
      const int64_t r1 = (i + 1) * RB < p.m ? (i + 1) * RB : p.m;
      const bool fits = i < nblk && (i == b || (!(sb && i % sb == 0) &&
                                                (hash_ok(p, r1 - b * RB, ci) || noted_ok(p, r1 - b * RB, ci))));
      const uint64_t no = __ballot(!fits);
      f = no ? __ffsll((long long)no) - 1 : kWave;
      if (f > 0) c = (uint32_t)__builtin_amdgcn_readlane((int)ci, f - 1);
      e += f;
    }
    before += c;
    if (c > 0) {
      const int64_t r0 = b * RB;
      const int64_t r1 = e * RB < p.m ? e * RB : p.m;
      if (lane == 0) {
        if (!bitmap_ok(p, r1 - r0, c) && !hash_ok(p, r1 - r0, c)) atomicOr(err, 4u);
        if (out) {
          Part P;
          P.off = base_off + run;
          P.t = t;
          P.c = (int32_t)c;
          P.r0 = (int32_t)r0;
          P.r1 = (int32_t)r1;
          P.mode = choose_mode(p, r1 - r0, c) | note;
          P.slice = p.slice_blocks ? (int32_t)(b / p.slice_blocks) : 0;
          P.bmi = bmi;
          P.b0 = b0;
          P.nb = nb;
          out[np] = P;
        }
      }
      ++np;
      run += c;
    }
    b = e;
  }
  return np;
}

// Number of parts of every column above the mid ones (list positions
// [0, npos)), or the parts themselves (parts given).  The first cut_blocks
// workgroups take the columns with row-block counts, a wave each with the
// counts in LDS (a thread each, walking them one by one in memory, took 0.21 ms
// on R-MAT scale 20, and 57 us on 128 long columns); the others the rest, a
// thread each.
// In the counting pass, setup_acc (if given) receives the sums over the cut
// columns of (B entries x parts) and of their multiplications, which tell
// how many range set-ups the multi-part launch makes per product.
constexpr int kCutBlk = 1024;  // row blocks held in LDS (more are read from memory)

__global__ void __launch_bounds__(256) k_parts(Operand B, PartCfg p, PartCfg ps, const int32_t* list, int64_t npos,
                                               int64_t multi_begin, int64_t multi_end, unsigned cut_blocks, int64_t nbm,
                                               const int64_t* cnt, const int64_t* off, const uint32_t* blkcnt,
                                               int64_t* nparts, const int64_t* poff, Part* parts, const int64_t* mults,
                                               unsigned long long* setup_acc, unsigned* err) {
  __shared__ uint32_t s_blk[4][kCutBlk];  // prefix sums of the counts
  unsigned long long my_setup = 0, my_mults = 0;
  // a column in one part
  auto whole = [&](int64_t pos, int32_t t, int64_t c, const PartCfg& q) {
    if (!parts) {
      if (!(bitmap_ok(q, q.m, c) || hash_ok(q, q.m, c))) atomicOr(err, 4u);
      return;
    }
    Part P;
    P.off = off[t];
    P.t = t;
    P.c = (int32_t)c;
    P.r0 = 0;
    P.r1 = (int32_t)q.m;
    P.mode = choose_mode(q, q.m, c) | note_mode(mults[t], c);
    P.slice = q.nslice;  // full row range: any queue
    P.bmi = pos - multi_begin < nbm ? (int32_t)(pos - multi_begin) : -1;
    P.b0 = slot_begin(B, t);
    P.nb = (int32_t)(slot_begin(B, t + 1) - P.b0);
    parts[poff[pos]] = P;
  };
  if (blockIdx.x < cut_blocks) {
    const int w = threadIdx.x / kWave, lane = lane_id();
    for (int64_t pos = multi_begin + (int64_t)blockIdx.x * 4 + w; pos < multi_end; pos += (int64_t)cut_blocks * 4) {
      const int32_t t = list[pos];
      const int64_t c = cnt[t];
      int64_t np = c > 0;
      PartCfg q = p;
      q.hash_span = span_limit(p, c);
      if (c > 0 && !(bitmap_ok(q, q.m, c) || hash_ok(q, q.m, c))) {
        const int64_t cb0 = slot_begin(B, t), nb = slot_begin(B, t + 1) - cb0;
        const uint32_t* blk = blkcnt + (pos - multi_begin) * p.nblk;
        if (p.nblk <= kCutBlk) {
          uint32_t carry = 0;
          for (int i0 = 0; i0 < p.nblk; i0 += kWave) {
            const int i = i0 + lane;
            const uint32_t s = carry + (uint32_t)wave_incl_scan(i < p.nblk ? (int32_t)blk[i] : 0);
            if (i < p.nblk) s_blk[w][i] = s;
            carry = (uint32_t)__builtin_amdgcn_readlane((int)s, kWave - 1);
          }
          wave_sync();
        }
        Part* out = parts ? parts + poff[pos] : nullptr;
        const int32_t bmi = pos - multi_begin < nbm ? (int32_t)(pos - multi_begin) : -1;
        const int note = parts ? note_mode(mults[t], c) : 0;
        np = p.nblk <= kCutBlk ? cut_parts<true>(q, s_blk[w], t, off[t], out, note, bmi, cb0, (int32_t)nb, err)
                               : cut_parts<false>(q, blk, t, off[t], out, note, bmi, cb0, (int32_t)nb, err);
        if (setup_acc && np > 1 && lane == 0) {
          my_setup += (unsigned long long)nb * (unsigned long long)np;
          my_mults += (unsigned long long)mults[t];
        }
        wave_sync();
      } else if (c > 0 && lane == 0) {
        whole(pos, t, c, q);
      }
      if (!parts && lane == 0) nparts[pos] = np;
    }
  } else {
    const int64_t stride = (int64_t)(gridDim.x - cut_blocks) * blockDim.x;
    for (int64_t pos = multi_end + (int64_t)(blockIdx.x - cut_blocks) * blockDim.x + threadIdx.x; pos < npos;
         pos += stride) {
      const int32_t t = list[pos];
      const int64_t c = cnt[t];
      if (c > 0) whole(pos, t, c, ps);
      if (!parts) nparts[pos] = c > 0;
    }
  }
  if (setup_acc) {  // one pair of atomics per workgroup
    __shared__ unsigned long long s_acc[2];
    if (threadIdx.x < 2) s_acc[threadIdx.x] = 0;
    __syncthreads();
    if (my_setup) atomicAdd(&s_acc[0], my_setup);
    if (my_mults) atomicAdd(&s_acc[1], my_mults);
    __syncthreads();
    if (threadIdx.x < 2 && s_acc[threadIdx.x]) atomicAdd(&setup_acc[threadIdx.x], s_acc[threadIdx.x]);
  }
}

// ------------------------------------------------------------------ buckets
// With a tall-skinny B, every part of a cut column walks all of the column's
// B entries although the few rows of each A(:,k) reach few parts.  Bucket
// mode lists, per part, only the B entries whose A column has rows in the
// part's row range: about one list entry per multiplication instead of one
// range set-up per B entry and part.
//   k_bucket_map:   per cut column, the part of every row block (-1: none);
//   k_bucket<FILL>: per B entry of a cut column, each part it reaches gets a
//                   count (FILL false) or the entry's index (FILL true);
//   k_bucket_parts: points every part of a cut column at its bucket.
// Cut columns are the list positions [multi_begin, multi_end) with more
// than one part.
__global__ void k_bucket_map(PartCfg p, const int64_t* np, const int64_t* poff, int64_t multi_begin,
                             int64_t multi_end, const Part* parts, int32_t* map) {
  for (int64_t pos = multi_begin + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; pos < multi_end;
       pos += (int64_t)gridDim.x * blockDim.x) {
    int32_t* mp = map + (pos - multi_begin) * p.nblk;
    for (int64_t b = 0; b < p.nblk; ++b) mp[b] = -1;
    if (np[pos] <= 1) continue;
    for (int64_t i = poff[pos]; i < poff[pos + 1]; ++i) {
      const int64_t bl0 = parts[i].r0 >> p.rbshift;
      const int64_t bl1 = ((int64_t)parts[i].r1 + (1ll << p.rbshift) - 1) >> p.rbshift;
      for (int64_t b = bl0; b < bl1 && b < p.nblk; ++b) mp[b] = (int32_t)(i - poff[pos]);
    }
  }
}

// One workgroup takes a strided share of one cut column's B entries and
// counts, per part, in LDS: the counting pass then adds its counts to bcnt,
// the filling pass reserves a range of each part's bucket (one atomic per
// part and workgroup) and walks its B entries again to fill the ranges.
// Columns with more than kBucketLds parts use global atomics per entry.
constexpr int kBucketLds = 4096;

template <bool FILL>
__global__ void __launch_bounds__(256) k_bucket(Operand B, ProdSrc S, PartCfg p, const int32_t* list,
                                                const int64_t* np, const int64_t* poff, int64_t multi_begin,
                                                int64_t multi_end, const Part* parts, const int32_t* map,
                                                unsigned* bcnt, const int64_t* boff, unsigned* bfill,
                                                int32_t* qlist, int64_t qcap, unsigned* err) {
  __shared__ unsigned s_cnt[kBucketLds];
  __shared__ int64_t s_base[FILL ? kBucketLds : 1];
  for (int64_t pos = multi_begin + blockIdx.y; pos < multi_end; pos += gridDim.y) {
    const int64_t npp = np[pos];
    if (npp <= 1) continue;
    const int32_t t = list[pos];
    const int64_t cb0 = slot_begin(B, t), cb1 = slot_begin(B, t + 1);
    const int64_t pbeg = poff[pos];
    const int32_t* mp = map + (pos - multi_begin) * p.nblk;
    const bool local = npp <= kBucketLds;
    // calls f(j) for every part j of the column that B entry q reaches
    auto reach = [&](int64_t q, auto&& f) {
      const int64_t a0 = S.a0[q];
      const int32_t alen = S.alen[q];
      const int32_t sid = S.splits ? S.split[q] : -1;
      if (sid >= 0 && alen > 2 * npp) {  // long A column: probe each part through the split table
        const int32_t* sp = S.splits + (int64_t)sid * S.sstride;
        for (int64_t j = 0; j < npp; ++j) {
          const Part& pj = parts[pbeg + j];
          const int32_t e0 = sp[pj.r0 >> S.rbshift];
          const int32_t e1 = sp[pj.r1 >= S.m ? S.sstride - 1 : (pj.r1 >> S.rbshift)];
          if (e1 > e0) f(j);
        }
      } else {  // short A column: walk its rows (sorted, so its parts come in order)
        int32_t last = -1;
        for (int32_t e = 0; e < alen; ++e) {
          const int32_t j = mp[S.air[a0 + e] >> S.rbshift];
          if (j >= 0 && j != last) {
            f(j);
            last = j;
          }
        }
      }
    };
    const int64_t q0 = cb0 + blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int64_t qs = (int64_t)gridDim.x * blockDim.x;
    if (!local) {  // uniform for the workgroup
      for (int64_t q = q0; q < cb1; q += qs)
        reach(q, [&](int64_t j) {
          if (FILL) {
            const int64_t at = boff[pbeg + j] + atomicAdd(&bfill[pbeg + j], 1u);
            if (at < qcap)
              qlist[at] = (int32_t)q;
            else
              atomicOr(err, 32u);
          } else {
            atomicAdd(&bcnt[pbeg + j], 1u);
          }
        });
      continue;
    }
    for (int64_t j = threadIdx.x; j < npp; j += blockDim.x) s_cnt[j] = 0;
    __syncthreads();
    for (int64_t q = q0; q < cb1; q += qs) reach(q, [&](int64_t j) { atomicAdd(&s_cnt[j], 1u); });
    __syncthreads();
    for (int64_t j = threadIdx.x; j < npp; j += blockDim.x) {
      const unsigned c = s_cnt[j];
      if (!FILL) {
        if (c) atomicAdd(&bcnt[pbeg + j], c);
      } else {
        s_base[j] = c ? boff[pbeg + j] + atomicAdd(&bfill[pbeg + j], c) : 0;
        s_cnt[j] = 0;
      }
    }
    __syncthreads();
    if (FILL) {
      for (int64_t q = q0; q < cb1; q += qs)
        reach(q, [&](int64_t j) {
          const int64_t at = s_base[j] + atomicAdd(&s_cnt[j], 1u);
          if (at < qcap)
            qlist[at] = (int32_t)q;
          else
            atomicOr(err, 32u);
        });
      __syncthreads();
    }
  }
}

__global__ void k_bucket_parts(const int64_t* np, const int64_t* poff, int64_t multi_begin, int64_t multi_end,
                               const unsigned* bcnt, const int64_t* boff, Part* parts) {
  for (int64_t pos = multi_begin + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; pos < multi_end;
       pos += (int64_t)gridDim.x * blockDim.x) {
    if (np[pos] <= 1) continue;
    for (int64_t i = poff[pos]; i < poff[pos + 1]; ++i) {
      parts[i].b0 = boff[i];
      parts[i].nb = (int32_t)bcnt[i];
      parts[i].mode |= 2;
    }
  }
}

struct LoadBucket {
  const unsigned* p;
  __device__ int64_t operator()(int64_t i) const { return (int64_t)p[i]; }
};

// ------------------------------------------------------------------ numeric: parts
// Most parts per work-queue ticket.  A launch takes one part per ticket until
// every workgroup of its grid would get two of them: with fewer parts a ticket
// of four leaves workgroups idle while others take four parts in turn (R-MAT
// scale 14: 176 parts on 44 of 176 workgroups, 172 us; scale 20 has 1900 parts
// per workgroup and keeps four, which save ticket round trips).
constexpr int kPartBatch = 4;
constexpr int kMaxQueues = 65;  // of the multi-part launch: at most 64 row slices and a shared queue

template <typename T>
__device__ __forceinline__ void block_bitonic_sort(uint64_t* a, int n2) {
  for (int k = 2; k <= n2; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = threadIdx.x; i < (n2 >> 1); i += blockDim.x) {
        const int lo = 2 * i - (i & (j - 1));
        const int hi = lo + j;
        const bool asc = (lo & k) == 0;
        const uint64_t x = a[lo], y = a[hi];
        if ((x > y) == asc) {
          a[lo] = y;
          a[hi] = x;
        }
      }
      __syncthreads();
    }
  }
}

// One workgroup per part (dynamic work queue).  Bitmap mode: mark rows,
// popcount prefix gives each row its rank = output position, accumulate
// values by rank, write rows and values in order.  Hash mode: accumulate
// into an open-addressing table, then rank its rows by a two-level bitmap
// (up to kRankSpan rows) or sort (row, slot) keys.
template <bool OFF32>
using PartRanges = RangeLdsT<kQChunkWide, kNumWin, OFF32, true>;

// Static LDS of the kernel, rounded up: with 32-bit positions two workgroups
// of the default 72 KiB part budget share a CU's 160 KiB.
constexpr int64_t kPartLds32 = 8192, kPartLds64 = 10240;
static_assert(sizeof(PartRanges<true>) + 480 <= kPartLds32 && sizeof(PartRanges<false>) + 480 <= kPartLds64, "static LDS");

template <int SR, typename T, bool OFF32>
__global__ void __launch_bounds__(1024) k_numeric_parts(Operand A, Operand B, ProdSrc S,
                                                        const Part* parts, const int64_t* qoff,
                                                        int64_t plo, int64_t phi, int nq, int nhome, int batch,
                                                        unsigned long long* qctr,
                                                        const uint64_t* gbm, int64_t gbm_words,
                                                        const int32_t* qlist, int64_t part_lds, int32_t* cir, T* cnum,
                                                        unsigned* err) {
  using SR_ = Semiring<SR, T>;
  constexpr bool kVal = SR != SPX_OR_AND;
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ int64_t s_pi;
  __shared__ int s_nbat;
  __shared__ Part s_batch[kPartBatch];
  __shared__ int64_t red[1024 / kWave + 1];
  __shared__ int32_t red32[1024 / kWave + 1];
  __shared__ unsigned s_ctr;
  __shared__ PartRanges<OFF32> s_rng;
  const T* an = (const T*)A.num;
  const T* bn = (const T*)B.num;
  // work queues: queue k holds parts [qoff[k], qoff[k+1]) (without qoff: one
  // queue of [plo, phi), its bounds passed by value); a workgroup
  // starts with its home queue (blockIdx.x % nhome: workgroups are placed on
  // the XCDs round robin, so one queue's rows of A stay in one L2), then
  // takes the shared queue nq-1, then helps the others.
  const int home = nhome > 1 ? (int)(blockIdx.x % nhome) : 0;
  // A ticket is a batch of up to `batch` (<= kPartBatch) consecutive parts
  // (often of one column), whose descriptors are loaded together.
  int qi = 0;
  for (;;) {
    if (threadIdx.x == 0) {
      int64_t got = -1;
      int nbat = 0;
      while (qi < nq) {
        const int q = qi == 0 ? home : (qi == 1 ? nq - 1 : (home + qi - 1) % (nq - 1));
        const int64_t qlo = qoff ? qoff[q] : plo, qhi = qoff ? qoff[q + 1] : phi;
        const int64_t first = qlo + (int64_t)atomicAdd(&qctr[q], (unsigned long long)batch);
        if (first < qhi) {
          got = first;
          nbat = (int)(qhi - first < batch ? qhi - first : batch);
          break;
        }
        ++qi;
      }
      s_pi = got;
      s_nbat = nbat;
    }
    __syncthreads();
    const int64_t pfirst = s_pi;
    const int nbat = s_nbat;
    if (pfirst < 0) break;
    if ((int)threadIdx.x < nbat) s_batch[threadIdx.x] = parts[pfirst + threadIdx.x];
    __syncthreads();
    for (int bi = 0; bi < nbat; ++bi) {
    Part P;
    {
      const Part& Q = s_batch[bi];
      P.off = uniform(Q.off);
      P.c = uniform(Q.c);
      P.r0 = uniform(Q.r0);
      P.r1 = uniform(Q.r1);
      P.mode = uniform(Q.mode);
      P.bmi = uniform(Q.bmi);
      P.nb = uniform(Q.nb);
      P.b0 = uniform(Q.b0);
    }
    const int64_t b0 = P.b0, b1 = P.b0 + P.nb;
    const int32_t* qx = (P.mode & 2) ? qlist : nullptr;  // a bucketed part visits only its bucket
    const int64_t span = (int64_t)P.r1 - P.r0;
    const bool full = (P.r0 == 0 && P.r1 == (int32_t)A.m);
    const int c = P.c;
    if ((P.mode & 1) == 0) {
      const int W = (int)((span + 63) >> 6);
      uint64_t* bm = (uint64_t*)lds;
      uint16_t* pre = (uint16_t*)(bm + W);
      T* vals = (T*)(lds + W * 8 + ((W * 2 + 7) & ~7));
      // Rows in rank order.  Where the part leaves room for them (2 bytes per output) and
      // the column has not too many products for an output (note_mode), every product
      // notes the low 16 bits of its row beside its value; the high bits follow from the
      // ranks at the multiples of 65536 rows.  Else, and for patterns, the rows are read
      // off the bitmap: its words hold one or two rows each, so lanes wait for the
      // fullest word at every step (about 50 vector instructions per 64 outputs against 12).
      uint16_t* low = (uint16_t*)(vals + c);
      const bool noted = kVal && (P.mode & 4) && (char*)(low + c) <= (char*)lds + part_lds;
      // rank of each product's row: all bitmap words first, then the adds
      auto acc = [&](const int32_t (&r)[8], const T (&a)[8], const T (&bv)[8]) {
        uint64_t w[8];
        int pr[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const uint32_t d = (uint32_t)(r[u] - P.r0);
          const uint32_t wi = d < (uint32_t)span ? d >> 6 : 0u;
          w[u] = bm[wi];
          pr[u] = pre[wi];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const uint32_t d = (uint32_t)(r[u] - P.r0);
          const int rank = pr[u] + __popcll(w[u] & ((1ull << (d & 63)) - 1ull));
          if (d < (uint32_t)span && rank < c) {
            SR_::lds_acc(&vals[rank], SR_::mul(a[u], bv[u]));
            if (noted) low[rank] = (uint16_t)d;  // the same from every product of the row
          }
        }
      };
      // the row set: the count phase's stored bitmap, else marked here
      const bool stored = gbm != nullptr && P.bmi >= 0;
      const int qchunk = (int)blockDim.x < S.qchunk ? (int)blockDim.x : S.qchunk;
      // A stored part of one chunk loads its ranges and its bitmap together and numbers
      // both in one scan: the part waits on a chain of memory latencies (two workgroups
      // fit a CU), and this takes one of them and three barriers out.
      const bool fused = kVal && stored && b1 - b0 <= qchunk;
      FirstChunk marked{0, false};
      int64_t at = 0;
      int32_t len = 0;
      T bq = T(0);
      if (fused) {
        if ((int)threadIdx.x < P.nb) {
          const int64_t q = qx ? (int64_t)qx[b0 + threadIdx.x] : b0 + threadIdx.x;
          load_range<T, SR_::kUsesB>(S, bn, q, P.r0, P.r1, full, at, len, bq);
        }
        for (int k = threadIdx.x; k < kNumWin; k += blockDim.x) s_rng.bits[k] = 0;
      }
      if (stored) {
        const uint64_t* g = gbm + (int64_t)P.bmi * gbm_words + (P.r0 >> 6);
        for (int i0 = threadIdx.x; i0 < W; i0 += 8 * blockDim.x) {  // 8 loads in flight per thread
          uint64_t v[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int i = i0 + k * (int)blockDim.x;
            v[k] = i < W ? g[i] : 0ull;
          }
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int i = i0 + k * (int)blockDim.x;
            if (i < W) bm[i] = v[k];
          }
        }
      } else {
        for (int i = threadIdx.x; i < W; i += blockDim.x) bm[i] = 0;
      }
      if constexpr (kVal)
        for (int i = threadIdx.x; i < c; i += blockDim.x) vals[i] = SR_::ident();
      __syncthreads();
      if (!stored) {
        block_products<8, T, false, SR_::kUsesB>(
            S, an, bn, b0, b1, P.r0, P.r1, full, s_rng, red, qx, &marked, [&](const int32_t(&r)[8], const T(&)[8], const T(&)[8]) {
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                const uint32_t d = (uint32_t)(r[u] - P.r0);
                if (d < (uint32_t)span) atomicOr((unsigned long long*)&bm[d >> 6], 1ull << (d & 63));
              }
            });
      }
      // exclusive popcount prefix per word (and the numbers of the ranges)
      const int per = (W + blockDim.x - 1) / blockDim.x;
      const int w0 = threadIdx.x * per;
      const int w1 = w0 + per < W ? w0 + per : W;
      int32_t s = 0, tot;
      for (int i = w0; i < w1; ++i) s += __popcll(bm[i]);
      int64_t rsum = 0, rpre = 0;
      int32_t run = block_excl_scan1(s, red32, &tot, range_word(len), red, &rpre, &rsum);
      for (int i = w0; i < w1; ++i) {
        pre[i] = (uint16_t)run;
        run += __popcll(bm[i]);
      }
      if (threadIdx.x == 0 && tot != c) atomicOr(err, 8u);
      if constexpr (kVal) {
        if (!fused) __syncthreads();
        // the chunks of ranges: those loaded above, those the marking pass left in LDS,
        // or loaded now
        for (int64_t qc = b0; qc < b1; qc += qchunk) {
          int64_t total = marked.total, ex = 0;
          int32_t rk = 0;
          if (!marked.all) {
            if (!fused) {
              for (int k = threadIdx.x; k < kNumWin; k += blockDim.x) s_rng.bits[k] = 0;
              len = 0;
              if (qc + threadIdx.x < b1 && (int)threadIdx.x < qchunk) {
                const int64_t q = qx ? (int64_t)qx[qc + threadIdx.x] : qc + threadIdx.x;
                load_range<T, SR_::kUsesB>(S, bn, q, P.r0, P.r1, full, at, len, bq);
              }
              rpre = block_excl_scan1(range_word(len), red, &rsum);
            }
            total = rsum & (((int64_t)1 << kRangeBits) - 1);
            ex = rpre & (((int64_t)1 << kRangeBits) - 1);
            rk = (int32_t)(rpre >> kRangeBits);
            if (len > 0) {
              s_rng.base[rk] = (typename PartRanges<OFF32>::Off)(at - ex);
              if constexpr (SR_::kUsesB) reinterpret_cast<T*>(&s_rng.bval[rk])[0] = bq;
            }
          }
          product_tiles<8, T, SR_::kUsesA, SR_::kUsesB>(S, an, !marked.all, total, ex, len, rk, s_rng, acc);
        }
        // C is written once, coalesced: streaming stores keep the L2 for A's gathers
        // (a part's scattered hash-mode writes stay ordinary: streamed partial lines
        // cost more than they save)
        for (int i = threadIdx.x; i < c; i += blockDim.x) __builtin_nontemporal_store(vals[i], &cnum[P.off + i]);
        if (noted) {
          const int nhi = (int)((span - 1) >> 16);  // pre[1024 k]: rank of the first row at or above 65536 k
          int32_t hi = P.r0;
          int k = 0, next = nhi > 0 ? (int)pre[1024] : 0x7fffffff;
          for (int i = threadIdx.x; i < c; i += blockDim.x) {
            while (i >= next) {
              ++k;
              hi += 65536;
              next = k < nhi ? (int)pre[1024 * (k + 1)] : 0x7fffffff;
            }
            __builtin_nontemporal_store(hi + (int32_t)low[i], &cir[P.off + i]);
          }
          __syncthreads();
          continue;
        }
        __syncthreads();
      }
      if constexpr (!kVal) __syncthreads();
      // rows in rank order: staged in the value area, then written coalesced
      int32_t* rows = (int32_t*)vals;
      for (int i = w0; i < w1; ++i) {
        uint64_t word = bm[i];
        int rk = pre[i];
        while (word) {
          const int bit = __ffsll((long long)word) - 1;
          word &= word - 1;
          if (rk < c) rows[rk] = P.r0 + i * 64 + bit;
          ++rk;
        }
      }
      __syncthreads();
      for (int i = threadIdx.x; i < c; i += blockDim.x) __builtin_nontemporal_store(rows[i], &cir[P.off + i]);
      __syncthreads();
    } else {
      int p2 = 64;
      while (p2 < c) p2 <<= 1;
      const uint32_t Sz = 2u * p2;
      const int log2s = 31 - __clz(Sz);
      uint32_t* keys = (uint32_t*)lds;
      T* vals = (T*)(lds + Sz * 4);
      unsigned char* tail = lds + Sz * 4 + ((Sz * sizeof(T) * (kVal ? 1 : 0) + 7) & ~7u);
      // row ranks by a two-level bitmap (spans up to kRankSpan rows): level 1
      // marks the nonempty 64-row groups, level 2 holds one word per nonempty
      // group; popcount prefixes of both give each row its rank.  Longer spans
      // sort (row, slot) keys instead.
      const bool ranked = span <= kRankSpan;
      const int n1 = (int)((span + 4095) >> 12);
      uint64_t* l2w = (uint64_t*)tail;
      uint16_t* l2p = (uint16_t*)(tail + p2 * 8);
      uint64_t* l1w = (uint64_t*)(tail + p2 * 10);
      uint16_t* l1p = (uint16_t*)(tail + p2 * 10 + (kRankSpan >> 9));
      uint64_t* sortb = (uint64_t*)tail;
      // (Sz is a multiple of 128, so 16 bytes at a time)
      for (uint32_t i = threadIdx.x; i < Sz / 4; i += blockDim.x)
        reinterpret_cast<uint4*>(keys)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
      if constexpr (kVal)
        for (uint32_t i = threadIdx.x; i < Sz; i += blockDim.x) vals[i] = SR_::ident();
      if (ranked) {
        for (int i = threadIdx.x; i < p2; i += blockDim.x) l2w[i] = 0;
        for (int i = threadIdx.x; i < n1; i += blockDim.x) l1w[i] = 0;
      }
      if (threadIdx.x == 0) s_ctr = 0;
      __syncthreads();
      block_products<4, T, SR_::kUsesA, SR_::kUsesB>(
          S, an, bn, b0, b1, P.r0, P.r1, full, s_rng, red, qx, nullptr, [&](const int32_t(&r)[4], const T(&a)[4], const T(&bv)[4]) {
            uint32_t h[4], old[4];
            bool in[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {  // first probes of the four windows together
              in[u] = (uint32_t)(r[u] - P.r0) < (uint32_t)span;
              h[u] = hash_row(r[u], log2s);
              old[u] = in[u] ? atomicCAS(&keys[h[u]], ~0u, (uint32_t)r[u]) : (uint32_t)r[u];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (!in[u]) continue;
              const uint32_t key = (uint32_t)r[u];
              uint32_t at = h[u], was = old[u];
              // a loop over two scalars (with an exit that wrote to the arrays, the compiler
              // moved all of them at every probe: 2000 products took 23.4k cycles, 17.8k
              // without batched first probes)
              for (uint32_t left = Sz; was != ~0u && was != key && left; --left) {
                at = (at + 1) & (Sz - 1);
                was = atomicCAS(&keys[at], ~0u, key);
              }
              if (was != ~0u && was != key) {
                atomicOr(err, 16u);
                continue;
              }
              if constexpr (kVal) SR_::lds_acc(&vals[at], SR_::mul(a[u], bv[u]));
              if (ranked && was == ~0u) {  // a new row: level 1 marks its group
                const uint32_t g = (key - (uint32_t)P.r0) >> 6;
                atomicOr((unsigned long long*)&l1w[g >> 6], 1ull << (g & 63));
              }
            }
          });
      if (ranked) {
        int64_t ng;  // nonempty groups
        {
          const int per = (n1 + (int)blockDim.x - 1) / (int)blockDim.x;
          const int w0 = threadIdx.x * per, w1 = w0 + per < n1 ? w0 + per : n1;
          int64_t sum = 0;
          for (int w = w0; w < w1; ++w) sum += __popcll(l1w[w]);
          int64_t run = block_excl_scan1(sum, red, &ng);
          for (int w = w0; w < w1; ++w) {
            l1p[w] = (uint16_t)run;
            run += __popcll(l1w[w]);
          }
        }
        __syncthreads();
        // level 2: the rows of each nonempty group.  Threads hold the keys of
        // their slots from here on (eight each; a part with more writes straight
        // from the table below).
        const bool held = Sz <= 8 * blockDim.x;
        uint32_t key[8];
        auto group = [&](uint32_t k) {  // index of row k's group among the nonempty ones
          const uint32_t g = (k - (uint32_t)P.r0) >> 6;
          return (int)l1p[g >> 6] + __popcll(l1w[g >> 6] & ((1ull << (g & 63)) - 1ull));
        };
        if (held) {
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const uint32_t i = q * blockDim.x + threadIdx.x;
            uint4 v = make_uint4(~0u, ~0u, ~0u, ~0u);
            if (i < Sz / 4) v = reinterpret_cast<const uint4*>(keys)[i];
            key[4 * q] = v.x;
            key[4 * q + 1] = v.y;
            key[4 * q + 2] = v.z;
            key[4 * q + 3] = v.w;
          }
#pragma unroll
          for (int k = 0; k < 8; ++k)
            if (key[k] != ~0u) {
              const int gi = group(key[k]);
              if (gi < p2) atomicOr((unsigned long long*)&l2w[gi], 1ull << ((key[k] - (uint32_t)P.r0) & 63));
            }
        } else {
          for (uint32_t i = threadIdx.x; i < Sz; i += blockDim.x)
            if (keys[i] != ~0u) {
              const int gi = group(keys[i]);
              if (gi < p2) atomicOr((unsigned long long*)&l2w[gi], 1ull << ((keys[i] - (uint32_t)P.r0) & 63));
            }
        }
        __syncthreads();
        int64_t found;
        {
          const int n2 = ng < p2 ? (int)ng : p2;
          const int per = (n2 + (int)blockDim.x - 1) / (int)blockDim.x;
          const int w0 = threadIdx.x * per, w1 = w0 + per < n2 ? w0 + per : n2;
          int64_t sum = 0;
          for (int w = w0; w < w1; ++w) sum += __popcll(l2w[w]);
          int64_t run = block_excl_scan1(sum, red, &found);
          for (int w = w0; w < w1; ++w) {
            l2p[w] = (uint16_t)run;
            run += __popcll(l2w[w]);
          }
        }
        __syncthreads();
        if (threadIdx.x == 0 && found != c) atomicOr(err, 32u);
        auto rank_of = [&](uint32_t k) {  // output position of row k, c or more if it has none
          const int gi = group(k);
          return gi < p2 ? (int)l2p[gi] + __popcll(l2w[gi] & ((1ull << ((k - (uint32_t)P.r0) & 63)) - 1ull)) : c;
        };
        if (held) {
          // values and rows go through the LDS in rank order, over the table, so that
          // C is written coalesced (straight from the table, 64 lanes wrote to as many lines)
          T v[8];
          if constexpr (kVal) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
              v[k] = key[k] != ~0u ? vals[4 * ((k / 4) * blockDim.x + threadIdx.x) + k % 4] : T(0);
          }
          __syncthreads();
          T* vout = vals;  // 2 c values fit there, so c values and c rows do
          int32_t* rout = kVal ? (int32_t*)(vals + c) : (int32_t*)keys;
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            if (key[k] == ~0u) continue;
            const int rank = rank_of(key[k]);
            if (rank < c) {
              rout[rank] = (int32_t)key[k];
              if constexpr (kVal) vout[rank] = v[k];
            }
          }
          __syncthreads();
          for (int i = threadIdx.x; i < c; i += blockDim.x) {
            __builtin_nontemporal_store(rout[i], &cir[P.off + i]);
            if constexpr (kVal) __builtin_nontemporal_store(vout[i], &cnum[P.off + i]);
          }
        } else {
          for (uint32_t i = threadIdx.x; i < Sz; i += blockDim.x) {
            if (keys[i] == ~0u) continue;
            const int rank = rank_of(keys[i]);
            if (rank < c) {
              cir[P.off + rank] = (int32_t)keys[i];
              if constexpr (kVal) cnum[P.off + rank] = vals[i];
            }
          }
        }
      } else {
        for (uint32_t i = threadIdx.x; i < Sz; i += blockDim.x) {
          const uint32_t key = keys[i];
          if (key != 0xffffffffu) {
            const unsigned p = atomicAdd(&s_ctr, 1u);
            if ((int)p < p2) sortb[p] = ((uint64_t)key << 32) | i;
          }
        }
        __syncthreads();
        const int found = (int)s_ctr;
        if (threadIdx.x == 0 && found != c) atomicOr(err, 32u);
        for (int i = found + threadIdx.x; i < p2; i += blockDim.x) sortb[i] = ~0ull;
        __syncthreads();
        block_bitonic_sort<T>(sortb, p2);
        for (int i = threadIdx.x; i < c; i += blockDim.x) {
          const uint64_t k = sortb[i];
          cir[P.off + i] = (int32_t)(k >> 32);
          if constexpr (kVal) cnum[P.off + i] = vals[k & 0xffffffffu];
        }
      }
      __syncthreads();
    }
    }
  }
}

// ------------------------------------------------------------------ output pointers
// CSC output: cp[j] = start of column j.  For a DCSC B, column j's start is
// the offset of the first slot whose column id is >= j.
// Clears the exec's queue counters for the plan's next exec.
__device__ __forceinline__ void reset_queues(unsigned long long* qctr) {
  if (blockIdx.x == 0 && threadIdx.x <= kMaxQueues) qctr[threadIdx.x] = 0;
}

__global__ void k_write_csc_cp(Operand B, const int64_t* off, int64_t nslots, int64_t n, void* cp, int32_t ptr_t,
                               unsigned long long* qctr) {
  reset_queues(qctr);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j <= n; j += stride) {
    int64_t t = j;
    if (B.fmt == SPX_DCSC) {
      int64_t lo = 0, hi = nslots;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)B.jc[mid] < j)
          lo = mid + 1;
        else
          hi = mid;
      }
      t = lo;
    }
    store_ptr(cp, ptr_t, j, off[t]);
  }
}

// DCSC output: nonempty slot t becomes entry zoff[t] of jc / cp.
__global__ void k_write_dcsc(Operand B, const int64_t* cnt, const int64_t* off, const int64_t* zoff, int64_t nslots,
                             int32_t* jc, void* cp, int32_t ptr_t, unsigned long long* qctr) {
  reset_queues(qctr);
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < nslots; t += stride) {
    if (cnt[t] > 0) {
      const int64_t u = zoff[t];
      jc[u] = (int32_t)slot_col(B, t);
      store_ptr(cp, ptr_t, u, off[t]);
    }
    if (t == nslots - 1) store_ptr(cp, ptr_t, zoff[nslots], off[nslots]);
  }
}

struct Summary {
  unsigned long long mults;
  unsigned long long nnz_tiny;
  unsigned long long nnz_multi;  // entries of C in columns with row-block counts
  unsigned long long setup;      // sum over cut columns of (B entries x parts)
  unsigned long long cut_mults;  // multiplications of the cut columns
  unsigned err;
  unsigned pad;
};

// Column pointers from the exact counts: off = exclusive scan of cnt, zoff =
// of the nonempty flags (DCSC output; else only its total), nnz_tiny and nnz_multi =
// sums over the columns of at most tiny_max products and over those of more than
// multi_min (which get row-block counts).  One pass of block sums and one that
// applies them, for all results (a scan each and a sum took five launches).
// totals: the spread counters of the multiplications, nnz_tiny and nnz_multi.
__global__ void __launch_bounds__(kScanThreads) k_cnt_reduce(const int64_t* cnt, const int64_t* mults, int64_t tiny_max,
                                                             int64_t multi_min, int64_t n, int64_t* sums,
                                                             int64_t* zsums, unsigned long long* totals) {
  __shared__ int64_t red[4][kScanThreads / kWave];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  int64_t s = 0, z = 0, ti = 0, mu = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
    if (i < n) {
      const int64_t c = cnt[i];
      s += c;
      z += c > 0;
      const int64_t m = mults[i];
      if (m <= tiny_max) ti += c;
      if (m > multi_min) mu += c;
    }
  }
  s = wave_sum(s);
  z = wave_sum(z);
  ti = wave_sum(ti);
  mu = wave_sum(mu);
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) {
    red[0][w] = s;
    red[1][w] = z;
    red[2][w] = ti;
    red[3][w] = mu;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < kScanThreads / kWave; ++k) {
      s += red[0][k];
      z += red[1][k];
      ti += red[2][k];
      mu += red[3][k];
    }
    sums[blockIdx.x] = s;
    zsums[blockIdx.x] = z;
    if (ti) atomicAdd(spread(totals + kSpreadWords), (unsigned long long)ti);
    if (mu) atomicAdd(spread(totals + 2 * kSpreadWords), (unsigned long long)mu);
  }
}

// carry / zcarry: the scanned block sums; else sums / zsums: the block sums.
// Also adds up the spread totals.
__global__ void __launch_bounds__(kScanThreads) k_cnt_apply(const int64_t* cnt, int64_t n, const int64_t* carry,
                                                            const int64_t* zcarry, const int64_t* sums,
                                                            const int64_t* zsums, int64_t* off, int64_t* zoff,
                                                            int zfull, const unsigned long long* totals,
                                                            Summary* sum) {
  __shared__ int64_t red[kScanThreads / kWave + 1];
  if (blockIdx.x == 0 && threadIdx.x < 3) {
    unsigned long long s = 0;
    for (int i = 0; i < kSpread; ++i) s += totals[threadIdx.x * kSpreadWords + i * 16];
    *(threadIdx.x == 0 ? &sum->mults : threadIdx.x == 1 ? &sum->nnz_tiny : &sum->nnz_multi) = s;
  }
  const int64_t cin = carry ? carry[blockIdx.x] : carry_from_sums(sums, blockIdx.x, red);
  const int64_t zin = zcarry ? zcarry[blockIdx.x] : carry_from_sums(zsums, blockIdx.x, red);
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int64_t v[kScanItems];
  int64_t s = 0, z = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? cnt[base + k] : 0;
    s += v[k];
    z += v[k] > 0;
  }
  int64_t total, ztotal;
  int64_t run = block_excl_scan(s, red, &total) + cin;
  int64_t zrun = block_excl_scan(z, red, &ztotal) + zin;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) {
      off[base + k] = run;
      if (zfull) zoff[base + k] = zrun;
    }
    run += v[k];
    zrun += v[k] > 0;
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == blockDim.x - 1) {
    off[n] = run;
    zoff[n] = zrun;
  }
}

// Both for up to kSmallSlots columns, by one workgroup of 1024.
__global__ void __launch_bounds__(1024) k_cnt_small(const int64_t* cnt, const int64_t* col_mults, int64_t tiny_max,
                                                    int64_t multi_min, int n, int64_t* off, int64_t* zoff, int zfull,
                                                    const unsigned long long* totals, Summary* sum) {
  __shared__ int64_t red[1024 / kWave + 1];
  __shared__ unsigned long long s_tot[2];  // entries of the tiny and of the cut columns
  if (threadIdx.x < 2) s_tot[threadIdx.x] = 0;
  const int per = (n + 1023) / 1024;  // columns per thread
  const int base = (int)threadIdx.x * per;
  int64_t v[kSmallPer];
  int64_t s = 0, z = 0, ti = 0, mi = 0;
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k) {
    const bool in = k < per && base + k < n;
    v[k] = in ? cnt[base + k] : 0;
    const int64_t mu = in ? col_mults[base + k] : 0;
    s += v[k];
    z += v[k] > 0;
    if (mu <= tiny_max) ti += v[k];
    if (mu > multi_min) mi += v[k];
  }
  ti = wave_incl_scan(ti);
  mi = wave_incl_scan(mi);
  int64_t total, ztotal;
  int64_t run = block_excl_scan(s, red, &total);
  if (lane_id() == kWave - 1) {
    if (ti) atomicAdd(&s_tot[0], (unsigned long long)ti);
    if (mi) atomicAdd(&s_tot[1], (unsigned long long)mi);
  }
  int64_t zrun = block_excl_scan(z, red, &ztotal);
#pragma unroll
  for (int k = 0; k < kSmallPer; ++k)
    if (k < per && base + k < n) {
      off[base + k] = run;
      if (zfull) zoff[base + k] = zrun;
      run += v[k];
      zrun += v[k] > 0;
    }
  if (threadIdx.x == 0) {
    unsigned long long m = 0;
    for (int i = 0; i < kSpread; ++i) m += totals[i * 16];
    sum->mults = m;
    sum->nnz_tiny = s_tot[0];
    sum->nnz_multi = s_tot[1];
    off[n] = total;
    zoff[n] = ztotal;
  }
}

// Counting sort of the multi-part list by row slice (work queue).
__global__ void k_part_hist(const Part* parts, int64_t n, unsigned long long* hist) {
  __shared__ unsigned h[66];
  for (int i = threadIdx.x; i < 66; i += blockDim.x) h[i] = 0;
  __syncthreads();
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    atomicAdd(&h[parts[i].slice], 1u);
  __syncthreads();
  for (int i = threadIdx.x; i < 66; i += blockDim.x)
    if (h[i]) atomicAdd(&hist[i], (unsigned long long)h[i]);
}

// Exclusive offsets of nb bins, written to cursor and to qoff (+ qoff[nb]).
__global__ void k_hist_offsets(unsigned long long* hist, int64_t nb, int64_t base, int64_t* qoff) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    unsigned long long run = 0;
    for (int64_t b = 0; b < nb; ++b) {
      const unsigned long long c = hist[b];
      hist[b] = run;
      qoff[b] = base + (int64_t)run;
      run += c;
    }
    qoff[nb] = base + (int64_t)run;
  }
}

// Per block: rank inside the block by LDS atomics, one global atomic per bin.
__global__ void k_part_scatter(const Part* in, int64_t n, unsigned long long* cursor, Part* out) {
  __shared__ unsigned h[66];
  __shared__ unsigned long long base[66];
  for (int64_t t0 = (int64_t)blockIdx.x * blockDim.x; t0 < n; t0 += (int64_t)gridDim.x * blockDim.x) {
    for (int i = threadIdx.x; i < 66; i += blockDim.x) h[i] = 0;
    __syncthreads();
    const int64_t i = t0 + threadIdx.x;
    Part p{};
    unsigned rk = 0;
    if (i < n) {
      p = in[i];
      rk = atomicAdd(&h[p.slice], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < 66; b += blockDim.x)
      if (h[b]) base[b] = atomicAdd(&cursor[b], (unsigned long long)h[b]);
    __syncthreads();
    if (i < n) out[base[p.slice] + rk] = p;
    __syncthreads();
  }
}

}  // namespace spx

// ==================================================================== host
using namespace spx;

namespace spx {

enum { kEvPlan0, kEvPlan1, kEvExec0, kEvMulti, kEvParts, kEvTiny, kEvPtr, kNumEv };

struct GemmPlan : spx_plan {
  explicit GemmPlan(const spx_ctx* c) : spx_plan(c, kPlanGemm) {
    if (c && c->profile) {
      profile = true;
      for (auto& e : ev) (void)hipEventCreate(&e);
    }
  }
  ~GemmPlan() override {
    if (profile)
      for (auto& e : ev) (void)hipEventDestroy(e);
  }
  void mark(int i, hipStream_t st) {
    if (profile) (void)hipEventRecord(ev[i], st);
  }
  bool profile = false;
  bool ran_parts = false, ran_tiny = false;
  hipEvent_t ev[kNumEv] = {};
  Operand A{}, B{};
  int32_t sr = 0, vt = 0, c_fmt = 0;
  spx_tuning tune{};
  int64_t nslots = 0, nnz = 0, nzc = 0, mults = 0, nparts = 0, psplit = 0, nnz_tiny = 0, nnz_multi = 0;
  int64_t binoff_h[kNumBins + 1] = {};
  int64_t* bq_a0 = nullptr;
  int32_t* bq_alen = nullptr;
  int32_t* bq_split = nullptr;
  int32_t* splits = nullptr;
  ProdSrc src{};
  int64_t* aux = nullptr;
  int64_t* mults_d = nullptr;
  int64_t* cnt = nullptr;
  int64_t* off = nullptr;
  int64_t* zoff = nullptr;
  int32_t* list = nullptr;
  int64_t* binoff = nullptr;
  Part* parts = nullptr;
  int64_t* qoff_multi = nullptr;  // bounds of the multi-part launch's queues (several row slices only)
  unsigned long long* qctr = nullptr;  // [kMaxQueues + 1] zero between execs
  bool queues_spent = false;           // unless an exec failed and could not clear them (see QueueGuard)
  int32_t nq_multi = 1, nslice = 1, nslice_req = 1;
  Summary* sum = nullptr;
  unsigned long long* totals = nullptr;  // spread counters: multiplications, entries of the tiny and the cut columns
  int64_t L = 0, L_single = 0;
  int32_t* qlist = nullptr;  // B entries of the parts of bucketed columns, grouped by part
  uint64_t* gbm = nullptr;  // stored row bitmaps of the bitmap-counted columns
  int64_t gbm_words = 0;    // 64-bit words per stored bitmap
};

// The last launch of an exec clears the queue counters for the next one.  An exec
// that returns before it leaves this to clear them: the next one would else find
// the queues empty and skip its parts without an error.
struct QueueGuard {
  GemmPlan* plan;
  hipStream_t st;
  ~QueueGuard() {
    if (plan) plan->queues_spent = zero_words(st, {{plan->qctr, kMaxQueues + 1}}) != SPX_OK;
  }
};

int check_mat(const spx_mat* X, const char* name) {
  if (!X) return fail(SPX_EINVAL, std::string(name) + " is NULL");
  if (X->m < 0 || X->n < 0 || X->nnz < 0 || X->m >= (1ll << 31) || X->n >= (1ll << 31))
    return fail(SPX_EINVAL, std::string(name) + ": bad dimensions");
  if (X->fmt != SPX_CSC && X->fmt != SPX_DCSC) return fail(SPX_EINVAL, std::string(name) + ": bad format");
  if (X->ptr_t != SPX_PTR_I32 && X->ptr_t != SPX_PTR_I64) return fail(SPX_EINVAL, std::string(name) + ": bad ptr_t");
  if (X->val_t < SPX_VAL_F32 || X->val_t > SPX_VAL_BOOL) return fail(SPX_EINVAL, std::string(name) + ": bad val_t");
  if (X->ptr_t == SPX_PTR_I32 && X->nnz >= (1ll << 31)) return fail(SPX_EOVERFLOW, std::string(name) + ": nnz needs I64 pointers");
  if (X->fmt == SPX_DCSC && (X->nzc < 0 || X->nzc > X->n || (X->nzc > 0 && !X->jc)))
    return fail(SPX_EINVAL, std::string(name) + ": bad DCSC nzc/jc");
  if (!X->cp) return fail(SPX_EINVAL, std::string(name) + ": cp is NULL");
  if (X->nnz > 0 && !X->ir) return fail(SPX_EINVAL, std::string(name) + ": ir is NULL");
  if (X->nnz > 0 && X->val_t != SPX_VAL_BOOL && !X->num) return fail(SPX_EINVAL, std::string(name) + ": num is NULL");
  return SPX_OK;
}

int build_aux(const Operand& X, Scratch& scr, hipStream_t st, int64_t** aux, int64_t* chunk) {
  *aux = nullptr;
  *chunk = 1;
  if (X.fmt != SPX_DCSC) return SPX_OK;
  *chunk = std::max<int64_t>(1, ceil_div(std::max<int64_t>(X.n, 1), std::max<int64_t>(X.nzc, 1)));
  const int64_t naux = ceil_div(std::max<int64_t>(X.n, 1), *chunk);
  SPX_TRY(scr.get_n(naux + 1, aux));
  k_build_aux<<<grid_for(naux + 1, 256), 256, 0, st>>>(X.jc, X.nzc, *chunk, naux, *aux);
  SPX_HIP(hipGetLastError());
  return SPX_OK;
}

// Most outputs of a hash-mode part in L bytes (hash_bytes steps at the powers of two).
static int32_t hash_most(int64_t L, int64_t sz) {
  int64_t p2 = 32;
  while (hash_bytes(2 * p2, sz) <= L) p2 *= 2;
  return p2 >= 64 ? (int32_t)p2 : 0;
}

// Column pointers of C (see k_cnt_reduce).
static int scan_counts(GemmPlan* P, Scratch& scr, hipStream_t st) {
  const int64_t n = P->nslots;
  // the products above which a column gets row-block counts (see multi_end)
  const int64_t multi_min =
      std::min<int64_t>(P->tune.hash_count_max, std::max<int64_t>(P->tune.single_part_max, kMidMax));
  if (n <= 0) return zero_words(st, {{P->off, 1}, {P->zoff, 1}});
  if (n <= kSmallSlots) {
    k_cnt_small<<<1, 1024, 0, st>>>(P->cnt, P->mults_d, P->tune.tiny_max, multi_min, (int)n, P->off, P->zoff,
                                    P->c_fmt == SPX_DCSC, P->totals, P->sum);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
  }
  const int64_t nb = ceil_div(n, kScanTile);
  int64_t *sums = nullptr, *zsums = nullptr, *carry = nullptr, *zcarry = nullptr;
  SPX_TRY(scr.get_many({Scratch::part(&sums, nb), Scratch::part(&zsums, nb)}));
  k_cnt_reduce<<<(unsigned)nb, kScanThreads, 0, st>>>(P->cnt, P->mults_d, P->tune.tiny_max, multi_min, n, sums, zsums,
                                                      P->totals);
  SPX_HIP(hipGetLastError());
  if (nb > kFusedCarry) {
    SPX_TRY(scr.get_many({Scratch::part(&carry, nb + 1), Scratch::part(&zcarry, nb + 1)}));
    SPX_TRY(exclusive_scan(LoadI64{sums}, nb, carry, scr, st));
    SPX_TRY(exclusive_scan(LoadI64{zsums}, nb, zcarry, scr, st));
  }
  k_cnt_apply<<<(unsigned)nb, kScanThreads, 0, st>>>(P->cnt, n, carry, zcarry, sums, zsums, P->off, P->zoff,
                                                     P->c_fmt == SPX_DCSC, P->totals, P->sum);
  SPX_HIP(hipGetLastError());
  return SPX_OK;
}

// Waits for the stream and reads the plan's summary together with the
// given extra device words (one read-back launch).
int summary_sync(GemmPlan* P, hipStream_t st, Summary* host, std::initializer_list<DevWord> extra = {},
                 int64_t* extra_out = nullptr) {
  static_assert(sizeof(Summary) == 6 * sizeof(int64_t), "the summary is read as six words");
  DevWord w[kMaxReadRanges];
  int n = 0, nx = 0;
  for (const DevWord& d : extra) {
    w[n++] = d;
    nx += d.count;
  }
  w[n++] = DevWord{P->sum, 8, 6};
  int64_t out[kMaxReadWords];
  SPX_TRY(read_device_words(st, w, n, out));
  for (int i = 0; i < nx; ++i) extra_out[i] = out[i];
  std::memcpy(host, out + nx, sizeof(Summary));
  return SPX_OK;
}

}  // namespace spx

extern "C" void spx_default_tuning(spx_tuning* t) {
  std::memset(t, 0, sizeof(*t));
  t->tiny_max = 64;
  t->hash_count_max = 1 << 13;
  t->single_part_max = 1024;
  t->part_lds_bytes = 72 * 1024;
  t->count_threads = 256;
  t->bitmap_threads = 512;
  t->part_threads = 512;
  t->single_threads = 256;
  t->bitmap_chunk_log2 = 0;
  t->xcd_slices = 1;
  t->bitmap_store_mb = 32768;
}

template <int SR, typename T>
static int launch_numeric(GemmPlan* P, spx_mat* C, hipStream_t st) {
  int32_t* cir = C->ir;
  T* cnum = (T*)C->num;
  unsigned* err = &P->sum->err;
  const int cus = device_cu_count();
  // parts of multi-part columns [0, psplit), single-part columns [psplit, nparts)
  // (the queue counters are zero: cleared by the plan, then by every exec's last launch or QueueGuard)
  for (int r = 0; r < 2; ++r) {
    const int64_t n0 = r == 0 ? 0 : P->psplit, n1 = r == 0 ? P->psplit : P->nparts;
    if (n1 <= n0) continue;
    const int blk = r == 0 ? P->tune.part_threads : P->tune.single_threads;
    const int64_t L = r == 0 ? P->L : P->L_single;
    const int64_t fixed = P->src.off32 ? kPartLds32 : kPartLds64;
    const int per_cu = (int)std::max<int64_t>(1, std::min<int64_t>((160 * 1024) / (L + fixed), 2048 / blk));
    int64_t grid = std::min<int64_t>(n1 - n0, (int64_t)cus * per_cu);
    if (r == 0 && P->nslice > 1) grid = std::max<int64_t>(P->nslice, grid / P->nslice * P->nslice);
    const int64_t* qoff = r == 0 ? P->qoff_multi : nullptr;
    const int nq = qoff ? P->nq_multi : 1;
    unsigned long long* qctr = r == 0 ? P->qctr : P->qctr + kMaxQueues;
    const int batch = (int)std::max<int64_t>(1, std::min<int64_t>(kPartBatch, (n1 - n0) / (2 * grid)));
    if (P->src.off32)  // A's positions fit 29 bits: gathers through 32-bit offsets
      hipLaunchKernelGGL((k_numeric_parts<SR, T, true>), dim3((unsigned)grid), dim3(blk), (size_t)L, st, P->A, P->B,
                         P->src, P->parts, qoff, n0, n1, nq, r == 0 ? P->nslice : 1, batch, qctr,
                         P->gbm, P->gbm_words, P->qlist, L, cir, cnum, err);
    else
      hipLaunchKernelGGL((k_numeric_parts<SR, T, false>), dim3((unsigned)grid), dim3(blk), (size_t)L, st, P->A, P->B,
                         P->src, P->parts, qoff, n0, n1, nq, r == 0 ? P->nslice : 1, batch, qctr,
                         P->gbm, P->gbm_words, P->qlist, L, cir, cnum, err);
    SPX_HIP(hipGetLastError());
    if (r == 0) P->mark(kEvMulti, st);
  }
  if (P->psplit == 0) P->mark(kEvMulti, st);
  for (int b = kBinMid; b < kBinTiny; ++b)  // mid columns, the longest first
    SPX_TRY(launch_mid(P->sr, P->vt, 8 >> (b - kBinMid), P->A, P->B, P->src, P->list, P->binoff_h[b],
                       P->binoff_h[b + 1], P->off, cir, cnum, st));
  P->mark(kEvParts, st);
  const int64_t ntiny = P->binoff_h[kBinTiny + 1] - P->binoff_h[kBinTiny];
  if (ntiny > 0) {
    hipLaunchKernelGGL((k_tiny<SR, T, false>), dim3(grid_for(ntiny, 8, (int64_t)cus * 64)), dim3(256), 0, st, P->A,
                       P->B, P->bq_a0, P->bq_alen, P->mults_d, P->list, P->binoff, P->cnt, P->off, cir, cnum);
    SPX_HIP(hipGetLastError());
  }
  P->mark(kEvTiny, st);
  return SPX_OK;
}

static int dispatch_numeric(GemmPlan* P, spx_mat* C, hipStream_t st) {
#define SPX_CASE(SRV, VTV, TY) \
  if (P->sr == SRV && P->vt == VTV) return launch_numeric<SRV, TY>(P, C, st);
  SPX_CASE(SPX_PLUS_TIMES, SPX_VAL_F32, float)
  SPX_CASE(SPX_PLUS_TIMES, SPX_VAL_F64, double)
  SPX_CASE(SPX_PLUS_TIMES, SPX_VAL_I64, int64_t)
  SPX_CASE(SPX_MIN_PLUS, SPX_VAL_F32, float)
  SPX_CASE(SPX_MIN_PLUS, SPX_VAL_F64, double)
  SPX_CASE(SPX_MIN_PLUS, SPX_VAL_I64, int64_t)
  SPX_CASE(SPX_SELECT2ND, SPX_VAL_F32, float)
  SPX_CASE(SPX_SELECT2ND, SPX_VAL_F64, double)
  SPX_CASE(SPX_SELECT2ND, SPX_VAL_I64, int64_t)
  SPX_CASE(SPX_SELECT1ST, SPX_VAL_F32, float)
  SPX_CASE(SPX_SELECT1ST, SPX_VAL_F64, double)
  SPX_CASE(SPX_SELECT1ST, SPX_VAL_I64, int64_t)
  if (P->sr == SPX_OR_AND || P->vt == SPX_VAL_BOOL) return launch_numeric<SPX_OR_AND, float>(P, C, st);
#undef SPX_CASE
  return fail(SPX_EUNSUPPORTED, "semiring / value type combination not provided");
}

// Result value type of a product, or -1 when the combination is not provided.
static int result_type(int32_t sr, const spx_mat* A, const spx_mat* B) {
  switch (sr) {
    case SPX_PLUS_TIMES:
    case SPX_MIN_PLUS:
      if (A->val_t != B->val_t || A->val_t == SPX_VAL_BOOL) return -1;
      return A->val_t;
    case SPX_SELECT2ND: return B->val_t;
    case SPX_SELECT1ST: return A->val_t;
    case SPX_OR_AND: return SPX_VAL_BOOL;
    default: return -1;
  }
}

extern "C" int spx_spgemm_plan(const spx_ctx* ctx, const spx_mat* A, const spx_mat* B, int32_t semiring,
                               int32_t c_fmt, const spx_tuning* tuning, spx_plan** plan, int64_t* nnz_c,
                               int64_t* nzc_c) {
  if (!plan) return fail(SPX_EINVAL, "plan is NULL");
  *plan = nullptr;
  SPX_TRY(check_mat(A, "A"));
  SPX_TRY(check_mat(B, "B"));
  if (A->n != B->m) return fail(SPX_EINVAL, "inner dimensions differ: A is m x k, B must be k x n");
  if (c_fmt != SPX_CSC && c_fmt != SPX_DCSC) return fail(SPX_EINVAL, "bad output format");
  const int vt = result_type(semiring, A, B);
  if (vt < 0) return fail(SPX_EUNSUPPORTED, "semiring / value type combination not provided");
  spx_tuning tune;
  spx_default_tuning(&tune);
  if (tuning) tune = *tuning;
  if (tune.tiny_max < 0 || tune.tiny_max > 64) return fail(SPX_EINVAL, "tiny_max must be in [0, 64]");
  if (tune.hash_count_max < tune.tiny_max || tune.hash_count_max > (1 << 14))
    return fail(SPX_EINVAL, "hash_count_max must be in [tiny_max, 16384]");
  if (tune.single_part_max < 64 || tune.single_part_max > 4096 || (tune.single_part_max & (tune.single_part_max - 1)))
    return fail(SPX_EINVAL, "single_part_max must be a power of two in [64, 4096]");
  if (tune.range_chunk != 0 && tune.range_chunk != kQChunk && tune.range_chunk != kQChunkWide)
    return fail(SPX_EINVAL, "range_chunk must be 0, 256 or 512");
  for (int th : {tune.count_threads, tune.bitmap_threads, tune.part_threads, tune.single_threads})
    if (th % 64 || th < 64 || th > 1024) return fail(SPX_EINVAL, "thread counts must be multiples of 64 in [64, 1024]");

  if (ctx && ctx->validate) {
    int32_t ok = 0;
    SPX_TRY(spx_check(ctx, A, &ok));
    if (!ok) return fail(SPX_EINVAL, "A is not canonical");
    SPX_TRY(spx_check(ctx, B, &ok));
    if (!ok) return fail(SPX_EINVAL, "B is not canonical");
  }
  auto* P = new GemmPlan(ctx);
  std::unique_ptr<GemmPlan> guard(P);
  hipStream_t st = stream_of(ctx);
  Scratch& scr = P->scratch;
  P->A = make_operand(A);
  P->B = make_operand(B);
  P->sr = semiring;
  P->vt = vt;
  P->c_fmt = c_fmt;
  P->tune = tune;
  const int sz = value_size(vt);
  const int64_t m = A->m;
  P->nslots = nslots_of(P->B);
  const int64_t nslots = P->nslots;
  const int cus = device_cu_count();

  // Row blocks: the largest power of two <= 2^14 such that one dense block
  // fits a part in bitmap mode.
  int64_t L = tune.part_lds_bytes;
  if (L > 160 * 1024 - kPartLds64) L = 160 * 1024 - kPartLds64;
  int rb = 14;
  while (rb > 6 && ((1ll << rb) * sz + ((1ll << rb) / 64) * 10 + 256) > L) --rb;
  if (((1ll << rb) * sz + ((1ll << rb) / 64) * 10 + 256) > L) return fail(SPX_EINVAL, "part_lds_bytes too small");
  const bool off32 = A->nnz < (1ll << 29) && !tune.force_off64;
  // 64-bit ranges take 2 KiB more: leave them out of the part budget if a dense row block still fits
  if (!off32 && ((1ll << rb) * sz + ((1ll << rb) / 64) * 10 + 256) <= L - (kPartLds64 - kPartLds32))
    L -= kPartLds64 - kPartLds32;
  P->L = L;
  int sp_log2 = 6;
  while ((1 << sp_log2) < tune.single_part_max) ++sp_log2;
  {
    const int64_t p2 = tune.single_part_max, S2 = 2 * p2;
    P->L_single = S2 * 4 + ((S2 * sz + 7) & ~7ll) + p2 * 10 + (kRankSpan >> 9) + (kRankSpan >> 11) + 64;
    if (P->L_single > 160 * 1024 - 8192) return fail(SPX_EINVAL, "single_part_max too large for LDS");
  }
  const int64_t nblk = std::max<int64_t>(1, ceil_div(m, 1ll << rb));
  P->nslice_req = std::max(1, std::min(tune.xcd_slices, 64));
  P->mark(kEvPlan0, st);

  unsigned long long *bincount = nullptr, *binfill = nullptr, *nlong = nullptr;
  int32_t* longs = nullptr;  // slots with more than kLongSlot B entries
  SPX_TRY(scr.get_many({Scratch::part(&P->sum, 1), Scratch::part(&P->bq_a0, B->nnz),
                        Scratch::part(&P->bq_alen, B->nnz),
                        Scratch::part(&P->mults_d, nslots), Scratch::part(&P->cnt, nslots),
                        Scratch::part(&P->off, nslots + 1), Scratch::part(&P->zoff, nslots + 1),
                        Scratch::part(&P->list, nslots), Scratch::part(&P->binoff, kNumBins + 1),
                        Scratch::part(&bincount, kNumBins), Scratch::part(&binfill, kNumBins),
                        Scratch::part(&longs, std::max<int64_t>(nslots, 1)), Scratch::part(&nlong, 1),
                        Scratch::part(&P->qctr, kMaxQueues + 1), Scratch::part(&P->totals, 3 * kSpreadWords)}));
  // bin offsets stay zero when there are no slots (k_bin_fill writes them otherwise)
  SPX_TRY(zero_words(st, {{P->sum, (int64_t)(sizeof(Summary) / 8)}, {bincount, kNumBins}, {binfill, kNumBins},
                          {P->cnt, std::max<int64_t>(nslots, 1)}, {nlong, 1}, {P->binoff, kNumBins + 1},
                          {P->qctr, kMaxQueues + 1}, {P->totals, 3 * kSpreadWords}}));
  unsigned* err = &P->sum->err;

  // AUX index for a DCSC A
  int64_t chunk = 1;
  SPX_TRY(build_aux(P->A, scr, st, &P->aux, &chunk));
  const int32_t sstride = (int32_t)nblk + 1;
  P->src = ProdSrc{A->ir, P->bq_a0, P->bq_alen, nullptr, nullptr, sstride, rb, (int32_t)m,
                   off32 ? 1 : 0, tune.range_chunk == kQChunk ? kQChunk : kQChunkWide};
  BinCfg bc{tune.tiny_max, tune.hash_count_max};
  const bool small = nslots <= kSmallSlots;
  if (nslots > 0 && small && B->m <= kSmallSlots) {
    k_slots_small<<<grid_for(nslots, 4), 256, 0, st>>>(P->A, P->B, P->aux, chunk, P->bq_a0, P->bq_alen, (int)nslots,
                                                       P->mults_d, P->totals, longs, nlong, err);
    SPX_HIP(hipGetLastError());
  } else if (nslots > 0) {
    if (B->nnz > 0) {
      k_rowinfo<<<grid_for(B->nnz, 256, (int64_t)cus * 32), 256, 0, st>>>(P->A, P->B, P->aux, chunk, P->bq_a0,
                                                                           P->bq_alen, err);
      SPX_HIP(hipGetLastError());
    }
    k_slot_mults<<<grid_for(nslots * 8, 256, (int64_t)cus * 16), 256, 0, st>>>(P->B, P->bq_alen, nslots, P->mults_d,
                                                                              P->totals, longs, nlong);
    SPX_HIP(hipGetLastError());
    k_slot_mults_long<<<(unsigned)cus * 8, 256, 0, st>>>(P->B, P->bq_alen, longs, nlong, P->mults_d, P->totals);
    SPX_HIP(hipGetLastError());
  }
  if (nslots > 0 && small) {
    k_bin_small<<<1, 1024, 0, st>>>(P->mults_d, (int)nslots, bc, P->binoff, P->list);
    SPX_HIP(hipGetLastError());
  } else if (nslots > 0) {
    k_bin_count<<<grid_for(nslots, 256, (int64_t)cus * 8), 256, 0, st>>>(P->mults_d, nslots, bc, bincount);
    SPX_HIP(hipGetLastError());
    k_bin_fill<<<grid_for(ceil_div(nslots, kFillPer), 256, (int64_t)cus * 8), 256, 0, st>>>(
        P->mults_d, nslots, bc, bincount, P->binoff, binfill, P->list);
    SPX_HIP(hipGetLastError());
  }
  // sync 1: bin sizes and the total number of multiplications
  Summary hs{};
  static_assert(sizeof(P->binoff_h) == (kNumBins + 1) * sizeof(int64_t), "bin offsets are read as words");
  SPX_TRY(summary_sync(P, st, &hs, {{P->binoff, 8, kNumBins + 1}}, P->binoff_h));
  if (hs.err & 1u) return fail(SPX_EINVAL, "B has a row index outside A's columns");
  const int64_t* bo = P->binoff_h;
  // columns with more than single_part_max products get row-block counts
  const int64_t multi_begin = bo[0], multi_end = bo[std::min(kBinHash0 + 14 - sp_log2, kBinMid)];
  const int64_t nmulti = multi_end - multi_begin;
  uint32_t* blkcnt = nullptr;
  if (nmulti > 0) {
    if ((double)nmulti * (double)nblk * 4.0 > 8e9) return fail(SPX_EUNSUPPORTED, "row-block table too large");
    SPX_TRY(scr.get_n(nmulti * nblk + 1, &blkcnt));
  }
  const int64_t nbitmap = bo[kBinHash0] - bo[0];
  // bitmap chunks: a power of two of rows, a multiple of the row block and of 128;
  // 0 = one chunk per row slice
  int want = tune.bitmap_chunk_log2;
  if (want <= 0) {  // auto: one chunk per row slice, at most 2^18 rows (four workgroups per CU)
    want = 0;
    while ((1ll << want) < ceil_div(m, std::max(1, P->nslice_req))) ++want;
    want = std::min(want, 18);
  }
  const int clog_min = std::max(rb, 7);  // whole 16-byte stores (k_count_bitmap)
  int clog = std::max<int>(clog_min, std::min<int>(want, 20));
  while (clog > clog_min && (1ll << (clog - 1)) >= m) --clog;
  const int64_t nchunks = std::max<int64_t>(1, ceil_div(m, 1ll << clog));
  unsigned long long* bqctr = nullptr;  // per-chunk column counters of the bitmap count
  if (nbitmap > 0) SPX_TRY(scr.get_n(nchunks, &bqctr));
  // split table of the long columns of A that these columns name
  const bool split = nmulti > 0 && A->nnz > kSplitMin;
  const int64_t nslots_a = nslots_of(P->A);
  int32_t *flag = nullptr, *slot_of_split = nullptr;
  int64_t* sid_off = nullptr;
  if (split) {
    const int64_t cap = std::min(A->nnz / (kSplitMin + 1) + 1, B->nnz);  // distinct long columns named by B
    SPX_TRY(scr.get_many({Scratch::part(&flag, nslots_a + 1), Scratch::part(&sid_off, nslots_a + 1),
                          Scratch::part(&slot_of_split, cap), Scratch::part(&P->bq_split, B->nnz),
                          Scratch::part(&P->splits, cap * sstride)}));
  }
  if (nmulti > 0)
    SPX_TRY(zero_words(st, {{blkcnt, ceil_div(nmulti * nblk, 2)}, {flag, split ? ceil_div(nslots_a, 2) : 0},
                            {bqctr, nbitmap > 0 ? nchunks : 0}}));
  if (split) {
    const unsigned sb = grid_for(nmulti, 16, (int64_t)cus * 16);
    const unsigned lb = kLongShare * grid_for(std::min(nslots, B->nnz / kLongSlot), 1, cus);
    k_split_mark<<<sb + lb, 256, 0, st>>>(P->A, P->B, P->aux, chunk, P->list, multi_begin, multi_end, longs, nlong, lb,
                                          P->bq_alen, flag);
    SPX_HIP(hipGetLastError());
    SPX_TRY(exclusive_scan(LoadFlag{flag}, nslots_a, sid_off, scr, st));
    k_split_rows<<<grid_for(nslots_a, 256, (int64_t)cus * 32), 256, 0, st>>>(nslots_a, sid_off, flag, slot_of_split);
    SPX_HIP(hipGetLastError());
    // flat where such columns are not rare: R-MAT 2^20 squared (most are) 134 us by list, 38
    // flat; 16,384 columns, all such, 3.25 | 3.03 ms in all; among 2^20 columns no difference
    // from n/65536 to n/4 of them, where B has two entries a column
    const int flat = nmulti > nslots / 64;
    k_split_assign<<<flat ? grid_for(B->nnz, 1024, (int64_t)cus * 16) : sb + lb, 256, 0, st>>>(
        P->A, P->B, P->aux, chunk, P->list, multi_begin, multi_end, longs, nlong, lb, flat, P->bq_alen, flag,
        P->bq_split);
    SPX_HIP(hipGetLastError());
    k_split_fill<<<grid_for(std::min(nslots_a, B->nnz) * kWave, 256, (int64_t)cus * 32), 256, 0, st>>>(
        P->A, sid_off + nslots_a, slot_of_split, P->splits, sstride, rb);
    SPX_HIP(hipGetLastError());
    P->src.split = P->bq_split;
    P->src.splits = P->splits;
  }

  // exact counts
  const int64_t ntiny = bo[kBinTiny + 1] - bo[kBinTiny];
  if (ntiny > 0) {
    k_tiny<SPX_OR_AND, float, true><<<grid_for(ntiny, 8, (int64_t)cus * 64), 256, 0, st>>>(
        P->A, P->B, P->bq_a0, P->bq_alen, P->mults_d, P->list, P->binoff, P->cnt, nullptr, nullptr, nullptr);
    SPX_HIP(hipGetLastError());
  }
  SPX_TRY(launch_mid_count(P->B, P->src, P->mults_d, P->list, bo[kBinMid], bo[kBinTiny], P->cnt, err, st));
  // hash-counted columns: a launch per table size, so that each runs at its own
  // occupancy; few columns go in one launch sized for the largest (four launches
  // of 13 to 355 columns took 60 us one after the other)
  ProdSrc hsrc = P->src;
  hsrc.qchunk = kQChunk;
  const auto count_hash = [&](int bin, int64_t beg, int64_t end) -> int {
    const int log2s = kHashLog2Max - (bin - kBinHash0);
    const size_t lds = ((size_t)4 << log2s) + (nblk <= 1024 ? (size_t)nblk * 4 : 0);
    const int blk = log2s >= 15 ? 1024 : (log2s >= 13 ? std::max(tune.count_threads, 512) : tune.count_threads);
    const int64_t fixed = (off32 ? sizeof(HashRanges<true>) : sizeof(HashRanges<false>)) + 256;
    const int per_cu = std::max<int>(1, std::min<int>((int)((160 * 1024) / (lds + fixed)), 2048 / blk));
    const auto kern = off32 ? k_count_hash<true> : k_count_hash<false>;
    kern<<<(unsigned)std::min<int64_t>(end - beg, (int64_t)cus * per_cu), blk, lds, st>>>(
        P->B, hsrc, P->mults_d, P->list, beg, end, multi_begin, multi_end, rb, nblk, blkcnt, P->cnt, err);
    SPX_HIP(hipGetLastError());
    return SPX_OK;
  };
  const bool together = bo[kBinMid] - bo[kBinHash0] <= 4 * (int64_t)cus;
  for (int b = kBinHash0; b < kBinMid; ++b) {
    if (bo[b + 1] == bo[b]) continue;
    SPX_TRY(count_hash(b, bo[b], together ? bo[kBinMid] : bo[b + 1]));
    if (together) break;
  }
  if (nbitmap > 0) {
    const size_t lds = (((size_t)1 << clog) + 127) / 128 * 16 + (((size_t)1 << clog) >> rb) * 4 + 16;
    const int64_t fixed = (off32 ? sizeof(BitmapRanges<true>) : sizeof(BitmapRanges<false>)) + 256;
    const int per_cu = std::max<int>(1, std::min<int>((int)((160 * 1024) / (lds + fixed)), 2048 / tune.bitmap_threads));
    int64_t bgrid = std::min<int64_t>(nbitmap * nchunks, (int64_t)cus * per_cu);
    bgrid = std::max<int64_t>(nchunks, bgrid / nchunks * nchunks);
    // keep the bitmaps for the numeric phase when they fit the cap
    const int64_t words = ceil_div(m, 128) * 2;  // 16-byte rows
    if (tune.bitmap_store_mb > 0 && (double)nbitmap * words * 8.0 <= (double)tune.bitmap_store_mb * 1048576.0) {
      if (scr.get_n(nbitmap * words, &P->gbm) == SPX_OK)
        P->gbm_words = words;
      else
        P->gbm = nullptr;  // not enough memory: recompute instead
    }
    ProdSrc bsrc = P->src;
    bsrc.qchunk = kQChunkWide;
    const auto kern = off32 ? k_count_bitmap<true> : k_count_bitmap<false>;
    kern<<<(unsigned)bgrid, tune.bitmap_threads, lds, st>>>(
        P->B, bsrc, P->list, P->binoff, m, clog, rb, nblk, blkcnt, (unsigned long long*)P->cnt,
        (uint32_t*)P->gbm, 2 * P->gbm_words, bqctr);
    SPX_HIP(hipGetLastError());
  }
  // column pointers and nonempty-column offsets
  SPX_TRY(scan_counts(P, scr, st));
  // parts of the columns above the mid ones: list positions [0, bo[kBinMid])
  const int64_t npos = bo[kBinMid];
  int64_t *np = nullptr, *poff = nullptr;
  int nslice = std::max(1, std::min(tune.xcd_slices, 64));
  int64_t slice_blocks = ceil_div(nblk, nslice);
  nslice = (int)ceil_div(nblk, slice_blocks);
  if (nslice <= 1) slice_blocks = 0;
  P->nslice = nslice;
  // Parts leave room for noted rows (9% more parts) where every workgroup gets many of
  // them.  Without | with room, in all: R-MAT scale 20 squared 46.3 | 45.5 ms, scale 18 5.94 |
  // 5.82, scale 16 equal; 16,384 columns through R-MAT 2.73 | 2.65, 2048 514 | 503 us; but
  // through uniform columns, whose bitmap words are evenly full, 2048 541 | 564 us and
  // 16,384 2.87 | 3.03 ms.
  const int32_t note = sz > 0 && nmulti >= 16 * (int64_t)cus ? 2 : 0;
  PartCfg pc{L, m, sz, rb, nblk, slice_blocks, nslice, hash_most(L, sz), m, note, 0};
  PartCfg pcs{P->L_single, m, sz, rb, nblk, 0, nslice, hash_most(P->L_single, sz), m, 0, 0};
  const unsigned cut_blocks = nmulti > 0 ? grid_for(nmulti, 4, (int64_t)cus * 8) : 0;
  const unsigned pgrid = cut_blocks + (npos > multi_end ? grid_for(npos - multi_end, 256, (int64_t)cus * 8) : 0);
  if (npos > 0) {
    SPX_TRY(scr.get_n(npos, &np));
    SPX_TRY(scr.get_n(npos + 1, &poff));
    k_parts<<<pgrid, 256, 0, st>>>(P->B, pc, pcs, P->list, npos, multi_begin, multi_end,
                                                                    cut_blocks, P->gbm ? nbitmap : 0, P->cnt,
                                                                    P->off, blkcnt, np, nullptr, nullptr, P->mults_d,
                                                                    &P->sum->setup, err);
    SPX_HIP(hipGetLastError());
    SPX_TRY(exclusive_scan(LoadI64{np}, npos, poff, scr, st));
  }
  // sync 2: sizes
  int64_t tail[4] = {0, 0, 0, 0};
  if (npos > 0)
    SPX_TRY(summary_sync(P, st, &hs, {{P->off + nslots, 8}, {P->zoff + nslots, 8}, {poff + npos, 8},
                                      {poff + multi_end, 8}}, tail));
  else
    SPX_TRY(summary_sync(P, st, &hs, {{P->off + nslots, 8}, {P->zoff + nslots, 8}}, tail));
  if (hs.err & 4u) return fail(SPX_EUNSUPPORTED, "a row block is too dense for the LDS budget");
  P->mults = (int64_t)hs.mults;
  P->nnz = tail[0];
  P->nzc = tail[1];
  P->nparts = tail[2];
  P->psplit = tail[3];
  P->nnz_tiny = (int64_t)hs.nnz_tiny;
  P->nnz_multi = (int64_t)hs.nnz_multi;
  if (P->nparts > 0) {
    SPX_TRY(scr.get_n(P->nparts, &P->parts));
    k_parts<<<pgrid, 256, 0, st>>>(P->B, pc, pcs, P->list, npos, multi_begin, multi_end,
                                                                    cut_blocks, P->gbm ? nbitmap : 0, P->cnt,
                                                                    P->off, blkcnt, nullptr, poff, P->parts,
                                                                    P->mults_d, nullptr, err);
    SPX_HIP(hipGetLastError());
    // bucket mode: range set-ups would outnumber multiplications 3 to 2
    // (building the lists costs about three walks over the cut columns' rows;
    // measured on R-MAT times tall-skinny B, the lists pay off above ~1.3)
    const int64_t nmulti = multi_end - multi_begin;
    const bool bucket_auto = tune.bucket_parts == 0 && hs.cut_mults > 0 && 2 * hs.setup > 3 * hs.cut_mults;
    if (P->psplit > 0 && (bucket_auto || tune.bucket_parts > 0) && nblk <= 4096 && nmulti * nblk <= (1ll << 27) &&
        B->nnz < (1ll << 31) && hs.cut_mults > 0) {
      int32_t* map = nullptr;
      unsigned *bcnt = nullptr, *bfill = nullptr;
      int64_t* boff = nullptr;
      SPX_TRY(scr.get_n(nmulti * nblk, &map));
      SPX_TRY(scr.get_n(P->psplit, &bcnt));
      SPX_TRY(scr.get_n(P->psplit, &bfill));
      SPX_TRY(scr.get_n(P->psplit + 1, &boff));
      SPX_TRY(scr.get_n((int64_t)hs.cut_mults, &P->qlist));  // a B entry reaches at most alen parts
      SPX_TRY(fill_u32(bcnt, P->psplit, 0, st));
      SPX_TRY(fill_u32(bfill, P->psplit, 0, st));
      k_bucket_map<<<grid_for(nmulti, 256, 4096), 256, 0, st>>>(pc, np, poff, multi_begin, multi_end, P->parts, map);
      SPX_HIP(hipGetLastError());
      const dim3 bgrid(64, (unsigned)std::min<int64_t>(nmulti, 4096));
      k_bucket<false><<<bgrid, 256, 0, st>>>(P->B, P->src, pc, P->list, np, poff, multi_begin, multi_end, P->parts,
                                              map, bcnt, nullptr, nullptr, nullptr, 0, err);
      SPX_HIP(hipGetLastError());
      SPX_TRY(exclusive_scan(LoadBucket{bcnt}, P->psplit, boff, scr, st));
      k_bucket<true><<<bgrid, 256, 0, st>>>(P->B, P->src, pc, P->list, np, poff, multi_begin, multi_end, P->parts,
                                             map, nullptr, boff, bfill, P->qlist, (int64_t)hs.cut_mults, err);
      SPX_HIP(hipGetLastError());
      k_bucket_parts<<<grid_for(nmulti, 256, 4096), 256, 0, st>>>(np, poff, multi_begin, multi_end, bcnt, boff,
                                                                  P->parts);
      SPX_HIP(hipGetLastError());
      SPX_TRY(summary_sync(P, st, &hs));
      if (hs.err & 32u) return fail(SPX_EDEVICE, "bucket lists exceeded their bound");
    }
    // work queues of the multi-part launch: one per row slice plus a
    // shared one (parts spanning all rows); the single-part launch has one
    P->nq_multi = pc.nslice + 1;
    if (P->psplit > 0 && pc.nslice > 1) {
      SPX_TRY(scr.get_n(P->nq_multi + 1, &P->qoff_multi));
      unsigned long long* hist = nullptr;
      Part* sorted = nullptr;
      SPX_TRY(scr.get_n(P->nq_multi + 1, &hist));
      SPX_TRY(scr.get_n(P->nparts, &sorted));
      SPX_TRY(fill_i64((int64_t*)hist, P->nq_multi + 1, 0, st));
      k_part_hist<<<grid_for(P->psplit, 256, 4096), 256, 0, st>>>(P->parts, P->psplit, hist);
      k_hist_offsets<<<1, 64, 0, st>>>(hist, P->nq_multi, 0, P->qoff_multi);
      k_part_scatter<<<grid_for(P->psplit, 256, 4096), 256, 0, st>>>(P->parts, P->psplit, hist, sorted);
      SPX_HIP(hipGetLastError());
      if (P->nparts > P->psplit)
        SPX_HIP(hipMemcpyAsync(sorted + P->psplit, P->parts + P->psplit, sizeof(Part) * (P->nparts - P->psplit),
                               hipMemcpyDeviceToDevice, st));
      P->parts = sorted;
    }
  }
  P->mark(kEvPlan1, st);
  if (nnz_c) *nnz_c = P->nnz;
  if (nzc_c) *nzc_c = P->nzc;
  *plan = guard.release();
  return SPX_OK;
}

extern "C" int spx_spgemm_exec(spx_plan* plan, spx_mat* C) {
  if (!plan || plan->kind != kPlanGemm) return fail(SPX_EINVAL, "not a SpGEMM plan");
  auto* P = static_cast<GemmPlan*>(plan);
  if (!C) return fail(SPX_EINVAL, "C is NULL");
  if (C->m != P->A.m || C->n != P->B.n) return fail(SPX_EINVAL, "C has the wrong dimensions");
  if (C->fmt != P->c_fmt) return fail(SPX_EINVAL, "C's format differs from the planned one");
  if (C->val_t != P->vt) return fail(SPX_EINVAL, "C's value type differs from the product's");
  if (C->ptr_t != SPX_PTR_I32 && C->ptr_t != SPX_PTR_I64) return fail(SPX_EINVAL, "bad C ptr_t");
  if (C->ptr_t == SPX_PTR_I32 && P->nnz >= (1ll << 31)) return fail(SPX_EOVERFLOW, "nnz(C) needs I64 pointers");
  if (!C->cp || (P->nnz > 0 && !C->ir) || (P->nnz > 0 && P->vt != SPX_VAL_BOOL && !C->num) ||
      (C->fmt == SPX_DCSC && P->nzc > 0 && !C->jc))
    return fail(SPX_EINVAL, "C buffers missing");
  C->nnz = P->nnz;
  C->nzc = C->fmt == SPX_DCSC ? P->nzc : 0;
  hipStream_t st = stream_of(&P->ctx);
  if (P->queues_spent) SPX_TRY(zero_words(st, {{P->qctr, kMaxQueues + 1}}));
  P->queues_spent = false;
  QueueGuard queues{P, st};
  P->mark(kEvExec0, st);
  P->ran_parts = P->ran_tiny = false;
  if (P->nnz > 0) SPX_TRY(dispatch_numeric(P, C, st));
  else {
    P->mark(kEvMulti, st);
    P->mark(kEvParts, st);
    P->mark(kEvTiny, st);
  }
  if (C->fmt == SPX_CSC) {
    k_write_csc_cp<<<grid_for(C->n + 1, 256, 65536), 256, 0, st>>>(P->B, P->off, P->nslots, C->n, C->cp, C->ptr_t,
                                                                         P->qctr);
  } else if (P->nslots > 0) {
    k_write_dcsc<<<grid_for(P->nslots, 256, 65536), 256, 0, st>>>(P->B, P->cnt, P->off, P->zoff, P->nslots, C->jc,
                                                                   C->cp, C->ptr_t, P->qctr);
  } else {
    if (C->ptr_t == SPX_PTR_I64)
      SPX_TRY(fill_i64((int64_t*)C->cp, 1, 0, st));
    else
      SPX_TRY(fill_u32((uint32_t*)C->cp, 1, 0, st));
  }
  SPX_HIP(hipGetLastError());
  queues.plan = nullptr;
  P->mark(kEvPtr, st);
  return SPX_OK;
}

extern "C" int spx_plan_get_times(spx_plan* plan, spx_times* times) {
  if (!plan || !times) return fail(SPX_EINVAL, "NULL argument");
  std::memset(times, 0, sizeof(*times));
  if (plan->kind == kPlanSum) plan = const_cast<spx_plan*>(sum_plan_inner(plan));
  if (plan->kind == kPlanContract) plan = const_cast<spx_plan*>(contract_plan_inner(plan));
  if (plan->kind != kPlanGemm) return fail(SPX_EINVAL, "not a SpGEMM plan");
  auto* P = static_cast<GemmPlan*>(plan);
  if (!P->profile) return fail(SPX_EINVAL, "plan was not created with ctx->profile set");
  SPX_HIP(hipEventSynchronize(P->ev[kEvPlan1]));
  SPX_HIP(hipEventElapsedTime(&times->symbolic_ms, P->ev[kEvPlan0], P->ev[kEvPlan1]));
  if (hipEventQuery(P->ev[kEvPtr]) == hipErrorNotReady) SPX_HIP(hipEventSynchronize(P->ev[kEvPtr]));
  float t = 0;
  if (hipEventElapsedTime(&t, P->ev[kEvExec0], P->ev[kEvPtr]) != hipSuccess) {
    (void)hipGetLastError();
    return SPX_OK;  // exec has not run
  }
  SPX_HIP(hipEventElapsedTime(&times->numeric_parts_ms, P->ev[kEvExec0], P->ev[kEvParts]));
  SPX_HIP(hipEventElapsedTime(&times->numeric_multi_ms, P->ev[kEvExec0], P->ev[kEvMulti]));
  SPX_HIP(hipEventElapsedTime(&times->numeric_tiny_ms, P->ev[kEvParts], P->ev[kEvTiny]));
  SPX_HIP(hipEventElapsedTime(&times->pointers_ms, P->ev[kEvTiny], P->ev[kEvPtr]));
  return SPX_OK;
}

extern "C" int spx_plan_get_info(const spx_plan* plan, spx_plan_info* info) {
  if (!plan || !info) return fail(SPX_EINVAL, "NULL argument");
  std::memset(info, 0, sizeof(*info));
  if (plan->kind == kPlanSum) plan = sum_plan_inner(plan);
  if (plan->kind == kPlanContract) plan = contract_plan_inner(plan);
  if (plan->kind != kPlanGemm) return SPX_OK;
  auto* P = static_cast<const GemmPlan*>(plan);
  const int64_t* bo = P->binoff_h;
  info->mults = P->mults;
  info->nnz = P->nnz;
  info->nzc = P->nzc;
  info->cols_empty = bo[kBinEmpty + 1] - bo[kBinEmpty];
  info->cols_tiny = bo[kBinTiny + 1] - bo[kBinTiny];
  info->cols_medium = bo[kBinTiny] - bo[kBinHash0];
  info->cols_heavy = bo[kBinHash0] - bo[0];
  info->heavy_parts = P->nparts + bo[kBinTiny] - bo[kBinMid];  // a mid column is one part
  info->nnz_tiny = P->nnz_tiny;
  info->nnz_multi = P->nnz_multi;
  info->multi_parts = P->psplit;
  return SPX_OK;
}

extern "C" void spx_plan_destroy(spx_plan* plan) { delete plan; }

const int64_t* spx::gemm_plan_offsets(const spx_plan* plan) {
  if (!plan || plan->kind != kPlanGemm) return nullptr;
  return static_cast<const GemmPlan*>(plan)->off;
}

extern "C" int spx_spgemm(const spx_ctx* ctx, const spx_mat* A, const spx_mat* B, int32_t semiring, int32_t c_fmt,
                          spx_mat* C) {
  if (!C) return fail(SPX_EINVAL, "C is NULL");
  spx_plan* plan = nullptr;
  int64_t nnz = 0, nzc = 0;
  SPX_TRY(spx_spgemm_plan(ctx, A, B, semiring, c_fmt, nullptr, &plan, &nnz, &nzc));
  std::unique_ptr<spx_plan> guard(plan);
  auto* P = static_cast<GemmPlan*>(plan);
  OutAlloc oa(ctx);
  spx_mat out{};
  out.m = A->m;
  out.n = B->n;
  out.fmt = c_fmt;
  out.ptr_t = SPX_PTR_I64;
  out.val_t = P->vt;
  const int64_t ncp = (c_fmt == SPX_CSC ? B->n : nzc) + 1;
  SPX_TRY(oa.get((size_t)ncp * 8, &out.cp));
  SPX_TRY(oa.get((size_t)std::max<int64_t>(nnz, 1) * 4, reinterpret_cast<void**>(&out.ir)));
  if (P->vt != SPX_VAL_BOOL) SPX_TRY(oa.get((size_t)std::max<int64_t>(nnz, 1) * value_size(P->vt), &out.num));
  if (c_fmt == SPX_DCSC) SPX_TRY(oa.get((size_t)std::max<int64_t>(nzc, 1) * 4, reinterpret_cast<void**>(&out.jc)));
  SPX_TRY(spx_spgemm_exec(plan, &out));
  oa.keep();
  *C = out;
  return SPX_OK;
}
