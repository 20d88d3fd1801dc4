// SpRef B = A(I,J) (Section 4) as the selection-matrix product R*A*Q, with
// R = sparse(1:len(I), I, 1) and Q = sparse(J, 1:len(J), 1).
//
// The product is evaluated right to left, R*(A*Q), and fused:
//   * A*Q: column q of A*Q is column J(q) of A (Q has one nonzero per column),
//     so it is a gather of A's columns -- no arithmetic;
//   * R*(AQ): R has one nonzero per row, so every entry (i, v) of column q
//     is copied to the rows p with I(p) = i.  The transpose of R in
//     compressed form (for each row index i the list of p with I(p) = i, in
//     any order) is built once by a counting scatter over I.
// Every output entry receives exactly one product (flops(R*A) = nnz(R*A)),
// so there is no semiring addition and the values are copied bit for bit.
// A position p occurs at most once in an output column, so ordering the
// column's (p, source) pairs by p is all that is left: by a wave in registers
// (up to 512 entries), by rank in an LDS bitmap over the positions or an LDS
// sort (up to 4096), or, for longer columns, by scanning p in order and
// probing A(:,J(q)) by binary search.
#include <algorithm>

#include "common.h"
#include "operand.h"
#include "plan.h"
#include "scan.h"
#include "wave.h"

namespace spx {

constexpr int kRefSmall = 64;
constexpr int kRefMid = 512;
constexpr int kRefMedium = 4096;
// Output classes; columns without entries are in none.
enum { kClsSmall = 0, kClsMid = 1, kClsMedium = 2, kClsLarge = 3, kNumCls = 4 };
// A column gathering more entries of A than kRefWide is never left to one wave.
constexpr int32_t kRefWide = 4096;
// Columns gathering more than kRefSplit entries are counted by kRefShare workgroups each.
constexpr int32_t kRefSplit = 256;
constexpr int kRefShare = 8;

struct SprefPlan : spx_plan {
  explicit SprefPlan(const spx_ctx* c) : spx_plan(c, kPlanSpref) {}
  Operand A{};
  const int32_t* I = nullptr;
  const int32_t* J = nullptr;
  int64_t lenI = 0, lenJ = 0, nnz = 0;
  uint32_t* rcnt = nullptr;  // [m] positions p with I(p) = i
  int32_t* rbeg = nullptr;   // [m] where they start in rpos (set where rcnt > 0)
  int32_t* rpos = nullptr;   // [lenI] positions grouped by I(p)
  int64_t* qa0 = nullptr;    // [lenJ] start of A(:,J(q))
  int32_t* qlen = nullptr;   // [lenJ] its length
  int64_t* cnt = nullptr;    // [lenJ] nnz(B(:,q))
  int64_t* off = nullptr;    // [lenJ+1]
  int32_t* list = nullptr;   // [kNumCls][lenJ] columns of each class, in any order
  int64_t ncls[kNumCls] = {};
  unsigned* err = nullptr;
};

// One pass over I and J: range checks (error bits 1 and 2); for every p its
// rank among the positions seen so far of row I(p); for every q where
// A(:,J(q)) starts and how long it is, columns longer than kRefSplit also
// being listed (their counts start from zero).
__global__ void k_ref_start(Operand A, const int64_t* aux, int64_t chunk, const int32_t* I, int64_t lenI,
                            const int32_t* J, int64_t lenJ, uint32_t* rcnt, int32_t* rank, int64_t* qa0, int32_t* qlen,
                            int64_t* cnt, int32_t* wide, unsigned long long* nwide, unsigned* err) {
  for (int64_t x = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; x < lenI + lenJ;
       x += (int64_t)gridDim.x * blockDim.x) {
    if (x < lenI) {
      const int32_t i = I[x];
      if (i < 0 || i >= A.m)
        atomicOr(err, 1u);
      else
        rank[x] = (int32_t)atomicAdd(&rcnt[i], 1u);
    } else {
      const int64_t q = x - lenI;
      const int32_t k = J[q];
      int64_t a0 = 0, a1 = 0;
      if (k < 0 || k >= A.n)
        atomicOr(err, 2u);
      else
        column_range(A, aux, chunk, k, a0, a1);
      qa0[q] = a0;
      qlen[q] = (int32_t)(a1 - a0);
      if (a1 - a0 > kRefSplit) {
        cnt[q] = 0;
        wide[atomicAdd(nwide, 1ull)] = (int32_t)q;
      }
    }
  }
}

// The first position of every row claims the row's slots of rpos, one atomic
// per workgroup and round.  (A scan over all m row counts read and wrote 50 MB
// for 2^22 rows, and left 8-byte pointers to look up twice per gathered entry.)
constexpr int kClaimPer = 4;
__global__ void __launch_bounds__(256) k_ref_claim(const int32_t* I, int64_t lenI, int64_t m, const uint32_t* rcnt,
                                                   const int32_t* rank, int32_t* rbeg, unsigned* total) {
  __shared__ uint32_t red[256 / kWave + 1];
  __shared__ uint32_t s_base;
  for (int64_t p0 = (int64_t)blockIdx.x * 256 * kClaimPer; p0 < lenI; p0 += (int64_t)gridDim.x * 256 * kClaimPer) {
    int32_t i[kClaimPer];
    uint32_t n[kClaimPer], mine = 0;
#pragma unroll
    for (int k = 0; k < kClaimPer; ++k) {
      const int64_t p = p0 + k * 256 + threadIdx.x;
      i[k] = p < lenI ? I[p] : -1;
      if (i[k] >= m) i[k] = -1;
      if (i[k] >= 0 && rank[p] != 0) i[k] = -1;
    }
#pragma unroll
    for (int k = 0; k < kClaimPer; ++k) {
      n[k] = i[k] >= 0 ? rcnt[i[k]] : 0;
      mine += n[k];
    }
    uint32_t tot;
    uint32_t at = block_excl_scan(mine, red, &tot);
    if (threadIdx.x == 0) s_base = tot ? atomicAdd(total, tot) : 0;
    __syncthreads();
    at += s_base;
#pragma unroll
    for (int k = 0; k < kClaimPer; ++k) {
      if (i[k] >= 0) rbeg[i[k]] = (int32_t)at;
      at += n[k];
    }
    __syncthreads();
  }
}

__global__ void k_ref_scatter(const int32_t* I, int64_t lenI, int64_t m, const int32_t* rank, const int32_t* rbeg,
                              int32_t* rpos) {
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < lenI; p += (int64_t)gridDim.x * blockDim.x) {
    const int32_t i = I[p];
    if (i >= 0 && i < m) rpos[rbeg[i] + rank[p]] = (int32_t)p;
  }
}

// nnz(B(:,q)) = sum over the entries (i, v) of A(:,J(q)) of |{p : I(p) = i}|.
// Groups of 16 lanes take a column each (most gather a few entries); the
// longer ones (the list wide) are shared by kRefShare workgroups each, the
// first wide_blocks ones.
__global__ void __launch_bounds__(256) k_ref_count(const Operand A, const int64_t* qa0, const int32_t* qlen,
                                                   const uint32_t* rcnt, int64_t lenJ, const int32_t* wide,
                                                   const unsigned long long* nwide, unsigned wide_blocks,
                                                   unsigned long long* cnt) {
  constexpr int G = 16;
  if (blockIdx.x >= wide_blocks) {
    const int gl = lane_id() & (G - 1);
    const int64_t grp = ((int64_t)(blockIdx.x - wide_blocks) * blockDim.x + threadIdx.x) / G;
    const int64_t ngrp = (int64_t)(gridDim.x - wide_blocks) * blockDim.x / G;
    for (int64_t q = grp; q < lenJ; q += ngrp) {
      const int64_t a0 = qa0[q];
      const int32_t al = qlen[q];
      if (al > kRefSplit) continue;
      int64_t s = 0;
      for (int32_t e0 = gl; e0 < al; e0 += 4 * G) {  // four rows in flight per lane
        int32_t i[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) i[k] = e0 + k * G < al ? A.ir[a0 + e0 + k * G] : -1;
#pragma unroll
        for (int k = 0; k < 4; ++k) s += i[k] >= 0 ? rcnt[i[k]] : 0u;
      }
#pragma unroll
      for (int d = 1; d < G; d <<= 1) s += __shfl_xor(s, d, G);
      if (gl == 0) cnt[q] = (unsigned long long)s;
    }
  } else {
    const unsigned lb = blockIdx.x, nlb = wide_blocks;  // a multiple of kRefShare
    const int64_t n = (int64_t)*nwide;
    const int32_t step = kRefShare * 256;
    for (int64_t w = lb / kRefShare; w < n; w += nlb / kRefShare) {
      const int32_t q = wide[w];
      const int64_t a0 = qa0[q];
      const int32_t al = qlen[q];
      int64_t s = 0;
      for (int64_t e0 = (int64_t)(lb % kRefShare) * 256 + threadIdx.x; e0 < al; e0 += 4 * step) {
        int32_t i[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) i[k] = e0 + (int64_t)k * step < al ? A.ir[a0 + e0 + (int64_t)k * step] : -1;
#pragma unroll
        for (int k = 0; k < 4; ++k) s += i[k] >= 0 ? rcnt[i[k]] : 0u;
      }
      s = wave_sum(s);
      if (lane_id() == 0 && s) atomicAdd(&cnt[q], (unsigned long long)s);
    }
  }
}

// Class of a column with s > 0 outputs gathering al entries of A.
__device__ __forceinline__ int ref_class(int64_t s, int32_t al) {
  if (s > kRefMedium) return kClsLarge;
  return al > kRefWide || s > kRefMid ? kClsMedium : s > kRefSmall ? kClsMid : kClsSmall;
}

// Column pointers (exclusive scan of cnt; carry: the scanned block sums, else
// sums: the block sums) and the class lists in one pass.  The class counts of
// a thread's kScanItems columns are packed in 16-bit fields, so one workgroup
// scan ranks every column in its class and one atomic per class and workgroup
// claims its slots.
__global__ void __launch_bounds__(kScanThreads) k_ref_apply(const int64_t* cnt, const int32_t* qlen, int64_t n,
                                                            const int64_t* carry, const int64_t* sums, int64_t* off,
                                                            unsigned long long* ncls, int32_t* list) {
  static_assert(kScanTile < (1 << 16), "16-bit class counts");
  __shared__ int64_t red[kScanThreads / kWave + 1];
  __shared__ uint64_t redc[kScanThreads / kWave + 1];
  __shared__ unsigned long long s_base[kNumCls];
  const int64_t cin = carry ? carry[blockIdx.x] : carry_from_sums(sums, blockIdx.x, red);
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  int64_t v[kScanItems];
  int c[kScanItems];
  int64_t s = 0;
  uint64_t mine = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    v[k] = base + k < n ? cnt[base + k] : 0;
    c[k] = v[k] > 0 ? ref_class(v[k], qlen[base + k]) : -1;
    s += v[k];
    if (c[k] >= 0) mine += 1ull << (16 * c[k]);
  }
  int64_t total;
  uint64_t tot;
  int64_t run = block_excl_scan(s, red, &total) + cin;
  uint64_t ex = block_excl_scan(mine, redc, &tot);
  if (threadIdx.x < kNumCls) {
    const unsigned long long x = (tot >> (16 * threadIdx.x)) & 0xffffull;
    s_base[threadIdx.x] = x ? atomicAdd(&ncls[threadIdx.x], x) : 0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    if (base + k < n) off[base + k] = run;
    run += v[k];
    if (c[k] >= 0) {
      list[c[k] * n + (int64_t)s_base[c[k]] + (int64_t)((ex >> (16 * c[k])) & 0xffffull)] = (int32_t)(base + k);
      ex += 1ull << (16 * c[k]);
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == blockDim.x - 1) off[n] = run;
}

// ------------------------------------------------------------------ one wave per column
// Gathers the column's (p, source) pairs into the wave's LDS: first the
// entries of A whose row is selected (a few in a hundred when I is short), 256
// looked up at a time, then their positions.  Writes at most CAP pairs to p[]
// and e[] (e: offset in A's column) and returns their number; hi and he are
// scratch of CAP entries.
template <int CAP>
__device__ __forceinline__ int gather_pairs(const Operand& A, int64_t a0, int32_t al, const uint32_t* rcnt,
                                            const int32_t* rbeg, const int32_t* rpos, int32_t* hi, int32_t* he,
                                            int32_t* p, int32_t* e) {
  const int lane = lane_id();
  int nh = 0;
  for (int32_t e0 = 0; e0 < al; e0 += 4 * kWave) {
    int32_t i[4];
    uint32_t rc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int32_t x = e0 + k * kWave + lane;
      i[k] = x < al ? A.ir[a0 + x] : -1;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) rc[k] = i[k] >= 0 ? rcnt[i[k]] : 0u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t hit = __ballot(rc[k] != 0);
      const int h = nh + __popcll(hit & lanemask_lt());
      if (rc[k] && h < CAP) {
        hi[h] = i[k];
        he[h] = e0 + k * kWave + lane;
      }
      nh += __popcll(hit);
    }
  }
  if (nh > CAP) nh = CAP;  // cannot happen: every selected entry has an output
  wave_sync();
  int total = 0;
  for (int h0 = 0; h0 < nh; h0 += kWave) {
    const int h = h0 + lane;
    const int32_t i = h < nh ? hi[h] : 0, x = h < nh ? he[h] : 0;
    const int n = h < nh ? (int)rcnt[i] : 0;
    const int32_t beg = h < nh ? rbeg[i] : 0;
    const int incl = wave_incl_scan(n);
    for (int r = 0; r < n; ++r) {
      const int slot = total + incl - n + r;
      if (slot < CAP) {
        p[slot] = rpos[beg + r];
        e[slot] = x;
      }
    }
    total += __builtin_amdgcn_readlane(incl, kWave - 1);
  }
  wave_sync();
  return total < CAP ? total : CAP;
}

// Orders the pairs by p (K: 32-bit keys when p leaves room for the slot) and
// writes the column; hi and he take them in order, for coalesced stores.
template <int R, typename K>
__device__ __forceinline__ void write_sorted(const Operand& A, int64_t a0, int n, const int32_t* p, const int32_t* e,
                                             int32_t* hi, int32_t* he, int64_t o, int vb, int32_t* bir, void* bnum) {
  constexpr int kLog = R == 1 ? 6 : R == 2 ? 7 : R == 4 ? 8 : 9;
  static_assert((1 << kLog) == kWave * R, "slots fill the key's low bits");
  const int lane = lane_id();
  K key[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int i = k * kWave + lane;
    key[k] = i < n ? ((K)(uint32_t)p[i] << kLog) | (K)i : ~K(0);
  }
  sort_regs<R, K>(key, lane);
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int i = lane * R + k;
    if (i < n) {
      hi[i] = (int32_t)(key[k] >> kLog);
      he[i] = e[(int)(key[k] & (kWave * R - 1))];
    }
  }
  wave_sync();
  for (int i = lane; i < n; i += kWave) {
    bir[o + i] = hi[i];
    copy_value(A.num, a0 + he[i], bnum, o + i, vb);
  }
  wave_sync();  // the LDS is rewritten for the next column
}

// CLS: the small columns (at most 64 entries) or the mid ones (at most 512).
template <int CLS>
__global__ void __launch_bounds__(256) k_ref_wave(Operand A, const int64_t* qa0, const int32_t* qlen,
                                                  const uint32_t* rcnt, const int32_t* rbeg, const int32_t* rpos,
                                                  const int32_t* list, int64_t n, int64_t lenI, const int64_t* off,
                                                  int vb, int32_t* bir, void* bnum) {
  constexpr int CAP = CLS == kClsSmall ? kRefSmall : kRefMid;
  __shared__ int32_t s_hi[4][CAP], s_he[4][CAP], s_p[4][CAP], s_e[4][CAP];
  const int w = threadIdx.x / kWave;
  int32_t *hi = s_hi[w], *he = s_he[w], *p = s_p[w], *e = s_e[w];
  const bool narrow = lenI <= (1ll << 32) / CAP;
  for (int64_t pos = (int64_t)blockIdx.x * 4 + w; pos < n; pos += (int64_t)gridDim.x * 4) {
    const int32_t q = list[pos];
    const int64_t a0 = qa0[q], o = off[q];
    const int c = gather_pairs<CAP>(A, a0, qlen[q], rcnt, rbeg, rpos, hi, he, p, e);
    if constexpr (CLS == kClsSmall) {
      if (narrow)
        write_sorted<1, uint32_t>(A, a0, c, p, e, hi, he, o, vb, bir, bnum);
      else
        write_sorted<1, uint64_t>(A, a0, c, p, e, hi, he, o, vb, bir, bnum);
    } else if (!narrow) {
      write_sorted<8, uint64_t>(A, a0, c, p, e, hi, he, o, vb, bir, bnum);
    } else if (c <= 128) {
      write_sorted<2, uint32_t>(A, a0, c, p, e, hi, he, o, vb, bir, bnum);
    } else if (c <= 256) {
      write_sorted<4, uint32_t>(A, a0, c, p, e, hi, he, o, vb, bir, bnum);
    } else {
      write_sorted<8, uint32_t>(A, a0, c, p, e, hi, he, o, vb, bir, bnum);
    }
  }
}

// ------------------------------------------------------------------ one workgroup per column
// Columns of at most 4096 entries that gather too many entries of A, or have
// too many outputs, for a wave.  The pairs are collected in LDS in any order
// (slots by an LDS counter, so no thread waits for another while gathering:
// with a block scan per round a hub column of 38312 entries took 150 us).
// Their ranks come from a bitmap over the positions when it fits (lenI up to
// kRankBits: one mark per pair and a popcount prefix), else from an LDS sort.
constexpr int kRefThreads = 1024;
constexpr int64_t kRankBits = 1 << 19;

__global__ void __launch_bounds__(kRefThreads) k_ref_medium(Operand A, const int64_t* qa0, const int32_t* qlen,
                                                            const uint32_t* rcnt, const int32_t* rbeg,
                                                            const int32_t* rpos, const int32_t* list, int64_t n,
                                                            int64_t lenI, const int64_t* off, int vb, int32_t* bir,
                                                            void* bnum) {
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ unsigned s_n;
  __shared__ int32_t red[kRefThreads / kWave + 1];
  const bool ranked = lenI <= kRankBits;
  const int W = (int)((lenI + 63) >> 6);  // words of the bitmap
  int32_t* s_e = (int32_t*)lds;                             // [kRefMedium] offset in A's column
  int32_t* s_p = s_e + kRefMedium;                          // ranked: [kRefMedium] position
  uint64_t* bm = (uint64_t*)(s_p + kRefMedium);             // ranked: [W] bitmap, then [W] 16-bit prefixes
  uint16_t* pre = (uint16_t*)(bm + W);
  uint64_t* s_key = (uint64_t*)(s_e + kRefMedium);          // else: [kRefMedium] (position, slot)
  for (int64_t pos = blockIdx.x; pos < n; pos += gridDim.x) {
    const int32_t q = list[pos];
    const int64_t a0 = qa0[q], o = off[q];
    const int32_t al = qlen[q];
    if (threadIdx.x == 0) s_n = 0;
    if (ranked)
      for (int i = threadIdx.x; i < W; i += kRefThreads) bm[i] = 0;
    __syncthreads();
    for (int64_t e0 = threadIdx.x; e0 < al; e0 += 8 * kRefThreads) {  // eight entries in flight per thread
      int32_t i[8];
      uint32_t rc[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) i[k] = e0 + k * kRefThreads < al ? A.ir[a0 + e0 + k * kRefThreads] : -1;
#pragma unroll
      for (int k = 0; k < 8; ++k) rc[k] = i[k] >= 0 ? rcnt[i[k]] : 0u;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (rc[k] == 0) continue;
        const unsigned at = atomicAdd(&s_n, rc[k]);
        const int32_t beg = rbeg[i[k]];
        for (uint32_t r = 0; r < rc[k] && at + r < (unsigned)kRefMedium; ++r) {
          const int32_t p = rpos[beg + r];
          s_e[at + r] = (int32_t)(e0 + k * kRefThreads);
          if (ranked) {
            s_p[at + r] = p;
            atomicOr((unsigned long long*)&bm[p >> 6], 1ull << (p & 63));
          } else {
            s_key[at + r] = ((uint64_t)(uint32_t)p << 32) | (at + r);
          }
        }
      }
    }
    __syncthreads();
    const int c = s_n < (unsigned)kRefMedium ? (int)s_n : kRefMedium;
    if (ranked) {
      const int per = (W + kRefThreads - 1) / kRefThreads;
      const int w0 = (int)threadIdx.x * per, w1 = w0 + per < W ? w0 + per : W;
      int32_t s = 0, tot;
      for (int i = w0; i < w1; ++i) s += __popcll(bm[i]);
      int32_t run = block_excl_scan1(s, red, &tot);
      for (int i = w0; i < w1; ++i) {
        pre[i] = (uint16_t)run;
        run += __popcll(bm[i]);
      }
      __syncthreads();
      for (int s2 = threadIdx.x; s2 < c; s2 += kRefThreads) {
        const int32_t p = s_p[s2];
        const int rank = pre[p >> 6] + __popcll(bm[p >> 6] & ((1ull << (p & 63)) - 1ull));
        bir[o + rank] = p;
        copy_value(A.num, a0 + s_e[s2], bnum, o + rank, vb);
      }
    } else {
      int p2 = 64;
      while (p2 < c) p2 <<= 1;
      for (int s = c + (int)threadIdx.x; s < p2; s += kRefThreads) s_key[s] = ~0ull;
      __syncthreads();
      for (int k = 2; k <= p2; k <<= 1) {
        for (int j = k >> 1; j > 0; j >>= 1) {
          for (int t = threadIdx.x; t < (p2 >> 1); t += kRefThreads) {
            const int lo = 2 * t - (t & (j - 1));
            const int hi = lo + j;
            const bool asc = (lo & k) == 0;
            const uint64_t x = s_key[lo], y = s_key[hi];
            if ((x > y) == asc) {
              s_key[lo] = y;
              s_key[hi] = x;
            }
          }
          __syncthreads();
        }
      }
      for (int s = threadIdx.x; s < c; s += kRefThreads) {
        const uint64_t k = s_key[s];
        bir[o + s] = (int32_t)(k >> 32);
        copy_value(A.num, a0 + s_e[k & 0xffffffffu], bnum, o + s, vb);
      }
    }
    __syncthreads();
  }
}

// Long columns: walk p = 0..lenI-1 in order; B(p,q) exists iff row I(p)
// is stored in A(:,J(q)) (binary search).  Output is in p order directly.
__global__ void __launch_bounds__(1024) k_ref_large(Operand A, const int64_t* qa0, const int32_t* qlen,
                                                    const int32_t* I, int64_t lenI, const int32_t* list, int64_t n,
                                                    const int64_t* off, int vb, int32_t* bir, void* bnum) {
  __shared__ int64_t red[1024 / kWave + 1];
  for (int64_t pos = blockIdx.x; pos < n; pos += gridDim.x) {
    const int32_t q = list[pos];
    const int64_t a0 = qa0[q];
    const int32_t al = qlen[q];
    const int32_t* col = A.ir + a0;
    int64_t run = off[q];
    for (int64_t pc = 0; pc < lenI; pc += blockDim.x) {
      const int64_t p = pc + threadIdx.x;
      int64_t found = -1;
      if (p < lenI) {
        const int32_t i = I[p];
        int32_t lo = 0, hi = al;
        while (lo < hi) {
          const int32_t mid = (lo + hi) >> 1;
          if (col[mid] < i)
            lo = mid + 1;
          else
            hi = mid;
        }
        if (lo < al && col[lo] == i) found = a0 + lo;
      }
      int64_t ctot;
      const int64_t excl = block_excl_scan((int64_t)(found >= 0), red, &ctot);
      if (found >= 0) {
        bir[run + excl] = (int32_t)p;
        copy_value(A.num, found, bnum, run + excl, vb);
      }
      run += ctot;
    }
  }
}

__global__ void k_write_cp(const int64_t* off, int64_t n, void* cp, int32_t ptr_t) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j <= n; j += (int64_t)gridDim.x * blockDim.x)
    store_ptr(cp, ptr_t, j, off[j]);
}

}  // namespace spx

using namespace spx;

extern "C" int spx_spref_plan(const spx_ctx* ctx, const spx_mat* A, const int32_t* I, int64_t lenI, const int32_t* J,
                              int64_t lenJ, spx_plan** plan, int64_t* nnz_b) {
  if (!plan) return fail(SPX_EINVAL, "plan is NULL");
  *plan = nullptr;
  SPX_TRY(check_mat(A, "A"));
  if (lenI < 0 || lenJ < 0 || lenI >= (1ll << 31) || lenJ >= (1ll << 31)) return fail(SPX_EINVAL, "bad index length");
  if ((lenI > 0 && !I) || (lenJ > 0 && !J)) return fail(SPX_EINVAL, "index vector is NULL");
  if (A->m > (1ll << 30)) return fail(SPX_EUNSUPPORTED, "SpRef needs m <= 2^30 (dense row map)");
  if (ctx && ctx->validate) {
    int32_t ok = 0;
    SPX_TRY(spx_check(ctx, A, &ok));
    if (!ok) return fail(SPX_EINVAL, "A is not canonical");
  }
  auto* P = new SprefPlan(ctx);
  std::unique_ptr<SprefPlan> guard(P);
  hipStream_t st = stream_of(ctx);
  Scratch& scr = P->scratch;
  P->A = make_operand(A);
  P->I = I;
  P->J = J;
  P->lenI = lenI;
  P->lenJ = lenJ;
  const int64_t m = A->m;
  const int cus = device_cu_count();
  unsigned long long *ncls = nullptr, *nwide = nullptr;
  int32_t *rank = nullptr, *wide = nullptr;
  unsigned* claimed = nullptr;
  const int64_t nblocks = ceil_div(lenJ, kScanTile);
  int64_t *sums = nullptr, *carry = nullptr;
  SPX_TRY(scr.get_many({Scratch::part(&nwide, 1), Scratch::part(&ncls, kNumCls), Scratch::part(&P->err, 4),
                        Scratch::part(&claimed, 4), Scratch::part(&P->rcnt, m + 1), Scratch::part(&P->rbeg, m),
                        Scratch::part(&rank, lenI), Scratch::part(&P->rpos, lenI), Scratch::part(&P->qa0, lenJ),
                        Scratch::part(&P->qlen, lenJ), Scratch::part(&P->cnt, lenJ), Scratch::part(&P->off, lenJ + 1),
                        Scratch::part(&P->list, kNumCls * lenJ), Scratch::part(&wide, lenJ),
                        Scratch::part(&sums, nblocks)}));
  SPX_TRY(zero_words(st, {{nwide, 1}, {ncls, kNumCls}, {P->err, 2}, {claimed, 2}, {P->rcnt, ceil_div(m, 2)},
                          {P->off, 1}}));
  int64_t *aux = nullptr, chunk = 1;
  SPX_TRY(build_aux(P->A, scr, st, &aux, &chunk));
  if (lenI + lenJ > 0) {
    k_ref_start<<<grid_for(lenI + lenJ, 256, 4096), 256, 0, st>>>(P->A, aux, chunk, I, lenI, J, lenJ, P->rcnt, rank,
                                                                  P->qa0, P->qlen, P->cnt, wide, nwide, P->err);
    SPX_HIP(hipGetLastError());
  }
  if (lenI > 0) {  // transpose of R: the positions grouped by row
    k_ref_claim<<<grid_for(lenI, 256 * kClaimPer, 4096), 256, 0, st>>>(I, lenI, m, P->rcnt, rank, P->rbeg, claimed);
    SPX_HIP(hipGetLastError());
    k_ref_scatter<<<grid_for(lenI, 256, 4096), 256, 0, st>>>(I, lenI, m, rank, P->rbeg, P->rpos);
    SPX_HIP(hipGetLastError());
  }
  if (lenJ > 0) {
    const unsigned sb = grid_for(lenJ, 16, (int64_t)cus * 16);
    const unsigned lb = kRefShare * grid_for(std::min(lenJ, A->nnz / kRefSplit), 1, cus);
    k_ref_count<<<sb + lb, 256, 0, st>>>(P->A, P->qa0, P->qlen, P->rcnt, lenJ, wide, nwide, lb,
                                         (unsigned long long*)P->cnt);
    SPX_HIP(hipGetLastError());
    if (nblocks > 1) {
      k_scan_reduce<LoadI64><<<(unsigned)nblocks, kScanThreads, 0, st>>>(LoadI64{P->cnt}, lenJ, sums);
      SPX_HIP(hipGetLastError());
    }
    if (nblocks > kFusedCarry) {
      SPX_TRY(scr.get_n(nblocks + 1, &carry));
      SPX_TRY(exclusive_scan(LoadI64{sums}, nblocks, carry, scr, st));
    }
    k_ref_apply<<<(unsigned)nblocks, kScanThreads, 0, st>>>(P->cnt, P->qlen, lenJ, carry, sums, P->off, ncls, P->list);
    SPX_HIP(hipGetLastError());
  }
  int64_t h[kNumCls + 2] = {};
  SPX_TRY(read_device_words(st, {{ncls, 8, kNumCls}, {P->off + lenJ, 8}, {P->err, 4}}, h));
  if (h[kNumCls + 1] & 1) return fail(SPX_EINVAL, "I has an index outside [0, m)");
  if (h[kNumCls + 1] & 2) return fail(SPX_EINVAL, "J has an index outside [0, n)");
  for (int c = 0; c < kNumCls; ++c) P->ncls[c] = h[c];
  const int64_t nnz = h[kNumCls];
  P->nnz = nnz;
  if (nnz_b) *nnz_b = nnz;
  *plan = guard.release();
  return SPX_OK;
}

extern "C" int spx_spref_exec(spx_plan* plan, spx_mat* B) {
  if (!plan || plan->kind != kPlanSpref) return fail(SPX_EINVAL, "not a SpRef plan");
  auto* P = static_cast<SprefPlan*>(plan);
  if (!B) return fail(SPX_EINVAL, "B is NULL");
  if (B->m != P->lenI || B->n != P->lenJ || B->fmt != SPX_CSC) return fail(SPX_EINVAL, "B must be lenI x lenJ CSC");
  if (B->val_t != P->A.val_t) return fail(SPX_EINVAL, "B's value type must be A's");
  if (B->ptr_t == SPX_PTR_I32 && P->nnz >= (1ll << 31)) return fail(SPX_EOVERFLOW, "nnz(B) needs I64 pointers");
  if (!B->cp || (P->nnz > 0 && (!B->ir || (B->val_t != SPX_VAL_BOOL && !B->num))))
    return fail(SPX_EINVAL, "B buffers missing");
  B->nnz = P->nnz;
  B->nzc = 0;
  hipStream_t st = stream_of(&P->ctx);
  const int vb = value_size(P->A.val_t);
  const int cus = device_cu_count();
  const int64_t* nc = P->ncls;
  const auto list = [&](int c) { return P->list + c * P->lenJ; };
  // the workgroup columns (few and long) run beside the one-wave classes
  SideJoin side{nullptr, st};
  if (nc[kClsMedium] > 0) {
    hipStream_t ms = st;
    if (nc[kClsSmall] + nc[kClsMid] > 0) {
      SPX_TRY(side_fork(st, &side.ss));
      ms = side.ss->s;
    }
    const int64_t W = ceil_div(P->lenI, 64);
    const size_t lds = P->lenI <= kRankBits ? (size_t)(8 * kRefMedium + 10 * W + 16) : (size_t)12 * kRefMedium;
    const int64_t per_cu = lds > 78 * 1024 ? 1 : 2;
    k_ref_medium<<<(unsigned)std::min<int64_t>(nc[kClsMedium], (int64_t)cus * per_cu), kRefThreads, lds, ms>>>(
        P->A, P->qa0, P->qlen, P->rcnt, P->rbeg, P->rpos, list(kClsMedium), nc[kClsMedium], P->lenI, P->off, vb, B->ir,
        B->num);
    SPX_HIP(hipGetLastError());
  }
  if (nc[kClsSmall] > 0) {
    k_ref_wave<kClsSmall><<<grid_for(nc[kClsSmall], 4, (int64_t)cus * 16), 256, 0, st>>>(
        P->A, P->qa0, P->qlen, P->rcnt, P->rbeg, P->rpos, list(kClsSmall), nc[kClsSmall], P->lenI, P->off, vb, B->ir,
        B->num);
    SPX_HIP(hipGetLastError());
  }
  if (nc[kClsMid] > 0) {
    k_ref_wave<kClsMid><<<grid_for(nc[kClsMid], 4, (int64_t)cus * 8), 256, 0, st>>>(
        P->A, P->qa0, P->qlen, P->rcnt, P->rbeg, P->rpos, list(kClsMid), nc[kClsMid], P->lenI, P->off, vb, B->ir,
        B->num);
    SPX_HIP(hipGetLastError());
  }
  if (nc[kClsLarge] > 0) {
    k_ref_large<<<grid_for(nc[kClsLarge], 1, (int64_t)cus * 2), 1024, 0, st>>>(
        P->A, P->qa0, P->qlen, P->I, P->lenI, list(kClsLarge), nc[kClsLarge], P->off, vb, B->ir, B->num);
    SPX_HIP(hipGetLastError());
  }
  SPX_TRY(side.join());
  k_write_cp<<<grid_for(P->lenJ + 1, 256, 65536), 256, 0, st>>>(P->off, P->lenJ, B->cp, B->ptr_t);
  SPX_HIP(hipGetLastError());
  return SPX_OK;
}

extern "C" int spx_spref(const spx_ctx* ctx, const spx_mat* A, const int32_t* I, int64_t lenI, const int32_t* J,
                         int64_t lenJ, spx_mat* B) {
  if (!B) return fail(SPX_EINVAL, "B is NULL");
  spx_plan* plan = nullptr;
  int64_t nnz = 0;
  SPX_TRY(spx_spref_plan(ctx, A, I, lenI, J, lenJ, &plan, &nnz));
  std::unique_ptr<spx_plan> guard(plan);
  OutAlloc oa(ctx);
  spx_mat out{};
  out.m = lenI;
  out.n = lenJ;
  out.fmt = SPX_CSC;
  out.ptr_t = SPX_PTR_I64;
  out.val_t = A->val_t;
  const int vb = value_size(A->val_t);
  SPX_TRY(oa.get((size_t)(lenJ + 1) * 8, &out.cp));
  SPX_TRY(oa.get((size_t)std::max<int64_t>(nnz, 1) * 4, reinterpret_cast<void**>(&out.ir)));
  if (vb) SPX_TRY(oa.get((size_t)std::max<int64_t>(nnz, 1) * vb, &out.num));
  SPX_TRY(spx_spref_exec(plan, &out));
  oa.keep();
  *B = out;
  return SPX_OK;
}
