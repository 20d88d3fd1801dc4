// SpGEMM columns of 65 to 512 products: one wave per column.
//
// A workgroup per column spends most of its time on a dozen barriers and
// dependent loads for work that fills two to eight registers of one wave, and
// its LDS (sized for the largest column it may meet) leaves three to five
// columns in flight per CU.  Here every wave takes its own column without a
// barrier: 16 to 32 columns are in flight per CU.  The count inserts the rows
// into an LDS table of the wave; the numeric pass sorts (row, product) keys in
// registers and folds the runs of equal rows.  Both wait on dependent loads (B
// pointers, A ranges, A's rows and values), so what counts is the number of
// waves in flight.
#include <algorithm>

#include "mid.h"
#include "plan.h"

namespace spx {

// The A ranges of up to 64 B entries, in the wave's LDS.
template <typename T, int MAXP>
struct WaveRanges {
  int64_t base[kWave];      // position in A of the entry's product 0, less its product number in the chunk
  T bval[kWave];            // B's value
  uint32_t own[MAXP / 4];   // bytes: 1 + the entry whose first product this is, else 0
};

// Walks the products of one column (at most MAXP): B's entries in chunks of 64
// (one per lane), the products of a chunk in windows of 64, U windows in flight
// together.  A lane finds its product's entry by a maximum scan over the marks
// of the entries' first products.  f(p, r, a, b): p is the column's product
// number of lane 0 in window 0, r[u] the row (-1: no product), a[u] and b[u]
// the values.  Returns the number of products.
template <int U, int MAXP, typename T, bool LOADA, bool LOADB, class F>
__device__ __forceinline__ int wave_products(const ProdSrc& S, const T* an, const T* bn, int64_t b0, int64_t b1,
                                             WaveRanges<T, MAXP>& R, F&& f) {
  const int lane = lane_id();
  uint8_t* own = reinterpret_cast<uint8_t*>(R.own);
  int done = 0;
  for (int64_t qc = b0; qc < b1; qc += kWave) {
    const int64_t q = qc + lane;
    const bool inq = q < b1;
    const int al = inq ? S.alen[q] : 0;
    const int64_t a0 = inq ? S.a0[q] : 0;
    T bq = T(0);
    if constexpr (LOADB) bq = inq ? bn[q] : T(0);
    const int incl = wave_incl_scan(al);
    int ctot = __builtin_amdgcn_readlane(incl, 63);
    if (ctot == 0) continue;
    if (ctot > MAXP - done) ctot = MAXP - done;  // cannot happen: the caller checked the column's products
    for (int i = lane; i * 4 < ctot; i += kWave) R.own[i] = 0;
    R.base[lane] = a0 - (incl - al);
    if constexpr (LOADB) R.bval[lane] = bq;
    wave_sync();
    if (al > 0 && incl - al < ctot) own[incl - al] = (uint8_t)(lane + 1);
    wave_sync();
    int carry = 0;
    for (int w = 0; w < ctot; w += U * kWave) {
      int o[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = w + u * kWave + lane;
        o[u] = p < ctot ? (int)own[p] : 0;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int s = group_scan<kWave>(o[u], 0, [](int x, int y) { return x > y ? x : y; });
        o[u] = s > carry ? s : carry;
        carry = __builtin_amdgcn_readlane(o[u], 63);
      }
      int32_t r[U];
      T a[U], b[U];
      int64_t e[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = w + u * kWave + lane;
        e[u] = R.base[o[u] - 1] + p;  // the first product of a chunk is marked, so o >= 1
        b[u] = T(0);
        if constexpr (LOADB) b[u] = R.bval[o[u] - 1];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int p = w + u * kWave + lane;
        r[u] = -1;
        a[u] = T(0);
        if (p < ctot) {
          r[u] = S.air[e[u]];
          if constexpr (LOADA) a[u] = an[e[u]];
        }
      }
      f(done + w, r, a, b);
    }
    done += ctot;
    wave_sync();  // the ranges are rewritten by the next chunk
  }
  return done;
}

// ------------------------------------------------------------------ count
// Distinct rows by insertion into the wave's table of 2^s keys, at least twice
// the number of products.
__global__ void __launch_bounds__(256) k_mid_count(Operand B, ProdSrc S, const int64_t* mults, const int32_t* list,
                                                   int64_t beg, int64_t end, int64_t* cnt, unsigned* err) {
  __shared__ __align__(16) uint32_t s_tab[4][1 << kMidHashLog2];
  __shared__ WaveRanges<float, kMidMax> s_rng[4];
  const int w = threadIdx.x / kWave, lane = lane_id();
  uint32_t* tab = s_tab[w];
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  for (int64_t pos = beg + (int64_t)blockIdx.x * 4 + w; pos < end; pos += nwaves) {
    const int32_t t = list[pos];
    const int64_t mu = mults[t];
    const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1);
    int log2s = ceil_log2_u64((uint64_t)mu) + 1;
    log2s = __builtin_amdgcn_readfirstlane(log2s < 8 ? 8 : (log2s > kMidHashLog2 ? kMidHashLog2 : log2s));
    const int TS = 1 << log2s;
    for (int i = lane; i < TS / 4; i += kWave) reinterpret_cast<uint4*>(tab)[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    wave_sync();
    int mine = 0;
    wave_products<4, kMidMax, float, false, false>(
        S, nullptr, nullptr, b0, b1, s_rng[w], [&](int, const int32_t(&r)[4], const float(&)[4], const float(&)[4]) {
          // first probes of the four windows together
          uint32_t h[4], old[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            h[u] = ((uint32_t)r[u] * 0x9E3779B1u) >> (32 - log2s);
            old[u] = r[u] >= 0 ? atomicCAS(&tab[h[u]], ~0u, (uint32_t)r[u]) : (uint32_t)r[u];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            for (int probe = 1; old[u] != ~0u && old[u] != (uint32_t)r[u]; ++probe) {
              if (probe > TS) {  // cannot happen: the table has twice the products' slots
                atomicOr(err, 2u);
                break;
              }
              h[u] = (h[u] + 1) & (TS - 1);
              old[u] = atomicCAS(&tab[h[u]], ~0u, (uint32_t)r[u]);
            }
            mine += r[u] >= 0 && old[u] == ~0u;
          }
        });
    const int total = __builtin_amdgcn_readlane(wave_incl_scan(mine), 63);
    if (lane == 0) cnt[t] = total;
    wave_sync();  // the table is cleared for the next column
  }
}

// ------------------------------------------------------------------ numeric
// Previous lane's value (DPP wave shift; 0 in lane 0).
__device__ __forceinline__ int lane_prev(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xF, 0xF, false); }

// One column per wave: gather the products into LDS, sort (row, product)
// keys, fold each run of equal rows and write the column in order.  K is
// uint32_t when the rows leave log2(64 R) bits for the product number, else
// uint64_t.
template <int SR, typename T, int R, typename K>
__device__ __forceinline__ void mid_column(const Operand& A, const Operand& B, const ProdSrc& S, int64_t b0, int64_t b1,
                                           int64_t o, int32_t* cir, T* cnum, T* s_x, T* s_v,
                                           WaveRanges<T, kWave * R>& rng) {
  using SR_ = Semiring<SR, T>;
  constexpr bool kVal = SR != SPX_OR_AND;
  constexpr int MAXP = kWave * R;
  constexpr int U = R < 4 ? R : 4;
  constexpr int kLog = R == 2 ? 7 : R == 4 ? 8 : 9;
  static_assert((1 << kLog) == MAXP, "product numbers fill the key's low bits");
  const int lane = lane_id();
  int32_t* s_row = reinterpret_cast<int32_t*>(s_x);  // rows by product, then the sums by rank
  const int total = wave_products<U, MAXP, T, SR_::kUsesA, SR_::kUsesB>(
      S, (const T*)A.num, (const T*)B.num, b0, b1, rng, [&](int p0, const int32_t(&r)[U], const T(&a)[U], const T(&b)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (r[u] < 0) continue;
          s_row[p0 + u * kWave + lane] = r[u];
          if constexpr (kVal) s_v[p0 + u * kWave + lane] = SR_::mul(a[u], b[u]);
        }
      });
  wave_sync();
  K key[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int i = k * kWave + lane;
    key[k] = i < total ? ((K)(uint32_t)s_row[i] << kLog) | (K)i : ~K(0);
  }
  sort_regs<R, K>(key, lane);
  int32_t row[R];
  T v[R];
#pragma unroll
  for (int k = 0; k < R; ++k) {
    row[k] = (int32_t)(key[k] >> kLog);
    v[k] = T(0);
    if constexpr (kVal) v[k] = lane * R + k < total ? s_v[(int)(key[k] & (MAXP - 1))] : T(0);
  }
  // heads of the runs of equal rows, and their ranks
  const int32_t before = lane_prev(row[R - 1]);
  bool head[R];
  int nh = 0;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const int pos = lane * R + k;
    head[k] = pos < total && (pos == 0 || row[k] != (k == 0 ? before : row[k > 0 ? k - 1 : 0]));
    nh += head[k];
  }
  const int hincl = wave_incl_scan(nh);
  const int c = __builtin_amdgcn_readlane(hincl, 63);
  // the keys are in registers and the values too: s_x takes the sums by rank,
  // s_v the rows by rank
  wave_sync();
  int32_t* rows = reinterpret_cast<int32_t*>(s_v);
  int rank = hincl - nh - 1;  // the run that reaches into this lane
  // Lanes cut a run into pieces, so a piece starts from the neutral element and folds
  // as the LDS does: started from its own first product, a NaN there hid the rest.
  T lead = T(0), acc = T(0);
  bool leads = false;
#pragma unroll
  for (int k = 0; k < R; ++k) {
    const bool in = lane * R + k < total;
    if (head[k]) {
      ++rank;
      rows[rank] = row[k];
      acc = SR_::fold(SR_::ident(), v[k]);
    } else if (k == 0) {
      acc = SR_::fold(SR_::ident(), v[0]);
      leads = in;
    } else if (in) {
      acc = SR_::fold(acc, v[k]);
    }
    if constexpr (kVal) {
      const bool last = k == R - 1 || head[k + 1 < R ? k + 1 : k] || lane * R + k + 1 >= total;
      if (in && last) {
        if (rank == hincl - nh - 1)
          lead = acc;  // started in an earlier lane
        else
          s_x[rank] = acc;
      }
    }
  }
  wave_sync();
  if constexpr (kVal) {
    if (leads) SR_::lds_acc(&s_x[hincl - nh - 1], lead);
    wave_sync();
  }
  for (int i = lane; i < c; i += kWave) {
    cir[o + i] = rows[i];
    if constexpr (kVal) cnum[o + i] = s_x[i];
  }
  wave_sync();  // the LDS is rewritten for the next column
}

template <int SR, typename T, int R>
__global__ void __launch_bounds__(256) k_mid(Operand A, Operand B, ProdSrc S, const int32_t* list, int64_t beg,
                                             int64_t end, const int64_t* off, int32_t* cir, T* cnum) {
  constexpr int MAXP = kWave * R;
  __shared__ __align__(16) T s_x[4][MAXP];
  __shared__ __align__(16) T s_v[4][MAXP];
  __shared__ WaveRanges<T, MAXP> s_rng[4];
  const int w = threadIdx.x / kWave;
  const int64_t nwaves = (int64_t)gridDim.x * 4;
  const bool narrow = A.m <= (1ll << 32) / MAXP;
  for (int64_t pos = beg + (int64_t)blockIdx.x * 4 + w; pos < end; pos += nwaves) {
    const int32_t t = list[pos];
    const int64_t b0 = slot_begin(B, t), b1 = slot_begin(B, t + 1), o = off[t];
    if (narrow)
      mid_column<SR, T, R, uint32_t>(A, B, S, b0, b1, o, cir, cnum, s_x[w], s_v[w], s_rng[w]);
    else
      mid_column<SR, T, R, uint64_t>(A, B, S, b0, b1, o, cir, cnum, s_x[w], s_v[w], s_rng[w]);
  }
}

// ------------------------------------------------------------------ host
int launch_mid_count(const Operand& B, const ProdSrc& S, const int64_t* mults, const int32_t* list, int64_t beg,
                     int64_t end, int64_t* cnt, unsigned* err, hipStream_t st) {
  if (end <= beg) return SPX_OK;
  k_mid_count<<<grid_for(end - beg, 4, (int64_t)device_cu_count() * 8), 256, 0, st>>>(B, S, mults, list, beg, end, cnt,
                                                                                      err);
  SPX_HIP(hipGetLastError());
  return SPX_OK;
}

template <int SR, typename T>
static int launch_mid_t(int regs, const Operand& A, const Operand& B, const ProdSrc& S, const int32_t* list, int64_t beg,
                        int64_t end, const int64_t* off, int32_t* cir, T* cnum, hipStream_t st) {
  const unsigned grid = grid_for(end - beg, 4, (int64_t)device_cu_count() * 8);
  if (regs == 2)
    hipLaunchKernelGGL((k_mid<SR, T, 2>), dim3(grid), dim3(256), 0, st, A, B, S, list, beg, end, off, cir, cnum);
  else if (regs == 4)
    hipLaunchKernelGGL((k_mid<SR, T, 4>), dim3(grid), dim3(256), 0, st, A, B, S, list, beg, end, off, cir, cnum);
  else
    hipLaunchKernelGGL((k_mid<SR, T, 8>), dim3(grid), dim3(256), 0, st, A, B, S, list, beg, end, off, cir, cnum);
  SPX_HIP(hipGetLastError());
  return SPX_OK;
}

int launch_mid(int32_t sr, int32_t vt, int regs, const Operand& A, const Operand& B, const ProdSrc& S,
               const int32_t* list, int64_t beg, int64_t end, const int64_t* off, int32_t* cir, void* cnum,
               hipStream_t st) {
  if (end <= beg) return SPX_OK;
#define SPX_CASE(SRV, VTV, TY) \
  if (sr == SRV && vt == VTV) return launch_mid_t<SRV, TY>(regs, A, B, S, list, beg, end, off, cir, (TY*)cnum, st);
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
#undef SPX_CASE
  return launch_mid_t<SPX_OR_AND, float>(regs, A, B, S, list, beg, end, off, cir, (float*)cnum, st);
}

}  // namespace spx
