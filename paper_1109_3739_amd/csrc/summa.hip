// Sparse SUMMA stage accumulation on one GPU (Section 3.3, Algorithm 2).
//
// On a sqrt(p) x sqrt(p) grid, processor (i,j) accumulates
// C_ij = C_ij + A_ik * B_kj over the stages k.  When all stage blocks of one
// processor are resident in HBM, the stages are one product over a longer
// inner dimension:
//     sum_k A_k * B_k = [A_1 A_2 ... A_K] * [B_1; B_2; ...; B_K].
// Every output column then gathers the products of all stages into one LDS
// accumulator (the accumulators of the stage products stay live across the
// stages), so no partial C_ij is written, re-read or merged.
//
// The plan builds the two concatenated patterns once:
//   * left:  DCSC, m x sum(b_k); the stored columns of every A_k, moved to
//            the stage's column range (its row ids and values are A_k's,
//            one after the other).  A CSC block's empty columns are listed too:
//            a look-up finds them with length zero, and leaving them out would
//            take a scan and a read-back of their number;
//   * right: CSC, sum(b_k) x n; column j lists B_1(:,j), B_2(:,j) + b_1, ...
//            in stage order, so rows stay ascending.
// and a SpGEMM plan over them.  Exec copies the values of the stage blocks
// into the concatenations and runs the SpGEMM numeric phase.
#include <algorithm>
#include <cstring>
#include <vector>

#include "common.h"
#include "operand.h"
#include "plan.h"
#include "scan.h"

namespace spx {

struct SumPlan : spx_plan {
  explicit SumPlan(const spx_ctx* c) : spx_plan(c, kPlanSum) {}
  ~SumPlan() override {
    if (gemm) spx_plan_destroy(gemm);
  }
  int32_t count = 0;
  int vb_a = 0, vb_b = 0;
  std::vector<Operand> a_h, b_h;  // the stage blocks
  std::vector<int64_t> base_h;    // nnz bases of the A_k and B_k, slot bases, column bases, B's slot bases (count+1 each)
  std::vector<char> table_h;      // those, as copied to the device
  Operand* a_d = nullptr;
  Operand* b_d = nullptr;
  int64_t* anzb = nullptr;   // [count+1] nnz bases of the A_k
  int64_t* bnzb = nullptr;   // [count+1] nnz bases of the B_k
  int64_t* slotb = nullptr;  // [count+1] slot bases of the A_k
  int64_t* colb = nullptr;   // [count+1] column bases of the A_k (= row bases of the B_k)
  int64_t* bslotb = nullptr;  // [count+1] slot bases of the B_k
  int32_t* ajc = nullptr;
  int64_t* acp = nullptr;
  int32_t* air = nullptr;
  void* anum = nullptr;
  int64_t* bcp = nullptr;
  int32_t* bir = nullptr;
  void* bnum = nullptr;
  int64_t* bmap = nullptr;  // position in the right concatenation of every B_k entry
  spx_plan* gemm = nullptr;
};

// The left concatenation: column ids and pointers of every stage's slots, and
// the row ids of its entries.  The work of a stage is small (8 stages of 2^17
// columns: 0.9 M entries), so launches bound the plan: one takes all stages here
// and below (stage = blockIdx.y).  With a launch or copy per stage that product
// took 1.68 ms, with these 1.39.
__global__ void k_sum_left(const Operand* a, const int64_t* slotb, const int64_t* colb, const int64_t* anzb, int count,
                           int32_t* jc, int64_t* cp, int32_t* ir) {
  for (int k = blockIdx.y; k < count; k += gridDim.y) {
    const Operand X = a[k];
    const int64_t ns = slotb[k + 1] - slotb[k], ne = anzb[k + 1] - anzb[k];
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = i0; t < ns; t += step) {
      jc[slotb[k] + t] = (int32_t)(colb[k] + slot_col(X, t));
      cp[slotb[k] + t] = anzb[k] + slot_begin(X, t);
    }
    for (int64_t e = i0; e < ne; e += step) ir[anzb[k] + e] = X.ir[e];
    if (k == count - 1 && i0 == 0) cp[slotb[count]] = anzb[count];
  }
}

// Column lengths of all stages of B (which share the n columns): len[k n + j],
// zero on entry.
__global__ void k_sum_right_count(const Operand* b, int count, int64_t n, uint32_t* len) {
  for (int k = blockIdx.y; k < count; k += gridDim.y) {
    const Operand X = b[k];
    const int64_t ns = nslots_of(X);
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < ns; t += (int64_t)gridDim.x * blockDim.x)
      len[k * n + slot_col(X, t)] = (uint32_t)(slot_begin(X, t + 1) - slot_begin(X, t));
  }
}

// Per column: the lengths become the stages' offsets in the column, and cnt[j]
// what they end at.
__global__ void k_sum_right_offsets(int count, int64_t n, uint32_t* len, int64_t* cnt) {
  for (int64_t j = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
    uint32_t run = 0;  // a column has fewer than 2^31 entries (its rows are below 2^31)
    for (int k = 0; k < count; ++k) {
      const uint32_t x = len[k * n + j];
      len[k * n + j] = run;
      run += x;
    }
    cnt[j] = run;
  }
}

// The offsets of one stage's stored columns only, off[t] for slot t, where
// cnt[j] holds the entries of the stages before it (one launch per stage, in order).
__global__ void k_sum_right_chain(Operand X, int64_t* cnt, uint32_t* off) {
  const int64_t ns = nslots_of(X);
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < ns; t += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = slot_col(X, t), before = cnt[j];
    off[t] = (uint32_t)before;
    cnt[j] = before + slot_begin(X, t + 1) - slot_begin(X, t);
  }
}

// Places every stage's columns (rows moved down by the stage's row base) at
// their offsets: off[k n + j], or with bslot off[bslot[k] + t].  A wave takes
// four slots at a time, one per 16-lane group; slots of more than 64 entries
// then take the whole wave.
__global__ void __launch_bounds__(256) k_sum_right_place(const Operand* b, const int64_t* colb, const int64_t* bnzb,
                                                         int count, int64_t n, const int64_t* bcp, const uint32_t* off,
                                                         const int64_t* bslot, int32_t* ir, int64_t* map) {
  const int lane = lane_id(), gl = lane & 15;
  const int64_t w0 = (blockIdx.x * (int64_t)blockDim.x + threadIdx.x) / kWave;
  const int64_t nw = (int64_t)gridDim.x * blockDim.x / kWave;
  for (int k = blockIdx.y; k < count; k += gridDim.y) {
    const Operand X = b[k];
    const int64_t ns = nslots_of(X), rowb = colb[k];
    int64_t* mp = map + bnzb[k];
    for (int64_t base = w0 * 4; base < ns; base += nw * 4) {
      const int64_t t = base + (lane >> 4);
      int64_t s0 = 0, s1 = 0, dst = 0;
      if (t < ns) {
        s0 = slot_begin(X, t);
        s1 = slot_begin(X, t + 1);
        const int64_t j = slot_col(X, t);
        dst = bcp[j] + off[bslot ? bslot[k] + t : k * n + j];
      }
      const bool whole = s1 - s0 > kWave;
      if (!whole)
        for (int64_t e = s0 + gl; e < s1; e += 16) {
          ir[dst + (e - s0)] = (int32_t)(X.ir[e] + rowb);
          mp[e] = dst + (e - s0);
        }
      uint64_t rest = __ballot(whole && gl == 0);
      while (rest) {  // uniform
        const int src = __ffsll((unsigned long long)rest) - 1;
        rest &= rest - 1;
        const int64_t a0 = __shfl(s0, src), a1 = __shfl(s1, src), d = __shfl(dst, src);
        for (int64_t e = a0 + lane; e < a1; e += kWave) {
          ir[d + (e - a0)] = (int32_t)(X.ir[e] + rowb);
          mp[e] = d + (e - a0);
        }
      }
    }
  }
}

// Values of both concatenations: the left one's stages lie one after the
// other, the right one's scatter through the map.
__global__ void k_sum_vals(const Operand* a, const int64_t* anzb, int va, void* aout, const Operand* b,
                           const int64_t* bnzb, const int64_t* map, int vb, void* bout, int count) {
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  for (int k = blockIdx.y; k < count; k += gridDim.y) {
    if (va) {
      const int64_t len = anzb[k + 1] - anzb[k];
      const void* src = a[k].num;
      for (int64_t e = i0; e < len; e += step) copy_value(src, e, aout, anzb[k] + e, va);
    }
    if (vb) {
      const int64_t len = bnzb[k + 1] - bnzb[k];
      const void* src = b[k].num;
      for (int64_t e = i0; e < len; e += step) copy_value(src, e, bout, map[bnzb[k] + e], vb);
    }
  }
}

// Where a stage's part of a column begins comes from a table of all stages' column
// lengths (two launches for all stages), or from a launch per stage over its stored
// columns only.  The table is taken while the stages store at least an eighth of its
// columns, so that no pass or buffer is proportional to (stages x columns) of
// hypersparse blocks; and while it is short all the same, since launches are dear.
// Plan and exec by table | by stage: 8 stages of 2^17 entries, DCSC, n = 2^20 416 | 433
// us, 2^21 488 | 470, 2^24 1630 | 1230; 64 of 2^14, n = 2^19 649 | 720; in CSC, n = 2^22
// 2515 | 2835.  Always by table, n = 2^27 took 19.2 ms, now 6.9.
constexpr int64_t kLenCols = 1ll << 20;
constexpr int64_t kLenTable = 1ll << 26;  // words, 256 MiB
static bool by_table(int64_t stored, int64_t n, int count) {
  return 8 * stored >= n * count || (n <= kLenCols && n * count <= kLenTable);
}

// Grid over the elements of the largest stage (x) and the stages (y).
static dim3 stage_grid(int64_t widest, int per_block, int count) {
  return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(widest, per_block), 2048)),
              (unsigned)std::min(count, 64));
}

const spx_plan* sum_plan_inner(const spx_plan* plan) { return static_cast<const SumPlan*>(plan)->gemm; }

}  // namespace spx

using namespace spx;

extern "C" int spx_spgemm_sum_plan(const spx_ctx* ctx, int32_t count, const spx_mat* A, const spx_mat* B,
                                   int32_t semiring, int32_t c_fmt, const spx_tuning* tuning, spx_plan** plan,
                                   int64_t* nnz_c, int64_t* nzc_c) {
  if (!plan) return fail(SPX_EINVAL, "plan is NULL");
  *plan = nullptr;
  if (count < 1 || !A || !B) return fail(SPX_EINVAL, "need count >= 1 stage blocks");
  int64_t inner = 0, anz = 0, bnz = 0, slots = 0;
  for (int k = 0; k < count; ++k) {
    SPX_TRY(check_mat(&A[k], "A_k"));
    SPX_TRY(check_mat(&B[k], "B_k"));
    if (A[k].m != A[0].m || B[k].n != B[0].n) return fail(SPX_EINVAL, "stage blocks must share m (A) and n (B)");
    if (A[k].n != B[k].m) return fail(SPX_EINVAL, "inner dimensions of a stage differ");
    if (A[k].val_t != A[0].val_t || B[k].val_t != B[0].val_t)
      return fail(SPX_EINVAL, "stage blocks must share value types");
    inner += A[k].n;
    anz += A[k].nnz;
    bnz += B[k].nnz;
  }
  if (inner >= (1ll << 31)) return fail(SPX_EUNSUPPORTED, "the summed inner dimension must be below 2^31");
  if (ctx && ctx->validate) {
    for (int k = 0; k < count; ++k) {
      int32_t ok = 0;
      SPX_TRY(spx_check(ctx, &A[k], &ok));
      if (!ok) return fail(SPX_EINVAL, "A_k is not canonical");
      SPX_TRY(spx_check(ctx, &B[k], &ok));
      if (!ok) return fail(SPX_EINVAL, "B_k is not canonical");
    }
  }
  auto* P = new SumPlan(ctx);
  std::unique_ptr<SumPlan> guard(P);
  hipStream_t st = stream_of(ctx);
  Scratch& scr = P->scratch;
  P->count = count;
  P->vb_a = value_size(A[0].val_t);
  P->vb_b = value_size(B[0].val_t);
  const int64_t m = A[0].m, n = B[0].n;
  P->base_h.assign(5 * (count + 1), 0);
  int64_t* const anzb = P->base_h.data();
  int64_t *const bnzb = anzb + count + 1, *const slotb = bnzb + count + 1, *const colb = slotb + count + 1;
  int64_t* const bslotb = colb + count + 1;
  int64_t wide_a = 0, wide_b = 0, wide_bs = 0;  // largest stage: A's slots or entries, B's entries, B's slots
  for (int k = 0; k < count; ++k) {
    P->a_h.push_back(make_operand(&A[k]));
    P->b_h.push_back(make_operand(&B[k]));
    slotb[k + 1] = slotb[k] + nslots_of(P->a_h[k]);
    colb[k + 1] = colb[k] + A[k].n;
    anzb[k + 1] = anzb[k] + A[k].nnz;
    bnzb[k + 1] = bnzb[k] + B[k].nnz;
    bslotb[k + 1] = bslotb[k] + nslots_of(P->b_h[k]);
    wide_a = std::max({wide_a, nslots_of(P->a_h[k]), A[k].nnz});
    wide_b = std::max(wide_b, B[k].nnz);
    wide_bs = std::max(wide_bs, nslots_of(P->b_h[k]));
  }
  slots = slotb[count];
  const bool tabled = by_table(bslotb[count], n, count);
  // stage tables in one copy (the host bytes live as long as the plan)
  const size_t ops = sizeof(Operand) * count, bases = sizeof(int64_t) * P->base_h.size();
  P->table_h.resize(2 * ops + bases);
  std::memcpy(P->table_h.data(), P->a_h.data(), ops);
  std::memcpy(P->table_h.data() + ops, P->b_h.data(), ops);
  std::memcpy(P->table_h.data() + 2 * ops, P->base_h.data(), bases);
  char* table = nullptr;
  int64_t* cnt = nullptr;
  uint32_t* off = nullptr;  // offsets of the stages' columns: the table, or one per stored column
  SPX_TRY(scr.get_many({Scratch::part(&table, (int64_t)P->table_h.size()), Scratch::part(&P->ajc, slots),
                        Scratch::part(&P->acp, slots + 1), Scratch::part(&P->air, anz), Scratch::part(&cnt, n),
                        Scratch::part(&P->bcp, n + 1), Scratch::part(&P->bir, bnz), Scratch::part(&P->bmap, bnz),
                        Scratch::part(&off, tabled ? count * n + 1 : bslotb[count])}));
  if (P->vb_a) SPX_TRY(scr.get(std::max<int64_t>(anz, 1) * P->vb_a, &P->anum));
  if (P->vb_b) SPX_TRY(scr.get(std::max<int64_t>(bnz, 1) * P->vb_b, &P->bnum));
  static_assert(sizeof(Operand) % sizeof(int64_t) == 0, "the bases follow the operands");
  P->a_d = reinterpret_cast<Operand*>(table);
  P->b_d = P->a_d + count;
  P->anzb = reinterpret_cast<int64_t*>(table + 2 * ops);
  P->bnzb = P->anzb + count + 1;
  P->slotb = P->bnzb + count + 1;
  P->colb = P->slotb + count + 1;
  P->bslotb = P->colb + count + 1;
  SPX_HIP(hipMemcpyAsync(table, P->table_h.data(), P->table_h.size(), hipMemcpyHostToDevice, st));

  // left concatenation (DCSC)
  k_sum_left<<<stage_grid(wide_a, 256, count), 256, 0, st>>>(P->a_d, P->slotb, P->colb, P->anzb, count, P->ajc, P->acp,
                                                             P->air);
  SPX_HIP(hipGetLastError());
  // right concatenation (CSC)
  if (n > 0 && tabled) {
    SPX_TRY(zero_words(st, {{off, ceil_div(count * n, 2)}}));
    k_sum_right_count<<<stage_grid(wide_bs, 256, count), 256, 0, st>>>(P->b_d, count, n, off);
    SPX_HIP(hipGetLastError());
    k_sum_right_offsets<<<grid_for(n, 256, 4096), 256, 0, st>>>(count, n, off, cnt);
    SPX_HIP(hipGetLastError());
  } else if (n > 0) {
    SPX_TRY(zero_words(st, {{cnt, n}}));
    for (int k = 0; k < count; ++k) {
      const int64_t ns = nslots_of(P->b_h[k]);
      if (ns == 0 || B[k].nnz == 0) continue;
      k_sum_right_chain<<<grid_for(ns, 256, 4096), 256, 0, st>>>(P->b_h[k], cnt, off + bslotb[k]);
      SPX_HIP(hipGetLastError());
    }
  }
  SPX_TRY(exclusive_scan(LoadI64{cnt}, n, P->bcp, scr, st));
  if (bnz > 0) {
    k_sum_right_place<<<stage_grid(wide_bs, 16, count), 256, 0, st>>>(P->b_d, P->colb, P->bnzb, count, n, P->bcp, off,
                                                                      tabled ? nullptr : P->bslotb, P->bir, P->bmap);
    SPX_HIP(hipGetLastError());
  }

  // one SpGEMM over the concatenations
  spx_mat Ac{}, Bc{};
  Ac.m = m;
  Ac.n = inner;
  Ac.nnz = anz;
  Ac.nzc = slots;
  Ac.fmt = SPX_DCSC;
  Ac.ptr_t = SPX_PTR_I64;
  Ac.val_t = A[0].val_t;
  Ac.jc = P->ajc;
  Ac.cp = P->acp;
  Ac.ir = P->air;
  Ac.num = P->anum;
  Bc.m = inner;
  Bc.n = n;
  Bc.nnz = bnz;
  Bc.fmt = SPX_CSC;
  Bc.ptr_t = SPX_PTR_I64;
  Bc.val_t = B[0].val_t;
  Bc.cp = P->bcp;
  Bc.ir = P->bir;
  Bc.num = P->bnum;
  spx_ctx c2 = ctx ? *ctx : spx_ctx{};
  c2.validate = 0;
  SPX_TRY(spx_spgemm_plan(&c2, &Ac, &Bc, semiring, c_fmt, tuning, &P->gemm, nnz_c, nzc_c));
  *plan = guard.release();
  return SPX_OK;
}

extern "C" int spx_spgemm_sum_exec(spx_plan* plan, spx_mat* C) {
  if (!plan || plan->kind != kPlanSum) return fail(SPX_EINVAL, "not a stage-sum plan");
  auto* P = static_cast<SumPlan*>(plan);
  hipStream_t st = stream_of(&P->ctx);
  int64_t widest = 0;
  for (int k = 0; k < P->count; ++k)
    widest = std::max({widest, P->vb_a ? P->a_h[k].nnz : 0, P->vb_b ? P->b_h[k].nnz : 0});
  if (widest > 0) {
    k_sum_vals<<<stage_grid(widest, 256, P->count), 256, 0, st>>>(P->a_d, P->anzb, P->vb_a, P->anum, P->b_d, P->bnzb,
                                                                  P->bmap, P->vb_b, P->bnum, P->count);
    SPX_HIP(hipGetLastError());
  }
  return spx_spgemm_exec(P->gemm, C);
}
