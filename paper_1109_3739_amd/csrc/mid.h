// Output columns of 65 to 512 products, formed by one wave each (mid.hip).
#pragma once

#include "common.h"
#include "operand.h"
#include "wave.h"

namespace spx {

// Most products of a mid column: its hash-count bin has a table of at most
// 2^kMidHashLog2 keys.
constexpr int kMidHashLog2 = 10;
constexpr int kMidMax = 1 << (kMidHashLog2 - 1);

// Distinct rows of the columns list[beg, end) (at most kMidMax products each).
int launch_mid_count(const Operand& B, const ProdSrc& S, const int64_t* mults, const int32_t* list, int64_t beg,
                     int64_t end, int64_t* cnt, unsigned* err, hipStream_t st);

// Values and rows of the columns list[beg, end), at most 64 * regs products
// each (regs = 2, 4 or 8), written at off[column].
int launch_mid(int32_t sr, int32_t vt, int regs, const Operand& A, const Operand& B, const ProdSrc& S,
               const int32_t* list, int64_t beg, int64_t end, const int64_t* off, int32_t* cir, void* cnum,
               hipStream_t st);

}  // namespace spx
