// Shared between the code generator and the launcher: where each value sits in
// the kernel's argument block (an array of 8-byte slots passed by value).
#pragma once

#include <string>
#include <vector>

#include "ir.h"

namespace gr {

struct ArgLayout {
  std::vector<int> ptr;        // per access group: slot of the buffer pointer
  std::vector<int> base;       // per access group: slot of the base element offset
  std::vector<int> coef;       // per access group: first of `ncoef[g]` coefficient slots
  std::vector<int> ncoef;
  int out = 0;                 // output pointer
  int dims = 0;                // first of `rank` extents
  int consts = 0;              // first constant slot
  int extra = 0;               // kind-specific: GEMV {M, K, workspace, slabs}; REDUCE {outputs, length, workspace, splits};
                               // SCAN {lines, chunk length, workspace, chunks}
  int ocoef = 0;               // SCAN, MAP: first of `rank` output strides
  int obase = 0;               // MAP: element offset of the output's first element
  int total = 0;
};

ArgLayout arg_layout(const GroupPlan& g);

// Rows of the scalar operand that a workgroup of a pair kernel (gen_rowred_pairs) takes, at most.
// (LDS for 256 lanes' results: 20 KiB, seven workgroups per compute unit.  Blocks of 32 against 16 rows, us: 262144 x 32
// pairs of 16 elements 19.2 / 15.0, 292509 x 24 of 11 16.3 / 13.3, 65536 x 64 of 64 23.4 / 23.8, 973632 x 24 of 3 27.5 / 30.4.)
constexpr int kPairBlock = 16;
// Blocks of 256 of the lanes' rows from which on those of the same rows share an XCD.
constexpr int kPairSpread = 16;

// Lanes of a workgroup of the column reductions (REDUCE mode 0).
constexpr int kReduceLanes = 512;

// Splits of a reduction from which on the kernel that combines the partial results of 1024 outputs and more takes several lanes per output.
constexpr int kCombineSplits = 16;

// Chunks of a scanned line up to which, and lines from which on, a lane, not a workgroup, scans their totals.
constexpr int kScanFewChunks = 16, kScanManyLines = 4096;

// Columns up to which the kernel that combines the partial vectors of a matrix-vector product takes four of them per workgroup instead of sixteen.
constexpr int kCombineFew = 384;

// Ragged extents that a direct-to-LDS matrix product has compiled in (GroupPlan::NP): values of k beyond whole steps of 16, and
// dimensions, no multiple of four, along which an operand is contiguous.
constexpr int kGemmRestK = 16, kGemmShiftM = 32, kGemmShiftN = 64;

// Lanes of a workgroup of a matrix product's kernel.
inline unsigned gemm_threads(const GroupPlan& g) { return g.VR == 4 ? 64u * (g.UC > 1 ? (unsigned)g.UC : 4u) : (g.VR == 2 && g.UC == 2 ? 512u : 256u); }

// 'Z': no leaf dimension follows this iteration dimension; '1': unit stride; 'G': anything else.
char access_class(const AccessGroup& ag, int dim);

// Row-resident sums of squares accumulate with one fused multiply-add per element, as the contractions do: the instruction whose
// square phase `s` sums, -1 where the phase sums anything else.  (A square is not negative, so a sum overflows, or is not
// a number, exactly when it does with the square rounded first.  Rows of 1024 lanes add pairs of elements first.
// Squared distances, their minima and the launch of those included, us: 262144 points to 32 centres in 16 dimensions 20.2 -> 19.6, 100000 to 60 in
// 40 26.7 -> 24.1, 65536 to 64 in 64 26.3 -> 23.9; relative error 4.8e-8 -> 4.7e-8.)
int square_root_of(const GroupPlan& g, int s);

// Whether loads of this access group carry the non-temporal hint.
bool nontemporal_group(const GroupPlan& g, int group);

}  // namespace gr
