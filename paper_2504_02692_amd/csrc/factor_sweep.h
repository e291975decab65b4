// The factor sweep of gptaq_prepare (factor_sweep.hip).
#pragma once
#include "common.h"
#include "split_rows.h"

namespace gptaq {

// F: n x n, upper triangle: H + lambda I in, U out.  Everything else but `split` is scratch.
struct FactorSweep {
  double* F; int64_t ldf; int n;
  int32_t* info;                     // set to 1 + index of the first pivot that is not positive, unless set already
  double *V, *T, *Uob;               // kFactorTileBytes, kHalfTileBytes, kFactorBlock^2
  int32_t* sync;                     // kBlockSyncBytes a block, zeros
  I8Operand Vs[3], UJ[2], Ucol[2], Urow;   // digits: of V_I,OB, U_OB,J and the columns of U_OB,OB (three and two blocks' in turn), of its rows
  SplitRows split;                   // taken beside the first block
};
hipError_t launch_factor_sweep(const FactorSweep& w, hipStream_t s);

}  // namespace gptaq
