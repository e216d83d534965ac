// The column-reduction sweep (pass 2) of the importance scoring: see score_sweep.h.
#include "score_sweep.h"

namespace speckv {

hipError_t launch_column_sweep(const ScoreArgs &A, hipStream_t st) { return dispatch_sweep<2>(A, st); }

}  // namespace speckv
