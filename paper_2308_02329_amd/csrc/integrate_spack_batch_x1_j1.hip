// Instantiates the packed streamed-J integrators of batches for 1 state and 1 coupling term.
#include "integrate_spack.h"

namespace chym {
SpackBatchFn lookup_spack_batch_1_1(int tpw) { return spack_batch_lookup<1, 1>(tpw); }
}  // namespace chym
