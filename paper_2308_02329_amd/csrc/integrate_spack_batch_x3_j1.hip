// Instantiates the packed streamed-J integrators of batches for 3 state and 1 coupling term.
#include "integrate_spack.h"

namespace chym {
SpackBatchFn lookup_spack_batch_3_1(int tpw) { return spack_batch_lookup<3, 1>(tpw); }
}  // namespace chym
