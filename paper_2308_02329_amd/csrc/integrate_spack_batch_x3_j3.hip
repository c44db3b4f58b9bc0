// Instantiates the packed streamed-J integrators of batches for 3 state and 3 coupling terms.
#include "integrate_spack.h"

namespace chym {
SpackBatchFn lookup_spack_batch_3_3(int tpw) { return spack_batch_lookup<3, 3>(tpw); }
}  // namespace chym
