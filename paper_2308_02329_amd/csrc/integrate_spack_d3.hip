// Instantiates the packed streamed-J integrators for d = 3.
#include "integrate_spack.h"

namespace chym {
SpackFn lookup_spack_3(int tpw, int xs, int js) { return spack_lookup<3>(tpw, xs, js); }
}  // namespace chym
