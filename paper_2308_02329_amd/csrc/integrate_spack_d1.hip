// Instantiates the packed streamed-J integrators for d = 1.
#include "integrate_spack.h"

namespace chym {
SpackFn lookup_spack_1(int tpw, int xs, int js) { return spack_lookup<1>(tpw, xs, js); }
}  // namespace chym
