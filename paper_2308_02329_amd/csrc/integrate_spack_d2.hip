// Instantiates the packed streamed-J integrators for d = 2.
#include "integrate_spack.h"

namespace chym {
SpackFn lookup_spack_2(int tpw, int xs, int js) { return spack_lookup<2>(tpw, xs, js); }
}  // namespace chym
