// Instantiates the packed streamed-J integrators for d = 4.
#include "integrate_spack.h"

namespace chym {
SpackFn lookup_spack_4(int tpw, int xs, int js) { return spack_lookup<4>(tpw, xs, js); }
}  // namespace chym
