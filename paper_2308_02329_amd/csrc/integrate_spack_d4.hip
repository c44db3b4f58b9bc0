// Instantiates the packed streamed-J integrators for d = 4.
#include "integrate_spack.h"

namespace chym {
SpackFn lookup_spack_4(int tiles, int xs, int js) { return spack_lookup<4>(tiles, xs, js); }
}  // namespace chym
