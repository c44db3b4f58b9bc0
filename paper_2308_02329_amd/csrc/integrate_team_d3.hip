// Instantiates the team integrators for d = 3.
#include "integrate_team.h"

namespace chym {
TeamFn lookup_team_3(int tiles, int xs, int js, bool pack, bool map) {
    return team_lookup<3>(tiles, xs, js, pack, map);
}
}  // namespace chym
