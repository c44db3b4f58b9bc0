// Instantiates the team integrators for d = 2.
#include "integrate_team.h"

namespace chym {
TeamFn lookup_team_2(int tiles, int xs, int js, bool pack, bool map) {
    return team_lookup<2>(tiles, xs, js, pack, map);
}
}  // namespace chym
