// Instantiates the team integrators for d = 1.
#include "integrate_team.h"

namespace chym {
TeamFn lookup_team_1(int tiles, int xs, int js, bool pack, bool map) {
    return team_lookup<1>(tiles, xs, js, pack, map);
}
}  // namespace chym
