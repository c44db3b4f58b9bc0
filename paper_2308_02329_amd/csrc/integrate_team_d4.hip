// Instantiates the team integrators for d = 4.
#include "integrate_team.h"

namespace chym {
TeamFn lookup_team_4(int tiles, int xs, int js, bool pack, bool map) {
    return team_lookup<4>(tiles, xs, js, pack, map);
}
}  // namespace chym
