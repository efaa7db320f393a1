// Instantiations of the team kernels (dsq_team_impl.h) for one family of compressors.
#include "dsq_team_impl.h"

namespace dsq {

void team_plans_quant4(int block, int n, std::vector<TilePlan>& plans) {
    team_plans_for_kind<DS_COMP_QUANT_MAXABS, 4>(block, n, plans);
}

}  // namespace dsq
