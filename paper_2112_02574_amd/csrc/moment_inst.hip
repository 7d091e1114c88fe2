// moment_inst.hip -- instantiates the moment-field step of one storage format
// and stencil order (SCMC_INST_STORE, SCMC_INST_ORDER, set by the build).
#include "moment_impl.h"

namespace scmc {
template struct MomOps<SCMC_INST_STORE, SCMC_INST_ORDER>;
}  // namespace scmc
