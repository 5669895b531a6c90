// The Lloyd kernel for rows of up to 48 features (one translation unit per row length: they compile side
// by side).
#include "kb_cluster_lloyd.h"

namespace kb {
template hipError_t launch_lloyd<3>(const ClusterArgs&, const LloydForm&, hipStream_t);
}  // namespace kb
