// fp32 gradient kernel of the learner for hidden size 64
#include "learn_block.h"

namespace msrl {
MSRL_BLOCK_LAUNCHER(64)
}  // namespace msrl
