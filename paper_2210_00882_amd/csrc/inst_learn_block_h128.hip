// fp32 gradient kernel of the learner for hidden size 128
#include "learn_block.h"

namespace msrl {
MSRL_BLOCK_LAUNCHER(128)
}  // namespace msrl
