// fp32 gradient kernel of the learner for hidden size 256
#include "learn_block.h"

namespace msrl {
MSRL_BLOCK_LAUNCHER(256)
}  // namespace msrl
