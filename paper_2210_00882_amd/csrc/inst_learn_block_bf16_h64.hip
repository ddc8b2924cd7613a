// bf16 gradient kernel of the learner for hidden size 64
#include "learn_block_bf16.h"

namespace msrl {
MSRL_BLOCK_BF16_LAUNCHER(64)
}  // namespace msrl
