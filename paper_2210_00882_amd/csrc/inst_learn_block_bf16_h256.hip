// bf16 gradient kernel of the learner for hidden size 256
#include "learn_block_bf16.h"

namespace msrl {
MSRL_BLOCK_BF16_LAUNCHER(256)
}  // namespace msrl
