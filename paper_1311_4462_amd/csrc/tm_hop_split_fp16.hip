// FP16 instantiations of the direction-split hop kernel.
#include "tm_hop_split.inc.h"

namespace twm {
TM_SPLIT_DEFINE(TM_FP16)
}
