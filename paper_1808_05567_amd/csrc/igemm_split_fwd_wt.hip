// The split kernel on the forward pass's weights, for backward passes without a launch that transforms them.
#include "igemm_split.h"

namespace convmi {

#define SPLIT_FW true
static const SplitEntry g_split_fwd_wt[] = {SPLIT_TABLE};
const SplitEntry *igemm_split_fwd_wt_entries(int *count)
{
    *count = (int)(sizeof(g_split_fwd_wt) / sizeof(g_split_fwd_wt[0]));
    return g_split_fwd_wt;
}

}  // namespace convmi
