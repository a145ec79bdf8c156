// More compiled on-chip kernels: more than ten channels at the depths that are affordable there (11-20 at depth 2, 11
// and 12 at depth 3), a lane per word of length depth - 1 with its d children.  They serve final mode only (see wide_on_chip_wanted
// in sig_api.hip); stream mode of these shapes stays with the level-scan family.
#include "sig_onchip.h"

namespace sig {

namespace {
const OnChipKernelInfo kTable[] = {
    SIG_ON_CHIP_FINAL_ENTRY(11, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(12, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(13, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(14, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(15, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(16, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(17, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(18, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(19, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(20, 2, 1),
    SIG_ON_CHIP_FINAL_ENTRY(11, 3, 2),
    SIG_ON_CHIP_FINAL_ENTRY(12, 3, 2),
    {0, 0, 0, 0, 0, 0, nullptr, nullptr, nullptr},
};
}  // namespace

const OnChipKernelInfo *on_chip_table_wide() { return kTable; }

}  // namespace sig
