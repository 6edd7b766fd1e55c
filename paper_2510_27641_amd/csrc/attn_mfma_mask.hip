// Matrix-core attention: the variants for kept-mask source, d = 128.
#include "attn_mfma_kernel.h"

namespace specattn {

const void *attn_mfma_mask(int form, int nqt, int layout, bool f16)
{
    return form == MANY ? variant<128, MASK, MANY>(nqt, layout, f16) : variant<128, MASK, FEW_POSITIONS>(nqt, layout, f16);
}

}  // namespace specattn
