// Matrix-core attention: the variants for up to 64 rows with chunk lists or without lists.
#include "attn_mfma_kernel.h"

namespace specattn {

const void *attn_mfma_few_any(int d, int nqt, int layout, bool f16)
{
    return d == 64 ? variant<64, LIST, FEW_ANY>(nqt, layout, f16) : variant<128, LIST, FEW_ANY>(nqt, layout, f16);
}

}  // namespace specattn
