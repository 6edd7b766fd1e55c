// Matrix-core attention: the variants for any number of rows, lists of every kind.
#include "attn_mfma_kernel.h"

namespace specattn {

const void *attn_mfma_many(int d, int nqt, int layout, bool f16)
{
    return d == 64 ? variant<64, LIST, MANY>(nqt, layout, f16) : variant<128, LIST, MANY>(nqt, layout, f16);
}

}  // namespace specattn
