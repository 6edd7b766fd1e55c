// Matrix-core attention: the variants for kept-mask source, d = 128.
#include "attn_mfma_kernel.h"

namespace specattn {

const void *attn_mfma_mask_128(int nqt, int layout, bool f16) { return variant<128, MASK>(nqt, layout, f16); }

}  // namespace specattn
