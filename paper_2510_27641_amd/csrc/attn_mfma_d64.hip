// Matrix-core attention: the variants for index lists, d = 64.
#include "attn_mfma_kernel.h"

namespace specattn {

const void *attn_mfma_list_64(int nqt, int layout, bool f16) { return variant<64, LIST>(nqt, layout, f16); }

}  // namespace specattn
