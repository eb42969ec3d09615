// kb_mat_dir.hip -- the matrix-core workgroup kernel (kb_mat.h) for directed graphs without arc labels.
#include "kb_mat.h"

namespace gedk {
namespace mat {

const void *mat_kernel_dir(const MatConfig &m, bool fast) {
    return fast ? mat_select<false, true, true>(m) : mat_select<false, true, false>(m);
}

}  // namespace mat
}  // namespace gedk
