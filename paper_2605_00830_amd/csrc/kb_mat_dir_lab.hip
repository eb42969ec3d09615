// kb_mat_dir_lab.hip -- the matrix-core workgroup kernel (kb_mat.h) for directed graphs with arc labels.
#include "kb_mat.h"

namespace gedk {
namespace mat {

const void *mat_kernel_dir_lab(const MatConfig &m, bool fast) {
    return fast ? mat_select<true, true, true>(m) : mat_select<true, true, false>(m);
}

}  // namespace mat
}  // namespace gedk
