// kb_mat_lab.hip -- the matrix-core workgroup kernel (kb_mat.h) for undirected graphs with edge labels.
#include "kb_mat.h"

namespace gedk {
namespace mat {

const void *mat_kernel_lab(const MatConfig &m, bool fast) {
    return fast ? mat_select<true, false, true>(m) : mat_select<true, false, false>(m);
}

}  // namespace mat
}  // namespace gedk
