// kb_mat.hip -- host side of the matrix-core workgroup kernel (kb_mat.h) and
// its instantiations for undirected graphs without edge labels.
#include <algorithm>

#include "kb_mat.h"

namespace gedk {
namespace mat {

const void *mat_kernel_plain(const MatConfig &m, bool fast) {
    return fast ? mat_select<false, false, true>(m) : mat_select<false, false, false>(m);
}

}  // namespace mat

using namespace mat;

namespace {

MatConfig mat_config(const BlockShape &s) {
    MatConfig m;
    const int W = std::max(4, s.W), K = s.K;
    if (s.PL > 2 || W > 16 || K < 1) return m;
    const bool wide = s.BT > kBlockThreads;
    if (K <= 16) m = MatConfig{W, 1, 1, 4};
    else if (K <= 32) m = MatConfig{W, 1, 2, 2};
    else if (K <= 64) m = wide ? MatConfig{W, 1, 4, 2} : MatConfig{W, 1, 4, 1};
    else if (K <= 128) m = MatConfig{W, 1, 8, 1};
    else if (K <= 256) m = MatConfig{W, 2, 8, 1};
    else if (K <= 512 && W <= 8) m = MatConfig{W, 4, 8, 1};
    else if (K <= 1024 && W == 4) m = MatConfig{W, 4, 16, 1};
    return m;
}

int slots_of(const MatConfig &m) { return 16 * m.NT * m.SW; }

MatLds lds_for(const BlockShape &s, const MatConfig &m) {
    MatLds L{};
    const int W = m.W, KS = slots_of(m), NA = s.PL > 0 ? 3 : 1, WU = s.directed ? W / 2 : W;
    const int KP = KS % 64 == 0 ? KS + 16 : (KS == 32 ? 48 : KS);
    const int n1 = std::max(s.nmax1, 1);
    int off = 0;
    auto take = [&](int bytes) {
        const int o = off;
        off += (bytes + 15) & ~15;
        return o;
    };
    const int URS = 32 * WU + 16;
    L.rows = take(NA * W * URS * 4);
    L.lc = take(URS * 4);
    L.img = take(W * KP * 4);
    L.phi = take(NA * W * KP * 4);
    L.le = take((WU + 1) * KP * 4);
    L.lt = take((WU + 1) * KP * 4);
    L.anc = take((n1 + BL - 1) / BL * KS * 2);
    L.cur = take(BL * KS * 2);
    L.com = take(n1 * 2);
    L.nbr = take(n1 * (s.directed ? 2 : 1) * 2);
    L.nbc = take(n1 * (s.directed ? 2 : 1));
    L.pc = take(NA * W * 4);
    L.ped = take(KS * 4);
    L.nsub = take(KS * 4);
    L.sel = take(KS * 4);
    L.bytes = off;
    return L;
}

constexpr int kMatLdsBytes = 158 * 1024;

const void *mat_kernel(const BlockShape &s, const MatConfig &m, bool fast) {
    if (s.PL > 0) return s.directed ? mat_kernel_dir_lab(m, fast) : mat_kernel_lab(m, fast);
    return s.directed ? mat_kernel_dir(m, fast) : mat_kernel_plain(m, fast);
}

// fp4 code of the integer m (0.5 m in E2M1), or -1.
int fp4_code(int64_t m) {
    const int sign = m < 0 ? 8 : 0;
    switch (m < 0 ? -m : m) {
        case 0: return 0;
        case 1: return sign | 1;
        case 2: return sign | 2;
        case 3: return sign | 3;
        case 4: return sign | 4;
        case 6: return sign | 5;
        case 8: return sign | 6;
        case 12: return sign | 7;
        default: return -1;
    }
}

}  // namespace

bool mat_supported(const BlockShape &s) {
    const MatConfig m = mat_config(s);
    return m.W != 0 && lds_for(s, m).bytes <= kMatLdsBytes && mat_kernel(s, m, true) != nullptr;
}

size_t mat_workspace_bytes(const BlockShape &s) {
    const MatConfig m = mat_config(s);
    return ((size_t)std::max(s.nmax1, 1) * (size_t)slots_of(m) * 2 + 255) / 256 * 256;
}

hipError_t mat_max_resident(const BlockShape &s, int *blocks_per_cu) {
    const MatConfig m = mat_config(s);
    const int threads = 64 * m.SW * m.UW, lds = lds_for(s, m).bytes;
    int f = 0, g = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&f, mat_kernel(s, m, true), threads, lds);
    if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&g, mat_kernel(s, m, false), threads, lds);
    *blocks_per_cu = std::min(f, g);
    return e;
}

hipError_t launch_mat(const BlockShape &s, const DbView &src, const DbView &dst, const WorkItem *work, int nwork,
                      int *queue, Costs c, int last_complete, void *workspace, size_t ws_stride, Outputs out,
                      int grid, hipStream_t stream) {
    const MatConfig m = mat_config(s);
    if (m.W == 0 || grid <= 0 || ws_stride != mat_workspace_bytes(s)) return hipErrorInvalidValue;
    MatArgs a{};
    a.src = src;
    a.dst = dst;
    a.work = work;
    a.nwork = nwork;
    a.queue = queue;
    a.c = c;
    a.K = s.K;
    a.last_complete = last_complete;
    a.ws = static_cast<char *>(workspace);
    a.ws_stride = ws_stride;
    a.L = lds_for(s, m);
    a.out = out;
    // the largest PED of any pair of these orders, and whether the costs fit
    // the matrix operands
    const int64_t vmax = std::max({c.vsub, c.vdel, c.vins}), emax = std::max({c.esub, c.edel, c.eins});
    const int64_t e1 = (int64_t)s.nmax1 * (s.nmax1 - 1), e2 = (int64_t)s.nmax2 * (s.nmax2 - 1);
    const int64_t bound = vmax * ((int64_t)s.nmax1 + s.nmax2) + emax * (s.directed ? e1 + e2 : (e1 + e2) / 2);
    a.pedbound = (uint32_t)std::min<int64_t>(bound, 0x7fffffff);
    const bool lab = s.PL > 0;
    const int64_t ci = c.eins, cp = lab ? (int64_t)c.esub - c.edel : -(int64_t)c.edel, cs = lab ? -(int64_t)c.esub : 0;
    int64_t g = 0;
    for (int64_t x : {ci, cp, cs}) {
        x = x < 0 ? -x : x;
        while (x) {
            const int64_t r = g % x;
            g = x;
            x = r;
        }
    }
    if (g == 0) g = 1;
    a.code_img = fp4_code(ci / g);
    a.code_phi = fp4_code(cp / g);
    a.code_same = fp4_code(cs / g);
    a.unit = (float)g;
    const bool fast = bound < kFastBound && a.code_img >= 0 && a.code_phi >= 0 && a.code_same >= 0;
    const void *k = mat_kernel(s, m, fast);
    if (!k) return hipErrorInvalidValue;
    void *args[] = {&a};
    return hipLaunchKernel(k, dim3(grid), dim3(64 * m.SW * m.UW), args, (size_t)a.L.bytes, stream);
}

}  // namespace gedk
