// kb_mat.hip -- host side of the matrix-core workgroup kernel (kb_mat.h) and
// its instantiations for undirected graphs without edge labels.
#include <algorithm>

#include "kb_mat.h"

namespace gedk {
namespace mat {

const void *mat_kernel_plain(const MatConfig &m, bool fast) {
    return fast ? mat_select<false, false, true>(m) : mat_select<false, false, false>(m);
}

bool slot_codes(const Costs &c, bool labels, SlotCodes *out) {
    // nibbles of weight m (0 .. 3) for spread_slot: 2 m, m, m / 2 and 2 m in fp4
    static const uint32_t mag[4] = {0x0000u, CODE_ONE, 0x6246u, 0x7357u};
    const int64_t w[3] = {c.eins, labels ? (int64_t)c.esub - c.edel : -(int64_t)c.edel, labels ? -(int64_t)c.esub : 0};
    int e = 0;   // unit 2^e: the largest that divides the three
    while (e < 21 && (((w[0] | w[1] | w[2]) >> e) & 1) == 0) ++e;
    uint32_t code[3];
    for (int k = 0; k < 3; ++k) {
        const int64_t unit = (int64_t)1 << e, m = w[k] / unit;
        if (w[k] % unit != 0 || m < -3 || m > 3) return false;
        code[k] = mag[m < 0 ? -m : m] | (m < 0 ? 0x8888u : 0u);
    }
    out->img = code[0];
    out->phi = code[1];
    out->same = code[2];
    out->unit_exp = SC_ONE + e;
    return true;
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

int lds_bytes(const BlockShape &s, const MatConfig &m) {
    const int KS = slots_of(m), blocks = (std::max(s.nmax1, 1) + BL - 1) / BL;
    return mat_lds(m.W, KS, s.PL > 0 ? 3 : 1, s.directed ? 2 : 1).anc + blocks * KS * (KS > 256 ? 2 : 1);
}

constexpr int kMatLdsBytes = 158 * 1024;

const void *mat_kernel(const BlockShape &s, const MatConfig &m, bool fast) {
    if (s.PL > 0) return s.directed ? mat_kernel_dir_lab(m, fast) : mat_kernel_lab(m, fast);
    return s.directed ? mat_kernel_dir(m, fast) : mat_kernel_plain(m, fast);
}

}  // namespace

bool mat_supported(const BlockShape &s) {
    const MatConfig m = mat_config(s);
    return m.W != 0 && lds_bytes(s, m) <= kMatLdsBytes && mat_kernel(s, m, true) != nullptr;
}

size_t mat_workspace_bytes(const BlockShape &s) {
    const MatConfig m = mat_config(s);
    return ((size_t)std::max(s.nmax1, 1) * (size_t)slots_of(m) * 2 + 255) / 256 * 256;
}

hipError_t mat_max_resident(const BlockShape &s, int *blocks_per_cu) {
    const MatConfig m = mat_config(s);
    // (the grid is sized for the matrix form of the costs; the other needs
    // more registers, and a grid beyond what is resident at once only queues)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, mat_kernel(s, m, true), 64 * m.SW * m.UW,
                                                        lds_bytes(s, m));
}

namespace {

// The largest PED of any pair of the shape's orders.
int64_t ped_bound(const BlockShape &s, const Costs &c) {
    const int64_t vmax = std::max({c.vsub, c.vdel, c.vins}), emax = std::max({c.esub, c.edel, c.eins});
    const int64_t e1 = (int64_t)s.nmax1 * (s.nmax1 - 1), e2 = (int64_t)s.nmax2 * (s.nmax2 - 1);
    return vmax * ((int64_t)s.nmax1 + s.nmax2) + emax * (s.directed ? e1 + e2 : (e1 + e2) / 2);
}

}  // namespace

bool mat_fast(const BlockShape &s, const Costs &c) {
    SlotCodes codes;
    return ped_bound(s, c) < kFastBound && slot_codes(c, s.PL > 0, &codes);
}

const void *mat_kernel_for(const BlockShape &s, const Costs &c) { return mat_kernel(s, mat_config(s), mat_fast(s, c)); }

hipError_t launch_mat(const BlockShape &s, const DbView &src, const DbView &dst, const WorkItem *work, int nwork,
                      int *queue, Costs c, int last_complete, void *workspace, size_t ws_stride, Outputs out,
                      int grid, hipStream_t stream) {
    const MatConfig m = mat_config(s);
    if (m.W == 0 || grid <= 0 || ws_stride < mat_workspace_bytes(s)) return hipErrorInvalidValue;
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
    a.ws_stride = mat_workspace_bytes(s);   // (what the caller has a workgroup may be more)
    a.out = out;
    a.pedbound = (uint32_t)std::min<int64_t>(ped_bound(s, c), 0x7fffffff);
    SlotCodes codes;
    slot_codes(c, s.PL > 0, &codes);   // (used where mat_fast holds)
    a.code_img = codes.img;
    a.code_phi = codes.phi;
    a.code_same = codes.same;
    a.unit_exp = codes.unit_exp;
    const void *k = mat_kernel_for(s, c);
    if (!k) return hipErrorInvalidValue;
    void *args[] = {&a};
    return hipLaunchKernel(k, dim3(grid), dim3(64 * m.SW * m.UW), args, (size_t)lds_bytes(s, m), stream);
}

}  // namespace gedk
