// kb_mat.h -- workgroup-per-pair K-Best search with the children scored on
// the matrix cores: targets of up to 512 vertices (directed: 256), up to four
// edge-label codes, K as far as mat_config() has an instantiation.
//
// A level's children are two contractions over g2's vertices v,
//   kept[s][u]  = sum_v Phi_s[v] A2[u][v]     |Phi & N2(u)|
//   inimg[s][u] = sum_v Img_s[v] A2[u][v]     |Img & N2(u)|
// (and, with edge labels, one per label code c: Phi_c against the rows of
// code c), which the PED of child (s, u) takes linearly:
//   PED_s + lc(u) + edel (deg - kept) + eins (inimg - kept) + esub (kept - same).
// The 0/1 operands are fp4 (E2M1) matrices of the 16x16x128 MFMA: 32 bits of a
// set become four registers of nibbles by (w >> j) & 0x11111111 (value 0.5,
// lifted to 1 by the block scale), the same permutation of v on both sides.
// FAST: eins, -edel (+ esub) and -esub are each 0 to 3 times one power of two
// (fp4 holds 0, 1, 2, 3, 4, 6, 8, 12 times 0.5, and the spread bits stand for
// 0.5 to 2; the power of two is the block scale), so they ride in the slot
// operand and one chain gives the whole child but for its base; otherwise the
// counts come out separately and the PED is formed in int32: two chains and
// more registers, 1.5 to 4 times as long (200 pairs of 130..250 vertices at
// K = 64: 1,656 us FAST, 3,757 with edge costs of 15; 7,500 with the candidate
// matrix).  All sums are whole numbers below 2^24: the f32 accumulators are
// exact.  Used vertices are
// struck out by one more MFMA, a unit matrix times Img at scale 2^24.
//
// A wave holds NT tiles of 16 slots (their operands in registers) and walks
// the tiles of 16 target vertices; each child is kept as one byte
// x = clamp((PED - b) >> sh, 0, 127) in registers, four per word, so no
// candidate matrix exists.  b is the least parent PED plus the previous
// level's T - m0, less 63, and sh = 0: T - m0 moves by about 4 to 12 from level
// to level on the random graphs measured (at most 46 on 200- to 500-vertex
// pairs), so the K-th child almost always falls inside the bytes' exact range;
// if not, coarse passes from the least parent PED (a bound of every child)
// narrow it 6 bits at a time until it is exact.
//
// The threshold is searched on the bytes (SWAR compare and popcount, two
// thresholds per round, steered by the least child plus the last level's
// T - least child).  Survivors are marked in per-slot bit masks over u in LDS
// and emitted slot by slot in ascending u with the tie quota counted from the
// first slot: generation order, as in every other kernel.  Their PEDs are
// recomputed in int32 from the sets, so the bytes only select.
//
// The mapping is not copied level by level.  Images of the last (incomplete)
// block of 8 levels are per-slot rows in LDS; a complete block's rows go to
// the workspace once, indexed by the slots of its last level, and each slot
// carries one ancestor index per block (gathered from its parent's).  A block
// whose ancestors have all become one slot is the same for the whole beam: it
// leaves the window for the common mapping, whose part of Phi is built once
// per level instead of once per slot.  (Measured window: 35 to 85 levels on
// 200- to 450-vertex pairs at K = 256, against half of n1 for a full copy.)
//
// Images that became common are used in every slot, so their vertices need no
// scoring: target vertices stand in the rows, labels and used bits by position,
// and every CB = 4 blocks the common ones move behind the others (in place,
// order kept, so generation order is still ascending position).  The tiles past
// the nact positions left are skipped.  Fewer blocks at a time would seldom free
// a group of tiles (32 or 64 vertices).  (Mean nact at 500 vertices and K = 256:
// 369; at 250 and K = 64: 177.  With the clamp as one med3 instead of min and
// the max that quiets NaN: 256 pairs of 100..500 vertices, K = 256 14,181 ->
// 12,555 us; 512 of 65..250, K = 64 2,165 -> 2,060; 3000 of 10..70, which have
// no level for it, 746 -> 740.)
//
// Measured against the candidate-matrix kernel of kb_block.hip (same box, us
// a launch): 256 pairs of 100..500 vertices at K = 256 80,050 -> 12,350; 512
// pairs of 65..250 at K = 64 9,220 -> 1,810; and before the positions closed up
// 400 pairs of 65..128 at K = 1024 20,034 -> 6,379; 100 labelled pairs of
// 300..500 at K = 64 131,104 -> 12,191; 200 labelled directed pairs of 130..250
// at K = 80 41,755 -> 5,939.  A launch lasts as long as its largest pair.  A
// level of 500 vertices (p = 0.1) at K = 256 is 48.6 thousand cycles, 405
// positions left: 23.8 in the scoring (7.4 of it waiting for the SIMD's other
// wave), 4.9 in 1.13 threshold rounds, 4.4 marking survivors, 3.1 emitting, 6.8
// in the update, 5.0 on the neighbours and Phi, 0.6 closing up.  The matrix
// instructions (16 cycles each) and the vector ones hardly overlap on this part:
// a stream of both takes 0.93 of the two alone added up.  Over a launch the
// matrix pipes of the CUs at work are busy 15 % of the time, the vector pipes 54 %.
#pragma once

#include "ged_internal.h"
#include "wave_common.h"

namespace gedk {
namespace mat {

using namespace wv;

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));

constexpr uint32_t NIB = 0x11111111u;
constexpr uint32_t HI = 0x80808080u;
constexpr uint32_t DEAD = 0x7f7f7f7fu;      // four children that never survive
constexpr uint32_t DEL16 = 0xffffu;
constexpr int XCAP = 127;                   // byte of a child above the range
constexpr int DELU = 1023;                  // survivor record's vertex of the deletion child
constexpr int BL = 8;                       // levels per mapping block
constexpr int CB = 4;                       // mapping blocks whose images leave the positions together
constexpr int SC_ONE = 127;                 // E8M0 scales 1, 2^24
constexpr int SC_BIG = 127 + 24;
constexpr uint32_t CODE_ONE = 0x4124u;      // slot operand's nibbles of weight 1 (spread_slot)
constexpr float FBIG = 16777216.f;
constexpr int64_t kFastBound = (int64_t)1 << 22;   // PEDs below this stay exact in f32 with 1 / 2^sh parts

// Slot stride of the LDS arrays: the four k-groups of an operand on different banks.
constexpr int slot_pad(int KS) { return KS % 64 == 0 ? KS + 16 : (KS == 32 ? 48 : KS); }

// Byte offsets in dynamic LDS, constants of an instantiation (a row of W words,
// KS slots, NA sets, ND rows of a vertex); the ancestor rows, whose number goes
// with the largest source, come last.
struct MatLds {
    int rows, lc, l1, l2, r1, act, img, use, phi, le, lt, cur, com, nbr, nbc, pc, ped, nsub, sel, anc;
};
constexpr MatLds mat_lds(int W, int KS, int NA, int ND) {
    MatLds L{};
    const int WU = W / ND, URS = 32 * WU + 16, KP = slot_pad(KS), N1 = GED_MAX_VERTICES_BATCH;
    int off = 0;
    auto take = [&off](int bytes) {
        const int o = off;
        off += (bytes + 15) & ~15;
        return o;
    };
    L.rows = take(NA * W * URS * 4);
    L.lc = take(URS * 4);
    L.l1 = take(N1 * 4);
    L.l2 = take(URS * 4);
    L.r1 = take(2 * ND * NA * (N1 / 32) * 4);
    L.act = take(URS * 2);
    L.img = take(W * KP * 4);
    L.use = take(WU * KP * 4);
    L.phi = take(NA * W * KP * 4);
    L.le = take((WU + 1) * KP * 4);
    L.lt = take((WU + 1) * KP * 4);
    L.cur = take(BL * KS * 2);
    L.com = take(N1 * 2);
    L.nbr = take(N1 * ND * 2);
    L.nbc = NA > 1 ? take(N1 * ND) : off;
    L.pc = take(NA * W * 4);
    L.ped = take(KS * 4);
    L.nsub = take(KS * 4);
    L.sel = take(KS * 4);
    L.anc = off;
    return L;
}

struct MatArgs {
    DbView src, dst;
    const WorkItem *work;
    int nwork;
    int *queue;
    Costs c;
    int K;
    int last_complete;
    char *ws;
    size_t ws_stride;
    Outputs out;
    uint32_t pedbound;   // no PED of the launch exceeds it
    // FAST: the slot operand's nibbles (spread_slot) for Img \ Phi, Phi, Phi_c,
    // and the power of two (E8M0) of their unit
    uint32_t code_img, code_phi, code_same;
    int unit_exp;
};

// One chain step; the operands' scales are E8M0 bytes.
__device__ __forceinline__ v4f mfma_fp4(const uint32_t (&a)[4], const uint32_t (&b)[4], v4f c, int sa, int sb) {
    v8i x = {}, y = {};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        x[j] = (int)a[j];
        y[j] = (int)b[j];
    }
    return __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(x, y, c, 4, 4, 0, sa, 0, sb);
}

// The 32 bits of w as fp4 numbers, bit i in register i % 4.  The row side
// leaves the bits where they are, so that a word takes five instructions
// instead of seven: they stand for 0.5, 1, 2 and (shifted down) 0.5 ...
__device__ __forceinline__ void spread_row(uint32_t w, uint32_t (&e)[4]) {
    e[0] = w & NIB;
    e[1] = w & (NIB << 1);
    e[2] = w & (NIB << 2);
    e[3] = (w >> 3) & NIB;
}
// ... and the slot side makes up for it: a weight m is 2 m, m, m / 2 and 2 m
// (fp4 has them for m = 0 .. 3), nibble j of `code` for register j.
__device__ __forceinline__ void spread_slot(uint32_t w, uint32_t code, uint32_t (&e)[4]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) e[j] = ((w >> j) & NIB) * ((code >> (4 * j)) & 15u);
}
// (weight 1)
__device__ __forceinline__ void spread_one(uint32_t w, uint32_t (&e)[4]) {
    e[0] = (w << 2) & (NIB << 2);
    e[1] = w & (NIB << 1);
    e[2] = (w >> 2) & NIB;
    e[3] = (w >> 1) & (NIB << 2);
}

__device__ __forceinline__ uint32_t below(int i, int kw) {
    const int rem = i - kw * 32;
    return rem >= 32 ? 0xffffffffu : (rem <= 0 ? 0u : ((1u << rem) - 1u));
}

__device__ __forceinline__ unsigned long long wave_min64(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long w = (unsigned long long)__shfl_xor((long long)v, o);
        v = w < v ? w : v;
    }
    return v;
}

// Sum over the N neighbouring lanes of a slot, in each of them (N a power of two,
// at most a row of 16): DPP within a quad, then the mirrors, whose lanes hold
// the other half's sum.  (Lane shuffles go through LDS, one round trip a step.)
template <int N>
__device__ __forceinline__ uint32_t parts_sum(uint32_t v) {
    static_assert(N == 1 || N == 2 || N == 4 || N == 8 || N == 16, "lanes of a slot");
    if (N > 1) v += dpp_ror<0xb1>(v);    // quad_perm 1 0 3 2
    if (N > 2) v += dpp_ror<0x4e>(v);    // quad_perm 2 3 0 1
    if (N > 4) v += dpp_ror<0x141>(v);   // row_half_mirror
    if (N > 8) v += dpp_ror<0x140>(v);   // row_mirror
    return v;
}

// A slot index, in a byte while that holds it.
template <bool WIDE> struct AncOf { using type = uint8_t; };
template <> struct AncOf<true> { using type = uint16_t; };

// W: words of a row (directed: out-half, then in-half); a wave holds NT tiles
// of 16 slots; SW waves split the slots, UW the target tiles.
// MINW: waves per SIMD the registers are held to, four where that costs no
// spills (two registers with directed label planes), so that two 512-thread
// workgroups fit a CU.
template <int W, int NT, int SW, int UW, bool LAB, bool DIR, bool FAST,
          int MINW = (FAST && NT == 1 && (W == 4 || (W == 8 && !LAB))) ? 4 : 2>
__global__ __launch_bounds__(64 * SW * UW, MINW) void kb_mat_kernel(MatArgs a) {
    constexpr int KS = 16 * NT * SW;            // slots
    constexpr int T = 64 * SW * UW;
    constexpr int NWV = SW * UW;
    constexpr int PARTS = T / KS;               // threads per slot in the update
    constexpr int KST = W / 4;                  // 128-vertex steps of a contraction
    constexpr int WU = DIR ? W / 2 : W;         // words that name target vertices
    constexpr int NTL = 2 * WU / UW;            // target tiles of a wave
    constexpr int KP = slot_pad(KS);
    constexpr int NA = LAB ? 3 : 1;             // sets: Phi / rows, and two label planes
    constexpr int ND = DIR ? 2 : 1;             // rows of a vertex (out, in)
    constexpr int W1 = GED_MAX_VERTICES_BATCH / 32;   // words of a source row
    constexpr int CW = (WU + PARTS) / PARTS;    // mask words of an emitting thread
    constexpr int NS = LAB ? 5 : (FAST ? 1 : 2);   // slot operands (FAST: combined first; else Phi, Img first)
    constexpr int NOP = LAB ? (FAST ? 5 : 6) : NS; // ... with four label codes after them
    constexpr int NCAND = NTL + 1;              // words of a slot tile: target tiles, then the deletion
    constexpr int NWP = (W + PARTS - 1) / PARTS;
    // ancestor rows a thread moves per step: 16 a slot cover most windows (mean 3.5
    // blocks at K = 64, 9 at 256), and each further one is code that finds no row
    // (16 a thread instead: 512 pairs of 65..250, K = 64, 2,026 against 1,862 us)
    constexpr int MAXA = PARTS >= 4 ? 4 : 16 / PARTS;
    static_assert(W % 4 == 0 && KS <= T && 8 % UW == 0 && (2 * WU) % UW == 0, "shape");
    // what the packed words below rest on
    static_assert(16 * NT * (32 * WU / UW + 1) < 65536, "a wave's children: 16 bits of a threshold count");
    static_assert(GED_MAX_K < 2048 && T * GED_MAX_K <= 1 << 21, "children below T in 11 bits, ties in the 21 above");
    static_assert(32 * W < 1024, "counts over a row: 10 bits each");
    static_assert(32 * WU < DELU && GED_MAX_K <= 1 << 21, "survivor record: slot above 10 bits of vertex");
    static_assert(KS <= (KS > 256 ? 65536 : 256), "ancestor index");

    constexpr MatLds L = mat_lds(W, KS, NA, ND);
    extern __shared__ uint32_t s_dyn[];
    __shared__ uint32_t s_red[2][NWV];
    __shared__ unsigned long long s_red64[NWV];
    __shared__ int s_item, s_neq, s_nw[2];
    __shared__ uint32_t s_gone[WU], s_rm[WU];   // vertices, positions that leave
    __shared__ int s_sumV[2];
    __shared__ uint32_t s_min[2];
    char *lds = reinterpret_cast<char *>(s_dyn);
    uint32_t *s_rows = reinterpret_cast<uint32_t *>(lds + L.rows);   // [NA][W][urs], by position
    float *s_lc = reinterpret_cast<float *>(lds + L.lc);             // label cost of u (FAST: float, else int bits)
    int *s_lci = reinterpret_cast<int *>(lds + L.lc);
    int *s_l1 = reinterpret_cast<int *>(lds + L.l1);                 // vertex labels of g1, g2
    int *s_l2 = reinterpret_cast<int *>(lds + L.l2);
    uint32_t *s_r1 = reinterpret_cast<uint32_t *>(lds + L.r1);       // [2][ND * NA][W1] row of v_i, by level parity
    uint16_t *s_act = reinterpret_cast<uint16_t *>(lds + L.act);     // target vertex of a position (nact of them, ascending)
    uint32_t *s_img = reinterpret_cast<uint32_t *>(lds + L.img);     // [W][KP]
    uint32_t *s_use = reinterpret_cast<uint32_t *>(lds + L.use);     // [WU][KP] Img by position (past nact: used)
    uint32_t *s_phi = reinterpret_cast<uint32_t *>(lds + L.phi);     // [NA][W][KP] the window's part of Phi
    uint32_t *s_le = reinterpret_cast<uint32_t *>(lds + L.le);       // [WU + 1][KP] children at most T (last: deletion)
    uint32_t *s_lt = reinterpret_cast<uint32_t *>(lds + L.lt);       // ... below T
    using Anc = typename AncOf<(KS > 256)>::type;
    Anc *s_anc = reinterpret_cast<Anc *>(lds + L.anc);               // [blocks][KS]
    uint16_t *s_cur = reinterpret_cast<uint16_t *>(lds + L.cur);     // [BL][KS]
    uint16_t *s_com = reinterpret_cast<uint16_t *>(lds + L.com);     // common mapping
    uint16_t *s_nbr = reinterpret_cast<uint16_t *>(lds + L.nbr);     // window neighbours of v_i (bit 15: in-arc)
    uint8_t *s_nbc = reinterpret_cast<uint8_t *>(lds + L.nbc);       // their label codes
    uint32_t *s_pc = reinterpret_cast<uint32_t *>(lds + L.pc);       // [NA][W] the common part of Phi
    int *s_ped = reinterpret_cast<int *>(lds + L.ped);
    int *s_nsub = reinterpret_cast<int *>(lds + L.nsub);
    int *s_sel = reinterpret_cast<int *>(lds + L.sel);               // survivor: parent << 10 | vertex
    constexpr int URS = 32 * WU + 16;           // stride of a row word over u: the four k-groups on different banks

    const int t0 = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(t0 >> 6);
    const int sw = wid % SW, uw = UW == 1 ? 0 : wid / SW;
    uint16_t *phi_g = reinterpret_cast<uint16_t *>(a.ws + (size_t)blockIdx.x * a.ws_stride);   // [n1][KS]
    const int K = a.K;
    const Costs c = a.c;

    for (bool first = true;; first = false) {
        const int t = t0;
        int item = (int)blockIdx.x;
        if (!first) {
            if (t == 0) s_item = pull_item(a.queue, a.nwork);
            __syncthreads();
            item = __builtin_amdgcn_readfirstlane(s_item);
            __syncthreads();
        }
        if (item >= a.nwork) break;
        const WorkItem wi = a.work[item];
        const GraphRec g1 = a.src.graphs[wi.src];
        const GraphRec g2 = a.dst.graphs[wi.dst];
        const int n1 = g1.n, n2 = g2.n, w1 = g1.w, w2 = g2.w;
        const uint32_t *A1 = a.src.adj + g1.adj;
        const uint32_t *A2 = a.dst.adj + g2.adj;
        const int *L1 = a.src.vlab + g1.vlab;
        const int *L2 = a.dst.vlab + g2.vlab;
        const int P = a.dst.planes;
        const size_t pl1 = (size_t)n1 * w1, pl2 = (size_t)n2 * w2;
        const uint32_t *A1in = A1 + (size_t)(1 + a.src.planes) * pl1;
        const uint32_t *A2in = A2 + (size_t)(1 + P) * pl2;

        for (int x = t; x < NA * W * URS; x += T) {
            const int b = x / (W * URS), r = x % (W * URS), kk = r / URS, u = r % URS;
            const bool in = DIR && kk >= WU;
            const int kr = in ? kk - WU : kk;
            s_rows[x] = (u < n2 && kr < w2 && b <= P) ? (in ? A2in : A2)[(size_t)b * pl2 + (size_t)u * w2 + kr] : 0u;
        }
        for (int x = t; x < URS; x += T) s_l2[x] = x < n2 ? L2[x] : 0;
        for (int x = t; x < n1; x += T) s_l1[x] = L1[x];
        // word k of set b (row, label planes) of g1 vertex v's out- or in-row
        auto source_word = [&](int v, int x) -> uint32_t {
            const int k = x % W1, b = x / W1 % NA, d = x / (W1 * NA);
            return (v < n1 && k < w1 && b <= P) ? (d ? A1in : A1)[(size_t)b * pl1 + (size_t)v * w1 + k] : 0u;
        };
        for (int x = t; x < ND * NA * W1; x += T) s_r1[x] = source_word(0, x);
        for (int x = t; x < W * KP; x += T) {
            const int kk = x / KP;
            s_img[x] = 0u;
            if (kk < WU) s_use[x] = ~below(n2, kk);
        }
        for (int x = t; x < URS; x += T) s_act[x] = (uint16_t)x;
        for (int x = t; x < NA * W * KP; x += T) s_phi[x] = 0u;
        for (int x = t; x < (WU + 1) * KP; x += T) {
            s_le[x] = 0u;
            s_lt[x] = 0u;
        }
        for (int x = t; x < NA * W; x += T) s_pc[x] = 0u;
        for (int x = t; x < KS; x += T) {
            s_ped[x] = 0;
            s_nsub[x] = 0;
        }
        if (t == 0) {
            s_neq = 0;
            s_sumV[0] = s_sumV[1] = 0;
            s_min[0] = s_min[1] = 0xffffffffu;
        }
        int nb = 1, m0 = 0, V = n2 + 1, nact = n2;
        int b0 = 0, nblk = 0;       // window blocks [b0, nblk)
        int cb = 0;                 // blocks whose images have left the positions
        int dlt = 0, spr = 0;       // last level's T - m0, T - least child
        long long ce = 0;
        __syncthreads();

        // image of g1 vertex j under slot s, for j in the window or common
        auto image = [&](int j, int s) -> uint32_t {
            if (j >= BL * nblk) return s_cur[(j - BL * nblk) * KS + s];
            return phi_g[(size_t)j * KS + s_anc[(j / BL) * KS + s]];
        };
        // g2 edges (arcs) inside Img of slot us, split over its parts: twice the count
        auto inside = [&](int s, int part) -> int {
            uint32_t im[W];
#pragma unroll
            for (int k = 0; k < W; ++k) im[k] = s_img[k * KP + s];
            uint32_t e = 0;
            for (int at = part; at < n2; at += PARTS) {
                const int u = s_act[at];
                if (!((s_img[(u >> 5) * KP + s] >> (u & 31)) & 1u)) continue;
#pragma unroll
                for (int k = 0; k < W; ++k) e += (uint32_t)__popc(im[k] & s_rows[k * URS + at]);
            }
            return (int)parts_sum<PARTS>(e);
        };

        for (int i = 0; i < n1; ++i) {
            // the thread's index is opaque in each level: addresses are formed
            // where they are used instead of being kept for the whole pair
            int t = t0;
            asm volatile("" : "+v"(t));
            const int lane = t & 63, q = lane >> 4, col = lane & 15;
            const int us = t / PARTS, part = t % PARTS;   // slot and share of the update's threads
            const int c0 = BL * b0;
            const int lab1 = s_l1[i];
            const uint32_t *R1 = s_r1 + (i & 1) * (ND * NA * W1);
            // the next vertex's row, in flight during the level
            const uint32_t rown = t < ND * NA * W1 ? source_word(i + 1, t) : 0u;
            int degP = 0;
            if (lane < W1) {
                degP = __popc(R1[lane] & below(i, lane));
                if (DIR) degP += __popc(R1[NA * W1 + lane] & below(i, lane));
            }
            degP = (int)wave_sum((uint32_t)degP);
            const int del_cost = c.vdel + c.edel * degP;

            // ---------------- the common part of Phi, the window's neighbours, label costs
            for (int j = t; j < c0; j += T) {
                const uint32_t x = s_com[j];
#pragma unroll
                for (int d = 0; d < ND; ++d) {
                    const uint32_t *R = R1 + d * (NA * W1) + (j >> 5);
                    if (x == DEL16 || !((R[0] >> (j & 31)) & 1u)) continue;
                    const int xw = (int)(x >> 5) + (d ? WU : 0);
                    atomicOr(&s_pc[xw], 1u << (x & 31));
#pragma unroll
                    for (int b = 1; b < NA; ++b)
                        if ((R[b * W1] >> (j & 31)) & 1u) atomicOr(&s_pc[b * W + xw], 1u << (x & 31));
                }
            }
            if (wid == NWV - 1) {
                // images in the complete blocks first, then those of the current one
                int base = 0;
#pragma unroll 1
                for (int part2 = 0; part2 < 2; ++part2) {
                    const int jl = part2 ? BL * nblk : c0, jh = part2 ? i : BL * nblk;
#pragma unroll
                    for (int d = 0; d < ND; ++d) {
                        for (int kw = jl >> 5; kw * 32 < jh; ++kw) {
                            const uint32_t *R = R1 + d * (NA * W1) + kw;
                            const uint32_t bits = R[0] & below(jh, kw) & ~below(jl, kw);
                            const bool mine = lane < 32 && ((bits >> lane) & 1u);
                            const unsigned long long m = __ballot(mine);
                            if (mine) {
                                const int rank = (int)__builtin_amdgcn_mbcnt_lo((unsigned)m, 0u);
                                s_nbr[base + rank] = (uint16_t)((kw * 32 + lane) | (d << 15));
                                if (LAB) {
                                    int code = 0;
#pragma unroll
                                    for (int b = 1; b < NA; ++b) code |= (int)((R[b * W1] >> lane) & 1u) << (b - 1);
                                    s_nbc[base + rank] = (uint8_t)code;
                                }
                            }
                            base += __popcll(m);
                        }
                    }
                    if (lane == 0) s_nw[part2] = base;
                }
            }
            for (int u = t; u < URS; u += T) {
                const int lc = (u < nact && lab1 != s_l2[u]) ? c.vsub : 0;
                if (FAST) s_lc[u] = (float)lc;
                else s_lci[u] = lc;
            }
            if (b0 < nblk && us < nb && s_anc[b0 * KS + us] != s_anc[b0 * KS]) s_neq = 1;
            __syncthreads();

            // ---------------- the window's part of Phi, slot by slot
            {
                const int nwb = s_nw[0], nw = s_nw[1], slot = t % KS, p0 = t / KS;
                auto mark = [&](uint32_t x, int nj, int at) {
                    if (x == DEL16) return;   // deleted, or past the list
                    const int xw = (int)(x >> 5) + ((DIR && (nj >> 15)) ? WU : 0);
                    const uint32_t bit = 1u << (x & 31);
                    atomicOr(&s_phi[xw * KP + slot], bit);
                    if (LAB) {
                        const int code = s_nbc[at];
                        if (code & 1) atomicOr(&s_phi[(W + xw) * KP + slot], bit);
                        if (code & 2) atomicOr(&s_phi[(2 * W + xw) * KP + slot], bit);
                    }
                };
                // (LB rows of the complete blocks in flight together)
                constexpr int LB = PARTS >= 4 ? 4 : 8;
                if (slot < nb) {
                    for (int kb = p0; kb < nwb; kb += LB * PARTS) {
                        uint32_t x[LB];
                        int nj[LB];
#pragma unroll
                        for (int k = 0; k < LB; ++k) {
                            const int kk = kb + k * PARTS;
                            nj[k] = s_nbr[min(kk, nwb - 1)];
                            const int j = nj[k] & 0x7fff;
                            x[k] = phi_g[(size_t)j * KS + s_anc[(j / BL) * KS + slot]];
                            x[k] = kk < nwb ? x[k] : DEL16;
                        }
#pragma unroll
                        for (int k = 0; k < LB; ++k) mark(x[k], nj[k], kb + k * PARTS);
                    }
                    for (int kk = nwb + p0; kk < nw; kk += PARTS) {
                        const int nj = s_nbr[kk];
                        mark(s_cur[((nj & 0x7fff) - BL * nblk) * KS + slot], nj, kk);
                    }
                }
                // a block with one ancestor left joins the common mapping
                if (b0 < nblk && s_neq == 0) {
                    if (t < BL) s_com[BL * b0 + t] = phi_g[(size_t)(BL * b0 + t) * KS + s_anc[b0 * KS]];
                    ++b0;
                }
            }
            __syncthreads();

            ce += V;
            int nb_new;
            if (a.last_complete && i == n1 - 1) {
                // ---------------- complete-then-minimum last level: the least
                // total (Sec. 4.4.1), first in generation order
                unsigned long long bk = ~0ull;
                if (us < nb) {
                    const int e0 = inside(us, part) / 2, ns = s_nsub[us];
                    for (int at = part; at <= nact; at += PARTS) {
                        int d = s_ped[us], left = g2.m - e0, used = ns;
                        if (at < nact) {
                            if ((s_use[(at >> 5) * KP + us] >> (at & 31)) & 1u) continue;
                            int kept = 0, inimg = 0, relab = 0;
                            for (int k = 0; k < W; ++k) {
                                const uint32_t row = s_rows[k * URS + at];
                                const uint32_t ph = s_phi[k * KP + us] | s_pc[k];
                                kept += __popc(ph & row);
                                inimg += __popc(s_img[k * KP + us] & row);
                                if (LAB) {
                                    const uint32_t f0 = (s_phi[(W + k) * KP + us] | s_pc[W + k]) ^ s_rows[(W + k) * URS + at];
                                    const uint32_t f1 = (s_phi[(2 * W + k) * KP + us] | s_pc[2 * W + k]) ^ s_rows[(2 * W + k) * URS + at];
                                    relab += __popc(ph & row & (f0 | f1));
                                }
                            }
                            d += (lab1 != s_l2[at] ? c.vsub : 0) + c.edel * (degP - kept) + c.eins * (inimg - kept) +
                                 c.esub * relab;
                            left -= inimg;
                            ++used;
                        } else {
                            d += del_cost;
                        }
                        const int total = d + c.vins * (n2 - used) + c.eins * left;
                        const unsigned long long key = ((unsigned long long)(unsigned)total << 32) |
                                                       (unsigned)((us << 10) | at);
                        bk = key < bk ? key : bk;
                    }
                }
                bk = wave_min64(bk);
                if (lane == 0) s_red64[wid] = bk;
                __syncthreads();
                if (t == 0) {
                    unsigned long long m = s_red64[0];
#pragma unroll
                    for (int k = 1; k < NWV; ++k) m = s_red64[k] < m ? s_red64[k] : m;
                    const int low = (int)(m & 0xffffffffu);
                    s_sel[0] = (low & 1023) == nact ? (low | DELU) : low;
                }
                nb_new = 1;
            } else {
                int quota = 0;
                if (V <= K) {
                    // every child survives: the free vertices and the deletion
                    for (int x = t; x < (WU + 1) * KS; x += T) {
                        const int k = x / KS, s = x % KS;
                        if (s < nb) {
                            const uint32_t m = k < WU ? ~s_use[k * KP + s] : 1u;
                            s_le[k * KP + s] = m;
                            s_lt[k * KP + s] = m;
                        }
                    }
                    dlt = spr = 0;
                } else {
                    // ---------------- score: bytes of all children, in registers
                    uint32_t cand[NT][NCAND];
                    int b = max(m0, m0 + dlt - 63), sh = 0;
                    int tb = 0;            // threshold byte
                    bool coarse = false;
                    for (;;) {
                        float yminf = FBIG;
                        int ymini = 0x7fffffff;
                        const float inv = FAST ? __builtin_ldexpf(1.f, -sh) : 1.f;
                        const int sc = FAST ? a.unit_exp - sh : SC_ONE;   // scale of the weights
                        // the conversion to a byte rounds to nearest: half a
                        // unit less its own step below makes it a floor
                        const float bias = FAST ? 0.5f - 0.5f * inv : 0.f;
                        uint32_t B[NT][NOP][KST][4];
                        float basef[NT];
                        int basei[NT];
#pragma unroll
                        for (int n = 0; n < NT; ++n) {
                            const int slot = (sw * NT + n) * 16 + col;
                            basei[n] = s_ped[slot] + c.edel * degP - b;
                            basef[n] = slot < nb ? (float)basei[n] * inv - bias : FBIG;
#pragma unroll
                            for (int ks = 0; ks < KST; ++ks) {
                                const int k = 4 * ks + q;
                                const uint32_t im = s_img[k * KP + slot];
                                const uint32_t ph = s_phi[k * KP + slot] | s_pc[k];
                                if (FAST) {
                                    if (a.code_img == CODE_ONE && a.code_phi == (CODE_ONE | 0x8888u)) {
                                        // weights 1 and -1: Phi sets the sign (Phi is in Img)
                                        spread_one(im, B[n][0][ks]);
#pragma unroll
                                        for (int j = 0; j < 4; ++j) B[n][0][ks][j] |= ((ph >> j) & NIB) << 3;
                                    } else {
                                        uint32_t x[4];
                                        spread_slot(im & ~ph, a.code_img, B[n][0][ks]);
                                        spread_slot(ph, a.code_phi, x);
#pragma unroll
                                        for (int j = 0; j < 4; ++j) B[n][0][ks][j] |= x[j];
                                    }
                                } else {
                                    spread_one(ph, B[n][0][ks]);
                                    spread_one(im, B[n][1][ks]);
                                }
                                if (LAB) {
                                    const uint32_t f0 = s_phi[(W + k) * KP + slot] | s_pc[W + k];
                                    const uint32_t f1 = s_phi[(2 * W + k) * KP + slot] | s_pc[2 * W + k];
#pragma unroll
                                    for (int l = 0; l < 4; ++l) {
                                        const uint32_t m = ph & ((l & 1) ? f0 : ~f0) & ((l & 2) ? f1 : ~f1);
                                        if (FAST) spread_slot(m, a.code_same, B[n][NOP - 4 + l][ks]);
                                        else spread_one(m, B[n][NOP - 4 + l][ks]);
                                    }
                                }
                            }
                        }
                        // (unit matrix of the strike-out step: row `col` of an even tile)
                        uint32_t e_lo[4];
                        spread_row(1u << col, e_lo);
                        // (opaque, so that the tiles' bounds are compared where
                        // they are needed and not kept for the whole pair)
                        int nav = __builtin_amdgcn_readfirstlane(nact), qv = q;
                        asm volatile("" : "+s"(nav), "+v"(qv));
                        constexpr int TG = 8 / UW;           // tiles of a 128-vertex group
                        constexpr int TP = TG >= 4 && W == 16 ? 4 : (TG > 1 ? 2 : 1);   // tiles in flight
#pragma unroll
                        for (int g = 0; g < (2 * WU + 7) / 8; ++g) {
                            uint32_t bd[NT][4];
#pragma unroll
                            for (int n = 0; n < NT; ++n)
                                spread_one(4 * g + qv < WU ? s_use[(4 * g + qv) * KP + (sw * NT + n) * 16 + col] : 0u, bd[n]);
#pragma unroll
                            for (int kk = 0; kk < TG; kk += TP) {
                                const int k0 = g * TG + kk;   // this wave's tiles k0 .. k0 + TP - 1
                                if (k0 >= NTL) continue;
                                // a few tiles' operands at a time
                                __builtin_amdgcn_sched_barrier(0);
                                if (16 * (k0 * UW + uw) >= nav) {
#pragma unroll
                                    for (int h = 0; h < TP; ++h)
#pragma unroll
                                        for (int n = 0; n < NT; ++n)
                                            if (k0 + h < NTL) cand[n][k0 + h] = DEAD;
                                    continue;
                                }
                                v4f dd[TP][NT], kp[TP][NT], ii[TP][NT], same[TP][NT];
                                uint32_t rw[TP][KST], rp0[TP][KST], rp1[TP][KST];
                                v4f lcv[TP];
#pragma unroll
                                for (int h = 0; h < TP; ++h) {
                                    if (k0 + h >= NTL) continue;
                                    const int tile = (k0 + h) * UW + uw;
#pragma unroll
                                    for (int ks = 0; ks < KST; ++ks) {
                                        const int at = (4 * ks + qv) * URS + 16 * tile + col;
                                        rw[h][ks] = s_rows[at];
                                        if (LAB) {
                                            rp0[h][ks] = s_rows[W * URS + at];
                                            rp1[h][ks] = s_rows[2 * W * URS + at];
                                        }
                                    }
                                    lcv[h] = *reinterpret_cast<const v4f *>(&s_lc[16 * tile + 4 * qv]);
                                }
#pragma unroll
                                for (int h = 0; h < TP; ++h) {
                                    if (k0 + h >= NTL) continue;
                                    const int tile = (k0 + h) * UW + uw;
                                    uint32_t Ad[4];
                                    const bool here = qv == ((tile >> 1) & 3);
#pragma unroll
                                    for (int j = 0; j < 4; ++j) Ad[j] = here ? ((tile & 1) ? e_lo[j] << 16 : e_lo[j]) : 0u;
#pragma unroll
                                    for (int n = 0; n < NT; ++n) {
                                        const v4f z = v4f{0.f, 0.f, 0.f, 0.f};
                                        dd[h][n] = z;
                                        if (FAST) {
#pragma unroll
                                            for (int r = 0; r < 4; ++r) dd[h][n][r] = __builtin_fmaf(lcv[h][r], inv, basef[n]);
                                        }
                                        // FAST: dd is the child; else the mark of a used vertex, and
                                        // the counts |Phi & N2(u)|, |Img & N2(u)|, same apart
                                        dd[h][n] = mfma_fp4(Ad, bd[n], dd[h][n], SC_BIG, SC_ONE);
                                        kp[h][n] = ii[h][n] = same[h][n] = z;
                                    }
                                }
#pragma unroll
                                for (int ks = 0; ks < KST; ++ks)
#pragma unroll
                                    for (int h = 0; h < TP; ++h) {
                                        if (k0 + h >= NTL) continue;
                                        uint32_t A[4];
                                        spread_row(rw[h][ks], A);
#pragma unroll
                                        for (int n = 0; n < NT; ++n) {
                                            if (FAST) {
                                                dd[h][n] = mfma_fp4(A, B[n][0][ks], dd[h][n], SC_ONE, sc);
                                            } else {
                                                kp[h][n] = mfma_fp4(A, B[n][0][ks], kp[h][n], SC_ONE, SC_ONE);
                                                ii[h][n] = mfma_fp4(A, B[n][1][ks], ii[h][n], SC_ONE, SC_ONE);
                                            }
                                        }
                                        if (LAB) {
#pragma unroll
                                            for (int l = 0; l < 4; ++l) {
                                                if (FAST && l >= 2 && P < 2) continue;   // one plane: two codes
                                                spread_row(rw[h][ks] & ((l & 1) ? rp0[h][ks] : ~rp0[h][ks]) &
                                                               ((l & 2) ? rp1[h][ks] : ~rp1[h][ks]), A);
#pragma unroll
                                                for (int n = 0; n < NT; ++n) {
                                                    if (FAST) dd[h][n] = mfma_fp4(A, B[n][NOP - 4 + l][ks], dd[h][n], SC_ONE, sc);
                                                    else same[h][n] = mfma_fp4(A, B[n][NOP - 4 + l][ks], same[h][n], SC_ONE, SC_ONE);
                                                }
                                            }
                                        }
                                    }
#pragma unroll
                                for (int h = 0; h < TP; ++h)
#pragma unroll
                                    for (int n = 0; n < NT; ++n) {
                                        if (k0 + h >= NTL) continue;
                                        uint32_t w = 0u;
                                        if (FAST) {
                                            // (med3: fminf of a matrix result costs a second
                                            // instruction, which quiets a NaN that cannot be)
                                            float y[4];
#pragma unroll
                                            for (int r = 0; r < 4; ++r) {
                                                y[r] = __builtin_amdgcn_fmed3f(dd[h][n][r], -1.f, (float)XCAP);
                                                w = __builtin_amdgcn_cvt_pk_u8_f32(y[r], r, w);
                                            }
                                            yminf = fminf(yminf, fminf(fminf(y[0], y[1]), fminf(y[2], y[3])));
                                        } else {
                                            const bool dead = (sw * NT + n) * 16 + col >= nb;
#pragma unroll
                                            for (int r = 0; r < 4; ++r) {
                                                const int kept = (int)kp[h][n][r];
                                                int y = basei[n] + __float_as_int(lcv[h][r]) + c.eins * ((int)ii[h][n][r] - kept) - c.edel * kept;
                                                if (LAB) y += c.esub * (kept - (int)same[h][n][r]);
                                                y = (dead || dd[h][n][r] > 0.5f) ? 0x7fffffff : y;
                                                ymini = min(ymini, y);
                                                w |= (uint32_t)min(max(y >> sh, 0), XCAP) << (8 * r);
                                            }
                                        }
                                        cand[n][k0 + h] = w;
                                    }
                                // alternate the pipes' instructions: 31.0 -> 29.7 thousand
                                // cycles a level at 500 vertices, K = 256 (no gain on
                                // shorter chains)
                                if (FAST && TP == 4) {
#pragma unroll
                                    for (int z = 0; z < TP * NT * (KST * (LAB ? 5 : 1) + 1); ++z) {
                                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                                        __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                                    }
                                }
                            }
                        }
                        // the deletion children, one byte per slot
#pragma unroll
                        for (int n = 0; n < NT; ++n) {
                            const int slot = (sw * NT + n) * 16 + col;
                            const bool mine = q == 0 && uw == 0 && slot < nb;
                            const int y = s_ped[slot] + del_cost - b;
                            cand[n][NTL] = mine ? (0x7f7f7f00u | (uint32_t)min(max(y >> sh, 0), XCAP)) : DEAD;
                            if (mine) {
                                if (FAST) yminf = fminf(yminf, (float)y * inv - bias);
                                else ymini = min(ymini, y);
                            }
                        }
                        int ylow;   // lower bound of the least byte (exact when sh = 0 and not below 0)
                        {
                            // (held to 2^30 on both sides, so that its offset below cannot wrap: a child
                            // may lie up to 2^31 below b, and anything below 0 says the same)
                            const int yl = FAST ? (int)floorf(fminf(yminf, 1.0e6f))
                                                : max(min(ymini >> sh, 1000000), -0x40000000);
                            const uint32_t wm = wave_umin((uint32_t)yl + 0x40000000u);
                            if (lane == 0) s_red[0][wid] = wm;
                            __syncthreads();
                            uint32_t m = s_red[0][0];
#pragma unroll
                            for (int k = 1; k < NWV; ++k) m = min(m, s_red[0][k]);
                            ylow = (int)(m - 0x40000000u);
                        }

                        // ---------------- the smallest byte t with at least K children at or below it
                        int lo = max(sh == 0 ? ylow : ylow - 1, 0), hi = XCAP;
                        const int off = lo;
                        int ta = max(min(spr + off, XCAP - 1) - 1, off), tc = min(ta + 1, XCAP - 1);
                        int par = 1;
                        for (int s = 1; lo < hi; s <<= 1) {
                            const uint32_t Ca = ((uint32_t)ta * 0x01010101u) | HI, Cb = ((uint32_t)tc * 0x01010101u) | HI;
                            uint32_t ca = 0u, cb = 0u;
#pragma unroll
                            for (int k8 = 0; k8 < NTL; k8 += 8) {
                                if (k8 > 0 && 16 * k8 * UW >= nact) break;   // past the last tile
#pragma unroll
                                for (int n = 0; n < NT; ++n)
#pragma unroll
                                    for (int k = k8; k < k8 + 8 && k < NTL; ++k) {
                                        ca += (uint32_t)__popc((Ca - cand[n][k]) & HI);
                                        cb += (uint32_t)__popc((Cb - cand[n][k]) & HI);
                                    }
                            }
#pragma unroll
                            for (int n = 0; n < NT; ++n) {
                                ca += (uint32_t)__popc((Ca - cand[n][NTL]) & HI);
                                cb += (uint32_t)__popc((Cb - cand[n][NTL]) & HI);
                            }
                            const uint32_t w = wave_sum(ca | (cb << 16));
                            if (lane == 0) s_red[par][wid] = w;
                            __syncthreads();
                            int na = 0, nc = 0;
#pragma unroll
                            for (int k = 0; k < NWV; ++k) {
                                const uint32_t v = s_red[par][k];
                                na += (int)(v & 0xffffu);
                                nc += (int)(v >> 16);
                            }
                            par ^= 1;
                            if (nc >= K) hi = min(hi, tc);
                            else lo = max(lo, tc + 1);
                            if (na >= K) hi = min(hi, ta);
                            else lo = max(lo, ta + 1);
                            if (lo >= hi) break;
                            if (hi == XCAP) {
                                ta = min(lo + s - 1, XCAP - 1);
                                tc = min(lo + 2 * s, XCAP - 1);
                            } else if (lo == off) {
                                tc = hi - 1;
                                ta = max(hi - 1 - s, off);
                            } else {
                                const int span = hi - lo;
                                ta = lo + (span - 1) / 3;
                                tc = lo + (2 * span - 1) / 3;
                            }
                        }
                        __syncthreads();   // the last round's sums are read before the next pass writes
                        // exact when the range is exact and T lies inside it
                        // (byte 0 also stands for children below b)
                        if (sh == 0 && lo < XCAP && (lo > 0 || ylow >= 0)) {
                            tb = lo;
                            dlt = b + tb - m0;
                            spr = tb - ylow;
                            break;
                        }
                        if (!coarse) {
                            coarse = true;
                            b = m0;
                            sh = 0;
                            while (((a.pedbound - (uint32_t)m0) >> sh) >= (uint32_t)XCAP) ++sh;
                        } else {
                            // bucket `lo` becomes the range, one byte up: byte 0 takes what is below it
                            const int sn = max(sh - 6, 0);
                            b += (lo << sh) - (1 << sn);
                            sh = sn;
                        }
                        spr = 0;
                    }

                    // ---------------- survivors' bits
                    const uint32_t Cle = ((uint32_t)tb * 0x01010101u) | HI;
                    const uint32_t Clt = tb > 0 ? (((uint32_t)tb - 1u) * 0x01010101u) | HI : DEAD;
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        const int slot = (sw * NT + n) * 16 + col;
#pragma unroll
                        for (int k4 = 0; k4 < NCAND; k4 += 4) {
                            if (k4 > 0 && k4 + 4 <= NTL && 16 * k4 * UW >= nact) continue;
                            // most words hold no survivor: one test for four
                            uint32_t f[4], any = 0u;
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                f[k] = k4 + k < NCAND ? (Cle - cand[n][k4 + k < NCAND ? k4 + k : 0]) & HI : 0u;
                                any |= f[k];
                            }
                            if (!any) continue;
#pragma unroll
                            for (int k = 0; k < 4; ++k) {
                                if (k4 + k >= NCAND || !f[k]) continue;
                                const uint32_t flt = (Clt - cand[n][k4 + k]) & HI;
                                const int tile = (k4 + k) * UW + uw;
                                const int row = k4 + k < NTL ? (tile >> 1) * KP + slot : WU * KP + slot;
                                const int shf = k4 + k < NTL ? 16 * (tile & 1) + 4 * q : 0;
                                atomicOr(&s_le[row], (__builtin_amdgcn_udot4(f[k], 0x08040201u, 0u, false) >> 7) << shf);
                                if (flt)
                                    atomicOr(&s_lt[row], (__builtin_amdgcn_udot4(flt, 0x08040201u, 0u, false) >> 7) << shf);
                            }
                        }
                    }
                }
                __syncthreads();

                // ---------------- emission in generation order: slot, vertex, the
                // deletion last; a thread takes CW words of its slot's masks.
                // One scan of (children below T, ties at T), the ties capped at K
                uint32_t ml[CW], me[CW];
                int lt = 0, eq = 0;
#pragma unroll
                for (int k = 0; k < CW; ++k) {
                    const int w = part * CW + k;
                    const uint32_t m = w <= WU ? s_lt[w * KP + us] : 0u;
                    ml[k] = m;
                    me[k] = (w <= WU ? s_le[w * KP + us] : 0u) & ~m;
                    lt += __popc(ml[k]);
                    eq += __popc(me[k]);
                }
                const uint32_t both = (uint32_t)lt | ((uint32_t)min(eq, K) << 11);
                uint32_t pre = (uint32_t)wave_excl_scan((int)both);
                if (lane == 63) s_red[0][wid] = pre + both;
                __syncthreads();
                uint32_t all = 0u;
#pragma unroll
                for (int k = 0; k < NWV; ++k) {
                    const uint32_t x = s_red[0][k];
                    pre += k < wid ? x : 0u;
                    all += x;
                }
                nb_new = min(V, K);
                if (lt + eq > 0) {
                    quota = nb_new - (int)(all & 2047u);            // ties at T that survive
                    const int eqb = min((int)(pre >> 11), quota);   // ... of the threads before
                    int keq = min(quota - eqb, eq);
                    int pos = (int)(pre & 2047u) + eqb;
#pragma unroll
                    for (int k = 0; k < CW; ++k) {
                        uint32_t m = keq > 0 ? ml[k] | me[k] : ml[k];
                        while (m) {
                            const uint32_t bit = m & (0u - m);
                            m ^= bit;
                            if (me[k] & bit) {
                                if (keq == 0) continue;
                                --keq;
                            }
                            const int w = part * CW + k;
                            s_sel[pos++] = (us << 10) | (w < WU ? 32 * w + (int)__builtin_ctz(bit) : DELU);
                        }
                    }
                }
            }
            __syncthreads();

            // ---------------- update: the new slots gather their parents' state ...
            const int par = i & 1;
            const bool live = us < nb_new;
            int p = 0, at = DELU, nped = 0, nns = 0;
            uint32_t nim[NWP], nus[NWP];
            uint16_t cv[(BL + PARTS - 1) / PARTS];
            const int r8 = i % BL;      // row of this level in its block
            if (live) {
                const int sel = s_sel[us];
                p = sel >> 10;
                at = sel & 1023;
            }
            const bool sub = at < nact;
            const int u = sub ? (int)s_act[at] : n2;
            {
                int kept = 0, inimg = 0, relab = 0;
#pragma unroll
                for (int k = 0; k < NWP; ++k) {
                    const int w = part + k * PARTS;
                    nim[k] = nus[k] = 0u;
                    if (w < WU && live) {
                        nus[k] = s_use[w * KP + p];
                        if (sub && w == (at >> 5)) nus[k] |= 1u << (at & 31);
                    }
                    if (w < W && live) {
                        const uint32_t im = s_img[w * KP + p];
                        nim[k] = im;
                        if (sub) {
                            const uint32_t row = s_rows[w * URS + at];
                            const uint32_t ph = s_phi[w * KP + p] | s_pc[w];
                            kept += __popc(ph & row);
                            inimg += __popc(im & row);
                            if (LAB) {
                                const uint32_t f0 = (s_phi[(W + w) * KP + p] | s_pc[W + w]) ^ s_rows[(W + w) * URS + at];
                                const uint32_t f1 = (s_phi[(2 * W + w) * KP + p] | s_pc[2 * W + w]) ^ s_rows[(2 * W + w) * URS + at];
                                relab += __popc(ph & row & (f0 | f1));
                            }
                            if (w == (u >> 5) || (DIR && w == (u >> 5) + WU)) nim[k] |= 1u << (u & 31);
                        }
                    }
                }
                // (none of the three reaches 1024)
                const uint32_t sum = parts_sum<PARTS>((uint32_t)(kept | (inimg << 10) | (relab << 20)));
                kept = (int)(sum & 1023u);
                inimg = (int)((sum >> 10) & 1023u);
                relab = (int)(sum >> 20);
                if (live) {
                    nped = s_ped[p];
                    nns = s_nsub[p] + (sub ? 1 : 0);
                    if (sub)
                        nped += (lab1 != s_l2[at] ? c.vsub : 0) + c.edel * (degP - kept) + c.eins * (inimg - kept) +
                                c.esub * relab;
                    else
                        nped += del_cost;
#pragma unroll
                    for (int k = 0; k < (BL + PARTS - 1) / PARTS; ++k) {
                        const int r = part + k * PARTS;
                        cv[k] = r < r8 ? s_cur[r * KS + p] : (uint16_t)0;
                    }
                }
                const int vs = wave_sum((live && part == 0) ? (uint32_t)(n2 - nns + 1) : 0u);
                const uint32_t mn = wave_umin((live && part == 0) ? (uint32_t)nped : 0xffffffffu);
                if (lane == 0) {
                    atomicAdd(&s_sumV[par], vs);
                    atomicMin(&s_min[par], mn);
                }
            }
            // ... and write it, all at once (the ancestor rows in steps)
            Anc av[MAXA];
            bool rest = true;
            for (int g = b0; rest; g += MAXA * PARTS) {
#pragma unroll
                for (int k = 0; k < MAXA; ++k) {
                    const int r = g + part + k * PARTS;
                    av[k] = (r < nblk && live) ? s_anc[r * KS + p] : (Anc)0;
                }
                __syncthreads();
                if (g == b0) {
                    if (live) {
#pragma unroll
                        for (int k = 0; k < NWP; ++k) {
                            const int w = part + k * PARTS;
                            if (w < W) s_img[w * KP + us] = nim[k];
                            if (w < WU) s_use[w * KP + us] = nus[k];
                        }
                        const uint16_t xi = sub ? (uint16_t)u : (uint16_t)DEL16;
                        const bool full = r8 == BL - 1;
#pragma unroll
                        for (int k = 0; k < (BL + PARTS - 1) / PARTS; ++k) {
                            const int r = part + k * PARTS;
                            if (r > r8) continue;
                            const uint16_t x = r == r8 ? xi : cv[k];
                            if (full) phi_g[(size_t)(i - r8 + r) * KS + us] = x;
                            else s_cur[r * KS + us] = x;
                        }
                        if (part == 0) {
                            s_ped[us] = nped;
                            s_nsub[us] = nns;
                            if (full) s_anc[nblk * KS + us] = (Anc)us;
                        }
                    }
#pragma unroll
                    for (int k = 0; k < NWP; ++k) {
                        const int w = part + k * PARTS;
                        if (w < W) {
#pragma unroll
                            for (int b = 0; b < NA; ++b) s_phi[(b * W + w) * KP + us] = 0u;
                        }
                    }
                    for (int w = part; w <= WU; w += PARTS) {
                        s_le[w * KP + us] = 0u;
                        s_lt[w * KP + us] = 0u;
                    }
                    if (t < NA * W) s_pc[t] = 0u;
                    if (t < ND * NA * W1) s_r1[((i + 1) & 1) * (ND * NA * W1) + t] = rown;
                    if (t == 0) {
                        s_neq = 0;
                        s_sumV[par ^ 1] = 0;
                        s_min[par ^ 1] = 0xffffffffu;
                    }
                }
                if (live) {
#pragma unroll
                    for (int k = 0; k < MAXA; ++k) {
                        const int r = g + part + k * PARTS;
                        if (r < nblk) s_anc[r * KS + us] = av[k];
                    }
                }
                rest = g + MAXA * PARTS < nblk;
            }
            if (r8 == BL - 1) ++nblk;
            nb = nb_new;
            __syncthreads();
            V = s_sumV[par];
            m0 = (int)s_min[par];

            // ---------------- images common to the whole beam are used in every
            // slot: they go behind the other positions, and every slot's bits
            // close up (CB blocks at a time: fewer would free no group of tiles;
            // not for the last levels, where it would cost more than it saves)
            if (b0 - cb >= CB && i + 2 * BL < n1) {
                if (t < WU) s_gone[t] = 0u;
                __syncthreads();
                for (int x = BL * cb + t; x < BL * b0; x += T) {
                    const uint32_t v = s_com[x];
                    if (v != DEL16) atomicOr(&s_gone[v >> 5], 1u << (v & 31));
                }
                __syncthreads();
                constexpr int AE = (32 * WU + T - 1) / T;   // positions of a thread
                uint16_t ua[AE];
                int lb[AE], to[AE];
#pragma unroll
                for (int k = 0; k < AE; ++k) {
                    const int x = t + k * T;
                    ua[k] = 0;
                    lb[k] = 0;
                    if (x < nact) {
                        ua[k] = s_act[x];
                        lb[k] = s_l2[x];
                    }
                    const unsigned long long m =
                        __ballot(x < nact && ((s_gone[ua[k] >> 5] >> (ua[k] & 31)) & 1u));
                    if ((lane & 31) == 0 && x < 32 * WU) s_rm[x >> 5] = (uint32_t)(lane ? m >> 32 : m);
                }
                __syncthreads();
                int out = 0;
#pragma unroll
                for (int w = 0; w < WU; ++w) out += __popc(s_rm[w]);
#pragma unroll
                for (int k = 0; k < AE; ++k) {
                    const int x = t + k * T;
                    int before = 0;
#pragma unroll
                    for (int w = 0; w < WU; ++w) before += __popc(s_rm[w] & below(x, w));
                    const bool leaves = x < nact && ((s_rm[x >> 5] >> (x & 31)) & 1u);
                    to[k] = leaves ? nact - out + before : x - before;
                    if (x < nact) {
                        s_act[to[k]] = ua[k];
                        s_l2[to[k]] = lb[k];
                    }
                }
#pragma unroll 1
                for (int r = 0; r < NA * W; r += 4) {
                    uint32_t rv[AE][4];
#pragma unroll
                    for (int k = 0; k < AE; ++k)
#pragma unroll
                        for (int z = 0; z < 4; ++z) rv[k][z] = t + k * T < nact ? s_rows[(r + z) * URS + t + k * T] : 0u;
                    __syncthreads();
#pragma unroll
                    for (int k = 0; k < AE; ++k)
#pragma unroll
                        for (int z = 0; z < 4; ++z)
                            if (t + k * T < nact) s_rows[(r + z) * URS + to[k]] = rv[k][z];
                }
                // one thread a slot: positions taken out from the highest on, a
                // used one shifted in at the top
                if (t < KS) {
                    uint32_t wv[WU];
#pragma unroll
                    for (int k = 0; k < WU; ++k) wv[k] = s_use[k * KP + t];
#pragma unroll
                    for (int w = WU - 1; w >= 0; --w) {
                        uint32_t m = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_rm[w]);
                        while (m) {
                            const int b = 31 - __builtin_clz(m);
                            m ^= 1u << b;
                            const uint32_t low = (1u << b) - 1u;   // bits that stay
#pragma unroll
                            for (int k = w; k < WU; ++k) {
                                const uint32_t up = k + 1 < WU ? wv[k + 1 < WU ? k + 1 : 0] : 0xffffffffu;
                                const uint32_t sh = (wv[k] >> 1) | (up << 31);
                                wv[k] = k == w ? (wv[k] & low) | (sh & ~low) : sh;
                            }
                        }
                    }
#pragma unroll
                    for (int k = 0; k < WU; ++k) s_use[k * KP + t] = wv[k];
                }
                nact -= out;
                cb = b0;
                __syncthreads();
            }
        }

        // ---------------- completion: insert what is left of g2, pick the best leaf
        const int us = t / PARTS, part = t % PARTS;
        unsigned long long best = ~0ull;
        if (us < nb) {
            const int e2 = inside(us, part);
            const int total = s_ped[us] + c.vins * (n2 - s_nsub[us]) + c.eins * (g2.m - e2 / 2);
            best = ((unsigned long long)(unsigned)total << 32) | (unsigned)us;
        }
        best = wave_min64(best);
        if ((t & 63) == 0) s_red64[wid] = best;
        __syncthreads();
        best = s_red64[0];
#pragma unroll
        for (int k = 1; k < NWV; ++k) best = s_red64[k] < best ? s_red64[k] : best;
        const int bs = (int)(best & 0xffffffffu);
        if (t == 0) {
            a.out.dist[wi.out] = (int)(best >> 32);
            if (a.out.cand) a.out.cand[wi.out] = ce;
        }
        for (int j = t; j < n1; j += T) {
            const uint32_t x = j < BL * b0 ? (uint32_t)s_com[j] : image(j, bs);
            a.out.map[wi.map_off + j] = x == DEL16 ? -1 : (int)x;
        }
        __syncthreads();
    }
}

// The slot operand's nibbles for these costs (plain: Img \ Phi and Phi; with
// edge labels also Phi_c): false if they are not small multiples of a power of
// two.
struct SlotCodes {
    uint32_t img = 0, phi = 0, same = 0;
    int unit_exp = SC_ONE;
};
bool slot_codes(const Costs &c, bool labels, SlotCodes *out);

struct MatConfig {
    int W = 0, NT = 0, SW = 0, UW = 0;   // W == 0: no instantiation
};

template <bool LAB, bool DIR, bool FAST>
const void *mat_select(const MatConfig &m) {
#define GEDK_M(w, nt, sw, uw)                                  \
    if (m.W == w && m.NT == nt && m.SW == sw && m.UW == uw)     \
        return reinterpret_cast<const void *>(&kb_mat_kernel<w, nt, sw, uw, LAB, DIR, FAST>);
#define GEDK_MW(nt, sw, uw) GEDK_M(4, nt, sw, uw) GEDK_M(8, nt, sw, uw) GEDK_M(16, nt, sw, uw)
    GEDK_MW(1, 1, 4) GEDK_MW(1, 2, 2) GEDK_MW(1, 4, 1) GEDK_MW(1, 4, 2)
    GEDK_M(4, 1, 8, 1) GEDK_M(8, 1, 8, 1) GEDK_M(4, 2, 8, 1) GEDK_M(8, 2, 8, 1) GEDK_M(4, 4, 8, 1)
    // the largest states: LDS holds them without label planes, some with those of
    // directed graphs, whose rows are half as many
    if constexpr (!LAB) { GEDK_M(16, 2, 8, 1) }
    if constexpr (!LAB || DIR) { GEDK_M(16, 1, 8, 1) GEDK_M(8, 4, 8, 1) GEDK_M(4, 4, 16, 1) }
#undef GEDK_MW
#undef GEDK_M
    return nullptr;
}

// The instantiations for undirected / directed graphs without / with edge
// labels, each in a source of its own.
const void *mat_kernel_plain(const MatConfig &m, bool fast);
const void *mat_kernel_lab(const MatConfig &m, bool fast);
const void *mat_kernel_dir(const MatConfig &m, bool fast);
const void *mat_kernel_dir_lab(const MatConfig &m, bool fast);

}  // namespace mat
}  // namespace gedk
