// kb_widem.hip -- the whole-device search of one pair (kb_wide.hip) for larger
// targets without edge labels, with the children scored on the matrix cores:
// the paper's runtime-versus-size experiment (500 vertices at K = 5000).
//
// The scoring is that of kb_mat.h (fp4 0/1 operands, exact f32 sums; eins and
// edel small multiples of one power of two), and so is the mapping: images of
// the last incomplete block of 8 levels as rows that are gathered from level to
// level, complete blocks written once and reached through one ancestor index
// per block, blocks that the whole beam shares moved to the common mapping.  A
// level is three kernels, the first two on a grid of (64 slots) x (128 target
// vertices), a wave holding 16 slots:
//   expand   Phi of the 64 slots (stored for the others), every child's PED,
//            an LDS histogram above the least parent PED, added to one of HC
//            copies (atomics on one address are serialised, about 10 ns each).
//            A workgroup with children past the histogram's range (HB values)
//            scores them again, HB values at a time, into the far histogram:
//            exact counts of every value, and their sums per HB of them.
//   mark     the threshold T from the histogram, by every workgroup (should
//            the K-th child lie past its range: from the far one, first the
//            sums, then one group's values); then scores again -- cheaper than a
//            candidate matrix of 4 bytes a child, written once and read twice --
//            and stores, per slot, a bit per vertex for children at most T and
//            below T, and their counts per 64 slots.
//   update   every workgroup adds up the counts before its 64 slots, places its
//            survivors in generation order (slot, vertex ascending, the deletion
//            last, ties at T while the quota lasts) and writes them, four
//            threads a slot; one more workgroup prepares the next level's
//            neighbour lists and the common part of its Phi.
// A kernel here is a few microseconds of dependent loads, so each begins with
// every load that needs no answer.
//
// Two 500-vertex graphs at K = 5000 (MI355X): 39.6 ms with kb_wide.hip's kernels
// (79 us a level), 17.0 ms so: 13.0 us of expand, 12.0 of mark and 9.4 of update
// a level, each a chain of about six dependent loads and a launch; scoring all
// 2.5 million children is about 1 us of it.
#include <algorithm>

#include "kb_mat.h"

namespace gedk {
namespace {

using namespace mat;

constexpr int WT = 256;
constexpr int NWV = WT / 64;
constexpr int HB = 4096;          // histogram bins; the last one also counts what is above
constexpr int HC = 2;             // copies
constexpr uint32_t FAR = (uint32_t)kFastBound;   // values of the far histogram (no PED of the search reaches it)
constexpr int FC = (int)(FAR / HB);              // ... and sums of HB of them
constexpr int GS = 64;            // slots of a workgroup
constexpr int GP = GS + 16;       // their LDS stride
constexpr int CT = 8;             // target tiles of a workgroup (128 vertices)
constexpr int CWD = 4;            // ... words
constexpr int RS = 32 * CWD + 16; // LDS stride of a row word over a chunk's vertices
constexpr int MAXN = GED_MAX_VERTICES;
constexpr uint32_t NONE = 0xffffffffu;
constexpr int UBITS = 11;         // record: slot << UBITS | vertex (n2: the deletion)
static_assert(MAXN < 1 << UBITS && (int64_t)kWideMaxK << UBITS <= (int64_t)1 << 32, "record");
static_assert((int64_t)kWideMaxK * (MAXN + 1) < (int64_t)1 << 32, "children of a level: 32 bits");
constexpr uint32_t kCommonMost = 1u << 16;   // beams whose oldest block is looked at

struct Level {
    uint32_t B, m0, mmax;    // parents, their least and largest PED
    uint32_t quota;          // children equal to the threshold that survive
    uint32_t b0;             // first block not yet common
    uint32_t far;            // the level has children past the histogram
    uint32_t pad[2];
};

// What a level needs of v_i and the common mapping, made while the level before
// is written.
struct Prep {
    uint32_t deg;            // earlier neighbours of v_i
    uint32_t nwb, nw;        // window neighbours: in complete blocks, and all
    uint32_t pad;
    uint32_t pc[MAXN / 32];  // images of the common ones
    uint16_t nbr[MAXN];      // the window's, those of complete blocks first
};

struct Ctx {
    const uint32_t *a1;
    const int32_t *l1;
    const uint32_t *a2;
    const int32_t *l2;
    int n1, w1, n2, w2, m2;
    Costs c;
    uint32_t pedmax;
    uint32_t code_img, code_phi;
    int unit_exp;
    uint32_t K, Kp;
    int blocks;              // mapping blocks of n1
    uint32_t *ped[2], *nsub[2];
    uint32_t *img[2];        // [W][Kp]
    uint16_t *cur[2];        // [BL][Kp] images of the incomplete block
    uint32_t *anc[2];        // [blocks][Kp] slot of the block's last level
    uint16_t *phi;           // [n1][Kp] complete blocks
    uint16_t *com;           // [n1] common mapping
    uint32_t *sets;          // [W][Kp] Phi of the level
    uint32_t *le, *lt;       // [W + 1][Kp] children at most T, below T (last word: the deletion)
    uint32_t *cnt;           // [2][groups] below T, equal to T per 64 slots
    uint32_t *rec;           // [Kp]
    uint32_t *hist;          // [HC][HB]
    Level *st;
    Prep *prep;
    unsigned long long *ce, *best;   // best: a key per workgroup
    int32_t *out_dist, *out_map;
    int64_t *out_cand;
    uint32_t *far, *farc;    // [FAR] children past the histogram, by value above the least parent PED; [FC] sums
};

__device__ __forceinline__ uint32_t sgpr(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

template <int NW>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *s_tmp, uint32_t *total) {
    const int wid = threadIdx.x >> 6;
    const uint32_t x = (uint32_t)wave_excl_scan((int)v);
    if ((threadIdx.x & 63) == 63) s_tmp[wid] = x + v;
    __syncthreads();
    uint32_t pre = 0u, tot = 0u;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
        const uint32_t t = s_tmp[k];
        pre += k < wid ? t : 0u;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return pre + x;
}

__device__ __forceinline__ uint32_t degree(const Ctx &c, int i) {
    const int lane = threadIdx.x & 63;
    return wave_sum(lane < c.w1 ? (uint32_t)__popc(c.a1[(size_t)i * c.w1 + lane] & below(i, lane)) : 0u);
}

__global__ __launch_bounds__(WT) void wm_init(Ctx c) {
    const int t = blockIdx.x * WT + threadIdx.x, T = gridDim.x * WT;
    for (int l = t; l <= c.n1; l += T) {
        Level s = {};
        s.B = l == 0 ? 1u : 0u;
        c.st[l] = s;
    }
    for (int b = t; b < HC * HB; b += T) c.hist[b] = 0u;
    if (c.pedmax >= (uint32_t)(HB - 1)) {   // (else no level has values past the histogram)
        const uint32_t end = (c.pedmax / HB + 1u) * HB;   // whole sums
        for (uint32_t b = t; b < end; b += T) c.far[b] = 0u;
        for (int b = t; b < FC; b += T) c.farc[b] = 0u;
    }
    for (int k = t; k < c.w2; k += T) c.img[0][(size_t)k * c.Kp] = 0u;
    for (int k = t; k < (int)(sizeof(Prep) / 4); k += T) reinterpret_cast<uint32_t *>(c.prep)[k] = 0u;
    if (t == 0) {
        c.ped[0][0] = 0u;
        c.nsub[0][0] = 0u;
        *c.ce = 0ull;
    }
}

// The level's 64 slots against 128 target vertices: operands staged in LDS.
template <int W>
struct Tile {
    static constexpr int KST = W / 4;
    uint32_t *s_rows;   // [W][RS]
    float *s_lc;        // [RS]
    uint32_t *s_phi;    // [W][GP]

    __device__ __forceinline__ void stage_rows(const Ctx &c, int i, int u0) const {
        const int t = threadIdx.x;
        for (int x = t; x < W * 32 * CWD; x += WT) {
            const int uu = x / W, k = x % W, u = u0 + uu;
            s_rows[k * RS + uu] = (u < c.n2 && k < c.w2) ? c.a2[(size_t)u * c.w2 + k] : 0u;
        }
        const int lab1 = c.l1[i];
        if (t < 32 * CWD) s_lc[t] = (u0 + t < c.n2 && c.l2[u0 + t] != lab1) ? (float)c.c.vsub : 0.f;
    }

    // This lane's slot: its words of Img, the chunk's own once more for the
    // strike-out, and its PED.  Loaded before anything is waited for: rows past
    // the beam hold what they did before, and are not looked at.
    struct Slot {
        uint32_t im[KST], own, ped;
        __device__ __forceinline__ void load(const Ctx &c, int i, uint32_t s0, int u0) {
            const int lane = threadIdx.x & 63, q = lane >> 4, ls = (threadIdx.x >> 6) * 16 + (lane & 15), cur = i & 1;
            const uint32_t s = s0 + (uint32_t)ls;   // below Kp
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
                const int k = 4 * ks + q;
                im[ks] = k < c.w2 ? c.img[cur][(size_t)k * c.Kp + s] : 0u;
            }
            const int kd = (u0 >> 5) + q;
            own = (kd < c.w2 ? c.img[cur][(size_t)kd * c.Kp + s] : 0u) | ~below(c.n2, kd);   // past n2: used
            ped = c.ped[cur][s];
        }
    };

    // f(k, y): the four children 16 k + 4 q .. + 3 of this lane's slot, y their
    // PEDs plus `shift` (used vertices and dead slots near 2^24), for the
    // chunk's tiles in turn
    template <class F>
    __device__ __forceinline__ void score(const Ctx &c, const Slot &sl, int t, uint32_t s0, uint32_t B, int u0, float shift, F f) const {
        const int lane = t & 63, wid = __builtin_amdgcn_readfirstlane(t >> 6);
        const int q = lane >> 4, col = lane & 15, ls = wid * 16 + col;
        uint32_t Bo[KST][4], bd[4];
#pragma unroll
        for (int ks = 0; ks < KST; ++ks) {
            const uint32_t ph = s_phi[(4 * ks + q) * GP + ls];
            if (c.code_img == CODE_ONE && c.code_phi == (CODE_ONE | 0x8888u)) {
                spread_one(sl.im[ks], Bo[ks]);
#pragma unroll
                for (int j = 0; j < 4; ++j) Bo[ks][j] |= ((ph >> j) & NIB) << 3;
            } else {
                uint32_t x[4];
                spread_slot(sl.im[ks] & ~ph, c.code_img, Bo[ks]);
                spread_slot(ph, c.code_phi, x);
#pragma unroll
                for (int j = 0; j < 4; ++j) Bo[ks][j] |= x[j];
            }
        }
        spread_one(sl.own, bd);
        const float base = s0 + (uint32_t)ls < B ? (float)sl.ped + shift : FBIG;
        uint32_t e_lo[4];
        spread_row(1u << col, e_lo);
#pragma unroll
        for (int k = 0; k < CT; ++k) {
            if (u0 + 16 * k >= c.n2) break;
            uint32_t A[4], Ad[4];
            const bool here = q == ((k >> 1) & 3);
#pragma unroll
            for (int j = 0; j < 4; ++j) Ad[j] = here ? ((k & 1) ? e_lo[j] << 16 : e_lo[j]) : 0u;
            const v4f lc = *reinterpret_cast<const v4f *>(&s_lc[16 * k + 4 * q]);
            v4f y;
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = lc[r] + base;
            y = mfma_fp4(Ad, bd, y, SC_BIG, SC_ONE);
#pragma unroll
            for (int ks = 0; ks < KST; ++ks) {
                spread_row(s_rows[(4 * ks + q) * RS + 16 * k + col], A);
                y = mfma_fp4(A, Bo[ks], y, SC_ONE, c.unit_exp);
            }
            f(k, y);
        }
    }
};

// Bins that the children of a level can reach above the least parent PED.
__device__ __forceinline__ int level_bins(const Ctx &c, const Level &L, int i, uint32_t deg) {
    const uint64_t inc_sub = (uint64_t)c.c.vsub + (uint64_t)c.c.edel * deg + (uint64_t)c.c.eins * (uint64_t)min(i, c.n2);
    const uint64_t inc_del = (uint64_t)c.c.vdel + (uint64_t)c.c.edel * deg;
    uint64_t R = (uint64_t)(L.mmax - L.m0) + (inc_sub > inc_del ? inc_sub : inc_del);
    R = R < c.pedmax ? R : c.pedmax;
    return (int)(R < (uint64_t)(HB - 1) ? R : (uint64_t)(HB - 1)) + 1;
}

// ------------------------------------------------------------------ expand
// hist: 0 = only Phi (the complete-then-minimum last level).
template <int W>
__global__ __launch_bounds__(WT) void wm_expand(Ctx c, int i, int chunks, int groups, int hist) {
    __shared__ uint32_t s_rows[W * RS], s_phi[W * GP];
    __shared__ __attribute__((aligned(16))) float s_lc[RS];
    __shared__ uint32_t s_hist[HB], s_next, s_past;
    __shared__ uint16_t s_nbr[MAXN];
    const int t = threadIdx.x, slot = t % GS, p0 = t / GS;
    constexpr int PT = WT / GS;
    const int chunk = blockIdx.x % chunks, group = blockIdx.x / chunks;
    const uint32_t s0 = (uint32_t)group * GS;
    const int u0 = chunk * 32 * CWD, cur = i & 1, nblk = i / BL;
    const Tile<W> tile{s_rows, s_lc, s_phi};
    // everything that needs no answer first
    typename Tile<W>::Slot sl;
    const Level L = c.st[i];
    const int nwb = (int)c.prep->nwb, nw = (int)c.prep->nw;
    const uint32_t deg = sgpr(c.prep->deg);
    sl.load(c, i, s0, u0);
    s_nbr[t] = c.prep->nbr[t];
    for (int k = p0; k < W; k += PT) s_phi[k * GP + slot] = c.prep->pc[k];
    if (hist) tile.stage_rows(c, i, u0);
    const uint32_t B = sgpr(L.B), m0 = sgpr(L.m0);
    if (s0 >= B) return;
    const int nbins = (int)sgpr((uint32_t)level_bins(c, L, i, deg));
    for (int x = t; x < nbins; x += WT) s_hist[x] = 0u;
    for (int x = WT + t; x < nw; x += WT) s_nbr[x] = c.prep->nbr[x];
    if (chunk == 0 && t < 2) c.cnt[t * groups + group] = 0u;
    if (t == 0) s_past = 0u;
    __syncthreads();
    {
        const uint32_t s = min(s0 + (uint32_t)slot, B - 1u);
        auto put = [&](uint32_t x) {
            if (x != DEL16) atomicOr(&s_phi[(x >> 5) * GP + slot], 1u << (x & 31));
        };
        constexpr int LB = 8;
        for (int kb = p0; kb < nwb; kb += LB * PT) {
            uint32_t x[LB];
#pragma unroll
            for (int k = 0; k < LB; ++k) {
                const int kk = kb + k * PT;
                const int j = s_nbr[min(kk, nwb - 1)];
                x[k] = c.phi[(size_t)j * c.Kp + c.anc[cur][(size_t)(j / BL) * c.Kp + s]];
                x[k] = kk < nwb ? x[k] : DEL16;
            }
#pragma unroll
            for (int k = 0; k < LB; ++k) put(x[k]);
        }
        for (int kk = nwb + p0; kk < nw; kk += PT) put(c.cur[cur][(size_t)(s_nbr[kk] - BL * nblk) * c.Kp + s]);
    }
    __syncthreads();
    if (chunk == 0 && s0 + (uint32_t)slot < B)
        for (int k = p0; k < c.w2; k += PT) c.sets[(size_t)k * c.Kp + s0 + slot] = s_phi[k * GP + slot];
    if (!hist) return;

    const float shift = (float)((int)(deg * (uint32_t)c.c.edel) - (int)m0), top = (float)(nbins - 1);
    const bool over = nbins == HB;   // children past the last bin are possible
    tile.score(c, sl, t, s0, B, u0, shift, [&](int, const v4f &y) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (y[r] < 8388608.f) atomicAdd(&s_hist[(int)(over ? __builtin_amdgcn_fmed3f(y[r], 0.f, top) : y[r])], 1u);
    });
    // the deletions: one per slot, from the first k-group's lanes
    if (chunk == 0 && (t & 63) < 16 && s0 + (uint32_t)((t >> 6) * 16 + (t & 15)) < B) {
        const uint32_t d = sl.ped - m0 + (uint32_t)c.c.vdel + deg * (uint32_t)c.c.edel;
        atomicAdd(&s_hist[min(d, (uint32_t)(nbins - 1))], 1u);
    }
    __syncthreads();
    uint32_t *out = c.hist + (size_t)(blockIdx.x % HC) * HB;
    uint32_t near = 0u;   // children below the last bin (of HB)
    for (int b = t; b < nbins; b += WT) {
        const uint32_t h = s_hist[b];
        if (h) atomicAdd(&out[b], h);
        near += b < HB - 1 ? h : 0u;
    }
    if (!over || s_hist[HB - 1] == 0u) return;
    near = wave_sum(near);
    if ((t & 63) == 0) atomicAdd(&s_past, near);
    __syncthreads();
    // children of this workgroup past the histogram: HB values from `lo` on, then
    // from the least value above those, until there is none, or K are counted,
    // as the K-th of all children lies among them then (the slot's words are
    // loaded again rather than held in registers, as operands, from above on)
    if (s_past >= c.K) return;
    for (uint32_t lo = HB - 1;;) {
        __syncthreads();
        sl.load(c, i, s0, u0);
        for (int b = t; b < HB; b += WT) s_hist[b] = 0u;
        if (t == 0) s_next = NONE;
        __syncthreads();
        // (such levels have few values: the lanes that hold the first one's, then
        // those that hold the next one's, add as one)
        uint32_t above = NONE;
        auto take = [&](uint32_t d, bool live) {
            if (live && d >= lo + (uint32_t)HB) above = min(above, d);
            bool in = live && d - lo < (uint32_t)HB;
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const unsigned long long m = __ballot(in);
                if (m == 0ull) break;
                const int one = __builtin_ctzll(m);
                const uint32_t v = (uint32_t)__builtin_amdgcn_readlane((int)d, one);
                const unsigned long long same = __ballot(in && d == v);
                if ((t & 63) == one) atomicAdd(&s_hist[v - lo], (uint32_t)__popcll(same));
                in = in && d != v;
            }
            if (in) atomicAdd(&s_hist[d - lo], 1u);
        };
        int t2 = t;   // (opaque: nothing of a pass is formed before it and kept over the loop)
        asm volatile("" : "+v"(t2));
        tile.score(c, sl, t2, s0, B, u0, shift, [&](int, const v4f &y) {
#pragma unroll
            for (int r = 0; r < 4; ++r) take((uint32_t)(int)fminf(y[r], (float)FAR), y[r] < 8388608.f);
        });
        if (chunk == 0)
            take(sl.ped - m0 + (uint32_t)c.c.vdel + deg * (uint32_t)c.c.edel,
                 (t & 63) < 16 && s0 + (uint32_t)((t >> 6) * 16 + (t & 15)) < B);
        above = wave_umin(above);
        if ((t & 63) == 0 && above != NONE) atomicMin(&s_next, above);
        __syncthreads();
        const uint32_t next = s_next, c0 = lo / HB;   // the values' sums: c0, and c0 + 1
        uint32_t a = 0u, b1 = 0u;
        for (int b = t; b < HB; b += WT) {
            const uint32_t h = s_hist[b], v = lo + (uint32_t)b;
            if (h) atomicAdd(&c.far[v], h);   // (a child's value: below FAR)
            a += v / HB == c0 ? h : 0u;
            b1 += v / HB == c0 ? 0u : h;
        }
        a = wave_sum(a);
        b1 = wave_sum(b1);
        if ((t & 63) == 0) {
            if (a) atomicAdd(&c.farc[c0], a);
            if (b1) atomicAdd(&c.farc[c0 + 1u], b1);
            if (a + b1) atomicAdd(&s_past, a + b1);
        }
        if (next == NONE) return;
        __syncthreads();
        if (s_past >= c.K) return;
        lo = next;
    }
}

// ------------------------------------------------------------------ mark
// The level's threshold from its histogram, by every workgroup; *quota the
// ties that survive.  Workgroup 0 also writes the next level's size and bounds.
__device__ __forceinline__ uint32_t threshold(const Ctx &c, int i, const Level &L, uint32_t deg, uint32_t *s_bin) {
    __shared__ uint32_t s_tmp[NWV], s_res[2], s_first, s_last;
    const int t = threadIdx.x;
    const uint32_t K = c.K, B = sgpr(L.B), m0 = sgpr(L.m0);
    const int nbins = (int)sgpr((uint32_t)level_bins(c, L, i, deg));
    if (t == 0) {
        s_first = HB;
        s_last = 0u;
    }
    // the counts, coalesced, then a thread's own bins from LDS
    for (int b = t; b < nbins; b += WT) {
        uint32_t h = 0u;
#pragma unroll
        for (int k = 0; k < HC; ++k) h += c.hist[(size_t)k * HB + b];
        s_bin[b] = h;
    }
    __syncthreads();
    const int per = (nbins + WT - 1) / WT;
    uint32_t sum = 0u, first = HB, last = 0u;
    for (int q = 0; q < per; ++q) {
        const int b = t * per + q;
        const uint32_t h = b < nbins ? s_bin[b] : 0u;
        sum += h;
        if (h) {
            first = min(first, (uint32_t)b);
            last = (uint32_t)b;
        }
    }
    uint32_t V;
    const uint32_t pre = block_excl_scan<NWV>(sum, s_tmp, &V);
    if (sum) {
        atomicMin(&s_first, first);
        atomicMax(&s_last, last);
    }
    // the bin of the K-th count, given the counts below this thread's bins
    auto find = [&](uint32_t under, uint32_t mine, int n) {
        if (!(under < K && K <= under + mine)) return;
        for (int q = 0; q < n; ++q) {
            const int b = t * n + q;
            const uint32_t h = s_bin[b];   // (the K-th lies in a real bin)
            if (under + h >= K) {
                s_res[0] = (uint32_t)b;
                s_res[1] = under;
                break;
            }
            under += h;
        }
    };
    const bool all = V <= K;
    if (!all) find(pre, sum, per);
    __syncthreads();
    uint32_t T = all ? NONE : m0 + s_res[0], under = all ? 0u : s_res[1];
    if (nbins == HB && !all && s_res[0] == (uint32_t)(HB - 1)) {
        // the K-th child is past the range: its HB values, then its value
        constexpr int PER = FC / WT, PERV = HB / WT;
        uint32_t h[PER], mine = 0u, tot;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            h[q] = c.farc[t * PER + q];
            mine += h[q];
        }
        uint32_t at = under + block_excl_scan<NWV>(mine, s_tmp, &tot);
        if (at < K && K <= at + mine) {
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                if (at < K && K <= at + h[q]) {
                    s_res[0] = (uint32_t)(t * PER + q);
                    s_res[1] = at;
                }
                at += h[q];
            }
        }
        __syncthreads();
        const uint32_t first_value = s_res[0] * (uint32_t)HB;
        under = s_res[1];
        for (int b = t; b < HB; b += WT) s_bin[b] = c.far[first_value + (uint32_t)b];
        __syncthreads();
        mine = 0u;
        for (int q = 0; q < PERV; ++q) mine += s_bin[t * PERV + q];
        find(under + block_excl_scan<NWV>(mine, s_tmp, &tot), mine, PERV);
        __syncthreads();
        T = m0 + first_value + s_res[0];
        under = s_res[1];
    }
    if (blockIdx.x == 0 && t == 0) {
        Level *N = c.st + i + 1;
        c.st[i].quota = all ? 0u : K - under;
        c.st[i].far = s_last == (uint32_t)(HB - 1) ? 1u : 0u;
        N->B = min(V, K);
        N->m0 = m0 + s_first;
        // (the last bin also holds what is above it)
        N->mmax = all ? (s_last == (uint32_t)(HB - 1) ? c.pedmax : m0 + s_last) : T;
        *c.ce += V;
    }
    return T;
}

template <int W>
__global__ __launch_bounds__(WT) void wm_mark(Ctx c, int i, int chunks, int groups) {
    __shared__ uint32_t s_rows[W * RS], s_phi[W * GP];
    __shared__ __attribute__((aligned(16))) float s_lc[RS];
    __shared__ uint32_t s_bin[HB];
    __shared__ uint32_t s_le[CWD * GP], s_lt[CWD * GP];
    __shared__ uint32_t s_cnt[2];
    const int t = threadIdx.x, lane = t & 63, wid = __builtin_amdgcn_readfirstlane(t >> 6);
    const int chunk = blockIdx.x % chunks, group = blockIdx.x / chunks;
    const uint32_t s0 = (uint32_t)group * GS;
    const int u0 = chunk * 32 * CWD, cur = i & 1;
    const int slot = t % GS, p0 = t / GS;
    constexpr int PT = WT / GS;
    const uint32_t s = s0 + (uint32_t)slot;
    const Tile<W> tile{s_rows, s_lc, s_phi};
    typename Tile<W>::Slot sl;
    const Level L = c.st[i];
    const uint32_t deg = sgpr(c.prep->deg);
    sl.load(c, i, s0, u0);
    const uint32_t ped = c.ped[cur][s];
    tile.stage_rows(c, i, u0);
    for (int k = p0; k < W; k += PT) s_phi[k * GP + slot] = k < c.w2 ? c.sets[(size_t)k * c.Kp + s] : 0u;
    for (int x = t; x < CWD * GP; x += WT) {
        s_le[x] = 0u;
        s_lt[x] = 0u;
    }
    if (t < 2) s_cnt[t] = 0u;
    const uint32_t B = sgpr(L.B);
    if (s0 >= B) return;
    const uint32_t T = sgpr(threshold(c, i, L, deg, s_bin));   // (waits for the staging too)
    if (T != NONE) {
        // bytes: 0 below T, 1 at T, more above
        const float shift = (float)((int)(deg * (uint32_t)c.c.edel) - (int)T + 1);
        const int ls = wid * 16 + (lane & 15), q = lane >> 4;
        tile.score(c, sl, t, s0, B, u0, shift, [&](int k, const v4f &y) {
            uint32_t w = 0u;
#pragma unroll
            for (int r = 0; r < 4; ++r) w = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f(y[r], 0.f, (float)XCAP), r, w);
            const uint32_t fle = (0x81818181u - w) & HI;
            if (fle) {
                const uint32_t flt = (0x80808080u - w) & HI;
                const int at2 = (k >> 1) * GP + ls, sh = 16 * (k & 1) + 4 * q;
                atomicOr(&s_le[at2], (__builtin_amdgcn_udot4(fle, 0x08040201u, 0u, false) >> 7) << sh);
                if (flt) atomicOr(&s_lt[at2], (__builtin_amdgcn_udot4(flt, 0x08040201u, 0u, false) >> 7) << sh);
            }
        });
        __syncthreads();
    }
    // the masks of the chunk's words (every free vertex when all survive), and
    // the deletion with the first chunk
    uint32_t nl = 0u, ne = 0u;
    for (int k = p0; k < CWD; k += PT) {
        const int kw = (u0 >> 5) + k;
        if (kw >= c.w2 || s >= B) continue;
        uint32_t a = s_le[k * GP + slot], b = s_lt[k * GP + slot];
        if (T == NONE) a = b = ~c.img[cur][(size_t)kw * c.Kp + s] & below(c.n2, kw);
        c.le[(size_t)kw * c.Kp + s] = a;
        c.lt[(size_t)kw * c.Kp + s] = b;
        nl += (uint32_t)__popc(b);
        ne += (uint32_t)__popc(a & ~b);
    }
    if (chunk == 0 && p0 == 0 && s < B) {
        const uint32_t d = ped + (uint32_t)c.c.vdel + deg * (uint32_t)c.c.edel;
        const uint32_t a = d <= T ? 1u : 0u, b = d < T ? 1u : 0u;
        c.le[(size_t)c.w2 * c.Kp + s] = a;
        c.lt[(size_t)c.w2 * c.Kp + s] = b;
        nl += b;
        ne += a - b;
    }
    nl = wave_sum(nl);
    ne = wave_sum(ne);
    if (lane == 0) {
        atomicAdd(&s_cnt[0], nl);
        atomicAdd(&s_cnt[1], ne);
    }
    __syncthreads();
    if (t < 2 && s_cnt[t]) atomicAdd(&c.cnt[t * groups + group], s_cnt[t]);
}

// New slot s: parent p with v_i -> u (u >= n2: deleted), by the four threads
// `part` of one quarter wave.
__device__ __forceinline__ void write_slot(const Ctx &c, int i, uint32_t s, uint32_t p, int u, uint32_t deg, int b0, int part) {
    constexpr int PT = 4;
    const int cur = i & 1, nxt = cur ^ 1, nblk = i / BL, r8 = i % BL;
    const bool sub = u < c.n2, full = r8 == BL - 1;
    uint32_t kept = 0u, in = 0u;
    for (int k = part; k < c.w2; k += PT) {
        uint32_t im = c.img[cur][(size_t)k * c.Kp + p];
        if (sub) {
            const uint32_t row = c.a2[(size_t)u * c.w2 + k];
            kept += (uint32_t)__popc(row & c.sets[(size_t)k * c.Kp + p]);
            in += (uint32_t)__popc(row & im);
            if (k == (u >> 5)) im |= 1u << (u & 31);
        }
        c.img[nxt][(size_t)k * c.Kp + s] = im;
    }
#pragma unroll
    for (int o = 1; o < PT; o <<= 1) {
        kept += (uint32_t)__shfl_xor((int)kept, o);
        in += (uint32_t)__shfl_xor((int)in, o);
    }
    for (int r = part; r <= r8; r += PT) {
        const uint16_t x = r == r8 ? (sub ? (uint16_t)u : (uint16_t)DEL16) : c.cur[cur][(size_t)r * c.Kp + p];
        if (full) c.phi[(size_t)(i - r8 + r) * c.Kp + s] = x;
        else c.cur[nxt][(size_t)r * c.Kp + s] = x;
    }
    for (int b = b0 + part; b < nblk; b += PT) c.anc[nxt][(size_t)b * c.Kp + s] = c.anc[cur][(size_t)b * c.Kp + p];
    if (part == 0) {
        uint32_t d = c.ped[cur][p] + (uint32_t)c.c.edel * (deg - kept);
        if (sub) d += (c.l2[u] != c.l1[i] ? (uint32_t)c.c.vsub : 0u) + (uint32_t)c.c.eins * (in - kept);
        else d += (uint32_t)c.c.vdel;
        c.ped[nxt][s] = d;
        c.nsub[nxt][s] = c.nsub[cur][p] + (sub ? 1u : 0u);
        if (full) c.anc[nxt][(size_t)nblk * c.Kp + s] = s;
    }
}

// ------------------------------------------------------------------ update
// The next level's Prep, by one workgroup: whether the oldest block has one
// ancestor left in the whole beam, the common images of v = i + 1's earlier
// neighbours, and the window's neighbours.
template <int UT>
__device__ __forceinline__ void prepare(const Ctx &c, int i) {
    __shared__ uint32_t s_pc[MAXN / 32], s_same;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6, v = i + 1;
    int b0 = (int)c.st[i].b0;
    const uint32_t B = c.st[i].B;
    const uint32_t *R = c.a1 + (size_t)min(v, c.n1 - 1) * c.w1;
    const bool look = b0 < i / BL && B <= kCommonMost;
    if (t == 0) s_same = 1u;
    if (t < MAXN / 32) s_pc[t] = 0u;
    __syncthreads();
    if (look) {
        const uint32_t *a = c.anc[i & 1] + (size_t)b0 * c.Kp;
        const uint32_t a0 = a[0];
        uint32_t differ = 0u;
#pragma unroll 4
        for (uint32_t s = t; s < B; s += UT) differ |= a[s] ^ a0;
        if (differ) s_same = 0u;
    }
    __syncthreads();
    if (look && s_same != 0u) {
        const int j = BL * b0 + t;
        if (t < BL) c.com[j] = c.phi[(size_t)j * c.Kp + c.anc[i & 1][(size_t)b0 * c.Kp]];
        ++b0;
    }
    if (t == 0) c.st[v].b0 = (uint32_t)b0;
    __syncthreads();
    if (v >= c.n1) return;
    const int c0 = BL * b0, nblk = v / BL;
    for (int j = t; j < c0; j += UT) {
        if (!((R[j >> 5] >> (j & 31)) & 1u)) continue;
        const uint32_t x = c.com[j];
        if (x != DEL16) atomicOr(&s_pc[x >> 5], 1u << (x & 31));
    }
    if (wid == UT / 64 - 1) {
        int base = 0;
#pragma unroll 1
        for (int part = 0; part < 2; ++part) {
            const int jl = part ? BL * nblk : c0, jh = part ? v : BL * nblk;
            for (int kw = jl >> 5; kw * 32 < jh; ++kw) {
                const uint32_t bits = R[kw] & below(jh, kw) & ~below(jl, kw);
                const bool mine = lane < 32 && ((bits >> lane) & 1u);
                const unsigned long long m = __ballot(mine);
                if (mine) c.prep->nbr[base + (int)__builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)] = (uint16_t)(kw * 32 + lane);
                base += __popcll(m);
            }
            if (lane == 0) (part ? c.prep->nw : c.prep->nwb) = (uint32_t)base;
        }
        const uint32_t deg = degree(c, v);
        if (lane == 0) c.prep->deg = deg;
    }
    __syncthreads();
    if (t < MAXN / 32) c.prep->pc[t] = s_pc[t];
}

// The far histogram back to zero, after a level that used it: each
// workgroup (but the last) its share of the groups that hold anything.
template <int UT>
__device__ __forceinline__ void clear_far(const Ctx &c) {
    __shared__ uint32_t s_used[FC];
    for (int x = threadIdx.x; x < FC; x += UT) s_used[x] = c.farc[x];
    __syncthreads();
    for (uint32_t g = blockIdx.x; g < (uint32_t)FC; g += gridDim.x - 1) {
        if (s_used[g] == 0u) continue;   // (only its owner clears a sum)
        for (int x = threadIdx.x; x < HB; x += UT) c.far[(size_t)g * HB + x] = 0u;
        if (threadIdx.x == 0) c.farc[g] = 0u;
    }
}

// The last workgroup prepares the next level; deg comes with the launch's own
// reading of it, since Prep is being rewritten.
// UT threads: 1024 while there are few groups, since the survivors gather
// under few parents and a workgroup writes UT / 4 slots at a time.
template <int W, int UT>
__global__ __launch_bounds__(UT) void wm_update(Ctx c, int i, int groups) {
    __shared__ uint32_t s_tmp[4][UT / 64];
    constexpr int NWU = UT / 64, PT = UT / GS;
    constexpr int CWM = (W + 1 + PT - 1) / PT;   // mask words of a thread
    const int t = threadIdx.x, us = t / PT, part = t % PT, wid = t >> 6, lane = t & 63;
    if (blockIdx.x == gridDim.x - 1) {
        prepare<UT>(c, i);
        return;
    }
    const uint32_t s0 = (uint32_t)blockIdx.x * GS, s = s0 + (uint32_t)us;
    const Level L = c.st[i];
    const uint32_t Bn0 = c.st[i + 1].B;
    uint32_t ml[CWM], me[CWM], nl = 0u, ne = 0u;
#pragma unroll
    for (int k = 0; k < CWM; ++k) {
        const int kw = part * CWM + k;
        ml[k] = kw <= c.w2 ? c.lt[(size_t)kw * c.Kp + s] : 0u;
        me[k] = kw <= c.w2 ? c.le[(size_t)kw * c.Kp + s] : 0u;
    }
    // counts of the groups before this one
    uint32_t a = 0u, e = 0u;
    for (int g = t; g < (int)blockIdx.x; g += UT) {
        a += c.cnt[g];
        e += c.cnt[groups + g];
    }
    for (uint32_t b = blockIdx.x * UT + t; b < (uint32_t)(HC * HB); b += (gridDim.x - 1) * UT) c.hist[b] = 0u;
    const uint32_t deg = sgpr(degree(c, i));
    const uint32_t B = sgpr(L.B), quota = sgpr(L.quota), Bn = sgpr(Bn0);
    const int b0 = (int)sgpr(L.b0);
    if (sgpr(L.far)) clear_far<UT>(c);
    if (s0 >= B) return;
#pragma unroll
    for (int k = 0; k < CWM; ++k) {
        ml[k] = s < B ? ml[k] : 0u;
        me[k] = s < B ? me[k] & ~ml[k] : 0u;
        nl += (uint32_t)__popc(ml[k]);
        ne += (uint32_t)__popc(me[k]);
    }
    // one pass for the sums before the group and the scans inside it
    uint32_t pl = (uint32_t)wave_excl_scan((int)nl), pe = (uint32_t)wave_excl_scan((int)ne);
    a = wave_sum(a);
    e = wave_sum(e);
    if (lane == 63) {
        s_tmp[0][wid] = pl + nl;
        s_tmp[1][wid] = pe + ne;
        s_tmp[2][wid] = a;
        s_tmp[3][wid] = e;
    }
    __syncthreads();
    uint32_t LT = 0u, EQ = 0u, tl = 0u, te = 0u;
#pragma unroll
    for (int k = 0; k < NWU; ++k) {
        const uint32_t x = s_tmp[0][k], y = s_tmp[1][k];
        pl += k < wid ? x : 0u;
        pe += k < wid ? y : 0u;
        tl += x;
        te += y;
        LT += s_tmp[2][k];
        EQ += s_tmp[3][k];
    }
    const uint32_t out0 = LT + min(EQ, quota), out1 = LT + tl + min(EQ + te, quota);
    const uint32_t eqb = min(EQ + pe, quota);   // ties kept before this thread's words
    uint32_t keq = min(quota - eqb, ne);        // ... and among them
    uint32_t pos = LT + pl + eqb;
#pragma unroll
    for (int k = 0; k < CWM; ++k) {
        const int kw = part * CWM + k;
        uint32_t m = keq > 0u ? ml[k] | me[k] : ml[k];
        while (m) {
            const uint32_t bit = m & (0u - m);
            m ^= bit;
            if (me[k] & bit) {
                if (keq == 0u) continue;
                --keq;
            }
            const uint32_t u = kw < c.w2 ? (uint32_t)(32 * kw + __builtin_ctz(bit)) : (uint32_t)c.n2;
            if (pos < Bn) c.rec[pos] = (s << UBITS) | u;
            ++pos;
        }
    }
    __syncthreads();
    for (uint32_t x = out0 + (uint32_t)(t / 4); x < min(out1, Bn); x += UT / 4) {
        const uint32_t r = c.rec[x];
        write_slot(c, i, x, r >> UBITS, (int)(r & ((1u << UBITS) - 1u)), deg, b0, t & 3);
    }
}

// Edges of g2 inside slot s's Img, twice: the share of thread `part` of `parts`
// (the image's words in turn).
__device__ __forceinline__ uint32_t inside2(const Ctx &c, int cur, uint32_t s, int part, int parts) {
    uint32_t e = 0u;
    for (int kw = part; kw < c.w2; kw += parts) {
        uint32_t m = c.img[cur][(size_t)kw * c.Kp + s];
        while (m) {
            const int u = 32 * kw + __builtin_ctz(m);
            m &= m - 1u;
            for (int k = 0; k < c.w2; ++k)
                e += (uint32_t)__popc(c.a2[(size_t)u * c.w2 + k] & c.img[cur][(size_t)k * c.Kp + s]);
        }
    }
    return e;
}

// Sum over the four threads of a slot.
__device__ __forceinline__ uint32_t quad_sum(uint32_t v) {
    v += (uint32_t)__shfl_xor((int)v, 1);
    v += (uint32_t)__shfl_xor((int)v, 2);
    return v;
}

__device__ __forceinline__ void block_least(unsigned long long key, unsigned long long *out) {
    __shared__ unsigned long long s_key[NWV];
    key = wave_min64(key);
    if ((threadIdx.x & 63) == 0) s_key[threadIdx.x >> 6] = key;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 1; k < NWV; ++k) key = s_key[k] < key ? s_key[k] : key;
        *out = key;
    }
}

// ------------------------------------------------------------------ complete-then-minimum
// Last level with that option: every child's total (Sec. 4.4.1), CP threads a
// slot; the least (total, generation order) of each workgroup.  CP: four keep the
// slots' words coalesced (100 x 100 vertices, K = 200,000: 7.95 ms the search,
// 8.41 with 16); with few slots they would leave most of the device idle (5 x 1000
// at K = 2000: 1.48 ms the search so, 0.52 with 16 and without the second sum).
constexpr uint32_t kCompleteFew = 1u << 14;   // slots that 16 threads each serve
template <int CP>
__global__ __launch_bounds__(WT) void wm_complete(Ctx c, int i) {
    const int t = threadIdx.x, us = t / CP, part = t % CP, cur = i & 1;
    const uint32_t B = sgpr(c.st[i].B), s = (uint32_t)blockIdx.x * (WT / CP) + (uint32_t)us;
    const uint32_t deg = sgpr(degree(c, i));
    unsigned long long key = ~0ull;
    uint32_t children = 0u;
    if (s < B) {
        const uint32_t e0 = parts_sum<CP>(inside2(c, cur, s, part, CP)) / 2u, left = (uint32_t)c.n2 - c.nsub[cur][s];
        const uint32_t ped = c.ped[cur][s], eins = (uint32_t)c.c.eins, edel = (uint32_t)c.c.edel;
        const int lab1 = c.l1[i];
        for (int u = part; u <= c.n2; u += CP) {
            uint32_t total = ped + deg * edel + (uint32_t)c.c.vins * left + eins * ((uint32_t)c.m2 - e0);   // (the deletion's)
            if (u < c.n2) {
                if ((c.img[cur][(size_t)(u >> 5) * c.Kp + s] >> (u & 31)) & 1u) continue;
                // its edges into Img, inserted or kept now, are not inserted at the end
                uint32_t kept = 0u;
                for (int k = 0; k < c.w2; ++k) kept += (uint32_t)__popc(c.a2[(size_t)u * c.w2 + k] & c.sets[(size_t)k * c.Kp + s]);
                total += (c.l2[u] != lab1 ? (uint32_t)c.c.vsub : 0u) - (uint32_t)c.c.vins - (edel + eins) * kept;
            } else {
                total += (uint32_t)c.c.vdel;
            }
            const unsigned long long k = ((unsigned long long)total << 32) | ((s << UBITS) | (uint32_t)u);
            key = k < key ? k : key;
        }
        children = part == 0 ? left + 1u : 0u;
    }
    children = wave_sum(children);
    if ((t & 63) == 0) atomicAdd(c.ce, (unsigned long long)children);
    block_least(key, c.best + blockIdx.x);
}

__device__ __forceinline__ unsigned long long least_key(const Ctx &c, int groups) {
    __shared__ unsigned long long s_least;
    unsigned long long key = ~0ull;
    for (int b = threadIdx.x; b < groups; b += WT) key = c.best[b] < key ? c.best[b] : key;
    block_least(key, &s_least);
    __syncthreads();
    return s_least;
}

// The winner becomes the only survivor.
__global__ __launch_bounds__(WT) void wm_pick(Ctx c, int i, int groups) {
    const uint32_t r = (uint32_t)(least_key(c, groups) & 0xffffffffull);
    const uint32_t deg = sgpr(degree(c, i));
    const int b0 = (int)c.st[i].b0;
    if (threadIdx.x < 4) write_slot(c, i, 0u, r >> UBITS, (int)(r & ((1u << UBITS) - 1u)), deg, b0, threadIdx.x);
    if (threadIdx.x == 0) {
        c.st[i + 1].B = 1u;
        c.st[i + 1].b0 = (uint32_t)b0;
    }
}

// ------------------------------------------------------------------ final
__global__ __launch_bounds__(WT) void wm_final_keys(Ctx c) {
    const int t = threadIdx.x, us = t / 4, part = t % 4, cur = c.n1 & 1;
    const uint32_t B = sgpr(c.st[c.n1].B), s = (uint32_t)blockIdx.x * GS + (uint32_t)us, at = min(s, B - 1u);
    const uint32_t e = quad_sum(inside2(c, cur, at, part, 4)) / 2u;
    unsigned long long key = ~0ull;
    if (s < B)
        key = ((unsigned long long)(c.ped[cur][s] + (uint32_t)c.c.vins * ((uint32_t)c.n2 - c.nsub[cur][s]) +
                                    (uint32_t)c.c.eins * ((uint32_t)c.m2 - e)) << 32) | s;
    block_least(key, c.best + blockIdx.x);
}

__global__ __launch_bounds__(WT) void wm_final_map(Ctx c, int groups) {
    const unsigned long long best = least_key(c, groups);
    const uint32_t slot = (uint32_t)(best & 0xffffffffull);
    const int cur = c.n1 & 1, nblk = c.n1 / BL, b0 = (int)c.st[c.n1].b0;
    if (threadIdx.x == 0) {
        *c.out_dist = (int32_t)(best >> 32);
        if (c.out_cand) *c.out_cand = (int64_t)*c.ce;
    }
    for (int j = threadIdx.x; j < c.n1; j += WT) {
        const int b = j / BL;
        const uint32_t x = b < b0 ? c.com[j]
                                  : (b < nblk ? c.phi[(size_t)j * c.Kp + c.anc[cur][(size_t)b * c.Kp + slot]]
                                              : c.cur[cur][(size_t)(j % BL) * c.Kp + slot]);
        c.out_map[j] = x == DEL16 ? -1 : (int32_t)x;
    }
}

// ------------------------------------------------------------------ host side

struct Layout {
    size_t ped[2], nsub[2], img[2], cur[2], anc[2], phi, com, sets, le, lt, cnt, rec, hist, st, prep, ce, best, far, farc, total;
};

uint32_t slot_stride(int K) { return (uint32_t)((K + GS - 1) / GS) * GS; }

Layout layout(int n1, int w2, uint32_t Kp) {
    Layout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    const size_t groups = Kp / GS, blocks = (size_t)(n1 + BL - 1) / BL;
    for (int k = 0; k < 2; ++k) {
        L.ped[k] = take((size_t)Kp * 4);
        L.nsub[k] = take((size_t)Kp * 4);
        L.img[k] = take((size_t)w2 * Kp * 4);
        L.cur[k] = take((size_t)BL * Kp * 2);
        L.anc[k] = take(blocks * Kp * 4);
    }
    L.phi = take((size_t)n1 * Kp * 2);
    L.com = take((size_t)n1 * 2);
    L.sets = take((size_t)w2 * Kp * 4);
    L.le = take((size_t)(w2 + 1) * Kp * 4);
    L.lt = take((size_t)(w2 + 1) * Kp * 4);
    L.cnt = take(2 * groups * 4);
    L.rec = take((size_t)Kp * 4);
    L.hist = take((size_t)HC * HB * 4);
    L.st = take((size_t)(n1 + 1) * sizeof(Level));
    L.prep = take(sizeof(Prep));
    L.ce = take(8);
    L.best = take(std::max<size_t>(groups, kCompleteFew / (WT / 16)) * 8);
    // (last: few levels touch them, and between the others they would put what
    // every level touches on further pages, 0.4 us of each of its launches)
    L.farc = take((size_t)FC * 4);
    L.far = take((size_t)FAR * 4);
    L.total = off;
    return L;
}

template <int W>
hipError_t levels(const Ctx &c, bool last_complete, hipStream_t stream) {
    // (up to 16 MB to clear: 64 values a thread)
    const uint32_t far = c.pedmax >= (uint32_t)(HB - 1) ? c.pedmax + 1u : 0u;
    hipLaunchKernelGGL(wm_init, dim3(std::max(32u, far / (64 * WT))), dim3(WT), 0, stream, c);
    const int chunks = (c.n2 + 32 * CWD - 1) / (32 * CWD), groups = (int)(c.Kp / GS);
    uint64_t bound = 1;   // parents at level i are at most min(K, (n2 + 1)^i)
    for (int i = 0; i < c.n1; ++i) {
        const int g = (int)((bound + GS - 1) / GS);
        const bool last = last_complete && i == c.n1 - 1;
        hipLaunchKernelGGL(wm_expand<W>, dim3(last ? g : g * chunks), dim3(WT), 0, stream, c, i, last ? 1 : chunks, groups, last ? 0 : 1);
        if (last) {
            const int gc = bound <= kCompleteFew ? (int)((bound + WT / 16 - 1) / (WT / 16)) : g;
            if (bound <= kCompleteFew) hipLaunchKernelGGL(wm_complete<16>, dim3(gc), dim3(WT), 0, stream, c, i);
            else hipLaunchKernelGGL(wm_complete<WT / GS>, dim3(gc), dim3(WT), 0, stream, c, i);
            hipLaunchKernelGGL(wm_pick, dim3(1), dim3(WT), 0, stream, c, i, gc);
            bound = 1;
            break;
        }
        hipLaunchKernelGGL(wm_mark<W>, dim3(g * chunks), dim3(WT), 0, stream, c, i, chunks, groups);
        if (g <= 512)
            hipLaunchKernelGGL((wm_update<W, 1024>), dim3(g + 1), dim3(1024), 0, stream, c, i, groups);
        else
            hipLaunchKernelGGL((wm_update<W, 256>), dim3(g + 1), dim3(256), 0, stream, c, i, groups);
        const uint64_t grown = bound * (uint64_t)(c.n2 + 1);
        bound = grown < c.K ? grown : c.K;
    }
    const int g = (int)((bound + GS - 1) / GS);
    hipLaunchKernelGGL(wm_final_keys, dim3(g), dim3(WT), 0, stream, c);
    hipLaunchKernelGGL(wm_final_map, dim3(1), dim3(WT), 0, stream, c, g);
    return hipGetLastError();
}

}  // namespace

size_t widem_workspace_bytes(int n1, int w2, int K) { return layout(n1, w2, slot_stride(K)).total; }

bool widem_takes(const GraphRec &g1, const GraphRec &g2, int planes, Costs c, int K, uint64_t pedmax) {
    if (planes != 0 || g2.n <= kWide1MaxN2 || pedmax >= (uint64_t)kFastBound) return false;
    // the largest beams on small targets: here a level costs about 20 ns per 64
    // slots whatever the target (workgroups of few children), while the candidate
    // matrix's share goes with n2 and its mapping copies with n1.  Equal, measured,
    // at K = 235,000 for 33 x 33 vertices (n1 x n2), 290,000 for 100 x 33, 520,000
    // for 200 x 33, 330,000 for 48 x 48, 400,000 for 56 x 56; at two million slots
    // 18.3 against 10.7 ms (33 x 33), 23.1 against 15.7 (40 x 40); from 64 target
    // vertices on here is at most 4 % behind and up to twice as fast.
    if (g2.n <= 60 && (int64_t)K * (7400 - 75 * g2.n - 14 * std::min(g1.n, 240)) > 1000000000) return false;
    // the largest increment of a level: while the bins hold it, the least child
    // (the least parent's) lies among them, so a level's bins start at its least
    // parent PED exactly.  Children past the bins go to the far histogram.
    const int64_t inc = (int64_t)c.vsub + (int64_t)c.vdel + (int64_t)std::max(c.edel, c.esub) * std::min(g1.n - 1, g1.m) +
                        (int64_t)c.eins * std::min(g1.n, g2.n);
    SlotCodes s;
    return inc <= 3 * HB / 4 && slot_codes(c, false, &s);
}

hipError_t launch_widem(const DbView &src, const DbView &dst, const GraphRec &g1, const GraphRec &g2, Costs costs, int K,
                        int last_complete, uint32_t pedmax, void *ws, size_t ws_bytes, int32_t *dist, int32_t *map,
                        int64_t *cand, hipStream_t stream) {
    const uint32_t Kp = slot_stride(K);
    const Layout L = layout(g1.n, g2.w, Kp);
    SlotCodes s;
    if (K < 1 || K > kWideMaxK || L.total > ws_bytes || g1.n > MAXN || g2.n > MAXN || pedmax >= FAR ||
        !slot_codes(costs, false, &s))
        return hipErrorInvalidValue;
    char *base = static_cast<char *>(ws);
    Ctx c{};
    c.a1 = src.adj + g1.adj;
    c.l1 = src.vlab + g1.vlab;
    c.a2 = dst.adj + g2.adj;
    c.l2 = dst.vlab + g2.vlab;
    c.n1 = g1.n;
    c.w1 = g1.w;
    c.n2 = g2.n;
    c.w2 = g2.w;
    c.m2 = g2.m;
    c.c = costs;
    c.pedmax = pedmax;
    c.code_img = s.img;
    c.code_phi = s.phi;
    c.unit_exp = s.unit_exp;
    c.K = (uint32_t)K;
    c.Kp = Kp;
    for (int k = 0; k < 2; ++k) {
        c.ped[k] = reinterpret_cast<uint32_t *>(base + L.ped[k]);
        c.nsub[k] = reinterpret_cast<uint32_t *>(base + L.nsub[k]);
        c.img[k] = reinterpret_cast<uint32_t *>(base + L.img[k]);
        c.cur[k] = reinterpret_cast<uint16_t *>(base + L.cur[k]);
        c.anc[k] = reinterpret_cast<uint32_t *>(base + L.anc[k]);
    }
    c.phi = reinterpret_cast<uint16_t *>(base + L.phi);
    c.com = reinterpret_cast<uint16_t *>(base + L.com);
    c.sets = reinterpret_cast<uint32_t *>(base + L.sets);
    c.le = reinterpret_cast<uint32_t *>(base + L.le);
    c.lt = reinterpret_cast<uint32_t *>(base + L.lt);
    c.cnt = reinterpret_cast<uint32_t *>(base + L.cnt);
    c.rec = reinterpret_cast<uint32_t *>(base + L.rec);
    c.hist = reinterpret_cast<uint32_t *>(base + L.hist);
    c.far = reinterpret_cast<uint32_t *>(base + L.far);
    c.farc = reinterpret_cast<uint32_t *>(base + L.farc);
    c.st = reinterpret_cast<Level *>(base + L.st);
    c.prep = reinterpret_cast<Prep *>(base + L.prep);
    c.ce = reinterpret_cast<unsigned long long *>(base + L.ce);
    c.best = reinterpret_cast<unsigned long long *>(base + L.best);
    c.out_dist = dist;
    c.out_map = map;
    c.out_cand = cand;
    const bool lc = last_complete != 0;
    if (g2.w <= 4) return levels<4>(c, lc, stream);
    if (g2.w <= 8) return levels<8>(c, lc, stream);
    if (g2.w <= 16) return levels<16>(c, lc, stream);
    return levels<32>(c, lc, stream);
}

}  // namespace gedk
