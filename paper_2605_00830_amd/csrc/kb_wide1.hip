// kb_wide1.hip -- the whole-device search of one pair (kb_wide.hip) for targets
// of up to 32 vertices whose PEDs fit the histogram (below 4096): the paper's
// runtime-versus-K experiment, two 20-vertex graphs at K up to 1.2 million.
//
// Here a parent's whole state is a handful of words (PED, Img, Phi and its
// label planes), so a child costs fewer instructions to score again than its
// PED costs to store and load: no candidate matrix exists.  Three kernels per
// level:
//   count   finds the threshold T from the level's histogram (every workgroup
//           by itself), marks each parent's children at most T and below T in
//           two masks, and counts them per workgroup.
//   emit    every workgroup adds up the counts before its own and writes its
//           survivors' records in generation order (parents in beam order,
//           vertex ascending, the deletion last, ties at T while the quota
//           lasts).
//   update  a thread per new slot (so a parent of many survivors costs no more
//           than others): its words and mapping, the next level's Phi, gathered
//           from the mapping as it is copied (a byte per vertex, four to a word,
//           0xff = deleted), and, while all that is in registers, the next
//           level's histogram.  The values of a level are few (some tens), so
//           lanes would meet on the same LDS counter: each adds in its own
//           column of counters (as many columns as the range leaves room for).
// Workgroup b of count and emit owns the same contiguous range of parent tiles,
// so the beam stays in generation order.
//
// Two 20-vertex graphs at K = 1.2 million (MI355X): 2,325 us with the candidate
// matrix of kb_wide.hip, 975 us so; a level of 1.2 million parents is 14 us of
// count (13 instructions a child), 12 us of emit and 23 us of update (it moves
// about 75 MB).  Not kept: emit and update in one kernel, a workgroup writing
// its own parents' survivors (53 us for the two: survivors gather under few
// parents).
#include <algorithm>

#include "ged_internal.h"
#include "wave_common.h"

namespace gedk {
namespace {

using namespace wv;

constexpr int WT = 256;
constexpr int NWV = WT / 64;
constexpr int HB = kWide1Bound;       // histogram bins: every PED of the search is below
constexpr int HWORDS = 4096;          // LDS counters of a workgroup (eight workgroups fit a CU)
constexpr int MAXG = 2048;            // workgroups of a level
// Copies of the level's histogram: atomics on one address are serialised at
// the memory side, about 10 ns each, and 2048 workgroups add to every bin of
// the range (update 33.5 us a level with one copy, 23 with 16).
constexpr int HC = 16;
constexpr uint32_t NONE = 0xffffffffu;
constexpr uint32_t DEL8 = 0xffu;
static_assert(kWide1MaxN2 <= 32 && (uint32_t)kWide1MaxN2 < DEL8, "an image: a bit of a word, a byte");
static_assert((int64_t)kWideMaxK << 6 <= (int64_t)1 << 32, "record");

struct Level {
    uint32_t B;      // parents
    uint32_t m0;     // least parent PED
    uint32_t mmax;   // largest
    uint32_t T;      // threshold (NONE: every child survives)
    uint32_t quota;  // children equal to T that survive
    uint32_t pad[3];
};

struct Ctx {
    const uint32_t *a1;   // g1 rows, then its label planes
    const int32_t *l1;
    const uint32_t *a2;   // g2 rows (one word each), then its label planes
    const int32_t *l2;
    int n1, w1, n2, m2, planes;
    Costs c;
    uint32_t pedmax;
    uint32_t K, Kp;       // beam width, slot stride
    uint32_t *ped[2], *img[2];
    uint32_t *sets[2];    // [1 + planes][Kp] Phi and its label planes of the coming level
    uint32_t *phi[2];     // [ceil(n1 / 4)][Kp] images, a byte each
    uint32_t *blk;        // [2][MAXG] children below T, equal to T of each workgroup
    uint32_t *hist[2];    // [HC][HB] by level parity
    uint32_t *rec;        // [Kp] survivor records
    uint32_t *lem, *ltm;  // [Kp] substitutions at most T, below T of each parent
    Level *st;
    unsigned long long *ce;
    unsigned long long *best;   // [MAXG] least key of each workgroup
    int32_t *out_dist, *out_map;
    int64_t *out_cand;
};

__device__ __forceinline__ uint32_t sgpr(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }

__device__ __forceinline__ uint32_t block_sum(uint32_t v, uint32_t *s_tmp) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) s_tmp[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t r = 0u;
#pragma unroll
    for (int k = 0; k < NWV; ++k) r += s_tmp[k];
    __syncthreads();
    return r;
}

__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *s_tmp, uint32_t *total) {
    const uint32_t x = (uint32_t)wave_excl_scan((int)v);
    if ((threadIdx.x & 63) == 63) s_tmp[threadIdx.x >> 6] = x + v;
    __syncthreads();
    uint32_t pre = 0u, tot = 0u;
#pragma unroll
    for (int k = 0; k < NWV; ++k) {
        const uint32_t t = s_tmp[k];
        pre += k < (int)(threadIdx.x >> 6) ? t : 0u;
        tot += t;
    }
    __syncthreads();
    *total = tot;
    return pre + x;
}

// Word k of g1 vertex v's row: its neighbours below `lim`.
__device__ __forceinline__ uint32_t earlier_word(const Ctx &c, int v, int k, int lim) {
    const uint32_t r = c.a1[(size_t)v * c.w1 + k];
    const int lo = 32 * k;
    if (lim >= lo + 32) return r;
    if (lim <= lo) return 0u;
    return r & ((1u << (lim - lo)) - 1u);
}

// What scoring a level's children takes: lane u of every wave holds target
// vertex u's row and label planes, read back as scalars at constant lanes (the
// child loops are unrolled, so they stay in scalar registers over a workgroup's
// tiles; scalar loads inside the loops would wait for the LDS counters too),
// the vertices whose label differs from v_i's as a mask, and the degree of
// v_i into earlier vertices.
template <int PL>
struct Score {
    static constexpr int PLA = PL > 0 ? PL : 1;
    uint32_t rows, planes[PLA];
    uint32_t differ, valid, vsub, deg;
    __device__ __forceinline__ void load(const Ctx &c, int i) {
        const int u = threadIdx.x & 63;
        const bool in = u < c.n2;
        rows = in ? c.a2[u] : 0u;
#pragma unroll
        for (int b = 0; b < PLA; ++b) planes[b] = (PL > 0 && in && b < c.planes) ? c.a2[(size_t)(1 + b) * c.n2 + u] : 0u;
        differ = (uint32_t)__ballot(in && c.l2[u] != c.l1[i]);
        valid = c.n2 >= 32 ? 0xffffffffu : (1u << c.n2) - 1u;
        vsub = (uint32_t)c.c.vsub;
        deg = 0u;
        for (int k = 0; k < c.w1; ++k) deg += (uint32_t)__popc(earlier_word(c, i, k, i));
        deg = sgpr(deg);
    }
    __device__ __forceinline__ uint32_t row(int u) const { return (uint32_t)__builtin_amdgcn_readlane((int)rows, u); }
    __device__ __forceinline__ uint32_t lc(int u) const { return ((differ >> u) & 1u) ? vsub : 0u; }
    __device__ __forceinline__ uint32_t plane(int b, int u) const {
        return PL > 0 ? (uint32_t)__builtin_amdgcn_readlane((int)planes[b], u) : 0u;
    }
};

// f(u) for every target vertex, and a few past the last (rows of 0), highest
// first, unrolled.
template <class F>
__device__ __forceinline__ void each_target(int n2, F f) {
#pragma unroll
    for (int u0 = 28; u0 >= 0; u0 -= 4) {
        if (u0 < n2) {
#pragma unroll
            for (int k = 3; k >= 0; --k) f(u0 + k);
        }
    }
}

// A parent's words.
template <int PL>
struct Parent {
    static constexpr int PLA = PL > 0 ? PL : 1;
    uint32_t ped, img, ph, pb[PLA];
    __device__ __forceinline__ void load(const Ctx &c, int cur, uint32_t p) {
        ped = c.ped[cur][p];
        img = c.img[cur][p];
        ph = c.sets[cur][p];
#pragma unroll
        for (int b = 0; b < PLA; ++b) pb[b] = (PL > 0 && b < c.planes) ? c.sets[cur][(size_t)(1 + b) * c.Kp + p] : 0u;
    }
    // base + eins |(Img \ Phi) & row| - edel |Phi & row| + esub |Phi & row & relabelled|:
    // the PED of the child that substitutes this row's vertex, but for the label
    // cost (all costs below 2^24: a PED stays below 4096)
    __device__ __forceinline__ uint32_t child(uint32_t base, uint32_t row, const uint32_t (&pl)[PLA], uint32_t eins,
                                              uint32_t nedel, uint32_t esub) const {
        uint32_t d = msub_cost<true>((uint32_t)__popc(ph & row), nedel,
                                     mad_cost<true>((uint32_t)__popc((img & ~ph) & row), eins, base));
        if (PL > 0) {
            uint32_t diff = 0u;
#pragma unroll
            for (int b = 0; b < PLA; ++b) diff |= pb[b] ^ pl[b];
            d = mad_cost<true>((uint32_t)__popc(ph & row & diff), esub, d);
        }
        return d;
    }
    // ... target vertex u (the same in every lane)
    __device__ __forceinline__ uint32_t child_of(uint32_t base, const Score<PL> &sc, int u, uint32_t eins,
                                                 uint32_t nedel, uint32_t esub) const {
        uint32_t pl[PLA];
#pragma unroll
        for (int b = 0; b < PLA; ++b) pl[b] = sc.plane(b, u);
        return child(base, sc.row(u), pl, eins, nedel, esub);
    }
};

// A workgroup's histogram: 2^lg columns per bin, as many as the level's range
// leaves room for, a lane adding in its own (or shared by few).
struct Hist {
    uint32_t *s_hist;
    int nbins, lg;
    __device__ __forceinline__ void clear() {
        lg = 6;
        while ((nbins << lg) > HWORDS) --lg;
        for (int x = threadIdx.x; x < (nbins << lg); x += WT) s_hist[x] = 0u;
    }
    __device__ __forceinline__ void flush(uint32_t *hist) const {
        for (int b = threadIdx.x; b < nbins; b += WT) {
            uint32_t h = 0u;
            for (int k = 0; k < (1 << lg); ++k) h += s_hist[(b << lg) + ((k + b) & ((1 << lg) - 1))];
            if (h) atomicAdd(&hist[(blockIdx.x % HC) * HB + b], h);
        }
    }
    // the children of one parent; m0 is the level's least parent PED
    template <int PL>
    __device__ __forceinline__ void add(const Ctx &c, const Score<PL> &sc, const Parent<PL> &pa, uint32_t m0, bool live) const {
        // (in units of a bin's columns: sums are addresses)
        uint32_t *mine = s_hist + (threadIdx.x & ((1 << lg) - 1));
        const uint32_t edel = (uint32_t)c.c.edel << lg;
        const uint32_t eins = sgpr((uint32_t)c.c.eins << lg), nedel = sgpr(0u - edel), esub = sgpr((uint32_t)c.c.esub << lg);
        const uint32_t base = ((pa.ped - m0) << lg) + __umul24(sc.deg, edel);
        const uint32_t fr = live ? sc.valid & ~pa.img : 0u;
        each_target(c.n2, [&](int u) {
            const uint32_t d = pa.child_of(base, sc, u, eins, nedel, esub) + (sc.lc(u) << lg);
            if ((fr >> u) & 1u) atomicAdd(&mine[d], 1u);
        });
        if (live) atomicAdd(&mine[base + ((uint32_t)c.c.vdel << lg)], 1u);
    }
};

// The bins that a search can use (up to its PED bound) in every copy of a
// histogram, by T threads.  (All 64 K counters by the one workgroup of a small
// beam's level took 5 us a level, and 20 before the first.)
__device__ __forceinline__ void clear_hist(const Ctx &c, uint32_t *hist, uint32_t t, uint32_t T) {
    const int lg = 32 - __builtin_clz(c.pedmax | 1u);
    for (uint32_t x = t; x < (uint32_t)HC << lg; x += T) hist[(x >> lg) * HB + (x & ((1u << lg) - 1u))] = 0u;
}

__global__ __launch_bounds__(WT) void wide1_init(Ctx c) {
    const int t = blockIdx.x * WT + threadIdx.x, T = gridDim.x * WT;
    for (int l = t; l <= c.n1; l += T) {
        Level s = {};
        s.B = l == 0 ? 1u : 0u;
        c.st[l] = s;
    }
    for (int k = 0; k < 2; ++k) clear_hist(c, c.hist[k], (uint32_t)t, (uint32_t)T);
    if (t <= c.planes) c.sets[0][(size_t)t * c.Kp] = 0u;
    if (t == 0) {
        c.ped[0][0] = 0u;
        c.img[0][0] = 0u;
        *c.ce = 0ull;
    }
}

// Edges of g2 inside Img, twice.
template <int PL>
__device__ __forceinline__ uint32_t inside2(const Ctx &c, const Score<PL> &sc, uint32_t img) {
    uint32_t e = 0u;
    each_target(c.n2, [&](int u) { e += ((img >> u) & 1u) ? (uint32_t)__popc(img & sc.row(u)) : 0u; });
    return e;
}

// Values of a level lie in [m0, m0 + range(...)]: a substitution adds at most
// the label cost, every earlier edge deleted or relabelled and every edge to
// Img inserted; a deletion its edges.
__device__ __forceinline__ int level_bins(const Ctx &c, const Level &L, int i, uint32_t deg) {
    const uint64_t inc_sub = (uint64_t)c.c.vsub + (uint64_t)max(c.c.edel, c.c.esub) * deg +
                             (uint64_t)c.c.eins * (uint64_t)min(i, c.n2);
    const uint64_t inc_del = (uint64_t)c.c.vdel + (uint64_t)c.c.edel * deg;
    uint64_t R = (uint64_t)(L.mmax - L.m0) + (inc_sub > inc_del ? inc_sub : inc_del);
    R = R < c.pedmax ? R : c.pedmax;
    return (int)R + 1;   // at most HB
}

// ------------------------------------------------------------------ hist
// The first level's histogram (its one parent).
template <int PL>
__global__ __launch_bounds__(WT) void wide1_hist(Ctx c) {
    __shared__ uint32_t s_hist[HWORDS];
    const Level L = c.st[0];
    Score<PL> sc;
    sc.load(c, 0);
    Hist h{s_hist, (int)sgpr((uint32_t)level_bins(c, L, 0, sc.deg)), 0};
    h.clear();
    __syncthreads();
    Parent<PL> pa;
    pa.load(c, 0, 0u);
    h.add<PL>(c, sc, pa, 0u, threadIdx.x == 0);
    __syncthreads();
    h.flush(c.hist[0]);
}

// ------------------------------------------------------------------ count
template <int PL>
__global__ __launch_bounds__(WT) void wide1_count(Ctx c, int i, int per) {
    __shared__ uint32_t s_tmp[NWV], s_res[2], s_first, s_last;
    const int t = threadIdx.x;
    const Level L = c.st[i];
    const uint32_t B = sgpr(L.B), m0 = sgpr(L.m0), K = c.K;
    if (t == 0) {
        s_first = HB;
        s_last = 0u;
        s_res[0] = NONE;
        s_res[1] = 0u;
    }
    __syncthreads();
    Score<PL> sc;
    sc.load(c, i);
    const int nbins = (int)sgpr((uint32_t)level_bins(c, L, i, sc.deg));
    // the bin of the K-th smallest child; V, the least and the largest value
    const int pb = (nbins + WT - 1) / WT;   // bins of a thread
    uint32_t sum = 0u, first = HB, last = 0u;
    auto bin = [&](int b) -> uint32_t {
        uint32_t h = 0u;
        if (b < nbins) {
#pragma unroll
            for (int k = 0; k < HC; ++k) h += c.hist[i & 1][k * HB + b];
        }
        return h;
    };
    for (int k = 0; k < pb; ++k) {
        const int b = t * pb + k;
        const uint32_t h = bin(b);
        sum += h;
        if (h) {
            first = min(first, (uint32_t)b);
            last = (uint32_t)b;
        }
    }
    uint32_t V;
    const uint32_t pre = block_excl_scan(sum, s_tmp, &V);
    if (sum) {
        atomicMin(&s_first, first);
        atomicMax(&s_last, last);
    }
    if (V > K && pre < K && K <= pre + sum) {
        uint32_t below = pre;
        for (int k = 0; k < pb; ++k) {
            const int b = t * pb + k;
            const uint32_t h = bin(b);
            if (below + h >= K) {
                s_res[0] = (uint32_t)b;
                s_res[1] = below;
                break;
            }
            below += h;
        }
    }
    __syncthreads();
    const uint32_t T = sgpr(s_res[0]);   // relative to m0; NONE: every child survives
    if (blockIdx.x == 0 && t == 0) {
        Level *N = c.st + i + 1;
        c.st[i].T = T;
        c.st[i].quota = T == NONE ? 0u : K - s_res[1];
        N->B = min(V, K);
        N->m0 = m0 + s_first;
        N->mmax = m0 + (T == NONE ? s_last : T);
        *c.ce += V;
    }
    const uint32_t eins = (uint32_t)c.c.eins, edel = (uint32_t)c.c.edel, esub = (uint32_t)c.c.esub, nedel = sgpr(0u - edel);
    const int Ts = T == NONE ? 0x3fffffff : (int)T;
    uint32_t lt = 0u, eq = 0u;
    for (int q = 0; q < per; ++q) {
        const uint32_t tile = blockIdx.x * (uint32_t)per + (uint32_t)q;
        if (tile * WT >= B) break;
        const uint32_t p = tile * WT + t;
        Parent<PL> pa;
        pa.load(c, i & 1, min(p, B - 1u));
        // bit u: child u at most T, below T (shifted in from the highest u on);
        // the label cost goes to the scalar side of the compare
        const uint32_t base = pa.ped - m0 + __umul24(sc.deg, edel);
        uint32_t le = 0u, l = 0u;
        each_target(c.n2, [&](int u) {
            const int d = (int)pa.child_of(base, sc, u, eins, nedel, esub), tu = Ts - (int)sc.lc(u);
            shift_in2(le, d <= tu, l, d < tu);
        });
        const uint32_t fr = p < B ? sc.valid & ~pa.img : 0u;
        le &= fr;
        l &= fr;
        if (p < B) {
            c.lem[p] = le;
            c.ltm[p] = l;
        }
        const int dd = (int)(base + (uint32_t)c.c.vdel);
        const uint32_t nl = (uint32_t)__popc(l) + (p < B && dd < Ts ? 1u : 0u);
        lt += nl;
        eq += (uint32_t)__popc(le) + (p < B && dd <= Ts ? 1u : 0u) - nl;
    }
    const uint32_t a = block_sum(lt, s_tmp), b = block_sum(eq, s_tmp);
    if (t == 0) {
        c.blk[blockIdx.x] = a;
        c.blk[MAXG + blockIdx.x] = b;
    }
}

// New slot s: parent p's state with v_i -> u (u = n2: deleted), and the Phi
// sets of level i + 1 for it; written if `live`, and returned.
template <int PL>
__device__ __forceinline__ Parent<PL> write_slot(const Ctx &c, int i, bool live, uint32_t s, uint32_t p, uint32_t u,
                                                 uint32_t deg, const uint32_t (*s_tab)[32], const uint32_t *s_nb) {
    constexpr int PLA = Score<PL>::PLA, CH = 8;
    const int cur = i & 1, nxt = cur ^ 1, v = i + 1, words = (i >> 2) + 1;
    // (the mapping's words go eight at a time: that many loads in flight)
    uint32_t x[CH];
#pragma unroll
    for (int q = 0; q < CH; ++q) x[q] = 4 * q < i ? c.phi[cur][(size_t)q * c.Kp + p] : 0u;
    Parent<PL> pa;
    pa.load(c, cur, p);
    const bool sub = u < (uint32_t)c.n2;
    const uint32_t base = pa.ped + __umul24(deg, (uint32_t)c.c.edel);
    uint32_t d = base + (uint32_t)c.c.vdel;
    if (sub) {
        uint32_t pl[PLA];
#pragma unroll
        for (int b = 0; b < PLA; ++b) pl[b] = PL > 0 ? s_tab[2 + b][u] : 0u;
        d = pa.child(base, s_tab[0][u], pl, (uint32_t)c.c.eins, sgpr(0u - (uint32_t)c.c.edel), (uint32_t)c.c.esub) + s_tab[1][u];
        pa.img |= 1u << u;
    }
    pa.ped = d;
    if (live) {
        c.ped[nxt][s] = d;
        c.img[nxt][s] = pa.img;
    }
    uint32_t ph = 0u, pb[PLA];
#pragma unroll
    for (int b = 0; b < PLA; ++b) pb[b] = 0u;
    const uint32_t img8 = sub ? u : DEL8;
    for (int w0 = 0; w0 < words; w0 += CH) {
        if (w0 > 0) {
#pragma unroll
            for (int q = 0; q < CH; ++q) x[q] = 4 * (w0 + q) < i ? c.phi[cur][(size_t)(w0 + q) * c.Kp + p] : 0u;
        }
#pragma unroll
        for (int q = 0; q < CH; ++q) {
            const int w = w0 + q;
            if (w >= words) continue;
            if (w == (i >> 2)) {
                const int at = 8 * (i & 3);
                x[q] = (x[q] & ~(0xffu << at)) | (img8 << at);
            }
            if (live) c.phi[nxt][(size_t)w * c.Kp + s] = x[q];
            if (v >= c.n1) continue;
            // v's earlier neighbours among vertices 4 w .. 4 w + 3 (s_nb: row of
            // v below v, then its label planes)
            const int k = w >> 3, sh = 4 * (w & 7);
            const uint32_t nb = sgpr((s_nb[k] >> sh) & 15u);
            if (!nb) continue;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (!((nb >> j) & 1u)) continue;
                const uint32_t y = (x[q] >> (8 * j)) & 0xffu;
                const uint32_t bit = y == DEL8 ? 0u : 1u << (y & 31u);
                ph |= bit;
#pragma unroll
                for (int b = 0; b < PLA; ++b)
                    if (PL > 0) pb[b] |= ((s_nb[(1 + b) * c.w1 + k] >> (sh + j)) & 1u) ? bit : 0u;
            }
        }
    }
    pa.ph = ph;
#pragma unroll
    for (int b = 0; b < PLA; ++b) pa.pb[b] = pb[b];
    if (v < c.n1 && live) {
        c.sets[nxt][s] = ph;
#pragma unroll
        for (int b = 0; b < PLA; ++b)
            if (PL > 0 && b < c.planes) c.sets[nxt][(size_t)(1 + b) * c.Kp + s] = pb[b];
    }
    return pa;
}

// The level's table by vertex (row, label cost, planes) for lanes that want
// different vertices.
template <int PL>
__device__ __forceinline__ void share(const Score<PL> &sc, uint32_t (*s_tab)[32]) {
    const int t = threadIdx.x;
    if (t < 32) {
        s_tab[0][t] = sc.rows;
        s_tab[1][t] = sc.lc(t);
#pragma unroll
        for (int b = 0; b < Score<PL>::PLA; ++b) s_tab[2 + b][t] = sc.planes[b];
    }
}

// The row of v = i + 1 below v and its label planes.
template <int PL>
__device__ __forceinline__ void load_next(const Ctx &c, int i, uint32_t *s_nb) {
    const int v = i + 1, t = threadIdx.x;
    if (v < c.n1 && t < (1 + PL) * c.w1) {
        const int b = t / c.w1, k = t % c.w1;
        s_nb[t] = b == 0 ? earlier_word(c, v, k, v)
                         : (b <= c.planes ? c.a1[((size_t)b * c.n1 + v) * c.w1 + k] : 0u);
    }
}

// ------------------------------------------------------------------ emit
// Survivor records (parent << 6 | vertex, n2 for the deletion) in generation order.
template <int PL>
__global__ __launch_bounds__(WT) void wide1_emit(Ctx c, int i, int per) {
    __shared__ uint32_t s_tmp[NWV];
    const int t = threadIdx.x;
    const Level L = c.st[i];
    const uint32_t B = sgpr(L.B), m0 = sgpr(L.m0), T = sgpr(L.T), quota = sgpr(L.quota);
    const int Ts = T == NONE ? 0x3fffffff : (int)T;
    Score<PL> sc;
    sc.load(c, i);
    clear_hist(c, c.hist[i & 1], blockIdx.x * WT + t, gridDim.x * WT);
    // children below T, equal to T of the workgroups before this one
    uint32_t a = 0u, e = 0u;
    for (uint32_t b = t; b < blockIdx.x; b += WT) {
        a += c.blk[b];
        e += c.blk[MAXG + b];
    }
    uint32_t LT = block_sum(a, s_tmp), EQ = block_sum(e, s_tmp);
    for (int q = 0; q < per; ++q) {
        const uint32_t tile = blockIdx.x * (uint32_t)per + (uint32_t)q;
        if (tile * WT >= B) break;
        const uint32_t p = tile * WT + t;
        uint64_t le = 0ull, lt = 0ull;
        if (p < B) {
            const int dd = (int)(c.ped[i & 1][p] - m0 + __umul24(sc.deg, (uint32_t)c.c.edel) + (uint32_t)c.c.vdel);
            le = (uint64_t)c.lem[p] | ((uint64_t)(dd <= Ts ? 1u : 0u) << 32);
            lt = (uint64_t)c.ltm[p] | ((uint64_t)(dd < Ts ? 1u : 0u) << 32);
        }
        const uint32_t nlt = (uint32_t)__popcll(lt), neq = (uint32_t)__popcll(le) - nlt;
        uint32_t tot;   // (at most 33 a thread: halves of a word)
        const uint32_t pre = block_excl_scan(nlt | (neq << 16), s_tmp, &tot);
        const uint32_t keptb = min(EQ + (pre >> 16), quota);   // ties kept before the parent
        uint32_t keq = min(quota - keptb, neq);               // ... and of the parent
        uint32_t pos = LT + (pre & 0xffffu) + keptb;
        uint64_t m = keq > 0u ? le : lt;
        while (m) {
            const int u = (int)__builtin_ctzll(m);
            m &= m - 1ull;
            if (!((lt >> u) & 1ull)) {
                if (keq == 0u) continue;
                --keq;
            }
            if (pos < c.K) c.rec[pos] = (p << 6) | (uint32_t)(u < 32 ? u : c.n2);
            ++pos;
        }
        LT += tot & 0xffffu;
        EQ += tot >> 16;
    }
}

// ------------------------------------------------------------------ update
// A thread per new slot.  hist: also count the new slots' children for the
// next level.
template <int PL>
__global__ __launch_bounds__(WT) void wide1_update(Ctx c, int i, int hist) {
    __shared__ uint32_t s_nb[(1 + PL) * (GED_MAX_VERTICES / 32)], s_tab[2 + Score<PL>::PLA][32];
    __shared__ uint32_t s_hist[HWORDS];
    const int t = threadIdx.x;
    const Level N = c.st[i + 1];
    const uint32_t Bn = sgpr(N.B), m1 = sgpr(N.m0), Bp = sgpr(c.st[i].B);
    Score<PL> sc, sn;
    load_next<PL>(c, i, s_nb);
    sc.load(c, i);
    share(sc, s_tab);
    Hist h{s_hist, 0, 0};
    if (hist) {
        sn.load(c, i + 1);
        h.nbins = (int)sgpr((uint32_t)level_bins(c, N, i + 1, sn.deg));
        h.clear();
    }
    __syncthreads();
    // (lanes past the beam repeat its last slot, unwritten: the targets' rows
    // are read across lanes)
    for (uint32_t x0 = blockIdx.x * WT; x0 < Bn; x0 += gridDim.x * WT) {
        const uint32_t s = x0 + t, r = c.rec[min(s, Bn - 1u)];
        const bool live = s < Bn;
        const Parent<PL> pa = write_slot<PL>(c, i, live, s, min(r >> 6, Bp - 1u), r & 63u, sc.deg, s_tab, s_nb);
        if (hist) h.add<PL>(c, sn, pa, m1, live);
    }
    __syncthreads();
    if (hist) h.flush(c.hist[(i + 1) & 1]);
}

// ------------------------------------------------------------------ complete-then-minimum
// Last level with that option: every child's total (Sec. 4.4.1); the least
// (total, generation order) lands in *best.
template <int PL>
__global__ __launch_bounds__(WT) void wide1_complete(Ctx c, int i, int per) {
    __shared__ unsigned long long s_key[NWV];
    __shared__ uint32_t s_tmp[NWV];
    const int t = threadIdx.x, cur = i & 1;
    const uint32_t B = sgpr(c.st[i].B);
    Score<PL> sc;
    sc.load(c, i);
    unsigned long long key = ~0ull;
    uint32_t children = 0u;
    for (int q = 0; q < per; ++q) {
        const uint32_t tile = blockIdx.x * (uint32_t)per + (uint32_t)q;
        if (tile * WT >= B) break;
        const uint32_t p = tile * WT + t;
        const bool live = p < B;
        Parent<PL> pa;
        pa.load(c, cur, min(p, B - 1u));
        const uint32_t base = pa.ped + __umul24(sc.deg, (uint32_t)c.c.edel);
        const uint32_t left = (uint32_t)c.n2 - (uint32_t)__popc(pa.img), e0 = inside2(c, sc, pa.img) / 2u;
        children += live ? left + 1u : 0u;
        auto take = [&](uint32_t total, int u, bool in) {
            const unsigned long long k = ((unsigned long long)total << 32) | ((p << 6) | (uint32_t)u);
            key = in && k < key ? k : key;
        };
        const uint32_t vins = (uint32_t)c.c.vins, eins = (uint32_t)c.c.eins, out = (uint32_t)c.m2 - e0;
        const uint32_t nedel = sgpr(0u - (uint32_t)c.c.edel);
        const uint32_t fr = live ? sc.valid & ~pa.img : 0u;
        each_target(c.n2, [&](int u) {
            const uint32_t add = (uint32_t)__popc(pa.img & sc.row(u));
            const uint32_t d = pa.child_of(base, sc, u, eins, nedel, (uint32_t)c.c.esub) + sc.lc(u);
            take(d + vins * (left - 1u) + eins * (out - add), u, (fr >> u) & 1u);
        });
        take(base + (uint32_t)c.c.vdel + vins * left + eins * out, c.n2, live);
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long other = (unsigned long long)__shfl_xor((long long)key, o);
        key = other < key ? other : key;
    }
    if ((t & 63) == 0) s_key[t >> 6] = key;
    const uint32_t V = block_sum(children, s_tmp);
    if (t == 0) {
        unsigned long long m = s_key[0];
#pragma unroll
        for (int k = 1; k < NWV; ++k) m = s_key[k] < m ? s_key[k] : m;
        c.best[blockIdx.x] = m;
        atomicAdd(c.ce, (unsigned long long)V);
    }
}

// The least of the workgroups' keys, in every thread.
__device__ __forceinline__ unsigned long long least_key(const Ctx &c, int groups) {
    __shared__ unsigned long long s_key[NWV];
    unsigned long long key = ~0ull;
    for (int b = threadIdx.x; b < groups; b += WT) key = c.best[b] < key ? c.best[b] : key;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long other = (unsigned long long)__shfl_xor((long long)key, o);
        key = other < key ? other : key;
    }
    if ((threadIdx.x & 63) == 0) s_key[threadIdx.x >> 6] = key;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NWV; ++k) key = s_key[k] < key ? s_key[k] : key;
    return key;
}

// The winner becomes the only survivor.
template <int PL>
__global__ __launch_bounds__(WT) void wide1_pick(Ctx c, int i, int groups) {
    __shared__ uint32_t s_nb[(1 + PL) * (GED_MAX_VERTICES / 32)], s_tab[2 + Score<PL>::PLA][32];
    Score<PL> sc;
    load_next<PL>(c, i, s_nb);
    sc.load(c, i);
    share(sc, s_tab);
    const uint32_t r = (uint32_t)(least_key(c, groups) & 0xffffffffull);
    (void)write_slot<PL>(c, i, threadIdx.x == 0, 0u, r >> 6, r & 63u, sc.deg, s_tab, s_nb);
    if (threadIdx.x != 0) return;
    c.st[i + 1].B = 1u;
}

// ------------------------------------------------------------------ final
// Every leaf's total; the least (total, slot) wins.
__global__ __launch_bounds__(WT) void wide1_final_keys(Ctx c, int per) {
    __shared__ unsigned long long s_key[NWV];
    const int cur = c.n1 & 1, t = threadIdx.x;
    const uint32_t B = sgpr(c.st[c.n1].B);
    Score<0> sc;
    sc.rows = (t & 63) < c.n2 ? c.a2[t & 63] : 0u;
    unsigned long long key = ~0ull;
    for (int q = 0; q < per; ++q) {
        const uint32_t s = (blockIdx.x * (uint32_t)per + (uint32_t)q) * WT + t;
        const uint32_t at = min(s, B - 1u), img = c.img[cur][at];
        const uint32_t left = (uint32_t)c.n2 - (uint32_t)__popc(img);
        const uint32_t total = c.ped[cur][at] + (uint32_t)c.c.vins * left +
                               (uint32_t)c.c.eins * ((uint32_t)c.m2 - inside2(c, sc, img) / 2u);
        const unsigned long long k = ((unsigned long long)total << 32) | s;
        key = s < B && k < key ? k : key;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        const unsigned long long other = (unsigned long long)__shfl_xor((long long)key, o);
        key = other < key ? other : key;
    }
    if ((t & 63) == 0) s_key[t >> 6] = key;
    __syncthreads();
    if (t == 0) {
        unsigned long long m = s_key[0];
#pragma unroll
        for (int k = 1; k < NWV; ++k) m = s_key[k] < m ? s_key[k] : m;
        c.best[blockIdx.x] = m;
    }
}

__global__ __launch_bounds__(WT) void wide1_final_map(Ctx c, int groups) {
    const int cur = c.n1 & 1;
    const unsigned long long best = least_key(c, groups);
    const uint32_t slot = (uint32_t)(best & 0xffffffffull);
    if (threadIdx.x == 0) {
        *c.out_dist = (int32_t)(best >> 32);
        if (c.out_cand) *c.out_cand = (int64_t)*c.ce;
    }
    for (int j = threadIdx.x; j < c.n1; j += WT) {
        const uint32_t x = (c.phi[cur][(size_t)(j >> 2) * c.Kp + slot] >> (8 * (j & 3))) & 0xffu;
        c.out_map[j] = x == DEL8 ? -1 : (int32_t)x;
    }
}

// ------------------------------------------------------------------ host side

struct Layout {
    size_t ped[2], img[2], sets[2], phi[2], blk, hist[2], lem, ltm, rec, st, ce, best, total;
};

Layout layout(int n1, int planes, uint32_t Kp) {
    Layout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += (bytes + 255) & ~(size_t)255;
        return o;
    };
    for (int k = 0; k < 2; ++k) {
        L.ped[k] = take((size_t)Kp * 4);
        L.img[k] = take((size_t)Kp * 4);
        L.sets[k] = take((size_t)(1 + planes) * Kp * 4);
        L.phi[k] = take((size_t)((n1 + 3) / 4) * Kp * 4);
    }
    L.blk = take((size_t)2 * MAXG * 4);
    for (int k = 0; k < 2; ++k) L.hist[k] = take((size_t)HC * HB * 4);
    L.lem = take((size_t)Kp * 4);
    L.rec = take((size_t)Kp * 4);
    L.ltm = take((size_t)Kp * 4);
    L.st = take((size_t)(n1 + 1) * sizeof(Level));
    L.ce = take(8);
    L.best = take((size_t)MAXG * 8);
    L.total = off;
    return L;
}

uint32_t slot_stride(int K) { return (uint32_t)((K + WT - 1) / WT) * WT; }

template <int PL>
hipError_t levels(const Ctx &c, bool last_complete, int cus, hipStream_t stream) {
    hipLaunchKernelGGL(wide1_init, dim3(1 + c.pedmax / 256), dim3(WT), 0, stream, c);
    uint64_t bound = 1;   // parents at level i are at most min(K, (n2 + 1)^i)
    // workgroups: eight per CU, each with a few tiles, so that the counters'
    // columns and the threshold are paid for once per several tiles
    auto split = [&](uint64_t parents, int *grid, int *per) {
        const int tiles = (int)((parents + WT - 1) / WT);
        const int most = std::min(MAXG, 8 * cus);
        *per = (tiles + most - 1) / most;
        *grid = (tiles + *per - 1) / *per;
    };
    int grid, per;
    const int scored = last_complete ? c.n1 - 1 : c.n1;   // levels that select
    if (scored > 0) hipLaunchKernelGGL(wide1_hist<PL>, dim3(1), dim3(WT), 0, stream, c);
    for (int i = 0; i < c.n1; ++i) {
        split(bound, &grid, &per);
        if (last_complete && i == c.n1 - 1) {
            hipLaunchKernelGGL(wide1_complete<PL>, dim3(grid), dim3(WT), 0, stream, c, i, per);
            hipLaunchKernelGGL(wide1_pick<PL>, dim3(1), dim3(WT), 0, stream, c, i, grid);
            bound = 1;
            break;
        }
        hipLaunchKernelGGL(wide1_count<PL>, dim3(grid), dim3(WT), 0, stream, c, i, per);
        hipLaunchKernelGGL(wide1_emit<PL>, dim3(grid), dim3(WT), 0, stream, c, i, per);
        const uint64_t grown = bound * (uint64_t)(c.n2 + 1);
        bound = grown < c.K ? grown : c.K;
        const int ugrid = (int)std::min<uint64_t>((bound + WT - 1) / WT, (uint64_t)8 * cus);
        hipLaunchKernelGGL(wide1_update<PL>, dim3(ugrid), dim3(WT), 0, stream, c, i, i + 1 < scored ? 1 : 0);
    }
    split(bound, &grid, &per);
    hipLaunchKernelGGL(wide1_final_keys, dim3(grid), dim3(WT), 0, stream, c, per);
    hipLaunchKernelGGL(wide1_final_map, dim3(1), dim3(WT), 0, stream, c, grid);
    return hipGetLastError();
}

}  // namespace

size_t wide1_workspace_bytes(int n1, int planes, int K) { return layout(n1, planes, slot_stride(K)).total; }

hipError_t launch_wide1(const DbView &src, const DbView &dst, const GraphRec &g1, const GraphRec &g2, Costs costs, int K,
                        int last_complete, uint32_t pedmax, void *ws, size_t ws_bytes, int32_t *dist, int32_t *map,
                        int64_t *cand, int cus, hipStream_t stream) {
    const int planes = dst.planes;
    const uint32_t Kp = slot_stride(K);
    const Layout L = layout(g1.n, planes, Kp);
    if (K < 1 || K > kWideMaxK || L.total > ws_bytes || g2.n > kWide1MaxN2 || pedmax >= (uint32_t)HB ||
        g1.n > GED_MAX_VERTICES || cus < 1)
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
    c.m2 = g2.m;
    c.planes = planes;
    c.c = costs;
    c.pedmax = pedmax;
    c.K = (uint32_t)K;
    c.Kp = Kp;
    for (int k = 0; k < 2; ++k) {
        c.ped[k] = reinterpret_cast<uint32_t *>(base + L.ped[k]);
        c.img[k] = reinterpret_cast<uint32_t *>(base + L.img[k]);
        c.sets[k] = reinterpret_cast<uint32_t *>(base + L.sets[k]);
        c.phi[k] = reinterpret_cast<uint32_t *>(base + L.phi[k]);
    }
    c.blk = reinterpret_cast<uint32_t *>(base + L.blk);
    for (int k = 0; k < 2; ++k) c.hist[k] = reinterpret_cast<uint32_t *>(base + L.hist[k]);
    c.lem = reinterpret_cast<uint32_t *>(base + L.lem);
    c.rec = reinterpret_cast<uint32_t *>(base + L.rec);
    c.ltm = reinterpret_cast<uint32_t *>(base + L.ltm);
    c.st = reinterpret_cast<Level *>(base + L.st);
    c.ce = reinterpret_cast<unsigned long long *>(base + L.ce);
    c.best = reinterpret_cast<unsigned long long *>(base + L.best);
    c.out_dist = dist;
    c.out_map = map;
    c.out_cand = cand;
    if (planes == 0) return levels<0>(c, last_complete != 0, cus, stream);
    if (planes <= 2) return levels<2>(c, last_complete != 0, cus, stream);
    return levels<4>(c, last_complete != 0, cus, stream);
}

}  // namespace gedk
