// Reachability kernels of the learned reset proposal: breadth-first search on
// C-free bitsets, by one wavefront in its registers, or (maps whose searches do
// not fit a wavefront's registers) by a workgroup in LDS.
// Each search level dilates the frontier by one 4-neighbour move with word
// shifts (left/right within a row, carries across words) and row offsets
// (up/down), masks it with the C-free cells not yet reached, and stops as soon
// as the target bit appears, the frontier empties or the depth limit is reached.
#include <limits.h>
#include <math.h>

#include "mlp_internal.hpp"
#include "philox.hpp"
#include "reach_internal.hpp"

namespace navsim {
namespace {

constexpr double kPiR = 3.14159265358979323846;
constexpr double kTwo32 = 4294967296.0;

__device__ __forceinline__ bool cell_bit(const uint32_t *b, const ReachDesc &d, int cell) {
    const int i = cell % d.W, j = cell / d.W;
    return (b[j * d.wpr + (i >> 5)] >> (i & 31)) & 1u;
}

__device__ __forceinline__ void set_cell(uint32_t *b, const ReachDesc &d, int cell) {
    const int i = cell % d.W, j = cell / d.W;
    b[j * d.wpr + (i >> 5)] |= 1u << (i & 31);
}

__device__ __forceinline__ uint16_t bf16_bits(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return 0x7fc0u;
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ void stage_free(const ReachParams &rp, const ReachDesc &d, uint32_t *fb) {
    const uint32_t *g = rp.bits + d.bit_off;
    for (int w = threadIdx.x; w < d.words; w += blockDim.x) fb[w] = g[w];
}

// One search level: nx = (frontier moved by one step) & C-free & ~visited,
// visited |= nx, over the words of rows r0..r1 and word columns c0..c1 only
// (the caller's box holds every bit the level can set; nx, vis and fr are
// zero outside it).  Returns the OR of this thread's nx words.
__device__ uint32_t search_level(const ReachDesc &d, const uint32_t *fb, uint32_t *vis,
                                 const uint32_t *fr, uint32_t *nx, int r0, int r1, int c0,
                                 int c1) {
    uint32_t any = 0;
    const int wpr = d.wpr, nw = c1 - c0 + 1, total = (r1 - r0 + 1) * nw;
    const float inv_nw = 1.0f / (float)nw;
    for (int q = threadIdx.x; q < total; q += blockDim.x) {
        int rr = (int)((float)q * inv_nw);
        if (rr * nw > q) --rr;
        if ((rr + 1) * nw <= q) ++rr;
        const int r = r0 + rr, c = c0 + (q - rr * nw), w = r * wpr + c;
        const uint32_t f = fr[w];
        uint32_t g = (f << 1) | (f >> 1);
        if (c > 0) g |= fr[w - 1] >> 31;
        if (c + 1 < wpr) g |= fr[w + 1] << 31;
        if (r > 0) g |= fr[w - wpr];
        if (r + 1 < d.H) g |= fr[w + wpr];
        const uint32_t n = g & fb[w] & ~vis[w];
        nx[w] = n;
        vis[w] |= n;
        any |= n;
    }
    return any;
}

// Rows and word columns that level `level` (>= 1 moves from cell a) can reach.
struct SearchBox {
    int r0, r1, c0, c1;
};

__device__ __forceinline__ SearchBox level_box(const ReachDesc &d, int a, int level) {
    const int i = a % d.W, j = a / d.W;
    SearchBox b;
    b.r0 = max(j - level, 0);
    b.r1 = min(j + level, d.H - 1);
    b.c0 = max(i - level, 0) >> 5;
    b.c1 = min(i + level, d.W - 1) >> 5;
    return b;
}

// Clears vis, fr and nx and seeds vis and fr with cell a (which must be C-free).
__device__ void search_start(const ReachDesc &d, uint32_t *vis, uint32_t *fr, uint32_t *nx,
                             int a) {
    uint4 *v4 = reinterpret_cast<uint4 *>(vis), *f4 = reinterpret_cast<uint4 *>(fr),
          *n4 = reinterpret_cast<uint4 *>(nx);
    const uint4 z = make_uint4(0u, 0u, 0u, 0u);
    for (int w = threadIdx.x; w < (d.words + 3) / 4; w += blockDim.x) {
        v4[w] = z;
        f4[w] = z;
        n4[w] = z;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        set_cell(vis, d, a);
        set_cell(fr, d, a);
    }
    __syncthreads();
}

// Hop count from C-free a to b within max_hops moves, else -1 (uniform
// across the workgroup).  A 4-neighbour path is at least as long as the
// Manhattan distance, so a farther b is rejected without a search, and level
// L only touches the box of cells within L moves of a.
__device__ int hops_to(const ReachDesc &d, const uint32_t *fb, uint32_t *vis, uint32_t *fr,
                       uint32_t *nx, int a, int b, int max_hops) {
    if (a == b) return 0;
    const int man = abs(a % d.W - b % d.W) + abs(a / d.W - b / d.W);
    if (man > max_hops) return -1;
    search_start(d, vis, fr, nx, a);
    for (int level = 0; level < max_hops; ++level) {
        const SearchBox bx = level_box(d, a, level + 1);
        const uint32_t any = search_level(d, fb, vis, fr, nx, bx.r0, bx.r1, bx.c0, bx.c1);
        const int more = __syncthreads_or(any != 0u);
        if (cell_bit(nx, d, b)) return level + 1;
        if (!more) return -1;
        uint32_t *t = fr;
        fr = nx;
        nx = t;
    }
    return -1;
}

__device__ __forceinline__ double centre_dist(const ReachDesc &d, int a, int b) {
    const double dx = (double)(b % d.W - a % d.W) * (double)d.s;
    const double dy = (double)(b / d.W - a / d.W) * (double)d.s;
    return sqrt(dx * dx + dy * dy);
}

// The exact check of (a, b) for bin k: hop count when valid, else -1.
__device__ int check_pair(const ReachParams &rp, const ReachDesc &d, const uint32_t *fb,
                          uint32_t *vis, uint32_t *fr, uint32_t *nx, int a, int b, int k) {
    if (a < 0 || b < 0 || !cell_bit(fb, d, a) || !cell_bit(fb, d, b)) return -1;
    if (centre_dist(d, a, b) < rp.gmd) return -1;
    const int h = hops_to(d, fb, vis, fr, nx, a, b, rp.bin_hi[k]);
    return (h >= 0 && rp.hop_bin[h] == k) ? h : -1;
}

// Nearest C-free cell to c: least |di| + |dj|, then least index; -1 if none.
__device__ int snap_cell(const ReachDesc &d, const uint32_t *fb, int c, int *s_min) {
    if (cell_bit(fb, d, c)) return c;
    const int i0 = c % d.W, j0 = c / d.W;
    for (int r = 1; r <= d.W + d.H; ++r) {
        __syncthreads();
        if (threadIdx.x == 0) *s_min = INT_MAX;
        __syncthreads();
        for (int q = threadIdx.x; q < 4 * r; q += blockDim.x) {
            const int side = q / r, t = q % r;
            int di, dj;
            if (side == 0) {
                di = r - t;
                dj = t;
            } else if (side == 1) {
                di = -t;
                dj = r - t;
            } else if (side == 2) {
                di = t - r;
                dj = -t;
            } else {
                di = t;
                dj = t - r;
            }
            const int i = i0 + di, j = j0 + dj;
            if (i >= 0 && i < d.W && j >= 0 && j < d.H && cell_bit(fb, d, j * d.W + i))
                atomicMin(s_min, j * d.W + i);
        }
        __syncthreads();
        const int m = *s_min;
        if (m != INT_MAX) return m;
    }
    return -1;
}

__device__ __forceinline__ int decode_axis(float y, int n) {
    const double v = (double)y * (double)n;
    if (v != v) return 0;
    const double f = floor(v);
    return f < 0.0 ? 0 : (f > (double)(n - 1) ? n - 1 : (int)f);
}

__device__ __forceinline__ float decode_heading(float y) {
    double t = (double)y;
    t = t != t ? 0.0 : (t < -1.0 ? -1.0 : (t > 1.0 ? 1.0 : t));
    return (float)(t * kPiR);
}

__device__ __forceinline__ float cell_x(const ReachDesc &d, int c) {
    return (float)(((double)(c % d.W) + 0.5) * (double)d.s);
}

__device__ __forceinline__ float cell_y(const ReachDesc &d, int c) {
    return (float)(((double)(c / d.W) + 0.5) * (double)d.s);
}

__global__ __launch_bounds__(kReachThreads) void label_kernel(ReachParams rp, const int32_t *map,
                                                              uint32_t first_sid, int32_t *start,
                                                              int32_t *goal, int32_t *hops) {
    extern __shared__ uint4 lds4[];  // 16-byte aligned: the searches clear it 16 bytes at a time
    uint32_t *lds = reinterpret_cast<uint32_t *>(lds4);
    __shared__ unsigned long long s_best[kReachMaxBins];
    const int i = blockIdx.x, tid = threadIdx.x;
    const int mk = map[i];
    const ReachDesc d = rp.maps[(mk >= 0 && mk < rp.num_maps) ? mk : 0];
    const uint32_t sid = first_sid + (uint32_t)i;
    if (d.free_cnt == 0 || mk < 0 || mk >= rp.num_maps) {
        if (rp.any_label) return;  // label_wave_kernel wrote these
        if (tid < rp.nbins) {
            goal[(int64_t)i * rp.nbins + tid] = -1;
            hops[(int64_t)i * rp.nbins + tid] = -1;
        }
        if (tid == 0) start[i] = -1;
        return;
    }
    if (d.label_ok) return;  // and those
    uint32_t *fb = lds, *vis = fb + kReachMaxWords, *fr = vis + kReachMaxWords,
             *nx = fr + kReachMaxWords;
    uint32_t c[4] = {sid, 0u, 0u, 6u};
    philox4x32_10(c, rp.key0, rp.key1);
    const int a = rp.free_cells[d.free_off + pick_of(c[0], d.free_cnt)];
    stage_free(rp, d, fb);
    if (tid < kReachMaxBins) s_best[tid] = ~0ull;
    search_start(d, vis, fr, nx, a);
    for (int level = 0; level < rp.max_hops; ++level) {
        const SearchBox bx = level_box(d, a, level + 1);
        const uint32_t any = search_level(d, fb, vis, fr, nx, bx.r0, bx.r1, bx.c0, bx.c1);
        const int h = level + 1;
        const int k = rp.hop_bin[h];
        if (k >= 0 && any) {
            // the words this thread wrote in search_level (same box, same
            // order), so no barrier is needed before reading them
            unsigned long long best = ~0ull;
            const int nw = bx.c1 - bx.c0 + 1, total = (bx.r1 - bx.r0 + 1) * nw;
            const float inv_nw = 1.0f / (float)nw;
            for (int qi = tid; qi < total; qi += blockDim.x) {
                int rr = (int)((float)qi * inv_nw);
                if (rr * nw > qi) --rr;
                if ((rr + 1) * nw <= qi) ++rr;
                const int row = bx.r0 + rr, wc = bx.c0 + (qi - rr * nw);
                uint32_t n = nx[row * d.wpr + wc];
                const int col0 = wc * 32;
                while (n) {
                    const int bit = __ffs(n) - 1;
                    n &= n - 1u;
                    const int cell = row * d.W + col0 + bit;
                    if (centre_dist(d, a, cell) < rp.gmd) continue;
                    uint32_t q[4] = {sid, (uint32_t)cell, 0u, 5u};
                    philox4x32_10(q, rp.key0, rp.key1);
                    const unsigned long long v = ((unsigned long long)q[0] << 32) |
                                                 ((unsigned long long)cell << 16) |
                                                 (unsigned long long)h;
                    best = v < best ? v : best;
                }
            }
            if (best != ~0ull) atomicMin(&s_best[k], best);
        }
        if (!__syncthreads_or(any != 0u)) break;
        uint32_t *t = fr;
        fr = nx;
        nx = t;
    }
    __syncthreads();
    if (tid < rp.nbins) {
        const unsigned long long v = s_best[tid];
        goal[(int64_t)i * rp.nbins + tid] = v == ~0ull ? -1 : (int32_t)((v >> 16) & 0xffffu);
        hops[(int64_t)i * rp.nbins + tid] = v == ~0ull ? -1 : (int32_t)(v & 0xffffu);
    }
    if (tid == 0) start[i] = a;
}

// ---------------------------------------------------------------------------
// Searches in one wavefront's registers, on the packed bitsets.  The 4-neighbour
// grid is bipartite: a level's frontier lies on one checkerboard colour and the
// next one on the other, so the two colours are kept apart and a level touches
// only half of the map's bits.  Within a packed row, cell p of the colour that
// receives the level neighbours cells p of the rows above and below and cells p
// and p - 1 (or p and p + 1, by the row's parity) of its own row in the other
// colour.  The lanes of the wavefront hold NW words of each colour: NW / P whole
// rows of P words, of the window of the map that a path of at most max_hops
// moves can touch (see search_hops), so a small bin's search runs in 2 x 4
// words a lane where the whole of a 256 x 256 map takes 2 x 16.  A row's carries
// stay in the lane and only the rows next to the lane's first and last come from
// the lanes beside it (cross-lane moves).  No LDS and no workgroup barrier per
// level.
//
// The searches are bound by VALU issue: about 4.5 instructions per word and
// level (a funnel shift, an or of three, two three-operand logic operations, and
// the frontier's emptiness every other level), against 6.5 on twice the words
// with both colours in one bitset.  8,192 requests on 64 maps of 256 x 256 cells:
// 3,454 -> 1,072 us; 490 requests inside a step of 32,768 envs, head round 312 ->
// 117 us and the tail rounds 217 -> 100 us (the whole step 935 -> 624 us).

template <int N>
using Words = uint32_t __attribute__((ext_vector_type(N)));
typedef __attribute__((address_space(3))) const uint32_t LdsWord;
typedef __attribute__((address_space(3))) const int LdsInt;

// One level into the words of colour CB (rows counted from an even row): nx =
// the cells of `un` (C-free, not reached) with a neighbour in the frontier f of
// the other colour; they leave un.  Returns the OR of the lane's nx words.
template <int P, int NW, int CB>
__device__ __forceinline__ uint32_t packed_level(const Words<NW> &f, Words<NW> &nx, Words<NW> &un,
                                                 int lane) {
    constexpr int R = NW / P;  // rows per lane
    static_assert(R == 1 || R % 2 == 0, "a lane's first row is even, or lanes alternate");
    uint32_t up[P], dn[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        // DPP wavefront shifts by one lane (wave_shr:1, wave_shl:1), 0 past the ends
        up[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f[NW - P + k], 0x138, 0xf, 0xf, true);
        dn[k] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)f[k], 0x130, 0xf, 0xf, true);
    }
    uint32_t any = 0u;
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const int k = j % P;
        const uint32_t prev = k > 0 ? f[k > 0 ? j - 1 : 0] : 0u;
        const uint32_t next = k < P - 1 ? f[k < P - 1 ? j + 1 : 0] : 0u;
        const uint32_t lower = __builtin_amdgcn_alignbit(f[j], prev, 31u);
        const uint32_t upper = __builtin_amdgcn_alignbit(next, f[j], 1u);
        const bool odd = R == 1 ? ((lane + CB) & 1) != 0 : ((j / P + CB) & 1) != 0;
        const uint32_t t = f[j] | (odd ? upper : lower) | (j >= P ? f[j >= P ? j - P : 0] : up[k]) |
                           (j + P < NW ? f[j + P < NW ? j + P : 0] : dn[k]);
        nx[j] = t & un[j];
        un[j] &= ~t;
        any |= nx[j];
    }
    return any;
}

// A window of a map's packed bitsets (H rows of pk words per colour, pwords
// words in all): rows from the even row j0, word columns from cw0.
struct Window {
    int j0, cw0, H, pk, pwords;
};

// The C-free words of a window, both colours (words outside the map are 0).
template <int P, int NW, typename Ptr>
__device__ __forceinline__ void load_window(Ptr fb, const Window &w, Words<NW> &un0,
                                            Words<NW> &un1, int lane) {
    const int r0 = w.j0 + lane * (NW / P);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const int row = r0 + j / P, col = w.cw0 + j % P;
        const bool in = row < w.H && col < w.pk;
        const int q = in ? row * w.pk + col : 0;
        const uint32_t v0 = fb[q], v1 = fb[q + w.pwords];
        un0[j] = in ? v0 : 0u;
        un1[j] = in ? v1 : 0u;
    }
}

// Hop count from cell (ia, ja) to (ib, jb) (both C-free, not the same) within
// max_hops moves, else -1 (uniform across the wavefront).
template <int P, int NW>
__device__ __forceinline__ int window_hops(LdsWord *fb, const Window &w, int ia, int ja, int ib,
                                           int jb, int max_hops, int lane, int c, LdsInt *s_won,
                                           const int *g_won) {
    Words<NW> f0, f1, un0, un1;
    load_window<P, NW>(fb, w, un0, un1, lane);
    const int ca = (ia + ja) & 1, cb = (ib + jb) & 1;
    const int wa = (ja - w.j0) * P + (ia >> 6) - w.cw0, wb = (jb - w.j0) * P + (ib >> 6) - w.cw0;
    const uint32_t ba = 1u << ((ia >> 1) & 31);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const uint32_t seed = wa == lane * NW + j ? ba : 0u;
        f0[j] = ca == 0 ? seed : 0u;
        f1[j] = ca == 0 ? 0u : seed;
        un0[j] &= ~f0[j];
        un1[j] &= ~f1[j];
    }
    // b is reached when its bit leaves un, at a level into its own colour; its
    // register index is the same on every lane (one relative register move)
    const int lb = wb / NW, xb = wb % NW, sb = (ib >> 1) & 31;
    auto reached = [&](const Words<NW> &un) {
        return (((uint32_t)__builtin_amdgcn_readlane((int)un[xb], lb) >> sb) & 1u) == 0u;
    };
    int level = 0;
    if (ca == 1) {  // the first move leaves colour 1
        if (max_hops < 1) return -1;
        level = 1;
        (void)packed_level<P, NW, 0>(f1, f0, un0, lane);
        if (cb == 0 && reached(un0)) return 1;
    }
    while (level < max_hops) {
        // a lower candidate of the round (s_won, LDS) or of the request (g_won,
        // device memory: other workgroups' rounds) already passed: this one
        // cannot win (looked at every 8 levels)
        if ((level & 6) == 0) {
            if (s_won && __atomic_load_n(s_won, __ATOMIC_RELAXED) < c) return -1;
            if (g_won && __atomic_load_n(g_won, __ATOMIC_RELAXED) < c) return -1;
        }
        (void)packed_level<P, NW, 1>(f0, f1, un1, lane);
        ++level;
        if (cb == 1 && reached(un1)) return level;
        if (level >= max_hops) break;
        // once a level is empty the next one is too: looked at every other level
        const uint32_t any = packed_level<P, NW, 0>(f1, f0, un0, lane);
        ++level;
        if (cb == 0 && reached(un0)) return level;
        if (__ballot(any != 0u) == 0ull) break;
    }
    return -1;
}

// The smallest register layout for a window of ncw word columns and nr rows
// (the map's pair_ok / label_ok says that one holds it).
#define NAVSIM_PACKED_SHAPES(X, ncw, nr) \
    if ((ncw) <= 1) {                    \
        if ((nr) <= 256) X(1, 4)         \
        else if ((nr) <= 512) X(1, 8)    \
        else X(1, 16)                    \
    } else if ((ncw) <= 2) {             \
        if ((nr) <= 128) X(2, 4)         \
        else if ((nr) <= 256) X(2, 8)    \
        else X(2, 16)                    \
    } else if ((ncw) <= 4) {             \
        if ((nr) <= 128) X(4, 8)         \
        else X(4, 16)                    \
    } else if ((ncw) <= 8) X(8, 16)      \
    else X(16, 16)

// window_hops in the window of the cells that a path of at most max_hops moves
// can touch: those within max_hops of a and b together (Manhattan distances),
// that is at most (max_hops - |a - b|) / 2 cells outside the box of a and b.
// Needs |a - b| <= max_hops; every argument is the same on every lane.  Inlined:
// as a call, 41 registers a search went to scratch and back (3 % slower).
__device__ __forceinline__ int search_hops(LdsWord *fb, int W, int H, int pk, int a,
                                                     int b, int max_hops, int c, LdsInt *s_won,
                                                     const int *g_won) {
    const int lane = threadIdx.x & 63;
    W = __builtin_amdgcn_readfirstlane(W);
    a = __builtin_amdgcn_readfirstlane(a);
    b = __builtin_amdgcn_readfirstlane(b);
    const int hi = __builtin_amdgcn_readfirstlane(max_hops);
    c = __builtin_amdgcn_readfirstlane(c);
    const int ia = a % W, ja = a / W, ib = b % W, jb = b / W;
    const int slack = (hi - abs(ia - ib) - abs(ja - jb)) >> 1;
    Window w;
    w.H = __builtin_amdgcn_readfirstlane(H);
    w.pk = __builtin_amdgcn_readfirstlane(pk);
    w.pwords = w.H * w.pk;
    w.j0 = max(min(ja, jb) - slack, 0) & ~1;
    w.cw0 = max(min(ia, ib) - slack, 0) >> 6;
    const int nr = min(max(ja, jb) + slack, w.H - 1) - w.j0 + 1;
    const int ncw = (min(max(ia, ib) + slack, W - 1) >> 6) - w.cw0 + 1;
#define NAVSIM_X(p, nw) return window_hops<p, nw>(fb, w, ia, ja, ib, jb, hi, lane, c, s_won, g_won);
    NAVSIM_PACKED_SHAPES(NAVSIM_X, ncw, nr)
#undef NAVSIM_X
}

// ---------------------------------------------------------------------------
// Labelling by one wavefront per start, for maps whose searches fit its
// registers: the levels of packed_level from the start, and for every cell that
// a level reaches one Philox word (the cell's random key in its bin), of which
// each bin keeps the smallest.  A level reaches a few cells of a few lanes, so
// they first go to a queue in LDS, one cell per lane and pass, and 64 at a time
// are drawn with every lane busy.  Bound by VALU issue: about 0.4 of it each in
// the draws and in the queue's passes, the rest in the levels.  16,384 starts on
// 64 maps of 256 x 256, 12 m: 29.1 -> 4.5 ms against a workgroup's search in LDS
// (a barrier per level, draws by the few threads that hold the level's words).
constexpr int kLabelQueue = 512;  // entries per wavefront: level << 16 | packed bit index
constexpr int kLabelWaves = 4;    // starts per workgroup
typedef __attribute__((address_space(3))) uint32_t LdsQueue;

template <int P, int NW>
__device__ __forceinline__ void label_window(const ReachParams &rp, const ReachDesc &d,
                                             const Window &w, int ia, int ja, uint32_t sid,
                                             int lane, LdsQueue *queue, int32_t *goal,
                                             int32_t *hops) {
    Words<NW> f0, f1, un0, un1;
    load_window<P, NW>(rp.packed + d.pk_off, w, un0, un1, lane);
    const int ca = (ia + ja) & 1, wa = (ja - w.j0) * P + (ia >> 6) - w.cw0;
    const uint32_t ba = 1u << ((ia >> 1) & 31);
#pragma unroll
    for (int j = 0; j < NW; ++j) {
        const uint32_t seed = wa == lane * NW + j ? ba : 0u;
        f0[j] = ca == 0 ? seed : 0u;
        f1[j] = ca == 0 ? 0u : seed;
        un0[j] &= ~f0[j];
        un1[j] &= ~f1[j];
    }
    const double s = (double)d.s;
    unsigned long long best = ~0ull, found = ~0ull;  // found: lane k holds bin k's result
    int head = 0, cnt = 0;                           // the queue's first entry and length
    // draws of the queue's first n <= 64 cells
    auto take = [&](int n) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const uint32_t code = queue[(head + lane) & (kLabelQueue - 1)];
        head = (head + n) & (kLabelQueue - 1);
        cnt -= n;
        if (lane >= n) return;
        const int wi = (int)(code & 0xffffu) >> 5, h = (int)(code >> 16);
        const int row = w.j0 + wi / P;
        const int col = 64 * (w.cw0 + wi % P) + 2 * (int)(code & 31u) + ((row + ca + h) & 1);
        const int cell = row * d.W + col;
        const double dx = (double)(col - ia) * s, dy = (double)(row - ja) * s;
        if (dx * dx + dy * dy < rp.gmd2) return;  // centre_dist below gmd
        uint32_t q[4] = {sid, (uint32_t)cell, 0u, 5u};
        philox4x32_10(q, rp.key0, rp.key1);
        const unsigned long long v = ((unsigned long long)q[0] << 32) |
                                     ((unsigned long long)cell << 16) | (unsigned long long)h;
        best = v < best ? v : best;
    };
    // the cells of a level that bin k counts, one per lane and pass
    auto put = [&](Words<NW> n, int level) {
        const uint32_t base = ((uint32_t)level << 16) + (uint32_t)(lane * NW * 32);
        uint32_t left;
        do {
            left = 0u;
#pragma unroll
            for (int j = 0; j < NW; ++j) {
                for (;;) {
                    const uint64_t m = __ballot(n[j] != 0u);
                    if (m == 0ull || cnt > kLabelQueue - 64) break;
                    if (n[j] != 0u) {
                        const int at = head + cnt +
                                       (int)__builtin_amdgcn_mbcnt_hi(
                                           (uint32_t)(m >> 32),
                                           __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                        queue[at & (kLabelQueue - 1)] =
                            base + (uint32_t)(32 * j) + (uint32_t)__builtin_ctz(n[j]);
                        n[j] &= n[j] - 1u;
                    }
                    cnt += __popcll(m);
                }
                left |= n[j];
            }
            while (cnt >= 64) take(64);
        } while (__ballot(left != 0u) != 0ull);
    };
    // the smallest key of bin k, kept by lane k
    auto close_bin = [&](int k) {
        if (k < 0) return;
        if (cnt > 0) take(cnt);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long v = __shfl_xor(best, o);
            best = v < best ? v : best;
        }
        if (lane == k) found = best;
        best = ~0ull;
    };
    int level = 0, k = -1;
    int next = rp.hop_bin[min(1, rp.max_hops)];  // bin of the next level, loaded a level ahead
    auto advance = [&](uint32_t any, const Words<NW> &nx) {
        ++level;
        const int b = __builtin_amdgcn_readfirstlane(next);
        next = rp.hop_bin[min(level + 1, rp.max_hops)];
        if (b != k) {
            close_bin(k);
            k = b;
        }
        if (__ballot(any != 0u) == 0ull) return false;
        if (b >= 0) put(nx, level);
        return level < rp.max_hops;
    };
    bool more = rp.max_hops > 0;
    if (more && ca == 1) more = advance(packed_level<P, NW, 0>(f1, f0, un0, lane), f0);
    while (more) {
        if (!advance(packed_level<P, NW, 1>(f0, f1, un1, lane), f1)) break;
        more = advance(packed_level<P, NW, 0>(f1, f0, un0, lane), f0);
    }
    close_bin(k);
    if (lane < rp.nbins) {
        goal[lane] = found == ~0ull ? -1 : (int32_t)((found >> 16) & 0xffffu);
        hops[lane] = found == ~0ull ? -1 : (int32_t)(found & 0xffffu);
    }
}

// Start i by wavefront i; starts on maps that the register search does not hold
// are left to label_kernel.
__global__ __launch_bounds__(64 * kLabelWaves) __attribute__((amdgpu_waves_per_eu(4)))
void label_wave_kernel(ReachParams rp, int n, const int32_t *map, uint32_t first_sid,
                       int32_t *start, int32_t *goal, int32_t *hops) {
    __shared__ uint32_t s_queue[kLabelWaves][kLabelQueue];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int i = (int)blockIdx.x * kLabelWaves + wave;
    if (i >= n) return;
    const int mk = __builtin_amdgcn_readfirstlane(map[i]);
    const bool known = mk >= 0 && mk < rp.num_maps;
    const ReachDesc d = rp.maps[known ? mk : 0];
    goal += (int64_t)i * rp.nbins;
    hops += (int64_t)i * rp.nbins;
    if (!known || d.free_cnt == 0) {
        if (lane < rp.nbins) {
            goal[lane] = -1;
            hops[lane] = -1;
        }
        if (lane == 0) start[i] = -1;
        return;
    }
    if (!d.label_ok) return;
    const uint32_t sid = first_sid + (uint32_t)i;
    uint32_t c[4] = {sid, 0u, 0u, 6u};
    philox4x32_10(c, rp.key0, rp.key1);
    const int a = __builtin_amdgcn_readfirstlane(
        rp.free_cells[d.free_off + pick_of(c[0], d.free_cnt)]);
    if (lane == 0) start[i] = a;
    const int ia = a % d.W, ja = a / d.W;
    Window w;
    w.H = d.H;
    w.pk = d.pk;
    w.pwords = d.pwords;
    w.j0 = max(ja - rp.max_hops, 0) & ~1;
    w.cw0 = max(ia - rp.max_hops, 0) >> 6;
    const int nr = min(ja + rp.max_hops, d.H - 1) - w.j0 + 1;
    const int ncw = (min(ia + rp.max_hops, d.W - 1) >> 6) - w.cw0 + 1;
    LdsQueue *queue = (LdsQueue *)s_queue[wave];
#define NAVSIM_X(p, nw) label_window<p, nw>(rp, d, w, ia, ja, sid, lane, queue, goal, hops);
    NAVSIM_PACKED_SHAPES(NAVSIM_X, ncw, nr)
#undef NAVSIM_X
}

// Packed bitsets of a map (both colours) into LDS, 16 bytes at a time.
__device__ __forceinline__ void stage_packed(const ReachParams &rp, const ReachDesc &d,
                                             uint4 *fb4) {
    const uint4 *g = reinterpret_cast<const uint4 *>(rp.packed + d.pk_off);
    for (int w = threadIdx.x; w < (2 * d.pwords + 3) / 4; w += blockDim.x) fb4[w] = g[w];
}

__device__ __forceinline__ bool packed_cell(const uint32_t *fb, const ReachDesc &d, int c) {
    const int i = c % d.W, j = c / d.W;
    return (fb[((i + j) & 1) * d.pwords + j * d.pk + (i >> 6)] >> ((i >> 1) & 31)) & 1u;
}

// Nearest C-free cell to c (least |di| + |dj|, then least index; -1 if none),
// by one wavefront: the cells of ring r split over the lanes, a ballot and a
// lane minimum.
__device__ int wave_snap(const ReachDesc &d, const uint32_t *fb, int c, int lane) {
    if (packed_cell(fb, d, c)) return c;
    const int i0 = c % d.W, j0 = c / d.W;
    for (int r = 1; r <= d.W + d.H; ++r) {
        int best = INT_MAX;
        for (int q = lane; q < 4 * r; q += 64) {
            const int side = q / r, t = q % r;
            const int di = side == 0 ? r - t : (side == 1 ? -t : (side == 2 ? t - r : t));
            const int dj = side == 0 ? t : (side == 1 ? r - t : (side == 2 ? -t : t - r));
            const int i = i0 + di, j = j0 + dj;
            if (i >= 0 && i < d.W && j >= 0 && j < d.H && packed_cell(fb, d, j * d.W + i))
                best = min(best, j * d.W + i);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) best = min(best, __shfl_xor(best, o));
        if (best != INT_MAX) return best;
    }
    return -1;
}

// The exact check of (a, b) for bin k by one wavefront (see check_pair).
__device__ int wave_check(const ReachParams &rp, const ReachDesc &d, const uint32_t *fb,
                          int a, int b, int k, int lane, int c = 0, const int *s_won = nullptr,
                          const int *g_won = nullptr) {
    if (a < 0 || b < 0 || !packed_cell(fb, d, a) || !packed_cell(fb, d, b)) return -1;
    if (centre_dist(d, a, b) < rp.gmd) return -1;
    const int hi = rp.bin_hi[k];
    int h;
    if (a == b) {
        h = 0;
    } else {
        const int man = abs(a % d.W - b % d.W) + abs(a / d.W - b / d.W);
        h = man > hi ? -1 : search_hops((LdsWord *)fb, d.W, d.H, d.pk, a, b, hi, c, (LdsInt *)s_won, g_won);
    }
    return (h >= 0 && rp.hop_bin[h] == k) ? h : -1;
}

// Candidate c of request i: network draw c < props (decoded, snapped), else
// rejection attempt c - props.  Returns the pair and the heading.
__device__ void candidate(const ReachParams &rp, const ProposeArgs &pa, const ReachDesc &d,
                          const uint32_t *fb, int i, int c, int lane, int &a, int &b,
                          float &th) {
    if (c < pa.props) {
        const float *y = pa.y + ((int64_t)i * pa.props + c) * 5;
        const int a0 = decode_axis(y[1], d.H) * d.W + decode_axis(y[0], d.W);
        const int b0 = decode_axis(y[4], d.H) * d.W + decode_axis(y[3], d.W);
        a = wave_snap(d, fb, a0, lane);
        b = wave_snap(d, fb, b0, lane);
        th = decode_heading(y[2]);
    } else {
        uint32_t q[4] = {pa.env[i], pa.episode[i], (uint32_t)(c - pa.props), 7u};
        philox4x32_10(q, rp.key0, rp.key1);
        a = rp.free_cells[d.free_off + pick_of(q[0], d.free_cnt)];
        b = rp.free_cells[d.free_off + pick_of(q[1], d.free_cnt)];
        th = (float)((((double)q[2] + 0.5) / kTwo32) * (2.0 * kPiR) - kPiR);
    }
}

// Proposals with one candidate per wavefront: candidates W r .. W r + W - 1
// (W wavefronts) are checked together and the lowest valid one wins, the
// result of checking them in order; `checks` counts as the sequential search
// does.
// Outputs of request i (row o): pair (a, b) and heading th, the winning
// candidate win (-1: none valid), its hop count h; checks as the sequential
// search counts them.
__device__ void write_request(const ProposeArgs &pa, const ReachDesc &d, int o, int win, int la,
                              int lb, int lh, float lth, int total) {
    float *p = pa.pose + (int64_t)o * 5;
    p[0] = la >= 0 ? cell_x(d, la) : 0.0f;
    p[1] = la >= 0 ? cell_y(d, la) : 0.0f;
    p[2] = lth;
    p[3] = lb >= 0 ? cell_x(d, lb) : 0.0f;
    p[4] = lb >= 0 ? cell_y(d, lb) : 0.0f;
    const int checks = win >= 0 ? win + 1 : total;
    if (pa.hops) pa.hops[o] = win >= 0 ? lh : -1;
    pa.source[o] = win;
    if (pa.checks) pa.checks[o] = checks;
    if (pa.stats) {
        atomicAdd(&pa.stats[0], 1ull);
        atomicAdd(&pa.stats[win < 0 ? 3 : (win < pa.props ? 1 : 2)], 1ull);
        atomicAdd(&pa.stats[4], (unsigned long long)checks);
    }
}

// W candidates c0 .. c0 + W - 1 of request i, one per wavefront; returns the
// lowest valid one (-1: none), with its pair, hop count and heading in the
// *_out arguments (every thread); with none valid and the request's last
// candidate (a rejection attempt) in this round, that attempt's pair and
// heading go there instead (the pair that stands when nothing is valid).
template <int W>
__device__ int check_round(const ReachParams &rp, const ProposeArgs &pa, const ReachDesc &d,
                           const uint32_t *fb, int i, int k, int c0, int total, int &a_out,
                           int &b_out, int &h_out, float &th_out, const int *g_won = nullptr) {
    __shared__ int s_ok[W], s_a[W], s_b[W], s_h[W];
    __shared__ float s_th[W];
    __shared__ int s_won;  // lowest candidate of the round found valid so far
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = c0 + wave;
    if (threadIdx.x == 0) s_won = INT_MAX;
    __syncthreads();
    int a = -1, b = -1, h = -1;
    float th = 0.0f;
    if (c < total) {
        candidate(rp, pa, d, fb, i, c, lane, a, b, th);
        // searches of higher candidates stop once a lower one has passed
        // (they cannot win); the winner and the check counts are unchanged
        h = wave_check(rp, d, fb, a, b, k, lane, c, &s_won, g_won);
        if (h >= 0 && lane == 0) atomicMin(&s_won, c);
    }
    if (lane == 0) {
        s_ok[wave] = (c < total && h >= 0) ? c : INT_MAX;
        s_a[wave] = a;
        s_b[wave] = b;
        s_h[wave] = h;
        s_th[wave] = th;
    }
    __syncthreads();
    int best = INT_MAX, bw = -1;
    for (int w = 0; w < W; ++w)
        if (s_ok[w] < best) {
            best = s_ok[w];
            bw = w;
        }
    int win = -1;
    if (bw >= 0) {
        win = best;
        a_out = s_a[bw];
        b_out = s_b[bw];
        h_out = s_h[bw];
        th_out = s_th[bw];
    } else if (total - 1 >= c0 && total - 1 < c0 + W && total - 1 >= pa.props) {
        // none valid: the last rejection attempt's pair stands
        const int w = total - 1 - c0;
        a_out = s_a[w];
        b_out = s_b[w];
        th_out = s_th[w];
    }
    __syncthreads();
    return win;
}

template <int W>
__device__ void propose_waves(const ReachParams &rp, const ProposeArgs &pa, const ReachDesc &d,
                              const uint32_t *fb, int i, int o, int k) {
    const int total = pa.props + (d.free_cnt > 0 ? pa.tries : 0);
    int win = -1, la = -1, lb = -1, lh = -1;
    float lth = 0.0f;
    int c0 = 0;
    for (int round = 0; c0 < total && win < 0; c0 += W, ++round) {
        if (pa.head_rounds > 0 && round == pa.head_rounds) {
            // the rest of this request's rounds go to the tail launch
            if (threadIdx.x == 0) {
                if (pa.n_pend) {
                    const int p = atomicAdd(pa.n_pend, 1);
                    pa.pend[p] = i;
                    pa.best[p] = INT_MAX;
                } else {
                    pa.checks[o] = -1;  // pending, see propose_tail_own_kernel
                    pa.source[o] = INT_MAX;
                    pa.hops[o] = -1;
                }
            }
            return;
        }
        win = check_round<W>(rp, pa, d, fb, i, k, c0, total, la, lb, lh, lth);
    }
    if (threadIdx.x == 0) write_request(pa, d, o, win, la, lb, lh, lth, total);
}

// One workgroup of W wavefronts per request.
template <int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4)))
void propose_kernel(ReachParams rp, ProposeArgs pa) {
    extern __shared__ uint4 lds4[];  // 16-byte aligned: the searches clear it 16 bytes at a time
    uint32_t *lds = reinterpret_cast<uint32_t *>(lds4);
    __shared__ int s_min;
    const int i = blockIdx.x, tid = threadIdx.x;
    if (pa.n_dev && i >= *pa.n_dev) return;  // past the requests counted on the device
    const int o = pa.slot ? pa.slot[i] : i;    // output row
    const int mk = pa.map[i], k = pa.bin[i];
    if (mk < 0 || mk >= rp.num_maps || k < 0 || k >= rp.nbins) {  // rejected request
        if (tid < 5) pa.pose[(int64_t)o * 5 + tid] = 0.0f;
        if (tid == 0) {
            if (pa.hops) pa.hops[o] = -1;
            pa.source[o] = -1;
            if (pa.checks) pa.checks[o] = 0;
            if (pa.stats) {
                atomicAdd(&pa.stats[0], 1ull);
                atomicAdd(&pa.stats[3], 1ull);
            }
        }
        return;
    }
    const ReachDesc d = rp.maps[mk];
    uint32_t *fb = lds, *vis = fb + kReachMaxWords, *fr = vis + kReachMaxWords,
             *nx = fr + kReachMaxWords;
    if (d.pair_ok) {  // searches in registers
        stage_packed(rp, d, lds4);
        __syncthreads();
        propose_waves<W>(rp, pa, d, lds, i, o, k);
        return;
    }
    stage_free(rp, d, fb);
    __syncthreads();
    int checks = 0, src = -1, ra = -1, rb = -1, rh = -1;
    float th = 0.0f;
    for (int j = 0; j < pa.props && src < 0; ++j) {
        const float *y = pa.y + ((int64_t)i * pa.props + j) * 5;
        const int a0 = decode_axis(y[1], d.H) * d.W + decode_axis(y[0], d.W);
        const int b0 = decode_axis(y[4], d.H) * d.W + decode_axis(y[3], d.W);
        const int a = snap_cell(d, fb, a0, &s_min);
        const int b = snap_cell(d, fb, b0, &s_min);
        ++checks;
        const int h = check_pair(rp, d, fb, vis, fr, nx, a, b, k);
        if (h >= 0) {
            src = j;
            ra = a;
            rb = b;
            rh = h;
            th = decode_heading(y[2]);
        }
    }
    for (int t = 0; t < pa.tries && src < 0 && d.free_cnt > 0; ++t) {
        uint32_t c[4] = {pa.env[i], pa.episode[i], (uint32_t)t, 7u};
        philox4x32_10(c, rp.key0, rp.key1);
        const int a = rp.free_cells[d.free_off + pick_of(c[0], d.free_cnt)];
        const int b = rp.free_cells[d.free_off + pick_of(c[1], d.free_cnt)];
        ++checks;
        const int h = check_pair(rp, d, fb, vis, fr, nx, a, b, k);
        ra = a;
        rb = b;
        th = (float)((((double)c[2] + 0.5) / kTwo32) * (2.0 * kPiR) - kPiR);
        if (h >= 0) {
            src = pa.props + t;
            rh = h;
        }
    }
    if (tid == 0) {
        float *p = pa.pose + (int64_t)o * 5;
        p[0] = ra >= 0 ? cell_x(d, ra) : 0.0f;
        p[1] = ra >= 0 ? cell_y(d, ra) : 0.0f;
        p[2] = th;
        p[3] = rb >= 0 ? cell_x(d, rb) : 0.0f;
        p[4] = rb >= 0 ? cell_y(d, rb) : 0.0f;
        if (pa.hops) pa.hops[o] = rh;
        pa.source[o] = src;
        if (pa.checks) pa.checks[o] = checks;
        if (pa.stats) {
            atomicAdd(&pa.stats[0], 1ull);
            atomicAdd(&pa.stats[src < 0 ? 3 : (src < pa.props ? 1 : 2)], 1ull);
            atomicAdd(&pa.stats[4], (unsigned long long)checks);
        }
    }
}

__global__ __launch_bounds__(1024) void compact_kernel(CompactArgs a) {
    // each thread takes 16 consecutive envs per pass (one 16-byte load of
    // their flags; bins read only for the flagged ones), and a workgroup
    // prefix sum of the per-thread counts places them in env order
    __shared__ int s_wave[16];
    __shared__ int s_base;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) {
        s_base = 0;
        if (a.n_pend) *a.n_pend = 0;
    }
    __syncthreads();
    const bool vec = (reinterpret_cast<uintptr_t>(a.defer) & 15u) == 0u;
    for (int e0 = 0; e0 < a.N; e0 += 1024 * 16) {
        const int eb = e0 + tid * 16;
        uint32_t m = 0u;  // bit i: env eb + i asks for a pair
        if (vec && eb + 16 <= a.N) {
            const uint4 v = *reinterpret_cast<const uint4 *>(a.defer + eb);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if ((w[q] >> (8 * b)) & 0xffu) m |= 1u << (4 * q + b);
        } else {
            for (int i = 0; i < 16; ++i)
                if (eb + i < a.N && a.defer[eb + i] != 0) m |= 1u << i;
        }
        for (uint32_t r = m; r != 0u; r &= r - 1u) {
            const int i = (int)__builtin_ctz(r);
            if (a.bin[eb + i] < 0) m &= ~(1u << i);
        }
        const int cnt = __popc(m);
        int inc = cnt;  // inclusive prefix sum over the wavefront
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int t = __shfl_up(inc, o);
            if (lane >= o) inc += t;
        }
        if (lane == 63) s_wave[wave] = inc;
        __syncthreads();
        int before = s_base, total = 0;
        for (int w = 0; w < 16; ++w) {
            const int c = s_wave[w];
            before += w < wave ? c : 0;
            total += c;
        }
        int pos = before + inc - cnt;
        for (uint32_t r = m; r != 0u; r &= r - 1u, ++pos) {
            const int e = eb + (int)__builtin_ctz(r);
            a.src[e] = -1;
            if (pos < a.cap) {
                a.env[pos] = (uint32_t)e;
                a.map[pos] = a.env_map[e];
                a.rbin[pos] = a.bin[e];
                a.episode[pos] = a.ep[e];
            }
        }
        __syncthreads();
        if (tid == 0) s_base += total;
        __syncthreads();
    }
    if (tid == 0) {
        const int count = s_base;
        *a.n_out = count < a.cap ? count : a.cap;
        if (a.stats) {
            atomicAdd(&a.stats[0], (unsigned long long)count);
            atomicAdd(&a.stats[1], (unsigned long long)(count > a.cap ? count - a.cap : 0));
        }
    }
}

__global__ void noise_kernel(NoiseArgs a, uint32_t key0, uint32_t key1) {
    const int nq = (a.nz + 3) / 4;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (a.clear && idx == 0) *a.clear = 0;
    const int n = a.n_dev ? min(a.n, *a.n_dev) : a.n;
    const int64_t rows = (int64_t)n * a.per;
    if (idx >= rows * nq) return;
    const int64_t r = idx / nq;
    const int q = (int)(idx % nq);
    const int i = (int)(r / a.per), j = (int)(r % a.per);
    uint32_t c[4] = {a.c0 ? a.c0[i] : (uint32_t)i, a.c1 ? a.c1[i] : a.c1_const,
                     ((uint32_t)j << 8) | (uint32_t)q, a.stream};
    philox4x32_10(c, key0, key1);
    for (int t = 0; t < 4; ++t) {
        const int col = 4 * q + t;
        if (col < a.nz) {
            const double u = ((double)c[t] + 0.5) / kTwo32;
            a.z[r * a.nz + col] = bf16_bits((float)(2.0 * u - 1.0));
        }
    }
    if (q == 0 && a.row_idx) {
        const int m = a.map[i], b = a.bin[i];
        a.row_idx[r] = (m >= 0 && m < a.num_maps && b >= 0 && b < a.nbins) ? m * a.nbins + b : 0;
    }
}

__global__ void pool_rows_kernel(int num_maps, int nbins, const float *pool, uint16_t *rows) {
    const int width = kPoolCells + nbins;
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)num_maps * nbins * width) return;
    const int64_t row = idx / width;
    const int col = (int)(idx % width);
    const int m = (int)(row / nbins), b = (int)(row % nbins);
    const float v = col < kPoolCells ? pool[(int64_t)m * kPoolCells + col]
                                     : (col - kPoolCells == b ? 1.0f : 0.0f);
    rows[idx] = bf16_bits(v);
}

__global__ void batch_kernel(BatchArgs a, uint32_t key0, uint32_t key1) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.batch) return;
    uint32_t c[4] = {a.step, (uint32_t)i, 0u, 10u};
    philox4x32_10(c, key0, key1);
    const int p = pick_of(c[0], a.num_pairs);
    int m = a.pair_map[p], b = a.pair_bin[p];
    const bool ok_mb = m >= 0 && m < a.num_maps && b >= 0 && b < a.nbins;
    const ReachDesc d = a.maps[ok_mb ? m : 0];
    int s = a.pair_start[p], g = a.pair_goal[p];
    const int cells = d.W * d.H;
    float *t = a.target + (int64_t)i * 5;
    if (!ok_mb || s < 0 || s >= cells || g < 0 || g >= cells) {
        a.map[i] = 0;
        a.bin[i] = 0;
        for (int q = 0; q < 5; ++q) t[q] = 0.0f;
        return;
    }
    a.map[i] = m;
    a.bin[i] = b;
    t[0] = (float)(((double)(s % d.W) + 0.5) / (double)d.W);
    t[1] = (float)(((double)(s / d.W) + 0.5) / (double)d.H);
    t[2] = 0.0f;
    t[3] = (float)(((double)(g % d.W) + 0.5) / (double)d.W);
    t[4] = (float)(((double)(g / d.W) + 0.5) / (double)d.H);
}

// One workgroup per target, one thread per draw (per <= 256).  The choice is the
// sequential scan's: draw 0 unless a later one is smaller (the first such on
// ties); a distance that is no number loses to every other, and stands when it
// is draw 0's.  1,024 targets of 128 draws: 31 us with one thread scanning a
// target's draws, 5.5 us (a launch) now.
__global__ __launch_bounds__(256) void select_kernel(SelectArgs a) {
    __shared__ unsigned long long s_best[4];
    __shared__ int s_j;
    const int i = blockIdx.x, tid = threadIdx.x;
    unsigned long long best = ~0ull;
    bool stays = false;
    if (tid < a.per) {
        const float *t = a.target + (int64_t)i * 5;
        const float *y = a.y + ((int64_t)i * a.per + tid) * 5;
        float dsum = 0.0f;
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            const float e = y[q] - t[q];
            dsum += a.w[q] * (e * e);
        }
        stays = tid == 0 && dsum != dsum;
        // dsum >= +0, so its bits order like its value
        const uint32_t bits = dsum != dsum ? 0x7f800000u : __float_as_uint(dsum);
        best = ((unsigned long long)bits << 32) | (unsigned long long)tid;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long v = __shfl_xor(best, o);
        best = v < best ? v : best;
    }
    if ((tid & 63) == 0) s_best[tid >> 6] = best;
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w) best = s_best[w] < best ? s_best[w] : best;
        s_j = stays ? 0 : (int)(best & 0xffffffffull);
        if (a.chosen) a.chosen[i] = s_j;
    }
    __syncthreads();
    const int j = s_j;
    const int width = kPoolCells + a.nbins + a.nz;
    const int m = a.map[i], b = a.bin[i];
    uint16_t *x = a.x + (int64_t)i * width;
    const uint16_t *z = a.z + ((int64_t)i * a.per + j) * a.nz;
    for (int col = tid; col < width; col += blockDim.x) {
        uint16_t v;
        if (col < kPoolCells)
            v = bf16_bits(a.pool[(int64_t)m * kPoolCells + col]);
        else if (col < kPoolCells + a.nbins)
            v = bf16_bits(col - kPoolCells == b ? 1.0f : 0.0f);
        else
            v = z[col - kPoolCells - a.nbins];
        x[col] = v;
    }
}

unsigned nblocks(int64_t n, int t) { return (unsigned)((n + t - 1) / t); }

constexpr size_t kSearchLds = 4u * kReachMaxWords * sizeof(uint32_t);

// LDS of the proposal kernels: the packed bitsets of the largest map; the LDS
// search's four bitsets when some map needs it.
size_t propose_lds(const ReachParams &rp) {
    const size_t packed = (2u * (size_t)rp.max_pwords + 3u) / 4u * 16u;
    return rp.all_pair ? packed : std::max(packed, kSearchLds);
}

}  // namespace

hipError_t launch_label(const ReachParams &rp, int n, const int32_t *map, uint32_t first_sid,
                        int32_t *start, int32_t *goal, int32_t *hops, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    if (rp.any_label) {
        hipLaunchKernelGGL(label_wave_kernel, dim3(nblocks(n, kLabelWaves)), dim3(64 * kLabelWaves),
                           0, s, rp, n, map, first_sid, start, goal, hops);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || rp.all_label) return e;
    }
    hipLaunchKernelGGL(label_kernel, dim3((unsigned)n), dim3(kReachThreads), kSearchLds, s, rp,
                       map, first_sid, start, goal, hops);
    return hipGetLastError();
}

// Tail round r of pending request i by one workgroup: the lowest valid candidate
// of the round with its pair, hop count and heading, or -1; a round that starts
// above a valid candidate already found (*best) is skipped, it cannot win.
template <int W>
__device__ __forceinline__ int tail_round(const ReachParams &rp, const ProposeArgs &pa, uint4 *lds4,
                                          int i, int r, const int *best, int &a, int &b, int &h,
                                          float &th) {
    __shared__ int s_skip;
    const int mk = pa.map[i], k = pa.bin[i];
    const ReachDesc d = rp.maps[mk];
    const int total = pa.props + (d.free_cnt > 0 ? pa.tries : 0);
    const int c0 = (pa.head_rounds + r) * W;
    // uniform across the workgroup: one read of *best, then a barrier before any
    // thread moves on
    if (threadIdx.x == 0) s_skip = c0 >= total || __atomic_load_n(best, __ATOMIC_RELAXED) < c0;
    __syncthreads();
    const bool skip = s_skip != 0;
    __syncthreads();
    if (skip) return -1;
    stage_packed(rp, d, lds4);
    __syncthreads();
    return check_round<W>(rp, pa, d, reinterpret_cast<uint32_t *>(lds4), i, k, c0, total, a, b, h,
                          th, best);
}

// Tail rounds: every (pending request, round) is one work item, taken by the
// workgroups of a fixed grid in round-major order (all requests' first tail
// round, then their second, ...), so a request's rounds run at once on
// different workgroups.  A round's lowest valid candidate goes to its slot and
// into the request's best index (atomic minimum).  Requests reach the pending
// list only from the register search, so the same path serves.
template <int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4)))
void propose_tail_kernel(ReachParams rp, ProposeArgs pa, int tail_rounds) {
    extern __shared__ uint4 lds4[];
    const int np = *pa.n_pend;
    const int items = np * tail_rounds;
    for (int g = blockIdx.x; g < items; g += gridDim.x) {
        const int p = g % np, r = g / np;
        int a = -1, b = -1, h = -1;
        float th = 0.0f;
        const int win = tail_round<W>(rp, pa, lds4, pa.pend[p], r, &pa.best[p], a, b, h, th);
        if (threadIdx.x == 0 && win >= 0) {
            pa.tail[(int64_t)p * tail_rounds + r] = make_int4(a, b, h, __float_as_int(th));
            atomicMin(&pa.best[p], win);
        }
        __syncthreads();  // the map in LDS is restaged by the next item
    }
}

// The same for a call of the rejection sampler alone, which has no workspace: a
// pending request's state lies in its own output rows until the final launch.
// checks is -1; source holds the lowest valid attempt found so far, or INT_MAX;
// hops, unsigned, that attempt's number << 16 | its hop count (both below 2^16).
// The pair and heading come from the attempt's number again.  Every workgroup
// looks through the marks itself and lists the pending requests in order, so all
// agree on the items' numbers (marks change only in the final launch).  A call thus
// allocates nothing, may be captured first and may overlap any other.
template <int W>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(4)))
void propose_tail_own_kernel(ReachParams rp, ProposeArgs pa, int tail_rounds) {
    extern __shared__ uint4 lds4[];
    constexpr int T = 64 * W, N = W == 8 ? kProposeWideMax : kOwnTailMax;
    static_assert(N % (4 * T) == 0 && N <= 1 << 16, "4 requests a thread and pass");
    __shared__ uint16_t s_req[N];
    __shared__ int s_cnt[N / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // ballots of the marks of requests q + j T .., their loads together
    const auto pending = [&](int q, uint64_t(&m)[4]) {
        int c[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) c[j] = pa.checks[min(q + j * T + tid, pa.n - 1)];
#pragma unroll
        for (int j = 0; j < 4; ++j) m[j] = __ballot(q + j * T + tid < pa.n && c[j] == -1);
    };
    uint64_t m[4];
    for (int q = 0; q < pa.n; q += 4 * T) {
        pending(q, m);
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (lane == 0) s_cnt[(q >> 6) + j * W + wave] = __popcll(m[j]);
    }
    __syncthreads();
    int np = 0;
    for (int q = 0; q < pa.n; q += 4 * T) {
        pending(q, m);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            int at = np;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int c = s_cnt[(q >> 6) + j * W + w];
                at += w < wave ? c : 0;
                np += c;
            }
            if ((m[j] >> lane) & 1ull)
                s_req[at + __popcll(m[j] & ((1ull << lane) - 1ull))] = (uint16_t)(q + j * T + tid);
        }
    }
    __syncthreads();
    const int items = np * tail_rounds;
    for (int g = blockIdx.x; g < items; g += gridDim.x) {
        const int i = s_req[g % np];
        int a = -1, b = -1, h = -1;
        float th = 0.0f;
        const int win = tail_round<W>(rp, pa, lds4, i, g / np, &pa.source[i], a, b, h, th);
        if (tid == 0 && win >= 0) {
            atomicMin(&pa.source[i], win);
            atomicMin(reinterpret_cast<uint32_t *>(&pa.hops[i]),
                      ((uint32_t)win << 16) | (uint32_t)h);
        }
        __syncthreads();  // the map in LDS is restaged by the next item
    }
}

// Pair and heading of rejection attempt t of request i.
__device__ void attempt_pair(const ReachParams &rp, const ProposeArgs &pa, const ReachDesc &d,
                             int i, int t, int &a, int &b, float &th) {
    uint32_t q[4] = {pa.env[i], pa.episode[i], (uint32_t)t, 7u};
    philox4x32_10(q, rp.key0, rp.key1);
    a = rp.free_cells[d.free_off + pick_of(q[0], d.free_cnt)];
    b = rp.free_cells[d.free_off + pick_of(q[1], d.free_cnt)];
    th = (float)((((double)q[2] + 0.5) / kTwo32) * (2.0 * kPiR) - kPiR);
}

// Outputs of the pending requests: the lowest valid candidate any tail round
// found, else the last rejection attempt's pair (as the sequential search).
__global__ void propose_final_kernel(ReachParams rp, ProposeArgs pa, int tail_rounds, int W) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= *pa.n_pend) return;
    const int i = pa.pend[p], o = pa.slot ? pa.slot[i] : i;
    const ReachDesc d = rp.maps[pa.map[i]];
    const int total = pa.props + (d.free_cnt > 0 ? pa.tries : 0);
    const int win = pa.best[p] == INT_MAX ? -1 : pa.best[p];
    int la = -1, lb = -1, lh = -1;
    float lth = 0.0f;
    if (win >= 0) {
        const int4 q = pa.tail[(int64_t)p * tail_rounds + win / W - pa.head_rounds];
        la = q.x;
        lb = q.y;
        lh = q.z;
        lth = __int_as_float(q.w);
    } else if (total - 1 >= pa.props) {
        attempt_pair(rp, pa, d, i, total - 1 - pa.props, la, lb, lth);
    }
    write_request(pa, d, o, win, la, lb, lh, lth, total);
}

__global__ void propose_final_own_kernel(ReachParams rp, ProposeArgs pa) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= pa.n || pa.checks[i] != -1) return;
    const ReachDesc d = rp.maps[pa.map[i]];
    const int win = pa.source[i] == INT_MAX ? -1 : pa.source[i];
    const int lh = (int)((uint32_t)pa.hops[i] & 0xffffu);
    int la, lb;
    float lth;
    attempt_pair(rp, pa, d, i, win >= 0 ? win : pa.tries - 1, la, lb, lth);
    write_request(pa, d, i, win, la, lb, lh, lth, pa.tries);
}

int propose_width(int n) { return n <= kProposeWideMax ? 8 : 4; }

// 8,192 requests, 32 draws and 64 attempts, with 1, 2, 3 and 6 head rounds of 4:
// 1,521, 1,455, 1,423 and 1,454 us (1,497 with every round in one launch; 3,000
// requests 735 against 1,023 us).
int propose_head_rounds(int n) { return n <= kProposeWideMax ? 1 : 3; }

hipError_t launch_propose_tail(const ReachParams &rp, const ProposeArgs &a, int tail_rounds,
                               hipStream_t s) {
    if (a.n <= 0 || tail_rounds <= 0) return hipSuccess;
    // a fixed grid: the pending count is only known on the device
    const unsigned g = (unsigned)std::min<int64_t>((int64_t)a.n * tail_rounds, 1024);
    const int W = propose_width(a.n);
    const dim3 grid(g), block(64 * W);
    if (!a.n_pend) {
        if (a.n > kOwnTailMax) return hipErrorInvalidValue;
        if (W == 8)
            hipLaunchKernelGGL(propose_tail_own_kernel<8>, grid, block, propose_lds(rp), s, rp, a,
                               tail_rounds);
        else
            hipLaunchKernelGGL(propose_tail_own_kernel<4>, grid, block, propose_lds(rp), s, rp, a,
                               tail_rounds);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(propose_final_own_kernel, dim3(nblocks(a.n, 256)), dim3(256), 0, s, rp, a);
        return hipGetLastError();
    }
    if (W == 8)
        hipLaunchKernelGGL(propose_tail_kernel<8>, dim3(g), dim3(512), propose_lds(rp), s, rp, a,
                           tail_rounds);
    else
        hipLaunchKernelGGL(propose_tail_kernel<4>, dim3(g), dim3(256), propose_lds(rp), s, rp, a,
                           tail_rounds);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(propose_final_kernel, dim3(nblocks(a.n, 256)), dim3(256), 0, s, rp, a,
                       tail_rounds, W);
    return hipGetLastError();
}

hipError_t launch_propose(const ReachParams &rp, const ProposeArgs &a, hipStream_t s) {
    if (a.n <= 0) return hipSuccess;
    // few requests (a step's resets): 8 candidates at a time shortens the
    // slowest requests, which set the launch's time; many (a batch): 4, fewer
    // checks past the first valid candidate
    if (propose_width(a.n) == 8)
        hipLaunchKernelGGL(propose_kernel<8>, dim3((unsigned)a.n), dim3(512), propose_lds(rp), s, rp, a);
    else
        hipLaunchKernelGGL(propose_kernel<4>, dim3((unsigned)a.n), dim3(256), propose_lds(rp), s, rp, a);
    return hipGetLastError();
}

hipError_t launch_compact(const CompactArgs &a, hipStream_t s) {
    hipLaunchKernelGGL(compact_kernel, dim3(1), dim3(1024), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_noise(const NoiseArgs &a, uint32_t key0, uint32_t key1, hipStream_t s) {
    const int64_t total = (int64_t)a.n * a.per * ((a.nz + 3) / 4);
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(noise_kernel, dim3(nblocks(total, 256)), dim3(256), 0, s, a, key0, key1);
    return hipGetLastError();
}

hipError_t launch_pool_rows(int num_maps, int nbins, const float *pool, uint16_t *rows,
                            hipStream_t s) {
    const int64_t total = (int64_t)num_maps * nbins * (kPoolCells + nbins);
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(pool_rows_kernel, dim3(nblocks(total, 256)), dim3(256), 0, s, num_maps,
                       nbins, pool, rows);
    return hipGetLastError();
}

hipError_t launch_batch(const BatchArgs &a, uint32_t key0, uint32_t key1, hipStream_t s) {
    if (a.batch <= 0) return hipSuccess;
    hipLaunchKernelGGL(batch_kernel, dim3(nblocks(a.batch, 256)), dim3(256), 0, s, a, key0, key1);
    return hipGetLastError();
}

hipError_t launch_select(const SelectArgs &a, hipStream_t s) {
    if (a.batch <= 0) return hipSuccess;
    hipLaunchKernelGGL(select_kernel, dim3((unsigned)a.batch), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace navsim
