// mr_ccl.hip -- connected components labeling (union-find) and area threshold
// (map + reduction), Table II; mr_ccl and mr_area_threshold in
// include/mr_ops.h.
//
// Union-find as Sec. II-B describes it: every foreground pixel starts as its
// own tree, trees of adjacent foreground pixels are merged with the smaller
// root becoming the root of the merged tree, and the labels are read from
// the flattened forest. Here a pixel's value in the forest is its linear
// index y * W + x, so every root is the smallest index of its tree and the
// labels (root + 1) do not depend on the order of the merges.
//
// The GPU version follows Sec. III-B's split, on horizontal runs instead of
// pixels: each 64 x 64 tile is merged by one wave in LDS (k_ccl_local: lane =
// row, a row's foreground is one 64-bit mask), then the trees that cross tile
// borders are merged in the global forest with device atomics (k_ccl_merge),
// and finally every pixel gets its run's root (k_ccl_write). The passes move
// what they must and little more: the image is read once (1 byte a pixel),
// the labels are written once (4 bytes a pixel), and between the passes only
// the row masks (1 bit a pixel) and the forest entries of the runs travel.
// The forest lives in the workspace and holds parent index + 1 for the
// pixels later steps look at: every run's first pixel (runs are cut at tile
// borders), and the foreground pixels of a tile's first row, last row and
// last column. All other entries are undefined. The row masks live in the
// label plane until the last pass: a tile's masks sit in the tile's own
// labels, which only that tile's wave reads (its masks first) and then writes.
// A merge links the larger of two roots below the smaller
// with an atomic minimum on the larger's parent; if another merge got there
// first, the atomic returns the new parent and the merge goes on from it.
// Parents stay below their children, so every walk ends at a root.
//
// Area threshold: the map step reads each pixel's label; the reduction counts
// pixels per label with device atomic adds into one counter per possible
// label (the workspace), adding a lane's run of equal labels in one atomic;
// the filter clears every pixel whose label's count is out of range.
#include <algorithm>
#include <cstdarg>
#include <cstdio>

#include "../../include/mr_ops.h"
#include "mr_internal.h"

using namespace mr;

namespace {

int cfail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return set_error(code, buf);
}

int chip(hipError_t e, const char *what) {
    return cfail(MR_EHIP, "%s: %s", what, hipGetErrorString(e));
}

size_t up256(size_t n) { return (n + 255) / 256 * 256; }

constexpr int CT = 64;              // tile side: a row is one 64-bit mask, lane = row
constexpr int CT_RUNS = CT / 2;     // a row holds at most this many runs
constexpr int CT_NODES = CT_RUNS + 1; // a row's nodes, one unused: rows lie a bank apart
constexpr int CT_WAVES = 4;         // tiles (waves) per workgroup
// Fewer tiles than this: a workgroup each, so that every CU gets one, and the
// last pass takes CT_WAVES waves a tile. 2048 x 2048 (1024 tiles), label and area
// threshold: 36.1 us so, 38.4 us with four tiles a workgroup; 4096 x 2048 the same
// (46.1 us); 16384 x 16384 (65536 tiles) 742 us so, 695 us with four.
constexpr uint32_t CT_FEW = 2048;
constexpr int WALKS = 4;            // walks to a root that a lane of the last pass makes at once
constexpr int CT_DENSE = 4;         // runs of a row above which a tile's workgroup shares it
constexpr uint32_t RANK = 1u << 31; // there: a place in the run list, not a label (below 2^31)

// ------------------------------------------------------------- local phase

// LDS handed between the lanes of one wave: program order and a compiler
// barrier (each wave works on its own part of the workgroup's LDS).
__device__ __forceinline__ void ccl_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ uint32_t lds_load(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The root of x's tree in the tile's LDS forest. Each second node passed is put below
// its parent's parent (plain stores, see gfind).
__device__ __forceinline__ uint32_t lfind(uint32_t *P, uint32_t x) {
    uint32_t p = lds_load(P + x);
    while (p != x) {
        const uint32_t g = lds_load(P + p);
        if (g == p) return p;
        __hip_atomic_store(P + x, g, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        x = g;
        p = lds_load(P + x);
    }
    return x;
}

// Merge the trees of a and b in the tile's LDS forest: the larger root goes
// below the smaller one.
__device__ __forceinline__ void lunion(uint32_t *P, uint32_t a, uint32_t b) {
    while (true) {
        a = lfind(P, a);
        b = lfind(P, b);
        if (a == b) return;
        if (a > b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        const uint32_t old = atomicMin(P + b, a);
        if (old == b) return; // b was still a root: linked
        b = old;              // b was linked meanwhile: go on from its parent
    }
}

// The run of a row (mask m) that holds column x: its first column.
__device__ __forceinline__ int run_start(uint64_t m, int x) {
    const uint64_t z = ~m & ((1ull << x) - 1);
    return z ? 64 - __builtin_clzll(z) : 0;
}

// A tile's run is a node of its LDS forest: its row and half its first
// column (two runs of a row start at least two columns apart). Nodes are
// ordered like the runs' first pixels.
__device__ __forceinline__ uint32_t run_node(int row, uint64_t m, int x) {
    return (uint32_t)(row * CT_NODES + (run_start(m, x) >> 1));
}

// The tile of this wave: its place and size in the image (32-bit: H * W is
// below 2^31).
struct CclTile {
    uint32_t y0, x0, h, w, nw; // nw: 32-bit words that hold a row's mask
    uint32_t first;            // linear index of its first pixel
    __device__ CclTile(uint32_t t, uint32_t tiles_x, uint32_t H, uint32_t W) {
        const uint32_t ty = t / tiles_x, tx = t - ty * tiles_x;
        y0 = ty * CT;
        x0 = tx * CT;
        h = std::min<uint32_t>(CT, H - y0);
        w = std::min<uint32_t>(CT, W - x0);
        nw = w > 32 ? 2 : 1;
        first = y0 * W + x0;
    }
    // Word j of the tile's masks (row j / nw), kept in the tile's own labels.
    __device__ uint32_t *word(uint32_t *labels, int64_t lpitch, uint32_t j) const {
        const uint32_t r = w == CT ? j >> 6 : j / w;
        return labels + (int64_t)(y0 + r) * lpitch + x0 + (j - r * w);
    }
    __device__ uint64_t mask(uint32_t *labels, int64_t lpitch, uint32_t row) const {
        if (nw == 1) return *word(labels, lpitch, row);
        return *word(labels, lpitch, 2 * row) |
               (uint64_t)*word(labels, lpitch, 2 * row + 1) << 32;
    }
};

// The unions of one tile from its row masks, by TW waves (thread th of them), and its
// forest entries. A thread has a row (TW = 1), or those runs of a row that begin in
// 16 of its columns. A run makes one union per run above it that it touches, made at the
// first pixel that reaches that run: with 4-connectivity a common column
// whose left neighbour is not common; with 8-connectivity a run's first pixel
// takes the run above it or above-left of it, and every later pixel only the
// run that begins above-right of it.
// A run's first union takes no atomic: the run is put below the run above it,
// and the chains that this makes down the tile's rows are halved three times (by four
// waves once: 300 x 411 pixels, half foreground at random, 15 us, 19 us when halved until
// they were flat) before they are walked (512 x 3712 pixels, 20 % foreground: 7.0 us,
// 15.8 us with every union by walk and atomic minimum).
template <int CONN, int TW>
__device__ __forceinline__ void ccl_tile(const CclTile &T, uint32_t W, int th, uint32_t *P,
                                         const uint64_t *row_of, uint32_t *__restrict__ F) {
    auto sync = [] {
        if (TW == 1) ccl_wave_sync();
        else __syncthreads();
    };
    const int row = TW == 1 ? th : th >> 2;
    const uint64_t mine = TW == 1 ? ~0ull : 0xFFFFull << (16 * (th & 3));
    const uint64_t m = row_of[row];
    const uint64_t up = row > 0 ? row_of[row - 1] : 0ull;
    const uint64_t first = m & ~(m << 1); // the runs' first pixels
    const uint64_t s = first & mine;
    // Columns at which a run makes a union: with the run above at the column
    // itself (uC), or above-left (uL) or above-right (uR) of it.
    uint64_t uC, uL = 0, uR = 0;
    if (CONN == 4) {
        uC = m & up;
        uC &= ~(uC << 1);
    } else {
        uL = first & (up << 1);
        uC = first & up & ~(up << 1);
        uR = m & (up >> 1) & ~up;
    }
    // the node of the run above that column x unites with (first: at x itself or
    // to its left, else to its right)
    auto above = [&](int x, bool right) -> uint32_t {
        return run_node(row - 1, up, right ? x + 1 : ((uL >> x) & 1) ? x - 1 : x);
    };
    // A run starts below the first run it unites with, which takes no atomic; the
    // chains this makes down the rows are halved before anyone
    // walks them; what a run touches besides is united then.
    const uint64_t at = uC | uL;
    uint64_t left = 0, right = 0; // what is left to unite
    for (uint64_t u = s; u; u &= u - 1) {
        const int x = __builtin_ctzll(u);
        const uint32_t node = (uint32_t)(row * CT_NODES + (x >> 1));
        // this run's columns
        const uint64_t gap = ~m & ~((2ull << x) - 1);
        const uint64_t run = (gap ? (gap & -gap) - 1 : ~0ull) & ~((1ull << x) - 1);
        uint64_t l = at & run, r = uR & run;
        uint32_t parent = node;
        if (l) {
            parent = above(__builtin_ctzll(l), false);
            l &= l - 1;
        } else if (r) {
            parent = above(__builtin_ctzll(r), true);
            r &= r - 1;
        }
        left |= l;
        right |= r;
        P[node] = parent;
    }
    sync();
#pragma unroll 1
    for (int k = 0; k < (TW == 1 ? 3 : 1); ++k) {
        for (uint64_t u = s; u; u &= u - 1) {
            const uint32_t node = (uint32_t)(row * CT_NODES + (__builtin_ctzll(u) >> 1));
            P[node] = P[P[node]];
        }
        sync();
    }
    if (TW > 1 || __ballot((left | right) != 0)) {
        for (uint64_t u = left; u; u &= u - 1) {
            const int x = __builtin_ctzll(u);
            lunion(P, run_node(row, m, x), above(x, false));
        }
        for (uint64_t u = right; u; u &= u - 1) {
            const int x = __builtin_ctzll(u);
            lunion(P, run_node(row, m, x), above(x, true));
        }
    }
    sync();
    // the forest entry of a node's root: root's linear index + 1
    auto entry = [&](uint32_t node) -> uint32_t {
        const uint32_t r = lfind(P, node);
        const uint32_t rr = r / CT_NODES, k = 2 * (r - rr * CT_NODES);
        const uint64_t rm = row_of[rr];
        // the run starts at column k, or else at k + 1
        const uint32_t x = k + (((rm & ~(rm << 1)) >> k & 1) ? 0 : 1);
        return T.first + rr * W + x + 1u;
    };
    for (uint64_t u = s; u; u &= u - 1) {
        const int x = __builtin_ctzll(u);
        F[T.first + row * W + x] = entry(row * CT_NODES + (x >> 1));
    }
    if (m >> 63 && (TW == 1 || (th & 3) == 3)) F[T.first + row * W + 63] = entry(run_node(row, m, 63));
    // first and last row, lane = column
    const int lane = threadIdx.x & 63;
    const uint64_t m0 = row_of[0], m1 = row_of[T.h - 1];
    if ((TW == 1 || th < 64) && (m0 >> lane) & 1) F[T.first + lane] = entry(run_node(0, m0, lane));
    if ((TW == 1 || th >= 192) && (m1 >> lane) & 1)
        F[T.first + (T.h - 1) * W + lane] = entry(run_node((int)T.h - 1, m1, lane));
}

// TW waves per tile. Four threads read a row (16 pixels each; a wave's load
// instruction covers 16 rows), so the whole tile is in flight with at most
// four loads a thread, and each thread packs its pixels' foreground into 16 bits.
// A tile without foreground stores its empty masks and is done, the others make their
// unions. Bound by the image read: 16384 x 16384 uint8 with 1.6 % foreground takes 78 us
// (3.4 TB/s of image). Per-pixel lanes on 32 x 64 tiles that loaded one byte a
// lane and stored every pixel's forest entry took 533 us.
// Dense tiles are bound by the walks in LDS: node rows one bank apart, and nodes passed on
// a walk put below their parent's parent, take 4096 x 4096 one-pixel stripes from 234 to
// 77 us, half foreground at random (conn 8) from 72 to 53 us. With few tiles, whose time is one
// tile's, four waves share a tile with rows of many runs: 300 x 411 pixels, half of them
// foreground at random, 33 -> 15 us.
template <int CONN, int TW>
__global__ __launch_bounds__(64 * CT_WAVES) void k_ccl_local(const uint8_t *__restrict__ img,
                                                             uint32_t H, uint32_t W, int64_t pitch,
                                                             uint32_t tiles_x, uint32_t n_tiles,
                                                             uint32_t *__restrict__ labels,
                                                             int64_t lpitch,
                                                             uint32_t *__restrict__ F) {
    constexpr int TILES = CT_WAVES / TW; // tiles a workgroup
    constexpr int NJ = 4 / TW;           // 16-pixel chunks a thread loads
    __shared__ uint32_t Ps[TILES][CT * CT_NODES];
    __shared__ uint64_t rows[TILES][CT];
    const int wv = threadIdx.x / (64 * TW), th = threadIdx.x % (64 * TW); // tile, thread of it
    const uint32_t t = blockIdx.x * TILES + wv;
    if (t >= n_tiles) return;
    const CclTile T(t, tiles_x, H, W);
    uint32_t *P = Ps[wv];
    uint64_t *row_of = rows[wv];
    {
        const int c0 = 16 * (th & 3);
        uint32_t bits[NJ];
        if (W >= 16) {
            // a chunk that leaves the image on the right loads the image's last
            // 16 columns, and its bits are shifted back
            const int cs = std::min(c0, (int)(W - 16) - (int)T.x0);
            const int back = std::min(16, c0 - cs);
            // Aligned words that hold the 16 pixels: a fifth word where the
            // pixels are not word-aligned (it holds the last of them, so no
            // word is read that holds none).
            uint4 d[NJ];
            uint32_t d4[NJ], sh[NJ];
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t r = std::min<uint32_t>(16 * j + (th >> 2), T.h - 1);
                const uintptr_t a = (uintptr_t)(img + (int64_t)(T.y0 + r) * pitch + (int64_t)T.x0 + cs);
                const uint32_t *q = (const uint32_t *)(a & ~(uintptr_t)3);
                sh[j] = (uint32_t)(a & 3);
                __builtin_memcpy(&d[j], q, 16);
                d4[j] = q[sh[j] ? 4 : 3];
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                bits[j] = (nonzero_bits(__builtin_amdgcn_alignbyte(d[j].y, d[j].x, sh[j])) |
                           nonzero_bits(__builtin_amdgcn_alignbyte(d[j].z, d[j].y, sh[j])) << 4 |
                           nonzero_bits(__builtin_amdgcn_alignbyte(d[j].w, d[j].z, sh[j])) << 8 |
                           nonzero_bits(__builtin_amdgcn_alignbyte(d4[j], d[j].w, sh[j])) << 12) >>
                          back;
        } else {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const uint32_t r = std::min<uint32_t>(16 * j + (th >> 2), T.h - 1);
                const uint8_t *p = img + (int64_t)(T.y0 + r) * pitch + T.x0;
                bits[j] = 0;
                for (int k = 0; k < 16 && c0 + k < (int)T.w; ++k)
                    bits[j] |= (p[c0 + k] ? 1u : 0u) << k;
            }
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const uint32_t r = 16 * j + (th >> 2);
            ((uint16_t *)row_of)[4 * r + (th & 3)] = (uint16_t)(r < T.h ? bits[j] : 0u);
        }
    }
    if (TW == 1) ccl_wave_sync();
    else __syncthreads();
    // the masks, in word order, coalesced
    for (uint32_t j = th; j < T.h * T.nw; j += 64 * TW) {
        const uint32_t *half = (const uint32_t *)row_of;
        *T.word(labels, lpitch, j) = T.nw == 2 ? half[j] : half[2 * j];
    }
    const uint64_t m = row_of[threadIdx.x & 63];
    if (__ballot(m != 0) == 0) return;
    // all four waves of a workgroup take a tile with rows of many runs, else one does
    if (TW == 1 || __ballot(__popcll(m & ~(m << 1)) > CT_DENSE) == 0) {
        if (th < 64) ccl_tile<CONN, 1>(T, W, th, P, row_of, F);
    } else {
        ccl_tile<CONN, TW>(T, W, th, P, row_of, F);
    }
}

// ------------------------------------------------------------- border phase

__device__ __forceinline__ uint32_t gload(const uint32_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root index of x's tree in the global forest (entries: parent index + 1). Each second
// pixel passed is put below its parent's parent. A plain store does: x is not a root and
// never becomes one again, what is stored is an ancestor of x, and a merge whose minimum
// on x's entry it overwrites goes on to merge with the parent that the minimum returned.
__device__ __forceinline__ uint32_t gfind(uint32_t *F, uint32_t x) {
    uint32_t p = gload(F + x) - 1u;
    while (p != x) {
        const uint32_t g = gload(F + p) - 1u;
        if (g == p) return p;
        __hip_atomic_store(F + x, g + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        x = g;
        p = gload(F + x) - 1u;
    }
    return x;
}

__device__ __forceinline__ void gunion(uint32_t *F, uint32_t a, uint32_t b) {
    while (true) {
        a = gfind(F, a);
        b = gfind(F, b);
        if (a == b) return;
        if (a > b) {
            const uint32_t t = a;
            a = b;
            b = t;
        }
        const uint32_t old =
            __hip_atomic_fetch_min(F + b, a + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - 1u;
        if (old == b) return;
        b = old;
    }
}

// One wave per tile joins it with the tiles to its left and above, from the
// row masks alone (the forest is read only where two pixels touch). Left
// border, lane = row: column c (this tile's first) against column l (the left
// tile's last). Two touching pixels of a row are joined unless the row above
// joins the same two runs of rows; a diagonal pair only where no straight
// pair connects the same pixels. Pairs that reach into the row above the tile
// belong to the first-row rule, lane = column: as in the local phase, one
// union per run above that a run touches (the row above is the last row of
// the tiles above; where its runs straddle a tile border, the left-border
// rule of those tiles joins them). Bound by the latency of the mask reads and
// the few walks: 34 us on that image (204 us when border pixels were found
// by reading the forest). Dense images are bound by the walks: shortened on the way
// (gfind), half foreground at random at 8192 x 8192 takes 116 us instead of 275.
// With few tiles a workgroup of two waves takes a tile, one for each border (300 x 411
// pixels, half of them foreground 18 -> 12 us).
template <int CONN, bool SPLIT>
__global__ __launch_bounds__(64 * CT_WAVES) void k_ccl_merge(uint32_t H, uint32_t W,
                                                             uint32_t tiles_x, uint32_t n_tiles,
                                                             uint32_t *labels, int64_t lpitch,
                                                             uint32_t *__restrict__ F) {
    const int lane = threadIdx.x & 63;
    // SPLIT: a workgroup of two waves a tile, one for each border
    const uint32_t wv = threadIdx.x >> 6;
    const uint32_t t = SPLIT ? blockIdx.x : blockIdx.x * CT_WAVES + wv;
    if (t >= n_tiles) return;
    const CclTile T(t, tiles_x, H, W);
    const uint32_t tx = T.x0 / CT;
    const bool in = (uint32_t)lane < T.h;
    const uint64_t m = in ? T.mask(labels, lpitch, lane) : 0ull;
    uint64_t l = 0;
    if (tx > 0) { // (a tile with one to its right is 64 wide)
        const CclTile L(t - 1, tiles_x, H, W);
        l = in ? L.mask(labels, lpitch, lane) : 0ull;
    }
    uint64_t up = 0;
    bool upL = false, upR = false; // the row above, left and right of the tile
    if (T.y0 > 0) {
        up = CclTile(t - tiles_x, tiles_x, H, W).mask(labels, lpitch, CT - 1);
        if (CONN == 8 && tx > 0)
            upL = CclTile(t - tiles_x - 1, tiles_x, H, W).mask(labels, lpitch, CT - 1) >> 63;
        if (CONN == 8 && tx + 1 < tiles_x)
            upR = CclTile(t - tiles_x + 1, tiles_x, H, W).mask(labels, lpitch, CT - 1) & 1;
    }
    if (!SPLIT || wv == 0) {
        const uint64_t cb = __ballot((m & 1) != 0), lb = __ballot((l >> 63) != 0);
        const uint64_t straight = cb & lb;
        const uint32_t p = T.first + lane * W;
        if (((straight & ~(straight << 1)) >> lane) & 1) gunion(F, p, p - 1);
        if (CONN == 8 && lane > 0) {
            const uint64_t d1 = cb & (lb << 1) & ~lb & ~(cb << 1); // (y, c) and (y - 1, l)
            const uint64_t d2 = lb & (cb << 1) & ~cb & ~(lb << 1); // (y, l) and (y - 1, c)
            if ((d1 >> lane) & 1) gunion(F, p, p - W - 1);
            if ((d2 >> lane) & 1) gunion(F, p - 1, p - W);
        }
    }
    if (T.y0 == 0 || (SPLIT && wv == 0)) return;
    const uint64_t m0 = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)m) |
                        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(m >> 32)) << 32;
    const uint32_t q = T.first + lane;
    if (CONN == 4) {
        const uint64_t c = m0 & up;
        if (((c & ~(c << 1)) >> lane) & 1) gunion(F, q, q - W);
    } else {
        const uint64_t s = m0 & ~(m0 << 1);
        const uint64_t aL = up << 1 | (upL ? 1ull : 0ull);
        const uint64_t aR = up >> 1 | (upR ? 1ull << 63 : 0ull);
        if (((s & aL) >> lane) & 1) gunion(F, q, q - W - 1);
        if (((s & up & ~aL) >> lane) & 1) gunion(F, q, q - W);
        if (((m0 & aR & ~up) >> lane) & 1) gunion(F, q, q - W + 1);
    }
}

// ------------------------------------------------------------ labels written

// One wave per tile: its row masks are read, the first pixels of its runs
// listed in LDS in order, and each listed run's root looked up in the forest
// by one lane; then every pixel takes its run's label from the list (the rank
// of its run in the row) and the tile's labels are written, 16 bytes a lane
// (on any dword: rows of any width and pitch). Bound by the label write: 196 us on that image
// (5.5 TB/s; the flatten pass it replaces read the plane the local phase had
// written and took 242 us). The stores are streaming: the plane is four times
// the last-level cache, and the call is 3 % faster than with cached ones.
// Two or eight tiles a workgroup instead of four: 3 to 4 % slower calls.
// With few tiles (CT_FEW) a tile is split over the workgroup's waves, ROWS rows
// each: 512 x 3712 pixels 6.3 us instead of 8.3 us. Dense tiles are bound by the walks:
// four at a time, and of a whole tile's component once, take half foreground at random
// at 8192 x 8192 from 249 to 111 us and one-pixel stripes from 558 to 166 us.
template <int ROWS>
__global__ __launch_bounds__(64 * CT_WAVES) void k_ccl_write(uint32_t H, uint32_t W,
                                                             uint32_t tiles_x, uint32_t n_tiles,
                                                             uint32_t *labels, int64_t lpitch,
                                                             const uint32_t *__restrict__ F) {
    __shared__ uint32_t lists[CT_WAVES][ROWS * CT_RUNS];
    __shared__ uint64_t rows[CT_WAVES][ROWS];
    __shared__ uint32_t bases[CT_WAVES][ROWS]; // runs in the rows above
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint32_t t = ROWS == CT ? blockIdx.x * CT_WAVES + wv : blockIdx.x;
    const uint32_t r0 = ROWS == CT ? 0u : wv * ROWS; // this wave's rows of the tile
    if (t >= n_tiles) return;
    const CclTile T(t, tiles_x, H, W);
    uint32_t *list = lists[wv];
    uint64_t *row_of = rows[wv];
    uint32_t *base_of = bases[wv];
    const bool in = lane < ROWS && r0 + lane < T.h;
    const uint64_t m = in ? T.mask(labels, lpitch, r0 + lane) : 0ull;
    const bool any = __ballot(m != 0) != 0;
    if (any) {
        const uint32_t first = T.first + r0 * W; // this wave's first pixel
        const uint64_t s = m & ~(m << 1);
        const uint32_t n = (uint32_t)__popcll(s);
        uint32_t end = n; // inclusive scan over the rows
#pragma unroll
        for (int k = 1; k < 64; k <<= 1) {
            const uint32_t o = __shfl_up(end, k);
            if (lane >= k) end += o;
        }
        const uint32_t total = __shfl(end, 63);
        uint32_t at = end - n;
        if (lane < ROWS) {
            row_of[lane] = m;
            base_of[lane] = at;
        }
        for (uint64_t u = s; u; u &= u - 1)
            list[at++] = T.first + (r0 + lane) * W + (uint32_t)__builtin_ctzll(u);
        ccl_wave_sync();
        // The forest is at rest here: plain loads
        if (total <= 64) {
            if ((uint32_t)lane < total) {
                uint32_t e = list[lane] + 1u, p = F[e - 1u];
                while (p != e) {
                    e = p;
                    p = F[e - 1u];
                }
                list[lane] = e;
            }
        } else {
            // WALKS at a time. A run whose parent lies in this wave's rows takes the
            // label of the parent's run, so that a component of the tile is walked to
            // its root once and not by each of its runs (split tiles: their rows are few).
            for (uint32_t i = lane; i < total; i += 64 * WALKS) {
                uint32_t e[WALKS], p[WALKS];
#pragma unroll
                for (int k = 0; k < WALKS; ++k) e[k] = list[std::min(i + 64 * k, total - 1)] + 1u;
#pragma unroll
                for (int k = 0; k < WALKS; ++k) p[k] = F[e[k] - 1u];
                bool on = false;
                uint32_t in_tile = 0; // bit k: list[..] is to be the rank in e[k]
#pragma unroll
                for (int k = 0; k < WALKS; ++k) {
                    const uint32_t d = p[k] - 1u - first, y = d / W, x = d - y * W;
                    if (ROWS == CT && p[k] != e[k] && p[k] > first && y < ROWS && x < T.w) {
                        const uint64_t rm = row_of[y];
                        e[k] = base_of[y] + (uint32_t)__popcll((rm & ~(rm << 1)) & ((2ull << x) - 1)) - 1u;
                        p[k] = e[k];
                        in_tile |= 1u << k;
                    }
                    on |= p[k] != e[k];
                }
                while (on) {
                    on = false;
                    uint32_t q[WALKS];
#pragma unroll
                    for (int k = 0; k < WALKS; ++k) q[k] = (in_tile >> k) & 1u ? p[k] : F[p[k] - 1u];
#pragma unroll
                    for (int k = 0; k < WALKS; ++k) {
                        e[k] = p[k];
                        p[k] = q[k];
                        on |= p[k] != e[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < WALKS; ++k)
                    if (i + 64 * k < total) list[i + 64 * k] = (in_tile >> k) & 1u ? e[k] | RANK : e[k];
            }
            ccl_wave_sync();
            for (uint32_t i = lane; ROWS == CT && i < total; i += 64) {
                uint32_t e = lds_load(list + i);
                if (!(e & RANK)) continue;
                do e = lds_load(list + (e & ~RANK)); // (parents come first: this ends)
                while (e & RANK);
                list[i] = e;
            }
        }
    }
    // (the masks have been read: the tile's loads are done before its stores)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    ccl_wave_sync();
    if (ROWS < CT) __syncthreads();
    auto label = [&](uint64_t rm, uint64_t rs, uint32_t base, int x) -> uint32_t {
        if (!((rm >> x) & 1)) return 0u;
        return list[base + (uint32_t)__popcll(rs & ((2ull << x) - 1)) - 1u];
    };
    const int c = 4 * (lane & 15);
#pragma unroll 4
    for (int j = 0; j < ROWS / 4; ++j) {
        const uint32_t r = 4 * j + (lane >> 4);
        v4u v = {0, 0, 0, 0};
        if (any) {
            const uint64_t rm = row_of[r];
            if ((rm >> c) & 15) {
                const uint64_t rs = rm & ~(rm << 1);
                const uint32_t b = base_of[r];
                v = v4u{label(rm, rs, b, c), label(rm, rs, b, c + 1), label(rm, rs, b, c + 2),
                        label(rm, rs, b, c + 3)};
            }
        }
        if (r0 + r >= T.h) continue;
        uint32_t *o = labels + (int64_t)(T.y0 + r0 + r) * lpitch + T.x0 + c;
        if (c + 4 <= (int)T.w) {
            __builtin_nontemporal_store(v, (v4u_dw *)o);
        } else {
            if (c < (int)T.w) o[0] = v.x;
            if (c + 1 < (int)T.w) o[1] = v.y;
            if (c + 2 < (int)T.w) o[2] = v.z;
        }
    }
}

// A walk over the H x W pixels of a pitched image in linear
// order: (y, x) of this lane's pixel, advanced by the grid's stride without
// a division per pixel (H * W < 2^31).
struct PixelWalk {
    uint32_t i, y, x, dy, dx, n, W;
    __device__ PixelWalk(int64_t H, int64_t Wd, uint32_t first, uint32_t stride) {
        W = (uint32_t)Wd;
        n = (uint32_t)(H * Wd);
        i = first;
        y = first / W;
        x = first - y * W;
        dy = stride / W;
        dx = stride - dy * W;
    }
    __device__ bool ok() const { return i < n; }
    __device__ void next(uint32_t stride) {
        i += stride;
        y += dy;
        x += dx;
        if (x >= W) {
            x -= W;
            ++y;
        }
    }
};

// --------------------------------------------------------------- area phase

// Clears n counters, 16 bytes a lane (p is 256-byte aligned), with streaming
// stores, which leave fewer dirty lines for the count to displace: clear and
// count of 16384 x 16384 labels take 164 + 197 us (142 + 236 us with cached
// stores; 185 + 236 us with cached 4-byte ones).
__global__ __launch_bounds__(256) void k_area_clear(int32_t *p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n / 4;
         i += (int64_t)gridDim.x * 256)
        __builtin_nontemporal_store(v4u{0, 0, 0, 0}, (v4u *)p + i);
    if (blockIdx.x == 0 && threadIdx.x < (n & 3)) p[n / 4 * 4 + threadIdx.x] = 0;
}

// Count pixels per label: a wave reads 64 consecutive pixels of the image in
// linear order (one per lane, coalesced); a lane whose label differs from
// the previous pixel's (or that starts a row or the wave's chunk) heads a
// run, and adds the run's length, up to the next head, with one atomic.
// Background (0) and out-of-range labels are not counted. A run that spans
// two chunks is added in two parts.
__global__ __launch_bounds__(256) void k_area_count(const int32_t *__restrict__ labels,
                                                    int64_t H, int64_t W, int64_t pitch,
                                                    int32_t *__restrict__ area) {
    const uint32_t N = (uint32_t)(H * W);
    const int lane = threadIdx.x & 63;
    const uint32_t wave = blockIdx.x * 4u + (threadIdx.x >> 6), waves = gridDim.x * 4u;
    const uint32_t stride = waves * 64u;
    // every lane of a wave stays in the loop while its chunk has pixels, so
    // the cross-lane steps below see the whole wave
    for (PixelWalk w(H, W, wave * 64u + lane, stride); w.i - lane < N; w.next(stride)) {
        const bool in = w.ok();
        const int32_t l = in ? labels[(int64_t)w.y * pitch + w.x] : 0;
        const int32_t prev = __shfl_up(l, 1);
        const bool head = in && (lane == 0 || w.x == 0 || l != prev);
        const uint64_t heads = __ballot(head);
        const uint64_t valid = __ballot(in);
        if (head && l > 0 && (uint32_t)l <= N) {
            const uint64_t later = lane == 63 ? 0ull : (heads >> (lane + 1)) << (lane + 1);
            const int end = later ? __builtin_ctzll(later) : 64 - __builtin_clzll(valid);
            atomicAdd(area + l, end - lane);
        }
    }
}

// The word path: a lane takes 16-byte words of 4 labels. LIN: rows follow each
// other without gaps (pitch = W), so the plane is one row of H * W labels, of
// any length; else W and the pitch are multiples of 4. A wave's chunk is 64
// words; runs are found across it, and a run that spans two chunks is added
// in two parts.
constexpr int AREA_UNROLL = 2;   // chunks of the count loaded together
constexpr int FILTER_UNROLL = 4; // words of the filter
constexpr uint32_t AREA_GROUP = 32; // most chunks a wave of the filter takes
constexpr unsigned AREA_BLOCKS = 1u << 22;
// The one-pixel kernels walk the plane with this many blocks at most: waves that run
// together then lie far apart, and fewer of them add to one label's counter at once
// (16384 x 16377 labels, rows 16384 apart, squares of 300 pixels: 1661 us, 2299 us with
// a block for every 256 pixels).
constexpr int64_t AREA_PIXEL_BLOCKS = 1 << 16;

template <bool LIN>
__device__ __forceinline__ int64_t area_word(uint32_t i, uint32_t Wq, int64_t pitch) {
    if (LIN) return 4 * (int64_t)i;
    const uint32_t y = i / Wq;
    return (int64_t)y * pitch + 4 * (int64_t)(i - y * Wq);
}

// Run heads are marked per label; a head's run ends at the next head in its
// lane, else at the first head of the next lane that has one, else at the
// chunk's end. AREA_UNROLL chunks are loaded at a time. With `marks`, each
// chunk leaves a mask of its words that hold a countable label, so that the
// filter reads only those. Bound by the label read: 217 us on 16384 x 16384
// labels, 1.6 % of them foreground (4.9 TB/s). One pass of two chunks a wave: four
// chunks, or a fixed grid of 4096 blocks walking the plane, made the call 1 and 13 %
// slower. On dense labels the atomics bound it: blocks take a large plane in eight bands, so
// that those which run together add to fewer of the same counters (squares of 300
// pixels 509 -> 256 us, 1.6 % foreground 204 -> 218 us), and a chunk of short runs goes
// through LDS, so that an atomic instruction's lanes hold neighbouring pixels, whose
// labels often share a cache line (one-pixel stripes at 11584 x 11584 901 -> 552 us).
template <bool LIN>
__global__ __launch_bounds__(256) void k_area_count4(const int32_t *__restrict__ labels,
                                                     uint32_t N, uint32_t NQ, uint32_t Wq,
                                                     int64_t pitch, int32_t *__restrict__ area,
                                                     uint64_t *__restrict__ marks,
                                                     uint32_t bands) {
    __shared__ int4 runs[4][2][64];
    const int lane = threadIdx.x & 63;
    const uint32_t chunks = (NQ + 63) / 64;
    const uint32_t blk = blockIdx.x % bands * (gridDim.x / bands) + blockIdx.x / bands;
    const uint32_t wave = blk * 4u + (threadIdx.x >> 6), waves = gridDim.x * 4u;
    for (uint32_t c0 = wave * AREA_UNROLL; c0 < chunks; c0 += waves * AREA_UNROLL) {
        int4 qs[AREA_UNROLL];
#pragma unroll
        for (int k = 0; k < AREA_UNROLL; ++k) {
            const uint32_t i = (c0 + k) * 64u + lane;
            qs[k] = int4{0, 0, 0, 0};
            if (i < NQ) qs[k] = *(const int4 *)(labels + area_word<LIN>(i, Wq, pitch));
        }
#pragma unroll
        for (int k = 0; k < AREA_UNROLL; ++k) {
            if (c0 + k >= chunks) break;
            const bool in = (c0 + k) * 64u + lane < NQ;
            const int4 q = qs[k];
            auto counts = [&](int32_t l) { return l > 0 && (uint32_t)l <= N; };
            const uint64_t some =
                __ballot(in && (counts(q.x) || counts(q.y) || counts(q.z) || counts(q.w)));
            if (marks && lane == 0) marks[c0 + k] = some;
            if (some == 0) continue;
            const int32_t prev = __shfl_up(q.w, 1);
            uint32_t hm = 0; // bit j: label j of this lane starts a run
            if (in) {
                hm = (lane == 0 || q.x != prev) ? 1u : 0u;
                hm |= (q.y != q.x ? 2u : 0u) | (q.z != q.y ? 4u : 0u) | (q.w != q.z ? 8u : 0u);
            }
            const int first = hm ? __builtin_ctz(hm) : 4;
            const uint64_t with_head = __ballot(hm != 0);
            const uint64_t valid = __ballot(in);
            const uint64_t later = lane == 63 ? 0ull : (with_head >> (lane + 1)) << (lane + 1);
            const int ln = later ? __builtin_ctzll(later) : lane;
            const int fn = __shfl(first, ln);
            const int next = later ? 4 * ln + fn : 4 * (64 - __builtin_clzll(valid));
            const int32_t lv[4] = {q.x, q.y, q.z, q.w};
            auto run = [&](int j) -> int32_t { // pixels of the run that label j starts
                const uint32_t rest = hm >> (j + 1);
                const int end = rest ? 4 * lane + j + 1 + __builtin_ctz(rest) : next;
                return end - (4 * lane + j);
            };
            if (__popcll(__ballot((hm & (hm - 1)) != 0)) > 16) {
                int4 *L = runs[threadIdx.x >> 6][0], *C = runs[threadIdx.x >> 6][1];
                int32_t len[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) len[j] = (hm >> j) & 1u && counts(lv[j]) ? run(j) : 0;
                L[lane] = q;
                C[lane] = int4{len[0], len[1], len[2], len[3]};
                ccl_wave_sync();
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int32_t c = ((const int32_t *)C)[64 * j + lane];
                    if (c) atomicAdd(area + ((const int32_t *)L)[64 * j + lane], c);
                }
                ccl_wave_sync();
                continue;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if ((hm >> j) & 1u && counts(lv[j])) atomicAdd(area + lv[j], run(j));
        }
    }
    // LIN: the labels past the last whole word
    if (LIN && blockIdx.x == 0 && threadIdx.x < (N & 3u)) {
        const int32_t l = labels[4 * (int64_t)NQ + threadIdx.x];
        if (l > 0 && (uint32_t)l <= N) atomicAdd(area + l, 1);
    }
}

__global__ __launch_bounds__(256) void k_area_filter(int32_t *__restrict__ labels, int64_t H,
                                                     int64_t W, int64_t pitch,
                                                     const int32_t *__restrict__ area,
                                                     int64_t lo, int64_t hi) {
    const int64_t N = H * W;
    const uint32_t stride = gridDim.x * 256u;
    for (PixelWalk w(H, W, blockIdx.x * 256u + threadIdx.x, stride); w.ok(); w.next(stride)) {
        int32_t *p = labels + (int64_t)w.y * pitch + w.x;
        const int32_t l = *p;
        if (l > 0 && (int64_t)l <= N) {
            const int64_t a = area[l];
            if (a < lo || a > hi) *p = 0;
        }
    }
}

// The word path of the filter: a word's 4 counter reads are in flight
// together, and it is written back only if one of its labels was cleared. With
// `marks` (see the count) a wave takes `group` chunks (32 of a large plane, fewer
// of a smaller one, so that it still spreads over the chip), lists the words that
// hold a label in LDS and deals them to its lanes, so that planes of mostly
// background are not read again; a wave with too many marked words (half of a large
// group's, three quarters of a small one's) and planes without marks go chunk by chunk. 16384 x 16384 labels: 1.6 % of
// them foreground 25 us with marks, 222 us reading every word; squares of 300
// pixels 412 us (535 us with 64 chunks a wave and one word a lane at a time; with four
// words a lane, 64 chunks take 21 and 446 us, 16 chunks 38 and 394 us).
template <bool LIN>
__global__ __launch_bounds__(256) void k_area_filter4(int32_t *__restrict__ labels, uint32_t N,
                                                      uint32_t NQ, uint32_t Wq, int64_t pitch,
                                                      const int32_t *__restrict__ area, int64_t lo,
                                                      int64_t hi, uint32_t group,
                                                      const uint64_t *__restrict__ marks) {
    constexpr uint32_t LIST = AREA_GROUP * 32; // listed words of a wave's AREA_GROUP * 64
    __shared__ uint16_t lists[4][LIST];
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint16_t *list = lists[wv];
    const uint32_t chunks = (NQ + 63) / 64;
    const uint32_t wave = blockIdx.x * 4u + wv, waves = gridDim.x * 4u;
    auto keep = [&](int32_t l) -> int32_t {
        if (l <= 0 || (uint32_t)l > N) return l;
        const int64_t a = area[l];
        return a < lo || a > hi ? 0 : l;
    };
    auto at = [&](uint32_t i) { return (int4 *)(labels + area_word<LIN>(i, Wq, pitch)); };
    auto filter = [&](int4 *p, int4 l) {
        const int4 o = {keep(l.x), keep(l.y), keep(l.z), keep(l.w)};
        if (o.x != l.x || o.y != l.y || o.z != l.z || o.w != l.w) *p = o;
    };
    for (uint32_t c0 = wave * group; c0 < chunks; c0 += waves * group) {
        if (marks) {
            const uint64_t w = (uint32_t)lane < group && c0 + lane < chunks ? marks[c0 + lane] : 0ull;
            const uint32_t n = (uint32_t)__popcll(w);
            uint32_t end = n;
#pragma unroll
            for (int k = 1; k < 64; k <<= 1) {
                const uint32_t o = __shfl_up(end, k);
                if (lane >= k) end += o;
            }
            const uint32_t total = __shfl(end, 63);
            if (total <= LIST && 4 * total <= 3 * 64 * group) {
                uint32_t e = end - n;
                for (uint64_t u = w; u; u &= u - 1)
                    list[e++] = (uint16_t)(lane * 64 + __builtin_ctzll(u));
                ccl_wave_sync();
                for (uint32_t i = lane; i < total; i += 64 * FILTER_UNROLL) {
                    int4 *p[FILTER_UNROLL], q[FILTER_UNROLL];
#pragma unroll
                    for (int j = 0; j < FILTER_UNROLL; ++j) {
                        p[j] = at(c0 * 64u + list[std::min(i + 64 * j, total - 1)]);
                        q[j] = int4{0, 0, 0, 0};
                        if (i + 64 * j < total) q[j] = *p[j];
                    }
#pragma unroll
                    for (int j = 0; j < FILTER_UNROLL; ++j)
                        if (i + 64 * j < total) filter(p[j], q[j]);
                }
                ccl_wave_sync();
                continue;
            }
        }
        for (uint32_t k = 0; k < group; k += FILTER_UNROLL) {
            int4 q[FILTER_UNROLL];
#pragma unroll
            for (int j = 0; j < FILTER_UNROLL; ++j) {
                const uint32_t i = (c0 + k + j) * 64u + lane;
                q[j] = int4{0, 0, 0, 0};
                if (k + j < group && i < NQ) q[j] = *at(i);
            }
#pragma unroll
            for (int j = 0; j < FILTER_UNROLL; ++j) {
                const uint32_t i = (c0 + k + j) * 64u + lane;
                if (k + j < group && i < NQ) filter(at(i), q[j]);
            }
        }
    }
    if (LIN && blockIdx.x == 0 && threadIdx.x < (N & 3u)) {
        int32_t *p = labels + 4 * (int64_t)NQ + threadIdx.x;
        const int32_t l = *p, o = keep(l);
        if (o != l) *p = o;
    }
}

unsigned grid_for(int64_t items, int64_t most) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + 255) / 256, most));
}

// The word path's marks, one bit per 16-byte word of labels, behind the areas.
// A workspace without room for them is still accepted; its filter reads every
// word.
size_t area_marks_bytes(int64_t n) { return up256((size_t)((n / 4 + 63) / 64) * 8); }

int check_labels_dims(int64_t H, int64_t W, int64_t pitch) {
    if (H < 1 || W < 1) return cfail(MR_EINVAL, "H and W must be >= 1");
    if (pitch < W) return cfail(MR_EINVAL, "pitch below W");
    if (H * W >= (1ll << 31) - 1) return cfail(MR_EINVAL, "H * W must be below 2^31 - 1");
    return MR_OK;
}

} // namespace

extern "C" {

size_t mr_ccl_workspace_bytes(int64_t H, int64_t W) {
    clear_error();
    if (check_labels_dims(H, W, W) != MR_OK) return 0;
    return up256((size_t)(H * W) * 4);
}

int mr_ccl(const void *img, void *labels, int64_t H, int64_t W, int64_t pitch,
           int64_t label_pitch, int conn, void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    if (pitch == 0) pitch = W;
    if (label_pitch == 0) label_pitch = W;
    int rc;
    if ((rc = check_labels_dims(H, W, pitch)) != MR_OK) return rc;
    if (label_pitch < W) return cfail(MR_EINVAL, "label_pitch below W");
    if (conn != 4 && conn != 8) return cfail(MR_EINVAL, "conn must be 4 or 8 (got %d)", conn);
    if (!img || !labels || !ws) return cfail(MR_EINVAL, "null pointer");
    if ((uintptr_t)labels % 4) return cfail(MR_EINVAL, "labels must be 4-byte aligned");
    if ((uintptr_t)ws % 256) return cfail(MR_EINVAL, "workspace must be 256-byte aligned");
    const size_t need = up256((size_t)(H * W) * 4);
    if (ws_bytes < need)
        return cfail(MR_ENOMEM, "workspace too small: %zu bytes given, %zu needed", ws_bytes, need);
    hipStream_t s = (hipStream_t)stream;
    uint32_t *F = (uint32_t *)ws, *L = (uint32_t *)labels;
    const uint32_t h = (uint32_t)H, w = (uint32_t)W;
    const uint32_t tx = (w + CT - 1) / CT, tiles = tx * ((h + CT - 1) / CT);
    const bool few = tiles < CT_FEW;
    const dim3 grid(few ? tiles : (tiles + CT_WAVES - 1) / CT_WAVES), wide(64 * CT_WAVES);
    auto launch = [&](auto local, auto merge, auto write) {
        hipLaunchKernelGGL(local, grid, wide, 0, s, (const uint8_t *)img, h, w, pitch, tx, tiles,
                           L, label_pitch, F);
        hipLaunchKernelGGL(merge, grid, few ? dim3(128) : wide, 0, s, h, w, tx, tiles, L, label_pitch,
                           F);
        hipLaunchKernelGGL(write, grid, wide, 0, s, h, w, tx, tiles, L, label_pitch, F);
    };
    const auto write = few ? k_ccl_write<CT / CT_WAVES> : k_ccl_write<CT>;
    if (conn == 8)
        launch(few ? k_ccl_local<8, CT_WAVES> : k_ccl_local<8, 1>,
               few ? k_ccl_merge<8, true> : k_ccl_merge<8, false>, write);
    else
        launch(few ? k_ccl_local<4, CT_WAVES> : k_ccl_local<4, 1>,
               few ? k_ccl_merge<4, true> : k_ccl_merge<4, false>, write);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MR_OK : chip(e, "ccl");
}

size_t mr_area_threshold_workspace_bytes(int64_t H, int64_t W) {
    clear_error();
    if (check_labels_dims(H, W, W) != MR_OK) return 0;
    return up256((size_t)(H * W + 1) * 4) + area_marks_bytes(H * W);
}

int mr_area_threshold(void *labels_inout, int64_t H, int64_t W, int64_t pitch, int64_t min_area,
                      int64_t max_area, void *ws, size_t ws_bytes, void *stream) {
    clear_error();
    if (pitch == 0) pitch = W;
    int rc;
    if ((rc = check_labels_dims(H, W, pitch)) != MR_OK) return rc;
    if (!labels_inout || !ws) return cfail(MR_EINVAL, "null pointer");
    if ((uintptr_t)labels_inout % 4) return cfail(MR_EINVAL, "labels must be 4-byte aligned");
    if ((uintptr_t)ws % 256) return cfail(MR_EINVAL, "workspace must be 256-byte aligned");
    const size_t need = up256((size_t)(H * W + 1) * 4);
    if (ws_bytes < need)
        return cfail(MR_ENOMEM, "workspace too small: %zu bytes given, %zu needed", ws_bytes, need);
    hipStream_t s = (hipStream_t)stream;
    int32_t *area = (int32_t *)ws;
    hipLaunchKernelGGL(k_area_clear, dim3(grid_for(H * W / 4 + 1, 1 << 22)), dim3(256), 0, s, area, H * W + 1);
    const uint32_t N = (uint32_t)(H * W), NQ = N / 4;
    const bool lin = pitch == W;
    if (NQ > 0 && (lin || (W % 4 == 0 && pitch % 4 == 0)) && (uintptr_t)labels_inout % 16 == 0) {
        int32_t *l = (int32_t *)labels_inout;
        const uint32_t wq = (uint32_t)(W / 4), chunks = (NQ + 63) / 64;
        // (small planes are filtered faster word by word: 512 x 3712 labels 3.9
        // against 4.8 us)
        uint64_t *marks = chunks >= 16384 && ws_bytes >= need + area_marks_bytes(H * W)
                              ? (uint64_t *)((char *)ws + need) : nullptr;
        // (2048 x 2048 labels, whose words still lie in the dies' L2s: 19 us in order, 25 us
        // in bands; squares of 300 pixels at 6000 x 6000 195 us in order, 172 us in bands)
        const uint32_t bands = chunks >= 131072 ? 8 : 1;
        const unsigned gc = (std::min<unsigned>((chunks + 4 * AREA_UNROLL - 1) / (4 * AREA_UNROLL),
                                                AREA_BLOCKS) + bands - 1) / bands * bands;
        // chunks a wave of the filter takes: 8 waves a SIMD before it grows
        const uint32_t group = std::max(1u, std::min(AREA_GROUP, chunks / 8192u));
        const unsigned gf = std::min<unsigned>((chunks + 4 * group - 1) / (4 * group), AREA_BLOCKS);
        if (lin) {
            hipLaunchKernelGGL(k_area_count4<true>, dim3(gc), dim3(256), 0, s, l, N, NQ, wq, pitch,
                               area, marks, bands);
            hipLaunchKernelGGL(k_area_filter4<true>, dim3(gf), dim3(256), 0, s, l, N, NQ, wq, pitch,
                               (const int32_t *)area, min_area, max_area, group, marks);
        } else {
            hipLaunchKernelGGL(k_area_count4<false>, dim3(gc), dim3(256), 0, s, l, N, NQ, wq, pitch,
                               area, marks, bands);
            hipLaunchKernelGGL(k_area_filter4<false>, dim3(gf), dim3(256), 0, s, l, N, NQ, wq,
                               pitch, (const int32_t *)area, min_area, max_area, group, marks);
        }
    } else {
        hipLaunchKernelGGL(k_area_count, dim3(grid_for(H * W, AREA_PIXEL_BLOCKS)), dim3(256), 0, s,
                           (const int32_t *)labels_inout, H, W, pitch, area);
        hipLaunchKernelGGL(k_area_filter, dim3(grid_for(H * W, AREA_PIXEL_BLOCKS)), dim3(256), 0, s,
                           (int32_t *)labels_inout, H, W, pitch, (const int32_t *)area,
                           min_area, max_area);
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? MR_OK : chip(e, "area threshold");
}

} // extern "C"
