// mr_dt.hip -- distance transform (Table II: IWPP, 8-connected);
// mr_distance_transform in include/mr_ops.h.
//
// D(p) = length in G-steps of the shortest path from p to a background
// pixel. As a wavefront propagation (Algorithm 1): background pixels start at
// 0 and foreground pixels at infinity, and a pixel q takes D(p) + 1 from a
// neighbour p whenever that is smaller (PropagationCondition D(p) + 1 < D(q),
// Update D(q) = D(p) + 1). Every value is at all times an upper bound of the
// true distance, and a state where no pixel can lower a neighbour is the
// true distance (along a shortest path each step can add at most 1), so any
// order of updates that runs to such a state gives the same, unique result.
//
// On the GPU a first pass (k_dt_first) settles every distance up to DW_MAX from
// the image's bits alone: a window of 128 x 128 pixels, eroded DW_MAX times,
// gives every pixel of its 96 x 96 interior its distance where that is at most
// DW_MAX, and that value is final, because a background pixel outside the
// window is further away than that. Pixels further from the background start
// unreached (infinity), and the tiles where they meet settled ones are listed.
// Those are left to rounds over 64 x 64 register tiles (a 62 x 62
// interior and a one-pixel halo) held by one wave each: lane = column,
// register = row. A visit loads the tile,
// sweeps down and up the registers (the three upper or lower
// neighbours through DPP lane shifts for 8-connectivity), transposes through
// LDS and sweeps right and left, which brings it to its fixed point; it stores
// the interior and marks for the next round every
// neighbouring tile whose halo it changed. Rounds run until one marks no
// tile; the host polls a small counter between batches of rounds.
#include <algorithm>
#include <cstdarg>
#include <cstdio>

#include "../../include/mr_ops.h"
#include "mr_internal.h"

using namespace mr;

namespace {

int dfail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return set_error(code, buf);
}

int dhip(hipError_t e, const char *what) {
    return dfail(MR_EHIP, "%s: %s", what, hipGetErrorString(e));
}

size_t up256(size_t n) { return (n + 255) / 256 * 256; }

constexpr int DS = 64, DI = DS - 2;     // register tile and its interior
constexpr uint32_t INF = 0x7FFFFFFFu;   // "not reached yet"; INF + 1 does not wrap
// Rounds per host poll. Squares of 300 pixels settle in the fifth round: 1000 x 1021
// pixels 147 us with 4 rounds, 122 us with 5, 124 us with 6; an image that needs two
// waits 2 us longer for each.
constexpr int DT_BATCH = 5;
constexpr int64_t DT_MAX_ROUNDS = 1 << 20;

// Per-call control words at the head of the workspace.
struct DtCtrl {
    uint32_t has_bg;     // some pixel of the image is background
    uint32_t pad[63];
    uint32_t marked[4];  // tiles marked for round r, at r mod 4 (r + 2's is cleared in r)
    uint32_t pad2[60];
};

// Lane i gets lane i-1's value (lane 0 keeps its own).
__device__ __forceinline__ uint32_t lane_left(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x138 /* wave_shr:1 */, 0xF,
                                                 0xF, false);
}
// Lane i gets lane i+1's value (lane 63 keeps its own).
__device__ __forceinline__ uint32_t lane_right(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x130 /* wave_shl:1 */, 0xF,
                                                 0xF, false);
}

template <int CONN>
__device__ __forceinline__ uint32_t reach(uint32_t prev_row) {
    // the smallest distance among the neighbours in the adjacent row, + 1
    uint32_t m = prev_row;
    if (CONN == 8) m = min(m, min(lane_left(prev_row), lane_right(prev_row)));
    return m + 1u;
}

// (one wave per block: LDS hand-offs between its lanes need program order
// and a compiler barrier, not a workgroup barrier)
__device__ __forceinline__ void dt_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void transpose(uint32_t (&A)[DS], uint32_t (*tb)[DS + 1], int lane) {
#pragma unroll
    for (int r = 0; r < DS; ++r) tb[r][lane] = A[r];
    dt_wave_sync();
#pragma unroll
    for (int c = 0; c < DS; ++c) A[c] = tb[lane][c];
    dt_wave_sync();
}

// ---------------------------------------------------------------- first pass

constexpr int DW = 128;            // window side: a row is four 32-bit words
constexpr int DW_MARGIN = 16;      // window pixels beyond the interior, each side
constexpr int DW_IN = DW - 2 * DW_MARGIN;
constexpr int DW_MAX = DW_MARGIN;  // largest distance the window settles
constexpr int DW_SLICES = 5;       // bits of a settled distance
constexpr int DW_WAVES = 4;        // windows (waves) per workgroup
constexpr int DW_ROW = DW_IN / 4 + 1; // dwords per row of the byte tile: odd, no bank conflicts
constexpr uint32_t DW_FAR = 0xFFu; // byte of a pixel further than DW_MAX
static_assert(DW_MAX < 1 << DW_SLICES && DW == 2 * 64, "a lane holds two rows");

// Lane i gets lane i-1's (i+1's) value; all ones come in at the wave's ends.
__device__ __forceinline__ uint32_t ones_from_left(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF,
                                                 false);
}
__device__ __forceinline__ uint32_t ones_from_right(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF,
                                                 false);
}

// One erosion of the window by the G-neighbourhood: E holds rows 2 lane (E[0])
// and 2 lane + 1 (E[1]), bit = column, set = foreground. What lies outside the
// window (or the image) is foreground: it never erodes anything.
template <int CONN>
__device__ __forceinline__ void erode_once(uint32_t (&E)[2][4]) {
    uint32_t h[2][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t lo = i > 0 ? E[r][i - 1] : ~0u, hi = i < 3 ? E[r][i + 1] : ~0u;
            h[r][i] = E[r][i] & __builtin_amdgcn_alignbit(E[r][i], lo, 31) &
                      __builtin_amdgcn_alignbit(hi, E[r][i], 1);
        }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        // 8-connectivity: the rows above and below, eroded along the row too
        const uint32_t a = CONN == 8 ? h[0][i] : E[0][i], b = CONN == 8 ? h[1][i] : E[1][i];
        const uint32_t up = ones_from_left(b), down = ones_from_right(a);
        const uint32_t both = h[0][i] & h[1][i];
        if (CONN == 8) {
            E[0][i] = both & up;
            E[1][i] = both & down;
        } else {
            E[0][i] = h[0][i] & b & up;
            E[1][i] = h[1][i] & a & down;
        }
    }
}

// One wave per window. Eight lanes read a row's 128 bytes (16 pixels each), the
// foreground goes to LDS as bits, and each lane takes two rows. With E_k the
// image eroded k times, a pixel's distance exceeds k iff E_k holds it, so bit j
// of the distance is the exclusive or of E_k over the k with 2^j | k + 1: the
// distances collect in bit slices, DW_SLICES words per 32 pixels, and the
// erosions stop once the interior is empty. The slices are spread to bytes
// (through LDS, four pixels a dword) and stored as 16 bytes a lane. Windows
// without foreground store zeros.
// Bound by the int32 plane's write: 16384 x 16384 uint8 with 1.6 % foreground
// takes 221 us, 6.1 TB/s of image read and distances written (418 us for a first
// round of register tiles, which also left 213 us of later rounds to do: a
// tile's halo is one pixel, so every object across a border was revisited).
template <int CONN>
__global__ __launch_bounds__(64 * DW_WAVES) void k_dt_first(
    const uint8_t *__restrict__ img, int64_t ipitch, int32_t *__restrict__ dist, int64_t dpitch,
    int64_t H, int64_t W, int64_t wtx, int64_t n_windows, int32_t ntx, int32_t nty,
    uint32_t *__restrict__ flags, DtCtrl *__restrict__ ctrl, uint32_t *__restrict__ lists) {
    __shared__ __align__(16) uint32_t lds[DW_WAVES][DW_IN * DW_ROW];
    static_assert(DW_IN * DW_ROW >= DW * 4, "the row bits share the byte tile's LDS");
    const int lane = threadIdx.x & 63;
    const int64_t wi = (int64_t)blockIdx.x * DW_WAVES + (threadIdx.x >> 6);
    if (wi >= n_windows) return;
    uint32_t *buf = lds[threadIdx.x >> 6];
    const int64_t wy = wi / wtx, wx = wi - wy * wtx;
    const int64_t y0 = wy * DW_IN, x0 = wx * DW_IN;           // interior's first pixel
    const int64_t wy0 = y0 - DW_MARGIN, wx0 = x0 - DW_MARGIN; // window's first pixel
    // the window's rows and columns that lie in the image: r_lo.. < r_hi, ...
    const int r_lo = wy0 < 0 ? (int)-wy0 : 0, r_hi = (int)std::min<int64_t>(DW, H - wy0);
    const int c_lo = wx0 < 0 ? (int)-wx0 : 0, c_hi = (int)std::min<int64_t>(DW, W - wx0);
    const uint8_t *wimg = img + wy0 * ipitch + wx0; // (dereferenced inside the image only)
    {
        const int c = 16 * (lane & 7);
        // the 16 pixels loaded: moved into the image where the chunk is partly
        // outside (images narrower than that go byte by byte), and their bits
        // shifted back
        const bool wide = c_hi - c_lo >= 16;
        const int cs = std::min(std::max(c, c_lo), c_hi - 16);
        const int back = std::min(16, cs > c ? cs - c : c - cs);
        const bool words = ((((uintptr_t)wimg) | (uintptr_t)ipitch | (uintptr_t)c_lo |
                             (uintptr_t)c_hi) & 3) == 0;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint32_t bits[8];
            if (wide) {
                uint4 d[8];
                uint32_t d4[8], sh[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int r = std::min(std::max(64 * half + 8 * j + (lane >> 3), r_lo), r_hi - 1);
                    const uintptr_t a = (uintptr_t)(wimg + r * ipitch + cs);
                    // aligned words that hold the pixels: a fifth one where the
                    // row is not word-aligned (it holds the last of them)
                    const uint32_t *q = (const uint32_t *)(a & ~(uintptr_t)3);
                    __builtin_memcpy(&d[j], q, 16);
                    sh[j] = words ? 0u : (uint32_t)(a & 3);
                    d4[j] = words ? 0u : q[sh[j] ? 4 : 3];
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    uint4 v = d[j];
                    if (!words) {
                        v.x = __builtin_amdgcn_alignbyte(d[j].y, d[j].x, sh[j]);
                        v.y = __builtin_amdgcn_alignbyte(d[j].z, d[j].y, sh[j]);
                        v.z = __builtin_amdgcn_alignbyte(d[j].w, d[j].z, sh[j]);
                        v.w = __builtin_amdgcn_alignbyte(d4[j], d[j].w, sh[j]);
                    }
                    const uint32_t w = nonzero_bits(v.x) | nonzero_bits(v.y) << 4 |
                                       nonzero_bits(v.z) << 8 | nonzero_bits(v.w) << 12;
                    bits[j] = cs >= c ? (w << back) | ((1u << back) - 1u)
                                      : (w >> back) | (0xFFFFu << (16 - back));
                }
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int r = std::min(std::max(64 * half + 8 * j + (lane >> 3), r_lo), r_hi - 1);
                    bits[j] = 0xFFFFu;
                    for (int k = 0; k < 16; ++k)
                        if (c + k >= c_lo && c + k < c_hi && wimg[r * ipitch + c + k] == 0)
                            bits[j] &= ~(1u << k);
                }
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int r = 64 * half + 8 * j + (lane >> 3);
                ((uint16_t *)buf)[8 * r + (lane & 7)] =
                    (uint16_t)(r >= r_lo && r < r_hi ? bits[j] : 0xFFFFu);
            }
        }
    }
    dt_wave_sync();
    uint32_t E[2][4], fg[2][4];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const uint4 w = *(const uint4 *)(buf + (2 * lane + r) * 4);
        E[r][0] = w.x;
        E[r][1] = w.y;
        E[r][2] = w.z;
        E[r][3] = w.w;
    }
    // (pixels outside the image read as foreground)
    uint32_t bg = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) bg |= ~(E[0][i] & E[1][i]);
    if (__ballot(bg != 0) != 0 && lane == 0 &&
        __hip_atomic_load(&ctrl->has_bg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
        atomicOr(&ctrl->has_bg, 1u);
    // the interior's pixels that lie in the image: column masks (uniform) and
    // whether this lane's two rows are among its rows
    uint32_t cm[4];
    const int i_lo = DW_MARGIN, i_hi = std::min(c_hi, DW_MARGIN + DW_IN);
    auto cols = [](int lo, int hi, int i) -> uint32_t { // bits lo..hi-1 of 128, word i
        const int a = std::max(0, std::min(32, lo - 32 * i)), b = std::max(0, std::min(32, hi - 32 * i));
        return (uint32_t)((1ull << b) - (1ull << a));
    };
#pragma unroll
    for (int i = 0; i < 4; ++i) cm[i] = cols(i_lo, i_hi, i);
    const int in_rows = std::min(r_hi - DW_MARGIN, DW_IN); // interior rows in the image
    const int ir = 2 * lane - DW_MARGIN;                   // interior row of E[0]
    const bool ok[2] = {ir >= 0 && ir < in_rows, ir + 1 >= 0 && ir + 1 < in_rows};
    auto inside_any = [&]() -> bool {
        uint32_t a = 0, b = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a |= E[0][i] & cm[i];
            b |= E[1][i] & cm[i];
        }
        return __ballot((ok[0] && a != 0) || (ok[1] && b != 0)) != 0;
    };
    const bool some = inside_any();
    bool far = false, last = false; // last: E ends eroded DW_MAX times
    if (some) {
        uint32_t S[DW_SLICES][2][4];
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                fg[r][i] = E[r][i] & cm[i];
                S[0][r][i] = E[r][i]; // k = 0
#pragma unroll
                for (int j = 1; j < DW_SLICES; ++j) S[j][r][i] = 0;
            }
        far = true;
#pragma unroll
        for (int k = 1; k <= DW_MAX; ++k) {
            erode_once<CONN>(E);
            last = k == DW_MAX; // what is left is further than DW_MAX
            if (!inside_any()) {
                far = false;
                break;
            }
            if (last) break;
#pragma unroll
            for (int j = 0; j < DW_SLICES; ++j)
                if ((k + 1) % (1 << j) == 0)
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int i = 0; i < 4; ++i) S[j][r][i] ^= E[r][i];
        }
        dt_wave_sync(); // every lane has read its row bits
        const bool mine = ir >= 0 && ir < DW_IN;
#pragma unroll
        for (int g = 0; g < DW_IN / 4; ++g) {
            const int wd = (DW_MARGIN + 4 * g) >> 5, sb = (DW_MARGIN + 4 * g) & 31;
            uint32_t v[2] = {0, 0};
            if (__ballot((((fg[0][wd] | fg[1][wd]) >> sb) & 15u) != 0) != 0) {
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    // a nibble's bits spread to the low bits of four bytes
                    auto spread = [&](uint32_t w) -> uint32_t {
                        return (__builtin_amdgcn_ubfe(w, sb, 4) * 0x204081u) & 0x01010101u;
                    };
#pragma unroll
                    for (int j = 0; j < DW_SLICES; ++j) v[r] |= spread(S[j][r][wd]) << j;
                    if (far) v[r] |= spread(E[r][wd]) * DW_FAR;
                }
            }
            if (mine) {
                buf[ir * DW_ROW + g] = v[0];
                buf[(ir + 1) * DW_ROW + g] = v[1];
            }
        }
        dt_wave_sync();
    }
    // 8 lanes a row, 16 bytes (four pixels) a lane and store
    const int c4 = 4 * (lane & 7);
    int32_t *out = dist + y0 * dpitch + x0;
#pragma unroll 2
    for (int it = 0; it < DW_IN / 8; ++it) {
        const int r = 8 * it + (lane >> 3);
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int c = 32 * j + c4;
            v4u v = {0, 0, 0, 0};
            if (some) {
                const uint32_t b = buf[r * DW_ROW + c / 4];
                v = v4u{b & 0xFFu, (b >> 8) & 0xFFu, (b >> 16) & 0xFFu, b >> 24};
                if (far)
#pragma unroll
                    for (int k = 0; k < 4; ++k) v[k] = v[k] == DW_FAR ? INF : v[k];
            }
            if (r >= in_rows) continue;
            int32_t *o = out + r * dpitch + c;
            const int left = i_hi - DW_MARGIN - c; // pixels of the row from here on
            if (left >= 4) {
                __builtin_nontemporal_store(v, (v4u_dw *)o);
            } else {
                if (left > 0) o[0] = (int32_t)v.x;
                if (left > 1) o[1] = (int32_t)v.y;
                if (left > 2) o[2] = (int32_t)v.z;
            }
        }
    }
    if (!last) return;
    // List for round 2 the register tiles (DI x DI interiors) that hold an unsettled
    // pixel next to a settled one: only there can a visit change anything yet, and
    // the wave goes on from there (an image of one large object without background
    // has none: 8192 x 8192 143 us, 305 us with all its tiles listed). Looked for in the
    // interior and the pixels around it: a pixel of the interior counts as settled
    // only if it is, and one around it as unsettled if it is, so of each such pair
    // the window whose interior holds the settled pixel finds the other. At most
    // 3 x 3 tiles.
    uint32_t next[2][4];
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) next[r][i] = E[r][i];
    erode_once<CONN>(next);
    const int f_lo = std::max(c_lo, DW_MARGIN - 1), f_hi = std::min(c_hi, DW_MARGIN + DW_IN + 1);
    const int g_lo = std::max(r_lo, DW_MARGIN - 1), g_hi = std::min(r_hi, DW_MARGIN + DW_IN + 1);
    uint32_t any = 0;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const bool in = 2 * lane + r >= g_lo && 2 * lane + r < g_hi;
            E[r][i] = in ? E[r][i] & ~next[r][i] & cols(f_lo, f_hi, i) : 0u;
            any |= E[r][i];
        }
    if (__ballot(any != 0) == 0) return;
    const int64_t ty0 = (y0 > 0 ? y0 - 1 : 0) / DI, tx0 = (x0 > 0 ? x0 - 1 : 0) / DI;
    bool want = false;
#pragma unroll 1
    for (int q = 0; q < 9; ++q) {
        // the tile's columns and rows in the window
        const int a = (int)((tx0 + q % 3) * DI - wx0), b = a + DI;
        const int ra = (int)((ty0 + q / 3) * DI - wy0), rb = ra + DI;
        uint32_t hit[2] = {0, 0};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t m = cols(a, b, i);
            hit[0] |= E[0][i] & m;
            hit[1] |= E[1][i] & m;
        }
        const int y = 2 * lane;
        const bool here =
            (y >= ra && y < rb && hit[0] != 0) || (y + 1 >= ra && y + 1 < rb && hit[1] != 0);
        const bool listed = __ballot(here) != 0;
        if (lane == q) want = listed;
    }
    if (want) { // (unsettled pixels lie in the image, so the tile exists)
        const int64_t n = (int64_t)ntx * nty;
        const int64_t t = (ty0 + lane / 3) * ntx + tx0 + lane % 3;
        if (atomicMax(flags + t, 2u) < 2u) {
            const uint32_t slot = atomicAdd(&ctrl->marked[2], 1u);
            if ((int64_t)slot < n) lists[slot] = (uint32_t)t;
        }
    }
}

// One visit of tile t by the calling wave (every lane, uniform t). A tile
// raised past `round` before its visit is left to the later round it is
// listed for. `tb` is the wave's transpose buffer.
template <int CONN>
__device__ __forceinline__ void dt_visit(int32_t *__restrict__ dist, int64_t dpitch, int64_t H,
                                         int64_t W, int32_t ntx, int32_t nty,
                                         uint32_t *__restrict__ flags, uint32_t round,
                                         DtCtrl *__restrict__ ctrl, uint32_t *__restrict__ lists,
                                         int64_t t, uint32_t (*tb)[DS + 1]) {
    const int lane = threadIdx.x;
    if (flags[t] != round) return;
    const int ty = (int)(t / ntx), tx = (int)(t - (int64_t)ty * ntx);
    const int64_t gy0 = (int64_t)ty * DI - 1, gx = (int64_t)tx * DI - 1 + lane;
    const bool xin = gx >= 0 && gx < W;
    const bool in_lane = lane >= 1 && lane <= DS - 2;

    // Pixels outside the image are never reached and never lower anything.
    // Every row is loaded from a clamped, in-bounds address and masked
    // afterwards. All 64 loads are issued before any of them is used (the
    // compiler otherwise placed each use, and a wait, right after its load).
    // Rows are addressed from the tile's first in-image row (a uniform base)
    // with 32-bit lane offsets, so a load in flight holds one address
    // register rather than two.
    uint32_t D[DS];
    const int64_t xc = gx < 0 ? 0 : (gx > W - 1 ? W - 1 : gx);
    const int64_t y_first = gy0 < 0 ? 0 : gy0;
    const int32_t *db = dist + y_first * dpitch;
    if (gy0 >= 0 && gy0 + DS <= H) {
        // every row inside the image: the row offset lives in a vector
        // register, stepped by one pitch per row, so that the 64 row offsets
        // are not all held (in scalar registers, which spill)
        const uint32_t pitch = (uint32_t)dpitch;
        uint32_t off = (uint32_t)xc;
#pragma unroll
        for (int r = 0; r < DS; ++r) {
            asm volatile("" : "+v"(off));
            D[r] = (uint32_t)db[off];
            off += pitch;
        }
    } else {
        // the top or bottom tile row: rows outside the image read the
        // nearest row inside it (masked below); the clamp is vector
        // arithmetic for the same reason
        int32_t g0 = (int32_t)(gy0 - y_first), hm = (int32_t)(H - 1 - y_first);
        asm volatile("" : "+v"(g0), "+v"(hm));
        const uint32_t pitch = (uint32_t)dpitch;
#pragma unroll
        for (int r = 0; r < DS; ++r) {
            const int32_t rel = min(max(g0 + r, 0), hm);
            const uint32_t off = (uint32_t)rel * pitch + (uint32_t)xc;
            D[r] = (uint32_t)db[off];
        }
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int r = 0; r < DS; ++r) asm volatile("" : "+v"(D[r]));
    // rows r_lo .. r_hi of the tile lie in the image; compared in vector
    // registers (as 64 scalar conditions they would be held and spilled)
    uint32_t r_lo = (uint32_t)(gy0 < 0 ? -gy0 : 0);
    uint32_t r_hi = (uint32_t)(H - 1 - gy0 < DS - 1 ? H - 1 - gy0 : DS - 1);
    asm volatile("" : "+v"(r_lo), "+v"(r_hi));
    // (0/1 arithmetic rather than comparisons: 64 rows of comparison masks
    // are held in scalar registers and spill)
    const uint32_t xin1 = xin ? 1u : 0u;
#pragma unroll
    for (int r = 0; r < DS; ++r) {
        // 1 for a row inside the image: neither r - r_lo nor r_hi - r is negative
        const uint32_t ok = xin1 & ~(((uint32_t)r - r_lo) | (r_hi - (uint32_t)r)) >> 31;
        D[r] = ok ? D[r] : INF;
    }
    // Pixels outside the image start unreached and may be lowered by the
    // sweeps like any other (a path through them is never shorter than one
    // along the image's edge, so they cannot shorten an inside distance), but
    // they are never stored and never count as a change. `valid` holds this
    // lane's interior pixels that lie in the image; rows 1.. are at or below
    // row 0 of the image, so only the bottom can run out.
    const bool col_ok = in_lane && xin;
    const int64_t rows_left = H - gy0 - 1; // interior rows inside the image
    const int last_row = rows_left < DS - 2 ? (int)rows_left : DS - 2;
    // (the bottom tile row compares each row with last_row in vector
    // registers: as scalar conditions the compiler keeps all 62 of them live
    // across the sweep loop, and they spill)
    auto vsum = [&]() {
        uint64_t sm = 0;
        if (last_row == DS - 2) {
#pragma unroll
            for (int r = 1; r < DS - 1; ++r) sm += D[r];
        } else {
            uint32_t lr = (uint32_t)last_row;
            asm volatile("" : "+v"(lr));
#pragma unroll
            for (int r = 1; r < DS - 1; ++r) sm += (uint32_t)r <= lr ? D[r] : 0u;
        }
        return col_ok ? sm : 0ull;
    };
    // border rows as loaded (what the neighbours' halos hold), and each
    // interior column's sum as loaded (distances only fall, so a column
    // changed iff its sum did)
    const uint32_t in_top = D[1], in_bot = D[DS - 2];
    const uint64_t sum_in = vsum();

    // Down and up sweeps (the neighbours in the adjacent row: three with
    // 8-connectivity, through lane shifts), then right and left sweeps on the
    // transposed tile (the in-row neighbour), once: between any two pixels of the
    // tile there is a shortest path of moves down (or up) only, diagonal and straight,
    // followed by moves along the row, so every interior pixel ends with the least
    // D(q) + d(q, p) over all pixels q of the tile, and by the triangle inequality a
    // second round of sweeps changes nothing. (8192 x 8192, squares of 300 pixels:
    // 628 us a call with a second round that confirmed it, 590 us without.)
#pragma unroll
    for (int r = 1; r < DS - 1; ++r) D[r] = min(D[r], reach<CONN>(D[r - 1]));
#pragma unroll
    for (int r = DS - 2; r >= 1; --r) D[r] = min(D[r], reach<CONN>(D[r + 1]));
    transpose(D, tb, lane); // lane = row, register = column
#pragma unroll
    for (int c = 1; c < DS - 1; ++c) D[c] = min(D[c], D[c - 1] + 1u);
#pragma unroll
    for (int c = DS - 2; c >= 1; --c) D[c] = min(D[c], D[c + 1] + 1u);
    transpose(D, tb, lane);
    const uint64_t sum = vsum();
    if (__ballot(sum != sum_in) == 0) return;
    if (in_lane && gx < W) {
        // rows gy0 + 1 .. are all >= 0; only the bottom may leave the image
        int32_t *drow = dist + (gy0 + 1) * dpitch;
        uint32_t off = (uint32_t)gx;
#pragma unroll
        for (int r = 1; r < DS - 1; ++r) {
            asm volatile("" : "+v"(off));
            if (r <= last_row) drow[off] = (int32_t)D[r];
            off += (uint32_t)dpitch;
        }
    }
    // mark for the next round every neighbour whose halo holds a border pixel
    // that changed here:
    // rows 1 and DS-2 (per lane), columns 1 and DS-2 (lanes 1 and DS-2),
    // and the corner pixels for the diagonal neighbours (8-connectivity)
    const uint64_t bt = __ballot(col_ok && D[1] != in_top);
    const uint64_t bb = __ballot(col_ok && last_row == DS - 2 && D[DS - 2] != in_bot);
    const uint64_t bc = __ballot(sum != sum_in);
    const uint32_t nxt = round + 1;
    bool want = false;
    int dy = 0, dx = 0;
    switch (lane) {
    case 1: want = bt != 0; dy = -1; break;
    case 2: want = bb != 0; dy = 1; break;
    case 3: want = (bc >> 1) & 1; dx = -1; break;
    case 4: want = (bc >> (DS - 2)) & 1; dx = 1; break;
    case 5: want = CONN == 8 && ((bt >> 1) & 1); dy = -1; dx = -1; break;
    case 6: want = CONN == 8 && ((bt >> (DS - 2)) & 1); dy = -1; dx = 1; break;
    case 7: want = CONN == 8 && ((bb >> 1) & 1); dy = 1; dx = -1; break;
    case 8: want = CONN == 8 && ((bb >> (DS - 2)) & 1); dy = 1; dx = 1; break;
    default: break;
    }
    const int ny = ty + dy, nx = tx + dx;
    if (want && ny >= 0 && ny < nty && nx >= 0 && nx < ntx) {
        const int64_t nb = (int64_t)ny * ntx + nx;
        // the first mark of a tile for round nxt lists it for that round
        if (atomicMax(flags + nb, nxt) < nxt) {
            const int64_t n = (int64_t)ntx * nty;
            const uint32_t slot = atomicAdd(&ctrl->marked[nxt & 3], 1u);
            if ((int64_t)slot < n) lists[(int64_t)(nxt & 1) * n + slot] = (uint32_t)nb;
        }
    }
}

// A round visits the
// tiles listed for it (each at most once: a tile is listed when its flag
// first reaches the round), a fixed grid of waves walking the list, so that
// a round with few marked tiles does not launch a wave per tile.
template <int CONN>
__global__ __launch_bounds__(64) void k_dt_round(int32_t *__restrict__ dist, int64_t dpitch,
                                                 int64_t H, int64_t W, int32_t ntx, int32_t nty,
                                                 uint32_t *__restrict__ flags, uint32_t round,
                                                 DtCtrl *__restrict__ ctrl,
                                                 uint32_t *__restrict__ lists) {
    __shared__ uint32_t tb[DS][DS + 1];
    const int64_t n = (int64_t)ntx * nty;
    const int64_t cnt = std::min<int64_t>(ctrl->marked[round & 3], n);
    if (blockIdx.x == 0 && threadIdx.x == 0) ctrl->marked[(round + 2) & 3] = 0;
    const uint32_t *list = lists + (int64_t)(round & 1) * n;
    for (int64_t i = blockIdx.x; i < cnt; i += gridDim.x)
        dt_visit<CONN>(dist, dpitch, H, W, ntx, nty, flags, round, ctrl, lists, (int64_t)list[i],
                       tb);
}

__global__ void k_dt_clear(DtCtrl *c, uint32_t *flags, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) {
        c->has_bg = 0;
        for (int k = 0; k < 4; ++k) c->marked[k] = 0;
    }
    for (int64_t k = i; k < n; k += (int64_t)gridDim.x * blockDim.x) flags[k] = 0;
}

__global__ void k_dt_fill(int32_t *dist, int64_t dpitch, int64_t H, int64_t W, int32_t v) {
    const int64_t n = H * W;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t y = i / W;
        dist[y * dpitch + (i - y * W)] = v;
    }
}

struct DtLayout {
    size_t ctrl = 0, flags = 0, lists = 0, total = 0;
    int64_t ntx = 0, nty = 0;
};

DtLayout dt_layout(int64_t H, int64_t W) {
    DtLayout L;
    L.ntx = (W + DI - 1) / DI;
    L.nty = (H + DI - 1) / DI;
    L.ctrl = 0;
    L.flags = up256(sizeof(DtCtrl));
    L.lists = L.flags + up256((size_t)(L.ntx * L.nty) * 4);
    L.total = L.lists + up256((size_t)(L.ntx * L.nty) * 8); // one list per round parity
    return L;
}

hipError_t dt_first(int conn, const uint8_t *img, int64_t ipitch, int32_t *dist, int64_t dpitch,
                    int64_t H, int64_t W, const DtLayout &L, uint32_t *flags, uint32_t *lists,
                    DtCtrl *ctrl, hipStream_t s) {
    const int64_t wtx = (W + DW_IN - 1) / DW_IN, n = wtx * ((H + DW_IN - 1) / DW_IN);
    const dim3 g((unsigned)((n + DW_WAVES - 1) / DW_WAVES)), b(64 * DW_WAVES);
    if (conn == 8)
        hipLaunchKernelGGL(k_dt_first<8>, g, b, 0, s, img, ipitch, dist, dpitch, H, W, wtx, n,
                           (int32_t)L.ntx, (int32_t)L.nty, flags, ctrl, lists);
    else
        hipLaunchKernelGGL(k_dt_first<4>, g, b, 0, s, img, ipitch, dist, dpitch, H, W, wtx, n,
                           (int32_t)L.ntx, (int32_t)L.nty, flags, ctrl, lists);
    return hipGetLastError();
}

hipError_t dt_round(int conn, int32_t *dist, int64_t dpitch, int64_t H, int64_t W,
                    const DtLayout &L, uint32_t *flags, uint32_t *lists, uint32_t round,
                    DtCtrl *ctrl, hipStream_t s) {
    // a fixed grid walks the round's list (the count is on the
    // device); 8192 waves (measured against 2048 to 32768)
    const dim3 g((unsigned)std::min<int64_t>(L.ntx * L.nty, 8192));
    if (conn == 8)
        hipLaunchKernelGGL(k_dt_round<8>, g, dim3(64), 0, s, dist, dpitch, H, W, (int32_t)L.ntx,
                           (int32_t)L.nty, flags, round, ctrl, lists);
    else
        hipLaunchKernelGGL(k_dt_round<4>, g, dim3(64), 0, s, dist, dpitch, H, W, (int32_t)L.ntx,
                           (int32_t)L.nty, flags, round, ctrl, lists);
    return hipGetLastError();
}

} // namespace

extern "C" {

size_t mr_distance_transform_workspace_bytes(int64_t H, int64_t W, int conn) {
    clear_error();
    if (H < 1 || W < 1 || (conn != 4 && conn != 8)) {
        dfail(MR_EINVAL, "bad arguments");
        return 0;
    }
    return dt_layout(H, W).total;
}

int mr_distance_transform(const void *img, void *dist, int64_t H, int64_t W, int64_t pitch,
                          int64_t dist_pitch, int conn, void *ws, size_t ws_bytes,
                          void *stream) {
    clear_error();
    if (pitch == 0) pitch = W;
    if (dist_pitch == 0) dist_pitch = W;
    if (H < 1 || W < 1) return dfail(MR_EINVAL, "H and W must be >= 1");
    if (pitch < W || dist_pitch < W) return dfail(MR_EINVAL, "a pitch is below W");
    if (conn != 4 && conn != 8) return dfail(MR_EINVAL, "conn must be 4 or 8 (got %d)", conn);
    if (!img || !dist || !ws) return dfail(MR_EINVAL, "null pointer");
    if ((uintptr_t)dist % 4) return dfail(MR_EINVAL, "dist must be 4-byte aligned");
    if ((uintptr_t)ws % 256) return dfail(MR_EINVAL, "workspace must be 256-byte aligned");
    const DtLayout L = dt_layout(H, W);
    if (L.ntx * L.nty >= (1ll << 31)) return dfail(MR_EINVAL, "image too large");
    if (ws_bytes < L.total)
        return dfail(MR_ENOMEM, "workspace too small: %zu bytes given, %zu needed", ws_bytes,
                     L.total);
    hipStream_t s = (hipStream_t)stream;
    DtCtrl *ctrl = (DtCtrl *)((char *)ws + L.ctrl);
    uint32_t *flags = (uint32_t *)((char *)ws + L.flags);
    uint32_t *lists = (uint32_t *)((char *)ws + L.lists);
    const uint8_t *im = (const uint8_t *)img;
    int32_t *d = (int32_t *)dist;
    const int64_t n = L.ntx * L.nty;
    hipLaunchKernelGGL(k_dt_clear, dim3((unsigned)std::min<int64_t>((n + 255) / 256 + 1, 4096)),
                       dim3(256), 0, s, ctrl, flags, n);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return dhip(e, "clear");
    // the first pass (round 1) settles what the windows can; later rounds visit
    // the tiles marked for them, DT_BATCH rounds per host poll of the marks
    uint32_t round = 1;
    if ((e = dt_first(conn, im, pitch, d, dist_pitch, H, W, L, flags, lists, ctrl, s)) != hipSuccess)
        return dhip(e, "first pass");
    DtCtrl h;
    while (true) {
        if ((e = hipMemcpyAsync(&h, ctrl, sizeof h, hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return dhip(e, "poll");
        // tiles the last round marked for the next one
        const uint32_t h_marked = h.marked[(round + 1) & 3];
        if (h_marked == 0) break;
        if ((int64_t)round > DT_MAX_ROUNDS)
            return dfail(MR_EHIP, "distance transform did not converge");
        // the next DT_BATCH rounds; a round that finds no tile marked for it
        // changes nothing, so a batch that overshoots the end is harmless
        for (int k = 0; k < DT_BATCH; ++k) {
            ++round;
            if ((e = dt_round(conn, d, dist_pitch, H, W, L, flags, lists, round, ctrl, s)) !=
                hipSuccess)
                return dhip(e, "round");
        }
    }
    if (!h.has_bg) {
        const int64_t items = H * W;
        hipLaunchKernelGGL(k_dt_fill, dim3((unsigned)std::min<int64_t>((items + 255) / 256, 65536)),
                           dim3(256), 0, s, d, dist_pitch, H, W, -1);
        if ((e = hipGetLastError()) != hipSuccess) return dhip(e, "fill");
    }
    return MR_OK;
}

} // extern "C"
