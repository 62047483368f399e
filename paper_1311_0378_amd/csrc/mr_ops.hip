// mr_ops.hip -- the regular operations of Table II and the reconstruction-based
// wrappers (include/mr_ops.h): h-dome, regional maxima, RGB to grayscale and
// opening by a 13 x 13 disk.
//
// All of these are streaming passes over HBM (Sec. V-C.1's regular,
// memory-bound class) except the reconstruction inside the wrappers, which
// runs on the engine of mr.h.
#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <type_traits>

#include "../../include/mr_ops.h"
#include "mr_internal.h"

using namespace mr;

namespace {

int ofail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    return set_error(code, buf);
}

int ohip(hipError_t e, const char *what) {
    return ofail(MR_EHIP, "%s: %s", what, hipGetErrorString(e));
}

size_t up256(size_t n) { return (n + 255) / 256 * 256; }

int check_dims(int64_t H, int64_t W, int64_t pitch, int64_t elem_bytes) {
    if (H < 1 || W < 1) return ofail(MR_EINVAL, "H and W must be >= 1 (got %lld x %lld)",
                                     (long long)H, (long long)W);
    if (pitch < W) return ofail(MR_EINVAL, "pitch %lld is below W %lld", (long long)pitch,
                                (long long)W);
    if ((double)H * (double)pitch * (double)elem_bytes >= 9.0e18)
        return ofail(MR_EINVAL, "image too large");
    return MR_OK;
}

unsigned grid_for(int64_t items, int per_block) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + per_block - 1) / per_block,
                                                            1 << 20));
}

// ------------------------------------------------------ h-dome, regional max

// Pixel keys of the two types (the key order is the pixel order; key 0 is
// the type's minimum).
template <typename T> struct K;
template <> struct K<uint8_t> {
    __device__ static uint32_t key(uint8_t v) { return v; }
    __device__ static uint8_t val(uint32_t k) { return (uint8_t)k; }
};
template <> struct K<int32_t> {
    __device__ static uint32_t key(int32_t v) { return (uint32_t)v ^ 0x80000000u; }
    __device__ static int32_t val(uint32_t k) { return (int32_t)(k ^ 0x80000000u); }
};

// The streaming passes of the wrappers, one kind each (the marker f - h is made by
// the reconstruction's first round, which finds out whether some pixel is above
// the type's minimum, *above):
//  P_DOME:   f <- f - r (the h-dome; r <= f everywhere, so 0 <= f - r <= h);
//  P_RMAX:   out = 255 where f > r (a dome of height 1), or everywhere when
//            no pixel is above the minimum (*above == 0); else 0.
// With WORDS every lane takes one 16-byte word of a row (planes whose base
// and pitch are multiples of 16 bytes; the u8 output of P_RMAX likewise, in
// 16 / sizeof(T)-byte pieces), else one pixel. A row's last word may be
// partial and goes pixel by pixel. Grid-stride over a grid of at most
// MAX_STREAM_BLOCKS blocks.
enum { P_DOME = 1, P_RMAX = 2 };
constexpr int64_t MAX_STREAM_BLOCKS = 4096;

template <typename T> struct alignas(16) Word {
    T e[16 / sizeof(T)];
};

template <typename T, int KIND>
__device__ __forceinline__ void pass_pixel(const T *f, const T *r, T *m, uint8_t *o, bool all_min,
                                           int64_t i, int64_t oi) {
    const uint32_t kf = K<T>::key(f[i]);
    if (KIND == P_DOME) {
        m[i] = (T)(int32_t)(kf - K<T>::key(r[i])); // m aliases f here
    } else {
        o[oi] = (all_min || kf > K<T>::key(r[i])) ? 255 : 0;
    }
}

// 0xFF in every byte of x that is nonzero, 0 in the others: the low seven
// bits of a byte plus 0x7F carry into its top bit iff they are nonzero, and
// the byte's own top bit covers the rest; no carry leaves a byte.
__device__ __forceinline__ uint32_t bytes_nonzero(uint32_t x) {
    const uint32_t top = (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
    return (top >> 7) * 0xFFu;
}

template <typename T, int KIND, bool WORDS>
__global__ __launch_bounds__(256) void k_stream_pass(const T *f, const T *r, T *m,
                                                     uint8_t *__restrict__ o, int64_t H,
                                                     int64_t W, int64_t pitch, int64_t out_pitch,
                                                     const uint32_t *above) {
    constexpr int EPW = WORDS ? 16 / (int)sizeof(T) : 1;
    const int64_t wpr = (W + EPW - 1) / EPW; // items per row
    const bool all_min = KIND == P_RMAX && *above == 0;
    for (int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; it < H * wpr;
         it += (int64_t)gridDim.x * blockDim.x) {
        const int64_t y = it / wpr, x0 = (it - y * wpr) * EPW;
        const int64_t i0 = y * pitch + x0, o0 = y * out_pitch + x0;
        if (WORDS && sizeof(T) == 1 && x0 + EPW <= W) {
            // uint8 dome and maxima on whole dwords: r <= f in every byte, so
            // f - r as 32-bit words subtracts byte by byte without borrows
            const uint4 wf = *(const uint4 *)(f + i0), wr = *(const uint4 *)(r + i0);
            uint4 d = {wf.x - wr.x, wf.y - wr.y, wf.z - wr.z, wf.w - wr.w};
            if (KIND == P_DOME) {
                *(uint4 *)(m + i0) = d;
            } else {
                *(uint4 *)(o + o0) = all_min ? uint4{~0u, ~0u, ~0u, ~0u}
                                             : uint4{bytes_nonzero(d.x), bytes_nonzero(d.y),
                                                     bytes_nonzero(d.z), bytes_nonzero(d.w)};
            }
        } else if (WORDS && x0 + EPW <= W) {
            const Word<T> wf = *(const Word<T> *)(f + i0), wr = *(const Word<T> *)(r + i0);
            if (KIND == P_DOME) {
                Word<T> wm;
#pragma unroll
                for (int e = 0; e < EPW; ++e)
                    wm.e[e] = (T)(int32_t)(K<T>::key(wf.e[e]) - K<T>::key(wr.e[e]));
                *(Word<T> *)(m + i0) = wm;
            } else { // (uint8 words went the other way: four pixels here)
                uint32_t v = 0;
#pragma unroll
                for (int e = 0; e < EPW; ++e)
                    v |= (all_min || K<T>::key(wf.e[e]) > K<T>::key(wr.e[e]) ? 255u : 0u) << (8 * (e & 3));
                *(uint32_t *)(o + o0) = v;
            }
        } else {
            for (int e = 0; e < EPW && x0 + e < W; ++e)
                pass_pixel<T, KIND>(f, r, m, o, all_min, i0 + e, o0 + e);
        }
    }
}

bool words_ok(const void *p, int64_t pitch_bytes) {
    return ((uintptr_t)p & 15) == 0 && (pitch_bytes & 15) == 0;
}

template <typename T, int KIND>
hipError_t stream_pass(const T *f, const T *r, T *m, uint8_t *o, int64_t H, int64_t W,
                       int64_t pitch, int64_t out_pitch, const uint32_t *above, hipStream_t s) {
    if (pitch == W && (KIND != P_RMAX || out_pitch == W)) { // rows without gaps: one long row
        W = pitch = out_pitch = H * W;
        H = 1;
    }
    // (a single row's pitch does not matter)
    const int64_t pb = H == 1 ? 0 : pitch * (int64_t)sizeof(T);
    bool words = words_ok(f, pb) && words_ok(r, pb) &&
                 (KIND == P_RMAX || words_ok(m, pb));
    if (KIND == P_RMAX)
        words = words && ((uintptr_t)o % (16 / sizeof(T))) == 0 &&
                (H == 1 || out_pitch % (int64_t)(16 / sizeof(T)) == 0);
    const int64_t epw = words ? 16 / (int64_t)sizeof(T) : 1;
    const int64_t items = H * ((W + epw - 1) / epw);
    const unsigned g =
        (unsigned)std::max<int64_t>(1, std::min<int64_t>((items + 255) / 256, MAX_STREAM_BLOCKS));
    if (words)
        hipLaunchKernelGGL((k_stream_pass<T, KIND, true>), dim3(g), dim3(256), 0, s, f, r, m, o,
                           H, W, pitch, out_pitch, above);
    else
        hipLaunchKernelGGL((k_stream_pass<T, KIND, false>), dim3(g), dim3(256), 0, s, f, r, m, o,
                           H, W, pitch, out_pitch, above);
    return hipGetLastError();
}

struct HdomeLayout {
    size_t recon = 0, plane = 0, flag = 0, total = 0;
};

int hdome_layout(int64_t H, int64_t W, int64_t pitch, int t, int conn, const mr_tune *tune,
                 HdomeLayout &L) {
    const size_t r = mr_workspace_bytes(MR_OP_RECON, H, W, (mr_dtype)t, conn, tune);
    if (r == 0) return MR_EINVAL; // the message is set
    L.recon = up256(r);
    L.plane = L.recon;
    L.flag = L.plane + up256((size_t)H * (size_t)pitch * (size_t)t);
    L.total = L.flag + 256;
    return MR_OK;
}

int hdome_common(const void *img, int64_t H, int64_t W, int64_t &pitch, int t, int conn,
                 void *ws, size_t ws_bytes, const mr_tune *tune, HdomeLayout &L) {
    clear_error();
    if (t != MR_U8 && t != MR_I32) return ofail(MR_EINVAL, "unknown pixel type %d", t);
    if (pitch == 0) pitch = W;
    int rc;
    if ((rc = check_dims(H, W, pitch, t)) != MR_OK) return rc;
    if (!img || !ws) return ofail(MR_EINVAL, "null image or workspace");
    if ((uintptr_t)ws % 256) return ofail(MR_EINVAL, "workspace must be 256-byte aligned");
    if ((uintptr_t)img % t) return ofail(MR_EINVAL, "image must be aligned to the pixel size");
    if ((rc = hdome_layout(H, W, pitch, t, conn, tune, L)) != MR_OK) return rc;
    if (ws_bytes < L.total)
        return ofail(MR_ENOMEM, "workspace too small: %zu bytes given, %zu needed", ws_bytes,
                     L.total);
    return MR_OK;
}

// ------------------------------------------------------------------ RGB2Gray

// BT.601 luma weights in 14-bit fixed point (0.299, 0.587, 0.114; sum 2^14)
constexpr uint32_t WR = 4899u, WG = 9617u, WB = 1868u;

__device__ __forceinline__ uint32_t luma(uint32_t r, uint32_t g, uint32_t b) {
    return (WR * r + WG * g + WB * b + 8192u) >> 14;
}

// 16 pixels per lane from three 16-byte words (48 bytes = 16 RGB triples),
// one 16-byte word out. Rows and both planes are 16-byte aligned; vec = the
// whole 16-pixel groups per row. The `rest` pixels past the last row's groups
// (of a plane without gaps, one long row) go one a lane.
__global__ __launch_bounds__(256) void k_rgb2gray16(const uint8_t *__restrict__ rgb,
                                                    int64_t rgb_pitch, uint8_t *__restrict__ gray,
                                                    int64_t gray_pitch, int64_t H, int64_t vec,
                                                    int rest) {
    if (blockIdx.x == 0 && (int)threadIdx.x < rest) {
        const int64_t x = vec * 16 + threadIdx.x;
        const uint8_t *p = rgb + (H - 1) * rgb_pitch + 3 * x;
        gray[(H - 1) * gray_pitch + x] = (uint8_t)luma(p[0], p[1], p[2]);
    }
    const int64_t items = H * vec;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < items;
         i += (int64_t)gridDim.x * 256) {
        const int64_t y = i / vec, g = i - y * vec;
        const uint4 *src = (const uint4 *)(rgb + y * rgb_pitch + g * 48);
        const uint4 a = src[0], b = src[1], c = src[2];
        const uint32_t w[12] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w, c.x, c.y, c.z, c.w};
        uint32_t o[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int p = 0; p < 16; ++p) {
            const int q = 3 * p; // byte index of this pixel's R
            const uint32_t r = (w[q >> 2] >> ((q & 3) * 8)) & 0xFFu;
            const uint32_t gg = (w[(q + 1) >> 2] >> (((q + 1) & 3) * 8)) & 0xFFu;
            const uint32_t bb = (w[(q + 2) >> 2] >> (((q + 2) & 3) * 8)) & 0xFFu;
            o[p >> 2] |= luma(r, gg, bb) << ((p & 3) * 8);
        }
        *(uint4 *)(gray + y * gray_pitch + g * 16) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// One pixel per lane, for unaligned planes and the columns past the last
// whole 16-pixel group (x0 = first column handled).
__global__ __launch_bounds__(256) void k_rgb2gray1(const uint8_t *__restrict__ rgb,
                                                   int64_t rgb_pitch, uint8_t *__restrict__ gray,
                                                   int64_t gray_pitch, int64_t H, int64_t x0,
                                                   int64_t W) {
    const int64_t cols = W - x0, items = H * cols;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < items;
         i += (int64_t)gridDim.x * 256) {
        const int64_t y = i / cols, x = x0 + (i - y * cols);
        const uint8_t *p = rgb + y * rgb_pitch + 3 * x;
        gray[y * gray_pitch + x] = (uint8_t)luma(p[0], p[1], p[2]);
    }
}

// -------------------------------------------------------- 13 x 13 disk

// The disk of radius 6 as rows: offset dy has half-width 6, 5, 5, 5, 4, 3, 0 at
// |dy| = 0..6 (dy^2 + dx^2 <= 36).
// One wave per workgroup. A wave's 64 lanes cover a window of 256 adjacent
// columns, 4 per lane, and it produces the 240 columns of lanes 2..61 for `th`
// rows: an extremum over 13 columns needs 6 columns on each side, and lanes 0,
// 1, 62 and 63 supply them. Per input row each lane loads the dword of its 4
// columns, forms the horizontal extrema of half-widths 1, 3, 4, 5 and 6 of its
// own columns, taking the few values it needs of the neighbouring lanes' columns
// by lane shifts (DPP, which the two-operand extrema take along), and combines
// them down the rows with three-operand extrema: the seven rows of half-width 5
// (row 0's half-width 6 covers its own) by a running extremum over 3 and 7
// rows, the others in 13 accumulators, one per output row still open, which
// take their values in pairs. That is 24 + 24 extrema for 4 pixels.
// Pixels outside the image read as the operation's identity (255 for the
// erosion, 0 for the dilation), which leaves the extrema over the inside offsets.
// Bound by instruction issue: 60 vector instructions a step and wave, which take 94 %
// of the issue slots while the chip is full; 16384 x 16384 takes 160 us a
// pass (3.4 TB/s), 238 us when 13 rows folded into 13 packed 16-bit accumulators
// (packed 16-bit extrema issue at half rate: two strips sharing 16-bit halves
// took 228 us). Without the die-wise order of the strips: 182 us.
constexpr int DK_OUT = 240;         // output columns per wave (lanes 2..61)
constexpr int DK_WAVES_PER_SIMD = 4; // by its registers

template <bool MIN> __device__ __forceinline__ uint32_t ext(uint32_t a, uint32_t b) {
    return MIN ? min(a, b) : max(a, b);
}
// (opaque: an accumulator's extrema are associative, and the compiler would
// gather them at the row that completes it, keeping all their operands alive)
template <bool MIN> __device__ __forceinline__ uint32_t ext3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    if (MIN)
        asm("v_min3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    else
        asm("v_max3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// Lane i gets lane i-1's value; lane i gets lane i+1's value. Lanes 0 and 63
// get 0 from the missing neighbour; only columns of lanes 0, 1, 62 and 63
// depend on those values, and they are not stored.
__device__ __forceinline__ uint32_t from_left(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF,
                                                 true);
}
__device__ __forceinline__ uint32_t from_right(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF,
                                                 true);
}

template <bool MIN>
__global__ __launch_bounds__(64, DK_WAVES_PER_SIMD) void k_disk13(const uint8_t *__restrict__ in,
                                                                  uint8_t *__restrict__ out,
                                                                  int64_t H, int64_t W,
                                                                  int64_t pitch, uint32_t tiles_x,
                                                                  uint32_t tiles, int th) {
    const uint32_t ident4 = MIN ? 0xFFFFFFFFu : 0u;
    const int lane = threadIdx.x;
    // (read back to scalars: the division runs on the vector unit)
    // Workgroups go to the eight dies in turn: each die takes a contiguous range of
    // strips, so that neighbouring strips, which share cache lines at both ends of
    // every row (240 columns are no whole lines), share them in one L2.
    const uint32_t per = gridDim.x / 8, tile = (blockIdx.x & 7) * per + blockIdx.x / 8;
    if (tile >= tiles) return;
    const uint32_t ty = (uint32_t)__builtin_amdgcn_readfirstlane(tile / tiles_x);
    const uint32_t tx = tile - ty * tiles_x;
    const int64_t y0 = (int64_t)ty * th;           // the strip's first output row
    const int64_t gx0 = (int64_t)tx * DK_OUT - 8;  // the window's first column
    const int x = 4 * lane;                        // this lane's first column in the window
    // rows of the image from y0 (as far as the strip reaches; 32-bit compares),
    // and the window's columns inside the image
    const int y_lo = (int)-std::min<int64_t>(y0, 1 << 30), y_hi = (int)std::min<int64_t>(H - y0, 1 << 30);
    const int x_lo = gx0 < 0 ? (int)-gx0 : 0, x_hi = (int)std::min<int64_t>(256, W - gx0);
    // Three forms of a strip. Dword-aligned rows: a row is one dword load per lane
    // from the row's uniform base, with nothing else to do where the window and
    // the input rows all lie inside the image (FAST); else rows outside the image
    // and columns outside it take the identity (their loads are moved to the
    // nearest row and dword inside). Other rows (SHIFTED): the
    // aligned dword below the lane's pixels, and the row's misalignment
    // shifted out with the next lane's dword.
    const int steps = th + 12; // (a multiple of 13: see disk_rows)
    const bool aligned = ((((uintptr_t)in) | (uintptr_t)pitch) & 3) == 0;
    const bool whole = x_lo == 0 && x_hi == 256 && y_lo <= -6 && y_hi >= th + 6;
    uint32_t inside = 0; // 0xFF in every byte whose column lies in the image
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (x + c >= x_lo && x + c < x_hi) inside |= 0xFFu << (8 * c);
    // The nearest row of the image (uniform; opaque, so that a row's address is
    // this base and a 32-bit lane offset, not a 64-bit address per lane and row).
    typedef const __attribute__((address_space(1))) uint8_t *row_t;
    const row_t in0 = (row_t)in + y0 * pitch + gx0;
    auto row_of = [&](int y) -> row_t { // y: from the strip's first output row
        row_t p = in0 + (int64_t)(y < y_lo ? y_lo : (y >= y_hi ? y_hi - 1 : y)) * pitch;
        asm volatile("" : "+s"(p));
        return p;
    };
    typedef const __attribute__((address_space(1))) uint32_t *word_t;

    // 13 accumulators per column in a ring: output row o (strip-relative) lives
    // in slot o mod 13. Step r's input row r - 6 opens output row r and
    // completes output row r - 12; the rows are walked 13 at a time so that
    // every slot index is a constant.
    const uint32_t ident = ident4 & 0xFFu;
    uint32_t acc[13][4];
    uint32_t e5p[2][4], t3[4][4]; // half-width 5: the rows before; threes of rows before
    uint32_t e3p[4], p7p[4];      // the row before: half-width 3; seven rows of half-width 5
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int k = 0; k < 13; ++k) acc[k][c] = ident;
        e5p[0][c] = e5p[1][c] = e3p[c] = p7p[c] = ident;
#pragma unroll
        for (int k = 0; k < 4; ++k) t3[k][c] = ident;
    }
    const bool stores = lane >= 2 && lane < 62 && x < x_hi;
    typedef __attribute__((address_space(1))) uint8_t *orow_t;
    auto strip = [&](auto kind) {
    constexpr bool FAST = decltype(kind)::value == 0, SHIFTED = decltype(kind)::value == 2;
    row_t next_in = in0 - 6 * pitch;                              // FAST: the next row to load
    orow_t next_out = (orow_t)out + (y0 - 12) * pitch + gx0;      // the next step's output row
#pragma unroll 1
    for (int r0 = 0; r0 < steps; r0 += 13) {
        uint32_t w[13]; // this lane's dwords of 13 rows
        const int ra = r0 - 6;
        if (FAST) {
#pragma unroll
            for (int rr = 0; rr < 13; ++rr) {
                // (one row at a time: the scheduler would hold all the addresses)
                w[rr] = *(word_t)(next_in + (uint32_t)x);
                next_in += pitch;
                asm volatile("" : "+s"(next_in));
            }
        } else {
            uint32_t after[13]; // (lane 63 has no next lane: the dword after its own)
#pragma unroll
            for (int rr = 0; rr < 13; ++rr) {
                row_t row = row_of(ra + rr);
                const int mis = SHIFTED ? (int)((uintptr_t)row & 3) : 0;
                // dwords of the row start at multiples of 4 from row - mis (gx0 is one)
                const int last = (x_hi - 1 + mis) & ~3;
                const int o = x < (x_lo & ~3) ? x_lo & ~3 : (x > last ? last : x);
                if (SHIFTED) {
                    row -= mis;
                    asm volatile("" : "+s"(row));
                }
                w[rr] = *(word_t)(row + (uint32_t)o);
                if (SHIFTED) after[rr] = *(word_t)(row + (uint32_t)std::min(256, last));
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int rr = 0; rr < 13; ++rr) {
                if (SHIFTED) {
                    const uint32_t mis = (uint32_t)((uintptr_t)row_of(ra + rr) & 3);
                    const uint32_t next = (uint32_t)__builtin_amdgcn_update_dpp(
                        (int)after[rr], (int)w[rr], 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
                    w[rr] = __builtin_amdgcn_alignbyte(next, w[rr], mis);
                    __builtin_amdgcn_sched_barrier(0);
                }
                w[rr] = (w[rr] & inside) | (ident4 & ~inside);
            }
        }
#pragma unroll
        for (int rr = 0; rr < 13; ++rr) {
            const int r = r0 + rr;
            const uint32_t v = FAST || (ra + rr >= y_lo && ra + rr < y_hi) ? w[rr] : ident4;
            uint32_t b[4], e1[4], e3[4], e4[4], e5[4], e6[4];
            b[0] = v & 0xFFu;
            b[1] = __builtin_amdgcn_ubfe(v, 8, 8);
            b[2] = __builtin_amdgcn_ubfe(v, 16, 8);
            b[3] = v >> 24;
            // e_w[c]: the extremum over columns c - w .. c + w
            {
                const uint32_t m01 = ext<MIN>(b[0], b[1]), m23 = ext<MIN>(b[2], b[3]);
                e1[0] = ext<MIN>(from_left(b[3]), m01);
                e1[1] = ext<MIN>(m01, b[2]);
                e1[2] = ext<MIN>(b[1], m23);
                e1[3] = ext<MIN>(from_right(b[0]), m23);
            }
            {
                const uint32_t m02 = ext<MIN>(e1[0], e1[2]), m13 = ext<MIN>(e1[1], e1[3]);
                e3[0] = ext<MIN>(from_left(e1[2]), m02);
                e3[1] = ext<MIN>(from_left(e1[3]), m13);
                e3[2] = ext<MIN>(from_right(e1[0]), m02);
                e3[3] = ext<MIN>(from_right(e1[1]), m13);
            }
            auto wider = [&](const uint32_t (&e)[4], uint32_t (&o)[4]) { // a column more each side
                o[0] = ext<MIN>(from_left(e[3]), e[1]);
                o[1] = ext<MIN>(e[0], e[2]);
                o[2] = ext<MIN>(e[1], e[3]);
                o[3] = ext<MIN>(from_right(e[0]), e[2]);
            };
            wider(e3, e4);
            wider(e4, e5);
            wider(e5, e6);
            auto slot = [&](int back) { return (rr - back + 26) % 13; }; // of output row r - back
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                // half-width 5 over rows r - 2 .. r, and r - 6 .. r
                const uint32_t p3 = ext3<MIN>(e5p[1][c], e5p[0][c], e5[c]);
                const uint32_t p7 = ext3<MIN>(t3[3][c], t3[1][c], p3);
                e5p[1][c] = e5p[0][c];
                e5p[0][c] = e5[c];
                t3[3][c] = t3[2][c];
                t3[2][c] = t3[1][c];
                t3[1][c] = t3[0][c];
                t3[0][c] = p3;
                uint32_t &a12 = acc[slot(12)][c], &a10 = acc[slot(10)][c], &a6 = acc[slot(6)][c];
                uint32_t &a2 = acc[slot(2)][c];
                // (the value of the row before goes with this row's: output row
                // r - 12 took half-width 3 one row above, and so on)
                a12 = ext3<MIN>(a12, e3p[c], b[c]);
                a10 = ext3<MIN>(a10, p7p[c], e4[c]);
                a6 = ext3<MIN>(a6, e6[c], e6[c]);
                a2 = ext3<MIN>(a2, e3p[c], e4[c]);
                e3p[c] = e3[c];
                p7p[c] = p7;
            }
            // output row r - 12 is complete: store it, then open row r
            if (r >= 12 && (FAST || r - 12 < y_hi) && stores) {
                const uint32_t *o = acc[slot(12)];
                const uint32_t q = __builtin_amdgcn_perm(o[2] | o[3] << 8, o[0] | o[1] << 8,
                                                         0x05040100u);
                typedef uint32_t u32_any __attribute__((aligned(1)));
                orow_t op = next_out + (uint32_t)x;
                if (FAST || x_hi == 256 || x + 4 <= x_hi) { // (a dword store on any byte)
                    *(__attribute__((address_space(1))) u32_any *)op = q;
                } else {
                    op[0] = (uint8_t)q;
                    if (x + 1 < x_hi) op[1] = (uint8_t)(q >> 8);
                    if (x + 2 < x_hi) op[2] = (uint8_t)(q >> 16);
                }
            }
            next_out += pitch;
            asm volatile("" : "+s"(next_out));
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[rr][c] = b[c];
            // (steps overlapped further by the scheduler would spill)
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    };
    if (aligned && whole)
        strip(std::integral_constant<int, 0>{});
    else if (aligned)
        strip(std::integral_constant<int, 1>{});
    else
        strip(std::integral_constant<int, 2>{});
}

// Rows per strip: 13 m - 12, so that its th + 12 steps are whole turns of the
// accumulator ring. The chip holds a fixed number of waves: the strips are cut so
// that they fill it a whole number of times, twice at least, and the number of
// times is the one with the fewest steps in all. (Filled once, the chip waits
// for the strips at the image's edges, which take longer: 16384 x 16384 takes
// 175 us filled once, 160 us twice or three times, 166 us five times. Strips
// of 64 rows, 4.3 fillings, took 218 us.)
int disk_rows(int64_t H, int64_t tx) {
    const int64_t cap = (int64_t)persistent_grid() / 2 * DK_WAVES_PER_SIMD; // (grid: 2 waves a SIMD)
    int64_t best = 1ll << 62;
    int th = 13 * 6 - 12;
    for (int64_t k = 2; k <= 8; ++k) {
        const int64_t strips = k * cap / tx;
        if (strips == 0) continue;
        const int64_t m = std::max<int64_t>(2, ((H + strips - 1) / strips + 12 + 12) / 13);
        if (m > 1 << 16) continue;
        if (k * m < best) {
            best = k * m;
            th = (int)(13 * m - 12);
        }
    }
    return th;
}

hipError_t launch_disk13(bool erode, const uint8_t *in, uint8_t *out, int64_t H, int64_t W,
                         int64_t pitch, hipStream_t s) {
    const int64_t tx = (W + DK_OUT - 1) / DK_OUT;
    const int th = disk_rows(H, tx);
    const int64_t n = tx * ((H + th - 1) / th);
    if (n >= (1ll << 31) - 8) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(n + 7) / 8 * 8);
    if (erode)
        hipLaunchKernelGGL(k_disk13<true>, grid, dim3(64), 0, s, in, out, H, W, pitch,
                           (uint32_t)tx, (uint32_t)n, th);
    else
        hipLaunchKernelGGL(k_disk13<false>, grid, dim3(64), 0, s, in, out, H, W,
                           pitch, (uint32_t)tx, (uint32_t)n, th);
    return hipGetLastError();
}

} // namespace

extern "C" {

size_t mr_hdome_workspace_bytes(int64_t H, int64_t W, int64_t pitch, mr_dtype t, int conn,
                                const mr_tune *tune) {
    clear_error();
    if (pitch == 0) pitch = W;
    if (check_dims(H, W, pitch, (int)t) != MR_OK) return 0;
    HdomeLayout L;
    if (hdome_layout(H, W, pitch, (int)t, conn, tune, L) != MR_OK) return 0;
    return L.total;
}

int mr_hdome(void *img_inout, int64_t H, int64_t W, int64_t pitch, mr_dtype t, int conn,
             int64_t h, void *ws, size_t ws_bytes, const mr_tune *tune, void *stream) {
    HdomeLayout L;
    int rc = hdome_common(img_inout, H, W, pitch, (int)t, conn, ws, ws_bytes, tune, L);
    if (rc != MR_OK) return rc;
    if (h < 0) return ofail(MR_EINVAL, "h must be >= 0 (got %lld)", (long long)h);
    // the dome f - R lies in [0, h]: for int32 pixels h must fit the type
    if ((int)t == MR_I32 && h > 0x7FFFFFFFll)
        return ofail(MR_EINVAL, "h must be at most 2^31 - 1 for int32 pixels");
    const uint32_t hk = h > 0xFFFFFFFFll ? 0xFFFFFFFFu : (uint32_t)h;
    hipStream_t s = (hipStream_t)stream;
    char *w = (char *)ws;
    void *marker = w + L.plane;
    uint32_t *flag = (uint32_t *)(w + L.flag);
    rc = recon_lowered(marker, img_inout, H, W, pitch, (int)t, conn, hk, flag, ws, L.recon, tune,
                       stream);
    if (rc != MR_OK) return rc;
    const hipError_t e = (int)t == MR_U8
        ? stream_pass<uint8_t, P_DOME>((const uint8_t *)img_inout, (const uint8_t *)marker,
                                       (uint8_t *)img_inout, nullptr, H, W, pitch, 0, flag, s)
        : stream_pass<int32_t, P_DOME>((const int32_t *)img_inout, (const int32_t *)marker,
                                       (int32_t *)img_inout, nullptr, H, W, pitch, 0, flag, s);
    return e == hipSuccess ? MR_OK : ohip(e, "h-dome output");
}

int mr_regional_maxima(const void *img, void *out_u8, int64_t H, int64_t W, int64_t pitch,
                       int64_t out_pitch, mr_dtype t, int conn, void *ws, size_t ws_bytes,
                       const mr_tune *tune, void *stream) {
    HdomeLayout L;
    int rc = hdome_common(img, H, W, pitch, (int)t, conn, ws, ws_bytes, tune, L);
    if (rc != MR_OK) return rc;
    if (!out_u8) return ofail(MR_EINVAL, "null output");
    if (out_pitch == 0) out_pitch = W;
    if (out_pitch < W) return ofail(MR_EINVAL, "out_pitch below W");
    hipStream_t s = (hipStream_t)stream;
    char *w = (char *)ws;
    void *marker = w + L.plane;
    uint32_t *flag = (uint32_t *)(w + L.flag);
    rc = recon_lowered(marker, img, H, W, pitch, (int)t, conn, 1u, flag, ws, L.recon, tune, stream);
    if (rc != MR_OK) return rc;
    const hipError_t e = (int)t == MR_U8
        ? stream_pass<uint8_t, P_RMAX>((const uint8_t *)img, (const uint8_t *)marker, nullptr,
                                       (uint8_t *)out_u8, H, W, pitch, out_pitch, flag, s)
        : stream_pass<int32_t, P_RMAX>((const int32_t *)img, (const int32_t *)marker, nullptr,
                                       (uint8_t *)out_u8, H, W, pitch, out_pitch, flag, s);
    return e == hipSuccess ? MR_OK : ohip(e, "regional maxima output");
}

int mr_rgb2gray(const void *rgb, int64_t rgb_pitch, void *gray, int64_t gray_pitch, int64_t H,
                int64_t W, void *stream) {
    clear_error();
    if (!rgb || !gray) return ofail(MR_EINVAL, "null image");
    if (rgb_pitch == 0) rgb_pitch = 3 * W;
    if (gray_pitch == 0) gray_pitch = W;
    int rc;
    if ((rc = check_dims(H, W, gray_pitch, 1)) != MR_OK) return rc;
    if (rgb_pitch < 3 * W) return ofail(MR_EINVAL, "rgb_pitch %lld is below 3 W",
                                        (long long)rgb_pitch);
    hipStream_t s = (hipStream_t)stream;
    const uint8_t *src = (const uint8_t *)rgb;
    uint8_t *dst = (uint8_t *)gray;
    int64_t x0 = 0;
    if (rgb_pitch == 3 * W && gray_pitch == W) { // rows without gaps: one long row
        W = gray_pitch = H * W;
        rgb_pitch = 3 * W;
        H = 1;
    }
    const bool al = (uintptr_t)src % 16 == 0 && (uintptr_t)dst % 16 == 0 &&
                    (H == 1 || (rgb_pitch % 16 == 0 && gray_pitch % 16 == 0));
    if (al && W >= 16) {
        const int64_t vec = W / 16;
        hipLaunchKernelGGL(k_rgb2gray16, dim3(grid_for(H * vec, 256)), dim3(256), 0, s, src,
                           rgb_pitch, dst, gray_pitch, H, vec, H == 1 ? (int)(W - vec * 16) : 0);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return ohip(e, "rgb2gray");
        x0 = H == 1 ? W : vec * 16;
    }
    if (x0 < W) {
        hipLaunchKernelGGL(k_rgb2gray1, dim3(grid_for(H * (W - x0), 256)), dim3(256), 0, s, src,
                           rgb_pitch, dst, gray_pitch, H, x0, W);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return ohip(e, "rgb2gray");
    }
    return MR_OK;
}

int mr_disk13(int op, const void *in, void *out, int64_t H, int64_t W, int64_t pitch,
              void *stream) {
    clear_error();
    if (op != MR_DISK_ERODE && op != MR_DISK_DILATE) return ofail(MR_EINVAL, "unknown op %d", op);
    if (!in || !out) return ofail(MR_EINVAL, "null image");
    if (pitch == 0) pitch = W;
    int rc;
    if ((rc = check_dims(H, W, pitch, 1)) != MR_OK) return rc;
    const char *a = (const char *)in, *b = (const char *)out;
    const size_t span = (size_t)((H - 1) * pitch + W);
    if (a < b + span && b < a + span) return ofail(MR_EINVAL, "in and out overlap");
    hipError_t e = launch_disk13(op == MR_DISK_ERODE, (const uint8_t *)in, (uint8_t *)out, H, W,
                                 pitch, (hipStream_t)stream);
    return e == hipSuccess ? MR_OK : ohip(e, "disk13");
}

size_t mr_open_disk13_workspace_bytes(int64_t H, int64_t W, int64_t pitch) {
    clear_error();
    if (pitch == 0) pitch = W;
    if (check_dims(H, W, pitch, 1) != MR_OK) return 0;
    return up256((size_t)H * (size_t)pitch);
}

int mr_open_disk13(const void *in, void *out, int64_t H, int64_t W, int64_t pitch, void *ws,
                   size_t ws_bytes, void *stream) {
    clear_error();
    if (pitch == 0) pitch = W;
    int rc;
    if ((rc = check_dims(H, W, pitch, 1)) != MR_OK) return rc;
    if (!ws) return ofail(MR_EINVAL, "null workspace");
    if ((uintptr_t)ws % 256) return ofail(MR_EINVAL, "workspace must be 256-byte aligned");
    const size_t need = up256((size_t)H * (size_t)pitch);
    if (ws_bytes < need)
        return ofail(MR_ENOMEM, "workspace too small: %zu bytes given, %zu needed", ws_bytes,
                     need);
    if ((rc = mr_disk13(MR_DISK_ERODE, in, ws, H, W, pitch, stream)) != MR_OK) return rc;
    return mr_disk13(MR_DISK_DILATE, ws, out, H, W, pitch, stream);
}

} // extern "C"
