// mr_kernels.hip -- gfx950 kernels of libmrecon.
//
// Pixels are handled as 32-bit unsigned keys whose order is the pixel order:
// uint8 v -> v, int32 v -> v ^ 0x80000000. Key 0 is the type's minimum, so it
// is the identity of max and stands for "no pixel" outside the image. The
// bitwise complement used by fill-holes is KMAX - key in key space.
//
// Four kernels carry the propagation (Algorithm 1 split into the regular and
// irregular phases of Sec. V-C.2):
//  * k_tile_round -- the regular phase. One wave owns a 64 x 64 tile of keys
//    held in registers (lane = column, register = row); the outer ring is the
//    halo. Down and up sweeps run along the registers with the diagonal
//    neighbours taken from the adjacent lanes by DPP; the tile is transposed
//    through LDS for the right and left sweeps. Sweeps repeat until the tile
//    is stable, then the interior is stored and the neighbours whose halo the
//    new border can still raise go on the next round's dirty list, which is
//    all that round visits.
//  * k_tile_queue -- the same visits without rounds: waves take tiles from a
//    device ring and mark neighbours straight into it, until none is left.
//  * k_seed -- one relaxation step over each tile still dirty after the last
//    round; every raised pixel is compacted by wave ballot into the tile's row
//    of the frontier bitmap, and the tile into the device frontier ring.
//  * k_queue -- persistent waves pop tiles from the ring, claim the set bits of
//    the tile's bitmap and propagate each claimed pixel to its neighbours with
//    atomic max updates; every raised neighbour is pushed back (bit set, its
//    tile enqueued once). The wave that retires the last entry stops them all.
#include <algorithm>

#include "mr_internal.h"

namespace mr {

template <typename T> struct Pix;
template <> struct Pix<uint8_t> {
    static constexpr uint32_t KMAX = 0xFFu;
    __device__ static __forceinline__ uint32_t key(uint8_t v) { return v; }
    __device__ static __forceinline__ uint8_t val(uint32_t k) { return (uint8_t)k; }
};
template <> struct Pix<int32_t> {
    static constexpr uint32_t KMAX = 0xFFFFFFFFu;
    __device__ static __forceinline__ uint32_t key(int32_t v) { return (uint32_t)v ^ 0x80000000u; }
    __device__ static __forceinline__ int32_t val(uint32_t k) { return (int32_t)(k ^ 0x80000000u); }
};

template <typename T> using gptr = __attribute__((address_space(1))) T *;
template <typename T> using cgptr = const __attribute__((address_space(1))) T *;

// Lane i receives lane i-1's value (lane 0 receives 0).
__device__ __forceinline__ uint32_t from_lower_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
}
// Lane i receives lane i+1's value (lane 63 receives 0).
__device__ __forceinline__ uint32_t from_upper_lane(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
}

// Data that earlier launches wrote and this one only reads (descriptors,
// owner tables, the dirty lists and list lengths of the round being run),
// read through the scalar cache: uniform loads that wait on the scalar
// counter, not on the vector memory counter behind this wave's own loads
// and stores.
template <typename X> using kptr = const __attribute__((address_space(4))) X *;
template <typename X> __device__ __forceinline__ kptr<X> kconst(const X *p) {
    return (kptr<X>)p;
}

// Field-wise copy (the implicit copy constructor does not bind to a
// constant-address-space object).
__device__ __forceinline__ ImgDesc desc_at(kptr<ImgDesc> d, int64_t k) {
    ImgDesc r;
    r.J = d[k].J;
    r.I = d[k].I;
    r.out = d[k].out;
    r.H = d[k].H;
    r.W = d[k].W;
    r.pJ = d[k].pJ;
    r.pI = d[k].pI;
    r.pO = d[k].pO;
    r.tile_base = d[k].tile_base;
    r.first_round = d[k].first_round;
    r.ntx = d[k].ntx;
    r.nty = d[k].nty;
    r.op = d[k].op;
    r.done = d[k].done;
    r.wide = d[k].wide;
    r.above = d[k].above;
    r.h = d[k].h;
    r.pad = 0;
    return r;
}
static_assert(sizeof(ImgDesc) == 120, "desc_at copies every field of ImgDesc");

// Descriptor of the image that owns `tile` (owner table, else binary search
// on tile_base).
__device__ __forceinline__ ImgDesc load_desc(Imgs imgs, int64_t tile) {
    const kptr<ImgDesc> d = kconst(imgs.d);
    if (imgs.owner) return desc_at(d, kconst(imgs.owner)[tile]);
    int lo = 0, hi = imgs.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (d[mid].tile_base <= tile) lo = mid;
        else hi = mid - 1;
    }
    return desc_at(d, lo);
}

// Coherent (device-scope) access to the working image, used while other
// waves update it with atomics.
template <typename T> struct Atom;
template <> struct Atom<int32_t> {
    __device__ static __forceinline__ uint32_t load_key(const int32_t *base, int64_t off) {
        const int32_t v = __hip_atomic_load(base + off, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return Pix<int32_t>::key(v);
    }
    // Raise the pixel to key k if it is lower; true if this call raised it.
    __device__ static __forceinline__ bool raise(int32_t *base, int64_t off, uint32_t k,
                                                 unsigned long long &retries) {
        (void)retries;
        const int32_t v = Pix<int32_t>::val(k);
        const int32_t old = __hip_atomic_fetch_max(base + off, v, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
        return old < v;
    }
};
template <> struct Atom<uint8_t> {
    __device__ static __forceinline__ uint32_t load_key(const uint8_t *base, int64_t off) {
        const uintptr_t a = (uintptr_t)(base + off);
        const uint32_t *w = (const uint32_t *)(a & ~(uintptr_t)3);
        const uint32_t sh = (uint32_t)(a & 3) * 8u;
        const uint32_t word = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return (word >> sh) & 0xFFu;
    }
    __device__ static __forceinline__ bool raise(uint8_t *base, int64_t off, uint32_t k,
                                                 unsigned long long &retries) {
        const uintptr_t a = (uintptr_t)(base + off);
        uint32_t *w = (uint32_t *)(a & ~(uintptr_t)3);
        const uint32_t sh = (uint32_t)(a & 3) * 8u;
        uint32_t old = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        while (true) {
            if (((old >> sh) & 0xFFu) >= k) return false;
            const uint32_t nw = (old & ~(0xFFu << sh)) | (k << sh);
            uint32_t expect = old;
            if (__hip_atomic_compare_exchange_strong(w, &expect, nw, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                return true;
            old = expect;
            ++retries;
        }
    }
};

// ------------------------------------------------------------------ tiles

// The tile kernels run one wave per block. LDS that some lanes write and
// others read needs only program order there (a wave's LDS operations are
// performed in the order they issue) and a compiler barrier; a workgroup
// barrier would also wait for every global load and store in flight.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}


// Buffer resource over `bytes` bytes (whole dwords) from a 16-byte aligned
// address, so every 16-byte chunk load is
// aligned and the per-dword range check matches whole memory words. Loads past
// the end, or at the huge offsets used for rows outside the image, return 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *p, uint64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, (short)0, (int)(uint32_t)bytes,
                                             0x00020000);
}

// Bytes from the aligned start of a uint8 plane's resource to the end of its
// last pixel's dword.
__device__ __forceinline__ uint64_t plane_bytes(const void *p, int64_t H, int64_t W,
                                                int64_t pitch) {
    return (((uint64_t)((uintptr_t)p & 15) + (uint64_t)((H - 1) * pitch + W)) + 3) & ~3ull;
}

// Any uint8 plane whose bytes a 32-bit buffer offset reaches can be staged.
__device__ __forceinline__ bool stage_ok(const ImgDesc &d) {
    return plane_bytes(d.I, d.H, d.W, d.pI) <= STAGE_MAX_BYTES &&
           plane_bytes(d.J, d.H, d.W, d.pJ) <= STAGE_MAX_BYTES;
}

// uint8 staging: the 64 pixels of tile row r (image row gy0 + r, columns gx0..)
// lie in five aligned 16-byte chunks. Lane r fetches them, shifts its words by
// the row's byte misalignment (rows of an odd pitch each have their own), and
// writes them to LDS displaced by its word misalignment, so that column c of
// the tile is byte c of the stage row whatever the plane's base and pitch.
// A stage row is an odd number of dwords, so the row writes (lane = row) and the
// column reads (lane = column) are both free of bank conflicts; of the words
// a row writes outside its 16, up to 3 come before it and 4 after it, and all
// land behind the pixels of a row (its own or the one before), or in the
// STAGE_PAD bytes before the first.
constexpr int SROW = 84;
// Cache policy of loads that must see other compute units' stores at device
// scope (sc1: not served from a compute unit's or a die's non-coherent cache).
constexpr int CPOL_DEVICE = 16;
constexpr int STAGE_PAD = 16;
constexpr int STAGE_BYTES = TS * SROW;
static_assert(STAGE_PAD + 2 * STAGE_BYTES <= TS * (TS + 1) * 4,
              "the stage must fit in the transpose buffer");

// Byte offset of pixel (gy, gx) from the plane's aligned start (mod 2^32: a
// tile at the image's left edge starts before its row, in row 0 before the
// plane, where the offset wraps out of the resource's range).
__device__ __forceinline__ uint32_t stage_offset(const void *p, int32_t gy, uint32_t pitch,
                                                 int64_t gx0) {
    return (uint32_t)((uintptr_t)p & 15) + (uint32_t)gy * pitch + (uint32_t)(int32_t)gx0;
}

// The five chunks of lane's row. The lane
// id goes through an empty asm so that nothing derived from it is hoisted out
// of the caller's tile loop: held across the sweeps, such values would be
// spilled, and every reload would wait for all memory operations in flight.
// Pixels of chunks outside the image are whatever lies there in the plane, or
// 0 out of its range; the tile masks them.
template <int CPOL = 0>
__device__ __forceinline__ void stage_issue(const void *p, int64_t gy0, int64_t gx0, int64_t H,
                                            int64_t W, int64_t pitch, int lane, v4u (&v)[5],
                                            bool live = true) {
    const __amdgpu_buffer_rsrc_t rs =
        plane_rsrc((const void *)((uintptr_t)p & ~(uintptr_t)15), plane_bytes(p, H, W, pitch));
    uint32_t ln = (uint32_t)lane;
    asm volatile("" : "+v"(ln));
    const int32_t gy = (int32_t)gy0 + (int32_t)ln;
    const bool rowok = live && gy >= 0 && gy < (int32_t)H;
    uint32_t off = rowok ? stage_offset(p, gy, (uint32_t)pitch, gx0) & ~15u : 0xFFFFFF00u;
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        v[k] = __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, CPOL);
        off += 16;
    }
}

// Row `lane` of the stage at st gets the words fetched by stage_issue, each
// exclusive-ored with `flip`.
__device__ __forceinline__ void stage_commit(const v4u (&v)[5], const void *p, int64_t gy0,
                                             int64_t gx0, int64_t pitch, int lane, uint8_t *st,
                                             uint32_t flip) {
    uint32_t ln = (uint32_t)lane;
    asm volatile("" : "+v"(ln));
    const uint32_t mis = stage_offset(p, (int32_t)gy0 + (int32_t)ln, (uint32_t)pitch, gx0) & 15u;
    uint32_t *w = (uint32_t *)(st + ln * SROW) - (mis >> 2);
    const uint32_t sh = mis & 3u;
    uint32_t x[21];
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        x[4 * k + 0] = v[k].x;
        x[4 * k + 1] = v[k].y;
        x[4 * k + 2] = v[k].z;
        x[4 * k + 3] = v[k].w;
    }
    x[20] = 0;
#pragma unroll
    for (int k = 0; k < 20; ++k) w[k] = __builtin_amdgcn_alignbyte(x[k + 1], x[k], sh) ^ flip;
}

// A tile's stage rows in flight, held by value (mask words, working-image
// words) so that they stay in registers between the visit that fetches them
// and the one that commits them.
struct StageWords {
    v4u i0, i1, i2, i3, i4, j0, j1, j2, j3, j4;
};

// Where tile t of image d lies: tile row and column.
__device__ __forceinline__ void tile_place(const ImgDesc &d, int64_t t, int &ty, int &tx) {
    const uint32_t lt = (uint32_t)(t - d.tile_base); // (tile ids are below 2^31)
    ty = (int)(lt / (uint32_t)d.ntx);
    tx = (int)(lt - (uint32_t)ty * (uint32_t)d.ntx);
}

// Issue the stage loads of tile t of image d (uint8); with
// live false every load is out of the buffer's range (zeros, no memory
// access), so that the count of loads does not depend on the path. CPOL is the
// working image's cache policy.
template <bool NEEDJ, int CPOL = 0>
__device__ __forceinline__ StageWords stage_fetch(const ImgDesc &d, int64_t t, int lane,
                                                  bool live = true) {
    int ty, tx;
    tile_place(d, t, ty, tx);
    const int64_t gy0 = (int64_t)ty * TI - 1, gx0 = (int64_t)tx * TI - 1;
    StageWords w;
    v4u v[5];
    stage_issue(d.I, gy0, gx0, d.H, d.W, d.pI, lane, v, live);
    w.i0 = v[0];
    w.i1 = v[1];
    w.i2 = v[2];
    w.i3 = v[3];
    w.i4 = v[4];
    if (NEEDJ) {
        stage_issue<CPOL>(d.J, gy0, gx0, d.H, d.W, d.pJ, lane, v, live);
        w.j0 = v[0];
        w.j1 = v[1];
        w.j2 = v[2];
        w.j3 = v[3];
        w.j4 = v[4];
    } else {
        w.j0 = w.j1 = w.j2 = w.j3 = w.j4 = v4u{0u, 0u, 0u, 0u};
    }
    return w;
}

// The fetched rows of tile t go to the stage (mask rows, then working-image
// rows); a fill-holes image's mask is complemented on the way.
template <bool NEEDJ>
__device__ __forceinline__ void stage_commit_words(const StageWords &w, const ImgDesc &d,
                                                   int64_t t, int lane, uint8_t *st, bool fill) {
    int ty, tx;
    tile_place(d, t, ty, tx);
    const int64_t gy0 = (int64_t)ty * TI - 1, gx0 = (int64_t)tx * TI - 1;
    const v4u vi[5] = {w.i0, w.i1, w.i2, w.i3, w.i4};
    stage_commit(vi, d.I, gy0, gx0, d.pI, lane, st + STAGE_PAD, fill ? ~0u : 0u);
    if (NEEDJ) {
        const v4u vj[5] = {w.j0, w.j1, w.j2, w.j3, w.j4};
        stage_commit(vj, d.J, gy0, gx0, d.pJ, lane, st + STAGE_PAD + STAGE_BYTES, 0u);
    }
}

// A working-image element; COH reads it device-coherent.
template <typename T, bool COH>
__device__ __forceinline__ T load_j(cgptr<T> p, uint32_t off) {
    if (COH) return __hip_atomic_load((T *)(p + off), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return p[off];
}
template <typename T, bool COH>
__device__ __forceinline__ void store_j(gptr<T> p, uint32_t off, T v) {
    if (COH) __hip_atomic_store((T *)(p + off), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else p[off] = v;
}

// Key k lowered by h, saturating at 0.
__device__ __forceinline__ uint32_t lower(uint32_t k, uint32_t h) {
    return __builtin_elementwise_sub_sat(k, h);
}

// How a visit starts; uniform, and constants in the kernels made for one kind.
struct VisitKind {
    bool fill, initial, lowered;
};

// A kernel's visit kind V: bit 0 initial, bit 1 fill-holes, bit 2 (with bit 0) a
// marker lowered from the mask; V < 0: as the tile's image and round say (with
// LOWERED for launches that may lower the mask: those of one uint8 image too
// large to stage; the code for it costs mixed batches 10 % where it is not needed).
template <int V, bool LOWERED>
__device__ __forceinline__ VisitKind visit_kind(const Imgs &imgs, const ImgDesc &d, uint32_t round) {
    if (V >= 0) return VisitKind{(bool)((V >> 1) & 1), (bool)(V & 1), (bool)((V >> 2) & 1)};
    const bool initial = d.first_round == (int64_t)round;
    return VisitKind{d.op == MR_OP_FILL, initial, LOWERED && initial && imgs.lowered};
}

// The register tile of one visit. `initial` builds the starting working image
// (reconstruction: min(marker, mask); fill-holes: the complement on the image
// border and the minimum inside; `lowered`: the mask lowered by d.h) instead of
// reading it; `fill` reads the input
// image and complements it into the mask. Outside pixels become key 0 in
// both planes, which keeps them at 0.
// The halo is not frozen: a sweep may raise a halo pixel from its in-tile
// neighbours. That is a true geodesic dilation step on real values, so every
// value stays at or below the reconstruction; halo values are never stored,
// and a tile at a fixed point against a raised halo is one against the stored
// halo as well (the dilation step is monotone).
// uint8 tiles are staged through LDS; int32 rows (which are 256-byte coalesced
// loads) and uint8 planes beyond a buffer offset's range go straight to
// registers from clamped, in-bounds addresses. For staged tiles inside the
// image the
// transposed mask IT (lane = row, register = column) and the loaded halo
// columns JL, JR (lane = row) are read straight from the stage, and `it_done`
// says so.
// From a stage that holds the tile's mask rows (complemented already for
// fill-holes) and working-image rows, written and synchronized: the register
// tile J, I
// (lane = column), and for tiles inside the image the transposed mask IT and
// the halo columns JL, JR (lane = row), with it_done set. Ends with a wave sync:
// the stage's memory is the transpose buffer afterwards.
__device__ __forceinline__ void stage_read(const ImgDesc &d, int64_t gy0, int64_t gx0, int lane,
                                           uint32_t (&J)[TS], uint32_t (&I)[TS],
                                           uint32_t (&IT)[TS], uint32_t &JL, uint32_t &JR,
                                           const uint8_t *stage, bool &it_done, VisitKind kind) {
    const bool fill = kind.fill, initial = kind.initial;
    const int64_t H = d.H, W = d.W;
    const int64_t gx = gx0 + lane;
    const bool xin = gx >= 0 && gx < W;
    const bool xedge = gx == 0 || gx == W - 1;
    // The whole tile, halo included, lies inside the image (wave-uniform):
    // no pixel needs the outside rule. A fill-holes image's first visit also
    // needs to know the image border, so it always takes the general path.
    const bool inside =
        !(fill && initial) && gy0 >= 0 && gy0 + TS <= H && gx0 >= 0 && gx0 + TS <= W;
    const uint8_t *stI = stage + STAGE_PAD, *stJ = stI + STAGE_BYTES;
    if (inside) {
#pragma unroll
        for (int r = 0; r < TS; ++r) {
            const uint32_t iv = stI[r * SROW + lane];
            uint32_t jv = kind.lowered ? 0u : stJ[r * SROW + lane];
            if (kind.lowered) jv = lower(iv, d.h);
            else if (initial) jv = min(jv, iv);
            J[r] = jv;
            I[r] = iv;
        }
        // lane = row: this lane's row of the mask, and the working image's
        // two halo pixels of that row
        const uint8_t *row = stI + lane * SROW;
#pragma unroll
        for (int c = 0; c < TS; ++c) IT[c] = row[c];
        const uint8_t *rowJ = stJ + lane * SROW;
        JL = rowJ[0];
        JR = rowJ[TS - 1];
        if (kind.lowered) {
            JL = lower(IT[0], d.h);
            JR = lower(IT[TS - 1], d.h);
        } else if (initial) {
            JL = min(JL, IT[0]);
            JR = min(JR, IT[TS - 1]);
        }
        it_done = true;
    } else {
#pragma unroll
        for (int r = 0; r < TS; ++r) {
            const int64_t gy = gy0 + r;
            const bool ok = xin && gy >= 0 && gy < H;
            const uint32_t iv = stI[r * SROW + lane];
            uint32_t jv = kind.lowered ? 0u : stJ[r * SROW + lane];
            if (kind.lowered)
                jv = lower(iv, d.h);
            else if (initial)
                jv = fill ? ((xedge || gy == 0 || gy == H - 1) ? iv : 0u) : min(jv, iv);
            J[r] = ok ? jv : 0u;
            I[r] = ok ? iv : 0u;
        }
    }
    wave_sync();
}

template <typename T, bool COH = false>
__device__ __forceinline__ void load_tile(const ImgDesc &d, int64_t t, int64_t gy0, int64_t gx0,
                                          int lane, uint32_t (&J)[TS], uint32_t (&I)[TS],
                                          uint32_t (&IT)[TS], uint32_t &JL, uint32_t &JR,
                                          uint8_t *stage, bool &it_done, VisitKind kind) {
    using P = Pix<T>;
    const bool fill = kind.fill, initial = kind.initial;
    if (sizeof(T) == 1 && stage_ok(d)) {
        const StageWords w = stage_fetch<true, COH ? CPOL_DEVICE : 0>(d, t, lane);
        stage_commit_words<true>(w, d, t, lane, stage, fill);
        wave_sync();
        stage_read(d, gy0, gx0, lane, J, I, IT, JL, JR, stage, it_done, kind);
        return;
    }
    const int64_t H = d.H, W = d.W;
    const int64_t gx = gx0 + lane;
    const bool xin = gx >= 0 && gx < W;
    const bool xedge = gx == 0 || gx == W - 1;
    const bool inside =
        !(fill && initial) && gy0 >= 0 && gy0 + TS <= H && gx0 >= 0 && gx0 + TS <= W;
    const uint32_t flip = fill ? P::KMAX : 0u;
    cgptr<T> Jp = (cgptr<T>)d.J;
    cgptr<T> Ip = (cgptr<T>)d.I;
    if (inside) {
        uint32_t oI = (uint32_t)gy0 * (uint32_t)d.pI + (uint32_t)gx;
        uint32_t oJ = (uint32_t)gy0 * (uint32_t)d.pJ + (uint32_t)gx;
#pragma unroll
        for (int r = 0; r < TS; ++r) {
            const uint32_t iv = P::key(Ip[oI]) ^ flip;
            uint32_t jv;
            if (kind.lowered) {
                jv = lower(iv, d.h);
            } else {
                jv = P::key(load_j<T, COH>(Jp, oJ));
                if (initial) jv = min(jv, iv);
            }
            J[r] = jv;
            I[r] = iv;
            oI += (uint32_t)d.pI;
            oJ += (uint32_t)d.pJ;
        }
        return;
    }
    const uint32_t xc = (uint32_t)(gx < 0 ? 0 : (gx > W - 1 ? W - 1 : gx));
    // int32: all rows are loaded before any is used. Left to itself the compiler
    // waits for each row before it loads the next, 64 memory latencies a visit to a
    // border tile: 21 int32 jobs on the server 1255 -> 855 us, 1152 x 473 192 -> 173
    // us. (uint8 tiles come here only from planes too large to stage.)
    constexpr bool AHEAD = sizeof(T) == 4;
    if (AHEAD) {
        auto clamped = [&](int r) {
            const int64_t gy = gy0 + r;
            return (uint32_t)(gy < 0 ? 0 : (gy > H - 1 ? H - 1 : gy));
        };
#pragma unroll
        for (int r = 0; r < TS; ++r) I[r] = (uint32_t)Ip[clamped(r) * (uint32_t)d.pI + xc];
        if (!(fill && initial) && !kind.lowered) {
#pragma unroll
            for (int r = 0; r < TS; ++r)
                J[r] = (uint32_t)load_j<T, COH>(Jp, clamped(r) * (uint32_t)d.pJ + xc);
        }
        asm volatile("" ::: "memory");
    }
#pragma unroll
    for (int r = 0; r < TS; ++r) {
        const int64_t gy = gy0 + r;
        const bool ok = xin && gy >= 0 && gy < H;
        const uint32_t yc = (uint32_t)(gy < 0 ? 0 : (gy > H - 1 ? H - 1 : gy));
        uint32_t iv = P::key(AHEAD ? (T)I[r] : Ip[yc * (uint32_t)d.pI + xc]) ^ flip;
        uint32_t jv;
        if (fill && initial) {
            jv = (xedge || yc == 0 || yc == (uint32_t)(H - 1)) ? iv : 0u;
        } else if (kind.lowered) {
            jv = lower(iv, d.h);
        } else {
            jv = P::key(AHEAD ? (T)J[r] : load_j<T, COH>(Jp, yc * (uint32_t)d.pJ + xc));
            if (initial) jv = min(jv, iv);
        }
        jv = ok ? jv : 0u;
        iv = ok ? iv : 0u;
        J[r] = jv;
        I[r] = iv;
    }
}

// Transpose a 64 x 64 register tile through LDS: afterwards lane l holds row
// l and register c holds column c.
__device__ __forceinline__ void transpose(uint32_t (&A)[TS], uint32_t (*tb)[TS + 1], int lane) {
#pragma unroll
    for (int r = 0; r < TS; ++r) tb[r][lane] = A[r];
    wave_sync();
#pragma unroll
    for (int c = 0; c < TS; ++c) A[c] = tb[lane][c];
    wave_sync();
}

// med3(j, n, i) = min(max(j, n), i) whenever j <= i, which holds for every
// key the kernels hold (the working image never exceeds the mask, and the
// frozen halo has i == j): one VALU instead of two.
__device__ __forceinline__ uint32_t med3(uint32_t j, uint32_t n, uint32_t i) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(j), "v"(n), "v"(i));
    return r;
}

// One 8-connected row step: med3(j, max of u over lanes l-1, l, l+1, i).
// Both lane shifts ride on DPP max instructions. The leading s_nop covers the
// DPP read-after-VALU-write hazard on u, which is written by the previous
// row's step immediately before.
__device__ __forceinline__ uint32_t step3(uint32_t j, uint32_t u, uint32_t i) {
    uint32_t r, t;
    asm("s_nop 1\n\t"
        "v_max_u32_dpp %1, %2, %2 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_max_u32_dpp %1, %2, %1 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_med3_u32 %0, %3, %1, %4"
        : "=v"(r), "=&v"(t)
        : "v"(u), "v"(j), "v"(i));
    return r;
}

// Max over lanes l-1, l, l+1 (0 beyond the wave's ends).
__device__ __forceinline__ uint32_t max3_lanes(uint32_t u) {
    uint32_t t;
    asm("s_nop 1\n\t"
        "v_max_u32_dpp %0, %1, %1 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n\t"
        "v_max_u32_dpp %0, %1, %0 wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"
        : "=&v"(t)
        : "v"(u));
    return t;
}

// The halo columns 0 and TS-1 of a register tile, lane = row: lanes 0 and
// TS-1 write their registers to LDS and every lane reads its row back.
__device__ __forceinline__ void halo_cols(const uint32_t (&A)[TS], uint32_t (*tb)[TS + 1],
                                          int lane, uint32_t &cl, uint32_t &cr) {
    uint32_t *buf = &tb[0][0];
    if (lane == 0 || lane == TS - 1) {
        uint32_t *dst = buf + (lane == 0 ? 0 : TS);
#pragma unroll
        for (int r = 0; r < TS; ++r) dst[r] = A[r];
    }
    wave_sync();
    cl = buf[lane];
    cr = buf[TS + lane];
    wave_sync();
}

// Sweeps along the registers. With DIAG, A[r] takes the max over the three
// lanes of the previous register (the 3 neighbours in the previous row), else
// only the same lane; the result is limited by B[r]. Values only rise, so
// callers detect change by comparing column sums.
template <bool DIAG>
__device__ __forceinline__ void sweep_fwd(uint32_t (&A)[TS], const uint32_t (&B)[TS]) {
#pragma unroll
    for (int r = 1; r < TS - 1; ++r)
        A[r] = DIAG ? step3(A[r], A[r - 1], B[r]) : med3(A[r], A[r - 1], B[r]);
}

template <bool DIAG>
__device__ __forceinline__ void sweep_bwd(uint32_t (&A)[TS], const uint32_t (&B)[TS]) {
#pragma unroll
    for (int r = TS - 2; r >= 1; --r)
        A[r] = DIAG ? step3(A[r], A[r + 1], B[r]) : med3(A[r], A[r + 1], B[r]);
}

// One relaxation step over the interior rows: every pixel against all its
// neighbours. With 8-connectivity the step reads the values from before it;
// with 4-connectivity the row above is already updated. Both are valid
// steps, and a step that changes nothing means every pixel in rows 1..TS-2 is
// stable against all its neighbours.
template <int CONN>
__device__ __forceinline__ void relax_once(uint32_t (&J)[TS], const uint32_t (&I)[TS]) {
    if (CONN == 8) {
        uint32_t hp = max3_lanes(J[0]), hc = max3_lanes(J[1]);
#pragma unroll
        for (int r = 1; r < TS - 1; ++r) {
            const uint32_t hn = max3_lanes(J[r + 1]);
            J[r] = med3(J[r], max(max(hp, hc), hn), I[r]);
            hp = hc;
            hc = hn;
        }
    } else {
#pragma unroll
        for (int r = 1; r < TS - 1; ++r)
            J[r] = med3(J[r], max(max(J[r - 1], J[r + 1]), max3_lanes(J[r])), I[r]);
    }
}

// Sum of the interior rows of a column. Keys only rise, so the sum rises iff
// some key changed; 62 keys below 2^32 cannot overflow 64 bits, and 62 u8 keys
// cannot overflow 32.
template <typename T>
__device__ __forceinline__ uint64_t col_sum(const uint32_t (&A)[TS]) {
    if (sizeof(T) == 1) {
        uint32_t s = 0;
#pragma unroll
        for (int r = 1; r < TS - 1; ++r) s += A[r];
        return s;
    }
    uint64_t s = 0;
#pragma unroll
    for (int r = 1; r < TS - 1; ++r) s += A[r];
    return s;
}

// Tiles newly made dirty by one wave wait in an LDS batch and go to the next
// round's list with one counter update per batch, not one per tile.
__device__ __forceinline__ int64_t band_lo(int64_t n_tiles, int b) {
    return (int64_t)b * n_tiles / NBANDS;
}

__device__ __forceinline__ int band_of(int64_t n_tiles, int64_t t) {
    int b = (int)(t * NBANDS / n_tiles);
    while (b + 1 < NBANDS && band_lo(n_tiles, b + 1) <= t) ++b;
    while (b > 0 && band_lo(n_tiles, b) > t) --b;
    return b;
}

constexpr int APP_CAP = 64;
struct Appender {
    uint32_t *buf;      // LDS, APP_CAP entries
    uint32_t cnt;       // wave-uniform
    uint32_t *list_out; // next round's dirty lists (band b's at its band start)
    uint32_t *counter;  // their lengths, NBANDS of them
    int64_t n_tiles;
    uint32_t *queued;   // tile-queue states: set to 1 for the listed tiles; or null
};

// Append the batch: each lane takes one entry, and each band present gets
// one counter update.
__device__ __forceinline__ void app_flush(Appender &a, int lane) {
    if (a.cnt == 0) return;
    asm volatile("" : "+v"(lane)); // (as in visit_tile)
    wave_sync();
    const bool valid = (uint32_t)lane < a.cnt;
    const uint32_t e = valid ? a.buf[lane] : 0u;
    const int be = valid ? band_of(a.n_tiles, e) : -1;
    // lane b < NBANDS reserves band b's share with one atomic; all of them
    // go out together, so the batch costs one round trip
    uint64_t mine = 0, under = 0;
#pragma unroll
    for (int b = 0; b < NBANDS; ++b) {
        const uint64_t m = __ballot(be == b);
        if (lane == b) mine = m;
        if (be == b) under = m & ((1ull << lane) - 1);
    }
    uint32_t base = 0;
    if (lane < NBANDS && mine) base = atomicAdd(a.counter + lane, (uint32_t)__popcll(mine));
    const uint32_t my_base = __shfl(base, be < 0 ? 0 : be);
    if (valid) {
        a.list_out[band_lo(a.n_tiles, be) + my_base + __popcll(under)] = e;
        if (a.queued) a.queued[e] = 1u;
    }
    wave_sync();
    a.cnt = 0;
}

// ------------------------------------------------------------ frontier ring

// The ring holds tile ids; a tile is in it at most once (the seed pass and
// the queue phase: its qflag is 1 from enqueue until a wave finishes with
// it; the tile queue: its state), so it never holds more than the launch's
// tile count, and the capacity exceeds that plus one ticket per wave. The
// pusher has made what the entry stands for visible first: device-scope
// atomics it waited for, device-coherent stores it waited for, or stores of
// an earlier launch.
__device__ __forceinline__ void ring_put(Ctrl *ctrl, uint32_t *ring, uint64_t cap, uint32_t t,
                                         unsigned long long pos) {
    uint32_t *slot = ring + (pos & (cap - 1));
    // (the first turn around the ring finds every slot as it was cleared)
    if (pos < cap) {
        __hip_atomic_store(slot, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    // The capacity bound means the slot is already free; the wait is a guard,
    // capped so that a broken bound cannot hang the device. Past the cap the
    // entry is refused rather than written over another: its work is lost,
    // counted as an overflow and raised as the watchdog status, so the call
    // reports an incomplete result instead of returning a wrong one quietly.
    for (uint32_t spin = 0;
         __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != Q_EMPTY; ++spin) {
        if (spin > (1u << 22)) {
            atomicAdd(&ctrl->ovf[t & (NCNT - 1)], 1ull);
            atomicAdd(&ctrl->watchdog, 1ull);
            __hip_atomic_fetch_add(&ctrl->pending.v, (unsigned long long)-1ll, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    __hip_atomic_store(slot, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One lane's entry.
__device__ __forceinline__ void ring_push(Ctrl *ctrl, uint32_t *ring, uint64_t cap, uint32_t t) {
    __hip_atomic_fetch_add(&ctrl->pending.v, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long pos =
        __hip_atomic_fetch_add(&ctrl->q_tail.v, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    ring_put(ctrl, ring, cap, t, pos);
}

// The whole wave: every lane with t != Q_EMPTY pushes it, with one update of the
// tail and of the pending count for all of them. The pending count's update has
// been performed before an entry can be seen.
__device__ __forceinline__ void ring_push(Ctrl *ctrl, uint32_t *ring, uint64_t cap, uint32_t t,
                                          int lane) {
    const uint64_t m = __ballot(t != Q_EMPTY);
    if (m == 0) return;
    unsigned long long pos = 0;
    if (lane < 2) // both updates in one instruction, performed together
        pos = __hip_atomic_fetch_add(lane == 0 ? &ctrl->q_tail.v : &ctrl->pending.v,
                                     (unsigned long long)__popcll(m), __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    pos = __shfl(pos, 0);
    if (t != Q_EMPTY) ring_put(ctrl, ring, cap, t, pos + __popcll(m & ((1ull << lane) - 1)));
}

// Wait until this wave's memory operations are done (its device-coherent
// stores visible to every compute unit); also a compiler barrier.
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Ring consumers take a ticket (the next position) and wait for that entry,
// so no two waves contend for one. An entry can legitimately take as long as
// the whole run (a long chain), so the watchdog fires only when nothing at all
// moved (ring_progress) for wait_us microseconds (100 MHz constant clock): then
// the wave gives up with Q_STOP. One lane per wave calls it.
constexpr uint32_t Q_STOP = 0xFFFFFFFEu;

// A wave's first ticket in the tile queue (later ones come with ring_retire); a workgroup
// draws those of its waves together, as one counter takes 20 us for 2048 draws. Tickets are
// drawn by workgroups that run, not dealt by number: an entry dealt to a wave that
// finds no room on the chip (another stream's waves may hold it, waiting on
// their own ring) would wait for good. Every thread of the workgroup calls it.
__device__ __forceinline__ unsigned long long ring_tickets(Ctrl *ctrl, unsigned waves) {
    __shared__ unsigned long long first;
    if (threadIdx.x == 0)
        first = __hip_atomic_fetch_add(&ctrl->q_head.v, (unsigned long long)waves,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return first + (threadIdx.x >> 6);
}

// Moves while a launch makes progress: entries pushed and the sweep iterations of
// its visits. (A wave of the tile queue that hands itself tile after tile pushes
// nothing, for as long as its chain lasts: seconds on a corridor that winds through
// a whole slide level.)
__device__ __forceinline__ unsigned long long ring_progress(const Ctrl *ctrl) {
    unsigned long long p =
        __hip_atomic_load(&ctrl->q_tail.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll 1
    for (int i = 0; i < NCNT; ++i)
        p += __hip_atomic_load(&ctrl->iters[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return p;
}

__device__ __forceinline__ uint32_t ring_take(Ctrl *ctrl, uint32_t *ring, uint64_t cap,
                                              unsigned long long h, unsigned long long wait_us) {
    uint32_t *slot = ring + (h & (cap - 1));
    // (nothing seen yet: the first interval ends with a look, never with giving up)
    unsigned long long t0 = wall_clock64(), seen = ~0ull;
    uint32_t t;
    for (unsigned long long spin = 0;; ++spin) {
        t = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t != Q_EMPTY) break;
        if ((spin & 63) == 63 && wall_clock64() - t0 > wait_us * 100ull) {
            const unsigned long long now = ring_progress(ctrl);
            if (now != seen) { // progress: wait on
                seen = now;
                t0 = wall_clock64();
                continue;
            }
            atomicAdd(&ctrl->watchdog, 1ull);
            return Q_STOP;
        }
        if (spin < 32)
            __builtin_amdgcn_s_sleep(1);
        else
            __builtin_amdgcn_s_sleep(8);
    }
    if (t != Q_STOP)
        __hip_atomic_store(slot, Q_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return t;
}

// Retire one processed entry and draw the next ticket, in one instruction (the
// whole wave; the ticket is lane 1's). The wave that retires the last entry
// writes a stop entry for each of the launch's `waves` waves (each holds at most
// one ticket past the last entry, this one's new ticket among them). `pending`
// counts the entries beyond the launch's `seeds`.
__device__ __forceinline__ unsigned long long ring_retire(Ctrl *ctrl, uint32_t *ring, uint64_t cap,
                                                          unsigned waves, uint32_t seeds,
                                                          int lane) {
    unsigned long long got = 0, base = 0;
    if (lane < 2)
        got = __hip_atomic_fetch_add(lane == 0 ? &ctrl->pending.v : &ctrl->q_head.v,
                                     lane == 0 ? (unsigned long long)-1ll : 1ull, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long ticket = __shfl(got, 1);
    if (__ballot(lane == 0 && got + seeds == 1) == 0) return ticket;
    if (lane == 0)
        base = __hip_atomic_fetch_add(&ctrl->q_tail.v, (unsigned long long)waves, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
    base = __shfl(base, 0);
    // (all lanes: 2048 stops written by one lane held the launch's end up by 50 us)
    for (unsigned k = lane; k < waves; k += 64)
        __hip_atomic_store(ring + ((base + k) & (cap - 1)), Q_STOP, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    return ticket;
}

// Tile queue: a tile's state is 0 (idle), 1 (queued), 2 (a wave visits it)
// or 3 (visited and marked again meanwhile: it goes back on the ring when the
// visit ends). A mark sets bit 0; the one that finds the tile idle enqueues it.
// Tile-queue visits read and write the working image device-coherent and
// wait for their stores before any mark, so a visit that a mark leads to
// sees the marking visit's pixels without cache-wide fences.
struct TailMarks {
    bool want = false; // this lane asks for tile nb (lane 0: for the visited tile itself)
    uint32_t nb = 0;
};

// One visit of one tile: load, sweep to a local fixed point (or the cap),
// store, and mark the neighbours whose halo changed: onto the next round's
// lists, or (TAIL) into the tile queue `tq`.
// Which tile this lane (0..8) asks to visit again: itself if the sweep cap
// stopped it, or the neighbour next to a changed border pixel that can still
// raise one of the neighbour's pixels in this tile's halo (min(mask, max of
// the adjacent border pixels) above the value the halo pixel had when this
// visit loaded it; pixels only rise, so a halo pixel that passes against its
// loaded value passes against its current one too). Rows 0 and TS-1 are
// checked in lanes 0..TS-1 (lane = column), columns 0 and TS-1 in lanes
// 0..TS-1 (lane = row), whose border columns 1 and TS-2 the last transpose
// left in LDS. Returns whether this lane wants tile `nb`.
template <int CONN>
__device__ __forceinline__ bool mark_decide(const ImgDesc &d, int lane, int ty, int tx,
                                            const uint32_t (&J)[TS], const uint32_t (&I)[TS],
                                            const uint32_t (&IT)[TS], uint32_t JT, uint32_t JB,
                                            uint32_t JL, uint32_t JR, uint32_t top_in,
                                            uint32_t bot_in, uint64_t col_in, uint64_t col_out,
                                            bool stable, uint32_t (*tb)[TS + 1], uint32_t &nb) {
    const bool in_lane = lane >= 1 && lane <= TS - 2;
    const uint64_t bt = __ballot(in_lane && J[1] != top_in);
    const uint64_t bb = __ballot(in_lane && J[TS - 2] != bot_in);
    const uint64_t bc = __ballot(col_out != col_in);
    const uint32_t b1 = in_lane ? J[1] : 0u, b2 = in_lane ? J[TS - 2] : 0u;
    const uint32_t c1 = in_lane ? tb[1][lane] : 0u, c2 = in_lane ? tb[TS - 2][lane] : 0u;
    const uint32_t nbT = CONN == 8 ? max3_lanes(b1) : b1, nbB = CONN == 8 ? max3_lanes(b2) : b2;
    const uint32_t nbL = CONN == 8 ? max3_lanes(c1) : c1, nbR = CONN == 8 ? max3_lanes(c2) : c2;
    const uint64_t rt = __ballot(med3(JT, nbT, I[0]) > JT);
    const uint64_t rb = __ballot(med3(JB, nbB, I[TS - 1]) > JB);
    // (after a relaxation step that still changed pixels at the sweep cap,
    // LDS holds the columns from before it: then every halo column counts)
    const uint64_t rl = stable ? __ballot(med3(JL, nbL, IT[0]) > JL) : ~0ull;
    const uint64_t rr = stable ? __ballot(med3(JR, nbR, IT[TS - 1]) > JR) : ~0ull;
    constexpr uint64_t EDGE = ~(1ull | (1ull << (TS - 1))); // lanes 1..TS-2
    bool want = false;
    int dy = 0, dx = 0;
    switch (lane) {
    case 0: want = !stable; break;
    case 1: want = bt != 0 && (rt & EDGE) != 0; dy = -1; break;
    case 2: want = bb != 0 && (rb & EDGE) != 0; dy = 1; break;
    case 3: want = ((bc >> 1) & 1) && (rl & EDGE) != 0; dx = -1; break;
    case 4: want = ((bc >> (TS - 2)) & 1) && (rr & EDGE) != 0; dx = 1; break;
    case 5: want = CONN == 8 && ((bt >> 1) & 1) && (rt & 1); dy = -1; dx = -1; break;
    case 6: want = CONN == 8 && ((bt >> (TS - 2)) & 1) && (rt >> (TS - 1)); dy = -1; dx = 1; break;
    case 7: want = CONN == 8 && ((bb >> 1) & 1) && (rb & 1); dy = 1; dx = -1; break;
    case 8: want = CONN == 8 && ((bb >> (TS - 2)) & 1) && (rb >> (TS - 1)); dy = 1; dx = 1; break;
    default: break;
    }
    const int ny = ty + dy, nx = tx + dx;
    want = want && ny >= 0 && ny < d.nty && nx >= 0 && nx < d.ntx;
    nb = want ? (uint32_t)(d.tile_base + (int64_t)ny * d.ntx + nx) : 0u;
    return want;
}

// The round path's marks: the wanted tiles get the next round in their
// epoch flag; the atomic maximum lets exactly one marker list a tile: the
// one that finds the flag below the next round. Returns the flag's previous
// value (the next round itself where this lane marks nothing), so that
// callers can compare it late and let the wait for the atomic overlap other
// work; the tile's id is in nb.
template <int CONN>
__device__ __forceinline__ uint32_t mark_neighbours(const ImgDesc &d, int lane, int ty, int tx,
                                                const uint32_t (&J)[TS], const uint32_t (&I)[TS],
                                                const uint32_t (&IT)[TS], uint32_t JT, uint32_t JB,
                                                uint32_t JL, uint32_t JR, uint32_t top_in,
                                                uint32_t bot_in, uint64_t col_in,
                                                uint64_t col_out, bool stable,
                                                uint32_t (*tb)[TS + 1], uint32_t *flags,
                                                uint32_t round, uint32_t &nb) {
    const bool want = mark_decide<CONN>(d, lane, ty, tx, J, I, IT, JT, JB, JL, JR, top_in,
                                        bot_in, col_in, col_out, stable, tb, nb);
    const uint32_t nxt = round + 1;
    uint32_t old = nxt;
    if (want) old = atomicMax(flags + nb, nxt);
    return old;
}

// PIPE (the pipelined round kernel; implies a stage the caller has written
// and synchronized): after the stores and once the marking atomics are issued
// the visit issues the stage loads of the next tile (*dn, tn) when has_next, and
// returns them; otherwise it returns zeros.
template <typename T, int CONN, bool TAIL = false, bool PIPE = false, bool NEEDJ = true>
__device__ __forceinline__ StageWords visit_tile(const ImgDesc &d, int64_t t, int lane,
                                                 uint32_t *__restrict__ flags, Appender &app,
                                                 Ctrl *__restrict__ ctrl, uint32_t round,
                                                 int max_iters, uint32_t (*tb)[TS + 1],
                                                 VisitKind kind, TailMarks *tm = nullptr,
                                                 const ImgDesc *dn = nullptr, int64_t tn = 0,
                                                 bool has_next = false) {
    StageWords pre{};
    using P = Pix<T>;
    const bool initial = kind.initial;
    // nothing derived from the lane id is hoisted out of the caller's tile
    // loop: held across the sweeps, such values would be spilled, and their
    // reloads would wait behind the stores of the visit
    asm volatile("" : "+v"(lane));
    int ty, tx;
    tile_place(d, t, ty, tx);
    const int64_t gy0 = (int64_t)ty * TI - 1, gx = (int64_t)tx * TI - 1 + lane;

    uint32_t J[TS], I[TS], IT[TS];
    uint32_t JL, JR; // loaded halo columns 0 and TS-1, lane = row
    bool it_done = false;
    if (PIPE) // the caller has written and synchronized the stage
        stage_read(d, gy0, (int64_t)tx * TI - 1, lane, J, I, IT, JL, JR, (const uint8_t *)tb,
                   it_done, kind);
    else
        load_tile<T, TAIL>(d, t, gy0, (int64_t)tx * TI - 1, lane, J, I, IT, JL, JR, (uint8_t *)tb,
                           it_done, kind);
    if (kind.lowered) { // (outside pixels are key 0)
        uint32_t any = 0;
#pragma unroll
        for (int r = 0; r < TS; ++r) any |= I[r];
        if (__ballot(any != 0) != 0 && lane == 0 &&
            __hip_atomic_load(d.above, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
            atomicOr(d.above, 1u);
    }
    if (!it_done) {
        // (before the mask transpose: fewer registers live)
        halo_cols(J, tb, lane, JL, JR);
#pragma unroll
        for (int r = 0; r < TS; ++r) IT[r] = I[r];
        transpose(IT, tb, lane);
    }
    // loaded halo rows 0 and TS-1 (the sweeps may raise them in registers)
    const uint32_t JT = J[0], JB = J[TS - 1];

    const bool in_lane = lane >= 1 && lane <= TS - 2;
    const uint32_t top_in = J[1], bot_in = J[TS - 2];
    const uint64_t col_in = col_sum<T>(J);
    uint64_t col_prev = col_in;

    bool stable = false, changed = false;
    // Down and up sweeps take the 3 (8-connectivity) or 1 (4-connectivity)
    // neighbours of the adjacent row; on the transposed tile the right and
    // left sweeps take only the in-row neighbour, because the vertical sweeps
    // already test the diagonal ones. A full iteration that changes nothing
    // therefore means every pixel is stable against all its neighbours.
    // A full iteration that changes something mostly leaves the tile at its
    // fixed point; one relaxation step against all neighbours confirms that
    // at a fraction of an iteration's cost (no transposes), and otherwise
    // the iterations go on.
    int it = 0;
    while (it < max_iters) {
        sweep_fwd<CONN == 8>(J, I);
        sweep_bwd<CONN == 8>(J, I);
        transpose(J, tb, lane);
        sweep_fwd<false>(J, IT);
        sweep_bwd<false>(J, IT);
        transpose(J, tb, lane);
        ++it;
        uint64_t col_now = col_sum<T>(J);
        // halo columns may rise too, but only the interior must settle
        bool ch = in_lane && col_now != col_prev;
        col_prev = col_now;
        if (__ballot(ch) == 0) {
            stable = true;
            break;
        }
        changed = true;
        // (int32 visits start checking after the second iteration, which
        // measures faster for them; a first visit at its sweep cap leaves
        // the check out: the tile is left unstable, and so listed again)
        if (sizeof(T) == 4 && it < 2) continue;
        if (initial && it >= max_iters) break;
        relax_once<CONN>(J, I);
        col_now = col_sum<T>(J);
        ch = in_lane && col_now != col_prev;
        col_prev = col_now;
        if (__ballot(ch) == 0) {
            stable = true;
            break;
        }
    }
    if (lane == 0) atomicAdd(&ctrl->iters[t & (NCNT - 1)], (unsigned long long)it);

    if (changed || initial) {
        gptr<T> Jw = (gptr<T>)d.J;
        if (in_lane && gx < d.W) {
            // rows gy0+1 .. gy0+62 are all >= 0; only the last tile row may
            // run past the image
            const int64_t left = d.H - gy0 - 1;
            const int rows = left < TS - 2 ? (int)left : TS - 2;
            uint32_t off = (uint32_t)(gy0 + 1) * (uint32_t)d.pJ + (uint32_t)gx;
            if (rows == TS - 2) {
#pragma unroll
                for (int r = 1; r < TS - 1; ++r) {
                    asm volatile("" : "+v"(off));
                    store_j<T, TAIL>(Jw, off, P::val(J[r]));
                    off += (uint32_t)d.pJ;
                }
            } else {
#pragma unroll
                for (int r = 1; r < TS - 1; ++r) {
                    asm volatile("" : "+v"(off));
                    if (r <= rows) store_j<T, TAIL>(Jw, off, P::val(J[r]));
                    off += (uint32_t)d.pJ;
                }
            }
        }
    }
    // PIPE: the next tile's stage loads go out after this tile's stores and
    // mark atomics (on every path, with no loads when there is no next tile),
    // so that waiting for the marks does not wait for them, and they are in
    // flight while the marks are waited for and the list is appended to.
    // Nothing of the next tile may be loaded earlier (its registers would be
    // live across the sweeps).
    auto fetch_next = [&]() {
        if (PIPE) {
            asm volatile("" ::: "memory");
            pre = stage_fetch<NEEDJ>(*dn, tn, lane, has_next);
        }
    };
    if (!changed && stable) {
        fetch_next();
        return pre;
    }
    if (!TAIL) {
        uint32_t nb = 0;
        const uint32_t old =
            mark_neighbours<CONN>(d, lane, ty, tx, J, I, IT, JT, JB, JL, JR, top_in, bot_in,
                                  col_in, col_prev, stable, tb, flags, round, nb);
        fetch_next();
        // (an opaque use: the comparison stays here, behind the loads that
        // fetch_next issued, rather than right after the atomic)
        uint32_t o = old;
        asm volatile("" : "+v"(o));
        const bool fresh = o < round + 1;
        const uint64_t fm = __ballot(fresh);
        if (fresh) app.buf[app.cnt + __popcll(fm & ((1ull << lane) - 1))] = nb;
        app.cnt += (uint32_t)__popcll(fm);
        return pre;
    }
    uint32_t tnb = 0;
    const bool want = mark_decide<CONN>(d, lane, ty, tx, J, I, IT, JT, JB, JL, JR, top_in, bot_in,
                                        col_in, col_prev, stable, tb, tnb);
    tm->want = want;
    tm->nb = tnb;
    return pre;
}

// The tiles a block of a round visits: band `band`'s list (or, with
// all_tiles, the whole band), entries local, local + per, ... below n, from
// list_in (band start already applied). A round that lists no more tiles
// than the grid has blocks, but more in some band than that band has blocks,
// gives each tile a block of its own: the tail of a flood often sits in one
// or two bands, whose blocks would otherwise visit its tiles one after
// another while the rest of the grid idles. Block g takes entry g of the
// band lists laid end to end. When every band fits its blocks, the bands'
// dealing already gives each tile a block, and keeps neighbouring tiles on
// one die's L2.
struct RoundWork {
    int band;
    int64_t local, per, n, lo;
    const uint32_t *list_in;
    bool fwd;
    // walk the band's tiles in order (static interleave, as in an all-tiles
    // round) and visit those whose epoch flag holds this round, instead of
    // reading the list
    bool walk;
};

// all_tiles: 1 visits every tile (an image's first round), 0 the dirty
// lists, 2 the dirty lists or, for a band that lists at least half its
// tiles, the walk. A list is built in marking order, which scatters the
// tiles visited at one time over the band; the walk visits neighbouring
// tiles together, so they share the cache lines their rows straddle.
// The walk relies on what launch sequences that start at round 1 guarantee:
// a tile is listed for round r exactly when its flag reached r in round
// r - 1. A flag raised again (to r + 1) before the walk reads it means the
// tile is in the next round's list as well, so leaving it to that round
// loses nothing.
__device__ __forceinline__ RoundWork round_work(int64_t n_tiles, const uint32_t *lists,
                                                const uint32_t *counts_in, int all_tiles,
                                                uint32_t round, uint32_t leave) {
    RoundWork w;
    w.band = blockIdx.x % NBANDS;
    w.local = blockIdx.x / NBANDS;
    w.per = gridDim.x / NBANDS;
    w.walk = false;
    if (all_tiles == 1) {
        w.n = band_lo(n_tiles, w.band + 1) - band_lo(n_tiles, w.band);
    } else {
        uint32_t c[NBANDS], total = 0, cmax = 0;
#pragma unroll
        for (int q = 0; q < NBANDS; ++q) {
            c[q] = kconst(counts_in)[q];
            total += c[q];
            cmax = c[q] > cmax ? c[q] : cmax;
        }
        if (total <= leave) { // left to the tile queue (see tail_leave)
            w.n = 0;
        } else if (total <= gridDim.x && cmax > (uint32_t)w.per) {
            uint32_t i = blockIdx.x, cb = c[0];
            int b = 0;
#pragma unroll
            for (int q = 0; q < NBANDS - 1; ++q)
                if (b == q && i >= c[q]) {
                    i -= c[q];
                    b = q + 1;
                    cb = c[q + 1];
                }
            w.band = b;
            w.local = i;
            w.per = cb > 0 ? cb : 1; // one iteration: entry i (or n - 1 - i backward)
            w.n = blockIdx.x < total ? cb : 0;
        } else {
            w.n = kconst(counts_in)[w.band];
            const int64_t nb = band_lo(n_tiles, w.band + 1) - band_lo(n_tiles, w.band);
            if (all_tiles == 2 && w.n > 0 && 2 * w.n >= nb) {
                w.walk = true;
                w.n = nb;
            }
        }
    }
    w.lo = band_lo(n_tiles, w.band);
    w.list_in = lists + (round & 1) * n_tiles + w.lo;
    // Odd rounds walk the band forward, even rounds backward: a tile stored
    // early in a round is read by tiles visited later in it, so information
    // travels down the image within odd rounds and up it within even ones,
    // as in a raster / anti-raster pair of scans.
    w.fwd = (round & 1) != 0;
    return w;
}

__device__ __forceinline__ int64_t round_tile(const RoundWork &w, int all_tiles, int64_t i) {
    const int64_t k = w.fwd ? i : w.n - 1 - i;
    return all_tiles == 1 || w.walk ? w.lo + k : (int64_t)kconst(w.list_in)[k];
}

// The block's tiles of a round, in order: band entries local, local + per,
// ... below n. A walk reads the epoch flags of 64 entries at once and keeps
// those that hold the round.
struct TileCursor {
    int64_t i;     // next entry; walk: first entry of the next batch
    int64_t wi;    // walk: first entry of the current batch
    uint64_t mask; // walk: bit j set if entry wi + j * per is to be visited
};

__device__ __forceinline__ TileCursor cursor_start(const RoundWork &w) {
    return TileCursor{w.local, w.local, 0ull};
}

// The next tile, or -1 when the block has none left (wave-uniform).
__device__ __forceinline__ int64_t cursor_next(TileCursor &c, const RoundWork &w, int all_tiles,
                                               const uint32_t *flags, uint32_t round, int lane) {
    if (!w.walk) {
        if (c.i >= w.n) return -1;
        const int64_t t = round_tile(w, all_tiles, c.i);
        c.i += w.per;
        return t;
    }
    while (c.mask == 0) {
        if (c.i >= w.n) return -1;
        uint32_t ln = (uint32_t)lane;
        asm volatile("" : "+v"(ln));
        const int64_t e = c.i + (int64_t)ln * w.per;
        bool take = false;
        if (e < w.n) {
            const int64_t t = w.lo + (w.fwd ? e : w.n - 1 - e);
            take = __hip_atomic_load(flags + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                   round;
        }
        c.mask = __ballot(take);
        c.wi = c.i;
        c.i += 64 * w.per;
    }
    const int j = __builtin_ctzll(c.mask);
    c.mask &= c.mask - 1;
    return round_tile(w, all_tiles, c.wi + (int64_t)j * w.per);
}

// One tile round on a persistent grid (two waves per SIMD). Block b serves
// band b % NBANDS and visits either every tile of the band (all_tiles) or the
// band's dirty list (see round_work). Tiles are dealt to the band's blocks by
// static interleave, so no block gets more than one tile above another. A
// tile builds its image's initial working values in the image's first round.
// V selects the visit (see visit_kind): -1 dispatches per tile on the image's op
// and first round (mixed batches, the server); otherwise for
// launches whose tiles all take the same visit, which keeps the other three
// variants' code, and their registers, out of the kernel.
template <typename T, int CONN, int V>
__global__ __launch_bounds__(64, 2) void k_tile_round(Imgs imgs, int64_t n_tiles,
                                                      uint32_t *__restrict__ flags,
                                                      uint32_t *__restrict__ lists,
                                                      const uint32_t *__restrict__ counts_in,
                                                      uint32_t *__restrict__ counts_out,
                                                      int all_tiles, Ctrl *__restrict__ ctrl,
                                                      uint32_t round, int max_iters,
                                                      uint32_t leave,
                                                      uint32_t *__restrict__ counts_clear,
                                                      uint32_t *__restrict__ queued) {
    if (counts_clear && blockIdx.x == 0 && threadIdx.x < NBANDS) counts_clear[threadIdx.x] = 0;
    __shared__ uint32_t tb[TS][TS + 1]; // transpose buffer (and load stage)
    __shared__ uint32_t abuf[APP_CAP];
    const int lane = threadIdx.x;
    const RoundWork w = round_work(n_tiles, lists, counts_in, all_tiles, round, leave);
    Appender app{abuf, 0, lists + ((round + 1) & 1) * n_tiles, counts_out, n_tiles,
                 V < 0 || (V & 1) ? queued : nullptr};
    TileCursor cur = cursor_start(w);
    for (int64_t t; (t = cursor_next(cur, w, all_tiles, flags, round, lane)) >= 0;) {
        const ImgDesc d = load_desc(imgs, t);
        if (!d.done)
            visit_tile<T, CONN>(d, t, lane, flags, app, ctrl, round, max_iters, tb,
                                visit_kind<V, sizeof(T) == 1>(imgs, d, round));
        if (app.cnt > APP_CAP - 9) app_flush(app, lane);
    }
    app_flush(app, lane);
}

// The same round for launches whose images are all uint8 (of a size the stage
// reaches), software-pipelined
// over the block's tiles: the stage loads of the next tile are issued during
// the current visit, behind its stores and marking atomics, so
// that their memory latency (and that of the next list entry and
// descriptor) overlaps the wait for the marks and the append to the list
// instead of starting the next visit. The loads land in registers that the
// sweeps no longer need; the next visit writes them to the stage. With V < 0
// (mixed batches, the server) a visit's kind is read from its image.
// Planes of any base and pitch take this kernel: a batch of 40 mixed tiles of
// odd sizes spends 502 us in its rounds (757 us when such planes were loaded
// byte by byte by k_tile_round), one 293 x 421 image 61 us instead of 120.
template <int CONN, int V>
__global__ __launch_bounds__(64, 2) void k_tile_round_pf(Imgs imgs, int64_t n_tiles,
                                                         uint32_t *__restrict__ flags,
                                                         uint32_t *__restrict__ lists,
                                                         const uint32_t *__restrict__ counts_in,
                                                         uint32_t *__restrict__ counts_out,
                                                         int all_tiles, Ctrl *__restrict__ ctrl,
                                                         uint32_t round, int max_iters,
                                                         uint32_t leave,
                                                         uint32_t *__restrict__ counts_clear,
                                                      uint32_t *__restrict__ queued) {
    if (counts_clear && blockIdx.x == 0 && threadIdx.x < NBANDS) counts_clear[threadIdx.x] = 0;
    constexpr bool needJ = V != 3 && V != 5;
    __shared__ uint32_t tb[TS][TS + 1]; // transpose buffer and load stage
    __shared__ uint32_t abuf[APP_CAP];
    const int lane = threadIdx.x;
    const RoundWork w = round_work(n_tiles, lists, counts_in, all_tiles, round, leave);
    Appender app{abuf, 0, lists + ((round + 1) & 1) * n_tiles, counts_out, n_tiles,
                 V < 0 || (V & 1) ? queued : nullptr};
    uint8_t *stage = (uint8_t *)tb;
    TileCursor cur = cursor_start(w);
    // the next tile to visit and its image (images that are done take no visit)
    auto next = [&](ImgDesc &d) -> int64_t {
        int64_t t;
        while ((t = cursor_next(cur, w, all_tiles, flags, round, lane)) >= 0) {
            d = load_desc(imgs, t);
            if (!d.done) break;
        }
        return t;
    };
    ImgDesc d{};
    int64_t t = next(d);
    if (t >= 0) {
        StageWords pre = stage_fetch<needJ>(d, t, lane);
        while (true) {
            const VisitKind kind = visit_kind<V, false>(imgs, d, round);
            // the fetched rows of tile t go to the stage; the previous visit's
            // last reads of the transpose buffer are behind this sync
            wave_sync();
            stage_commit_words<needJ>(pre, d, t, lane, stage, kind.fill);
            wave_sync();
            ImgDesc dn = d;
            int64_t tn = next(dn);
            const bool has = tn >= 0;
            if (!has) {
                tn = t;
                dn = d;
            }
            pre = visit_tile<uint8_t, CONN, false, true, needJ>(d, t, lane, flags, app, ctrl,
                                                                round, max_iters, tb, kind,
                                                                nullptr, &dn, tn, has);
            if (app.cnt > APP_CAP - 9) app_flush(app, lane);
            if (!has) break;
            t = tn;
            d = dn;
        }
    }
    app_flush(app, lane);
}

// ------------------------------------------------------------- tile queue

// Before a tile queue that follows several rounds: finds the round whose lists it
// starts from (`round`, or an earlier one whose tiles were left to the queue: no more
// than `leave`; the rounds after it had nothing to visit), and marks band b's (block
// b) listed tiles as queued.
__global__ void k_tile_queue_mark(const uint32_t *__restrict__ lists, Ctrl *ctrl, int64_t n_tiles,
                                  uint32_t round, uint32_t leave, uint32_t *__restrict__ state) {
    __shared__ uint32_t from;
    const int b = blockIdx.x;
    if (threadIdx.x == 0) {
        uint32_t r = 2;
        for (; r < round; ++r) {
            uint32_t total = 0;
#pragma unroll
            for (int q = 0; q < NBANDS; ++q) total += ctrl->round_tiles[r][q];
            if (total <= leave) break;
        }
        from = r;
        if (b == 0) ctrl->seed_round = r;
    }
    __syncthreads();
    const uint32_t n = ctrl->round_tiles[from][b];
    const uint32_t *list = lists + (from & 1) * n_tiles + band_lo(n_tiles, b);
    for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) state[list[i]] = 1u;
}

// Entry i of the lists of a round laid end to end (uniform).
__device__ __forceinline__ uint32_t listed_tile(const Ctrl *ctrl, const uint32_t *lists,
                                                int64_t n_tiles, uint32_t round, uint32_t i) {
    const auto c = kconst(ctrl->round_tiles[round]);
    uint32_t lo = 0; // entries of the bands before
    int64_t at = 0;
#pragma unroll
    for (int q = 0; q < NBANDS; ++q) {
        const uint32_t n = c[q];
        if (i >= lo && i < lo + n) at = band_lo(n_tiles, q) + (i - lo);
        lo += n;
    }
    return kconst(lists + (round & 1) * n_tiles)[at];
}

// The tile queue (the regular phase without rounds): each wave takes a tile
// off the lists it starts from (tickets below their length `seeds`) or off the ring,
// visits it like a tile round does, and marks the neighbours
// straight into the ring, so a chain of dependent tiles costs one visit per
// link instead of one round. A wave takes a ticket (the next ring position)
// and waits for that entry, so no two waves contend for an entry. The wave
// that retires the last queued-or-running tile writes a stop entry for every
// wave. The watchdog (ring_take) turns a stall into an error instead of a hang.
// Bound by the latency of a link, so a wave hands itself the first idle
// neighbour it marks instead of queueing it: on the holes of a 4096 x 4096
// tile, after 8 rounds, the queue takes 269 us (357 us with every neighbour
// through the ring). The whole launch ends when every wave has its stop: written
// by one lane, 2048 stops took 50 us. A wave that retires a tile draws its next
// ticket in the same instruction. Tickets read the lists themselves: a seed launch
// that copied them to the ring cost small calls 3 us (293 x 421 uint8: 58.8 -> 56.2 us).

// Waves per workgroup of the tile queue. int32 visits have no register to spare
// for telling the waves of a workgroup apart (27 spills become 50, h-dome of a
// 4096 x 4096 int32 tile 714 -> 767 us).
template <typename T> constexpr int TQ_WAVES = sizeof(T) == 1 ? 4 : 1;

template <typename T, int CONN, int V>
__global__ __launch_bounds__(64 * TQ_WAVES<T>, 2) void k_tile_queue(Imgs imgs, Ctrl *__restrict__ ctrl,
                                                      uint32_t *__restrict__ state,
                                                      uint32_t *__restrict__ ring, uint64_t cap,
                                                      int max_iters,
                                                      unsigned long long wait_us,
                                                      uint32_t round, uint32_t from,
                                                      const uint32_t *__restrict__ lists,
                                                      int64_t n_tiles) {
    __shared__ uint32_t tbs[TQ_WAVES<T>][TS][TS + 1];
    const int lane = threadIdx.x & 63;
    uint32_t (*tb)[TS + 1] = tbs[TQ_WAVES<T> == 1 ? 0 : threadIdx.x >> 6];
    // the round whose lists this launch starts from; 0: as k_tile_queue_mark found
    const uint32_t first_list = from ? from : *kconst(&ctrl->seed_round);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctrl->rounds = round - 1;
        if (from) ctrl->seed_round = from;
    }
    uint32_t seeds = 0;
#pragma unroll
    for (int q = 0; q < NBANDS; ++q) seeds += kconst(ctrl->round_tiles[first_list])[q];
    Appender app{nullptr, 0, nullptr, nullptr, 0, nullptr}; // unused: marks go to the ring
    unsigned long long visits = 0;
    // nothing listed: no wave will ever retire a tile and write the stops
    if (seeds == 0) return;
    uint32_t t = Q_EMPTY; // the tile this wave holds: its state is 2, it counts as pending
    unsigned long long ticket = ring_tickets(ctrl, TQ_WAVES<T>);
    while (true) {
        if (t == Q_EMPTY) {
            const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)ticket);
            if (ticket < seeds) {
                t = listed_tile(ctrl, lists, n_tiles, first_list, i);
            } else if (lane == 0) {
                t = ring_take(ctrl, ring, cap, ticket - seeds, wait_us);
            }
            t = (uint32_t)__builtin_amdgcn_readfirstlane(t); // (uniform: scalar descriptor loads)
            if (t == Q_STOP) break;
            // queued -> visited, performed before any pixel is read: a mark that
            // comes later finds state 2 and gets the tile visited again, one that
            // came earlier had its stores done before it
            if (lane == 0)
                (void)__hip_atomic_exchange(state + t, 2u, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
            wait_vmem();
        }
        const ImgDesc d = load_desc(imgs, t);
        TailMarks tm;
        if (!d.done) {
            ++visits;
            const bool fill = V >= 0 ? (V >> 1) & 1 : d.op == MR_OP_FILL;
            visit_tile<T, CONN, true>(d, t, lane, nullptr, app, ctrl, 0, max_iters, tb,
                                      VisitKind{fill, false, false}, &tm);
        }
        // the visits these marks lead to must see this visit's stores
        wait_vmem();
        // Marks and the release of this tile, all in flight together. The first
        // neighbour asked for is tried as this wave's next tile (idle ->
        // visited by this wave), without a way through the ring; lane 63
        // releases the tile (visited -> idle), unless the sweep cap stopped
        // its visit: then the wave keeps it.
        const uint64_t wm = __ballot(tm.want);
        const bool again = wm & 1;
        const uint64_t others = wm & ~1ull;
        const int first = others && !again ? __builtin_ctzll(others) : -1;
        const bool try_next = lane == first, release = lane == 63 && !again;
        uint32_t expect = release ? 2u : 0u;
        bool swapped = false;
        if (try_next || release)
            swapped = __hip_atomic_compare_exchange_strong(
                state + (release ? t : tm.nb), &expect, release ? 0u : 2u, __ATOMIC_RELAXED,
                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t prev = 1u;
        if (tm.want && lane != 0 && !try_next)
            prev = __hip_atomic_fetch_or(state + tm.nb, 1u, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
        uint32_t next = again ? t : Q_EMPTY;
        if (__ballot(try_next && swapped)) {
            next = (uint32_t)__builtin_amdgcn_readlane(tm.nb, first);
        } else if (first >= 0) {
            // queued, visited or marked already: an ordinary mark (by now the tile
            // may be idle again, and is then queued by this lane)
            if (try_next)
                prev = __hip_atomic_fetch_or(state + tm.nb, 1u, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
        }
        uint32_t push = prev == 0u ? tm.nb : Q_EMPTY;
        if (again) {
            // visited again by this wave: marks from before its loads are answered
            if (lane == 0)
                (void)__hip_atomic_exchange(state + t, 2u, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
        } else if (__ballot(release && !swapped)) {
            // marked while it was visited (state 3): this wave visits it again, or
            // queues it if it has another tile already
            if (next == Q_EMPTY) {
                next = t;
                if (lane == 0)
                    (void)__hip_atomic_exchange(state + t, 2u, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT);
            } else if (lane == 63) {
                __hip_atomic_store(state + t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                push = t;
            }
        }
        wait_vmem();
        ring_push(ctrl, ring, cap, push, lane);
        // one entry held before and, with a next tile, one held now
        if (next == Q_EMPTY) ticket = ring_retire(ctrl, ring, cap, gridDim.x * TQ_WAVES<T>, seeds,
                                              lane);
        t = next;
    }
    if (lane == 0 && visits)
        atomicAdd(&ctrl->tiles[(blockIdx.x * TQ_WAVES<T> + (threadIdx.x >> 6)) & (NCNT - 1)], visits);
}

// ------------------------------------------------------------------- seeds

// One relaxation step over each tile still dirty for `round`: every interior
// pixel takes min(I, max of J over itself and its neighbours). Raised pixels
// are stored, their bits form the tile's frontier bitmap rows, and the tile
// enters the ring. Tiles that are not dirty only clear their bitmap and flag.
template <typename T, int CONN>
__device__ __forceinline__ void seed_tile(const ImgDesc &d, int64_t t, int lane, Ctrl *ctrl,
                                          uint64_t *bitmap, uint32_t *qflag, uint32_t *ring,
                                          uint64_t cap, uint8_t *stage, bool fill) {
    using P = Pix<T>;
    int ty, tx;
    tile_place(d, t, ty, tx);
    const int64_t gy0 = (int64_t)ty * TI - 1, gx = (int64_t)tx * TI - 1 + lane;
    uint32_t J[TS], I[TS], IT[TS], JL, JR;
    bool it_done = false;
    load_tile<T>(d, t, gy0, (int64_t)tx * TI - 1, lane, J, I, IT, JL, JR, stage, it_done,
                 VisitKind{fill, false, false});
    uint64_t myrow = 0; // lane r ends up holding row r's bits
    uint32_t nseed = 0;
    gptr<T> Jw = (gptr<T>)d.J;
    uint32_t off = (uint32_t)gy0 * (uint32_t)d.pJ + (uint32_t)gx;
#pragma unroll
    for (int r = 1; r < TS - 1; ++r) {
        off += (uint32_t)d.pJ;
        uint32_t n = max(J[r - 1], J[r + 1]);
        n = max(n, max(from_lower_lane(J[r]), from_upper_lane(J[r])));
        if (CONN == 8) {
            n = max(n, max(from_lower_lane(J[r - 1]), from_upper_lane(J[r - 1])));
            n = max(n, max(from_lower_lane(J[r + 1]), from_upper_lane(J[r + 1])));
        }
        const uint32_t v = min(max(J[r], n), I[r]);
        // only this tile's own pixels: the halo columns belong to the
        // neighbours (outside pixels have I == J == 0 and never rise)
        const bool raised = lane >= 1 && lane <= TS - 2 && v > J[r];
        const uint64_t bits = __ballot(raised);
        if (raised) Jw[off] = P::val(v);
        if (lane == r) myrow = bits;
        nseed += (uint32_t)__popcll(bits);
    }
    bitmap[t * TS + lane] = myrow;
    if (lane == 0 && nseed) {
        qflag[t] = 1;
        __hip_atomic_fetch_add(&ctrl->seeds_total.v, (unsigned long long)nseed,
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // the queue runs in a later launch, which sees this one's stores
        ring_push(ctrl, ring, cap, (uint32_t)t);
    }
}

// One relaxation step over each tile dirty for `round` (the round after the
// last one run): every interior pixel takes min(I, max of J over itself and
// its neighbours). Raised pixels are stored, their bits form the tile's rows
// of the frontier bitmap (one ballot per row), and the tile enters the
// frontier ring. The bitmap and queue flags start cleared.
template <typename T, int CONN>
__global__ __launch_bounds__(64) void k_seed(Imgs imgs, int64_t n_tiles,
                                             const uint32_t *__restrict__ lists, uint32_t round,
                                             Ctrl *__restrict__ ctrl,
                                             uint64_t *__restrict__ bitmap,
                                             uint32_t *__restrict__ qflag,
                                             uint32_t *__restrict__ ring, uint64_t cap) {
    __shared__ __align__(16) uint8_t stage[STAGE_PAD + 2 * STAGE_BYTES];
    const int lane = threadIdx.x;
    const int band = blockIdx.x % NBANDS;
    const int64_t local = blockIdx.x / NBANDS, per = gridDim.x / NBANDS;
    const uint32_t *list_in = lists + (round & 1) * n_tiles + band_lo(n_tiles, band);
    const int64_t n = ctrl->round_tiles[round][band];
    for (int64_t i = local; i < n; i += per) {
        const int64_t t = list_in[i];
        const ImgDesc d = load_desc(imgs, t);
        if (d.done) continue;
        seed_tile<T, CONN>(d, t, lane, ctrl, bitmap, qflag, ring, cap, stage,
                           d.op == MR_OP_FILL);
    }
}

// ------------------------------------------------------------------- queue

constexpr int QWAVES = 4;                  // waves per queue workgroup
constexpr int LIST_CAP = TI * TI;          // claimed pixels of one tile

// Process one claimed pixel: propagate its value to every neighbour that it
// can raise (Algorithm 1's PropagationCondition / Update), pushing each
// neighbour actually raised.
template <typename T, int CONN>
__device__ __forceinline__ void relax_pixel(const ImgDesc &d, int64_t y, int64_t x, Ctrl *ctrl,
                                            uint64_t *bitmap, uint32_t *qflag, uint32_t *ring,
                                            uint64_t cap, uint32_t &npush,
                                            unsigned long long &retries) {
    using P = Pix<T>;
    T *Jw = (T *)d.J;
    cgptr<T> Ip = (cgptr<T>)d.I;
    const bool fill = d.op == MR_OP_FILL;
    // uint8 images with a widened plane raise 32-bit keys there
    uint32_t *Wd = sizeof(T) == 1 ? d.wide : nullptr;
    auto load_key = [&](int64_t yy, int64_t xx) -> uint32_t {
        if (Wd)
            return __hip_atomic_load(Wd + yy * d.W + xx, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
        return Atom<T>::load_key(Jw, yy * d.pJ + xx);
    };
    auto raise = [&](int64_t yy, int64_t xx, uint32_t k) -> bool {
        if (Wd)
            return __hip_atomic_fetch_max(Wd + yy * d.W + xx, k, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT) < k;
        return Atom<T>::raise(Jw, yy * d.pJ + xx, k, retries);
    };
    const uint32_t jp = load_key(y, x);
#pragma unroll
    for (int k = 0; k < CONN; ++k) {
        // edge neighbours first, then diagonals
        const int dy = (k == 0) ? -1 : (k == 1) ? 1 : (k < 4) ? 0 : (k < 6 ? -1 : 1);
        const int dx = (k < 2) ? 0 : (k == 2) ? -1 : (k == 3) ? 1 : ((k & 1) ? 1 : -1);
        const int64_t yy = y + dy, xx = x + dx;
        if (yy < 0 || yy >= d.H || xx < 0 || xx >= d.W) continue;
        const uint32_t jq = load_key(yy, xx);
        if (jq >= jp) continue;
        uint32_t iq = P::key(Ip[yy * d.pI + xx]);
        if (fill) iq = P::KMAX - iq;
        if (jq >= iq) continue;
        const uint32_t v = min(jp, iq);
        if (!raise(yy, xx, v)) continue;
        // push: set the pixel's frontier bit, enqueue its tile once
        const int tyq = (int)(yy / TI), txq = (int)(xx / TI);
        const int rq = (int)(yy - (int64_t)tyq * TI) + 1, lq = (int)(xx - (int64_t)txq * TI) + 1;
        const int64_t tq = d.tile_base + (int64_t)tyq * d.ntx + txq;
        const uint64_t bit = 1ull << lq;
        // the raise above returned, so it is done before the bit is set
        const uint64_t old = __hip_atomic_fetch_or(bitmap + tq * TS + rq, bit, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT);
        ++npush;
        if (old & bit) continue;
        if (__hip_atomic_exchange(qflag + tq, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
            ring_push(ctrl, ring, cap, (uint32_t)tq);
    }
}

template <typename T, int CONN>
__global__ __launch_bounds__(64 * QWAVES) void k_queue(Imgs imgs, Ctrl *__restrict__ ctrl,
                                                       uint64_t *__restrict__ bitmap,
                                                       uint32_t *__restrict__ qflag,
                                                       uint32_t *__restrict__ ring, uint64_t cap,
                                                       unsigned long long wait_us) {
    __shared__ uint16_t list[QWAVES][LIST_CAP];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint16_t *mylist = list[w];
    uint32_t npush = 0, npop = 0;
    unsigned long long retries = 0;
    const int cslot = (int)((blockIdx.x * QWAVES + w) & (NCNT - 1));
    // Every access that other waves' work depends on is a device-scope
    // atomic (pixels, bitmap rows, queue flags, ring), each waited for where
    // a later one must see it: no cache-wide fences. Nothing seeded: no wave
    // would ever retire an entry and write the stops.
    if (__hip_atomic_load(&ctrl->pending.v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0)
        return;

    // (each wave draws its own: with neighbouring tickets in one workgroup, chains of
    // tiles, whose links then stay on one compute unit, ran a fifth slower. Fill-holes at
    // 4096 x 4096, 8 rounds, then this: 24.8 ms so, 19.8 ms with single draws.)
    unsigned long long ticket = 0;
    if (lane == 0)
        ticket = __hip_atomic_fetch_add(&ctrl->q_head.v, 1ull, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
    ticket = __shfl(ticket, 0);
    while (true) {
        uint32_t t = Q_EMPTY;
        if (lane == 0) t = ring_take(ctrl, ring, cap, ticket, wait_us);
        t = __shfl(t, 0);
        if (t == Q_STOP) break;
        const ImgDesc d = load_desc(imgs, t);
        const int64_t lt = (int64_t)t - d.tile_base;
        const int ty = (int)(lt / d.ntx), tx = (int)(lt - (int64_t)ty * d.ntx);
        const int64_t gy0 = (int64_t)ty * TI - 1, gx0 = (int64_t)tx * TI - 1;
        uint64_t *rows = bitmap + (int64_t)t * TS;
        bool released = false;
        while (true) {
            uint64_t bits = __hip_atomic_exchange(rows + lane, 0ull, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT);
            if (__ballot(bits != 0) == 0) {
                if (released) break;
                // let pushes enqueue the tile again, then look once more (the
                // store is done before the rows are read again)
                if (lane == 0)
                    __hip_atomic_store(qflag + t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                wait_vmem();
                released = true;
                continue;
            }
            // compact the claimed bits into a pixel list (row << 8 | lane)
            const uint32_t c = (uint32_t)__popcll(bits);
            uint32_t off = c; // inclusive scan over lanes
#pragma unroll
            for (int s = 1; s < 64; s <<= 1) {
                const uint32_t o = __shfl_up(off, s);
                if (lane >= s) off += o;
            }
            const uint32_t total = __shfl(off, 63);
            off -= c;
            while (bits) {
                const int l = __ffsll((unsigned long long)bits) - 1;
                bits &= bits - 1;
                mylist[off++] = (uint16_t)((lane << 8) | l);
            }
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
            for (uint32_t base = 0; base < total; base += 64) {
                const uint32_t k = base + lane;
                if (k < total) {
                    const uint32_t e = mylist[k];
                    const int64_t y = gy0 + (e >> 8), x = gx0 + (e & 0xFF);
                    relax_pixel<T, CONN>(d, y, x, ctrl, bitmap, qflag, ring, cap, npush, retries);
                }
            }
            npop += total;
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            __builtin_amdgcn_wave_barrier();
            if (released) {
                // bits arrived after the release; own the tile again if nobody
                // re-enqueued it, else leave the rest to the new entry
                uint32_t prev = 0;
                if (lane == 0)
                    prev = __hip_atomic_exchange(qflag + t, 1u, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT);
                prev = __shfl(prev, 0);
                if (prev != 0) break;
                released = false;
            }
        }
        // everything this tile produced is pushed; retire the ring entry
        wait_vmem();
        ticket = ring_retire(ctrl, ring, cap, gridDim.x * QWAVES, 0, lane);
    }
    // fold the per-lane counters
    unsigned long long p = npush, r = retries;
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        p += __shfl_xor(p, s);
        r += __shfl_xor(r, s);
    }
    if (lane == 0) {
        atomicAdd(&ctrl->pushes[cslot], p);
        atomicAdd(&ctrl->pops[cslot], (unsigned long long)npop);
        atomicAdd(&ctrl->cas[cslot], r);
    }
}

// ------------------------------------------------------------ small kernels

__global__ void k_clear_u32(uint32_t *p, int64_t n, uint32_t v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void k_clear_ctrl(Ctrl *c, int64_t n_tiles) {
    unsigned long long *p = (unsigned long long *)c;
    const int n = (int)(sizeof(Ctrl) / sizeof(unsigned long long));
    for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
    __syncthreads();
    if (threadIdx.x < NBANDS)
        c->round_tiles[1][threadIdx.x] =
            (uint32_t)(band_lo(n_tiles, threadIdx.x + 1) - band_lo(n_tiles, threadIdx.x));
}

// The start of a launch sequence in one kernel: the control block (block 0;
// round 1 lists every tile of each band), the dirty flags, the queue
// flags and ring of the tile queue and the queue phase, and a single image's
// descriptor.
__global__ void k_clear_start(Ctrl *c, int64_t n_tiles, uint32_t *flags, uint32_t *qflag,
                              uint32_t *ring, int64_t ring_cap, ImgDesc *desc, ImgDesc d) {
    if (desc && blockIdx.x == 0 && threadIdx.x == 0) {
        *desc = d;
        if (d.above) *d.above = 0u;
    }
    if (blockIdx.x == 0) {
        unsigned long long *p = (unsigned long long *)c;
        const int n = (int)(sizeof(Ctrl) / sizeof(unsigned long long));
        for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0;
        __syncthreads();
        if (threadIdx.x < NBANDS)
            c->round_tiles[1][threadIdx.x] =
                (uint32_t)(band_lo(n_tiles, threadIdx.x + 1) - band_lo(n_tiles, threadIdx.x));
    }
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n_tiles; i += stride) {
        flags[i] = 0u;
        qflag[i] = 0u;
    }
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < ring_cap; i += stride)
        ring[i] = Q_EMPTY;
}

// The queue phase's widened planes (uint8 images): block t copies tile t's
// interior between J and the image's 32-bit plane, lane = column.
template <bool TO_WIDE>
__global__ __launch_bounds__(64) void k_widen(Imgs imgs, int64_t t0) {
    const int64_t t = t0 + blockIdx.x;
    const ImgDesc d = load_desc(imgs, t);
    if (!d.wide) return;
    const int lane = threadIdx.x;
    const int64_t lt = t - d.tile_base;
    const int64_t ty = lt / d.ntx, tx = lt - ty * d.ntx;
    const int64_t x = tx * TI + lane - 1;
    if (lane < 1 || lane > TI || x >= d.W) return;
    uint8_t *J = (uint8_t *)d.J;
    for (int64_t y = ty * TI, ye = std::min<int64_t>(y + TI, d.H); y < ye; ++y) {
        if (TO_WIDE)
            d.wide[y * d.W + x] = J[y * d.pJ + x];
        else
            J[y * d.pJ + x] = (uint8_t)d.wide[y * d.W + x];
    }
}

// Fill-holes epilogue: out = NOT J for every fill-holes image of the launch. Block t
// takes the 64 x 64 block number t - tile_base of its image (there are no more of
// those than tiles), 16 bytes a lane: J's rows are 16-byte aligned in the
// workspace, out's may start on any pixel. Bound by its launch on one tile's
// 2 x 16 MiB; a pixel a lane, 62 dependent rows a block, took 24 us there.
template <typename T>
__global__ __launch_bounds__(64) void k_fill_output(Imgs imgs, int64_t t0) {
    constexpr int E = 16 / (int)sizeof(T); // pixels a lane and step
    constexpr int LPR = TS / E;            // lanes a row
    const int64_t t = t0 + blockIdx.x;
    const int lane = threadIdx.x;
    const ImgDesc d = load_desc(imgs, t);
    if (d.op != MR_OP_FILL || d.done) return;
    const int64_t lt = t - d.tile_base, nbx = (d.W + TS - 1) / TS, by = lt / nbx;
    const int64_t x = (lt - by * nbx) * TS + E * (lane % LPR);
    if (x >= d.W) return;
#pragma unroll 4
    for (int r = lane / LPR; r < TS; r += 64 / LPR) {
        const int64_t y = by * TS + r;
        if (y >= d.H) break;
        // (~key is the key of the complement in both types: bitwise NOT of the bits)
        v4u v = *(const v4u *)((const T *)d.J + y * d.pJ + x);
        v = ~v;
        T *o = (T *)d.out + y * d.pO + x;
        if (x + E <= d.W) {
            __builtin_memcpy(o, &v, 16);
        } else {
            T e[E];
            __builtin_memcpy(e, &v, 16);
#pragma unroll
            for (int k = 0; k < E; ++k)
                if (x + k < d.W) o[k] = e[k];
        }
    }
}

__global__ void k_store_u64(unsigned long long *p, unsigned long long v) { *p = v; }

struct DescChunk {
    ImgDesc d[DESC_CHUNK];
    int n;
};

__global__ void k_put_descs(ImgDesc *dst, DescChunk c) {
    if ((int)threadIdx.x < c.n) dst[threadIdx.x] = c.d[threadIdx.x];
}

// ------------------------------------------------------------------ server

// Copy a job's inputs into its planes: 16 bytes a lane from any address, a row's last
// bytes one by one; blockIdx.y says which plane. Both planes of a 2048 x 2048 uint8 job
// (16 MiB moved) cost its launch and little more.
__global__ __launch_bounds__(256) void k_server_copy(char *a, const char *x, char *b,
                                                     const char *y, int64_t dp, int64_t sp,
                                                     int64_t row, uint32_t H) {
    char *dst = blockIdx.y ? b : a;
    const char *src = blockIdx.y ? y : x;
    const uint32_t vec = (uint32_t)((row + 15) / 16), items = H * vec;
    for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < items; i += gridDim.x * 256u) {
        const uint32_t r = i / vec;
        const int64_t c = 16 * (int64_t)(i - r * vec);
        const char *p = src + r * sp + c;
        char *o = dst + r * dp + c;
        if (c + 16 <= row) {
            v4u v;
            __builtin_memcpy(&v, p, 16);
            *(v4u *)o = v;
        } else {
            for (int64_t k = 0; c + k < row; ++k) o[k] = p[k];
        }
    }
}

// Admit images: image blockIdx.y's descriptor, owner[t] for its tiles, and every one
// of its tiles on the dirty list of `round` (where it builds its initial
// values). One thread per tile; a wave reserves its places in a band's list with
// one counter update.
struct AdmitChunk {
    ImgDesc d[DESC_CHUNK];
    int32_t slot[DESC_CHUNK];
};
__global__ __launch_bounds__(256) void k_server_admit(ImgDesc *descs, AdmitChunk c, uint32_t *owner,
                                                      uint32_t *flags, uint32_t *lists_round,
                                                      uint32_t *counts_round, int64_t n_tiles,
                                                      uint32_t round) {
    const ImgDesc &d = c.d[blockIdx.y];
    const int64_t nt = (int64_t)d.ntx * d.nty;
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int lane = threadIdx.x & 63;
    if (i == 0) descs[c.slot[blockIdx.y]] = d;
    const bool in = i < nt;
    const int64_t t = d.tile_base + i;
    const int b = in ? band_of(n_tiles, t) : -1;
    for (int q = 0; q < NBANDS; ++q) {
        const uint64_t m = __ballot(b == q);
        if (m == 0) continue;
        uint32_t pos = 0;
        if (lane == 0) pos = atomicAdd(counts_round + q, (uint32_t)__popcll(m));
        pos = __shfl(pos, 0) + (uint32_t)__popcll(m & ((1ull << lane) - 1));
        if (b == q) lists_round[band_lo(n_tiles, q) + pos] = (uint32_t)t;
    }
    if (!in) return;
    owner[t] = (uint32_t)c.slot[blockIdx.y];
    flags[t] = round;
}

// busy[image] = stamp for every image with a tile on the round's lists.
__global__ void k_server_status(const uint32_t *lists_round, const uint32_t *counts_round,
                                const uint32_t *owner, uint32_t *busy, int64_t n_tiles,
                                uint32_t stamp) {
    const int b = blockIdx.x % NBANDS;
    const int64_t per = (gridDim.x / NBANDS) * (int64_t)blockDim.x;
    const int64_t n = counts_round[b];
    const uint32_t *l = lists_round + band_lo(n_tiles, b);
    for (int64_t i = (blockIdx.x / NBANDS) * (int64_t)blockDim.x + threadIdx.x; i < n; i += per)
        busy[owner[l[i]]] = stamp;
}

// ---------------------------------------------------------------- launchers

int persistent_grid() {
    static int g = 0;
    if (!g) {
        int dev = 0, cus = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess &&
            cus > 0)
            g = cus * 8;
        else
            g = 2048;
    }
    return g;
}

hipError_t launch_server_copy(void *a, const void *x, void *b, const void *y, int64_t dp,
                              int64_t sp, int64_t row, int64_t H, hipStream_t s) {
    const int64_t items = H * ((row + 15) / 16);
    const dim3 grid((unsigned)std::min<int64_t>((items + 255) / 256, 2048), y ? 2 : 1);
    hipLaunchKernelGGL(k_server_copy, grid, dim3(256), 0, s, (char *)a, (const char *)x, (char *)b,
                       (const char *)y, dp, sp, row, (uint32_t)H);
    return hipGetLastError();
}

hipError_t launch_server_admit(ImgDesc *descs, const int32_t *slots, const ImgDesc *d, int n,
                               uint32_t *owner, uint32_t *flags, uint32_t *lists_round,
                               uint32_t *counts_round, int64_t n_tiles, uint32_t round,
                               hipStream_t s) {
    if (n < 1 || n > DESC_CHUNK) return hipErrorInvalidValue;
    AdmitChunk c{};
    int64_t most = 1;
    for (int i = 0; i < n; ++i) {
        c.d[i] = d[i];
        c.slot[i] = slots[i];
        most = std::max<int64_t>(most, (int64_t)d[i].ntx * d[i].nty);
    }
    hipLaunchKernelGGL(k_server_admit, dim3((unsigned)((most + 255) / 256), (unsigned)n), dim3(256), 0,
                       s, descs, c, owner, flags, lists_round, counts_round, n_tiles, round);
    return hipGetLastError();
}

hipError_t launch_server_status(const uint32_t *lists_round, const uint32_t *counts_round,
                                const uint32_t *owner, uint32_t *busy, int64_t n_tiles,
                                uint32_t stamp, hipStream_t s) {
    hipLaunchKernelGGL(k_server_status, dim3(NBANDS * 32), dim3(256), 0, s, lists_round,
                       counts_round, owner, busy, n_tiles, stamp);
    return hipGetLastError();
}

hipError_t launch_clear_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_clear_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_clear_ctrl(Ctrl *c, int64_t n_tiles, hipStream_t s) {
    hipLaunchKernelGGL(k_clear_ctrl, dim3(1), dim3(256), 0, s, c, n_tiles);
    return hipGetLastError();
}
hipError_t launch_clear_start(Ctrl *c, int64_t n_tiles, uint32_t *flags, uint32_t *qflag,
                              uint32_t *ring, int64_t ring_cap, ImgDesc *desc, const ImgDesc &d,
                              hipStream_t s) {
    const int64_t n = std::max<int64_t>(n_tiles, ring_cap);
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(k_clear_start, dim3((unsigned)blocks), dim3(256), 0, s, c, n_tiles, flags,
                       qflag, ring, ring_cap, desc, d);
    return hipGetLastError();
}

template <typename T, int CONN, int V>
static hipError_t tile_round_v(const Imgs &imgs, int64_t n_tiles, uint32_t *flags,
                               uint32_t *lists, const uint32_t *cin, uint32_t *cout, int all,
                               Ctrl *ctrl, uint32_t round, int max_iters, int grid,
                               hipStream_t s, uint32_t leave, uint32_t *clear, uint32_t *queued) {
    const int64_t want = std::max<int64_t>(NBANDS, (n_tiles + NBANDS - 1) / NBANDS * NBANDS);
    const unsigned g = (unsigned)(std::min<int64_t>(grid, want) / NBANDS * NBANDS);
    // (uint8 planes beyond the stage's range are rare: one kernel for all visits)
    constexpr int VR = sizeof(T) == 1 ? -1 : V;
    if (sizeof(T) == 1 && imgs.staged)
        hipLaunchKernelGGL((k_tile_round_pf<CONN, V>), dim3(g), dim3(64), 0, s, imgs,
                           n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, leave, clear, queued);
    else
        hipLaunchKernelGGL((k_tile_round<T, CONN, VR>), dim3(g), dim3(64), 0, s, imgs, n_tiles,
                           flags, lists, cin, cout, all, ctrl, round, max_iters, leave, clear, queued);
    return hipGetLastError();
}

template <typename T, int CONN>
static hipError_t tile_round_t(const Imgs &imgs, int64_t n_tiles, uint32_t *flags,
                               uint32_t *lists, const uint32_t *cin, uint32_t *cout, int all,
                               Ctrl *ctrl, uint32_t round, int max_iters, int grid,
                               hipStream_t s, int variant, uint32_t leave,
                               uint32_t *clear, uint32_t *queued) {
    switch (variant) {
    case 0: return tile_round_v<T, CONN, 0>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, leave, clear, queued);
    case 1: return tile_round_v<T, CONN, 1>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, leave, clear, queued);
    case 2: return tile_round_v<T, CONN, 2>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, leave, clear, queued);
    case 3: return tile_round_v<T, CONN, 3>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, leave, clear, queued);
    case 5: return tile_round_v<T, CONN, 5>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, leave, clear, queued);
    default: return tile_round_v<T, CONN, -1>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, leave, clear, queued);
    }
}

static hipError_t tile_round_any(int tbytes, int conn, const Imgs &imgs, int64_t n_tiles,
                                 uint32_t *flags, uint32_t *lists, const uint32_t *cin,
                                 uint32_t *cout, int all, Ctrl *ctrl, uint32_t round,
                                 int max_iters, int grid, hipStream_t s, int variant,
                                 uint32_t leave, uint32_t *clear, uint32_t *queued) {
    if (!ctrl) return hipErrorInvalidValue;
    if (tbytes == 1)
        return conn == 8 ? tile_round_t<uint8_t, 8>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, variant, leave, clear, queued)
                         : tile_round_t<uint8_t, 4>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, variant, leave, clear, queued);
    return conn == 8 ? tile_round_t<int32_t, 8>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, variant, leave, clear, queued)
                     : tile_round_t<int32_t, 4>(imgs, n_tiles, flags, lists, cin, cout, all, ctrl, round, max_iters, grid, s, variant, leave, clear, queued);
}

hipError_t launch_tile_round_ex(int tbytes, int conn, const Imgs &imgs, int64_t n_tiles,
                                uint32_t *flags, uint32_t *lists, const uint32_t *cin,
                                uint32_t *cout, uint32_t *clear, Ctrl *ctrl, uint32_t round,
                                int max_iters, int grid, hipStream_t s) {
    return tile_round_any(tbytes, conn, imgs, n_tiles, flags, lists, cin, cout, 0, ctrl, round,
                          max_iters, grid, s, -1, 0, clear, nullptr);
}

hipError_t launch_tile_round(int tbytes, int conn, const Imgs &imgs, int64_t n_tiles,
                             uint32_t *flags, uint32_t *lists, Ctrl *ctrl, uint32_t round,
                             int max_iters, int grid, hipStream_t s, int op_all, uint32_t leave,
                             uint32_t *queued) {
    // every image starts in round 1 here, so with one op for all of them the
    // visit is known for the whole launch
    const int variant = op_all < 0 ? -1 : ((op_all == MR_OP_FILL ? 2 : 0) | (round == 1 ? 1 : 0) |
                                           (round == 1 && imgs.lowered ? 4 : 0));
    // Round 1 visits every tile. Later int32 rounds may walk dense bands
    // (the lists of a sequence that starts at round 1 allow it): their
    // visits are bound by memory traffic, which the walk's order lowers.
    // uint8 visits are bound by issue and latency instead; there the walk
    // only adds visits (neighbours visited together see each other's halos
    // stale more often), so uint8 rounds keep the lists.
    return tile_round_any(tbytes, conn, imgs, n_tiles, flags, lists, ctrl->round_tiles[round],
                          ctrl->round_tiles[round + 1], round == 1 ? 1 : (tbytes == 4 ? 2 : 0), ctrl, round,
                          max_iters, grid, s, variant, leave, nullptr, queued);
}

template <typename T, int CONN, int V>
static hipError_t tile_queue_v(const Imgs &imgs, Ctrl *ctrl, uint32_t *state, uint32_t *ring,
                               uint64_t cap, int max_iters, int grid, unsigned long long wait_us,
                               hipStream_t s, uint32_t round, uint32_t from,
                               const uint32_t *lists, int64_t n_tiles) {
    hipLaunchKernelGGL((k_tile_queue<T, CONN, V>), dim3((unsigned)grid), dim3(64 * TQ_WAVES<T>), 0, s, imgs,
                       ctrl, state, ring, cap, max_iters, wait_us, round, from, lists, n_tiles);
    return hipGetLastError();
}
template <typename T, int CONN>
static hipError_t tile_queue_t(const Imgs &imgs, Ctrl *ctrl, uint32_t *state, uint32_t *ring,
                               uint64_t cap, int max_iters, int grid, unsigned long long wait_us,
                               hipStream_t s, int op_all, uint32_t round, uint32_t from,
                               const uint32_t *lists, int64_t n_tiles) {
    if (op_all == MR_OP_RECON)
        return tile_queue_v<T, CONN, 0>(imgs, ctrl, state, ring, cap, max_iters, grid, wait_us, s, round, from, lists, n_tiles);
    if (op_all == MR_OP_FILL)
        return tile_queue_v<T, CONN, 2>(imgs, ctrl, state, ring, cap, max_iters, grid, wait_us, s, round, from, lists, n_tiles);
    return tile_queue_v<T, CONN, -1>(imgs, ctrl, state, ring, cap, max_iters, grid, wait_us, s, round, from, lists, n_tiles);
}
hipError_t launch_tile_queue(int tbytes, int conn, const Imgs &imgs, int64_t n_tiles,
                             const uint32_t *lists, uint32_t round, Ctrl *ctrl, uint32_t *state,
                             uint32_t *ring, uint64_t cap, int max_iters, int grid,
                             unsigned long long wait_us, hipStream_t s, int op_all,
                             uint32_t leave, uint32_t from) {
    if (!ctrl || round > (uint32_t)MAX_ROUNDS + 1 || grid < 1 || n_tiles < 1)
        return hipErrorInvalidValue;
    // no more waves than tiles: a wave visits one tile at a time. uint8 launches
    // hold half the chip's: their lists are short (see tail_leave), and waves
    // without a tile only draw tickets and poll the ring (4096 x 4096 fill-holes
    // 310 us with 1024 waves, 327 us with 2048, erosion 633 and 645 us).
    if (tbytes == 1) grid = std::max(grid / 2, 1);
    const int wg = tbytes == 1 ? TQ_WAVES<uint8_t> : TQ_WAVES<int32_t>;
    grid = (int)((std::min<int64_t>(std::min<int64_t>(grid, RING_SLACK), n_tiles) + wg - 1) / wg);
    if (!from) {
        hipLaunchKernelGGL(k_tile_queue_mark, dim3(NBANDS), dim3(256), 0, s, lists, ctrl, n_tiles,
                           round, leave, state);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (tbytes == 1)
        return conn == 8 ? tile_queue_t<uint8_t, 8>(imgs, ctrl, state, ring, cap, max_iters, grid, wait_us, s, op_all, round, from, lists, n_tiles)
                         : tile_queue_t<uint8_t, 4>(imgs, ctrl, state, ring, cap, max_iters, grid, wait_us, s, op_all, round, from, lists, n_tiles);
    return conn == 8 ? tile_queue_t<int32_t, 8>(imgs, ctrl, state, ring, cap, max_iters, grid, wait_us, s, op_all, round, from, lists, n_tiles)
                     : tile_queue_t<int32_t, 4>(imgs, ctrl, state, ring, cap, max_iters, grid, wait_us, s, op_all, round, from, lists, n_tiles);
}

template <typename T, int CONN>
static hipError_t seed_t(const Imgs &imgs, int64_t n_tiles, const uint32_t *lists,
                         uint32_t round, Ctrl *ctrl, uint64_t *bitmap, uint32_t *qflag,
                         uint32_t *ring, uint64_t cap, int grid, hipStream_t s) {
    const int64_t want = std::max<int64_t>(NBANDS, (n_tiles + NBANDS - 1) / NBANDS * NBANDS);
    const unsigned g = (unsigned)(std::min<int64_t>(grid, want) / NBANDS * NBANDS);
    hipLaunchKernelGGL((k_seed<T, CONN>), dim3(g), dim3(64), 0, s, imgs, n_tiles, lists, round,
                       ctrl, bitmap, qflag, ring, cap);
    return hipGetLastError();
}

hipError_t launch_seed(int tbytes, int conn, const Imgs &imgs, int64_t n_tiles,
                       const uint32_t *lists, uint32_t round, Ctrl *ctrl, uint64_t *bitmap,
                       uint32_t *qflag, uint32_t *ring, uint64_t cap, int grid, hipStream_t s) {
    if (tbytes == 1)
        return conn == 8 ? seed_t<uint8_t, 8>(imgs, n_tiles, lists, round, ctrl, bitmap, qflag, ring, cap, grid, s)
                         : seed_t<uint8_t, 4>(imgs, n_tiles, lists, round, ctrl, bitmap, qflag, ring, cap, grid, s);
    return conn == 8 ? seed_t<int32_t, 8>(imgs, n_tiles, lists, round, ctrl, bitmap, qflag, ring, cap, grid, s)
                     : seed_t<int32_t, 4>(imgs, n_tiles, lists, round, ctrl, bitmap, qflag, ring, cap, grid, s);
}

__global__ void k_clear_u64(uint64_t *p, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

hipError_t launch_clear_u64(uint64_t *p, int64_t n, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, 8192);
    hipLaunchKernelGGL(k_clear_u64, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

template <typename T, int CONN>
static const void *queue_fn() {
    return (const void *)&k_queue<T, CONN>;
}

static const void *queue_kernel(int tbytes, int conn) {
    if (tbytes == 1) return conn == 8 ? queue_fn<uint8_t, 8>() : queue_fn<uint8_t, 4>();
    return conn == 8 ? queue_fn<int32_t, 8>() : queue_fn<int32_t, 4>();
}

int queue_max_blocks(int tbytes, int conn) {
    int per_cu = 0, dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, queue_kernel(tbytes, conn),
                                                     64 * QWAVES, 0) != hipSuccess)
        return 0;
    return per_cu * cus;
}

template <typename T, int CONN>
static hipError_t queue_t(const Imgs &imgs, Ctrl *ctrl, uint64_t *bitmap, uint32_t *qflag,
                          uint32_t *ring, uint64_t cap, int blocks, unsigned long long wait_us,
                          hipStream_t s) {
    hipLaunchKernelGGL((k_queue<T, CONN>), dim3((unsigned)blocks), dim3(64 * QWAVES), 0, s, imgs,
                       ctrl, bitmap, qflag, ring, cap, wait_us);
    return hipGetLastError();
}

hipError_t launch_queue(int tbytes, int conn, const Imgs &imgs, Ctrl *ctrl, uint64_t *bitmap,
                        uint32_t *qflag, uint32_t *ring, uint64_t cap, int blocks,
                        unsigned long long wait_us, hipStream_t s) {
    if (blocks < 1) return hipErrorInvalidValue;
    blocks = (int)std::min<int64_t>(blocks, RING_SLACK / QWAVES);
    if (tbytes == 1)
        return conn == 8 ? queue_t<uint8_t, 8>(imgs, ctrl, bitmap, qflag, ring, cap, blocks, wait_us, s)
                         : queue_t<uint8_t, 4>(imgs, ctrl, bitmap, qflag, ring, cap, blocks, wait_us, s);
    return conn == 8 ? queue_t<int32_t, 8>(imgs, ctrl, bitmap, qflag, ring, cap, blocks, wait_us, s)
                     : queue_t<int32_t, 4>(imgs, ctrl, bitmap, qflag, ring, cap, blocks, wait_us, s);
}

hipError_t launch_widen(const Imgs &imgs, int64_t n_tiles, bool to_wide, hipStream_t s) {
    for (int64_t t0 = 0; t0 < n_tiles; t0 += (int64_t)1 << 30) {
        const unsigned g = (unsigned)std::min<int64_t>(n_tiles - t0, (int64_t)1 << 30);
        if (to_wide)
            hipLaunchKernelGGL(k_widen<true>, dim3(g), dim3(64), 0, s, imgs, t0);
        else
            hipLaunchKernelGGL(k_widen<false>, dim3(g), dim3(64), 0, s, imgs, t0);
    }
    return hipGetLastError();
}

hipError_t launch_fill_output(int tbytes, const Imgs &imgs, int64_t n_tiles, hipStream_t s,
                              int64_t t0) {
    if (n_tiles <= 0) return hipSuccess;
    if (tbytes == 1)
        hipLaunchKernelGGL(k_fill_output<uint8_t>, dim3((unsigned)n_tiles), dim3(64), 0, s, imgs, t0);
    else
        hipLaunchKernelGGL(k_fill_output<int32_t>, dim3((unsigned)n_tiles), dim3(64), 0, s, imgs, t0);
    return hipGetLastError();
}

hipError_t launch_put_descs(ImgDesc *dst, const ImgDesc *v, int n, hipStream_t s) {
    for (int i = 0; i < n; i += DESC_CHUNK) {
        DescChunk c{};
        c.n = std::min(DESC_CHUNK, n - i);
        for (int k = 0; k < c.n; ++k) c.d[k] = v[i + k];
        hipLaunchKernelGGL(k_put_descs, dim3(1), dim3(DESC_CHUNK), 0, s, dst + i, c);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_store_u64(unsigned long long *p, unsigned long long v, hipStream_t s) {
    hipLaunchKernelGGL(k_store_u64, dim3(1), dim3(1), 0, s, p, v);
    return hipGetLastError();
}

} // namespace mr
