// ray.hpp -- per-lane ray generation and 3D-DDA state (device code).
//
// One lane owns one ray.  Set-up turns pixel (i, j) of a perspective into a
// voxel-unit segment O -> O + D clipped to the map (Sec. III, endpoint
// calculation), then into Amanatides-Woo traversal state.  Every operation
// is a single binary32 operation in a fixed order (the library is built
// with -ffp-contract=off, correctly rounded division and IEEE denormals), so
// the visited voxel sequence is a deterministic function of the inputs.
#pragma once

#include <type_traits>

#include "internal.hpp"

namespace nbt {

enum RayStatus : int { kRayOk = 0, kRayMiss = 1, kRayInvalid = 2 };

struct RayState {
    int ix, iy, iz;          // current voxel (real coordinates)
    int sx, sy, sz;          // step direction per axis (-1, 0, +1)
    float tx, ty, tz;        // parameter of the next face crossing per axis
    float dtx, dty, dtz;     // parameter distance between crossings per axis
    float t1;                // end of the clipped segment
};

__host__ __device__ __forceinline__ float sel_min(float a, float b) { return (b < a) ? b : a; }
__host__ __device__ __forceinline__ float sel_max(float a, float b) { return (b > a) ? b : a; }

// One axis of the slab clip.  Returns false when the ray runs parallel to
// this axis' faces outside the map.
__host__ __device__ __forceinline__ bool clip_axis(float O, float D, int n, float& t0, float& t1,
                                                   float& inv, bool& parallel) {
    parallel = fabsf(D) < 0x1p-100f;
    if (parallel) {
        inv = 0.0f;
        return (O >= 0.0f) && (O < (float)n);
    }
    inv = 1.0f / D;
    const float tA = (0.0f - O) * inv;
    const float tB = ((float)n - O) * inv;
    t0 = sel_max(t0, sel_min(tA, tB));
    t1 = sel_min(t1, sel_max(tA, tB));
    return true;
}

__host__ __device__ __forceinline__ void init_axis(float O, float D, float t0, float inv, bool parallel,
                                                   int n, int& idx, int& step, float& tmax, float& tdelta) {
    float f = floorf(O + t0 * D);
    f = sel_max(f, 0.0f);
    f = sel_min(f, (float)(n - 1));
    idx = (int)f;
    if (parallel) {
        step = 0;
        tmax = __builtin_inff();
        tdelta = __builtin_inff();
    } else {
        step = D > 0.0f ? 1 : -1;
        tdelta = fabsf(inv);
        tmax = ((float)(idx + (step > 0 ? 1 : 0)) - O) * inv;
    }
}

// Pixel of lane `lane` inside a (1 << tw_log2) x (64 >> tw_log2) tile: the
// lane bits are dealt alternately to x and y (x first) while both sides have
// bits left, so every aligned group of 4 lanes covers a 2 x 2 pixel block and
// every 16 lanes a 4 x 4 block (8 x 8 tiles).  Compact lane groups gather
// from fewer distinct cache lines than rows of 4 or 16 pixels.
__device__ __forceinline__ void tile_pixel(int lane, int tw_log2, int& lx, int& ly) {
    int x = 0, y = 0, bx = 0, by = 0;
    const int th_log2 = 6 - tw_log2;
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        const int bit = (lane >> b) & 1;
        const bool to_x = bx < tw_log2 && (by >= th_log2 || bx <= by);
        if (to_x) x |= bit << bx++;
        else y |= bit << by++;
    }
    lx = x;
    ly = y;
}

// pose: 12 floats (row-major R camera->world, then t).
__device__ __forceinline__ int setup_ray(const DevMap& m, const CamParams& c, const float* pose,
                                         int i, int j, RayState& r) {
    float u = 0.0f, v = 0.0f;
    if (c.W > 1) u = c.dh * ((float)(2 * i - (c.W - 1)) / (float)(c.W - 1));
    if (c.H > 1) v = c.dv * ((float)(2 * j - (c.H - 1)) / (float)(c.H - 1));

    const float org[3] = {m.ox, m.oy, m.oz};
    float O[3], D[3];
    bool finite = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float w = pose[3 * a + 0] * u;
        w = w + pose[3 * a + 1] * v;
        w = w + pose[3 * a + 2] * c.range;
        const float t = pose[9 + a];
        const float e = t + w;
        O[a] = (t - org[a]) * m.inv_s;
        const float E = (e - org[a]) * m.inv_s;
        D[a] = E - O[a];
        finite = finite && __builtin_isfinite(O[a]) && __builtin_isfinite(E) && __builtin_isfinite(D[a]);
    }
    if (!finite) return kRayInvalid;

    float t0 = 0.0f, t1 = 1.0f;
    float inv[3];
    bool par[3];
    const int n[3] = {m.nx, m.ny, m.nz};
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) inside = clip_axis(O[a], D[a], n[a], t0, t1, inv[a], par[a]) && inside;
    if (!inside || t0 > t1) return kRayMiss;

    init_axis(O[0], D[0], t0, inv[0], par[0], n[0], r.ix, r.sx, r.tx, r.dtx);
    init_axis(O[1], D[1], t0, inv[1], par[1], n[1], r.iy, r.sy, r.ty, r.dty);
    init_axis(O[2], D[2], t0, inv[2], par[2], n[2], r.iz, r.sz, r.tz, r.dtz);
    r.t1 = t1;
    return kRayOk;
}

// Buffer resource over the encoded grid: out-of-range offsets read 0 instead
// of faulting, which keeps any indexing mistake inside the map's allocation.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t map_rsrc(const DevMap& m) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)m.enc, (short)0, (int)m.bytes, 0x00020000);
}

__device__ __forceinline__ uint32_t load_word(__amdgpu_buffer_rsrc_t rs, uint32_t byte_off) {
    return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)byte_off, 0, 0);
}

__device__ __forceinline__ unsigned long long fnv1a_u32(unsigned long long h, uint32_t v) {
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        h ^= (unsigned long long)((v >> (8 * b)) & 0xFFu);
        h *= 0x100000001b3ULL;
    }
    return h;
}

constexpr unsigned long long kFnvBasis = 0xcbf29ce484222325ULL;

// Canonical linear index (z*ny + y)*nx + x of the voxel whose word sits at
// byte offset `off` of the encoded grid, in the map's storage order: the
// inverse of voxel_offset, written from the layout definitions rather than
// from the walk's per-axis deltas.  -1 for a border or padding word.
__device__ __forceinline__ int32_t offset_to_lin(const DevMap& m, uint32_t off) {
    const uint32_t w = off >> 2;
    uint32_t X, Y, Z;
    if (m.tl == 0) {
        X = w % (uint32_t)m.px;
        const uint32_t r = w / (uint32_t)m.px;
        Y = r % (uint32_t)m.py;
        Z = r / (uint32_t)m.py;
    } else {
        const uint32_t t = (uint32_t)m.tl, edge = 1u << t;
        const uint32_t in_tile = w & (edge * edge - 1u);
        const uint32_t r = w >> (2u * t);
        Z = r % (uint32_t)m.pz;
        const uint32_t tile = r / (uint32_t)m.pz;
        X = (tile % (uint32_t)m.nbx) * edge + (in_tile & (edge - 1u));
        Y = (tile / (uint32_t)m.nbx) * edge + (in_tile >> t);
    }
    const int x = (int)X - 1, y = (int)Y - 1, z = (int)Z - 1;
    if (x < 0 || y < 0 || z < 0 || x >= m.nx || y >= m.ny || z >= m.nz) return -1;
    return (z * m.ny + y) * m.nx + x;
}

// The same for the byte offset of a voxel's code (the inverse of code_offset).
__device__ __forceinline__ int32_t code_to_lin(const DevMap& m, uint32_t off) {
    const uint32_t X = (off & 3u) | (off >> 4 & 4u) | (off >> 9 & ((1u << (m.csy - 9)) - 1u)) << 3;
    const uint32_t Y = (off >> 2 & 1u) | (off >> 3 & 2u) | (off >> 5 & 4u) |
                       (off >> m.csy & ((1u << (m.csz - m.csy)) - 1u)) << 3;
    const uint32_t Z = (off >> 3 & 1u) | (off >> 4 & 2u) | (off >> 6 & 4u) | (off >> m.csz) << 3;
    const int x = (int)X - 1, y = (int)Y - 1, z = (int)Z - 1;
    if (x < 0 || y < 0 || z < 0 || x >= m.nx || y >= m.ny || z >= m.nz) return -1;
    return (z * m.ny + y) * m.nx + x;
}

// Parity mode of the throughput walks.  A walk instantiated with WalkTrace
// keeps, beside each gather in flight, the byte offset it was issued for and
// whether the generator was still inside the segment; every consumed visit
// is folded into the record from that offset (decoded by offset_to_lin), so
// the record shows the voxels the walk actually read, in its order.  Walks
// instantiated with NoTrace compile to the timed code.
struct NoTrace {};
struct WalkTrace {
    unsigned long long hash = kFnvBasis;   // FNV-1a-64 of the visited linear indices
    double gain = 0.0;                     // the visited words' gains, binary64 in visiting order
    uint32_t steps = 0;
    int32_t last = -1;                     // linear index of the last visit
    int reason = -1;                       // NBT_IG_RAY_*, -1 while walking
    uint32_t mismatch = 0;                 // union walk: visits whose bitset position names another voxel
    uint32_t box_bits = 0;                 // union walk: positions of the trajectory's box

    // slot consumed while the lane is still walking: word x read at `off`,
    // `live` = the generator had not passed the segment end when it issued it
    __device__ __forceinline__ void consume(const DevMap& m, uint32_t x, uint32_t off, bool live, float t1) {
        consume_at(x != kSentinel ? offset_to_lin(m, off) : -1, x, live, t1);
    }
    __device__ __forceinline__ void consume_at(int32_t lin, uint32_t x, bool live, float t1) {
        if (x != kSentinel) {
            hash = fnv1a_u32(hash, (uint32_t)lin);
            gain += (double)__uint_as_float(x & ~kOccBit);
            ++steps;
            last = lin;
        }
        if ((int)x < 0)
            reason = x != kSentinel ? NBT_IG_RAY_HIT
                   : live ? NBT_IG_RAY_EXIT : (t1 == 1.0f ? NBT_IG_RAY_END : NBT_IG_RAY_EXIT);
    }
    // end of the walk: a walk cut by its guard reports EXIT, as the reference walk does
    __device__ __forceinline__ void finish() {
        if (reason < 0) reason = NBT_IG_RAY_EXIT;
    }
};

template <class TR> constexpr bool traced() { return !std::is_same<TR, NoTrace>::value; }

// The parity record of one ray from its set-up status and walk record.
__device__ __forceinline__ void write_trace(nbt_ig_ray_digest* out, int status, const WalkTrace& rec) {
    nbt_ig_ray_digest d;
    d.hash = kFnvBasis;
    d.gain = 0.0;
    d.steps = 0;
    d.stop_lin = -1;
    d.reason = NBT_IG_RAY_MISS;
    d.reserved = 0;
    if (status == kRayInvalid) {
        d.reason = NBT_IG_RAY_INVALID;
        d.gain = __builtin_nan("");
    } else if (status == kRayOk) {
        d.hash = rec.hash;
        d.gain = rec.gain;
        d.steps = rec.steps;
        d.stop_lin = rec.last;
        d.reason = (uint32_t)rec.reason;
        d.reserved = rec.mismatch;
    }
    *out = d;
}

// Reason a walk stopped (matches NBT_IG_RAY_*).
enum WalkEnd : int { kEndHit = NBT_IG_RAY_HIT, kEndEnd = NBT_IG_RAY_END, kEndExit = NBT_IG_RAY_EXIT };

// Walks one ray.  Per visited voxel the encoded word is gathered and its gain
// added; the walk stops after an Occupied voxel, on the border sentinel (the
// previous voxel was the last), or when the next face crossing lies beyond
// the segment end.  The voxel coordinates are kept and addressed through
// voxel_offset (either layout); when TRACK is set visit(x, y, z, word) runs
// for every visited voxel.
template <bool TRACK, class Visit>
__device__ __forceinline__ int walk_ray(const DevMap& m, __amdgpu_buffer_rsrc_t rs, RayState& r,
                                        double& acc, uint32_t& steps, Visit&& visit) {
    const float dtx = r.dtx, dty = r.dty, dtz = r.dtz;
    float tx = r.tx, ty = r.ty, tz = r.tz;
    const float t1 = r.t1;
    const uint32_t guard = (uint32_t)(m.nx + m.ny + m.nz + 3);
    uint32_t n = 0;
    uint32_t bits;
    float tm;
    for (;;) {
        bits = load_word(rs, voxel_offset(m, r.ix, r.iy, r.iz));
        const bool sentinel = bits == kSentinel;
        const float g = sentinel ? 0.0f : __uint_as_float(bits & ~kOccBit);
        acc += (double)g;
        n += sentinel ? 0u : 1u;
        if constexpr (TRACK) {
            if (!sentinel) visit(r.ix, r.iy, r.iz, bits);
        }
        tm = fminf(fminf(tx, ty), tz);
        if ((int)bits < 0 || tm > t1 || n >= guard) break;
        const bool bx = (tx == tm);
        const bool by = !bx && (ty == tm);
        const bool bz = !bx && !by;
        const float nt = tm + (bx ? dtx : (by ? dty : dtz));
        tx = bx ? nt : tx;
        ty = by ? nt : ty;
        tz = bz ? nt : tz;
        r.ix += bx ? r.sx : 0;
        r.iy += by ? r.sy : 0;
        r.iz += bz ? r.sz : 0;
    }
    steps += n;
    if ((int)bits < 0) return bits == kSentinel ? kEndExit : kEndHit;
    if (tm > t1) return t1 == 1.0f ? kEndEnd : kEndExit;
    return kEndExit;
}

// Per-ray constants of the incremental map offset.  Linear layout: a step on
// axis a adds d[a] bytes.  Column orders (T x T tiles, T = 1 << TL): a z step
// adds dz (one layer of T*T words); an x or y step inside the tile adds dx or
// dy (the in-tile stride) and one across a tile face adds bigx or bigy.  The
// step crosses when the voxel's in-tile coordinate on that axis is T-1
// (forward) or 0 (backward), i.e. when ((off ^ flip) & mask) == 0, with the
// in-tile x and y in the fields tile_mask_x/y of the byte offset (TL bits
// each, from bit 2) and flip holding T-1 in the fields of the forward axes.
struct OffsetSteps {
    int dx, dy, dz;
    int bigx, bigy;
    uint32_t flip;
};

template <int TL> constexpr uint32_t tile_mask_x() { return ((1u << TL) - 1u) << 2; }
template <int TL> constexpr uint32_t tile_mask_y() { return ((1u << TL) - 1u) << (2 + TL); }

// TL: 0 for the linear order, else log2 of the column tile edge (m.tl).
template <int TL>
__device__ __forceinline__ OffsetSteps offset_steps(const DevMap& m, const RayState& r) {
    OffsetSteps o;
    if constexpr (TL == 0) {
        o.dx = r.sx * 4;
        o.dy = r.sy * m.px * 4;
        o.dz = r.sz * m.px * m.py * 4;
        o.bigx = o.bigy = 0;
        o.flip = 0;
    } else {
        constexpr int T = 1 << TL;
        constexpr int layer = 4 * T * T;       // bytes of one layer of a tile
        const int column = layer * m.pz;       // bytes of one tile's column
        o.dx = r.sx * 4;
        o.dy = r.sy * 4 * T;
        o.dz = r.sz * layer;
        o.bigx = r.sx * (column - 4 * (T - 1));
        o.bigy = r.sy * (column * m.nbx - 4 * T * (T - 1));
        o.flip = (r.sx > 0 ? tile_mask_x<TL>() : 0u) | (r.sy > 0 ? tile_mask_y<TL>() : 0u);
    }
    return o;
}

// One generator step of the pipelined walk: move to the next voxel unless
// the next face crossing lies beyond the segment end.  Past the end the
// generator points at offset 0, the sentinel word in the corner of the
// border (either layout), so every later gather reads "stop" without the
// loaded value ever being inspected here (which would force a wait for it).
//
// The three-way choice is made with the execution mask, as in code_step, and
// the lanes of x and of y alone test their tile's face: 17 VALU operations in
// column order, six of them compares or selects, where selects all through took 20,
// 13 of which issue at half rate.  A lane past the end keeps its t and
// so stays past it.  32 perspectives of 64x48 rays in a 64^3 map 16.0 -> 14.9 us,
// a batch of 64 maps 2.54 -> 2.50 ms, whose larger maps are walked by codes.
template <int TL>
__device__ __forceinline__ void dda_advance(float& tx, float& ty, float& tz, uint32_t& off,
                                            bool& alive, float t1, int dxo, int dyo, int dzo,
                                            int bxo, int byo, uint32_t flip,
                                            float dtx, float dty, float dtz) {
    float t;
    uint64_t all, a, b, past;
    if constexpr (TL == 0) {
        asm("v_min3_f32 %[t], %[tx], %[ty], %[tz]\n\t"
            "s_mov_b64 %[all], exec\n\t"
            "v_cmp_gt_f32_e64 %[past], %[t], %[t1]\n\t"
            "s_and_b64 exec, %[all], %[past]\n\t"
            "v_mov_b32_e32 %[off], 0\n\t"
            "s_andn2_b64 exec, %[all], %[past]\n\t"
            "s_mov_b64 %[b], exec\n\t"
            "v_cmpx_eq_f32_e64 %[a], %[tx], %[t]\n\t"          // the lanes that step on x
            "v_add_f32_e32 %[tx], %[tx], %[dtx]\n\t"
            "v_add_u32_e32 %[off], %[off], %[dxo]\n\t"
            "s_andn2_b64 exec, %[b], %[a]\n\t"
            "s_andn2_b64 %[b], %[b], %[a]\n\t"
            "v_cmpx_eq_f32_e64 %[a], %[ty], %[t]\n\t"          // of the others, those on y
            "v_add_f32_e32 %[ty], %[ty], %[dty]\n\t"
            "v_add_u32_e32 %[off], %[off], %[dyo]\n\t"
            "s_andn2_b64 exec, %[b], %[a]\n\t"                 // the rest on z
            "v_add_f32_e32 %[tz], %[tz], %[dtz]\n\t"
            "v_add_u32_e32 %[off], %[off], %[dzo]\n\t"
            "s_mov_b64 exec, %[all]\n\t"
            "s_nop 1"                                            // past may be read as a VALU operand next
            : [tx] "+v"(tx), [ty] "+v"(ty), [tz] "+v"(tz), [off] "+v"(off), [t] "=&v"(t), [all] "=&s"(all),
              [a] "=&s"(a), [b] "=&s"(b), [past] "=&s"(past)
            : [t1] "v"(t1), [dxo] "v"(dxo), [dyo] "v"(dyo), [dzo] "v"(dzo), [dtx] "v"(dtx), [dty] "v"(dty),
              [dtz] "v"(dtz)
            : "scc");
    } else {
        // x or y: the in-tile stride, or the tile-crossing delta at the tile
        // face; z: one layer.
        uint32_t d;
        uint64_t big;
        asm("v_min3_f32 %[t], %[tx], %[ty], %[tz]\n\t"
            "s_mov_b64 %[all], exec\n\t"
            "v_cmp_gt_f32_e64 %[past], %[t], %[t1]\n\t"
            "s_and_b64 exec, %[all], %[past]\n\t"
            "v_mov_b32_e32 %[off], 0\n\t"
            "s_andn2_b64 exec, %[all], %[past]\n\t"
            "s_mov_b64 %[b], exec\n\t"
            "v_cmpx_eq_f32_e64 %[a], %[tx], %[t]\n\t"
            "v_bitop3_b32 %[d], %[off], %[flip], %[mx] bitop3:0x28\n\t"      // (off ^ flip) & mask
            "v_cmp_eq_u32_e64 %[big], 0, %[d]\n\t"
            "v_add_f32_e32 %[tx], %[tx], %[dtx]\n\t"
            "s_nop 0\n\t"                                      // two states before `big` may be read
            "v_cndmask_b32_e64 %[d], %[dxo], %[bxo], %[big]\n\t"
            "v_add_u32_e32 %[off], %[off], %[d]\n\t"
            "s_andn2_b64 exec, %[b], %[a]\n\t"
            "s_andn2_b64 %[b], %[b], %[a]\n\t"
            "v_cmpx_eq_f32_e64 %[a], %[ty], %[t]\n\t"
            "v_bitop3_b32 %[d], %[off], %[flip], %[my] bitop3:0x28\n\t"
            "v_cmp_eq_u32_e64 %[big], 0, %[d]\n\t"
            "v_add_f32_e32 %[ty], %[ty], %[dty]\n\t"
            "s_nop 0\n\t"
            "v_cndmask_b32_e64 %[d], %[dyo], %[byo], %[big]\n\t"
            "v_add_u32_e32 %[off], %[off], %[d]\n\t"
            "s_andn2_b64 exec, %[b], %[a]\n\t"
            "v_add_f32_e32 %[tz], %[tz], %[dtz]\n\t"
            "v_add_u32_e32 %[off], %[off], %[dzo]\n\t"
            "s_mov_b64 exec, %[all]\n\t"
            "s_nop 1"
            : [tx] "+v"(tx), [ty] "+v"(ty), [tz] "+v"(tz), [off] "+v"(off), [t] "=&v"(t), [d] "=&v"(d),
              [all] "=&s"(all), [a] "=&s"(a), [b] "=&s"(b), [past] "=&s"(past), [big] "=&s"(big)
            : [t1] "v"(t1), [dxo] "v"(dxo), [bxo] "v"(bxo), [dyo] "v"(dyo), [byo] "v"(byo), [dzo] "v"(dzo),
              [flip] "v"(flip), [mx] "s"(tile_mask_x<TL>()), [my] "s"(tile_mask_y<TL>()), [dtx] "v"(dtx),
              [dty] "v"(dty), [dtz] "v"(dtz)
            : "scc");
    }
    alive = !__builtin_amdgcn_inverse_ballot_w64(past);
}

// Software-pipelined walk for the throughput kernels.  The voxel sequence of
// a ray depends only on its geometry, never on the map contents, so a
// generator runs P-1 voxels ahead of the consumer and keeps P gathers in
// flight per lane; the consumer adds gains in visiting order and stops at
// the first Occupied word or at a sentinel (the border, or the corner word
// the generator reads once the segment has ended).  Visits, gains and their
// order are exactly those of walk_ray (the sum is rounded differently, see
// below); only the reason is not reported, and the visit count only when
// COUNT is set.  Gathers past a stop are never
// consumed (and out-of-range ones read 0).  TL selects the map order (see offset_steps).
constexpr uint32_t kRunSlots = 8;

template <int P, bool COUNT, int TL, class TR = NoTrace>
__device__ __forceinline__ void walk_ray_pipelined(const DevMap& m, __amdgpu_buffer_rsrc_t rs,
                                                   const RayState& r, double& acc, uint32_t& steps,
                                                   TR* tr = nullptr) {
    static_assert(P == 2 || P == 4 || P == 8, "pipeline depth");
    const OffsetSteps o = offset_steps<TL>(m, r);
    const float dtx = r.dtx, dty = r.dty, dtz = r.dtz;
    const float t1 = r.t1;
    uint32_t off = voxel_offset(m, r.ix, r.iy, r.iz);
    float tx = r.tx, ty = r.ty, tz = r.tz;
    bool alive = true;     // the generator has not yet passed the segment end

    uint32_t w[P];
    // parity mode only: the offset of each gather in flight and whether the
    // generator was inside the segment when it issued it
    [[maybe_unused]] uint32_t wo[P];
    [[maybe_unused]] bool wl[P];
    w[0] = load_word(rs, off);
    if constexpr (traced<TR>()) {
        wo[0] = off;
        wl[0] = true;
    }
#pragma unroll
    for (int u = 1; u < P; ++u) {
        dda_advance<TL>(tx, ty, tz, off, alive, t1, o.dx, o.dy, o.dz, o.bigx, o.bigy, o.flip,
                           dtx, dty, dtz);
        w[u] = load_word(rs, off);
        if constexpr (traced<TR>()) {
            wo[u] = off;
            wl[u] = alive;
        }
    }
    uint32_t n = 0;
    // Every axis index moves one way only, so the border is reached within
    // nx + ny + nz steps; the group budget only guards that argument.
    uint32_t budget = (uint32_t)(m.nx + m.ny + m.nz + 3) / P + 2;
    bool run = true;
    // Gains are summed in binary32 over runs of kRunSlots consecutive slots and
    // each run's sum is added to the double accumulator.  The runs start at
    // fixed slot indices whatever P is, so every depth gives the same bits; a
    // sum of 8 non-negative terms is off by at most 7 units of 2^-24 relative.
    float part = 0.0f;
    uint32_t group = 0;
    // Lanes leave the loop between groups of P slots; inside a group every slot
    // runs for every lane still in the loop, with a lane that has stopped adding
    // nothing.  No slot is conditional, so slot u's word lives in one register
    // across iterations and each read waits only for its own gather (the P - 1
    // issued after it stay in flight).  A stopped lane issues at most P - 1
    // spare gathers before it leaves.
    while (run) {
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const uint32_t x = w[u];
            // a voxel visit, not the sentinel.  The IG-only walk skips the test:
            // the sentinel then adds its magnitude 2^-149, at most once per ray
            // (it stops the walk), so a ray sum and the IG are off by at most
            // 2^-149 absolute.
            const bool take = COUNT ? (run && x != kSentinel) : run;
            // the empty asm keeps each slot's read ahead of its refill (else the
            // reads sink to the end of the group and the refills need copies)
            uint32_t xs = take ? x : 0u;
            asm volatile("" : "+v"(xs));
            part += fabsf(__uint_as_float(xs));
            if constexpr (COUNT) n += take ? 1u : 0u;
            if constexpr (traced<TR>()) {
                if (run) tr->consume(m, x, wo[u], wl[u], t1);
            }
            run = run && (int)x >= 0;
            dda_advance<TL>(tx, ty, tz, off, alive, t1, o.dx, o.dy, o.dz, o.bigx, o.bigy, o.flip,
                               dtx, dty, dtz);
            w[u] = load_word(rs, off);
            if constexpr (traced<TR>()) {
                wo[u] = off;
                wl[u] = alive;
            }
        }
        if ((++group & (kRunSlots / P - 1)) == 0u) {
            acc += (double)part;
            part = 0.0f;
        }
        run = run && --budget != 0u;
    }
    acc += (double)part;
    if constexpr (COUNT) steps += n;
    if constexpr (traced<TR>()) tr->finish();
}

// One generator step of the code walk, for the lanes that execute it: past
// gets the lanes whose next crossing lies beyond their segment's end t1; they
// stay where they are.  The others step on the axis of that crossing (ties to
// the lower axis): its t gains dt and its field of the offset g one.
//
// Compares and selects on lane masks issue at about half the rate of additions and
// moves, so the three-way choice is made with the execution mask instead: the
// lanes of one axis add their dt and fetch the axis' mask, then the next
// axis' do.  The mask is what it was at the end.  17 VALU operations per
// voxel with the sum and the palette; selects took 24 by words.
__device__ __forceinline__ void code_step(float& tx, float& ty, float& tz, uint32_t& g, uint64_t& past, float t1,
                                          uint32_t mx, uint32_t my, uint32_t mz, float dtx, float dty, float dtz) {
    uint32_t mask, t;
    uint64_t all, a, b;
    asm("v_min3_f32 %[t], %[tx], %[ty], %[tz]\n\t"
        "s_mov_b64 %[all], exec\n\t"
        "v_cmp_gt_f32_e64 %[past], %[t], %[t1]\n\t"
        "s_andn2_b64 exec, %[all], %[past]\n\t"
        "s_mov_b64 %[b], exec\n\t"
        "v_mov_b32_e32 %[mask], %[mz]\n\t"
        "v_cmpx_eq_f32_e64 %[a], %[tx], %[t]\n\t"          // the lanes that step on x
        "v_add_f32_e32 %[tx], %[tx], %[dtx]\n\t"
        "v_mov_b32_e32 %[mask], %[mx]\n\t"
        "s_andn2_b64 exec, %[b], %[a]\n\t"
        "s_andn2_b64 %[b], %[b], %[a]\n\t"
        "v_cmpx_eq_f32_e64 %[a], %[ty], %[t]\n\t"          // of the others, those on y
        "v_add_f32_e32 %[ty], %[ty], %[dty]\n\t"
        "v_mov_b32_e32 %[mask], %[my]\n\t"
        "s_andn2_b64 exec, %[b], %[a]\n\t"                 // the rest on z
        "v_add_f32_e32 %[tz], %[tz], %[dtz]\n\t"
        "s_andn2_b64 exec, %[all], %[past]\n\t"
        "v_bitop3_b32 %[t], %[g], %[mask], %[g] bitop3:0xf3\n\t"   // g | ~mask
        "v_add_u32_e32 %[t], 1, %[t]\n\t"
        "v_bfi_b32 %[g], %[mask], %[t], %[g]\n\t"
        "s_mov_b64 exec, %[all]"
        : [tx] "+v"(tx), [ty] "+v"(ty), [tz] "+v"(tz), [g] "+v"(g), [mask] "=&v"(mask), [t] "=&v"(t),
          [all] "=&s"(all), [a] "=&s"(a), [b] "=&s"(b), [past] "=&s"(past)
        : [t1] "v"(t1), [mx] "s"(mx), [my] "s"(my), [mz] "s"(mz), [dtx] "v"(dtx), [dty] "v"(dty), [dtz] "v"(dtz)
        : "scc");
}

// The walk over a map's codes, software-pipelined as walk_ray_pipelined at
// depth 8: the same visits, the same gains in the same order and runs, the same
// 2^-149 where the IG-only walk meets the border.  pal: the map's palette in
// LDS.  A code is looked up one slot before its word is used.
//
// The walk covers one stretch of a ray: from the state in `r`, which is that of
// slot index K of the ray, it passes `skip` slots without visiting them and
// then visits `groups` groups of kRunSlots slots, fewer when the ray ends (a
// whole ray: K = skip = 0, and more groups than the map has voxels in a row).
// K + skip is a multiple of kRunSlots, so the runs summed in binary32 are
// those of the whole walk.  Returns whether the ray ended here: an Occupied
// voxel, the border or the segment's end.
template <bool COUNT, class TR = NoTrace>
__device__ __forceinline__ bool walk_ray_codes(const DevMap& m, const uint32_t* pal, const RayState& r, uint32_t skip,
                                               uint32_t groups, double& acc, uint32_t& steps, TR* tr = nullptr) {
    constexpr int P = kRunSlots;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)m.codes, (short)0, (int)m.code_bytes, 0x00020000);
    const float dtx = r.dtx, dty = r.dty, dtz = r.dtz, t1 = r.t1;
    const uint32_t mx = m.mx, my = m.my, mz = m.mz;
    const uint32_t flip = (r.sx < 0 ? mx : 0u) | (r.sy < 0 ? my : 0u) | (r.sz < 0 ? mz : 0u);
    uint32_t g = code_offset(m.csy, m.csz, (uint32_t)(r.ix + 1), (uint32_t)(r.iy + 1), (uint32_t)(r.iz + 1)) ^ flip;
    float tx = r.tx, ty = r.ty, tz = r.tz;
    auto load = [&] { return (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rs, (int)(g ^ flip), 0, 0); };
    bool refused = false;                        // the last slot passed already lay past the segment's end
    for (; skip > 0; --skip) {
        uint64_t ended;
        code_step(tx, ty, tz, g, ended, t1, mx, my, mz, dtx, dty, dtz);
        refused = __builtin_amdgcn_inverse_ballot_w64(ended);
    }

    uint32_t w[P];
    uint64_t past[P];                            // per slot: lanes that had left their segment when it was issued
    [[maybe_unused]] uint32_t wo[P];
    w[0] = load();
    past[0] = __ballot(refused);
    if constexpr (traced<TR>()) wo[0] = g ^ flip;
#pragma unroll
    for (int u = 1; u < P; ++u) {
        code_step(tx, ty, tz, g, past[u], t1, mx, my, mz, dtx, dty, dtz);
        w[u] = load();
        if constexpr (traced<TR>()) wo[u] = g ^ flip;
    }
    // the opaque zero keeps the codes 32 bits wide across the loop (else every
    // group begins by waiting for its last gather to widen them)
    uint32_t zero = 0;
    asm volatile("" : "+s"(zero));
#pragma unroll
    for (int u = 0; u < P; ++u) w[u] += zero;

    uint32_t n = 0;
    uint64_t live = __ballot(true);              // lanes still walking
    bool run = groups != 0u;
    bool over = false;
    uint32_t next = pal[w[0]];
    while (run) {
        float part = 0.0f;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const uint32_t x = next;
            const uint64_t gone = past[u];
            [[maybe_unused]] uint32_t at;
            if constexpr (traced<TR>()) at = wo[u];
            code_step(tx, ty, tz, g, past[u], t1, mx, my, mz, dtx, dty, dtz);
            w[u] = load();
            if constexpr (traced<TR>()) wo[u] = g ^ flip;
            next = pal[w[(u + 1) % P]];
            if constexpr (traced<TR>()) {
                if (__builtin_amdgcn_inverse_ballot_w64(live)) {
                    const bool in = !__builtin_amdgcn_inverse_ballot_w64(gone);
                    tr->consume_at(in && x != kSentinel ? code_to_lin(m, at) : -1, in ? x : kSentinel, in, t1);
                }
            }
            // lanes past their segment's end stop; the others add the gain and
            // stop at a set sign
            uint64_t all, took;
            asm volatile(
                "s_mov_b64 %[all], exec\n\t"
                "s_andn2_b64 %[took], %[live], %[gone]\n\t"
                "s_and_b64 exec, %[all], %[took]\n\t"
                "v_add_f32_e64 %[part], %[part], |%[x]|\n\t"
                "v_cmpx_le_i32_e64 %[live], 0, %[x]\n\t"
                "s_mov_b64 exec, %[all]\n\t"
                "s_nop 1"                        // the new mask may be read as a VALU operand next
                : [part] "+v"(part), [live] "+s"(live), [all] "=&s"(all), [took] "=&s"(took)
                : [gone] "s"(gone), [x] "v"(x)
                : "scc");
            if constexpr (COUNT) n += __builtin_amdgcn_inverse_ballot_w64(took) && x != kSentinel ? 1u : 0u;
        }
        acc += (double)part;
        over = !__builtin_amdgcn_inverse_ballot_w64(live);
        run = !over && --groups != 0u;
    }
    if constexpr (COUNT) steps += n;
    return over;
}

// walk_ray_pipelined over one stretch of a ray: starting at the state in `r`,
// which is that of slot index K of the ray, it passes `skip` slots without
// visiting them and then visits `groups` groups of kRunSlots slots (fewer
// when the ray ends).  K + skip is a multiple of kRunSlots, so the runs that
// are summed in binary32 are those of the whole walk.  Returns whether the
// ray ended here: an Occupied voxel, the border or the segment's end.
template <bool COUNT, int TL, class TR = NoTrace>
__device__ __forceinline__ bool walk_ray_stretch(const DevMap& m, __amdgpu_buffer_rsrc_t rs, const RayState& r,
                                                 uint32_t skip, uint32_t groups, double& acc, uint32_t& steps,
                                                 TR* tr = nullptr) {
    constexpr int P = kRunSlots;
    const OffsetSteps o = offset_steps<TL>(m, r);
    const float dtx = r.dtx, dty = r.dty, dtz = r.dtz;
    const float t1 = r.t1;
    uint32_t off = voxel_offset(m, r.ix, r.iy, r.iz);
    float tx = r.tx, ty = r.ty, tz = r.tz;
    bool alive = true;
    auto advance = [&] {
        dda_advance<TL>(tx, ty, tz, off, alive, t1, o.dx, o.dy, o.dz, o.bigx, o.bigy, o.flip, dtx, dty, dtz);
    };
    for (; skip > 0; --skip) advance();

    uint32_t w[P];
    [[maybe_unused]] uint32_t wo[P];
    [[maybe_unused]] bool wl[P];
#pragma unroll
    for (int u = 0; u < P; ++u) {
        if (u > 0) advance();
        w[u] = load_word(rs, off);
        if constexpr (traced<TR>()) {
            wo[u] = off;
            wl[u] = alive;
        }
    }
    uint32_t n = 0;
    bool run = groups != 0u;
    bool over = false;
    while (run) {
        float part = 0.0f;
#pragma unroll
        for (int u = 0; u < P; ++u) {
            const uint32_t x = w[u];
            const bool take = run && x != kSentinel;
            uint32_t xs = take ? x : 0u;
            asm volatile("" : "+v"(xs));          // as in walk_ray_pipelined
            part += fabsf(__uint_as_float(xs));
            if constexpr (COUNT) n += take ? 1u : 0u;
            if constexpr (traced<TR>()) {
                if (run) tr->consume(m, x, wo[u], wl[u], t1);
            }
            run = run && (int)x >= 0;
            advance();
            w[u] = load_word(rs, off);
            if constexpr (traced<TR>()) {
                wo[u] = off;
                wl[u] = alive;
            }
        }
        acc += (double)part;
        over = !run;
        run = run && --groups != 0u;
    }
    if constexpr (COUNT) steps += n;
    return over;
}

}  // namespace nbt
