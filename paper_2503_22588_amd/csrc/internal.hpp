// internal.hpp -- types shared by the library's translation units (not installed).
#pragma once

#include <algorithm>
#include <atomic>

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nbt_ig.h"

namespace nbt {

// Encoded voxel word: the Eq. 2 gain of the voxel as float32 bits, with the
// sign bit set for Occupied voxels (their gain 1-P is still in the low 31
// bits).  The one-voxel border around the map holds kSentinel, the negative
// of the smallest denormal (2^-149): no gain takes it (1-P of an Occupied
// voxel is 0 or at least 2^-24), so a single signed test per step catches
// both "stop after this voxel" and "the walk left the map", and a walk that
// needs no visit count may add its magnitude instead of testing for it.
constexpr uint32_t kSentinel = 0x80000001u;
constexpr uint32_t kOccBit = 0x80000000u;
constexpr uint32_t kGainOne = 0x3F800000u;   // 1.0f: the gain of an Unknown voxel

// Storage order of the encoded words over the padded grid (X, Y, Z) =
// (x+1, y+1, z+1):
//   kLayoutLinear  x fastest: (Z*py + Y)*px + X;
//   column orders  T x T columns (T = 2, 4, 8): the x-y plane is cut into
//                  T x T tiles of T*T words (x fastest), each tile stores
//                  its layers z after z, and tiles go x fastest over the
//                  tile grid: ((Y/T*nbx + X/T)*pz + Z)*T*T + (Y%T)*T + X%T.
//                  For T = 4 a 128-B line holds a 4x4x2 block and four
//                  aligned layers a contiguous 4x4x4 block (256 B); a z step
//                  is always one layer.
// Padding of x and y up to whole tiles holds the sentinel as well.
constexpr int kLayoutLinear = NBT_IG_LAYOUT_LINEAR;

// log2 of the tile edge of a column order; 0 for the linear order.
__host__ __device__ inline int layout_tile_log2(int layout) {
    return layout == NBT_IG_LAYOUT_COLUMN2 ? 1
         : layout == NBT_IG_LAYOUT_COLUMN4 ? 2
         : layout == NBT_IG_LAYOUT_COLUMN8 ? 3 : 0;
}
// The storage order to keep of `count` timed ones: the fastest, but an order only
// takes the place of the current one when it is faster by the share `margin`.
inline int pick_layout(const float* ms, int count, int current, float margin) {
    int best = current;
    for (int l = 0; l < count; ++l)
        if (ms[l] < ms[best] && ms[l] < ms[current] * (1.0f - margin)) best = l;
    return best;
}
inline bool valid_layout(int layout) { return layout >= NBT_IG_LAYOUT_LINEAR && layout <= NBT_IG_LAYOUT_COLUMN8; }

constexpr int kCostWaves = 16;
// States of one workgroup of the planner's cost terms: whole horizons where one
// fits 64 lanes (the workgroup then also sums their cost), else 64 states.
inline uint32_t cost_tile(uint32_t steps) { return steps <= 64 ? 64 / steps * steps : 64; }
// Waves that split a tile's perspectives: 10 perspectives each at least, and
// no more than the chip holds at once (24 a CU), since every workgroup pays
// for its barriers and the sums' way through LDS.  16 waves for all: 1e6 x 1
// states against 1 x 10 128 us, one wave 16; 30,000 x 20 against 1 x 100 150, two 30; 10,000 x 100
// against 10 x 500 1557, two 1138.  In a large call one wave alone is slower
// with many perspectives (1223 there), two are within 5 % of the best.  A
// launch has less than 2^32 threads: 1.1e9 states in horizons of 33 are done
// by one wave a tile.
inline int query_waves(uint32_t tiles, uint32_t nb, uint32_t np, int cu_count) {
    const uint64_t pairs = (uint64_t)nb * np, cu = (uint64_t)cu_count;
    const uint64_t least = tiles >= 32u * cu ? 2u : 4u;
    const uint64_t most = std::min(pairs / 10u, std::max(24u * cu / tiles, least));
    int w = kCostWaves;
    while (w > 1 && ((uint64_t)w > most || (uint64_t)tiles * (uint64_t)w * 64u >= (1ull << 32))) w /= 2;
    return w;
}

// A map also holds one byte per voxel, its code: the index of its word in a
// palette of the map's distinct words (kCodes entries; 0 is the sentinel, 1
// Unknown, the others filled by the encoding, free ones hold kCodeFree).  The
// perspective walk gathers codes and looks the words up in LDS, so a cache
// line holds four times the voxels.  Words and codes say the same; a map with more
// distinct words than the palette takes has its overflow flag set (the word
// after the palette) and is walked by its words.
//
// The byte offset of a voxel is made of bit fields of X, Y and Z: x0 x1 y0 z0
// y1 z1 x2 y2 z2 from bit 0, then the rest of X, of Y and of Z (16 bytes hold
// a block of 4x2x2 voxels, a 128-byte line 8x4x4).  With the fields of the
// axes that a ray follows backwards complemented, every step of the ray adds
// one to its axis' field: ((g | ~mask) + 1) & mask within mask, the same four
// operations for each axis, where strides would need a test for the tile's
// face.
constexpr uint32_t kCodes = 256;
constexpr uint32_t kCodeFree = 0xFFFFFFFFu;
constexpr uint32_t kPaletteWords = kCodes + 2;       // with the overflow flag and the count

__host__ __device__ inline uint32_t code_offset(int sy, int sz, uint32_t X, uint32_t Y, uint32_t Z) {
    const uint32_t lo = (X & 3u) | (Y & 1u) << 2 | (Z & 1u) << 3 | (Y & 2u) << 3 | (Z & 2u) << 4 | (X & 4u) << 4 |
                        (Y & 4u) << 5 | (Z & 4u) << 6;
    return lo | (X >> 3) << 9 | (Y >> 3) << sy | (Z >> 3) << sz;
}

// Device view of an encoded map (passed to kernels by value).
struct DevMap {
    const uint32_t* enc;    // encoded words in `layout` order
    uint32_t bytes;         // size of enc in bytes (< 2^32)
    int nx, ny, nz;         // real dimensions
    int px, py, pz;         // padded dimensions (n + 2)
    int layout;             // NBT_IG_LAYOUT_*
    int tl;                 // log2 of the tile edge of a column order, 0 for the linear order
    int nbx, nby;           // tiles per axis over the padded x-y plane (column orders)
    float inv_s;            // 1/voxel_size (binary32)
    float ox, oy, oz;       // origin
    const uint8_t* codes;   // nullptr: the map has none
    const uint32_t* palette;    // kCodes words, then the overflow flag and the count of words
    uint32_t code_bytes;    // size of codes in bytes
    uint32_t mx, my, mz;    // offset bits of each axis
    int csy, csz;           // lowest offset bit of Y >> 3 and of Z >> 3
};

// Byte offset of voxel (x, y, z), real coordinates in [-1, n] (the border
// included), in either layout.
__host__ __device__ inline uint32_t voxel_offset(const DevMap& m, int x, int y, int z) {
    const uint32_t X = (uint32_t)(x + 1), Y = (uint32_t)(y + 1), Z = (uint32_t)(z + 1);
    if (m.tl == 0) return ((Z * (uint32_t)m.py + Y) * (uint32_t)m.px + X) * 4u;
    const uint32_t t = (uint32_t)m.tl, lo = (1u << t) - 1u;
    const uint32_t tile = (Y >> t) * (uint32_t)m.nbx + (X >> t);
    return (((tile * (uint32_t)m.pz + Z) << (2u * t)) + ((Y & lo) << t | (X & lo))) * 4u;
}

// Endpoint-grid parameters derived once per launch on the host.
struct CamParams {
    int W, H;
    float dh, dv;           // range * tan(fov/2), binary32
    float range;
};

// Per-perspective reduction slot used when several workgroups share one
// perspective: fixed-point sums are order-independent, so the result is
// bit-identical whatever order the workgroups finish in.  The last
// workgroup of a perspective reads and clears its slot.
struct VpAccum {
    unsigned long long sum_fx;     // sum of ray gains * fix_scale, rounded per workgroup
    unsigned long long steps;
    unsigned int count;            // workgroups done
    unsigned int invalid;
};
// The scale of those sums: the power of two that keeps the most a perspective
// can gather (1 a visit, nx + ny + nz + 3 visits a ray) below 2^63.  2^39 for
// 64x48 rays in a 1024^3 map, 2^27 at the largest sizes accepted, so rounding
// a workgroup's sum costs no more than 2^-28 of one Unknown voxel's gain (a
// fixed 2^24 lost whole digits of perspectives that see small gains only).
__host__ __device__ inline double fix_scale(const DevMap& m, const CamParams& c) {
    const unsigned long long most = (unsigned long long)c.W * (unsigned long long)c.H *
                                    (unsigned long long)(m.nx + m.ny + m.nz + 3);
    return (double)(1ull << (__builtin_clzll(most) - 1));
}

// Launch shape of the viewpoint kernel.
struct VpLaunch {
    int waves = 4;          // waves per workgroup (1, 2, 4, 8)
    int tile_w_log2 = 3;    // pixel tile of one wave: (1<<tile_w_log2) x (64>>tile_w_log2)
    int tiles_per_wave = 0; // tiles one wave walks per workgroup; 0 = balanced for the camera
    int xcd_remap = 0;      // 0, or runs of this many consecutive workgroups per XCD
    int depth = 8;          // gathers in flight per lane (1, 2, 4, 8)
    bool operator==(const VpLaunch& o) const {
        return waves == o.waves && tile_w_log2 == o.tile_w_log2 && tiles_per_wave == o.tiles_per_wave &&
               xcd_remap == o.xcd_remap && depth == o.depth;
    }
};

// Shape of a call whose rays are walked in segments (ig_segments_kernel).
struct SegLaunch {
    int segs_log2;          // segments per ray; -1: the rays are not split
    int rays_log2;          // rays of a workgroup; its threads are rays * segments
    int flat;               // rays dealt in row-major order, else in square-ish pixel tiles
    uint32_t blocks;        // blocks of 8 crossings per axis and ray that the LDS table holds
    uint32_t groups;        // workgroups per perspective
};

// Voxel box of one trajectory's frusta (its bitset positions: x fastest).
struct TrajBox {
    int lx, ly, lz;          // min corner (voxels)
    int ax, ay, az;          // extent (voxels)
    uint32_t nbits;          // ax*ay*az, 0 for an empty trajectory
    uint32_t pad;
};

// Scratch of trajectories whose rays are split over several workgroups: a
// bitset region per trajectory (kTrajSplitWords words dealt evenly) and this
// slot, both cleared by the box pre-pass of every call.
constexpr uint32_t kTrajSplitMost = 2048;            // trajectories of a split call
constexpr uint32_t kTrajSplitWords = 32u << 20;      // bitset words of all of them (128 MiB)
constexpr int kTrajParts = 64;                       // workgroups that sum up one trajectory at most
struct TrajAccum {
    unsigned long long visits;
    unsigned int invalid, count;                     // count: parts that have written theirs
    unsigned long long gain[kTrajParts];             // binary64 bits
    unsigned long long occ_free[kTrajParts];         // occupied | free << 32
    unsigned long long unknown[kTrajParts];
};

// How a call of T trajectories is split; groups == 1: one workgroup each.
struct TrajSplit {
    uint32_t groups;         // workgroups that share one trajectory's rays
    uint32_t leading;        // workgroups before them that take the boxes beyond cap_words, or 0
    uint32_t parts;          // workgroups that sum up its bitset
    uint32_t cap_words;      // bitset words per trajectory; a larger box is left to one workgroup
    uint32_t* bits;
    TrajAccum* acc;
};

// ---- launchers (each defined next to its kernels) ----

// Writes m's words (enc) and, when it has them, its codes.  A new map's palette is
// started from a sample of the grid, later ones are kept or started again.
enum class PaletteStart { kept, first, again };
hipError_t launch_encode_map(const float* prob, uint32_t* enc, const DevMap& m, float occ_thr,
                             float free_thr, unsigned int* bad_flag, PaletteStart start, hipStream_t s);
// Copies an encoded map into another storage order (dst laid out as dstm).
hipError_t launch_relayout(const DevMap& src, uint32_t* dst, const DevMap& dstm, hipStream_t s);

// trace != nullptr: the parity instance of the same kernel, which also writes
// one record per ray (trace[p * N_E + k]).
hipError_t launch_eval_viewpoints(const DevMap& m, const CamParams& c, const float* poses,
                                  uint32_t n, float* ig_out, unsigned long long* steps_out,
                                  VpAccum* ws, const VpLaunch& L, hipStream_t s,
                                  nbt_ig_ray_digest* trace = nullptr);

SegLaunch plan_segments(const DevMap& m, const CamParams& c, uint32_t n, int cu_count);
hipError_t launch_eval_segments(const DevMap& m, const CamParams& c, const float* poses, uint32_t n,
                                float* ig_out, unsigned long long* steps_out, VpAccum* ws, const SegLaunch& L,
                                hipStream_t s, nbt_ig_ray_digest* trace);

// Zeroes n per-perspective reduction slots (a fill kernel: no memset node
// when the caller captures the stream).
hipError_t launch_clear_slots(VpAccum* ws, uint32_t n, hipStream_t s);

hipError_t launch_trace_rays(const DevMap& m, const CamParams& c, const float* poses, uint32_t n,
                             nbt_ig_ray_digest* out, hipStream_t s);

hipError_t launch_trace_paths(const DevMap& m, const CamParams& c, const float* poses, uint32_t n,
                              const uint32_t* rays, uint32_t count, uint32_t max_len,
                              int32_t* lin_out, uint32_t* len_out, hipStream_t s);

hipError_t launch_traj_boxes(const DevMap& m, const CamParams& c, const float* poses, uint32_t T,
                             uint32_t L, TrajBox* boxes, const TrajSplit& split, hipStream_t s);

// Static LDS of the union kernel (its reductions); the bitset gets the rest.
size_t traj_static_lds_bytes();
// The timed union kernel of a workgroup size (4, 8, 16 waves), for occupancy queries.
const void* traj_union_kernel_ptr(int waves);

// One workgroup per trajectory, its bitset in LDS pass_words words at a time
// (boxes of more bits take several passes); trace != nullptr: the parity
// instance, one record per ray at trace[(t * L + l) * N_E + k].
hipError_t launch_traj_union(int waves, const DevMap& m, const CamParams& c, const float* poses, uint32_t L,
                             uint32_t T, uint32_t pass_words, const TrajBox* boxes, float* ig_union,
                             uint32_t* counts, unsigned long long* visits, nbt_ig_ray_digest* trace,
                             const TrajSplit& split, hipStream_t s);

// Kernel entry points of the persistent batched launch (for graph nodes).
// coded: some of the maps have codes.
const void* batch_kernel_ptr(int waves, int depth, bool count, bool coded);
const void* batch_reset_ptr();

hipError_t launch_eval_cost(const float* id_pos, const float* id_ig, uint32_t nb, uint32_t np, float p,
                            const float* poses, uint32_t h, uint32_t k, const float poi[3], float tan_h,
                            float tan_v, float w_i, float eps, float* g_out, float* o_out, float* cost,
                            int cu_count, hipStream_t s);

// Number of workgroups a perspective is split into for a launch shape.
// Raises a kernel's dynamic-LDS limit to `bytes` on the current device when
// above the 64 KiB default, once per (kernel, device, size) seen; `cache`
// is the caller's per-kernel record of the largest size set per device.
inline hipError_t allow_dynamic_lds(const void* kernel, size_t bytes, std::atomic<size_t>* cache, int ncache) {
    if (bytes <= 64 * 1024) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < ncache && cache[dev].load(std::memory_order_relaxed) >= bytes) return hipSuccess;
    e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e == hipSuccess && dev >= 0 && dev < ncache) {
        size_t cur = cache[dev].load(std::memory_order_relaxed);
        while (cur < bytes && !cache[dev].compare_exchange_weak(cur, bytes)) {
        }
    }
    return e;
}

inline uint32_t vp_tiles(const CamParams& c, int tile_w_log2) {
    const int tw = 1 << tile_w_log2, th = 64 >> tile_w_log2;
    return (uint32_t)((c.W + tw - 1) / tw) * (uint32_t)((c.H + th - 1) / th);
}

// tiles_per_wave == 0: as few workgroups as 16 tiles per wave allow, with the
// tiles dealt evenly over them (no wave of a small camera left idle, no short
// last workgroup on a large one); when n perspectives (n > 0) would give
// fewer than 64 workgroups per CU, each perspective is split further (down to
// one tile per wave): small calls then fill the chip, and rays of uneven
// length (views that hit an object next to views into open space) spread
// over many short workgroups instead of a few long ones.
inline VpLaunch resolve_launch(const CamParams& c, VpLaunch L, uint32_t n = 0, int cu_count = 0) {
    if (L.tiles_per_wave > 0) return L;
    const uint32_t tiles = vp_tiles(c, L.tile_w_log2);
    const uint32_t waves = (uint32_t)L.waves;
    uint32_t groups = (tiles + waves * 16 - 1) / (waves * 16);
    const uint64_t want = 64ull * (uint64_t)(cu_count > 0 ? cu_count : 0);
    if (n > 0 && (uint64_t)n * groups < want) {
        const uint32_t most = (tiles + waves - 1) / waves;
        const uint64_t g = (want + n - 1) / n;
        groups = (uint32_t)(g < most ? g : most);
        if (groups < 1) groups = 1;
    }
    const uint32_t tpw = (tiles + waves * groups - 1) / (waves * groups);
    L.tiles_per_wave = (int)(tpw > 0 ? tpw : 1);
    return L;
}

inline uint32_t vp_groups(const CamParams& c, const VpLaunch& L0, uint32_t n = 0, int cu_count = 0) {
    const VpLaunch L = resolve_launch(c, L0, n, cu_count);
    const uint32_t per = (uint32_t)(L.waves * L.tiles_per_wave);
    return (vp_tiles(c, L.tile_w_log2) + per - 1) / per;
}

}  // namespace nbt
