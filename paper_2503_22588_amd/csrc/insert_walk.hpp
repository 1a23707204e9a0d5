// insert_walk.hpp -- the walk of one depth pixel's ray through the map, as
// the mark pass of the depth-image insertion runs it (insert.hip).  Host and
// device code: a CPU build walks the same rays with every store checked.
#pragma once

#include "ray.hpp"

namespace nbt {

// Entries of the table of voxels marked lately (see insert.hip), and the
// table slot (a byte offset) of a voxel, both given as 4 * linear index.
constexpr uint32_t kSeen = 4096;
__host__ __device__ __forceinline__ uint32_t seen_slot(uint32_t lin4) {
    return (lin4 ^ (lin4 >> 13)) & (4u * kSeen - 4u);
}

// Steps left on each axis before the map's face, one field per axis under a
// guard bit that the step beyond the face clears (its borrow), so that
// leaving the map is one test of three bits.  Fields of 9 bits fit maps of up to
// 512 voxels per axis into 32 bits, larger ones (4096 at most) use 64.
template <class T>
struct StepsLeft {
    static constexpr int kBits = sizeof(T) == 4 ? 10 : 16;
    static constexpr T kGuard = (T)1 << (kBits - 1) | (T)1 << (2 * kBits - 1) | (T)1 << (3 * kBits - 1);
    T v;
    __host__ __device__ StepsLeft(int x, int y, int z)
        : v(((T)x | (T)y << kBits | (T)z << (2 * kBits)) | kGuard) {}
    static __host__ __device__ T unit(bool x, bool y) {
        return x ? (T)1 : y ? (T)1 << kBits : (T)1 << (2 * kBits);
    }
    __host__ __device__ bool take(T u) {         // false: the step leaves the map
        v -= u;
        return (~v & kGuard) == 0;
    }
};

// Walks pixel (i, j) of measured depth d and marks the voxels it passes
// (byte 2v) and its return's (byte 2v + 1).  Seen: read(lin4) and
// write(lin4) of the table's entry for a voxel, pin() between a read and the
// step's arithmetic.  Mark: called with the byte to set.
//
// The walk has two parts.  The crossing that leaves the map on an axis with n
// steps left lies at t + n dt but for the rounding of at most 4096 additions,
// 2^-12 of it; below 2^-10 short of the first such crossing no step needs a test for
// the map's face, and the loop steps with selects alone, four voxels a turn.
// The bound is strict, so a ray whose first crossing leaves the map at t = 0 (a
// camera exactly on a face, looking out: no steps left, so t + n dt = 0 and no
// margin) takes no step there; in the subnormal range, where the margin may
// round away, the additions are exact.  The rest of the ray, a few voxels, is walked with the test.
template <class T, class Seen, class Mark>
__host__ __device__ __forceinline__ void insert_walk(const DevMap& m, const CamParams& c, const float* pose_in,
                                                     float d, int i, int j, Seen&& seen, Mark&& mark) {
    if (!(d > 0.0f)) return;                 // no measurement (NaN included)
    const float s = d / c.range;
    const bool ret = s < 1.0f;               // a return within range

    // the pixel's segment O -> E in voxel units, as in setup_ray
    float u = 0.0f, v = 0.0f;
    if (c.W > 1) u = c.dh * ((float)(2 * i - (c.W - 1)) / (float)(c.W - 1));
    if (c.H > 1) v = c.dv * ((float)(2 * j - (c.H - 1)) / (float)(c.H - 1));
    const float org[3] = {m.ox, m.oy, m.oz};
    float O[3], D[3];
    bool finite = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        float w = pose_in[3 * a + 0] * u;
        w = w + pose_in[3 * a + 1] * v;
        w = w + pose_in[3 * a + 2] * c.range;
        const float t = pose_in[9 + a];
        const float e = t + w;
        O[a] = (t - org[a]) * m.inv_s;
        const float E = (e - org[a]) * m.inv_s;
        D[a] = E - O[a];
        finite = finite && __builtin_isfinite(O[a]) && __builtin_isfinite(E) && __builtin_isfinite(D[a]);
    }
    if (!finite) return;                     // an invalid ray updates nothing

    float t0 = 0.0f, t1 = 1.0f;
    float inv[3];
    bool par[3];
    const int n[3] = {m.nx, m.ny, m.nz};
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) inside = clip_axis(O[a], D[a], n[a], t0, t1, inv[a], par[a]) && inside;
    const bool hit_inside = ret && s <= t1;  // the return lies inside the map
    if (ret) t1 = sel_min(t1, s);
    if (!inside || t0 > t1) return;

    int ix, iy, iz, sx, sy, sz;
    float tx, ty, tz, dtx, dty, dtz;
    init_axis(O[0], D[0], t0, inv[0], par[0], n[0], ix, sx, tx, dtx);
    init_axis(O[1], D[1], t0, inv[1], par[1], n[1], iy, sy, ty, dty);
    init_axis(O[2], D[2], t0, inv[2], par[2], n[2], iz, sz, tz, dtz);

    // 4 * the linear index: the table's byte offset; the marks of a voxel are at half of it
    uint32_t lin4 = (((uint32_t)iz * (uint32_t)m.ny + (uint32_t)iy) * (uint32_t)m.nx + (uint32_t)ix) * 4u;
    const int dlx = 4 * sx, dly = 4 * sy * m.nx, dlz = 4 * sz * m.nx * m.ny;
    const int rx = sx > 0 ? m.nx - 1 - ix : ix, ry = sy > 0 ? m.ny - 1 - iy : iy, rz = sz > 0 ? m.nz - 1 - iz : iz;
    uint32_t prev = ~0u, prev_seen = ~0u;        // the previous voxel and its table entry
    auto check = [&] {
        if (prev_seen != prev) {
            seen.write(prev);
            mark(prev >> 1);
        }
    };

    // no step below this leaves the map (an axis the ray is parallel to gives inf or NaN: no limit)
    const float exit = fminf(fminf(tx + (float)rx * dtx, ty + (float)ry * dty), tz + (float)rz * dtz);
    const float safe = fminf(t1, exit * (1.0f - 0x1p-10f));
    bool go = true;
    while (go) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t now = seen.read(lin4);
            seen.pin();                          // the walk's arithmetic comes after the read
            check();
            const float tm = fminf(fminf(tx, ty), tz);
            go = tm < safe;
            const bool ex = tx == tm, ey = ty == tm;
            const bool bx = go && ex, by = go && !ex && ey, bz = go && !ex && !ey;
            prev = go ? lin4 : ~0u;
            prev_seen = go ? now : ~0u;
            lin4 += (uint32_t)(bx ? dlx : by ? dly : bz ? dlz : 0);
            tx = tx + (bx ? dtx : 0.0f);
            ty = ty + (by ? dty : 0.0f);
            tz = tz + (bz ? dtz : 0.0f);
        }
    }
    check();
    const uint32_t row = (lin4 >> 2) / (uint32_t)m.nx;
    ix = (int)((lin4 >> 2) - row * (uint32_t)m.nx);
    iz = (int)(row / (uint32_t)m.ny);
    iy = (int)(row - (uint32_t)iz * (uint32_t)m.ny);
    StepsLeft<T> left(sx > 0 ? m.nx - 1 - ix : ix, sy > 0 ? m.ny - 1 - iy : iy, sz > 0 ? m.nz - 1 - iz : iz);
    prev = prev_seen = ~0u;
    bool last;
    for (;;) {
        const uint32_t now = seen.read(lin4);
        const float tm = fminf(fminf(tx, ty), tz);
        last = tm > t1;
        check();
        prev = lin4;
        prev_seen = now;
        if (last) break;
        const bool ax = tx == tm;
        const bool ay = !ax && ty == tm;
        tx = tx + (ax ? dtx : 0.0f);
        ty = ty + (ay ? dty : 0.0f);
        tz = tz + (ax || ay ? 0.0f : dtz);
        lin4 += (uint32_t)(ax ? dlx : ay ? dly : dlz);
        if (!left.take(StepsLeft<T>::unit(ax, ay))) break;
    }
    // the ray's last voxel: the return's, or one it passed
    if (last && hit_inside) mark((prev >> 1) + 1u);
    else check();
}

}  // namespace nbt
