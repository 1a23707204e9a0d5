// insert.hip -- map update by depth-image insertion (clamped log-odds occupancy update).
//
// The step before IG evaluation: the map is built from the camera's point
// clouds (Sec. II-III; the paper leaves the update to its occupancy-mapping
// library and gives no formulas).  Per scan (a pose and a W x H z-depth
// image):
//   - the return of pixel (i, j) lies on that pixel's endpoint ray (Sec. III,
//     endpoint calculation; the endpoint sits at z-depth d_Cam) at segment
//     parameter s = depth / d_Cam;
//   - depth NaN or <= 0: no measurement; s >= 1: no return within range, the
//     whole segment is carved free;
//   - the walk is the ray walk of the IG kernels (same set-up and stepping,
//     ties to the lower axis) ending at min(t1, s) and not stopping at
//     occupied voxels; its last voxel is hit when the return lies inside the
//     map, every other voxel it visits is free;
//   - each voxel marked in the scan moves once: log-odds + l_hit if any ray
//     hit it, else + l_miss, then clamped to [l_min, l_max] (binary32).
// Scans are applied in order.  Two passes per scan: a mark pass (one thread
// per pixel; two mark bytes per voxel, pass and return, each set by a plain
// byte store) and an apply pass (one thread per 8 voxels: it reads their
// marks, updates the marked log-odds values and clears the marks for the next
// scan; the last scan's also writes the probabilities when they are wanted).
#include "host.hpp"
#include "ray.hpp"

namespace nbt {

// Two mark bytes per voxel, set by plain byte stores (a byte store touches
// no neighbouring byte, and any number of rays may store the same 1):
// byte 2v says a ray passed voxel v, byte 2v + 1 that a ray's return lies in it.
// A voxel is visited by many rays of a scan (640x576 pixels into 2 cm voxels:
// some 74 M visits of 2 M voxels), so storing on every visit is bound by the
// address path.  A workgroup's 16x16 pixels meet the same voxels at nearly
// the same time: it keeps the voxels it has marked lately in a direct-mapped
// LDS table and stores only where the table shows another one.  An entry is
// written together with its voxel's store, so a hit always stands for a store
// that this workgroup makes; lanes and waves racing for an entry only repeat
// stores.  The table's answer for one voxel is looked at after the next
// one's read, which keeps its latency off the walk.
//
// The walk has two parts.  The crossing that leaves the map on an axis with n
// steps left lies at t + n dt but for the rounding of at most 4096 additions,
// 2^-12 of it; up to 2^-10 short of the first such crossing no step needs a test for
// the map's face, and the loop steps with selects alone, four voxels a turn.
// The rest of the ray, a few voxels, is walked with the test.
// 640x576 into 256^3 at 2 cm: 216 us a scan with a store on every visit, 70 now.
constexpr uint32_t kSeen = 4096;

// Table slot (a byte offset) of a voxel, both given as 4 * linear index.
__device__ __forceinline__ uint32_t seen_slot(uint32_t lin4) { return (lin4 ^ (lin4 >> 13)) & (4u * kSeen - 4u); }

// Steps left on each axis before the map's face, one field per axis under a
// guard bit that the step beyond the face clears (its borrow), so that
// leaving the map is one test of three bits.  Fields of 9 bits fit maps of up to
// 512 voxels per axis into 32 bits, larger ones (4096 at most) use 64.
template <class T>
struct StepsLeft {
    static constexpr int kBits = sizeof(T) == 4 ? 10 : 16;
    static constexpr T kGuard = (T)1 << (kBits - 1) | (T)1 << (2 * kBits - 1) | (T)1 << (3 * kBits - 1);
    T v;
    __device__ StepsLeft(int x, int y, int z)
        : v(((T)x | (T)y << kBits | (T)z << (2 * kBits)) | kGuard) {}
    static __device__ T unit(bool x, bool y) { return x ? (T)1 : y ? (T)1 << kBits : (T)1 << (2 * kBits); }
    __device__ bool take(T u) {                  // false: the step leaves the map
        v -= u;
        return (~v & kGuard) == 0;
    }
};

template <class T>
__global__ __launch_bounds__(256) void insert_mark_kernel(DevMap m, CamParams c,
                                                          const float* __restrict__ pose_in,
                                                          const float* __restrict__ depth,
                                                          uint8_t* __restrict__ marks) {
    __shared__ uint32_t s_seen[kSeen];
    for (uint32_t k = threadIdx.x; k < kSeen; k += 256u) s_seen[k] = ~0u;
    __syncthreads();
    // 16x16 pixels: four 8x8 tiles, one per wave
    const uint32_t wave = threadIdx.x >> 6, tiles_x = ((uint32_t)c.W + 15u) / 16u;
    int lx, ly;
    tile_pixel((int)(threadIdx.x & 63u), 3, lx, ly);
    const int i = (int)(blockIdx.x % tiles_x * 16u + (wave & 1u) * 8u) + lx;
    const int j = (int)(blockIdx.x / tiles_x * 16u + (wave >> 1) * 8u) + ly;
    if (i >= c.W || j >= c.H) return;
    const float d = depth[(size_t)j * (size_t)c.W + (size_t)i];
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
    unsigned char* seen = reinterpret_cast<unsigned char*>(s_seen);
    uint32_t prev = ~0u, prev_seen = ~0u;        // the previous voxel and its table entry
    auto check = [&] {
        if (prev_seen != prev) {
            *reinterpret_cast<uint32_t*>(seen + seen_slot(prev)) = prev;
            marks[prev >> 1] = 1;
        }
    };

    // no step up to here leaves the map (an axis the ray is parallel to gives inf or NaN: no limit)
    const float exit = fminf(fminf(tx + (float)rx * dtx, ty + (float)ry * dty), tz + (float)rz * dtz);
    const float safe = fminf(t1, exit * (1.0f - 0x1p-10f));
    bool go = true;
    while (go) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t now = *reinterpret_cast<const uint32_t*>(seen + seen_slot(lin4));
            __builtin_amdgcn_sched_barrier(0);   // the walk's arithmetic comes after the read
            check();
            const float tm = fminf(fminf(tx, ty), tz);
            go = tm <= safe;
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
        const uint32_t now = *reinterpret_cast<const uint32_t*>(seen + seen_slot(lin4));
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
    if (last && hit_inside) marks[(prev >> 1) + 1u] = 1;
    else check();
}

// One thread per 8 voxels (16 bytes of marks, 32 of values).  PROB: also the
// probability of every voxel.  vec: all three arrays are 16-byte aligned.
template <bool PROB>
__global__ __launch_bounds__(256) void insert_apply_kernel(uint32_t* __restrict__ marks,
                                                           float* __restrict__ L, float* __restrict__ P,
                                                           uint64_t nvox, nbt_ig_insert_params p, bool vec) {
    const uint64_t v0 = 8 * ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x);
    if (v0 >= nvox) return;
    auto moved = [&](float l, uint32_t mk) {     // mk: the voxel's (pass, return) bytes
        if (mk == 0u) return l;
        l = l + ((mk & 0xFF00u) ? p.l_hit : p.l_miss);
        l = (p.l_min > l) ? p.l_min : l;
        return (p.l_max < l) ? p.l_max : l;
    };
    auto prob = [](float l) { return 1.0f / (1.0f + expf(-l)); };
    if (vec && v0 + 8 <= nvox) {
        uint4* mv = reinterpret_cast<uint4*>(marks + v0 / 2);
        const uint4 mk = *mv;
        const bool any = (mk.x | mk.y | mk.z | mk.w) != 0u;
        if (!PROB && !any) return;
        float4* lv = reinterpret_cast<float4*>(L + v0);
        float4 a = lv[0], b = lv[1];
        if (any) {
            *mv = make_uint4(0u, 0u, 0u, 0u);
            a.x = moved(a.x, mk.x & 0xFFFFu);
            a.y = moved(a.y, mk.x >> 16);
            a.z = moved(a.z, mk.y & 0xFFFFu);
            a.w = moved(a.w, mk.y >> 16);
            b.x = moved(b.x, mk.z & 0xFFFFu);
            b.y = moved(b.y, mk.z >> 16);
            b.z = moved(b.z, mk.w & 0xFFFFu);
            b.w = moved(b.w, mk.w >> 16);
            lv[0] = a;
            lv[1] = b;
        }
        if constexpr (PROB) {
            float4* pv = reinterpret_cast<float4*>(P + v0);
            pv[0] = make_float4(prob(a.x), prob(a.y), prob(a.z), prob(a.w));
            pv[1] = make_float4(prob(b.x), prob(b.y), prob(b.z), prob(b.w));
        }
        return;
    }
    for (uint64_t v = v0; v < v0 + 8 && v < nvox; v += 2) {
        const uint32_t mk = marks[v / 2];
        if (mk) marks[v / 2] = 0u;
        for (uint64_t k = 0; k < 2 && v + k < nvox; ++k) {
            const uint32_t mine = (mk >> (16 * k)) & 0xFFFFu;
            if (!PROB && mine == 0u) continue;
            const float l = moved(L[v + k], mine);
            if (mine) L[v + k] = l;
            if constexpr (PROB) P[v + k] = prob(l);
        }
    }
}

__global__ __launch_bounds__(256) void logodds_to_prob_kernel(const float* __restrict__ L,
                                                              float* __restrict__ P, uint64_t nvox) {
    const uint64_t v = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nvox) return;
    P[v] = 1.0f / (1.0f + expf(-L[v]));
}

}  // namespace nbt

using namespace nbt;

extern "C" uint64_t nbt_ig_insert_workspace_words(const nbt_ig_map* map) {
    if (!map) return 0;
    return ((uint64_t)map->dm.nx * (uint64_t)map->dm.ny * (uint64_t)map->dm.nz + 1) / 2;
}

extern "C" nbt_ig_insert_params nbt_ig_insert_default_params(void) {
    // log(p / (1 - p)) for hit 0.7, miss 0.4 and the bounds 0.1192 and 0.971, in binary32
    return nbt_ig_insert_params{0x1.b1d106p-1f, -0x1.9f323ep-2f, -0x1.0000eap+1f, 0x1.c16974p+1f};
}

extern "C" int nbt_ig_insert_scans(const nbt_ig_map* map, const nbt_ig_camera* cam, const float* poses,
                                   const float* depth, uint32_t n_scans, const nbt_ig_insert_params* params,
                                   float* logodds, float* prob_out, uint32_t* workspace,
                                   uint64_t workspace_words, void* stream) {
    if (int rc = check_map(map)) return rc;
    CamParams c;
    if (int rc = check_camera(cam, &c)) return rc;
    if (!logodds || !workspace) return fail(NBT_IG_EINVAL, "logodds or workspace is NULL");
    if (workspace_words < nbt_ig_insert_workspace_words(map))
        return fail(NBT_IG_EINVAL, "workspace holds %llu words, the map needs %llu",
                    (unsigned long long)workspace_words,
                    (unsigned long long)nbt_ig_insert_workspace_words(map));
    if (n_scans > 0 && (!poses || !depth)) return fail(NBT_IG_EINVAL, "poses or depth is NULL");
    const nbt_ig_insert_params p = params ? *params : nbt_ig_insert_default_params();
    if (!std::isfinite(p.l_hit) || !std::isfinite(p.l_miss) || !std::isfinite(p.l_min) ||
        !std::isfinite(p.l_max) || !(p.l_min <= p.l_max))
        return fail(NBT_IG_EINVAL, "insertion parameters must be finite with l_min <= l_max");
    const uint64_t rays = (uint64_t)c.W * (uint64_t)c.H;
    const uint64_t nvox = (uint64_t)map->dm.nx * (uint64_t)map->dm.ny * (uint64_t)map->dm.nz;
    DeviceGuard g(map->ctx->device);
    if (!g.ok) return fail(NBT_IG_EDEVICE, "cannot select device %d", map->ctx->device);
    hipStream_t s = (hipStream_t)stream;
    const unsigned mark_blocks = (unsigned)((((uint64_t)c.W + 15) / 16) * (((uint64_t)c.H + 15) / 16));
    const unsigned apply_blocks = (unsigned)(((nvox + 7) / 8 + 255) / 256);
    const bool small = map->dm.nx <= 512 && map->dm.ny <= 512 && map->dm.nz <= 512;
    const bool vec = (((uintptr_t)workspace | (uintptr_t)logodds | (uintptr_t)prob_out) & 15u) == 0;
    for (uint32_t k = 0; k < n_scans; ++k) {
        auto mark = small ? insert_mark_kernel<uint32_t> : insert_mark_kernel<uint64_t>;
        hipLaunchKernelGGL(mark, dim3(mark_blocks), dim3(256), 0, s, map->dm, c, poses + 12 * (size_t)k,
                           depth + rays * k, reinterpret_cast<uint8_t*>(workspace));
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "insert_mark_kernel");
        auto apply = prob_out && k + 1 == n_scans ? insert_apply_kernel<true> : insert_apply_kernel<false>;
        hipLaunchKernelGGL(apply, dim3(apply_blocks), dim3(256), 0, s, workspace, logodds, prob_out, nvox, p, vec);
        e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "insert_apply_kernel");
    }
    if (prob_out && n_scans == 0) {
        hipLaunchKernelGGL(logodds_to_prob_kernel, dim3((unsigned)((nvox + 255) / 256)), dim3(256), 0, s,
                           logodds, prob_out, nvox);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e, "logodds_to_prob_kernel");
    }
    return NBT_IG_OK;
}
