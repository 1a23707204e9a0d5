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
#include "insert_walk.hpp"

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
// 640x576 into 256^3 at 2 cm: 216 us a scan with a store on every visit, 70 now
// (the walk itself: insert_walk.hpp).
struct SeenTable {
    unsigned char* at;                           // kSeen words in LDS
    __device__ uint32_t read(uint32_t lin4) const { return *reinterpret_cast<const uint32_t*>(at + seen_slot(lin4)); }
    __device__ void write(uint32_t lin4) const { *reinterpret_cast<uint32_t*>(at + seen_slot(lin4)) = lin4; }
    __device__ void pin() const { __builtin_amdgcn_sched_barrier(0); }
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
    insert_walk<T>(m, c, pose_in, depth[(size_t)j * (size_t)c.W + (size_t)i], i, j,
                   SeenTable{reinterpret_cast<unsigned char*>(s_seen)}, [&](uint32_t byte) { marks[byte] = 1; });
}

// One thread per 8 voxels (16 bytes of marks, 32 of values).  PROB: also the
// probability of every voxel (P may be L: a voxel's probability is stored after its
// log-odds).  vec: all three arrays are 16-byte aligned.
template <bool PROB>
__global__ __launch_bounds__(256) void insert_apply_kernel(uint32_t* __restrict__ marks, float* L, float* P,
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
