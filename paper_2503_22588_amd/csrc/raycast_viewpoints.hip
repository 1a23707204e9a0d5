// raycast_viewpoints.hip -- per-perspective IG and the parity-mode ray records.
//
// Work decomposition: a perspective's N_E rays are cut into pixel tiles of
// 64 rays, one tile per wavefront (one ray per lane).  Neighbouring pixels
// have nearly parallel rays, so a wave's 64 gathers per step fall into a
// few cache lines of the map.  A workgroup of WAVES waves covers
// WAVES*tiles_per_wave tiles of one perspective; a perspective with more
// tiles is split over several workgroups whose partial sums are combined in
// fixed point (order independent), the last one writing g_P = sum / N_E
// (Sec. III, IG calculation: the per-perspective mean of the ray gains).
#include <algorithm>
#include <cmath>
#include <tuple>
#include <type_traits>

#include "ray.hpp"
#include "reduce.hpp"

namespace nbt {

// Consecutive workgroup ids are dealt round-robin to the 8 XCDs, so the
// workgroups of one perspective would land on different L2s.  With a chunk
// C > 0 each XCD instead receives runs of C consecutive logical workgroups
// (runs interleaved across XCDs in launch order, so all XCDs still progress
// through the perspectives together); the incomplete last round keeps the
// identity order.  The mapping is a bijection on [0, nb).
__device__ __forceinline__ uint32_t xcd_logical(uint32_t bid, uint32_t nb, uint32_t chunk) {
    constexpr uint32_t kXcd = 8;
    const uint32_t round = kXcd * chunk;
    const uint32_t full = (nb / round) * round;
    if (bid >= full) return bid;
    const uint32_t xcd = bid % kXcd, slot = bid / kXcd;
    return ((slot / chunk) * kXcd + xcd) * chunk + slot % chunk;
}

// Sums the lanes of a workgroup of `waves` waves (at most WAVES) and writes
// perspective vp's result (groups == 1) or combines the sum with the other
// workgroups of the perspective (the last one writes).  Called uniformly by
// the whole block.
template <int WAVES>
__device__ __forceinline__ void vp_combine(int waves, double acc, uint32_t steps, bool invalid, uint32_t vp,
                                           uint32_t groups, double rays, double scale, float* __restrict__ ig_out,
                                           unsigned long long* __restrict__ steps_out,
                                           VpAccum* __restrict__ ws) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    acc = wave_sum(acc);
    steps = wave_sum_u32(steps);
    const bool wave_invalid = __ballot(invalid) != 0ull;

    __shared__ double s_acc[WAVES];
    __shared__ unsigned long long s_steps[WAVES];
    __shared__ int s_inv[WAVES];
    if (lane == 0) {
        s_acc[wave] = acc;
        s_steps[wave] = steps;
        s_inv[wave] = wave_invalid ? 1 : 0;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;

    double tot = 0.0;
    unsigned long long st = 0;
    int inv = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        if (w >= waves) break;
        tot += s_acc[w];
        st += s_steps[w];
        inv |= s_inv[w];
    }
    if (groups == 1) {
        ig_out[vp] = inv ? __builtin_nanf("") : (float)(tot / rays);
        if (steps_out) steps_out[vp] = st;
        return;
    }
    // The slot's fields are only ever touched by device-scope atomic
    // read-modify-writes, which every XCD performs at one point per address
    // (the counts come out exact across XCDs).  Each returned old value is
    // that address's value at the moment this RMW took its place there, so
    // once the three returns are in, this workgroup's sums are part of every
    // later RMW's view.  The count's increment is made to depend on those
    // returns (the empty asm consumes them and hands back the 1), which holds
    // the count's RMW until they have arrived; the last workgroup's count has
    // then come after every other workgroup's sums, and it reads them with
    // RMWs too.  No fence: a release fence at device scope writes back the
    // XCD's L2 in every workgroup, and the last one's acquire fence
    // invalidates it (the map's gathers of the other workgroups there then
    // miss); they cost 8-15 % of a call of 64-256 perspectives of 64x48 rays.
    VpAccum* a = ws + vp;
    const unsigned long long o_sum = atomicAdd(&a->sum_fx, __double2ull_rn(tot * scale));
    const unsigned long long o_steps = atomicAdd(&a->steps, st);
    const unsigned int o_inv = inv ? atomicOr(&a->invalid, 1u) : 0u;
    unsigned int one = 1u;
    asm volatile("" : "+v"(one) : "v"(o_sum), "v"(o_steps), "v"(o_inv));
    const unsigned int done = atomicAdd(&a->count, one);
    if (done == groups - 1) {
        const unsigned long long s = atomicExch(&a->sum_fx, 0ull);
        const unsigned long long stp = atomicExch(&a->steps, 0ull);
        const unsigned int iv = atomicExch(&a->invalid, 0u);
        atomicExch(&a->count, 0u);
        ig_out[vp] = iv ? __builtin_nanf("") : (float)(((double)s / scale) / rays);
        if (steps_out) steps_out[vp] = stp;
    }
}

// The map's palette in LDS (filled by the whole block), or nullptr when the
// map is to be walked by its words.  The flag and the palette are requested
// together.
__device__ __forceinline__ const uint32_t* load_palette(const DevMap& m, uint32_t (&s_pal)[kCodes]) {
    if (!m.codes) return nullptr;
    const uint32_t over = m.palette[kCodes];
    for (uint32_t k = 4u * threadIdx.x; k < kCodes; k += 4u * blockDim.x)
        *reinterpret_cast<uint4*>(&s_pal[k]) = *reinterpret_cast<const uint4*>(m.palette + k);
    __syncthreads();
    return over == 0u ? s_pal : nullptr;
}

// The rays of workgroup-slice g of perspective vp: WAVES waves walk their
// tiles, then the block's sum is written (groups == 1) or combined with the
// other slices of the perspective (last slice writes).  Called uniformly by
// the whole block.  TRACE (parity mode) also writes every ray's record to
// trace[vp * N_E + k], built by the walk below from the offsets it gathers;
// the walk and the IG arithmetic are those of the timed instance.
template <int WAVES, int DEPTH, bool COUNT, bool TRACE, bool CODED>
__device__ __forceinline__ void vp_group(const DevMap& m, const CamParams& c,
                                         const float (&pose)[12], uint32_t vp, uint32_t g,
                                         uint32_t groups, uint32_t tiles_x, uint32_t tiles,
                                         int tw_log2, int tpw, float* __restrict__ ig_out,
                                         unsigned long long* __restrict__ steps_out,
                                         VpAccum* __restrict__ ws, nbt_ig_ray_digest* __restrict__ trace,
                                         const uint32_t* pal) {
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int tw = 1 << tw_log2;
    const int th = 64 >> tw_log2;
    int lx, ly;
    tile_pixel(lane, tw_log2, lx, ly);
    const __amdgpu_buffer_rsrc_t rs = map_rsrc(m);

    double acc = 0.0;
    uint32_t steps = 0;
    bool invalid = false;
    for (int r = 0; r < tpw; ++r) {
        const uint32_t tile = (g * WAVES + (uint32_t)wave) * (uint32_t)tpw + (uint32_t)r;
        if (tile >= tiles) break;
        const int i = (int)(tile % tiles_x) * tw + lx;
        const int j = (int)(tile / tiles_x) * th + ly;
        if (i < c.W && j < c.H) {
            RayState ray;
            const int st = setup_ray(m, c, pose, i, j, ray);
            [[maybe_unused]] WalkTrace rec;
            if (st == kRayOk) {
                if constexpr (DEPTH == 1) {
                    if constexpr (TRACE) {
                        // the depth-1 walk addresses each voxel from its coordinates
                        rec.reason = walk_ray<true>(m, rs, ray, acc, steps, [&](int x, int y, int z, uint32_t word) {
                            rec.last = (z * m.ny + y) * m.nx + x;
                            rec.hash = fnv1a_u32(rec.hash, (uint32_t)rec.last);
                            rec.gain += (double)__uint_as_float(word & ~kOccBit);
                            ++rec.steps;
                        });
                    } else {
                        walk_ray<false>(m, rs, ray, acc, steps, [](int, int, int, uint32_t) {});
                    }
                } else {
                    auto walk = [&](auto tl) {
                        constexpr int TLv = decltype(tl)::value;
                        if constexpr (TRACE)
                            walk_ray_pipelined<DEPTH, COUNT, TLv, WalkTrace>(m, rs, ray, acc, steps, &rec);
                        else
                            walk_ray_pipelined<DEPTH, COUNT, TLv>(m, rs, ray, acc, steps);
                    };
                    bool coded = false;
                    if constexpr (CODED) {
                        if (pal) {           // uniform per workgroup
                            coded = true;
                            const uint32_t most = (uint32_t)(m.nx + m.ny + m.nz + 3) / kRunSlots + 2u;
                            if constexpr (TRACE) walk_ray_codes<COUNT, WalkTrace>(m, pal, ray, 0u, most, acc, steps, &rec);
                            else walk_ray_codes<COUNT>(m, pal, ray, 0u, most, acc, steps);
                            if constexpr (TRACE) rec.finish();
                        }
                    }
                    if (!coded) {
                        switch (m.tl) {      // the map's order; uniform per workgroup
                        case 1: walk(std::integral_constant<int, 1>{}); break;
                        case 2: walk(std::integral_constant<int, 2>{}); break;
                        case 3: walk(std::integral_constant<int, 3>{}); break;
                        default: walk(std::integral_constant<int, 0>{});
                        }
                    }
                }
            } else if (st == kRayInvalid) {
                invalid = true;
            }
            if constexpr (TRACE)
                write_trace(trace + (size_t)vp * ((size_t)c.W * c.H) + (size_t)j * c.W + i, st, rec);
        }
    }

    vp_combine<WAVES>(WAVES, acc, steps, invalid, vp, groups, (double)c.W * (double)c.H, fix_scale(m, c), ig_out,
                      steps_out, ws);
}

// CODED: the map has codes (walked by them unless its palette overflowed).
template <int WAVES, int DEPTH, bool COUNT, bool TRACE, bool CODED>
__global__ __launch_bounds__(WAVES * 64) void ig_viewpoints_kernel(
    DevMap m, CamParams c, const float* __restrict__ poses, uint32_t groups, uint32_t tiles_x,
    uint32_t tiles, int tw_log2, int tpw, int remap, float* __restrict__ ig_out,
    unsigned long long* __restrict__ steps_out, VpAccum* __restrict__ ws,
    nbt_ig_ray_digest* __restrict__ trace) {
    const uint32_t bid = remap > 0 ? xcd_logical(blockIdx.x, gridDim.x, (uint32_t)remap) : blockIdx.x;
    const uint32_t vp = bid / groups;
    const uint32_t g = bid - vp * groups;
    float pose[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) pose[k] = poses[12 * (size_t)vp + k];
    const uint32_t* pal = nullptr;
    if constexpr (CODED) {
        __shared__ __align__(16) uint32_t s_pal[kCodes];
        pal = load_palette(m, s_pal);
    }
    vp_group<WAVES, DEPTH, COUNT, TRACE, CODED>(m, c, pose, vp, g, groups, tiles_x, tiles,
                                         tw_log2, tpw, ig_out, steps_out, ws, trace, pal);
}

// Small calls: a ray's voxels are a serial chain (each step picks the next of
// three crossings), so a call of a few hundred rays lasts as long as its
// longest ray (100 perspectives of 6 rays through a 320^3 map: 39 us for some
// 250 steps, 10 us now) while most lanes of its waves idle.  Every ray is cut
// into S segments walked by S lanes at once.  What a segment needs to start
// is the exact traversal state there, and per axis the crossing parameters
// are a chain of single additions, independent of the other axes: three
// lanes of each ray first write the chains into an LDS table (an addition
// and a store per crossing), then each segment's lane looks up how many
// crossings of each axis lie below its threshold, which gives its voxel, its
// next crossings and its slot index K, all as the serial walk would reach
// them.  Segments start at the next multiple of kRunSlots slots, so the runs
// summed in binary32 and the visits are those of the unsplit walk.  Lanes
// beyond the segment in which a ray ended count nothing.
//
// A ray whose chain does not reach its end within the table (a pose whose
// rotation stretches it) is walked whole by its first lane.  In parity mode the
// segments run one after the other, handing the record on.
constexpr int kSegThreads = 256, kSegRays = 64;
template <bool COUNT, bool TRACE>
__global__ __launch_bounds__(kSegThreads) void ig_segments_kernel(DevMap m, CamParams c, const float* __restrict__ poses,
                                                          SegLaunch L, uint32_t tiles_x,
                                                          float* __restrict__ ig_out,
                                                          unsigned long long* __restrict__ steps_out,
                                                          VpAccum* __restrict__ ws,
                                                          nbt_ig_ray_digest* __restrict__ trace) {
    extern __shared__ float s_tab[];             // every eighth crossing: [block][axis][ray]
    __shared__ uint32_t s_len[3][kSegRays], s_slot[kSegThreads + kSegRays], s_end[kSegRays];
    const uint32_t rays = 1u << L.rays_log2, segs = 1u << L.segs_log2;
    const uint32_t vp = blockIdx.x / L.groups, g = blockIdx.x - vp * L.groups;
    const uint32_t r = threadIdx.x & (rays - 1u), seg = threadIdx.x >> L.rays_log2;
    int i, j;
    if (L.flat) {
        const uint32_t k = g * rays + r;
        i = (int)(k % (uint32_t)c.W);
        j = (int)(k / (uint32_t)c.W);
    } else {
        const int twl = (L.rays_log2 + 1) / 2, thl = L.rays_log2 - twl;
        i = (int)((g % tiles_x) << twl) + (int)(r & ((1u << twl) - 1u));
        j = (int)((g / tiles_x) << thl) + (int)(r >> twl);
    }
    float pose[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) pose[k] = poses[12 * (size_t)vp + k];
    RayState ray;
    int st = kRayMiss;
    const bool pixel = i < c.W && j < c.H;
    if (pixel) st = setup_ray(m, c, pose, i, j, ray);
    const bool ok = st == kRayOk;

    if (seg == 0u) s_end[r] = segs;
    for (uint32_t a = seg; a < 3u; a += segs) {
        uint32_t len = 0u;                       // 0: the chain does not reach the ray's end
        if (ok) {
            float t = a == 0u ? ray.tx : a == 1u ? ray.ty : ray.tz;
            const float dt = a == 0u ? ray.dtx : a == 1u ? ray.dty : ray.dtz;
            float* tab = s_tab + a * rays + r;
            for (uint32_t k = 0; k < L.blocks; ++k) {
                tab[3u * k * rays] = t;
#pragma unroll
                for (int u = 0; u < 8; ++u) t = t + dt;
                if (t > ray.t1) {
                    len = k + 1u;
                    break;
                }
            }
        }
        s_len[a][r] = len;
    }
    __syncthreads();

    const uint32_t lx = s_len[0][r], ly = s_len[1][r], lz = s_len[2][r];
    const bool split = ok && lx != 0u && ly != 0u && lz != 0u;
    uint32_t slot = 0u;                          // crossings before this segment
    bool here = ok && (split || seg == 0u);
    if (split && seg != 0u) {
        const float lo = fminf(fminf(ray.tx, ray.ty), ray.tz);
        const float T = lo + (ray.t1 - lo) * ((float)seg / (float)segs);
        uint32_t kx = 0u, ky = 0u, kz = 0u;      // blocks that begin below T per axis
        const float* tab = s_tab + r;
        for (uint32_t b = 1u << (31 - __clz((int)L.blocks)); b != 0u; b >>= 1) {
            const uint32_t px = kx + b, py = ky + b, pz = kz + b;
            // entries beyond a chain's length are not read
            const float vx = px <= lx ? tab[(3u * px - 3u) * rays] : T;
            const float vy = py <= ly ? tab[(3u * py - 2u) * rays] : T;
            const float vz = pz <= lz ? tab[(3u * pz - 1u) * rays] : T;
            kx = vx < T ? px : kx;
            ky = vy < T ? py : ky;
            kz = vz < T ? pz : kz;
        }
        // then crossing by crossing inside the last such block (none: block 0,
        // whose first crossing is not below T)
        kx = kx ? kx - 1u : 0u;
        ky = ky ? ky - 1u : 0u;
        kz = kz ? kz - 1u : 0u;
        ray.tx = tab[3u * kx * rays];
        ray.ty = tab[(3u * ky + 1u) * rays];
        ray.tz = tab[(3u * kz + 2u) * rays];
        kx *= 8u;
        ky *= 8u;
        kz *= 8u;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool bx = ray.tx < T, by = ray.ty < T, bz = ray.tz < T;
            kx += bx ? 1u : 0u;
            ky += by ? 1u : 0u;
            kz += bz ? 1u : 0u;
            ray.tx = ray.tx + (bx ? ray.dtx : 0.0f);
            ray.ty = ray.ty + (by ? ray.dty : 0.0f);
            ray.tz = ray.tz + (bz ? ray.dtz : 0.0f);
        }
        slot = kx + ky + kz;
        ray.ix += (int)kx * ray.sx;
        ray.iy += (int)ky * ray.sy;
        ray.iz += (int)kz * ray.sz;
        // out of the map: the ray has ended in an earlier segment
        here = (uint32_t)ray.ix < (uint32_t)m.nx && (uint32_t)ray.iy < (uint32_t)m.ny &&
               (uint32_t)ray.iz < (uint32_t)m.nz;
    }
    const uint32_t first = (slot + kRunSlots - 1u) / kRunSlots;       // its first group of slots
    const uint32_t most = (uint32_t)(m.nx + m.ny + m.nz + 3) / kRunSlots + 2u;
    s_slot[seg * rays + r] = split ? first : most;
    if (seg == segs - 1u) s_slot[segs * rays + r] = most;
    __syncthreads();
    const uint32_t next = max(s_slot[(seg + 1u) * rays + r], first);

    double acc = 0.0;
    uint32_t steps = 0;
    __shared__ __align__(16) uint32_t s_pal[kCodes];
    const uint32_t* pal = load_palette(m, s_pal);
    const __amdgpu_buffer_rsrc_t rs = map_rsrc(m);
    auto walk = [&](auto tl, auto* rec) {
        constexpr int TLv = decltype(tl)::value;
        using Rec = std::remove_pointer_t<decltype(rec)>;
        return walk_ray_stretch<COUNT, TLv, Rec>(m, rs, ray, first * kRunSlots - slot, next - first, acc, steps, rec);
    };
    auto walk_order = [&](auto* rec) {           // codes or the map's order; uniform per workgroup
        using Rec = std::remove_pointer_t<decltype(rec)>;
        if (pal)
            return walk_ray_codes<COUNT, Rec>(m, pal, ray, first * kRunSlots - slot, next - first, acc, steps, rec);
        switch (m.tl) {
        case 1: return walk(std::integral_constant<int, 1>{}, rec);
        case 2: return walk(std::integral_constant<int, 2>{}, rec);
        case 3: return walk(std::integral_constant<int, 3>{}, rec);
        default: return walk(std::integral_constant<int, 0>{}, rec);
        }
    };
    bool over = false;
    if constexpr (TRACE) {
        __shared__ __align__(16) unsigned char s_rec_bytes[kSegRays * sizeof(WalkTrace)];
        WalkTrace* s_rec = reinterpret_cast<WalkTrace*>(s_rec_bytes);
        if (seg == 0u) s_rec[r] = WalkTrace{};
        for (uint32_t k = 0; k < segs; ++k) {
            __syncthreads();
            if (seg == k && here && next > first && s_rec[r].reason < 0) {
                WalkTrace rec = s_rec[r];
                over = walk_order(&rec);
                s_rec[r] = rec;
            }
        }
        __syncthreads();
        if (seg == 0u && pixel) {
            WalkTrace rec = s_rec[r];
            if (ok) rec.finish();
            write_trace(trace + (size_t)vp * ((size_t)c.W * c.H) + (size_t)j * c.W + i, st, rec);
        }
    } else {
        NoTrace none;
        if (here && next > first) over = walk_order(&none);
    }
    if (over) atomicMin(&s_end[r], seg);
    __syncthreads();
    if (seg > s_end[r]) {
        acc = 0.0;
        steps = 0u;
    }
    vp_combine<kSegThreads / 64>((int)(blockDim.x >> 6), acc, steps, seg == 0u && st == kRayInvalid, vp, L.groups,
                                  (double)c.W * (double)c.H, fix_scale(m, c), ig_out, steps_out, ws);
}

// Persistent batched launch: many maps, a CSR of perspectives per map
// (offsets[k]..offsets[k+1]).  Work items are (perspective, slice) pairs in
// map-major order; each workgroup pops items from an atomic counter until
// the queue is empty, so uneven maps and perspective counts balance across
// the chip and co-resident workgroups share one map in L2.
// Seven waves per SIMD: left to itself the coded kernel takes 98 VGPRs (five
// waves; 64 maps 2.9 ms against 2.55).
template <int WAVES, int DEPTH, bool COUNT, bool CODED>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(CODED ? 7 : 1, CODED ? 7 : 8))) void ig_batch_kernel(
    const DevMap* __restrict__ maps, uint32_t n_maps, const uint32_t* __restrict__ offsets,
    uint32_t capacity, CamParams c, const float* __restrict__ poses, uint32_t groups,
    uint32_t tiles_x, uint32_t tiles, int tw_log2, int tpw, unsigned int* __restrict__ queue,
    float* __restrict__ ig_out, unsigned long long* __restrict__ steps_out,
    VpAccum* __restrict__ ws) {
    __shared__ uint32_t s_item, s_map;
    uint32_t total = offsets[n_maps];
    total = total < capacity ? total : capacity;
    const uint64_t items = (uint64_t)total * groups;
    const uint32_t* pal = nullptr;
    uint32_t pal_map = n_maps;              // the map whose palette is loaded
    for (;;) {
        __syncthreads();                    // previous item's reductions are done
        if (threadIdx.x == 0) {
            const uint32_t it = atomicAdd(queue, 1u);
            uint32_t mi = 0;
            if (it < items) {
                const uint32_t vp = it / groups;
                uint32_t lo = 0, hi = n_maps;          // largest k with offsets[k] <= vp
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) / 2;
                    if (offsets[mid] <= vp) lo = mid; else hi = mid;
                }
                mi = lo;
            }
            s_item = it;
            s_map = mi;
        }
        __syncthreads();
        const uint32_t it = s_item;
        if (it >= items) return;
        const uint32_t vp = it / groups;
        const uint32_t g = it - vp * groups;
        const DevMap m = maps[s_map];
        float pose[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) pose[k] = poses[12 * (size_t)vp + k];
        if constexpr (CODED) {
            __shared__ __align__(16) uint32_t s_pal[kCodes];
            if (s_map != pal_map) {         // (the barriers above: nobody reads the old one)
                pal_map = s_map;
                pal = load_palette(m, s_pal);
            }
        }
        vp_group<WAVES, DEPTH, COUNT, false, CODED>(m, c, pose, vp, g, groups, tiles_x, tiles,
                                             tw_log2, tpw, ig_out, steps_out, ws, nullptr, pal);
    }
}

__global__ void batch_reset_kernel(unsigned int* queue) { *queue = 0u; }

__global__ __launch_bounds__(256) void clear_slots_kernel(VpAccum* __restrict__ ws, uint32_t n) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < n) ws[i] = VpAccum{0ull, 0ull, 0u, 0u};
}

hipError_t launch_clear_slots(VpAccum* ws, uint32_t n, hipStream_t s) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(clear_slots_kernel, dim3((n + 255) / 256), dim3(256), 0, s, ws, n);
    return hipGetLastError();
}

// Parity mode: one thread per ray, full record per ray.
__global__ __launch_bounds__(256) void trace_rays_kernel(DevMap m, CamParams c,
                                                         const float* __restrict__ poses, uint32_t n,
                                                         nbt_ig_ray_digest* __restrict__ out) {
    const uint64_t rays = (uint64_t)c.W * (uint64_t)c.H;
    const uint64_t gid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= rays * n) return;
    const uint32_t vp = (uint32_t)(gid / rays);
    const uint32_t k = (uint32_t)(gid - (uint64_t)vp * rays);
    float pose[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) pose[q] = poses[12 * (size_t)vp + q];
    const int i = (int)(k % (uint32_t)c.W), j = (int)(k / (uint32_t)c.W);

    nbt_ig_ray_digest d;
    d.hash = kFnvBasis;
    d.gain = 0.0;
    d.steps = 0;
    d.stop_lin = -1;
    d.reason = NBT_IG_RAY_MISS;
    d.reserved = 0;
    RayState ray;
    const int st = setup_ray(m, c, pose, i, j, ray);
    if (st == kRayInvalid) {
        d.reason = NBT_IG_RAY_INVALID;
        d.gain = __builtin_nan("");
    } else if (st == kRayOk) {
        unsigned long long h = kFnvBasis;
        int32_t last = -1;
        double acc = 0.0;
        uint32_t steps = 0;
        const int reason = walk_ray<true>(m, map_rsrc(m), ray, acc, steps,
                                          [&](int x, int y, int z, uint32_t) {
                                              last = (z * m.ny + y) * m.nx + x;
                                              h = fnv1a_u32(h, (uint32_t)last);
                                          });
        d.hash = h;
        d.gain = acc;
        d.steps = steps;
        d.stop_lin = last;
        d.reason = (uint32_t)reason;
    }
    out[gid] = d;
}

__global__ __launch_bounds__(256) void trace_paths_kernel(DevMap m, CamParams c,
                                                          const float* __restrict__ poses, uint32_t n,
                                                          const uint32_t* __restrict__ sel,
                                                          uint32_t count, uint32_t max_len,
                                                          int32_t* __restrict__ lin_out,
                                                          uint32_t* __restrict__ len_out) {
    const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= count) return;
    const uint32_t vp = sel[2 * r], k = sel[2 * r + 1];
    const uint32_t rays = (uint32_t)c.W * (uint32_t)c.H;
    if (vp >= n || k >= rays) {
        len_out[r] = 0;
        return;
    }
    float pose[12];
#pragma unroll
    for (int q = 0; q < 12; ++q) pose[q] = poses[12 * (size_t)vp + q];
    RayState ray;
    uint32_t steps = 0;
    if (setup_ray(m, c, pose, (int)(k % (uint32_t)c.W), (int)(k / (uint32_t)c.W), ray) == kRayOk) {
        double acc = 0.0;
        int32_t* dst = lin_out + (size_t)r * max_len;
        uint32_t w = 0;
        walk_ray<true>(m, map_rsrc(m), ray, acc, steps, [&](int x, int y, int z, uint32_t) {
            if (w < max_len) dst[w] = (z * m.ny + y) * m.nx + x;
            ++w;
        });
    }
    len_out[r] = steps;
}

hipError_t launch_eval_viewpoints(const DevMap& m, const CamParams& c, const float* poses,
                                  uint32_t n, float* ig_out, unsigned long long* steps_out,
                                  VpAccum* ws, const VpLaunch& L0, hipStream_t s,
                                  nbt_ig_ray_digest* trace) {
    const VpLaunch L = resolve_launch(c, L0);
    const int tw = 1 << L.tile_w_log2, th = 64 >> L.tile_w_log2;
    const uint32_t tiles_x = (uint32_t)((c.W + tw - 1) / tw);
    const uint32_t tiles = tiles_x * (uint32_t)((c.H + th - 1) / th);
    const uint32_t groups = vp_groups(c, L);
    const dim3 grid((unsigned)((uint64_t)n * groups));
    const auto args = std::make_tuple(m, c, poses, groups, tiles_x, tiles, L.tile_w_log2,
                                      L.tiles_per_wave, L.xcd_remap, ig_out, steps_out, ws, trace);
    auto go = [&](auto kernel, int waves) {
        std::apply([&](auto... a) { hipLaunchKernelGGL(kernel, grid, dim3(waves * 64), 0, s, a...); },
                   args);
    };
    // Without steps_out the walk skips the per-voxel visit count.
    const bool count = steps_out != nullptr;
    // Only the walk at the default depth knows codes.
    const bool coded = m.codes != nullptr && L.depth == 8;
#define NBT_VP_GO(W, D)                                                                            \
    (coded ? NBT_VP_GO2(W, D, (D == 8)) : NBT_VP_GO2(W, D, false))
#define NBT_VP_GO2(W, D, CD)                                                                       \
    (trace ? (count ? go(ig_viewpoints_kernel<W, D, true, true, CD>, W)                            \
                    : go(ig_viewpoints_kernel<W, D, false, true, CD>, W))                          \
           : (count ? go(ig_viewpoints_kernel<W, D, true, false, CD>, W)                           \
                    : go(ig_viewpoints_kernel<W, D, false, false, CD>, W)))
#define NBT_VP_DEPTHS(W)                                  \
    case W:                                               \
        switch (L.depth) {                                \
            case 1: NBT_VP_GO(W, 1); break;               \
            case 2: NBT_VP_GO(W, 2); break;               \
            case 4: NBT_VP_GO(W, 4); break;               \
            case 8: NBT_VP_GO(W, 8); break;               \
            default: return hipErrorInvalidValue;         \
        }                                                 \
        break;
    switch (L.waves) {
        NBT_VP_DEPTHS(1)
        NBT_VP_DEPTHS(2)
        NBT_VP_DEPTHS(4)
        NBT_VP_DEPTHS(8)
        default:
            return hipErrorInvalidValue;
    }
#undef NBT_VP_GO
#undef NBT_VP_GO2
#undef NBT_VP_DEPTHS
    return hipGetLastError();
}

// Segments pay while the rays alone leave the chip waiting on single chains
// and the memory idle: calls of up to kSegMaxRays rays of some hundred
// voxels.  They are cut until there are about kSegLanes lanes, into 4 to 32
// segments of at least kSegVoxels voxels (the table, the state and up to 7
// slots before a segment's first group cost as much as some twenty).  Whole
// calls (us), unsplit and split, maps of 320^3 at 1 cm: 100 x 6 rays 39 and
// 10-11, 1000 x 6 76 and 19-21, 200 x 20 40 and 15-16, 100 x 86 42 and 22,
// 3000 x 6 89 and 45; one perspective of 19,200 rays 36 and 25.  Beyond, the
// map's lines are what the call waits for: 1000 x 20 41 and 41, 500 x 86 54
// and 69.  Short rays do not pay either: 8 x 3072 rays of up to 80 voxels 15
// and 15.5.
// A workgroup of one wave spreads best; it grows to four while a perspective
// would have more than 8 of them (one perspective's combine in turn, 35 ns each; 256
// perspectives at once 3 ns a workgroup, 4096 less than 1) or
// the call more than two per CU.
constexpr uint64_t kSegMaxRays = 32768, kSegLanes = 49152;
constexpr uint32_t kSegVoxels = 24;

SegLaunch plan_segments(const DevMap& m, const CamParams& c, uint32_t n, int cu_count) {
    SegLaunch L{-1, 0, 0, 0, 0};
    const uint64_t rays = (uint64_t)c.W * (uint64_t)c.H;
    const uint64_t all = rays * n;
    if (all == 0 || all > kSegMaxRays) return L;
    // crossings per axis: a ray of a rigid pose is at most this long, and leaves the map after n of them
    const double len = std::sqrt((double)c.dh * c.dh + (double)c.dv * c.dv + (double)c.range * c.range) * m.inv_s;
    const int side = std::max(m.nx, std::max(m.ny, m.nz));
    const double cross = len + 2.0 < (double)(side + 1) ? len + 2.0 : (double)(side + 1);
    const uint32_t voxels = (uint32_t)(1.5 * cross);
    int s = 5;
    while (s >= 2 && ((s > 2 && (all << s) > kSegLanes) || (voxels >> s) < kSegVoxels)) --s;
    if (s < 2) return L;
    L.blocks = (uint32_t)cross / 8u + 1u;
    L.segs_log2 = s;
    L.flat = rays <= 64 || c.W < 8 || c.H < 8;
    for (int r = 6 - s;; ++r) {
        const uint32_t tw = 1u << ((r + 1) / 2), th = 1u << (r - (r + 1) / 2);
        L.rays_log2 = r;
        L.groups = L.flat ? (uint32_t)((rays + (1ull << r) - 1) >> r)
                          : (((uint32_t)c.W + tw - 1) / tw) * (((uint32_t)c.H + th - 1) / th);
        const bool grow = L.groups > 8 || (uint64_t)n * L.groups > 2ull * (uint64_t)cu_count;
        if (r + s == 8 || L.groups == 1 || !grow) break;
    }
    if (((size_t)12 * L.blocks << L.rays_log2) > 60 * 1024) L.segs_log2 = -1;
    return L;
}

hipError_t launch_eval_segments(const DevMap& m, const CamParams& c, const float* poses, uint32_t n,
                                float* ig_out, unsigned long long* steps_out, VpAccum* ws, const SegLaunch& L,
                                hipStream_t s, nbt_ig_ray_digest* trace) {
    const dim3 grid(n * L.groups), block(1u << (L.rays_log2 + L.segs_log2));
    const size_t lds = (size_t)12 * L.blocks << L.rays_log2;
    const uint32_t tw = 1u << ((L.rays_log2 + 1) / 2), tiles_x = ((uint32_t)c.W + tw - 1) / tw;
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, lds, s, m, c, poses, L, tiles_x, ig_out, steps_out, ws, trace);
    };
    const bool count = steps_out != nullptr;
    if (trace) count ? go(ig_segments_kernel<true, true>) : go(ig_segments_kernel<false, true>);
    else count ? go(ig_segments_kernel<true, false>) : go(ig_segments_kernel<false, false>);
    return hipGetLastError();
}

const void* batch_kernel_ptr(int waves, int depth, bool count, bool coded) {
#define NBT_BK(W, D)                                                                               \
    if (waves == W && depth == D) {                                                                \
        if (coded && D == 8)                                                                       \
            return count ? (const void*)ig_batch_kernel<W, D, true, D == 8>                        \
                         : (const void*)ig_batch_kernel<W, D, false, D == 8>;                      \
        return count ? (const void*)ig_batch_kernel<W, D, true, false>                             \
                     : (const void*)ig_batch_kernel<W, D, false, false>;                           \
    }
    NBT_BK(1, 1) NBT_BK(1, 2) NBT_BK(1, 4) NBT_BK(1, 8)
    NBT_BK(2, 1) NBT_BK(2, 2) NBT_BK(2, 4) NBT_BK(2, 8)
    NBT_BK(4, 1) NBT_BK(4, 2) NBT_BK(4, 4) NBT_BK(4, 8)
    NBT_BK(8, 1) NBT_BK(8, 2) NBT_BK(8, 4) NBT_BK(8, 8)
#undef NBT_BK
    return nullptr;
}

const void* batch_reset_ptr() { return (const void*)batch_reset_kernel; }

hipError_t launch_trace_rays(const DevMap& m, const CamParams& c, const float* poses, uint32_t n,
                             nbt_ig_ray_digest* out, hipStream_t s) {
    const uint64_t total = (uint64_t)c.W * c.H * n;
    const uint64_t blocks = (total + 255) / 256;
    hipLaunchKernelGGL(trace_rays_kernel, dim3((unsigned)blocks), dim3(256), 0, s, m, c, poses, n, out);
    return hipGetLastError();
}

hipError_t launch_trace_paths(const DevMap& m, const CamParams& c, const float* poses, uint32_t n,
                              const uint32_t* rays, uint32_t count, uint32_t max_len,
                              int32_t* lin_out, uint32_t* len_out, hipStream_t s) {
    const uint32_t blocks = (count + 255) / 256;
    hipLaunchKernelGGL(trace_paths_kernel, dim3(blocks), dim3(256), 0, s, m, c, poses, n, rays,
                       count, max_len, lin_out, len_out);
    return hipGetLastError();
}

}  // namespace nbt
