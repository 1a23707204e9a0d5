// cost.hip -- planner-side IG terms of Sec. IV for many candidate horizons.
//
//   G(x)  Eq. 3: inverse-distance weighting of the perspectives' IG, summed
//         over the N_B buffered information distributions with weight
//         1/(N_B - u) (u = 0 oldest);
//   O(x)  cosine between the camera's viewing axis and the direction to the
//         PoI, 0 when the PoI is outside the field of view;
//   c_I   sum over a horizon's states of w_I / (O G + eps).
// ALU-bound: about 10 VALU operations (one of them a quarter-rate reciprocal)
// per (state, perspective) pair.  One lane per state and up to 16 waves per
// workgroup that split the perspectives: a planner's call
// has few states (256 horizons of 20 states are 86 workgroups), so the
// parallelism has to come from the perspectives.  A perspective's position
// and IG are the same for the whole wave and are read through scalar loads.
// The waves split the perspectives of as many distributions at a time as one row,
// so there are two barriers for 16 of them (split one by one, the workgroup
// waited 2.4 us per distribution for the wave that summed up the last).
// 256 x 20 states against 10 x 500 perspectives: 671 us with one thread per
// state over all perspectives (20 workgroups of 4 waves on the chip) and 5 us
// for the horizons' sum in a launch of its own; 29 us in this kernel, 17 in
// the one below.  1024 horizons: 55 us here, 58 there; 4096: 131 and 203.
#include "internal.hpp"

namespace nbt {

constexpr int kCostRun = 64;     // pairs summed in binary32 before they join the binary64 sum
constexpr int kCostBlock = 8;    // perspectives whose scalar loads are in flight together

// The outputs of the states one wave holds (lane's: q), and with `cost` those of the
// `horizons` whole horizons they are: every horizon's terms are summed in order.
__device__ __forceinline__ void state_outputs(bool active, uint32_t q, float g, float tx, float ty, float tz, int lane,
                                              uint32_t horizons, uint32_t steps,
                                              const float* __restrict__ poses, uint32_t q_count, float px, float py,
                                              float pz, float tan_h, float tan_v, float w_i, float eps,
                                              float* __restrict__ g_out, float* __restrict__ o_out,
                                              float* __restrict__ cost, double* s_term) {
    float o = 0.0f;
    if (active) {
        g_out[q] = g;
        // orientation factor: camera coordinates of the PoI, c = R^T (poi - t)
        const float* r = poses + 12 * (size_t)q;
        const float vx = px - tx, vy = py - ty, vz = pz - tz;
        const float cx = r[0] * vx + r[3] * vy + r[6] * vz;
        const float cy = r[1] * vx + r[4] * vy + r[7] * vz;
        const float cz = r[2] * vx + r[5] * vy + r[8] * vz;
        const float n = sqrtf(vx * vx + vy * vy + vz * vz);
        if (cz > 0.0f && n > 0.0f && fabsf(cx / cz) <= tan_h && fabsf(cy / cz) <= tan_v) o = cz / n;
        o_out[q] = o;
    }
    if (!cost) return;
    s_term[lane] = (double)w_i / ((double)o * (double)g + (double)eps);
    __builtin_amdgcn_wave_barrier();
    const uint32_t h = blockIdx.x * horizons + (uint32_t)lane;
    if ((uint32_t)lane < horizons && h < q_count / steps) {
        double s = 0.0;
        for (uint32_t j = 0; j < steps; ++j) s += s_term[(uint32_t)lane * steps + j];
        cost[h] = (float)s;
    }
}

// Sums of one wave over a stretch of one distribution's perspectives.
struct IdwSums {
    double num = 0.0, den = 0.0, num0 = 0.0;
    uint32_t cnt0 = 0;
    float fnum = 0.0f, fden = 0.0f;              // the run's, in binary32
    __device__ __forceinline__ void join() {
        num += (double)fnum;
        den += (double)fden;
        fnum = fden = 0.0f;
    }
};

template <bool P_TWO>
__device__ __forceinline__ void idw_weigh(IdwSums& a, float d2, float ig, float half_neg_p) {
    const float w = P_TWO ? __builtin_amdgcn_rcpf(d2) : __builtin_powf(d2, half_neg_p);
    a.fnum = __builtin_fmaf(ig, w, a.fnum);
    a.fden += w;
}

template <bool P_TWO>
__device__ __forceinline__ void idw_pair(IdwSums& a, float dx, float dy, float dz, float ig, float half_neg_p) {
    const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
    if (d2 == 0.0f && dx == 0.0f && dy == 0.0f && dz == 0.0f) {
        // exactly on the perspective: counts instead of weighing
        a.num0 += (double)ig;
        ++a.cnt0;
    } else {
        idw_weigh<P_TWO>(a, d2, ig, half_neg_p);
    }
}

// G of the states that this workgroup's lanes hold (`subs` lanes each, `states` apart): the
// perspectives of up to kCostWaves distributions form one row that the waves
// split evenly, so a wave's stretch touches at most two of them;
// add(sums, u, j0, j1) adds its share of perspectives j0..j1 - 1 of distribution u.  The
// total is in wave 0.
template <int WAVES, class Add>
__device__ __forceinline__ double idw_sum(uint32_t nb, uint32_t np, int lane, uint32_t wave, uint32_t states,
                                          uint32_t subs, Add&& add) {
    __shared__ double s_num[2][WAVES][64], s_den[2][WAVES][64], s_num0[2][WAVES][64];
    __shared__ uint32_t s_cnt0[2][WAVES][64];
    double g_sum = 0.0;                          // of the distributions this wave sums up
    for (uint32_t u0 = 0; u0 < nb; u0 += WAVES) {
        const uint32_t count = min(nb - u0, (uint32_t)WAVES), row = count * np;
        const uint32_t share = (row + WAVES - 1) / WAVES;
        uint32_t i = min(wave * share, row);
        const uint32_t end = min(i + share, row);
        for (uint32_t e = 0; i < end; ++e) {
            const uint32_t u = i / np, j0 = i - u * np, j1 = min(np, end - u * np);
            IdwSums a;
            add(a, u0 + u, j0, j1);
            s_num[e][wave][lane] = a.num;
            s_den[e][wave][lane] = a.den;
            s_num0[e][wave][lane] = a.num0;
            s_cnt0[e][wave][lane] = a.cnt0;
            i += j1 - j0;
        }
        __syncthreads();
        if (wave < count) {
            const uint32_t first = wave * np / share, last = (wave * np + np - 1) / share;
            double n = 0.0, d = 0.0, n0 = 0.0;
            uint32_t c0 = 0;
            for (uint32_t w = first; w <= last; ++w) {
                const uint32_t e = wave - w * share / np;
                n += s_num[e][w][lane];
                d += s_den[e][w][lane];
                n0 += s_num0[e][w][lane];
                c0 += s_cnt0[e][w][lane];
            }
            if (subs > 1u) {
                double tn = 0.0, td = 0.0, tn0 = 0.0;
                uint32_t tc0 = 0;
                for (uint32_t k = 0; k < subs; ++k) {
                    const int from = (int)(k * states + (uint32_t)lane % states);
                    tn += __shfl(n, from, 64);
                    td += __shfl(d, from, 64);
                    tn0 += __shfl(n0, from, 64);
                    tc0 += __shfl(c0, from, 64);
                }
                n = tn;
                d = td;
                n0 = tn0;
                c0 = tc0;
            }
            const double g_u = c0 ? n0 / (double)c0 : n / d;
            g_sum += g_u / (double)(nb - u0 - wave);
        }
        __syncthreads();                         // the partial sums are read
    }
    s_num[0][wave][lane] = g_sum;
    __syncthreads();
    g_sum = 0.0;
    if (wave == 0u) {
#pragma unroll
        for (int w = 0; w < WAVES; ++w) g_sum += s_num[0][w][lane];
    }
    return g_sum;
}

template <bool P_TWO, int WAVES>
__global__ __launch_bounds__(WAVES * 64) void idw_query_kernel(
    const float* __restrict__ id_pos, const float* __restrict__ id_ig, uint32_t nb, uint32_t np, float p,
    const float* __restrict__ poses, uint32_t q_count, uint32_t tile, uint32_t steps, float px, float py,
    float pz, float tan_h, float tan_v, float w_i, float eps, float* __restrict__ g_out,
    float* __restrict__ o_out, float* __restrict__ cost) {
    __shared__ double s_term[64];
    const int lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t q = blockIdx.x * tile + (uint32_t)lane;
    const bool active = (uint32_t)lane < tile && q < q_count;
    float tx = 0.0f, ty = 0.0f, tz = 0.0f;
    if (active) {
        tx = poses[12 * (size_t)q + 9];
        ty = poses[12 * (size_t)q + 10];
        tz = poses[12 * (size_t)q + 11];
    }
    const float half_neg_p = -0.5f * p;
    const double g = idw_sum<WAVES>(nb, np, lane, wave, 64u, 1u, [&](IdwSums& a, uint32_t u, uint32_t j0, uint32_t j1) {
        for (uint32_t r = j0; r < j1; r += kCostRun) {
            const uint32_t end = min(r + (uint32_t)kCostRun, j1);
            uint32_t j = r;
            // kCostBlock perspectives' scalar loads in flight together, and
            // one test for a coincident one among them
            for (; j + kCostBlock <= end; j += kCostBlock) {
                const float* pp = id_pos + 3 * ((size_t)u * np + j);
                const float* gp = id_ig + ((size_t)u * np + j);
                float e[3 * kCostBlock], ig[kCostBlock], d2[kCostBlock];
#pragma unroll
                for (int k = 0; k < 3 * kCostBlock; ++k) e[k] = pp[k];
#pragma unroll
                for (int k = 0; k < kCostBlock; ++k) ig[k] = gp[k];
                float least = __builtin_inff();
#pragma unroll
                for (int k = 0; k < kCostBlock; ++k) {
                    const float dx = e[3 * k] - tx, dy = e[3 * k + 1] - ty, dz = e[3 * k + 2] - tz;
                    d2[k] = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
                    least = fminf(least, d2[k]);
                }
                if (least > 0.0f) {
#pragma unroll
                    for (int k = 0; k < kCostBlock; ++k) idw_weigh<P_TWO>(a, d2[k], ig[k], half_neg_p);
                } else {
#pragma unroll 1
                    for (int k = 0; k < kCostBlock; ++k)
                        idw_pair<P_TWO>(a, pp[3 * k] - tx, pp[3 * k + 1] - ty, pp[3 * k + 2] - tz, gp[k], half_neg_p);
                }
            }
            for (; j < end; ++j) {
                const size_t s = (size_t)u * np + j;
                idw_pair<P_TWO>(a, id_pos[3 * s] - tx, id_pos[3 * s + 1] - ty, id_pos[3 * s + 2] - tz, id_ig[s],
                                half_neg_p);
            }
            a.join();
        }
    });
    if (wave != 0) return;
    state_outputs(active, q, (float)g, tx, ty, tz, lane, tile / steps, steps, poses, q_count, px, py, pz, tan_h, tan_v,
                  w_i, eps, g_out, o_out, cost, s_term);
}

// The same for calls whose tiles would leave compute units idle: a workgroup
// takes one horizon (of at most 32 states), its lanes being `subs` copies of
// the states that take different perspectives.  A wave stages 64 of its
// perspectives at a time in LDS, the next ones' loads in flight meanwhile (read by every
// lane from memory they would be bound by the address path).  256 x 20 states
// against 10 x 500 perspectives: 29 us in whole tiles, 17 so.
template <bool P_TWO>
__global__ __launch_bounds__(kCostWaves * 64) void idw_horizon_kernel(
    const float* __restrict__ id_pos, const float* __restrict__ id_ig, uint32_t nb, uint32_t np, float p,
    const float* __restrict__ poses, uint32_t q_count, uint32_t steps, uint32_t subs, float px, float py, float pz,
    float tan_h, float tan_v, float w_i, float eps, float* __restrict__ g_out, float* __restrict__ o_out,
    float* __restrict__ cost) {
    __shared__ float4 s_persp[kCostWaves][64];
    __shared__ double s_term[64];
    const int lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t sub = (uint32_t)lane / steps, state = (uint32_t)lane - sub * steps;
    const uint32_t q = blockIdx.x * steps + state;
    const bool active = sub < subs;              // the grid has whole horizons only
    float tx = 0.0f, ty = 0.0f, tz = 0.0f;
    if (active) {
        tx = poses[12 * (size_t)q + 9];
        ty = poses[12 * (size_t)q + 10];
        tz = poses[12 * (size_t)q + 11];
    }
    const float half_neg_p = -0.5f * p;
    const double g = idw_sum<kCostWaves>(nb, np, lane, wave, steps, subs, [&](IdwSums& a, uint32_t u, uint32_t j0, uint32_t j1) {
        float4 next = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        auto fetch = [&](uint32_t j) {
            if (j < j1) {
                const size_t s = (size_t)u * np + j;
                next = make_float4(id_pos[3 * s], id_pos[3 * s + 1], id_pos[3 * s + 2], id_ig[s]);
            }
        };
        fetch(j0 + (uint32_t)lane);
        for (uint32_t j = j0; j < j1; j += 64u) {
            s_persp[wave][lane] = next;
            __builtin_amdgcn_wave_barrier();
            fetch(j + 64u + (uint32_t)lane);
            const uint32_t len = min(j1 - j, 64u);
            if (active) {
                uint32_t k = sub;
                // one test for a coincident perspective among kCostBlock
                for (; k + (kCostBlock - 1) * subs < len; k += kCostBlock * subs) {
                    float4 v[kCostBlock];
                    float d2[kCostBlock], least = __builtin_inff();
#pragma unroll
                    for (int b = 0; b < kCostBlock; ++b) v[b] = s_persp[wave][k + b * subs];
#pragma unroll
                    for (int b = 0; b < kCostBlock; ++b) {
                        const float dx = v[b].x - tx, dy = v[b].y - ty, dz = v[b].z - tz;
                        d2[b] = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
                        least = fminf(least, d2[b]);
                    }
                    if (least > 0.0f) {
#pragma unroll
                        for (int b = 0; b < kCostBlock; ++b) idw_weigh<P_TWO>(a, d2[b], v[b].w, half_neg_p);
                    } else {
#pragma unroll
                        for (int b = 0; b < kCostBlock; ++b)
                            idw_pair<P_TWO>(a, v[b].x - tx, v[b].y - ty, v[b].z - tz, v[b].w, half_neg_p);
                    }
                }
                for (; k < len; k += subs) {
                    const float4 v = s_persp[wave][k];
                    idw_pair<P_TWO>(a, v.x - tx, v.y - ty, v.z - tz, v.w, half_neg_p);
                }
            }
            a.join();                            // at most 32 pairs a run
            __builtin_amdgcn_wave_barrier();
        }
    });
    if (wave != 0) return;
    state_outputs(active && sub == 0u, q, (float)g, tx, ty, tz, lane, 1u, steps, poses, q_count, px, py, pz, tan_h, tan_v,
                  w_i, eps, g_out, o_out, cost, s_term);
}

// Cost of horizons of more than 64 states.
__global__ __launch_bounds__(256) void horizon_cost_kernel(const float* __restrict__ g,
                                                           const float* __restrict__ o, uint32_t h,
                                                           uint32_t k, float w_i, float eps,
                                                           float* __restrict__ cost) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= h) return;
    double s = 0.0;
    for (uint32_t j = 0; j < k; ++j) {
        const size_t q = (size_t)i * k + j;
        s += (double)w_i / ((double)o[q] * (double)g[q] + (double)eps);
    }
    cost[i] = (float)s;
}

// One horizon per workgroup pays while all of them run at once and each has
// enough perspectives to split: 256 x 20 states against 10 x 500 17 us where
// tiles take 29, 300 x 20 28 and 28 (32 and 35 for p = 1), 512 x 20 31 and 30, 16 x 1 18 and 27; with 1 x 500 or fewer, or distributions of
// 16 perspectives, which leave most lanes of a wave's chunk of 64 idle, it takes
// longer (256 x 1: 9.7 and 7.2; 64 x 16 perspectives 82 and 11).
static bool horizon_alone(uint32_t h, uint32_t k, uint32_t nb, uint32_t np, int cu_count) {
    return k <= 32 && 2u * h <= 3u * (uint32_t)cu_count && np >= 128 && (uint64_t)nb * np >= 1000;
}

hipError_t launch_eval_cost(const float* id_pos, const float* id_ig, uint32_t nb, uint32_t np, float p,
                            const float* poses, uint32_t h, uint32_t k, const float poi[3], float tan_h,
                            float tan_v, float w_i, float eps, float* g_out, float* o_out, float* cost,
                            int cu_count, hipStream_t s) {
    const uint32_t q = h * k;
    const uint32_t tile = cost_tile(k);
    const uint32_t tiles = (q + tile - 1) / tile;
    auto go = [&](auto kernel, int waves) {
        hipLaunchKernelGGL(kernel, dim3(tiles), dim3(waves * 64), 0, s, id_pos, id_ig, nb, np,
                           p, poses, q, tile, k, poi[0], poi[1], poi[2], tan_h, tan_v, w_i, eps, g_out, o_out,
                           k <= 64 ? cost : nullptr);
    };
    if (horizon_alone(h, k, nb, np, cu_count)) {
        auto one = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(h), dim3(kCostWaves * 64), 0, s, id_pos, id_ig, nb, np, p, poses, q, k,
                               64 / k, poi[0], poi[1], poi[2], tan_h, tan_v, w_i, eps, g_out, o_out, cost);
        };
        if (p == 2.0f) one(idw_horizon_kernel<true>);
        else one(idw_horizon_kernel<false>);
        return hipGetLastError();
    }
    const bool two = p == 2.0f;
    switch (query_waves(tiles, nb, np, cu_count)) {
    case 1: two ? go(idw_query_kernel<true, 1>, 1) : go(idw_query_kernel<false, 1>, 1); break;
    case 2: two ? go(idw_query_kernel<true, 2>, 2) : go(idw_query_kernel<false, 2>, 2); break;
    case 4: two ? go(idw_query_kernel<true, 4>, 4) : go(idw_query_kernel<false, 4>, 4); break;
    case 8: two ? go(idw_query_kernel<true, 8>, 8) : go(idw_query_kernel<false, 8>, 8); break;
    default: two ? go(idw_query_kernel<true, 16>, 16) : go(idw_query_kernel<false, 16>, 16);
    }
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !cost || k <= 64) return e;
    hipLaunchKernelGGL(horizon_cost_kernel, dim3((h + 255) / 256), dim3(256), 0, s, g_out, o_out, h, k, w_i,
                       eps, cost);
    return hipGetLastError();
}

}  // namespace nbt
