// cost.hip -- planner-side IG terms of Sec. IV for many candidate horizons.
//
//   G(x)  Eq. 3: inverse-distance weighting of the perspectives' IG, summed
//         over the N_B buffered information distributions with weight
//         1/(N_B - u) (u = 0 oldest);
//   O(x)  cosine between the camera's viewing axis and the direction to the
//         PoI, 0 when the PoI is outside the field of view;
//   c_I   sum over a horizon's states of w_I / (O G + eps).
// ALU-bound: about 10 VALU operations (one of them a quarter-rate reciprocal)
// per (state, perspective) pair.  One lane per state and 16 waves per
// workgroup that split every distribution's perspectives: a planner's call
// has few states (256 horizons of 20 states are 85 workgroups), so the
// parallelism has to come from the perspectives.  A perspective's position
// and IG are the same for the whole wave and are read through scalar loads.
// 256 x 20 states against 10 x 500 perspectives: 671 us with one thread per
// state over all perspectives (20 workgroups of 4 waves on the chip) and 5 us
// for the horizons' sum in a launch of its own, 29 us a call now, all included.
#include "internal.hpp"

namespace nbt {

constexpr int kCostWaves = 16;
constexpr int kCostRun = 64;     // pairs summed in binary32 before they join the binary64 sum
constexpr int kCostBlock = 8;    // perspectives whose scalar loads are in flight together

// States of one workgroup: whole horizons where one fits 64 lanes (the
// workgroup then also sums their cost), else 64 states.
static uint32_t cost_tile(uint32_t steps) { return steps <= 64 ? 64 / steps * steps : 64; }

template <bool P_TWO>
__global__ __launch_bounds__(kCostWaves * 64) void idw_query_kernel(
    const float* __restrict__ id_pos, const float* __restrict__ id_ig, uint32_t nb, uint32_t np, float p,
    const float* __restrict__ poses, uint32_t q_count, uint32_t tile, uint32_t steps, float px, float py,
    float pz, float tan_h, float tan_v, float w_i, float eps, float* __restrict__ g_out,
    float* __restrict__ o_out, float* __restrict__ cost) {
    // partial sums of one distribution, two of them in turn: while one wave
    // reduces distribution u, the others go on to u + 1
    __shared__ double s_num[2][kCostWaves][64], s_den[2][kCostWaves][64], s_num0[2][kCostWaves][64];
    __shared__ uint32_t s_cnt0[2][kCostWaves][64];
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
    const uint32_t share = (np + kCostWaves - 1) / kCostWaves;
    const uint32_t j0 = min(wave * share, np), j1 = min(j0 + share, np);
    double g_sum = 0.0;                      // of the distributions this wave reduces
    for (uint32_t u = 0; u < nb; ++u) {
        double num = 0.0, den = 0.0, num0 = 0.0;
        uint32_t cnt0 = 0;
        for (uint32_t r = j0; r < j1; r += kCostRun) {
            float fnum = 0.0f, fden = 0.0f;
            const uint32_t end = min(r + (uint32_t)kCostRun, j1);
            auto weigh = [&](float d2, float ig) {
                const float w = P_TWO ? __builtin_amdgcn_rcpf(d2) : __builtin_powf(d2, half_neg_p);
                fnum = __builtin_fmaf(ig, w, fnum);
                fden += w;
            };
            auto pair = [&](float dx, float dy, float dz, float d2, float ig) {
                if (dx == 0.0f && dy == 0.0f && dz == 0.0f) {
                    // exactly on the perspective: counts instead of weighing
                    num0 += (double)ig;
                    ++cnt0;
                } else {
                    weigh(d2, ig);
                }
            };
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
                    for (int k = 0; k < kCostBlock; ++k) weigh(d2[k], ig[k]);
                } else {
#pragma unroll 1
                    for (int k = 0; k < kCostBlock; ++k) {
                        const float dx = pp[3 * k] - tx, dy = pp[3 * k + 1] - ty, dz = pp[3 * k + 2] - tz;
                        pair(dx, dy, dz, __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)), gp[k]);
                    }
                }
            }
            for (; j < end; ++j) {
                const size_t s = (size_t)u * np + j;
                const float dx = id_pos[3 * s] - tx, dy = id_pos[3 * s + 1] - ty, dz = id_pos[3 * s + 2] - tz;
                pair(dx, dy, dz, __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)), id_ig[s]);
            }
            num += (double)fnum;
            den += (double)fden;
        }
        const uint32_t b = u & 1u;
        s_num[b][wave][lane] = num;
        s_den[b][wave][lane] = den;
        s_num0[b][wave][lane] = num0;
        s_cnt0[b][wave][lane] = cnt0;
        __syncthreads();
        if (wave == u % kCostWaves) {
            num = den = num0 = 0.0;
            cnt0 = 0;
#pragma unroll
            for (int w = 0; w < kCostWaves; ++w) {
                num += s_num[b][w][lane];
                den += s_den[b][w][lane];
                num0 += s_num0[b][w][lane];
                cnt0 += s_cnt0[b][w][lane];
            }
            const double g_u = cnt0 ? num0 / (double)cnt0 : num / den;
            g_sum += g_u / (double)(nb - u);
        }
    }
    __syncthreads();                         // the last distribution's partial sums are read
    s_num[0][wave][lane] = g_sum;
    __syncthreads();
    if (wave != 0) return;
    g_sum = 0.0;
#pragma unroll
    for (int w = 0; w < kCostWaves; ++w) g_sum += s_num[0][w][lane];
    const float g = (float)g_sum;
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
    // every horizon of the tile: its states' terms in order
    s_term[lane] = (double)w_i / ((double)o * (double)g + (double)eps);
    __builtin_amdgcn_wave_barrier();
    const uint32_t h = blockIdx.x * (tile / steps) + (uint32_t)lane;
    if ((uint32_t)lane < tile / steps && h < q_count / steps) {
        double s = 0.0;
        for (uint32_t j = 0; j < steps; ++j) s += s_term[(uint32_t)lane * steps + j];
        cost[h] = (float)s;
    }
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

hipError_t launch_eval_cost(const float* id_pos, const float* id_ig, uint32_t nb, uint32_t np, float p,
                            const float* poses, uint32_t h, uint32_t k, const float poi[3], float tan_h,
                            float tan_v, float w_i, float eps, float* g_out, float* o_out, float* cost,
                            hipStream_t s) {
    const uint32_t q = h * k;
    const uint32_t tile = cost_tile(k);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((q + tile - 1) / tile), dim3(kCostWaves * 64), 0, s, id_pos, id_ig, nb, np,
                           p, poses, q, tile, k, poi[0], poi[1], poi[2], tan_h, tan_v, w_i, eps, g_out, o_out,
                           k <= 64 ? cost : nullptr);
    };
    if (p == 2.0f) go(idw_query_kernel<true>);
    else go(idw_query_kernel<false>);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !cost || k <= 64) return e;
    hipLaunchKernelGGL(horizon_cost_kernel, dim3((h + 255) / 256), dim3(256), 0, s, g_out, o_out, h, k, w_i,
                       eps, cost);
    return hipGetLastError();
}

}  // namespace nbt
