// map_encode.hip -- occupancy probabilities -> device-resident encoded map.
//
// Each voxel is classified once (Occupied if P > occ, Free if P < free,
// Unknown otherwise) and stored as its Eq. 2 gain (1-P, P or 1) in float32
// bits, with the sign bit set for Occupied.  A one-voxel border of sentinel
// words surrounds the map (and fills the tile padding of the column orders).  The
// walk then needs one 4-byte gather and one signed compare per voxel: no
// probability, no threshold and no bounds test is evaluated per step.
// Streaming kernel, about 8 B per voxel.
#include "internal.hpp"

namespace nbt {

// Word of a voxel with probability p.
__device__ __forceinline__ uint32_t encode_prob(float p, float occ_thr, float free_thr, bool& any_bad) {
    if (!(p >= 0.0f && p <= 1.0f)) {          // also rejects NaN
        any_bad = true;
        return kGainOne;
    }
    if (p > occ_thr) return __float_as_uint(1.0f - p) | kOccBit;
    if (p < free_thr) return __float_as_uint(p) & ~kOccBit;    // -0.0 is stored as +0.0
    return kGainOne;
}

// The palette of the map being encoded, copied to LDS: a word's code is the
// slot it is found in, from a hash of the word on.  The sampling pass has
// entered the words of kSampleCount voxels; a word it missed takes the first free slot by
// compare-and-swap on the palette in memory, so all workgroups agree (the
// copy only ever lags behind), one lane of a wave at a time: the others
// usually wait for the same word.  A search of kCodeProbes slots without
// success sets the overflow flag, and from then on no code matters.
constexpr uint32_t kCodeProbes = 24;

struct Palette {
    uint32_t key[kCodes];
    uint32_t over;
};

__device__ __forceinline__ uint32_t code_slot(uint32_t w) {
    const uint32_t h = (w * 0x9E3779B1u) >> 24;
    return h < 2u ? 2u : h;
}
__device__ __forceinline__ uint32_t next_slot(uint32_t slot) { return slot + 1u < kCodes ? slot + 1u : 2u; }

// False when the map has no codes, or is known to have too many words for them.
__device__ __forceinline__ bool palette_load(Palette& s, const DevMap& m) {
    if (!m.codes) return false;
    for (uint32_t k = threadIdx.x; k <= kCodes; k += blockDim.x) (k < kCodes ? s.key[k] : s.over) = m.palette[k];
    __syncthreads();
    return s.over == 0u;
}

__device__ __forceinline__ uint32_t find_code(Palette& s, const DevMap& m, uint32_t w) {
    if (w == kSentinel) return 0u;
    if (w == kGainOne) return 1u;
    uint32_t slot = code_slot(w);
    for (uint32_t n = 0; n < kCodeProbes && !s.over;) {
        const uint32_t k = s.key[slot];
        if (k == w) return slot;
        if (k == kCodeFree) {
            if ((threadIdx.x & 63u) == (uint32_t)__builtin_ctzll(__ballot(1))) {
                const uint32_t old = atomicCAS(const_cast<uint32_t*>(m.palette) + slot, kCodeFree, w);
                s.key[slot] = old == kCodeFree ? w : old;
            }
            continue;                            // look at the slot again
        }
        slot = next_slot(slot);
        ++n;
    }
    s.over = 1u;
    atomicOr(const_cast<uint32_t*>(m.palette) + kCodes, 1u);
    return 0u;
}

// Starts the palette of a new encoding from kSampleCount voxels spread over
// the grid: one workgroup, which reads them at once and enters their words in
// LDS.  A map of many different probabilities overflows here, and its
// encoding then spends nothing on codes.
constexpr uint32_t kSampleThreads = 1024, kSampleEach = 4, kSampleCount = kSampleThreads * kSampleEach;

__global__ __launch_bounds__(kSampleThreads) void palette_sample_kernel(const float* __restrict__ prob, DevMap m,
                                                                        float occ_thr, float free_thr,
                                                                        uint32_t* __restrict__ palette) {
    __shared__ uint32_t s_key[kCodes];
    __shared__ uint32_t s_over;
    const uint32_t t = threadIdx.x;
    if (t < kCodes) s_key[t] = t == 0u ? kSentinel : t == 1u ? kGainOne : kCodeFree;
    if (t == 0u) s_over = 0u;
    const uint64_t total = (uint64_t)m.nx * (uint64_t)m.ny * (uint64_t)m.nz;
    float p[kSampleEach];
#pragma unroll
    for (uint32_t k = 0; k < kSampleEach; ++k) {
        // a low-discrepancy walk over the grid (the golden ratio's multiples)
        const uint32_t h = (k * kSampleThreads + t) * 0x9E3779B9u;
        p[k] = prob[(uint64_t)h * total >> 32];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < kSampleEach; ++k) {
        bool bad = false;
        const uint32_t w = encode_prob(p[k], occ_thr, free_thr, bad);
        if (w == kGainOne) continue;
        uint32_t slot = code_slot(w), n = 0;
        for (; n < kCodeProbes && !s_over; ++n) {
            uint32_t old = s_key[slot];
            if (old == kCodeFree) old = atomicCAS(&s_key[slot], kCodeFree, w);
            if (old == kCodeFree || old == w) break;
            slot = next_slot(slot);
        }
        if (n == kCodeProbes) s_over = 1u;
    }
    __syncthreads();
    if (t < kCodes) palette[t] = s_key[t];
    if (t == 0u) palette[kCodes] = s_over;
}

// Padded coordinates of stored word idx.
__device__ __forceinline__ void word_coords(const DevMap& m, uint32_t idx, uint32_t& X, uint32_t& Y, uint32_t& Z) {
    if (m.tl == 0) {
        X = idx % (uint32_t)m.px;
        const uint32_t yz = idx / (uint32_t)m.px;
        Y = yz % (uint32_t)m.py;
        Z = yz / (uint32_t)m.py;
    } else {
        const uint32_t t = (uint32_t)m.tl;
        const uint32_t r = idx >> (2u * t), l = idx & ((1u << (2u * t)) - 1u);
        Z = r % (uint32_t)m.pz;
        const uint32_t tile = r / (uint32_t)m.pz;
        X = ((tile % (uint32_t)m.nbx) << t) + (l & ((1u << t) - 1u));
        Y = ((tile / (uint32_t)m.nbx) << t) + (l >> t);
    }
}

// Bound by memory (4 B read, 4 B written per voxel).  Threads are dealt to the
// padded grid's coordinates, so no index is divided (one thread per stored
// word spent most of its time on four divisions per word: 50 us for 256^3 in
// 4x4 columns, 33 now; 47 and 31 in linear order; with the codes 54 and 48,
// 7 of them for the sampling pass).
//
// Every thread steps through LAYERS layers, their loads in flight together: 4,
// or 1 for a map too small to fill the chip so (64^3 in columns: 6.2 us at 8 layers,
// 3.0 at 1).
//
// Linear order: a workgroup takes 64 words in x of 4 rows of y.
constexpr int kEncodeLayers = 4;
constexpr uint64_t kEncodeGroups = 2048;         // workgroups from which on they step through 4 layers

template <int LAYERS>
__global__ __launch_bounds__(256) void encode_linear_kernel(const float* __restrict__ prob,
                                                            uint32_t* __restrict__ enc, DevMap m, float occ_thr,
                                                            float free_thr, unsigned int* __restrict__ bad) {
    const int X = (int)(blockIdx.x * 64u + (threadIdx.x & 63u));
    const int Y = (int)(blockIdx.y * 4u + (threadIdx.x >> 6));
    const int Z0 = (int)blockIdx.z * LAYERS;
    __shared__ Palette s_pal;
    const bool coded = palette_load(s_pal, m);
    if (X >= m.px || Y >= m.py) return;
    const bool xy = X > 0 && Y > 0 && X <= m.nx && Y <= m.ny;
    float p[LAYERS];
#pragma unroll
    for (int k = 0; k < LAYERS; ++k) {
        const int Z = Z0 + k;
        p[k] = xy && Z > 0 && Z <= m.nz ? prob[((size_t)(Z - 1) * m.ny + (size_t)(Y - 1)) * m.nx + (size_t)(X - 1)]
                                        : 0.0f;
    }
    bool any_bad = false;
    uint32_t known = kSentinel, code = 0u;       // the last word looked up
#pragma unroll
    for (int k = 0; k < LAYERS; ++k) {
        const int Z = Z0 + k;
        if (Z >= m.pz) break;
        const bool in = xy && Z > 0 && Z <= m.nz;
        const uint32_t w = in ? encode_prob(p[k], occ_thr, free_thr, any_bad) : kSentinel;
        enc[((size_t)Z * m.py + (size_t)Y) * m.px + (size_t)X] = w;
        if (coded) {
            if (w != known) code = find_code(s_pal, m, known = w);
            const_cast<uint8_t*>(m.codes)[code_offset(m.csy, m.csz, (uint32_t)X, (uint32_t)Y, (uint32_t)Z)] =
                (uint8_t)code;
        }
    }
    if (any_bad) atomicOr(bad, 1u);
}

// Column orders: a thread writes pieces of four consecutive stored words (16
// bytes): four x of one row of a tile (a whole layer of a 2x2 tile).  A wave
// takes 64 consecutive pieces of one layer along x, then y, so that it reads
// whole row segments of the probabilities and writes whole tile rows, and
// steps through the layers, whose tile rows continue one another.
template <int TL, int LAYERS>
__global__ __launch_bounds__(256) void encode_column_kernel(const float* __restrict__ prob,
                                                            uint32_t* __restrict__ enc, DevMap m, float occ_thr,
                                                            float free_thr, unsigned int* __restrict__ bad) {
    constexpr int T = 1 << TL;
    constexpr int kRows = TL == 1 ? 1 : T;                 // pieces of a tile along y
    constexpr int kCols = TL == 3 ? 2 : 1;                 // and along x
    const int lane = (int)(threadIdx.x & 63u), wave = (int)(threadIdx.x >> 6);
    // 64 / kRows pieces along x, kRows along y: one row of tiles per wave
    const int px = (int)blockIdx.x * (64 / kRows) + lane % (64 / kRows), row = lane / (64 / kRows);
    const int tx = px / kCols, ty = (int)blockIdx.y;
    const int Z0 = ((int)blockIdx.z * 4 + wave) * LAYERS;
    __shared__ Palette s_pal;
    const bool coded = palette_load(s_pal, m);
    // (of a pair of 2x2 tiles one may lie beyond the grid: it helps to write the codes)
    const bool stored = tx < m.nbx;
    if (TL == 1 ? (tx & ~1) >= m.nbx : !stored) return;
    const int X = tx * T + (px % kCols) * 4, Y = ty * T + row;
    uint32_t* out = enc + ((size_t)(ty * m.nbx + tx) * m.pz << (2 * TL)) + row * T + (px % kCols) * 4;
    bool any_bad = false;
    uint32_t known = kSentinel, code = 0u;       // the last word looked up
    float p[LAYERS][4];
    // the piece's voxels: four x of row Y, or for 2x2 tiles two x of rows Y and Y + 1
    auto at = [&](int e, int& x, int& y) {
        x = X - 1 + (TL == 1 ? (e & 1) : e);
        y = Y - 1 + (TL == 1 ? (e >> 1) : 0);
        return (unsigned)x < (unsigned)m.nx && (unsigned)y < (unsigned)m.ny;
    };
#pragma unroll
    for (int k = 0; k < LAYERS; ++k) {
        const int z = Z0 + k - 1;
        const bool in_z = (unsigned)z < (unsigned)m.nz;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int x, y;
            p[k][e] = at(e, x, y) && in_z ? prob[((size_t)z * m.ny + (size_t)y) * m.nx + (size_t)x] : 0.0f;
        }
    }
    uint32_t codes[LAYERS];                      // the piece's four codes per layer
#pragma unroll
    for (int k = 0; k < LAYERS; ++k) {
        const int Z = Z0 + k, z = Z - 1;
        codes[k] = 0u;
        if (Z >= m.pz) continue;
        const bool in_z = (unsigned)z < (unsigned)m.nz;
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int x, y;
            w[e] = at(e, x, y) && in_z ? encode_prob(p[k][e], occ_thr, free_thr, any_bad) : kSentinel;
        }
        if (stored) *reinterpret_cast<uint4*>(out + ((size_t)Z << (2 * TL))) = make_uint4(w[0], w[1], w[2], w[3]);
        if (coded) {
            if (w[0] == known && w[1] == known && w[2] == known && w[3] == known) {
                codes[k] = code * 0x01010101u;   // most pieces of a map continue the one below
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (w[e] != known) code = find_code(s_pal, m, known = w[e]);
                    codes[k] |= code << (8 * e);
                }
            }
        }
    }
    if (coded) {
        uint8_t* co = const_cast<uint8_t*>(m.codes);
        auto place = [&](int y, int Z) { return co + code_offset(m.csy, m.csz, (uint32_t)X, (uint32_t)y, (uint32_t)Z); };
        if constexpr (LAYERS == 1) {
            if (Z0 < m.pz) {
                if constexpr (TL == 1) {         // two codes of each of two rows
                    *reinterpret_cast<uint16_t*>(place(Y, Z0)) = (uint16_t)codes[0];
                    *reinterpret_cast<uint16_t*>(place(Y + 1, Z0)) = (uint16_t)(codes[0] >> 16);
                } else {
                    *reinterpret_cast<uint32_t*>(place(Y, Z0)) = codes[0];
                }
            }
        } else if constexpr (TL == 1) {
            // two tiles of two layers are 16 consecutive codes: their lanes take every
            // other pair of layers (see below)
#pragma unroll
            for (int k = 0; k < LAYERS; k += 2) {
                const uint32_t o0 = (uint32_t)__shfl_xor((int)codes[k], 1, 64);
                const uint32_t o1 = (uint32_t)__shfl_xor((int)codes[k + 1], 1, 64);
                const int odd = tx & 1;
                if (odd != (k / 2 & 1) || Z0 + k >= m.pz) continue;
                const uint32_t a0 = odd ? o0 : codes[k], b0 = odd ? codes[k] : o0;
                const uint32_t a1 = odd ? o1 : codes[k + 1], b1 = odd ? codes[k + 1] : o1;
                *reinterpret_cast<uint4*>(place(Y, Z0 + k) - 2 * odd) =
                    make_uint4((a0 & 0xFFFFu) | b0 << 16, a0 >> 16 | (b0 & 0xFFFF0000u), (a1 & 0xFFFFu) | b1 << 16,
                               a1 >> 16 | (b1 & 0xFFFF0000u));
            }
        } else {
            // two rows of two layers are 16 consecutive codes: the lanes of a pair of
            // rows exchange theirs and take every other pair of layers (the last
            // one's second layer may lie in the padding of Z to whole blocks)
#pragma unroll
            for (int k = 0; k < LAYERS; k += 2) {
                const uint32_t o0 = (uint32_t)__shfl_xor((int)codes[k], 64 / kRows, 64);
                const uint32_t o1 = (uint32_t)__shfl_xor((int)codes[k + 1], 64 / kRows, 64);
                const int odd = row & 1;
                if (odd != (k / 2 & 1) || Z0 + k >= m.pz) continue;
                *reinterpret_cast<uint4*>(place(Y - odd, Z0 + k)) =
                    odd ? make_uint4(o0, codes[k], o1, codes[k + 1]) : make_uint4(codes[k], o0, codes[k + 1], o1);
            }
        }
    }
    if (any_bad) atomicOr(bad, 1u);
}

// One thread per destination word: the word of the same padded voxel in the
// source order (the sentinel for the padding of whole tiles).
__global__ __launch_bounds__(256) void relayout_kernel(const uint32_t* __restrict__ src, DevMap sm,
                                                       uint32_t* __restrict__ dst, DevMap dm) {
    const uint32_t total = dm.bytes / 4u;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t idx = blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
        uint32_t X, Y, Z;
        word_coords(dm, idx, X, Y, Z);
        uint32_t w = kSentinel;
        if (X < (uint32_t)dm.px && Y < (uint32_t)dm.py && Z < (uint32_t)dm.pz)
            w = src[voxel_offset(sm, (int)X - 1, (int)Y - 1, (int)Z - 1) / 4u];
        dst[idx] = w;
    }
}

hipError_t launch_relayout(const DevMap& src, uint32_t* dst, const DevMap& dstm, hipStream_t s) {
    const uint64_t total = dstm.bytes / 4u;
    uint64_t blocks = (total + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(relayout_kernel, dim3((unsigned)blocks), dim3(256), 0, s, src.enc, src, dst, dstm);
    return hipGetLastError();
}

template <int TL>
static void launch_encode_column(const float* prob, uint32_t* enc, const DevMap& m, float occ_thr, float free_thr,
                                 unsigned int* bad_flag, hipStream_t s) {
    constexpr unsigned kAlongX = 64 / (TL == 1 ? 1 : 1 << TL);
    const unsigned pieces = (unsigned)m.nbx * (TL == 3 ? 2u : 1u);
    const unsigned gx = (pieces + kAlongX - 1) / kAlongX, gy = (unsigned)m.nby, pz = (unsigned)m.pz;
    const unsigned gz = (pz + 4 * kEncodeLayers - 1) / (4 * kEncodeLayers);
    if ((uint64_t)gx * gy * gz >= kEncodeGroups)
        hipLaunchKernelGGL((encode_column_kernel<TL, kEncodeLayers>), dim3(gx, gy, gz), dim3(256), 0, s, prob, enc, m,
                           occ_thr, free_thr, bad_flag);
    else
        hipLaunchKernelGGL((encode_column_kernel<TL, 1>), dim3(gx, gy, (pz + 3) / 4), dim3(256), 0, s, prob, enc, m,
                           occ_thr, free_thr, bad_flag);
}

hipError_t launch_encode_map(const float* prob, uint32_t* enc, const DevMap& m, float occ_thr,
                             float free_thr, unsigned int* bad_flag, hipStream_t s) {
    if (m.codes) {
        hipLaunchKernelGGL(palette_sample_kernel, dim3(1), dim3(kSampleThreads), 0, s, prob, m, occ_thr, free_thr,
                           const_cast<uint32_t*>(m.palette));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    switch (m.tl) {
    case 1: launch_encode_column<1>(prob, enc, m, occ_thr, free_thr, bad_flag, s); break;
    case 2: launch_encode_column<2>(prob, enc, m, occ_thr, free_thr, bad_flag, s); break;
    case 3: launch_encode_column<3>(prob, enc, m, occ_thr, free_thr, bad_flag, s); break;
    default: {
        const unsigned gx = ((unsigned)m.px + 63) / 64, gy = ((unsigned)m.py + 3) / 4, pz = (unsigned)m.pz;
        const unsigned gz = (pz + kEncodeLayers - 1) / kEncodeLayers;
        if ((uint64_t)gx * gy * gz >= kEncodeGroups)
            hipLaunchKernelGGL(encode_linear_kernel<kEncodeLayers>, dim3(gx, gy, gz), dim3(256), 0, s, prob, enc, m,
                               occ_thr, free_thr, bad_flag);
        else
            hipLaunchKernelGGL(encode_linear_kernel<1>, dim3(gx, gy, pz), dim3(256), 0, s, prob, enc, m, occ_thr,
                               free_thr, bad_flag);
    }
    }
    return hipGetLastError();
}

}  // namespace nbt
