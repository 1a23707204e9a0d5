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

// Codes.  The palette in memory is a hash table of the map's words, whose slots
// are the codes; the words that follow it are the overflow flag and the count
// of words entered.  It lives on from one encoding to the next, so an encoding
// usually finds all its words there; a new one takes the first free slot from
// its hash on by compare-and-swap, so all workgroups agree.  A palette of
// kCodeMost words takes no more: the flag is set, and from then on no code
// matters.  Now and then (PaletteStart::again) a pass of one workgroup starts it
// anew from a sample of the grid, which ends an overflow and drops words no longer met.
//
// A workgroup holds the palette as an LDS table of 2048 entries.  A word's hash (an
// odd multiple of it, so one to one) gives its place by the upper 11 bits; the
// entry holds the lower 21, its distance from that place and the code, so it
// names the whole word, and one read and one comparison give the code.  With
// 224 words some 10 % lie one place on and 1 % further; words that crowd so
// that one finds no room within 7 places count as too many.  (At an eighth place a free
// entry, all ones, would pass for that of a word whose lower 21 bits are all ones.)
// Looked up by probing a copy of the palette, with the sampling pass in every encoding,
// 150 words scattered over 320^3 took 296 us and three 104, now 83 and 82.
//
// New words: thousands of workgroups meet them at once, and swaps of one address
// take 15 ns each.  So a workgroup gathers the words it lacks, a thread looks after each, and
// only one workgroup in 64 swaps right away; the others look once more first, or twice or
// three times (256^3 in 4x4 columns with 10 new words 54 us, without 40; 150-250 when
// every wave swapped).  A map fused from one depth image after another, whose words grow from 3 to
// 125 in 16 of them: 57 us an encoding, 80 with eight looks.
constexpr uint32_t kCodeProbes = 24;             // palette slots tried for a new word
constexpr uint32_t kCodeMost = 224;
constexpr uint32_t kTableBits = 11, kTableSize = 1u << kTableBits, kTableFar = (kTableSize >> 8) - 1u;
constexpr uint32_t kSetSize = 256;

struct CodeTable {
    uint32_t entry[kTableSize];
    uint32_t set[kSetSize];                      // words the workgroup lacks
    uint32_t over, lacks[2];                     // of the map when loaded; of a call of find_codes
};

__device__ __forceinline__ uint32_t code_slot(uint32_t w) {
    const uint32_t h = (w * 0x9E3779B1u) >> 24;
    return h < 2u ? 2u : h;
}
__device__ __forceinline__ uint32_t next_slot(uint32_t slot) { return slot + 1u < kCodes ? slot + 1u : 2u; }

// h: the word's hash, one to one; its upper bits are the place, the lower ones the entry's.
__device__ __forceinline__ uint32_t table_hash(uint32_t w) { return w * 0x9E3779B1u; }
__device__ __forceinline__ uint32_t table_at(uint32_t h, uint32_t far) {
    return ((h >> (32u - kTableBits)) + far) & (kTableSize - 1u);
}
// Below 256, the code: the entry found `far` places behind the word's own is the word's.
__device__ __forceinline__ uint32_t table_match(uint32_t entry, uint32_t h, uint32_t far) {
    return entry ^ (h << kTableBits | far << 8);
}

// False: no room near the word's place.
__device__ __forceinline__ bool table_enter(CodeTable& s, uint32_t w, uint32_t code) {
    const uint32_t h = table_hash(w);
    for (uint32_t far = 0; far < kTableFar; ++far) {
        const uint32_t e = h << kTableBits | far << 8 | code;
        const uint32_t old = atomicCAS(&s.entry[table_at(h, far)], kCodeFree, e);
        if (old == kCodeFree || old == e) return true;
    }
    return false;
}

// Fills the table (by the whole workgroup of 256).  False when the map is known to
// have too many words for codes.
__device__ __forceinline__ bool table_load(CodeTable& s, const DevMap& m) {
    const uint32_t t = threadIdx.x;
    const uint32_t w = m.palette[t];
    if (t == 0u) {
        s.over = m.palette[kCodes];              // one reading for all waves
        s.lacks[0] = s.lacks[1] = 0u;
    }
    uint4* e = reinterpret_cast<uint4*>(s.entry);
    for (uint32_t k = t; k < kTableSize / 4u; k += 256u) e[k] = make_uint4(kCodeFree, kCodeFree, kCodeFree, kCodeFree);
    __syncthreads();
    if (s.over) return false;
    if (w != kCodeFree && !table_enter(s, w, t)) atomicOr(const_cast<uint32_t*>(m.palette) + kCodes, 1u);
    __syncthreads();
    return true;
}

// Finds word w in the palette or enters it, and puts it into the table (by one
// thread).  False: too many words.
__device__ __forceinline__ bool learn_word(CodeTable& s, const DevMap& m, uint32_t w, uint32_t& polls) {
    uint32_t* palette = const_cast<uint32_t*>(m.palette);
    uint32_t slot = code_slot(w);
    for (uint32_t n = 0; n < kCodeProbes;) {
        uint32_t there = __hip_atomic_load(palette + slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (there == kCodeFree) {
            if (__hip_atomic_load(palette + kCodes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return false;
            if (polls != 0u) {
                --polls;
                __builtin_amdgcn_s_sleep(8);
                continue;
            }
            there = atomicCAS(palette + slot, kCodeFree, w);
            if (there == kCodeFree) {
                if (atomicAdd(palette + kCodes + 1, 1u) >= kCodeMost) return false;
                there = w;
            }
        }
        if (there == w) return table_enter(s, w, slot);
        slot = next_slot(slot);
        ++n;
    }
    return false;
}

// The codes of N words per lane, the whole workgroup together; `call` is 0 in its
// first call, 1 in a second.  False: too many words, the codes do not matter.
template <int N>
__device__ __forceinline__ bool find_codes(CodeTable& s, const DevMap& m, int call, const uint32_t (&w)[N],
                                           uint32_t (&code)[N]) {
    bool lacks = false;
#pragma unroll
    for (int i = 0; i < N; ++i) code[i] = s.entry[table_at(table_hash(w[i]), 0u)];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        code[i] = table_match(code[i], table_hash(w[i]), 0u);
        lacks = lacks || code[i] >= kCodes;
    }
    for (uint32_t far = 1; far < kTableFar && __ballot(lacks) != 0ull; ++far) {
        lacks = false;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t h = table_hash(w[i]);
            if (code[i] >= kCodes) code[i] = table_match(s.entry[table_at(h, far)], h, far);
            lacks = lacks || code[i] >= kCodes;
        }
    }
    if (lacks) s.lacks[call] = 1u;
    __syncthreads();
    if (s.lacks[call] == 0u) return true;
    const uint32_t t = threadIdx.x;
    s.set[t] = kCodeFree;
    // (the palette read when the table was loaded may be this XCD's old copy; here memory answers)
    if (t == 0u) s.over = __hip_atomic_load(m.palette + kCodes, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (s.over != 0u) return false;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (code[i] >= kCodes && *(volatile uint32_t*)&s.over == 0u) {
            const uint32_t h = table_hash(w[i]);
            uint32_t n = 0u;
            for (; n < kCodeProbes; ++n) {
                const uint32_t old = atomicCAS(&s.set[((h >> 24) + n) & (kSetSize - 1u)], kCodeFree, w[i]);
                if (old == kCodeFree || old == w[i]) break;
            }
            if (n == kCodeProbes) s.over = 1u;   // some 200 words in this workgroup alone
        }
    }
    __syncthreads();
    // one wave looks after them: every look at the palette in memory competes with all other workgroups'
    if (t < 64u) {
        const uint32_t id = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
        uint32_t polls = id % 64u == 0u ? 0u : id % 16u == 0u ? 1u : id % 4u == 0u ? 2u : 3u;
        bool room = s.over == 0u;
        for (uint32_t k = t; room && k < kSetSize; k += 64u)
            if (s.set[k] != kCodeFree) room = learn_word(s, m, s.set[k], polls);
        if (__ballot(!room) != 0ull && t == 0u) {
            s.over = 1u;
            atomicOr(const_cast<uint32_t*>(m.palette) + kCodes, 1u);
        }
    }
    __syncthreads();
    if (s.over != 0u) return false;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        if (code[i] < kCodes) continue;
        const uint32_t h = table_hash(w[i]);
        for (uint32_t far = 0; far < kTableFar && code[i] >= kCodes; ++far)
            code[i] = table_match(s.entry[table_at(h, far)], h, far);
    }
    return true;
}

constexpr uint32_t kSampleCount = 4096;

// The sampling pass: one workgroup reads kSampleCount voxels spread over the grid
// at once and enters their words in LDS.  6 us, most of it the launch and the loads.
constexpr uint32_t kSampleThreads = 1024, kSampleEach = kSampleCount / kSampleThreads;

__global__ __launch_bounds__(kSampleThreads) void palette_sample_kernel(const float* __restrict__ prob, DevMap m,
                                                                        float occ_thr, float free_thr, bool fresh,
                                                                        uint32_t* __restrict__ palette) {
    __shared__ uint32_t s_key[kCodes];
    __shared__ uint32_t s_count;
    const uint32_t t = threadIdx.x;
    if (t < kCodes) s_key[t] = t == 0u ? kSentinel : t == 1u ? kGainOne : kCodeFree;
    if (t == 0u) s_count = 2u;
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
        uint32_t slot = code_slot(w);
        for (uint32_t n = 0; n < kCodeProbes; ++n) {
            uint32_t old = s_key[slot];
            if (old == kCodeFree) {
                old = atomicCAS(&s_key[slot], kCodeFree, w);
                if (old == kCodeFree) atomicAdd(&s_count, 1u);
            }
            if (old == kCodeFree || old == w) break;
            if (*(volatile uint32_t*)&s_count > kCodeMost) break;
            slot = next_slot(slot);
        }
    }
    __syncthreads();
    if (t < kCodes) palette[t] = s_key[t];
    if (t == 0u) {
        // a sample of many words shows not nearly all of them: after an overflow it takes a
        // map of few to try again (a trial that fails costs 100-200 us)
        const uint32_t most = !fresh && palette[kCodes] ? kCodeMost / 4u : kCodeMost;
        palette[kCodes] = s_count > most ? 1u : 0u;
        palette[kCodes + 1] = s_count;
    }
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
// 4x4 columns, 30 now; 47 and 31 in linear order; with the codes 35 and 38).
// How many lanes lie along x depends on the map (lanes_along; with always 64 words to a
// row, 1 x 4000 x 4000 took 1490 us in linear order, 85 now).
//
// Every thread steps through LAYERS layers, their loads in flight together: 4,
// or 1 for a map without codes that is too small to fill the chip so (64^3 in
// columns: 6.2 us at 8 layers, 3.0 at 1).
//
// The codes of 1024 voxels are 8 whole lines (8x4x4 voxels each), which one
// instruction of a wave stores, 16 bytes a lane.
constexpr int kEncodeLayers = 4;
constexpr uint64_t kEncodeGroups = 2048;         // workgroups from which on they step through 4 layers

// Codes go through LDS as lines of 8 x ROWS x 4 voxels, x fastest: byte of
// voxel (x, y, z) of a region that is 2^lines_x of them wide.
template <int ROWS>
__device__ __forceinline__ uint32_t stage_byte(uint32_t x, uint32_t y, uint32_t z, uint32_t lines_x) {
    const uint32_t in = (x & 3u) | (y & 1u) << 2 | (z & 1u) << 3;       // of a 16-byte piece
    if constexpr (ROWS == 4)
        return (((y >> 2) << lines_x) + (x >> 3)) << 7 | in | (y & 2u) << 3 | (z & 2u) << 4 | (x & 4u) << 4;
    else
        return (((y >> 1) << lines_x) + (x >> 3)) << 6 | in | (z & 2u) << 3 | (x & 4u) << 3;
}

// Lane `piece` stores 16 bytes (4x2x2 voxels) of the region at (X0, Y0, Z0).
template <int ROWS>
__device__ __forceinline__ void store_codes(const DevMap& m, const uint4* stage, uint32_t piece, uint32_t X0,
                                            uint32_t Y0, uint32_t Z0, uint32_t lines_x) {
    const uint32_t line = piece >> (ROWS == 4 ? 3 : 2), in = ROWS == 4 ? piece : piece << 1;
    const uint32_t X = X0 + ((line & ((1u << lines_x) - 1u)) << 3) + (in & 4u);
    const uint32_t Y = Y0 + (line >> lines_x) * ROWS + (ROWS == 4 ? (in & 1u) << 1 : 0u), Z = Z0 + (in & 2u);
    if (X < (uint32_t)m.px && Y < (uint32_t)m.py && Z < (uint32_t)m.pz)
        *reinterpret_cast<uint4*>(const_cast<uint8_t*>(m.codes) + code_offset(m.csy, m.csz, X, Y, Z)) = stage[piece];
}

// Linear order: a workgroup takes 2^xl words in x of 256 >> xl rows of y.
template <int LAYERS, bool CODED>
__global__ __launch_bounds__(256) void encode_linear_kernel(
    const float* __restrict__ prob, uint32_t* __restrict__ enc, DevMap m, int xl, float occ_thr, float free_thr,
    unsigned int* __restrict__ bad) {
    const uint32_t x = threadIdx.x & ((1u << xl) - 1u), y = threadIdx.x >> xl;
    const int X0 = (int)(blockIdx.x << xl), Y0 = (int)(blockIdx.y * (256u >> xl)), Z0 = (int)blockIdx.z * LAYERS;
    const int X = X0 + (int)x, Y = Y0 + (int)y;
    const bool xy = X > 0 && Y > 0 && X <= m.nx && Y <= m.ny;
    [[maybe_unused]] CodeTable* table = nullptr;
    [[maybe_unused]] uint4* stage = nullptr;
    if constexpr (CODED) {
        static_assert(LAYERS == 4, "a line of codes has four layers");
        __shared__ CodeTable s_table;
        __shared__ uint4 s_stage[64];
        table = &s_table;
        stage = s_stage;
    }
    float p[LAYERS];
#pragma unroll
    for (int k = 0; k < LAYERS; ++k) {
        const int Z = Z0 + k;
        p[k] = xy && Z > 0 && Z <= m.nz ? prob[((size_t)(Z - 1) * m.ny + (size_t)(Y - 1)) * m.nx + (size_t)(X - 1)]
                                        : 0.0f;
    }
    bool any_bad = false;
    uint32_t w[LAYERS];
#pragma unroll
    for (int k = 0; k < LAYERS; ++k) {
        const int Z = Z0 + k;
        w[k] = xy && Z > 0 && Z <= m.nz ? encode_prob(p[k], occ_thr, free_thr, any_bad) : kSentinel;
        if (X < m.px && Y < m.py && Z < m.pz) enc[((size_t)Z * m.py + (size_t)Y) * m.px + (size_t)X] = w[k];
    }
    if (any_bad) atomicOr(bad, 1u);
    if constexpr (CODED) {
        if (!table_load(*table, m)) return;      // one answer for the workgroup
        uint32_t code[LAYERS];
        if (!find_codes(*table, m, 0, w, code)) return;
        uint8_t* bytes = reinterpret_cast<uint8_t*>(stage);
#pragma unroll
        for (int k = 0; k < LAYERS; ++k) bytes[stage_byte<4>(x, y, (uint32_t)k, (uint32_t)xl - 3u)] = (uint8_t)code[k];
        __syncthreads();
        if (threadIdx.x < 64u)
            store_codes<4>(m, stage, threadIdx.x, (uint32_t)X0, (uint32_t)Y0, (uint32_t)Z0, (uint32_t)xl - 3u);
    }
}

// Column orders: a thread writes pieces of four consecutive stored words (16
// bytes): four x of one row of a tile (a whole layer of a 2x2 tile).  A wave
// takes 2^xl pieces along x of 64 >> xl rows of them, so that it reads
// row segments of the probabilities and writes whole tile rows, and
// steps through the layers, whose tile rows continue one another.
template <int TL, int LAYERS, bool CODED>
__global__ __launch_bounds__(256) void encode_column_kernel(const float* __restrict__ prob,
                                                            uint32_t* __restrict__ enc, DevMap m, int xl, int zl,
                                                            float occ_thr, float free_thr,
                                                            unsigned int* __restrict__ bad) {
    constexpr int T = 1 << TL;
    constexpr int kWide = TL == 1 ? 2 : 4, kHigh = TL == 1 ? 2 : 1;     // voxels of a piece along x and y
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t x = (lane & ((1u << xl) - 1u)) * kWide, y = (lane >> xl) * kHigh;
    const uint32_t X0 = (blockIdx.x << xl) * kWide;
    const uint32_t Y0 = ((blockIdx.y << (2 - zl)) + (wave >> zl)) * (64u >> xl) * kHigh;
    const int Z0 = (int)((blockIdx.z << zl) + (wave & ((1u << zl) - 1u))) * LAYERS;
    const int X = (int)(X0 + x), Y = (int)(Y0 + y), tx = X >> TL, ty = Y >> TL;
    const bool stored = tx < m.nbx && ty < m.nby;
    uint32_t* out = enc + ((size_t)(ty * m.nbx + tx) * m.pz << (2 * TL)) + (Y & (T - 1)) * T + (X & (T - 1));
    bool any_bad = false, coded = false;
    [[maybe_unused]] CodeTable* table = nullptr;
    [[maybe_unused]] uint4* stage = nullptr;
    if constexpr (CODED) {
        static_assert(LAYERS == 4, "a line of codes has four layers");
        __shared__ CodeTable s_table;
        __shared__ uint4 s_stage[4][64];
        stage = s_stage[wave];
        table = &s_table;
        coded = table_load(s_table, m);
    }
    float p[4 * LAYERS];
    // the piece's voxels: four x of row Y, or for 2x2 tiles two x of rows Y and Y + 1
    auto at = [&](int e, int& vx, int& vy) {
        vx = X - 1 + (TL == 1 ? (e & 1) : e);
        vy = Y - 1 + (TL == 1 ? (e >> 1) : 0);
        return (unsigned)vx < (unsigned)m.nx && (unsigned)vy < (unsigned)m.ny;
    };
#pragma unroll
    for (int k = 0; k < LAYERS; ++k) {
        const int z = Z0 + k - 1;
        const bool in_z = (unsigned)z < (unsigned)m.nz;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            int vx, vy;
            p[4 * k + e] = at(e, vx, vy) && in_z ? prob[((size_t)z * m.ny + (size_t)vy) * m.nx + (size_t)vx] : 0.0f;
        }
    }
    // two layers at a time (all four keep 77 registers in use: six waves per SIMD)
    constexpr int HALF = LAYERS >= 2 ? 2 : 1;
    // (2x2 tiles: half lines; a wave of two rows of 128 writes its words in two thirds of the time of four of 64)
    constexpr int kRows = TL == 1 ? 2 : 4;
    const uint32_t lines_x = (uint32_t)xl - (TL == 1 ? 2u : 1u);
#pragma unroll
    for (int h = 0; h < LAYERS; h += HALF) {
        uint32_t w[4 * HALF];
#pragma unroll
        for (int k = 0; k < HALF; ++k) {
            const int Z = Z0 + h + k;
            const bool in_z = (unsigned)(Z - 1) < (unsigned)m.nz;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int vx, vy;
                w[4 * k + e] = at(e, vx, vy) && in_z ? encode_prob(p[4 * (h + k) + e], occ_thr, free_thr, any_bad)
                                                     : kSentinel;
            }
            if (stored && Z < m.pz)
                *reinterpret_cast<uint4*>(out + ((size_t)Z << (2 * TL))) =
                    make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
        }
        if constexpr (CODED) {
            if (!coded) continue;                // one answer for the workgroup
            uint32_t code[4 * HALF];
            coded = find_codes(*table, m, h / HALF, w, code);
#pragma unroll
            for (int k = 0; k < HALF; ++k) {
                uint8_t* to = reinterpret_cast<uint8_t*>(stage) + stage_byte<kRows>(x, y, (uint32_t)(h + k), lines_x);
                const uint32_t c = code[4 * k] | code[4 * k + 1] << 8 | code[4 * k + 2] << 16 | code[4 * k + 3] << 24;
                if constexpr (TL == 1) {         // two codes of each of two rows
                    *reinterpret_cast<uint16_t*>(to) = (uint16_t)c;
                    *reinterpret_cast<uint16_t*>(to + 4) = (uint16_t)(c >> 16);
                } else {
                    *reinterpret_cast<uint32_t*>(to) = c;
                }
            }
        }
    }
    if (any_bad) atomicOr(bad, 1u);
    if constexpr (CODED) {
        if (!coded || Z0 >= m.pz) return;        // the latter one for the wave
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        store_codes<kRows>(m, stage, lane, X0, Y0, (uint32_t)Z0, lines_x);
    }
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

// Lanes (their log2) along an axis of `count` items: the most whose last piece
// leaves no more than three sevenths of them idle.  Fewer waste less but read
// and write shorter rows: 17 x 300 x 3000 in linear order 45 us with 32 lanes
// to a row of 19 words, 69 with 8; 70 x 300 x 1000 63 us with 32 to 72, 68 with 64.
static int lanes_along(uint32_t count, int least, int most) {
    int l = most;
    while (l > least && 4u * (((count + (1u << l) - 1u) >> l) << l) > 7u * count) --l;
    return l;
}

template <int TL>
static void launch_encode_column(const float* prob, uint32_t* enc, const DevMap& m, float occ_thr, float free_thr,
                                 unsigned int* bad_flag, hipStream_t s) {
    constexpr int T = 1 << TL, kWide = TL == 1 ? 2 : 4, kHigh = TL == 1 ? 2 : 1;
    const uint32_t along = (uint32_t)(m.nbx * (T / kWide)), rows = (uint32_t)(m.nby * (T / kHigh));
    // with codes a wave's region is at least a line of them wide
    const int xl = lanes_along(along, !m.codes ? 0 : TL == 1 ? 2 : 1, TL == 1 ? 6 : TL == 2 ? 4 : 3);
    const unsigned gx = (along + (1u << xl) - 1u) >> xl, pz = (unsigned)m.pz;
    auto go = [&](auto kernel, unsigned layers) {
        // the four waves take layers above one another, or rows where there are too few layers
        const unsigned steps = (pz + layers - 1) / layers, zl = steps > 2 ? 2 : steps - 1;
        const unsigned high = (64u >> xl) << (2 - zl);
        hipLaunchKernelGGL(kernel, dim3(gx, (rows + high - 1) / high, (steps + (1u << zl) - 1) >> zl), dim3(256), 0, s,
                           prob, enc, m, xl, (int)zl, occ_thr, free_thr, bad_flag);
    };
    const uint64_t groups = (uint64_t)gx * ((rows + (64u >> xl) - 1u) / (64u >> xl)) * ((pz + 15) / 16);
    if (m.codes) go(encode_column_kernel<TL, kEncodeLayers, true>, kEncodeLayers);
    else if (groups >= kEncodeGroups) go(encode_column_kernel<TL, kEncodeLayers, false>, kEncodeLayers);
    else go(encode_column_kernel<TL, 1, false>, 1);
}

static void launch_encode_linear(const float* prob, uint32_t* enc, const DevMap& m, float occ_thr, float free_thr,
                                 unsigned int* bad_flag, hipStream_t s) {
    const int xl = lanes_along((uint32_t)m.px, m.codes ? 3 : 0, 6);
    const unsigned gx = ((unsigned)m.px + (1u << xl) - 1u) >> xl, pz = (unsigned)m.pz;
    const unsigned rows = 256u >> xl, gy = ((unsigned)m.py + rows - 1u) / rows, gz = (pz + kEncodeLayers - 1) / kEncodeLayers;
    auto go = [&](auto kernel, unsigned z) {
        hipLaunchKernelGGL(kernel, dim3(gx, gy, z), dim3(256), 0, s, prob, enc, m, xl, occ_thr, free_thr, bad_flag);
    };
    if (m.codes) go(encode_linear_kernel<kEncodeLayers, true>, gz);
    else if ((uint64_t)gx * gy * gz >= kEncodeGroups) go(encode_linear_kernel<kEncodeLayers, false>, gz);
    else go(encode_linear_kernel<1, false>, pz);
}

hipError_t launch_encode_map(const float* prob, uint32_t* enc, const DevMap& m, float occ_thr,
                             float free_thr, unsigned int* bad_flag, PaletteStart start, hipStream_t s) {
    if (m.codes && start != PaletteStart::kept) {
        hipLaunchKernelGGL(palette_sample_kernel, dim3(1), dim3(kSampleThreads), 0, s, prob, m, occ_thr, free_thr,
                           start == PaletteStart::first, const_cast<uint32_t*>(m.palette));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    switch (m.tl) {
    case 1: launch_encode_column<1>(prob, enc, m, occ_thr, free_thr, bad_flag, s); break;
    case 2: launch_encode_column<2>(prob, enc, m, occ_thr, free_thr, bad_flag, s); break;
    case 3: launch_encode_column<3>(prob, enc, m, occ_thr, free_thr, bad_flag, s); break;
    default: launch_encode_linear(prob, enc, m, occ_thr, free_thr, bad_flag, s);
    }
    return hipGetLastError();
}

}  // namespace nbt
