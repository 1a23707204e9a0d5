// Rules of the host side in a CPU build (host code only, no kernel), for tests.
#include "internal.hpp"

extern "C" int pick_layout(const float* ms, int count, int current, float margin) {
    return nbt::pick_layout(ms, count, current, margin);
}

// Threads of the cost terms' launch over `states` states in horizons of `steps`.
extern "C" unsigned long long cost_threads(uint32_t states, uint32_t steps, uint32_t nb, uint32_t np, int cu_count) {
    const uint32_t tile = nbt::cost_tile(steps), tiles = (states + tile - 1) / tile;
    return (unsigned long long)tiles * (unsigned long long)nbt::query_waves(tiles, nb, np, cu_count) * 64u;
}
