// Rules of the host side in a CPU build (host code only, no kernel), for tests.
#include "internal.hpp"

extern "C" int pick_layout(const float* ms, int count, int current, float margin) {
    return nbt::pick_layout(ms, count, current, margin);
}
