// The mark walk of the depth insertion in a CPU build (host code only, no
// kernel): one scan's marks, with every store checked against the mark array.
#include <cstdint>
#include <vector>

#include "insert_walk.hpp"

using namespace nbt;

namespace {

struct HostTable {
    uint32_t word[kSeen];
    uint32_t read(uint32_t lin4) const { return word[seen_slot(lin4) / 4]; }
    void write(uint32_t lin4) { word[seen_slot(lin4) / 4] = lin4; }
    void pin() const {}
};

}  // namespace

// marks: 2 bytes per voxel.  Returns the number of stores outside them (not made).
extern "C" int64_t mark_scan(int nx, int ny, int nz, float voxel, const float* origin, int W, int H, float tan_h,
                             float tan_v, float range, const float* pose, const float* depth, uint8_t* marks) {
    DevMap m{};
    m.nx = nx; m.ny = ny; m.nz = nz;
    m.inv_s = 1.0f / voxel;
    m.ox = origin[0]; m.oy = origin[1]; m.oz = origin[2];
    const CamParams c{W, H, range * tan_h, range * tan_v, range};
    const uint64_t bytes = 2 * (uint64_t)nx * (uint64_t)ny * (uint64_t)nz;
    int64_t outside = 0;
    auto mark = [&](uint32_t byte) {
        if (byte < bytes) marks[byte] = 1;
        else ++outside;
    };
    std::vector<HostTable> table(1);
    const bool small = nx <= 512 && ny <= 512 && nz <= 512;
    for (int j0 = 0; j0 < H; j0 += 16)               // a table for every 16x16 pixels, as on the device
        for (int i0 = 0; i0 < W; i0 += 16) {
            for (uint32_t& w : table[0].word) w = ~0u;
            for (int j = j0; j < j0 + 16 && j < H; ++j)
                for (int i = i0; i < i0 + 16 && i < W; ++i) {
                    const float d = depth[(int64_t)j * W + i];
                    if (small) insert_walk<uint32_t>(m, c, pose, d, i, j, table[0], mark);
                    else insert_walk<uint64_t>(m, c, pose, d, i, j, table[0], mark);
                }
        }
    return outside;
}
