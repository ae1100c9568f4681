// Which chunks of tets make a brick of the adjoint (host only).
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

namespace sta {

constexpr int kAdjointChunk = 16, kAdjointBrick = 128;
constexpr int kBrickChunks = kAdjointBrick / kAdjointChunk;

// The LDS of every brick is what the largest one needs, and where ids are in no
// order a brick of 128 tets shares nothing: 1,280 blocks, one workgroup on a
// compute unit.  So a brick of more blocks than let four workgroups fit is
// halved.  A half may still hold up to 640 blocks; it is halved again, if need
// be to a chunk of 160, where such bricks are few, so that they don't set the
// LDS of all.  A call on 384,000 tets, never halved / halved so / every tet
// gathering for itself: ids shuffled in windows of 64 113 / 94 / 125 us, of 512
// 232 / 146 / 194, of 4,096 326 / 206 / 297, all 422 / 332 / 479, only a fiftieth
// of them 152 / 80 / 95.
constexpr int kBrickMost = 568;

// order: the bricks' chunks, kBrickChunks places each, -1 past the last; blocks:
// of each brick.  Halves the bricks that are too large; false: there are none.
inline bool halve_large_bricks(std::vector<int32_t>& order, const std::vector<int32_t>& blocks)
{
    const std::size_t n = blocks.size();
    std::vector<int> chunks(n, 0);
    std::size_t large_halves = 0;
    for (std::size_t k = 0; k < n; ++k) {
        while (chunks[k] < kBrickChunks && order[k * kBrickChunks + chunks[k]] >= 0)
            ++chunks[k];
        large_halves += blocks[k] > kBrickMost && chunks[k] <= kBrickChunks / 2;
    }
    const int least = large_halves <= n / 4 ? 1 : kBrickChunks / 2;
    std::vector<int32_t> out;
    out.reserve(order.size());
    for (std::size_t k = 0; k < n; ++k) {
        const int32_t* c = order.data() + k * kBrickChunks;
        const int part = blocks[k] > kBrickMost && chunks[k] > least ? (chunks[k] + 1) / 2 : chunks[k];
        for (int i0 = 0; i0 < chunks[k]; i0 += part)
            for (int i = 0; i < kBrickChunks; ++i)
                out.push_back(i < part && i0 + i < chunks[k] ? c[i0 + i] : -1);
    }
    const bool halved = out.size() > order.size();
    order.swap(out);
    return halved;
}

}  // namespace sta
