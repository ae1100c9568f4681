// Which launches a frame takes (host only).
#pragma once

#include <algorithm>
#include <cstdint>

namespace sta {

// A frame of the elasticity operator.  One launch re-sums the ten blocks of every
// edited tet, each as often as edits share it, from lists of up to kFrameOnceEdits
// (one launch / two at 1, 300, 1,700, 2,304 random edits of 384,000 tets: 3.7 / 6.1,
// 5.0 / 8.9, 8.9 / 12.0, 13.1 / 13.3 us).  Two launches sum every block once, which
// counts where a vertex has many tets: 5,000 of them, 64, 768, 2,304 edits 115 / 108,
// 152 / 116, 257 / 133 us; 2,450, 768 77 / 65; but 968, 768 33 / 35; 512, 300 17 / 21.
// So meshes whose longest list of a vertex's tets is past kFrameOnceTets take two.
// A grid barrier between two phases of one launch costs more than a launch
// (15 to 23 us a frame) and is taken for longer lists if the caller asks for it, and
// for any if they limit its polls.
constexpr int32_t kFrameOnceEdits = 2304;
constexpr int64_t kFrameOnceTets = 1024;

enum class FrameRoute { once, two, barrier };

inline FrameRoute frame_route(int64_t edits, int64_t longest, bool fused, bool polls_limited)
{
    if (fused && polls_limited)
        return FrameRoute::barrier;
    if (edits <= kFrameOnceEdits && longest <= kFrameOnceTets)
        return FrameRoute::once;
    return fused ? FrameRoute::barrier : FrameRoute::two;
}

// The proxy operator's frame of one launch counts a changed tet's edges again
// over their tets, eight lanes each, and its vertices' active edges over theirs,
// 16 lanes each, 64 columns of the row at a time: so many rounds, each a chain of
// two round trips.  Two launches change counts and degrees by atomics whatever
// there is around.  Meshes of more rounds than this take them for every frame: two
// frames of 30 to 1,000 edits took, by one launch / two, 10 to 11 / 16 us at 2 to 5
// rounds, 16 to 20 / 16 to 24 at 12 to 14, 24 / 22 at 18, 34 / 22 at 27, and 13,000 / 21
// at the 12,000 of a vertex of 5,000 tets.
constexpr int64_t kProxyOnceRounds = 14;

inline int64_t proxy_edge_rounds(int64_t tets)
{
    return (tets + 7) / 8;
}

inline int64_t proxy_vertex_rounds(int64_t tets, int64_t columns)
{
    return ((tets + 15) / 16) * ((columns + 63) / 64);
}

}  // namespace sta
