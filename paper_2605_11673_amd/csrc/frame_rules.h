// Which launches a frame takes (host only).
#pragma once

#include <algorithm>
#include <cstdint>

namespace sta {

// The proxy operator's frame of one launch counts a changed tet's edges again
// over their tets, eight lanes each, and its vertices' active edges over theirs,
// 16 lanes each, 64 columns of the row at a time: so many rounds, each a chain of
// two round trips.  Two launches change counts and degrees by atomics whatever
// there is around.  Meshes of more rounds than this take them for every frame:
// two frames of 30 to 1,000 edits took, by one launch, 10 to 11 us at 2 to 5
// rounds, 13 at 10, 16 to 20 at 12 to 14, 24 at 18, 34 at 27, and 13 ms at the
// 12,000 of a vertex of 5,000 tets; by two, 13 to 16 us at any.
constexpr int64_t kProxyOnceRounds = 10;

inline int64_t proxy_edge_rounds(int64_t tets)
{
    return (tets + 7) / 8;
}

inline int64_t proxy_vertex_rounds(int64_t tets, int64_t columns)
{
    return ((tets + 15) / 16) * ((columns + 63) / 64);
}

}  // namespace sta
