// Connectivity of the active tetrahedra (paper Sec. 3.6: rebuilt from the
// current mask; Alg. 1 keeps it with the mask), on gfx950.
//
// The paper does not fix the adjacency; two are provided.  Vertex: two
// active tets are connected when they share a vertex (the components of the
// assembled operator), labelled by the component's smallest vertex.  Face:
// when they share a face (fragments in the sense of fracture), labelled by
// the component's smallest tet; the candidate pairs with a common vertex
// triple are found once on the host and kept on the device.
//
// Both are a union-find over parent pointers f.  Each workgroup first merges
// one window of tets, consecutive or near each other, in LDS and keeps one root
// per set it finds.
// Vertex: every vertex of the window then takes its set's root as its own,
// exchanging it for that of another window that holds the vertex: those two
// roots are to be united.  Face: the pairs that cross windows name two roots
// each.  Of a workgroup's many pairs of roots few are different, and only those
// are united.  Then every vertex (tet) climbs to its root, every
// window's root lowers that root's smallest id by its own, and the labels read
// that.  One wait per call, for the count, which the last launch writes to pinned
// memory.
//
// A union hooks one of two roots under the other with a compare and swap, and
// climbs on from what it finds there if that was no root any more, so one pass
// is complete.  Which one is hooked follows a fixed scattered order of the ids
// (priority): trees stay shallow, where hooking the larger id under the smaller
// makes chains as long as the row of windows.  Plain loads may see
// another XCD's stale copy of a pointer: that is an older ancestor, and only
// costs the swap that fails on it.  Climbing shortens paths with stores that
// race; they only replace a pointer of a vertex that is no root by one to
// another of its ancestors, and no swap takes such a vertex, so no union is
// lost.  Launch boundaries make all of it visible to what follows.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <vector>

#include "sta_internal.h"

namespace sta {
namespace {

constexpr int kBlock = 256;

unsigned blocks(int64_t n)
{
    return (unsigned)((n + kBlock - 1) / kBlock);
}

// Tets per workgroup of the first merge.  Larger windows leave fewer roots to
// unite: both adjacencies of a fracture mesh of 196,608 tets take 130, 107, 99
// us a call at 256, 512, 1,024 tets.
constexpr int kWindow = 1024;
constexpr int kSlots = 8192;  // hash slots of a window's vertices
static_assert(4 * kWindow < kSlots && kSlots == 1 << 13, "every vertex of a window finds a slot");

// Pointers go to ids of smaller priority only, so every climb and union ends.
__device__ __forceinline__ uint32_t priority(int x)
{
    return (uint32_t)x * 2654435761u;
}

// The root above x as far as this thread sees; paths are shortened on the way.
__device__ __forceinline__ int climb(int* f, int x)
{
    int prev = x, cur = f[x];
    if (cur == x)
        return x;
    for (int next = f[cur]; next != cur; next = f[cur]) {
        f[prev] = next;
        prev = cur;
        cur = next;
    }
    return cur;
}

__device__ __forceinline__ void unite(int* f, int a, int b)
{
    a = climb(f, a);
    b = climb(f, b);
    while (a != b) {
        if (priority(a) < priority(b)) {
            const int c = a;
            a = b;
            b = c;
        }
        const int old = atomicCAS(f + a, a, b);
        if (old == a)
            break;
        a = climb(f, old);
        b = climb(f, b);
    }
}

// The same in LDS.
__device__ __forceinline__ int climb_lds(volatile int* f, int x)
{
    int cur = f[x];
    if (cur == x)
        return x;
    for (int next = f[cur]; next != cur; next = f[cur]) {
        f[x] = next;
        x = cur;
        cur = next;
    }
    return cur;
}

__device__ __forceinline__ void unite_lds(int* f, int a, int b)
{
    a = climb_lds(f, a);
    b = climb_lds(f, b);
    while (a != b) {
        if (priority(a) < priority(b)) {
            const int c = a;
            a = b;
            b = c;
        }
        const int old = atomicCAS(f + a, a, b);
        if (old == a)
            break;
        a = climb_lds(f, old);
    }
}

// A pair of roots that this workgroup has not just united.  The table keeps
// the last pair of each place, so a pair may be new twice, but never unseen.
constexpr int kPairSlots = 1024;
__device__ __forceinline__ bool new_pair(unsigned long long* table, int a, int b)
{
    const unsigned long long key = (unsigned long long)(uint32_t)min(a, b) << 32 | (uint32_t)max(a, b);
    const uint32_t h = (priority(a) + priority(b)) >> 22;
    return atomicExch(table + h, key) != key;
}
static_assert(kPairSlots == 1 << (32 - 22), "the hash covers the table");

// own[i] = -1: vertex i is in no active tet.
__global__ __launch_bounds__(kBlock) void k_cc_init(int n, int* __restrict__ f, int* __restrict__ least,
                                                    int* __restrict__ own, uint32_t* __restrict__ count)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i == 0)
        *count = 0u;
    if (i < n) {
        f[i] = i;
        least[i] = INT32_MAX;
        own[i] = -1;
    }
}

// The slot of vertex x in a window's hash table.
__device__ __forceinline__ int find_slot(int* key, int x, bool* added = nullptr)
{
    unsigned h = priority(x) >> (32 - 13);
    for (;; h = (h + 1) & (kSlots - 1)) {  // ends: there are more slots than vertices
        const int old = atomicCAS(key + h, -1, x);
        if (added)
            *added = old == -1;
        if (old == -1 || old == x)
            return (int)h;
    }
}

// One window of tets: the vertices of its active tets in a hash table, merged
// there; then its roots with those of other windows.  Bound by latency: chains
// of LDS atomics, then of pointers to global roots.  22 us at 196,608 tets,
// where seeding every vertex from its tets and two to four hooking passes, each
// with a shortcut pass, took 13 + 62; the whole call 45 us at 384,000 tets, all
// active or half of them (62, 250 to 500 before).
//
// kOrdered: windows of the tets in the order given (below).  kMany: the roots'
// smallest ids are found where the pointers were, so that two workgroups fit on a
// compute unit, at the price of two more barriers (1 us); for more windows than
// compute units: 375 windows 52.6 -> 44.5 us a call, the 1,388 of a batch of 64
// meshes 104.7 -> 82.0 (93 by the hooking passes); one window 28.1, else 29.3.
constexpr int kManyWindows = 256;
template <bool kOrdered, bool kMany>
__global__ __launch_bounds__(kWindow) void k_cc_windows(DevView v, const int* __restrict__ order, int* f,
                                                        int* __restrict__ own, int* least)
{
    __shared__ int s_key[kSlots], s_f[kSlots], s_least[kMany ? 1 : kSlots];
    __shared__ unsigned long long s_pair[kPairSlots];
    const int i = blockIdx.x * kWindow + threadIdx.x, ii = min(i, v.n_tets - 1), e = kOrdered ? order[ii] : ii;
    const int4 t = v.T[e];
    const bool on = i < v.n_tets && v.mask[e];
    for (int h = threadIdx.x; h < kSlots; h += kWindow) {
        s_key[h] = -1;
        s_f[h] = h;
        if (!kMany)
            s_least[h] = INT32_MAX;
    }
    for (int h = threadIdx.x; h < kPairSlots; h += kWindow)
        s_pair[h] = ~0ull;
    __syncthreads();
    if (on) {
        const int x[4] = {t.x, t.y, t.z, t.w};
        int slot[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            slot[k] = find_slot(s_key, x[k]);
#pragma unroll
        for (int k = 1; k < 4; ++k)
            unite_lds(s_f, slot[0], slot[k]);
    }
    __syncthreads();
    constexpr int kMine = kSlots / kWindow;
    int at[kMine], root[kMine], other[kMine];
#pragma unroll
    for (int k = 0; k < kMine; ++k) {
        const int h = threadIdx.x + k * kWindow, x = s_key[h];
        at[k] = root[k] = other[k] = -1;
        if (x >= 0) {
            at[k] = climb_lds(s_f, h);
            if (!kMany)
                atomicMin(s_least + at[k], x);
            root[k] = s_key[at[k]];
            other[k] = atomicExch(own + x, root[k]);
        }
    }
    __syncthreads();
    if (kMany) {  // no pointer is followed any more
#pragma unroll
        for (int k = 0; k < kMine; ++k)
            if (at[k] == (int)threadIdx.x + k * kWindow)  // a root
                s_f[at[k]] = root[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kMine; ++k)
            if (at[k] >= 0 && at[k] != (int)threadIdx.x + k * kWindow)
                atomicMin(s_f + at[k], s_key[threadIdx.x + k * kWindow]);
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < kMine; ++k) {
        const int h = threadIdx.x + k * kWindow;
        if (kMany ? at[k] == h : s_least[h] != INT32_MAX)  // h is a root
            atomicMin(least + s_key[h], kMany ? s_f[h] : s_least[h]);
    }
#pragma unroll
    for (int k = 0; k < kMine; ++k)
        if (other[k] >= 0 && other[k] != root[k] && new_pair(s_pair, root[k], other[k]))
            unite(f, root[k], other[k]);
}

// Windows of tets that are near each other leave few roots to unite; of tets in
// no order, nearly every vertex of each is one, and a call on 384,000 tets took
// 940 us.  By their smallest vertex the tets are near each other again if the
// vertices' ids are: 49 us, 45 in order (71 by the hooking passes); and share at
// least that vertex if not: 200 (by id 350; 3,290).  The first call looks at some
// windows and keeps that order if it halves their vertices, for 0.1 ms.  Any
// order gives the same labels.
//
// Vertices of the candidates of every step-th window, into sum.
constexpr int kSpreadWindows = 64, kSpreadFrom = 16 * kWindow, kSpreadVertices = 1024;
template <bool kOrdered>
__global__ __launch_bounds__(kWindow) void k_cc_spread(DevView v, const int* __restrict__ order, int step, uint32_t* sum)
{
    __shared__ int s_key[kSlots];
    __shared__ uint32_t s_count;
    const int i = blockIdx.x * step * kWindow + threadIdx.x, ii = min(i, v.n_tets - 1);
    const int4 t = v.T[kOrdered ? order[ii] : ii];
    for (int h = threadIdx.x; h < kSlots; h += kWindow)
        s_key[h] = -1;
    if (threadIdx.x == 0)
        s_count = 0u;
    __syncthreads();
    if (i < v.n_tets) {
        const int x[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            bool added;
            (void)find_slot(s_key, x[k], &added);
            if (added)
                atomicAdd(&s_count, 1u);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0)
        atomicAdd(sum, s_count);
}

// Order by smallest vertex: counts per vertex, their running sums, places.
__global__ __launch_bounds__(kBlock) void k_cc_zero(int n, uint32_t* __restrict__ at)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < n)
        at[i] = 0u;
}

__global__ __launch_bounds__(kBlock) void k_cc_place(DevView v, uint32_t* at, int* __restrict__ order)
{
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= v.n_tets)
        return;
    const int4 t = v.T[e];
    const uint32_t p = atomicAdd(at + min(min(t.x, t.y), min(t.z, t.w)), 1u);
    if (order)
        order[p] = e;
}

__global__ __launch_bounds__(kWindow) void k_cc_sums(int n, uint32_t* __restrict__ at)
{
    __shared__ uint32_t s_sum[kWindow];
    const int t = threadIdx.x, per = (n + kWindow - 1) / kWindow;
    const int i0 = min(n, t * per), i1 = min(n, i0 + per);
    uint32_t mine = 0u;
    for (int i = i0; i < i1; ++i)
        mine += at[i];
    s_sum[t] = mine;
    __syncthreads();
    for (int d = 1; d < kWindow; d *= 2) {
        const uint32_t x = t >= d ? s_sum[t - d] : 0u;
        __syncthreads();
        s_sum[t] += x;
        __syncthreads();
    }
    uint32_t sum = s_sum[t] - mine;
    for (int i = i0; i < i1; ++i) {
        const uint32_t c = at[i];
        at[i] = sum;
        sum += c;
    }
}

// After the unions: of every id i the root, into own[i] (a root of i's window
// before; -1: not in an active tet, not an active tet), and of every root the
// smallest id and the count.  least[i] is set where i is a root of a window, to
// the smallest id of its set there.
__global__ __launch_bounds__(kBlock) void k_cc_roots(int n, int* __restrict__ own, const int* __restrict__ f,
                                                     int* least, uint32_t* count)
{
    __shared__ uint32_t s_count;
    if (threadIdx.x == 0)
        s_count = 0u;
    __syncthreads();
    const int i = blockIdx.x * kBlock + threadIdx.x;
    int r = -1, m = INT32_MAX;
    if (i < n) {
        r = own[i];
        m = least[i];
    }
    if (r >= 0) {
        for (int p = f[r]; p != r; p = f[r])
            r = p;
        own[i] = r;
    }
    // A root hears from all its windows' roots: in a wave one lane speaks for
    // the lanes with the same root (of two roots; lanes with further ones speak
    // for themselves), and only if its id can lower what it sees there.  (Where
    // tet ids are scattered and nearly every tet is a window's root, an atomic
    // each took 4.6 ms of a call.)
    bool speaks = m != INT32_MAX && r != i;  // least[i] is no root's, and stays
    for (int k = 0; k < 2; ++k) {
        const unsigned long long left = __ballot(speaks);
        if (left == 0)
            break;
        const int lead = __ffsll(left) - 1, lr = __shfl(r, lead, 64);
        const bool same = speaks && r == lr;
        int least_id = same ? m : INT32_MAX;
#pragma unroll
        for (int d = 32; d > 0; d >>= 1)
            least_id = min(least_id, __shfl_xor(least_id, d, 64));
        if ((int)(threadIdx.x & 63) == lead && least[lr] > least_id)
            atomicMin(least + lr, least_id);
        speaks = speaks && !same;
    }
    if (speaks && least[r] > m)
        atomicMin(least + r, m);
    if (m != INT32_MAX && r == i)
        atomicAdd(&s_count, 1u);
    __syncthreads();
    if (threadIdx.x == 0 && s_count)
        atomicAdd(count, s_count);
}

// Tet e's label: the smallest id at the root of its first vertex (-1 if
// inactive); and the count, to the host.
__global__ __launch_bounds__(kBlock) void k_cc_label(DevView v, const int* __restrict__ own,
                                                     const int* __restrict__ least, int32_t* __restrict__ label,
                                                     const uint32_t* __restrict__ count, uint32_t* host)
{
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e == 0)
        __hip_atomic_store(host, *count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (e < v.n_tets)
        label[e] = v.mask[e] ? least[own[v.T[e].x]] : -1;
}

// Face adjacency, one window of tets: the pairs inside it (pairs are sorted by
// their smaller tet; start: the first pair of each window).
__global__ __launch_bounds__(kWindow) void k_ccf_windows(int n_tets, const uint8_t* __restrict__ mask,
                                                         const int2* __restrict__ pairs,
                                                         const int64_t* __restrict__ start, int* __restrict__ own,
                                                         int* __restrict__ f, int* __restrict__ least,
                                                         uint32_t* __restrict__ count)
{
    __shared__ int s_f[kWindow], s_least[kWindow];
    __shared__ uint8_t s_on[kWindow];
    const int base = blockIdx.x * kWindow, e = base + threadIdx.x;
    if (e == 0)
        *count = 0u;
    s_f[threadIdx.x] = threadIdx.x;
    s_least[threadIdx.x] = INT32_MAX;
    s_on[threadIdx.x] = e < n_tets ? mask[e] : (uint8_t)0;
    const int64_t k1 = start[blockIdx.x + 1];
    __syncthreads();
    for (int64_t k = start[blockIdx.x] + threadIdx.x; k < k1; k += kWindow) {
        const int a = pairs[k].x - base, b = pairs[k].y - base;
        if (b < kWindow && s_on[a] && s_on[b])
            unite_lds(s_f, a, b);
    }
    __syncthreads();
    const int r = s_on[threadIdx.x] ? climb_lds(s_f, threadIdx.x) : -1;
    if (r >= 0)
        atomicMin(s_least + r, e);
    __syncthreads();
    if (e < n_tets) {
        own[e] = r >= 0 ? base + r : -1;
        f[e] = e;
        least[e] = s_least[threadIdx.x];
    }
}

// The pairs that cross windows, kCross per workgroup.  12 us at 196,608 tets
// (three to six hooking passes over all pairs took 62 before); the whole call
// 43 us at 384,000 tets, 70 with half of them active, 286 with scattered ids
// (101, 160, 939 before).
constexpr int kCrossLane = 4, kCross = kBlock * kCrossLane;
__global__ __launch_bounds__(kBlock) void k_ccf_cross(const int2* __restrict__ pairs, int64_t n_pairs,
                                                      const int* __restrict__ own, int* f)
{
    __shared__ unsigned long long s_pair[kPairSlots];
    for (int h = threadIdx.x; h < kPairSlots; h += kBlock)
        s_pair[h] = ~0ull;
    int2 p[kCrossLane];
    int a[kCrossLane], b[kCrossLane];
#pragma unroll
    for (int k = 0; k < kCrossLane; ++k)
        p[k] = pairs[min((int64_t)blockIdx.x * kCross + k * kBlock + threadIdx.x, n_pairs - 1)];
#pragma unroll
    for (int k = 0; k < kCrossLane; ++k) {
        a[k] = own[p[k].x];
        b[k] = own[p[k].y];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kCrossLane; ++k)
        if (a[k] >= 0 && b[k] >= 0 && a[k] != b[k] && new_pair(s_pair, a[k], b[k]))
            unite(f, a[k], b[k]);
}

__global__ __launch_bounds__(kBlock) void k_ccf_label(int n_tets, const int* __restrict__ own,
                                                      const int* __restrict__ least, int32_t* __restrict__ label,
                                                      const uint32_t* __restrict__ count, uint32_t* host)
{
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e == 0)
        __hip_atomic_store(host, *count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (e < n_tets) {
        const int r = own[e];
        label[e] = r >= 0 ? least[r] : -1;
    }
}

}  // namespace

// Candidate tet pairs with a common face (sorted vertex triple), every pair
// of tets on one triple, (smaller id, larger id), sorted.
std::vector<int2> host_face_pairs(const std::vector<int4>& T)
{
    struct Face {
        int a, b, c, e;
    };
    std::vector<Face> fs;
    fs.reserve(4 * T.size());
    for (size_t e = 0; e < T.size(); ++e) {
        std::array<int, 4> v = {T[e].x, T[e].y, T[e].z, T[e].w};
        std::sort(v.begin(), v.end());
        for (int skip = 0; skip < 4; ++skip) {
            int t[3], k = 0;
            for (int i = 0; i < 4; ++i)
                if (i != skip)
                    t[k++] = v[i];
            fs.push_back(Face{t[0], t[1], t[2], (int)e});
        }
    }
    std::sort(fs.begin(), fs.end(), [](const Face& x, const Face& y) {
        if (x.a != y.a) return x.a < y.a;
        if (x.b != y.b) return x.b < y.b;
        if (x.c != y.c) return x.c < y.c;
        return x.e < y.e;
    });
    std::vector<int2> pairs;
    for (size_t i = 0; i < fs.size();) {
        size_t j = i + 1;
        while (j < fs.size() && fs[j].a == fs[i].a && fs[j].b == fs[i].b && fs[j].c == fs[i].c)
            ++j;
        for (size_t u = i; u < j; ++u)
            for (size_t w = u + 1; w < j; ++w)
                if (fs[u].e != fs[w].e)
                    pairs.push_back(make_int2(fs[u].e, fs[w].e));
        i = j;
    }
    std::sort(pairs.begin(), pairs.end(),
              [](const int2& x, const int2& y) { return x.x != y.x ? x.x < y.x : x.y < y.y; });
    pairs.erase(std::unique(pairs.begin(), pairs.end(), [](const int2& x, const int2& y) { return x.x == y.x && x.y == y.y; }),
                pairs.end());
    return pairs;
}

// Face-adjacency labels (smallest tet id of the component, -1 if inactive)
// into label; the number of components into *host (pinned) once s is done.
// own, f, least: n_tets ints each; count: one word.
static hipError_t run_face_components(const DevView& v, const int2* pairs, int64_t n_pairs, const int64_t* start,
                                      int* own, int* f, int* least, uint32_t* count, uint32_t* host, int32_t* label,
                                      hipStream_t s)
{
    const dim3 windows(std::max(1, (v.n_tets + kWindow - 1) / kWindow)), tets(std::max(1u, blocks(v.n_tets)));
    hipLaunchKernelGGL(k_ccf_windows, windows, dim3(kWindow), 0, s, v.n_tets, v.mask, pairs, start, own, f, least,
                       count);
    if (n_pairs > 0)
        hipLaunchKernelGGL(k_ccf_cross, dim3((unsigned)((n_pairs + kCross - 1) / kCross)), dim3(kBlock), 0, s, pairs,
                           n_pairs, own, f);
    hipLaunchKernelGGL(k_cc_roots, tets, dim3(kBlock), 0, s, v.n_tets, own, f, least, count);
    hipLaunchKernelGGL(k_ccf_label, tets, dim3(kBlock), 0, s, v.n_tets, own, least, label, count, host);
    return hipGetLastError();
}

// The order of the tets for the windows, into *order (NULL: by id), once per
// context; word: a device word, at: n_nodes words of scratch.  Waits for s.
static hipError_t order_tets(const DevView& v, uint32_t* word, uint32_t* at, int** order, hipStream_t s)
{
    *order = nullptr;
    if (v.n_tets < kSpreadFrom)
        return hipSuccess;
    const int windows = (v.n_tets + kWindow - 1) / kWindow, looked = std::min(windows, kSpreadWindows);
    auto spread = [&](const int* by, uint32_t* sum) {
        hipLaunchKernelGGL(k_cc_zero, dim3(1), dim3(kBlock), 0, s, 1, word);
        hipLaunchKernelGGL((by ? k_cc_spread<true> : k_cc_spread<false>), dim3(looked), dim3(kWindow), 0, s, v, by,
                           windows / looked, word);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess)
            e = hipMemcpyAsync(sum, word, sizeof(uint32_t), hipMemcpyDeviceToHost, s);
        return e == hipSuccess ? hipStreamSynchronize(s) : e;
    };
    uint32_t by_id = 0u, by_vertex = 0u;
    hipError_t e = spread(nullptr, &by_id);
    if (e != hipSuccess || by_id <= (uint32_t)(looked * kSpreadVertices))
        return e;
    int* q = nullptr;
    if (hipMalloc((void**)&q, sizeof(int) * (size_t)v.n_tets) != hipSuccess) {
        (void)hipGetLastError();
        return hipSuccess;  // by id, as without an order
    }
    hipLaunchKernelGGL(k_cc_zero, dim3(blocks(v.n_nodes)), dim3(kBlock), 0, s, v.n_nodes, at);
    hipLaunchKernelGGL(k_cc_place, dim3(blocks(v.n_tets)), dim3(kBlock), 0, s, v, at, (int*)nullptr);
    hipLaunchKernelGGL(k_cc_sums, dim3(1), dim3(kWindow), 0, s, v.n_nodes, at);
    hipLaunchKernelGGL(k_cc_place, dim3(blocks(v.n_tets)), dim3(kBlock), 0, s, v, at, q);
    e = hipGetLastError();
    if (e == hipSuccess)
        e = spread(q, &by_vertex);
    if (e == hipSuccess && by_vertex <= by_id / 2)
        *order = q;
    else
        (void)hipFree(q);
    return e;
}

// Component labels into label (device, n_tets); *host and count as above; own,
// f, least: n_nodes ints each.
static hipError_t run_components(const DevView& v, const int* order, int* own, int* f, int* least, uint32_t* count,
                                 uint32_t* host, int32_t* label, hipStream_t s)
{
    const dim3 nodes(std::max(1u, blocks(v.n_nodes)));
    hipLaunchKernelGGL(k_cc_init, nodes, dim3(kBlock), 0, s, v.n_nodes, f, least, own, count);
    const int windows = (v.n_tets + kWindow - 1) / kWindow;
    auto merge = windows > kManyWindows ? (order ? k_cc_windows<true, true> : k_cc_windows<false, true>)
                                        : (order ? k_cc_windows<true, false> : k_cc_windows<false, false>);
    if (windows > 0)
        hipLaunchKernelGGL(merge, dim3(windows), dim3(kWindow), 0, s, v, order, f, own, least);
    hipLaunchKernelGGL(k_cc_roots, nodes, dim3(kBlock), 0, s, v.n_nodes, own, f, least, count);
    hipLaunchKernelGGL(k_cc_label, dim3(std::max(1u, blocks(v.n_tets))), dim3(kBlock), 0, s, v, own, least, label, count,
                       host);
    return hipGetLastError();
}

// Waits for s; the count that the labels' kernel left in pinned memory.
static sta_status read_count(sta_ctx* ctx, hipError_t e, const char* what, int64_t* n_components, hipStream_t s)
{
    if (e == hipSuccess)
        e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        ctx->errmsg = std::string(what) + hipGetErrorString(e);
        return STA_EHIP;
    }
    if (n_components)
        *n_components = *ctx->cc_host;
    return STA_OK;
}

}  // namespace sta

using namespace sta;

extern "C" sta_status sta_components(sta_ctx* ctx, int32_t* labels_dev, int64_t* n_components, void* stream)
{
    if (!ctx || (ctx->n_tets > 0 && !labels_dev))
        return STA_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t n = (size_t)(ctx->n_nodes ? ctx->n_nodes : 1);
    hipError_t e = hipSuccess;
    if (!ctx->cc_ws) {
        void* q = nullptr;
        e = hipMalloc(&q, sizeof(int32_t) * (3 * n + 1));  // the count, three words per vertex
        if (e != hipSuccess) {
            ctx->errmsg = std::string("connectivity workspace: ") + hipGetErrorString(e);
            return STA_ENOMEM;
        }
        ctx->owned.push_back(q);
        ctx->cc_ws = static_cast<int32_t*>(q);
    }
    if (!ctx->cc_host) {
        e = hipHostMalloc((void**)&ctx->cc_host, sizeof(uint32_t), hipHostMallocDefault);
        if (e != hipSuccess) {
            ctx->cc_host = nullptr;
            ctx->errmsg = std::string("connectivity host flag: ") + hipGetErrorString(e);
            return STA_ENOMEM;
        }
    }
    uint32_t* count = reinterpret_cast<uint32_t*>(ctx->cc_ws);
    int* own = ctx->cc_ws + 1;
    if (!ctx->cc_ordered) {
        e = order_tets(ctx->v, count, reinterpret_cast<uint32_t*>(own), &ctx->cc_order, s);
        if (ctx->cc_order)
            ctx->owned.push_back(ctx->cc_order);
        ctx->cc_ordered = e == hipSuccess;
    }
    if (e == hipSuccess)
        e = run_components(ctx->v, ctx->cc_order, own, own + n, own + 2 * n, count, ctx->cc_host, labels_dev, s);
    return read_count(ctx, e, "connectivity: ", n_components, s);
}

extern "C" sta_status sta_face_components(sta_ctx* ctx, int32_t* labels_dev, int64_t* n_components, void* stream)
{
    if (!ctx || (ctx->n_tets > 0 && !labels_dev))
        return STA_EINVAL;
    hipStream_t s = static_cast<hipStream_t>(stream);
    hipError_t e = hipSuccess;
    if (!ctx->ccf_ws) {
        // the candidate face pairs, once per context (the candidate pool is fixed)
        std::vector<int4> T((size_t)ctx->n_tets);
        if (ctx->n_tets > 0)
            e = hipMemcpy(T.data(), ctx->v.T, sizeof(int4) * T.size(), hipMemcpyDeviceToHost);
        if (e != hipSuccess) {
            ctx->errmsg = std::string("face connectivity: ") + hipGetErrorString(e);
            return STA_EHIP;
        }
        const std::vector<int2> pairs = host_face_pairs(T);
        const int64_t windows = std::max<int64_t>(1, (ctx->n_tets + kWindow - 1) / kWindow);
        std::vector<int64_t> start((size_t)windows + 1);
        for (int64_t w = 0, k = 0; w <= windows; ++w) {
            while (k < (int64_t)pairs.size() && pairs[k].x < w * kWindow)
                ++k;
            start[w] = k;
        }
        // the count, the pairs, each window's first pair, three words per tet
        void* q = nullptr;
        const size_t bytes = sizeof(int2) + sizeof(int2) * pairs.size() +
                             sizeof(int64_t) * start.size() + 3 * sizeof(int32_t) * (size_t)ctx->n_tets;
        e = hipMalloc(&q, bytes);
        if (e != hipSuccess) {
            ctx->errmsg = std::string("face connectivity workspace: ") + hipGetErrorString(e);
            return STA_ENOMEM;
        }
        ctx->owned.push_back(q);
        int2* pd = static_cast<int2*>(q) + 1;
        int64_t* sd = reinterpret_cast<int64_t*>(pd + pairs.size());
        if (!pairs.empty())
            e = hipMemcpy(pd, pairs.data(), sizeof(int2) * pairs.size(), hipMemcpyHostToDevice);
        if (e == hipSuccess)
            e = hipMemcpy(sd, start.data(), sizeof(int64_t) * start.size(), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            ctx->errmsg = std::string("face pairs upload: ") + hipGetErrorString(e);
            return STA_EHIP;
        }
        ctx->ccf_ws = static_cast<int32_t*>(q);
        ctx->ccf_pairs = pd;
        ctx->ccf_start = sd;
        ctx->ccf_root = reinterpret_cast<int32_t*>(sd + start.size());
        ctx->ccf_npairs = (int64_t)pairs.size();
    }
    if (!ctx->cc_host) {
        e = hipHostMalloc((void**)&ctx->cc_host, sizeof(uint32_t), hipHostMallocDefault);
        if (e != hipSuccess) {
            ctx->cc_host = nullptr;
            ctx->errmsg = std::string("connectivity host flag: ") + hipGetErrorString(e);
            return STA_ENOMEM;
        }
    }
    e = run_face_components(ctx->v, ctx->ccf_pairs, ctx->ccf_npairs, ctx->ccf_start, ctx->ccf_root,
                            ctx->ccf_root + ctx->n_tets, ctx->ccf_root + 2 * ctx->n_tets, reinterpret_cast<uint32_t*>(ctx->ccf_ws),
                            ctx->cc_host, labels_dev, s);
    return read_count(ctx, e, "face connectivity: ", n_components, s);
}
