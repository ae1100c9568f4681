// Adjoint of the assembly: slot cotangents gA = dL/dvalues -> dL/dlogE per tet
// and dL/dx per node.
//
// For an active tet with element matrix
//   A[3a+i][3b+j] = lamV g_ai g_bj + muV g_aj g_bi + [i=j] muV (g_a.g_b) + [a=b][i=j] m,
// lamV = lambda V dt^2, muV = mu V dt^2, m = rho V / 4, V = |det D| / 6,
// g_k = column k of G = D^-T (k = 1..3), g_0 = -(g_1 + g_2 + g_3), D = [x1-x0, x2-x0, x3-x0]:
// with Abar the 12x12 gather of gA over the tet's slots, B_ab = Abar_ab + Abar_ba^T (B_ba = B_ab^T) and
// C_ab = lambda dt^2 B_ab + mu dt^2 (B_ab^T + tr(B_ab) I):
//   u_ab = C_ab g_b,  P = sum_{a<b} g_a . u_ab + 1/2 sum_a g_a . u_aa,  P_m = 1/2 sum_a tr(B_aa),
//   dL/dlogE = V P                          (lambda, mu proportional to E = exp(logE)),
//   gbar_a = V sum_b u_ab,
//   Vbar = P + (rho/4) P_m,
//   Dbar = -G Gbar^T G + (Vbar sign(det) / 6) det G,  Gbar columns gbar_k - gbar_0,
//   xbar_k = column k of Dbar (k = 1..3), xbar_0 = -(xbar_1 + xbar_2 + xbar_3).
// Inactive tets contribute nothing.  Per-vertex xbar are stored at the tet's
// diagonal incidence positions and summed per node over the node's
// incidence segment in ascending tet id (fixed order, no floating atomics).
#include <hip/hip_runtime.h>

#include <mutex>
#include <string>

#include "sta_internal.h"

#pragma clang fp contract(off)

namespace sta {

namespace {

constexpr int kBlock = 256;

struct Geo {
    double g[4][3];
    double det, V;
};

__device__ __forceinline__ void geometry(const DevView& v, int4 t, Geo& G)
{
    const int id[4] = {t.x, t.y, t.z, t.w};
    double X[4][3];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        X[a][0] = v.xs[id[a]];
        X[a][1] = v.ys[id[a]];
        X[a][2] = v.zs[id[a]];
    }
    double d[4][3];
#pragma unroll
    for (int k = 1; k <= 3; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i)
            d[k][i] = X[k][i] - X[0][i];
    double c[4][3];
    const int nx[4][2] = {{0, 0}, {2, 3}, {3, 1}, {1, 2}};
#pragma unroll
    for (int k = 1; k <= 3; ++k) {
        const double* a = d[nx[k][0]];
        const double* b = d[nx[k][1]];
        c[k][0] = (a[1] * b[2]) - (a[2] * b[1]);
        c[k][1] = (a[2] * b[0]) - (a[0] * b[2]);
        c[k][2] = (a[0] * b[1]) - (a[1] * b[0]);
    }
    const double det = ((d[1][0] * c[1][0]) + (d[1][1] * c[1][1])) + (d[1][2] * c[1][2]);
    const double inv = 1.0 / det;
#pragma unroll
    for (int k = 1; k <= 3; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i)
            G.g[k][i] = c[k][i] * inv;
#pragma unroll
    for (int i = 0; i < 3; ++i)
        G.g[0][i] = -((G.g[1][i] + G.g[2][i]) + G.g[3][i]);
    G.det = det;
    G.V = fabs(det) / 6.0;
}

// The tet's sums over its blocks: both kernels below form the same B_ab and add
// them in the order of the block slots through here, so that a tet's results
// are the same bits whichever of them it falls to (a mesh alone and in a batch
// may differ in that).
struct TetSums {
    double P = 0.0, Pm = 0.0;
    double u[4][3] = {};
};
constexpr int kSlotA[10] = {0, 1, 2, 3, 0, 0, 0, 1, 1, 2}, kSlotB[10] = {0, 1, 2, 3, 1, 2, 3, 2, 3, 3};

__device__ __forceinline__ void add_block(TetSums& s, const Geo& G, int a, int b, const double (&B)[3][3],
                                          double lam_dt, double mu_dt)
{
    const double* ga = G.g[a];
    const double* gb = G.g[b];
    const double tr = (B[0][0] + B[1][1]) + B[2][2], t = mu_dt * tr;
    double C[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            C[i][j] = lam_dt * B[i][j] + mu_dt * B[j][i];
    double ua[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        ua[i] = ((C[i][0] * gb[0] + C[i][1] * gb[1]) + C[i][2] * gb[2]) + t * gb[i];
        s.u[a][i] += ua[i];
    }
    const double p = (ga[0] * ua[0] + ga[1] * ua[1]) + ga[2] * ua[2];
    if (a == b) {
        s.P += 0.5 * p;
        s.Pm += 0.5 * tr;
    } else {
        s.P += p;
#pragma unroll
        for (int i = 0; i < 3; ++i)
            s.u[b][i] += ((C[0][i] * ga[0] + C[1][i] * ga[1]) + C[2][i] * ga[2]) + t * ga[i];
    }
}

// dL/dlogE of the tet and its vertices' xbar from its sums.
__device__ __forceinline__ void store_tet(const DevView& v, const TetSums& s, const Geo& G, double* g_logE,
                                          double* xbar, const int* pos)
{
    *g_logE = G.V * s.P;
    const double Vbar = s.P + 0.25 * v.mat.rho * s.Pm;
    const double detbar = Vbar * (G.det < 0.0 ? -1.0 : 1.0) / 6.0;
    // Gbar columns k = 1..3: gbar_k - gbar_0 ; G columns g_k
    double Gm[3][3], Gb[3][3];  // [row i][col k-1]
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            Gm[i][k] = G.g[k + 1][i];
            Gb[i][k] = G.V * s.u[k + 1][i] - G.V * s.u[0][i];
        }
    // Dbar = -G Gbar^T G + detbar det G
    double T1[3][3];  // Gbar^T G
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            T1[i][j] = (Gb[0][i] * Gm[0][j] + Gb[1][i] * Gm[1][j]) + Gb[2][i] * Gm[2][j];
    double Db[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            Db[i][j] = -((Gm[i][0] * T1[0][j] + Gm[i][1] * T1[1][j]) + Gm[i][2] * T1[2][j]) +
                       detbar * G.det * Gm[i][j];
    double xb[4][3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        xb[1][i] = Db[i][0];
        xb[2][i] = Db[i][1];
        xb[3][i] = Db[i][2];
        xb[0][i] = -((Db[i][0] + Db[i][1]) + Db[i][2]);
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        double* dst = xbar + 3 * (size_t)pos[a];
        dst[0] = xb[a][0];
        dst[1] = xb[a][1];
        dst[2] = xb[a][2];
    }
}

// Zeros of an inactive tet.
__device__ __forceinline__ void store_inactive(double* g_logE, double* xbar, const int* pos)
{
    *g_logE = 0.0;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        double* dst = xbar + 3 * (size_t)pos[a];
        dst[0] = 0.0;
        dst[1] = 0.0;
        dst[2] = 0.0;
    }
}

// The tet's sums from its 144 cotangents.
__device__ __forceinline__ void gather_sums(TetSums& s, const DevView& v, const double* __restrict__ gA, int e, int4 T,
                                            const Geo& G, double lam_dt, double mu_dt)
{
    const int id[4] = {T.x, T.y, T.z, T.w};
    const int* eb = v.e2b + 10 * (size_t)e;
#pragma unroll
    for (int q = 0; q < 10; ++q) {
        // Abar_ab stands in the upper copy if vertex a is the smaller node, in the mirror otherwise
        const BlockDesc d = v.desc[eb[q]];
        const int a = kSlotA[q], b = kSlotB[q];
        const bool swap = id[a] > id[b];
        const int pa = swap ? d.lo : d.up, la = swap ? d.rlj : d.rl, pb = swap ? d.up : d.lo, lb = swap ? d.rl : d.rlj;
        double Aab[3][3], Aba[3][3], B[3][3];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                Aab[i][j] = gA[pa + i * la + j];
                Aba[i][j] = a == b ? Aab[i][j] : gA[pb + i * lb + j];
            }
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j)
                B[i][j] = Aab[i][j] + Aba[j][i];
        add_block(s, G, a, b, B, lam_dt, mu_dt);
    }
}

// Every tet gathers its 144 cotangents: for meshes of few bricks (below), which
// would leave most of the chip idle.  Workgroups of one wave, so that the waves
// are spread over the compute units: 16.1 us at 48,000 tets, 23.5 at 82,944,
// where workgroups of four took 17.2 and 26.2.
constexpr int kDirect = 64;
__global__ __launch_bounds__(kDirect) void k_adjoint_direct(DevView v, const int32_t* __restrict__ order,
                                                            int32_t n_chunks, const double* __restrict__ gA,
                                                            double* __restrict__ g_logE,
                                                            double* __restrict__ xbar)
{
    // each XCD takes one contiguous share of the chunk order, chunks that are
    // near in space: neighbouring tets share node blocks, so their cotangent
    // rows stay in one L2
    constexpr int kPer = kDirect / kAdjointChunk;
    const int slot = xcd_remap(blockIdx.x, gridDim.x) * kPer + threadIdx.x / kAdjointChunk;
    if (slot >= n_chunks)
        return;
    const int e = order[slot] * kAdjointChunk + (threadIdx.x % kAdjointChunk);
    if (e >= v.n_tets)
        return;
    const int* pos = v.e2p + 10 * (size_t)e;
    if (!v.mask[e]) {
        store_inactive(g_logE + e, xbar, pos);
        return;
    }
    const int4 t = v.T[e];
    Geo G;
    geometry(v, t, G);
    const double E = v.E[e];
    TetSums s;
    gather_sums(s, v, gA, e, t, G, (E * v.mat.clam) * v.mat.cdt, (E * v.mat.cmu) * v.mat.cdt);
    store_tet(v, s, G, g_logE + e, xbar, pos);
}

// A brick of kAdjointBrick tets that are near in space (kBrickChunks chunks of
// the Morton order) shares most of its blocks: 128
// tets name 1,280 blocks, about 330 of them different.  So the brick's
// different blocks are formed once, in LDS, and each tet reads its ten from
// there.
//
// Per brick the plan lists the row blocks to read (one per diagonal block, two
// per other block) in the order of their place in the values, so that lanes
// side by side read runs of the rows, as (position, row length, block number |
// kind), the blocks numbered in ascending id; and per tet slot ten references,
// block number | transpose << 15.  (Two lists, upper copies and mirrors, read
// every line of the rows twice: 78 instead of 72 us a call.)
constexpr int kBrickBlocks = 10 * kAdjointBrick, kBrickReads = 2 * kBrickBlocks;  // most a brick can have
// Fewer bricks (4 a compute unit) and every tet gathers for itself: the whole
// adjoint, gathered / by bricks, 12.0 / 15.6 us at 1,296 tets, 16.1 / 21.8 at
// 48,000, 28.3 / 31.5 at 105,456, 35.1 / 34.7 at 131,712, 39.6 / 42.4 at 162,000,
// 56.3 / 53.8 at 235,824 (this depends on how the cells' rows fall into chunks).
constexpr int kMinBricks = 1024;
// Fewer active tets of a brick gather for themselves (in a refinement superset
// most candidates are inactive): 384,000 tets of which 5, 10, 25, 50 per cent are
// active, at random, by bricks 60 us each, gathered 46, 47, 55, 67.
constexpr int kFewActive = 40;
constexpr int kBrickTable = 4096;  // hash slots while a brick's blocks are found
constexpr int kEntryWords = 3;
constexpr int kMirror = 1 << 15, kDiagonal = 1 << 14;
static_assert(kBrickBlocks < kBrickTable && kBrickBlocks < kDiagonal, "every block finds a place and a number");

// Tet of slot t of a brick, or -1.
__device__ __forceinline__ int brick_tet(const DevView& v, const int32_t* __restrict__ order, int brick, int t)
{
    const int c = order[brick * kBrickChunks + t / kAdjointChunk];
    const int e = c * kAdjointChunk + t % kAdjointChunk;
    return c >= 0 && e < v.n_tets ? e : -1;
}

// Ranks of kMine values per thread among the n different values of list.
template <int kMine>
__device__ __forceinline__ void rank_among(const int* list, int n, const int (&v)[kMine], int (&r)[kMine])
{
#pragma unroll
    for (int u = 0; u < kMine; ++u)
        r[u] = 0;
    for (int i = 0; i < n; ++i) {
        const int x = list[i];
#pragma unroll
        for (int u = 0; u < kMine; ++u)
            r[u] += x < v[u] ? 1 : 0;
    }
}

// Plan of one brick per workgroup.  fill = false: only how many row blocks it
// reads, into starts, and how many blocks it has, into entries; true: its
// entries, starts being the running sum by then, and its references.
template <bool kFill>
__global__ __launch_bounds__(kAdjointBrick) void k_adjoint_plan(DevView v, const int32_t* __restrict__ order,
                                                                AdjointPlan plan)
{
    __shared__ int s_key[kBrickTable];      // block of each hash slot, -1: free
    __shared__ uint16_t s_at[kBrickTable];  // its place in s_list
    __shared__ int s_list[kBrickBlocks], s_pos[kBrickReads];
    __shared__ uint16_t s_rank[kBrickBlocks], s_src[kBrickReads];
    __shared__ int s_n, s_m;
    constexpr int kMine = kBrickBlocks / kAdjointBrick;
    const int t = threadIdx.x, brick = blockIdx.x;
    for (int k = t; k < kBrickTable; k += kAdjointBrick)
        s_key[k] = -1;
    if (t == 0)
        s_n = s_m = 0;
    __syncthreads();
    const int e = brick_tet(v, order, brick, t);
    int slot[10];
#pragma unroll
    for (int q = 0; q < 10; ++q) {
        slot[q] = 0;
        if (e >= 0) {
            const int key = v.e2b[10 * (size_t)e + q];
            unsigned h = ((unsigned)key * 2654435761u) >> 20;
            for (;; h = (h + 1) & (kBrickTable - 1)) {  // ends: the table holds more than all references
                const int old = atomicCAS(&s_key[h], -1, key);
                if (old == -1) {
                    const int at = atomicAdd(&s_n, 1);
                    s_list[at] = key;
                    s_at[h] = (uint16_t)at;
                    atomicAdd(&s_m, key < v.nd ? 1 : 2);
                }
                if (old == -1 || old == key)
                    break;
            }
            slot[q] = (int)h;
        }
    }
    __syncthreads();
    const int n = s_n, m = s_m;
    if (!kFill) {
        if (t == 0) {
            plan.starts[brick] = m;
            plan.entries[brick] = n;
        }
        return;
    }
    int key[kMine], rank[kMine];
#pragma unroll
    for (int u = 0; u < kMine; ++u)
        key[u] = t + u * kAdjointBrick < n ? s_list[t + u * kAdjointBrick] : -1;
    rank_among<kMine>(s_list, n, key, rank);
    __syncthreads();
    if (t == 0)
        s_m = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kMine; ++u) {
        if (key[u] < 0)
            continue;
        const int i = t + u * kAdjointBrick;
        s_rank[i] = (uint16_t)rank[u];
        const BlockDesc d = v.desc[key[u]];
        const int at = atomicAdd(&s_m, d.kind == 0 ? 1 : 2);
        s_pos[at] = d.up;
        s_src[at] = (uint16_t)i;
        if (d.kind != 0) {
            s_pos[at + 1] = d.lo;
            s_src[at + 1] = (uint16_t)(i | kMirror);
        }
    }
    __syncthreads();
    constexpr int kPass = 5;  // row blocks ranked per thread and pass: a typical brick takes one
    for (int k0 = t; k0 - t < m; k0 += kPass * kAdjointBrick) {
        int pos[kPass], at[kPass];
#pragma unroll
        for (int u = 0; u < kPass; ++u)
            pos[u] = k0 + u * kAdjointBrick < m ? s_pos[k0 + u * kAdjointBrick] : -1;
        rank_among<kPass>(s_pos, m, pos, at);
#pragma unroll
        for (int u = 0; u < kPass; ++u) {
            if (pos[u] < 0)
                continue;
            const int src = s_src[k0 + u * kAdjointBrick], mirror = src & kMirror;
            const BlockDesc d = v.desc[s_list[src & ~kMirror]];
            int32_t* o = plan.entries + kEntryWords * ((size_t)plan.starts[brick] + at[u]);
            o[0] = pos[u];
            o[1] = mirror ? d.rlj : d.rl;
            o[2] = s_rank[src & ~kMirror] | (d.kind == 0 ? kDiagonal : mirror);
        }
    }
    const int4 T = e >= 0 ? v.T[e] : make_int4(0, 0, 0, 0);
    const int id[4] = {T.x, T.y, T.z, T.w};
#pragma unroll
    for (int q = 0; q < 10; ++q) {
        const unsigned swap = id[kSlotA[q]] > id[kSlotB[q]] ? 1u << 15 : 0u;
        plan.refs[((size_t)brick * 10 + q) * kAdjointBrick + t] =
            e >= 0 ? (uint16_t)(s_rank[s_at[slot[q]]] | swap) : (uint16_t)0;
    }
}

// One brick per workgroup, one tet per lane; s_blocks: the brick's blocks, 9
// doubles each, row node = the smaller node.  Bound by latency and by the
// address units at about 10 waves a CU: staging 20 k clocks, of which the
// reads are most, the tets' sums 8 k, the first chain 5 k.  At the fracture
// mesh of resolution 40 (384,000 tets) 50 us (64 with every tet gathering its
// 144 cotangents), the whole adjoint 72 (97).  Bricks of 64 tets, 8 rounds in
// flight, whole rows per lane and atomic adds in LDS measured 71 to 82.
__global__ __launch_bounds__(kAdjointBrick) void k_adjoint_element(DevView v, const int32_t* __restrict__ order,
                                                                   AdjointPlan plan,
                                                                   const double* __restrict__ gA,
                                                                   double* __restrict__ g_logE,
                                                                   double* __restrict__ xbar)
{
    extern __shared__ double s_blocks[];
    __shared__ int s_active[kAdjointBrick / 64];
    // each XCD takes one contiguous share of the bricks: neighbouring bricks share rows in its L2
    const int brick = xcd_remap(blockIdx.x, gridDim.x), t = threadIdx.x;
    const int e = brick_tet(v, order, brick, t);
    const int start = plan.starts[brick], m = plan.starts[brick + 1] - start;
    const int32_t* __restrict__ entries = plan.entries + (size_t)kEntryWords * start;
    // the tet's own data, in flight while the blocks are formed
    const int ee = e >= 0 ? e : 0;
    const uint8_t active = v.mask[ee];
    const int4 T = v.T[ee];
    const double E = v.E[ee];
    int pos[4];
    unsigned ref[10];
#pragma unroll
    for (int a = 0; a < 4; ++a)
        pos[a] = v.e2p[10 * (size_t)ee + a];
#pragma unroll
    for (int q = 0; q < 10; ++q)
        ref[q] = plan.refs[((size_t)brick * 10 + q) * kAdjointBrick + t];
    // three lanes per row block (its columns), 21 row blocks per wave and round,
    // kAhead rounds in flight: a typical brick's 600 row blocks at once.  The
    // upper copies are stored, then the mirrors added transposed (a diagonal
    // block's copy is both).  Loads past the last row block take its data.
    constexpr int kWaveBlocks = 21, kRound = kAdjointBrick / 64 * kWaveBlocks, kAhead = 15, kBatch = kAhead * kRound;
    const int j = (t & 63) % 3, first = (t & 63) < 63 ? (t >> 6) * kWaveBlocks + (t & 63) / 3 : 1 << 20;
    double x[kAhead][3];
    int what[kAhead], at[kAhead], rl[kAhead];
    auto load_entries = [&](int b0) {
#pragma unroll
        for (int w = 0; w < kAhead; ++w) {
            const int k = b0 + first + w * kRound;
            const int32_t* o = entries + kEntryWords * min(k, m - 1);
            at[w] = o[0];
            rl[w] = o[1];
            what[w] = o[2] | ((m - 1 - k) >> 31);  // -1 past the end
        }
    };
    auto load_rows = [&]() {
#pragma unroll
        for (int w = 0; w < kAhead; ++w)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                x[w][i] = gA[at[w] + i * rl[w] + j];
    };
    auto store_uppers = [&]() {
#pragma unroll
        for (int w = 0; w < kAhead; ++w)
            if (what[w] >= 0 && !(what[w] & kMirror)) {
                double* dst = s_blocks + 9 * (what[w] & (kDiagonal - 1)) + j;
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    dst[3 * i] = x[w][i];
            }
    };
    auto add_mirrors = [&]() {
#pragma unroll
        for (int w = 0; w < kAhead; ++w)
            if (what[w] >= 0 && (what[w] & (kMirror | kDiagonal))) {
                double* dst = s_blocks + 9 * (what[w] & (kDiagonal - 1)) + 3 * j;
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    dst[i] = dst[i] + x[w][i];
            }
    };
    load_entries(0);
    // few active tets gather for themselves
    const int mine = __popcll(__ballot(e >= 0 && active));
    if ((t & 63) == 0)
        s_active[t >> 6] = mine;
    __syncthreads();
    if (s_active[0] + s_active[1] < kFewActive) {
        if (e >= 0 && active) {
            Geo G;
            geometry(v, T, G);
            TetSums s;
            gather_sums(s, v, gA, e, T, G, (E * v.mat.clam) * v.mat.cdt, (E * v.mat.cmu) * v.mat.cdt);
            store_tet(v, s, G, g_logE + e, xbar, pos);
        } else if (e >= 0) {
            store_inactive(g_logE + e, xbar, pos);
        }
        return;
    }
    for (int b0 = kBatch; b0 < m; b0 += kBatch) {  // rows past the first batch are read twice
        load_entries(b0);
        load_rows();
        store_uppers();
    }
    if (m > kBatch)
        load_entries(0);
    load_rows();
    store_uppers();
    __syncthreads();
    add_mirrors();
    for (int b0 = kBatch; b0 < m; b0 += kBatch) {
        load_entries(b0);
        load_rows();
        add_mirrors();
    }
    Geo G;
    geometry(v, T, G);
    __syncthreads();
    if (e < 0)
        return;
    if (!active) {
        store_inactive(g_logE + e, xbar, pos);
        return;
    }
    const double lam_dt = (E * v.mat.clam) * v.mat.cdt;  // lambda dt^2
    const double mu_dt = (E * v.mat.cmu) * v.mat.cdt;    // mu dt^2
    TetSums s;
#pragma unroll
    for (int q = 0; q < 10; ++q) {
        const double* r = s_blocks + 9 * (ref[q] & 0x7fffu);
        const int x = ref[q] >> 15 ? 2 : 0;  // transposed: entries 1 3, 2 6 and 5 7 change places
        const double B[3][3] = {{r[0], r[1 + x], r[2 + 2 * x]},
                                {r[3 - x], r[4], r[5 + x]},
                                {r[6 - 2 * x], r[7 - x], r[8]}};
        add_block(s, G, kSlotA[q], kSlotB[q], B, lam_dt, mu_dt);
    }
    store_tet(v, s, G, g_logE + e, xbar, pos);
}

// dL/dx of node i, component c: its diagonal segment's xbar in ascending tet id.
// Terms are loaded kChunk at a time and then added in order, so that a
// segment costs a few memory round trips instead of one per term.
__global__ __launch_bounds__(kBlock) void k_adjoint_nodes(DevView v, const double* __restrict__ xbar,
                                                          double* __restrict__ g_x)
{
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= 3 * v.n_nodes)
        return;
    const int i = t / 3, c = t - 3 * (t / 3);
    const int b = v.ndiag[i];
    double acc = 0.0;
    if (b >= 0) {
        const BlockDesc d = v.desc[b];
        constexpr int kChunk = 8;
        for (int k0 = d.k0; k0 < d.k1; k0 += kChunk) {
            double x[kChunk];
#pragma unroll
            for (int j = 0; j < kChunk; ++j)
                x[j] = k0 + j < d.k1 ? xbar[3 * (size_t)(k0 + j) + c] : 0.0;
#pragma unroll
            for (int j = 0; j < kChunk; ++j)
                if (k0 + j < d.k1)
                    acc = acc + x[j];
        }
    }
    g_x[t] = acc;
}

// out[slot(r, c)] = alpha * a[r] * b[c] over the pattern.
__global__ __launch_bounds__(kBlock) void k_slot_outer(int n_rows, const int32_t* __restrict__ rowptr,
                                                       const int32_t* __restrict__ colidx, const double* __restrict__ a,
                                                       const double* __restrict__ b, double alpha,
                                                       double* __restrict__ out)
{
    const int r = blockIdx.x * (kBlock / 16) + threadIdx.x / 16;
    const int l = threadIdx.x & 15;
    if (r >= n_rows)
        return;
    const double ar = alpha * a[r];
    for (int s = rowptr[r] + l; s < rowptr[r + 1]; s += 16)
        out[s] = ar * b[colidx[s]];
}

}  // namespace

// 0: the mesh is too small for bricks.
int adjoint_bricks(int n_chunks)
{
    const int bricks = (n_chunks + kBrickChunks - 1) / kBrickChunks;
    return bricks < kMinBricks ? 0 : bricks;
}

hipError_t launch_adjoint_plan(const DevView& v, const int32_t* order, const AdjointPlan& plan, bool fill, hipStream_t s)
{
    if (plan.bricks == 0)
        return hipSuccess;
    if (fill)
        hipLaunchKernelGGL(k_adjoint_plan<true>, dim3(plan.bricks), dim3(kAdjointBrick), 0, s, v, order, plan);
    else
        hipLaunchKernelGGL(k_adjoint_plan<false>, dim3(plan.bricks), dim3(kAdjointBrick), 0, s, v, order, plan);
    return hipGetLastError();
}

hipError_t launch_adjoint(const DevView& v, const int32_t* order, int32_t n_chunks, const AdjointPlan& plan,
                          const double* gA, double* g_logE, double* g_x, double* xbar, hipStream_t s)
{
    if (v.n_tets > 0 && plan.bricks == 0)
        hipLaunchKernelGGL(k_adjoint_direct, dim3((n_chunks * kAdjointChunk + kDirect - 1) / kDirect), dim3(kDirect), 0, s,
                           v, order, n_chunks, gA, g_logE, xbar);
    else if (v.n_tets > 0)
        hipLaunchKernelGGL(k_adjoint_element, dim3(plan.bricks), dim3(kAdjointBrick), 9 * sizeof(double) * plan.most, s,
                           v, order, plan, gA, g_logE, xbar);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || v.n_nodes == 0)
        return e;
    hipLaunchKernelGGL(k_adjoint_nodes, dim3((3 * v.n_nodes + kBlock - 1) / kBlock), dim3(kBlock), 0, s, v, xbar,
                       g_x);
    return hipGetLastError();
}

hipError_t launch_slot_outer(int n_rows, const int32_t* rowptr, const int32_t* colidx, const double* a,
                             const double* b, double alpha, double* out, hipStream_t s)
{
    if (n_rows == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_slot_outer, dim3((n_rows + kBlock / 16 - 1) / (kBlock / 16)), dim3(kBlock), 0, s, n_rows,
                       rowptr, colidx, a, b, alpha, out);
    return hipGetLastError();
}

}  // namespace sta

// ---------------------------------------------------------------------------
// Adjoint without allocation: the per-vertex cotangents live in a fixed
// device array of the library instead of a context workspace.
// ---------------------------------------------------------------------------

namespace {

// 3 doubles per diagonal incidence (4 per tet): room for 524,288 tets.
constexpr size_t kNoAllocTets = size_t(1) << 19;
constexpr size_t kNoAllocDoubles = 12 * kNoAllocTets;  // 48 MiB

static __device__ __align__(256) double scratch[kNoAllocDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's copy of `scratch`, looked up once per
// device (the current one); NULL on failure.
double* scratch_for_current_device(hipError_t& err)
{
    int dev = -1;
    err = hipGetDevice(&dev);
    if (err != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        if (err == hipSuccess)
            err = hipErrorInvalidDevice;
        return nullptr;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess)
            return nullptr;
        g_scratch_ptr[dev] = static_cast<double*>(p);
    }
    return g_scratch_ptr[dev];
}

}  // namespace

extern "C" sta_status sta_adjoint_noalloc(sta_ctx* ctx, const double* gA_dev, double* g_logE_dev, double* g_x_dev,
                                          void* stream)
{
    if (!ctx || (ctx->nnz > 0 && !gA_dev) || (ctx->n_tets > 0 && !g_logE_dev) || (ctx->n_nodes > 0 && !g_x_dev))
        return STA_EINVAL;
    if ((size_t)ctx->n_tets > kNoAllocTets) {
        ctx->errmsg = "sta_adjoint_noalloc: " + std::to_string(ctx->n_tets) + " tets exceed the fixed workspace (" +
                      std::to_string(kNoAllocTets) + " tets); use sta_adjoint";
        return STA_EINVAL;
    }
    if (ctx->stale) {
        ctx->errmsg = "parameters changed: call sta_full_rebuild before sta_adjoint_noalloc";
        return STA_ESTALE;
    }
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess && dev != ctx->device) {
        ctx->errmsg = "sta_adjoint_noalloc: the current device is not the context's device";
        return STA_EINVAL;
    }
    double* xbar = e == hipSuccess ? scratch_for_current_device(e) : nullptr;
    if (!xbar) {
        ctx->errmsg = std::string("sta_adjoint_noalloc: workspace address: ") + hipGetErrorString(e);
        return STA_EHIP;
    }
    // every diagonal incidence's three entries are written by the element pass
    // before the node pass reads them, so nothing needs clearing
    e = sta::launch_adjoint(ctx->v, ctx->adj_order, ctx->adj_chunks, ctx->adj_plan, gA_dev, g_logE_dev, g_x_dev, xbar,
                            static_cast<hipStream_t>(stream));
    if (e != hipSuccess) {
        ctx->errmsg = std::string("sta_adjoint_noalloc launch: ") + hipGetErrorString(e);
        return STA_EHIP;
    }
    return STA_OK;
}
