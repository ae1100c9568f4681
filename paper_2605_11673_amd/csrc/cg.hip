// Jacobi-preconditioned conjugate gradients on the assembled CSR matrix (the
// paper's solve step: Sec. 4 and Alg. 1 solve A_t x_t = b_t by CG with a
// diagonal preconditioner).  Dofs whose diagonal is zero (nodes with no
// active tet: their rows and columns are all zero) are held at 0.
//
// All scalars stay on the device; each kernel returns at once when the
// solve has converged, so the host only synchronises every few iterations.
// Dot products use fixed reduction trees (a per-workgroup tree, then a sum
// over the workgroups' partials in index order): results are reproducible
// run to run.
//
// One iteration is two launches.  The matrix-vector product sums the previous
// update's partials of r.z and r.r (every workgroup the same way, so all get
// the same bits), checks convergence, forms beta, and builds the new search
// direction p = z + beta p on the fly.  The update then sums the product's
// partials of p.Ap into alpha and updates x, r, z with partials of r.z and
// r.r.  The product works per node: the three rows of a node share one column
// list (3x3 blocks), so a group of lanes walks the node's neighbours once,
// reading one neighbour and one record of its z and p for all three rows.
//
// Both kernels are bound by latency (their data, 72 MB of values and 2 MB a
// vector on the 207k-row fracture system, come from the Infinity Cache): every
// load that does not need the scalars is issued before the partials are
// summed, z and p of a node are one 48-byte record (two copies, written in
// turn), and each node's first 16 neighbours stand at a fixed place, so that
// the product is two round trips deep.  Sums over a workgroup go through
// cross-lane moves and one barrier.  Per iteration of the 207k-row system 20.6
// + 6.4 -> 15.4 + 5.8 us (the product at 5.3 TB/s), of a 5k-row one 6.5 + 4.5
// -> 4.6 + 3.3 us.  Loading a round's neighbours a round ahead, and product
// grids of 768 to 4,320 workgroups, gave 5.0 to 5.9 ms for a solve that takes
// 5.1 at 2,048.
#include <hip/hip_runtime.h>

#include "sta_internal.h"

namespace sta {

namespace {

typedef double dvec2 __attribute__((ext_vector_type(2)));

constexpr int kBlock = 256;
constexpr int kNodeLanes = kCgNeighbours;  // lanes per node (three CSR rows) in the matrix-vector product
constexpr int kGroups = kBlock / kNodeLanes;
#ifndef STA_CG_SPMV_GRID
#define STA_CG_SPMV_GRID 2048
#endif
#ifndef STA_CG_UPDATE_GRID
#define STA_CG_UPDATE_GRID 256
#endif
constexpr int kSpmvGridMax = STA_CG_SPMV_GRID;
constexpr int kUpdateGridMax = STA_CG_UPDATE_GRID;
static_assert(kUpdateGridMax <= kBlock, "one lane holds one partial of the update");

// x plus the x of the lane that a DPP control names.
template <int kCtrl>
__device__ __forceinline__ double add_dpp(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, 0xf, 0xf, false);
    return x + __longlong_as_double((long long)hi << 32 | (unsigned)lo);
}

// The same for the rows of 16 lanes that kRows names; others add 0.
template <int kCtrl, int kRows>
__device__ __forceinline__ double add_dpp_rows(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, kRows, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRows, 0xf, false);
    return x + __longlong_as_double((long long)hi << 32 | (unsigned)lo);
}

// Sum over each aligned group of 16 lanes, the same bits in all of them: lanes
// 1 and 2 apart (quad permutations), then the mirrored half row and row (all
// lanes of a quad, then of a half row, hold the same sum by then).
__device__ __forceinline__ double sum16(double x)
{
    x = add_dpp<0xB1>(x);   // quad_perm 1 0 3 2
    x = add_dpp<0x4E>(x);   // quad_perm 2 3 0 1
    x = add_dpp<0x141>(x);  // row_half_mirror
    return add_dpp<0x140>(x);  // row_mirror
}

__device__ __forceinline__ double sum64(double x)
{
    x = sum16(x);
    x = x + __shfl_xor(x, 16, 64);
    return x + __shfl_xor(x, 32, 64);
}

constexpr int kWaves = kBlock / 64;

// Workgroup sums of one or two values per thread, valid in every thread; sh
// (kWaves doubles per value) must not be in use.
__device__ __forceinline__ double block_sum(double x, double* sh)
{
    x = sum64(x);
    if ((threadIdx.x & 63) == 0)
        sh[threadIdx.x >> 6] = x;
    __syncthreads();
    return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

__device__ __forceinline__ void block_sum2(double x, double y, double* sh, double& sx, double& sy)
{
    x = sum64(x);
    y = sum64(y);
    if ((threadIdx.x & 63) == 0) {
        sh[threadIdx.x >> 6] = x;
        sh[kWaves + (threadIdx.x >> 6)] = y;
    }
    __syncthreads();
    sx = (sh[0] + sh[1]) + (sh[2] + sh[3]);
    sy = (sh[4] + sh[5]) + (sh[6] + sh[7]);
}

// This thread's share of partials[0..n): t, t + 256, ... in order, eight loads
// at a time before their additions.
__device__ __forceinline__ double share_of_partials(const double* __restrict__ p, int n)
{
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 8 * kBlock) {
        double t[8];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            t[k] = i + k * kBlock < n ? p[i + k * kBlock] : 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            acc = acc + t[k];
    }
    return acc;
}

__global__ __launch_bounds__(kBlock) void k_cg_init(CgView c, const double* __restrict__ b)
{
    __shared__ double sh[2 * kWaves];
    const int r = blockIdx.x * kBlock + threadIdx.x;
    double rz = 0.0, bb = 0.0;
    if (r < c.n) {
        const int pos = c.dpos[r];
        const double d = pos >= 0 ? c.vals[pos] : 0.0;
        const double di = d != 0.0 ? 1.0 / d : 0.0;
        const double br = d != 0.0 ? b[r] : 0.0;
        c.dinv[r] = di;
        c.x[r] = 0.0;
        c.r[r] = br;
        const double z = br * di;
        double* zp = c.zp + 6 * (size_t)(r / 3) + r % 3;
        zp[0] = z;
        zp[3] = 0.0;  // p_0 = z_0 + 0 * 0, formed by the first product
        rz = br * z;
        bb = br * br;
    }
    double s1, s2;
    block_sum2(rz, bb, sh, s1, s2);
    if (threadIdx.x == 0) {
        c.part[blockIdx.x] = s1;
        c.part[c.nparts + blockIdx.x] = s2;
    }
}

__global__ __launch_bounds__(kBlock) void k_cg_init_finish(CgView c, double rtol)
{
    __shared__ double sh[2 * kWaves];
    double rz, bb;
    block_sum2(share_of_partials(c.part, c.nparts), share_of_partials(c.part + c.nparts, c.nparts), sh, rz, bb);
    if (threadIdx.x == 0) {
        c.s->rz = rz;
        c.s->rzk[0] = rz;
        c.s->bnorm2 = bb;
        c.s->rr = bb;
        c.s->beta = 0.0;
        c.s->tol2 = (rtol * rtol) * bb;
        c.s->iters = 0;
        c.s->done = bb == 0.0 ? 1 : 0;
    }
}

// Iteration k, first launch.  For k > 0: r_k.z_k and r_k.r_k from the update's
// partials; stop if converged or k reaches max_iter; beta = (r_k.z_k) /
// (r_{k-1}.z_{k-1}).  Then p_new = z + beta p_old and q = A p_new, with the
// partials of p_new . q.  kNodeLanes lanes per node; lane l takes neighbours
// l, l + kNodeLanes, ...; the three row sums are combined by a fixed tree.  The
// records of copy cur are read, p_new goes into the other copy.
//
// Node groups of kGroups nodes: with at least kXcds workgroups each XCD walks
// one contiguous share of them (its workgroups in turn), so that neighbouring
// nodes, which gather the same records, stay in one L2; otherwise a plain
// grid-stride.  All groups of a workgroup run the same number of rounds.
__global__ __launch_bounds__(kBlock) void k_cg_spmv(CgView c, int k, int cur, int max_iter)
{
    __shared__ double sh[2 * kWaves], sh2[kWaves];
    const int nn = c.n / 3;
    const int group = threadIdx.x / kNodeLanes, l = threadIdx.x & (kNodeLanes - 1);
    const int ngroups = (nn + kGroups - 1) / kGroups;
    int g0 = blockIdx.x, g1 = ngroups, gstep = gridDim.x;
    if ((int)gridDim.x >= kXcds) {
        const int xcd = blockIdx.x % kXcds, G = gridDim.x;
        g0 = (int)((int64_t)ngroups * xcd / kXcds) + blockIdx.x / kXcds;
        g1 = (int)((int64_t)ngroups * (xcd + 1) / kXcds);
        gstep = G / kXcds + (xcd < G % kXcds ? 1 : 0);  // workgroups on this XCD
    }
    const double* __restrict__ zp = c.zp + (cur ? 2 * (size_t)c.n : 0);
    double* __restrict__ zp_new = c.zp + (cur ? 0 : 2 * (size_t)c.n);
    // what this lane needs of node group gi before the scalars are known
    struct Lane {
        int i, base, rl, j;         // node, its rows' start and length, neighbour (-1: none)
        dvec2 n[3];                 // the neighbour's z and p
        double v[3][3];             // the block
        double z, p, di;            // lanes 0..2: the node's own row
    };
    auto first_trip = [&](int gi, Lane& a) {
        const int i = gi * kGroups + group;
        a.i = i < nn && gi < g1 ? i : -1;
        const int ii = a.i >= 0 ? i : 0;
        a.base = c.rowptr[3 * ii];
        a.rl = c.rowptr[3 * ii + 1] - a.base;
        a.j = c.adj[kNodeLanes * (size_t)ii + l];
        const int own = l < 3 ? l : 0;
        a.z = zp[6 * (size_t)ii + own];
        a.p = zp[6 * (size_t)ii + 3 + own];
        a.di = c.dinv[3 * (size_t)ii + own];
    };
    auto second_trip = [&](Lane& a) {
        if (a.j >= 0 && a.i >= 0) {
            const dvec2* r = reinterpret_cast<const dvec2*>(zp + 6 * (size_t)a.j);
            const double* v = c.vals + a.base + 3 * l;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                a.n[q] = r[q];
#pragma unroll
                for (int w = 0; w < 3; ++w)
                    a.v[q][w] = v[q * a.rl + w];
            }
        }
    };
    Lane a;
    first_trip(g0 < g1 ? g0 : 0, a);
    double rz = 0.0, rr = 0.0;
    if (k > 0 && (int)threadIdx.x < c.nparts_u) {
        rz = c.part[c.nparts_s + threadIdx.x];
        rr = c.part[c.nparts_s + c.nparts_u + threadIdx.x];
    }
    const int done = c.s->done;
    const double tol2 = c.s->tol2, rz_old = c.s->rzk[(k - 1) & 1], rz0 = c.s->rzk[0], rr0 = c.s->rr;
    if (g0 >= g1)
        a.i = -1;
    second_trip(a);
    if (done)
        return;
    double beta = 0.0;
    if (k > 0) {
        block_sum2(rz, rr, sh, rz, rr);
    } else {
        rz = rz0;
        rr = rr0;
    }
    if ((k > 0 && rr <= tol2) || k >= max_iter) {
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            c.s->rr = rr;
            c.s->iters = k;
            c.s->done = 1;
        }
        return;
    }
    if (k > 0) {
        beta = rz / rz_old;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            c.s->rzk[k & 1] = rz;
            c.s->rr = rr;
            c.s->iters = k;
        }
    }
    double pq = 0.0;
    for (int gi = g0; gi < g1; gi += gstep) {
        if (gi != g0) {
            first_trip(gi, a);
            second_trip(a);
        }
        double s0 = 0.0, s1 = 0.0, s2 = 0.0;
        if (a.i >= 0) {
            if (a.j >= 0) {
                const double pj[3] = {a.n[0].x + beta * a.n[1].y, a.n[0].y + beta * a.n[2].x,
                                      a.n[1].x + beta * a.n[2].y};
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    s0 = s0 + a.v[0][q] * pj[q];
                    s1 = s1 + a.v[1][q] * pj[q];
                    s2 = s2 + a.v[2][q] * pj[q];
                }
            }
            for (int kk = l + kNodeLanes; 3 * kk < a.rl; kk += kNodeLanes) {  // past the first 16 neighbours
                const double* r = zp + 6 * (size_t)(c.colidx[a.base + 3 * kk] / 3);
                const double* v = c.vals + a.base + 3 * kk;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const double pj = r[q] + beta * r[3 + q];
                    s0 = s0 + v[q] * pj;
                    s1 = s1 + v[a.rl + q] * pj;
                    s2 = s2 + v[2 * a.rl + q] * pj;
                }
            }
        }
        s0 = sum16(s0);
        s1 = sum16(s1);
        s2 = sum16(s2);
        if (a.i >= 0 && l < 3) {
            const double acc = l == 0 ? s0 : (l == 1 ? s1 : s2);
            const double q = a.di != 0.0 ? acc : 0.0;
            const double pr = a.z + beta * a.p;
            zp_new[6 * (size_t)a.i + 3 + l] = pr;
            c.q[3 * a.i + l] = q;
            pq = pq + pr * q;
        }
    }
    const double s = block_sum(pq, sh2);
    if (threadIdx.x == 0)
        c.part[blockIdx.x] = s;
}

// Iteration k, second launch: alpha = (r_k.z_k) / (p.Ap) from the product's
// partials; x += alpha p_new, r -= alpha q, z = Dinv r (into p_new's copy);
// partials of r.z and r.r (grid-stride, each thread in ascending row order).
// Each thread loads its first kUpdateRows rows before the partials are summed,
// and further ones four at a time before it updates any of them.
constexpr int kUpdateRows = 4;
__global__ __launch_bounds__(kBlock) void k_cg_update(CgView c, int k, int cur)
{
    __shared__ double sh[2 * kWaves], sh2[kWaves];
    double* __restrict__ zp_new = c.zp + (cur ? 0 : 2 * (size_t)c.n);
    const int stride = gridDim.x * kBlock, i_first = blockIdx.x * kBlock + threadIdx.x;
    double xs[kUpdateRows], ps[kUpdateRows], rs[kUpdateRows], qs[kUpdateRows], ds[kUpdateRows];
    auto load_rows = [&](int i0) {
#pragma unroll
        for (int u = 0; u < kUpdateRows; ++u) {
            const int i = i0 + u * stride, ii = i < c.n ? i : 0;
            xs[u] = c.x[ii];
            ps[u] = zp_new[6 * (size_t)(ii / 3) + 3 + ii % 3];
            rs[u] = c.r[ii];
            qs[u] = c.q[ii];
            ds[u] = c.dinv[ii];
        }
    };
    const int done = c.s->done;
    const double rz_k = c.s->rzk[k & 1];
    const double share = share_of_partials(c.part, c.nparts_s);
    load_rows(i_first);
    if (done)
        return;
    const double alpha = rz_k / block_sum(share, sh2);
    double rz = 0.0, rr = 0.0;
    for (int i0 = i_first; i0 < c.n; i0 += kUpdateRows * stride) {
        if (i0 != i_first)
            load_rows(i0);
#pragma unroll
        for (int u = 0; u < kUpdateRows; ++u) {
            const int i = i0 + u * stride;
            if (i < c.n) {
                c.x[i] = xs[u] + alpha * ps[u];
                const double r = rs[u] - alpha * qs[u];
                c.r[i] = r;
                const double z = r * ds[u];
                zp_new[6 * (size_t)(i / 3) + i % 3] = z;
                rz = rz + r * z;
                rr = rr + r * r;
            }
        }
    }
    double s1, s2;
    block_sum2(rz, rr, sh, s1, s2);
    if (threadIdx.x == 0) {
        c.part[c.nparts_s + blockIdx.x] = s1;
        c.part[c.nparts_s + c.nparts_u + blockIdx.x] = s2;
    }
}

// A whole solve of a small system in one workgroup.  Rows t, t + kSmallBlock,
// ... of x, r and the preconditioner stay in thread t's registers, p and q in
// LDS, and so does the matrix: the blocks of the first kSmallHeld rounds of
// nodes (16 lanes per node as above) in registers, those of up to kSmallLds
// more in LDS.  Barriers take the place of launches: three per iteration.  The
// steps and the stopping rules are those of the launches above.
//
// Bound by its one compute unit: per iteration a chain of some 2 us (two
// divisions, three barriers, the sums over waves), and 0.3 us a round.  Whole
// solves, these launches / those above: 9 iterations of 24 rows 34 / 126 us, 27
// of 375 rows 83 / 237, 31 of 648 rows 120 / 293, 37 of 1,029 rows 190 / 349.
// Past the rounds that fit in registers and LDS the blocks would be read again
// in each iteration, at 1.6 us a round: 42 iterations of 1,536 rows took 442 us
// that way, 345 by the launches above, so there the rule draws its line; and
// where many nodes have many neighbours (cg_small_pays).
//
// Iterations k0 .. k1 - 1; a solve that is not done by then is kept in the
// workspace for the next launch, so that no launch runs for long.
constexpr int kSmallBlock = 512, kSmallWaves = kSmallBlock / 64, kSmallGroups = kSmallBlock / kNodeLanes;
constexpr int kSmallHeld = 8, kSmallLds = 3, kSmallNodes = (kSmallHeld + kSmallLds) * kSmallGroups;
static_assert(kSmallGroups == kCgSmallRound && kSmallHeld + kSmallLds == kCgSmallRounds, "cg_small_pays");
constexpr int kSmallRows = 3 * kSmallNodes, kSmallMine = (kSmallRows + kSmallBlock - 1) / kSmallBlock;

__device__ __forceinline__ double sum_waves(const double* sh)
{
    return ((sh[0] + sh[1]) + (sh[2] + sh[3])) + ((sh[4] + sh[5]) + (sh[6] + sh[7]));
}
static_assert(kSmallWaves == 8, "sum_waves");

// Sum over the wave, in lane 63 only.
__device__ __forceinline__ double sum_wave(double x)
{
    x = sum16(x);
    x = add_dpp_rows<0x142, 0xa>(x);     // row_bcast 15 into rows 1 and 3
    return add_dpp_rows<0x143, 0xc>(x);  // row_bcast 31 into rows 2 and 3
}

// Sums of three values over each aligned group of 16 lanes: x's in its lane 0,
// y's in lane 1, z's in lane 2 (after a step each, lanes keep one value only).
__device__ __forceinline__ double sum16_three(double x, double y, double z, int lane)
{
    x = add_dpp<0xB1>(x);  // quad_perm 1 0 3 2
    y = add_dpp<0xB1>(y);
    z = add_dpp<0xB1>(z);
    x = lane & 1 ? y : x;
    x = add_dpp<0x4E>(x);  // quad_perm 2 3 0 1
    z = add_dpp<0x4E>(z);
    x = lane & 2 ? z : x;
    x = add_dpp<0x124>(x);  // row_ror 4
    return add_dpp<0x128>(x);  // row_ror 8
}

__global__ __launch_bounds__(kSmallBlock) void k_cg_small(CgView c, const double* b, double* x_out, CgScalars* host,
                                                          double rtol, int k0, int k1, int max_iter)
{
    extern __shared__ double s_v[];  // per LDS round nine planes of kSmallBlock
    __shared__ double s_p[kSmallRows + 3], s_q[kSmallRows + 1];  // past the rows: 0, for lanes without a neighbour or node
    __shared__ double sh1[kSmallWaves], sh2[2 * kSmallWaves];
    const int t = threadIdx.x, wave = t >> 6, nn = c.n / 3, group = t / kNodeLanes, l = t & (kNodeLanes - 1);
    const int rounds = (nn + kSmallGroups - 1) / kSmallGroups;
    double x[kSmallMine], r[kSmallMine], di[kSmallMine];
    double rz = 0.0, rr = 0.0, rz_old = 0.0, bb = 0.0;
#pragma unroll
    for (int u = 0; u < kSmallMine; ++u) {
        const int i = t + u * kSmallBlock, ii = i < c.n ? i : 0, pos = c.dpos[ii];
        const double d = i < c.n && pos >= 0 ? c.vals[pos >= 0 ? pos : 0] : 0.0;
        di[u] = d != 0.0 ? 1.0 / d : 0.0;
        if (k0 == 0) {
            x[u] = 0.0;
            r[u] = d != 0.0 ? b[ii] : 0.0;
        } else {
            x[u] = c.x[ii];
            r[u] = i < c.n ? c.r[ii] : 0.0;
        }
        if (i < kSmallRows)
            s_p[i] = k0 == 0 ? 0.0 : c.zp[6 * (size_t)(ii / 3) + 3 + ii % 3];
        const double z = r[u] * di[u];
        rz = rz + r[u] * z;
        rr = rr + r[u] * r[u];
    }
    if (t < 3)
        s_p[kSmallRows + t] = 0.0;
    // of each round the place in s_p of this lane's neighbour, the block, and whether the node has more neighbours
    double v[kSmallHeld][9];
    int j[kSmallHeld + kSmallLds];
    unsigned more = 0u, live = 0u;
    auto load = [&](int w, double (&m)[9]) {
        const int i = w * kSmallGroups + group, ii = i < nn ? i : 0;
        const int base = c.rowptr[3 * ii], rl = c.rowptr[3 * ii + 1] - base, a = c.adj[kNodeLanes * (size_t)ii + l];
        const bool on = i < nn && a >= 0;
        j[w] = on ? 3 * a : kSmallRows;
        more |= i < nn && rl > 3 * kNodeLanes ? 1u << w : 0u;
        const int row = 3 * ii + (l < 3 ? l : 0), pos = c.dpos[row];
        live |= i < nn && l < 3 && pos >= 0 && c.vals[pos >= 0 ? pos : 0] != 0.0 ? 1u << w : 0u;
        const double* q = c.vals + (on ? base + 3 * l : 0);
#pragma unroll
        for (int k = 0; k < 9; ++k)
            m[k] = on ? q[(k / 3) * rl + k % 3] : 0.0;
    };
#pragma unroll
    for (int w = 0; w < kSmallHeld; ++w)
        load(w, v[w]);
#pragma unroll
    for (int w = 0; w < kSmallLds; ++w) {
        j[kSmallHeld + w] = kSmallRows;
        if (kSmallHeld + w < rounds) {
            double m[9];
            load(kSmallHeld + w, m);
#pragma unroll
            for (int k = 0; k < 9; ++k)
                s_v[(9 * w + k) * kSmallBlock + t] = m[k];
        }
    }
    if (k0 == 0) {
        const double wz = sum_wave(rz), wr = sum_wave(rr);
        if ((t & 63) == 63) {
            sh2[wave] = wz;
            sh2[kSmallWaves + wave] = wr;
        }
        __syncthreads();
        rz = sum_waves(sh2);
        bb = rr = sum_waves(sh2 + kSmallWaves);
    } else {
        rz = c.s->rzk[0];
        rz_old = c.s->rzk[1];
        rr = c.s->rr;
        bb = c.s->bnorm2;
    }
    const double tol2 = (rtol * rtol) * bb;
    bool done = k0 == 0 && bb == 0.0;
    int k = k0;
    while (!done) {
        if ((k > 0 && rr <= tol2) || k >= max_iter) {
            done = true;
            break;
        }
        if (k == k1)
            break;
        const double beta = k > 0 ? rz / rz_old : 0.0;
#pragma unroll
        for (int u = 0; u < kSmallMine; ++u) {
            const int i = t + u * kSmallBlock;
            if (i < kSmallRows)
                s_p[i] = (r[u] * di[u]) + beta * s_p[i];
        }
        __syncthreads();
        double pq = 0.0;
        auto node = [&](int w, const double (&m)[9]) {
            const double* pj = s_p + j[w];
            const int i = w * kSmallGroups + group, row = i < nn ? 3 * i + (l < 3 ? l : 0) : kSmallRows;
            const double pr = s_p[row];
            double s0 = 0.0, s1 = 0.0, s2 = 0.0;
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                s0 = s0 + m[q] * pj[q];
                s1 = s1 + m[3 + q] * pj[q];
                s2 = s2 + m[6 + q] * pj[q];
            }
            if (more >> w & 1u) {
                const int base = c.rowptr[3 * i], rl = c.rowptr[3 * i + 1] - base;
                for (int kk = l + kNodeLanes; 3 * kk < rl; kk += kNodeLanes) {  // past the first 16 neighbours
                    const double* e = s_p + c.colidx[base + 3 * kk];
                    const double* g = c.vals + base + 3 * kk;
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        s0 = s0 + g[q] * e[q];
                        s1 = s1 + g[rl + q] * e[q];
                        s2 = s2 + g[2 * rl + q] * e[q];
                    }
                }
            }
            const double acc = sum16_three(s0, s1, s2, t);
            const double q = live >> w & 1u ? acc : 0.0;
            if (l < 3)
                s_q[row] = q;
            pq = pq + pr * q;
        };
#pragma unroll
        for (int w = 0; w < kSmallHeld; ++w)
            if (w < rounds)
                node(w, v[w]);
#pragma unroll
        for (int w = 0; w < kSmallLds; ++w)
            if (kSmallHeld + w < rounds) {
                double m[9];
#pragma unroll
                for (int q = 0; q < 9; ++q)
                    m[q] = s_v[(9 * w + q) * kSmallBlock + t];
                node(kSmallHeld + w, m);
            }
        pq = sum_wave(pq);
        if ((t & 63) == 63)
            sh1[wave] = pq;
        __syncthreads();
        const double alpha = rz / sum_waves(sh1);
        double wz = 0.0, wr = 0.0;
#pragma unroll
        for (int u = 0; u < kSmallMine; ++u) {
            const int i = t + u * kSmallBlock;
            if (i < c.n) {
                x[u] = x[u] + alpha * s_p[i];
                r[u] = r[u] - alpha * s_q[i];
                wz = wz + r[u] * (r[u] * di[u]);
                wr = wr + r[u] * r[u];
            }
        }
        wz = sum_wave(wz);
        wr = sum_wave(wr);
        if ((t & 63) == 63) {
            sh2[wave] = wz;
            sh2[kSmallWaves + wave] = wr;
        }
        __syncthreads();
        rz_old = rz;
        rz = sum_waves(sh2);
        rr = sum_waves(sh2 + kSmallWaves);
        ++k;
    }
#pragma unroll
    for (int u = 0; u < kSmallMine; ++u) {
        const int i = t + u * kSmallBlock;
        if (i >= c.n)
            continue;
        if (done) {
            x_out[i] = x[u];
        } else {
            c.x[i] = x[u];
            c.r[i] = r[u];
            c.zp[6 * (size_t)(i / 3) + 3 + i % 3] = s_p[i];
        }
    }
    if (t == 0) {
        c.s->rzk[0] = rz;
        c.s->rzk[1] = rz_old;
        c.s->rr = rr;
        c.s->bnorm2 = bb;
        host->rr = rr;
        host->bnorm2 = bb;
        host->iters = k;
        host->done = done ? 1 : 0;
    }
}

__global__ __launch_bounds__(kBlock) void k_cg_output(CgView c, double* __restrict__ x)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < c.n)
        x[i] = c.x[i];
}

// Position of each row's diagonal entry in the CSR values (-1: unused node).
__global__ __launch_bounds__(kBlock) void k_diag_positions(DevView v, int32_t* __restrict__ dpos)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= 3 * v.n_nodes)
        return;
    const int i = r / 3, p = r - 3 * (r / 3);
    const int b = v.ndiag[i];
    dpos[r] = b >= 0 ? v.desc[b].up + p * v.desc[b].rl + p : -1;
}

// Each node's first kNodeLanes neighbours (itself included), -1 past the last.
__global__ __launch_bounds__(kBlock) void k_cg_adjacency(int n_nodes, const int32_t* __restrict__ rowptr,
                                                         const int32_t* __restrict__ colidx, int32_t* __restrict__ adj)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t i = t / kNodeLanes;
    if (i >= n_nodes)
        return;
    const int l = (int)(t % kNodeLanes), base = rowptr[3 * i], rl = rowptr[3 * i + 1] - base;
    adj[t] = 3 * l < rl ? colidx[base + 3 * l] / 3 : -1;
}

inline unsigned blocks(int64_t n, int per)
{
    return (unsigned)((n + per - 1) / per);
}

}  // namespace

hipError_t launch_diag_positions(const DevView& v, int32_t* dpos, hipStream_t s)
{
    if (v.n_nodes == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_diag_positions, dim3(blocks(3 * (int64_t)v.n_nodes, kBlock)), dim3(kBlock), 0, s, v, dpos);
    return hipGetLastError();
}

hipError_t launch_cg_adjacency(const DevView& v, const int32_t* rowptr, const int32_t* colidx, int32_t* adj,
                               hipStream_t s)
{
    if (v.n_nodes == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_cg_adjacency, dim3(blocks((int64_t)v.n_nodes * kNodeLanes, kBlock)), dim3(kBlock), 0, s,
                       v.n_nodes, rowptr, colidx, adj);
    return hipGetLastError();
}

// Matrix-vector product grid: one workgroup per 16 nodes, at most
// kSpmvGridMax; update grid: one per 256 rows, at most kUpdateGridMax.
int spmv_grid(int n)
{
    const int g = (int)blocks(n / 3, kBlock / kNodeLanes);
    return g < 1 ? 1 : (g > kSpmvGridMax ? kSpmvGridMax : g);
}

int update_grid(int n)
{
    const int g = (int)blocks(n, kBlock);
    return g < 1 ? 1 : (g > kUpdateGridMax ? kUpdateGridMax : g);
}

// Size of the partial-sum buffer: the start kernels' two halves, or the
// product's partials followed by the update's two halves.
int cg_partials(int n)
{
    const int a = 2 * (int)blocks(n, kBlock);
    const int b = spmv_grid(n) + 2 * update_grid(n);
    return a > b ? a : b;
}

hipError_t launch_cg_init(const CgView& c, const double* b, double rtol, hipStream_t s)
{
    hipLaunchKernelGGL(k_cg_init, dim3(blocks(c.n, kBlock)), dim3(kBlock), 0, s, c, b);
    hipLaunchKernelGGL(k_cg_init_finish, dim3(1), dim3(kBlock), 0, s, c, rtol);
    return hipGetLastError();
}

// Iterations first .. first+count-1 (the solve launches k = 0 .. max_iter;
// the product of k = max_iter only records the final residual).
hipError_t launch_cg_iterations(const CgView& c, int first, int count, int max_iter, hipStream_t s)
{
    for (int k = first; k < first + count; ++k) {
        const int cur = k & 1;  // which copy of p holds the previous direction
        hipLaunchKernelGGL(k_cg_spmv, dim3(c.nparts_s), dim3(kBlock), 0, s, c, k, cur, max_iter);
        hipLaunchKernelGGL(k_cg_update, dim3(c.nparts_u), dim3(kBlock), 0, s, c, k, cur);
    }
    return hipGetLastError();
}

// Iterations k0 .. k1 - 1 of a small solve, or its end; host: pinned.
hipError_t launch_cg_small(const CgView& c, const double* b, double* x, CgScalars* host, double rtol, int k0, int k1,
                           int max_iter, hipStream_t s)
{
    if (c.n > kSmallRows)
        return hipErrorInvalidValue;
    const int rounds = (c.n / 3 + kSmallGroups - 1) / kSmallGroups;
    const size_t lds = rounds > kSmallHeld ? sizeof(double) * 9 * kSmallBlock * (rounds - kSmallHeld) : 0;
    hipLaunchKernelGGL(k_cg_small, dim3(1), dim3(kSmallBlock), lds, s, c, b, x, host, rtol, k0, k1, max_iter);
    return hipGetLastError();
}

hipError_t launch_cg_output(const CgView& c, double* x, hipStream_t s)
{
    hipLaunchKernelGGL(k_cg_output, dim3(blocks(c.n, kBlock)), dim3(kBlock), 0, s, c, x);
    return hipGetLastError();
}

}  // namespace sta
