// gfx950 kernels for exact assembly of A_t = M_t + dt^2 K_t (paper Sec. 3.4
// eq. (8), implicit-Euler matrix of Sec. 6.2 eq. (9)).
//
// Data flow.  Each candidate tet has one 128-byte geometry record (basis
// gradients, scaled moduli, lumped mass).  A matrix entry is the sum, in
// ascending tet id from +0.0, of the entries of its active tets' element
// matrices, each formed from the tet's record where it is needed: nothing of
// the 78 values per tet is stored.  The full rebuild recomputes every record
// and sums every row; the streaming update re-sums the blocks that the edited
// tets cover.  Both form and add the same terms in the same order, so they
// agree bit for bit with each other and with a rebuild that skips inactive
// tets (an accumulator that starts at +0.0 never becomes -0.0, so adding
// +0.0 changes nothing).
//
// Floating point: contraction is off for this file and the element formula
// is evaluated in a fixed order (see include/stafem.h); only IEEE + - * / and
// |.| are used.
#include <hip/hip_runtime.h>

#include "edit_table.h"
#include "sta_internal.h"

#pragma clang fp contract(off)

namespace sta {

namespace {

constexpr int kBlock = 256;
constexpr int kEditLanes = 16;     // phase 1: one lane per block slot (10 used), power of two
// Claimed blocks are compacted per edit-phase wave (64 / kEditLanes = 4
// edits): at most 16 diagonal and 24 off-diagonal claims.
constexpr int kRegionDiag = 16, kRegionOff = 24, kRegion = kRegionDiag + kRegionOff;
constexpr int kRegionsPerBlock = kBlock / 64;

typedef double dvec2 __attribute__((ext_vector_type(2)));

struct Geo {
    double g[4][3];
    double lamV, muV, ml, det;
};

__device__ __forceinline__ void cross3(const double* a, const double* b, double* c)
{
    c[0] = (a[1] * b[2]) - (a[2] * b[1]);
    c[1] = (a[2] * b[0]) - (a[0] * b[2]);
    c[2] = (a[0] * b[1]) - (a[1] * b[0]);
}

// Basis gradients, scaled moduli and lumped mass of a tet from its vertex
// coordinates X and Young's modulus E, in the fixed order.
__device__ __forceinline__ void geometry_from(const DevView& v, const double (&X)[4][3], double E, Geo& G)
{
    double d[4][3];
#pragma unroll
    for (int k = 1; k <= 3; ++k)
#pragma unroll
        for (int i = 0; i < 3; ++i)
            d[k][i] = X[k][i] - X[0][i];
    double c[4][3];
    cross3(d[2], d[3], c[1]);
    cross3(d[3], d[1], c[2]);
    cross3(d[1], d[2], c[3]);
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
    const double V = fabs(det) / 6.0;
    const double lam = E * v.mat.clam;
    const double mu = E * v.mat.cmu;
    G.lamV = (lam * V) * v.mat.cdt;
    G.muV = (mu * V) * v.mat.cdt;
    G.ml = (v.mat.rho * V) * 0.25;
    G.det = det;
}

__device__ __forceinline__ void load_vertices(const DevView& v, int4 t, double (&X)[4][3])
{
    const int id[4] = {t.x, t.y, t.z, t.w};
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        X[a][0] = v.xs[id[a]];
        X[a][1] = v.ys[id[a]];
        X[a][2] = v.zs[id[a]];
    }
}

__device__ __forceinline__ void element_geometry(const DevView& v, int e, int4 t, Geo& G)
{
    double X[4][3];
    load_vertices(v, t, X);
    geometry_from(v, X, v.E[e], G);
}

__device__ __forceinline__ double dot3(const double* a, const double* b)
{
    return ((a[0] * b[0]) + (a[1] * b[1])) + (a[2] * b[2]);
}

// Entry (i, j) of the 3x3 block of row vertex a (gradient ga) and column
// vertex b (gradient gb); s = ga . gb; diag: a == b.
__device__ __forceinline__ double entry(const double* ga, const double* gb, double s, const Geo& G, int i, int j,
                                        bool diag)
{
    double v = (G.lamV * (ga[i] * gb[j])) + (G.muV * (ga[j] * gb[i]));
    if (i == j)
        v = v + (G.muV * s);
    if (diag && i == j)
        v = v + G.ml;
    return v;
}

__device__ __constant__ int kDiagP[6] = {0, 0, 0, 1, 1, 2};
__device__ __constant__ int kDiagQ[6] = {0, 1, 2, 1, 2, 2};

__device__ __forceinline__ BlockDesc load_desc(const BlockDesc* p)
{
    const int4* q = reinterpret_cast<const int4*>(p);
    const int4 a = q[0], b = q[1];
    BlockDesc d;
    d.k0 = a.x;
    d.k1 = a.y;
    d.up = a.z;
    d.rl = a.w;
    d.lo = b.x;
    d.rlj = b.y;
    d.kind = b.z;
    d.block = b.w;
    return d;
}

__device__ __forceinline__ void store_desc(BlockDesc* p, const BlockDesc& d)
{
    int4* q = reinterpret_cast<int4*>(p);
    q[0] = make_int4(d.k0, d.k1, d.up, d.rl);
    q[1] = make_int4(d.lo, d.rlj, d.kind, d.block);
}

__device__ __forceinline__ BlockDesc empty_desc()
{
    return BlockDesc{0, 0, 0, 0, 0, 0, -1, -1};
}

// ---------------------------------------------------------------------------
// Full rebuild
// ---------------------------------------------------------------------------

// Every candidate's geometry record.  One lane per tet; a wave stages its 64
// records in LDS (17 doubles apart, so that neither side conflicts) and stores
// them as whole lines: 12.4 us for 384,000 tets, 60 MB at 4.9 TB/s, where
// writing each tet's 78 values into its blocks' segments took 58 to 69.
__global__ __launch_bounds__(kBlock) void k_geometry(DevView v)
{
    constexpr int kStride = kGeoDoubles + 1;
    __shared__ double s_stage[kBlock / 64][64 * kStride];
    const int wg = xcd_remap(blockIdx.x, gridDim.x);
    const int base = wg * kBlock + (threadIdx.x & ~63);  // the wave's first tet
    if (base >= v.n_tets)
        return;
    const int lane = threadIdx.x & 63;
    const int nw = v.n_tets - base < 64 ? v.n_tets - base : 64;  // tets of this wave
    const int e = base + (lane < nw ? lane : nw - 1);
    Geo G;
    element_geometry(v, e, v.T[e], G);
    const bool degenerate = G.det == 0.0;
    if (degenerate && v.mask[e])
        atomicOr(&v.ctl->err, ERR_DEGENERATE);
    double* buf = s_stage[threadIdx.x >> 6];
#pragma unroll
    for (int k = 0; k < 12; ++k)
        buf[kStride * lane + k] = G.g[k / 3][k % 3];
    buf[kStride * lane + 12] = G.lamV;
    buf[kStride * lane + 13] = G.muV;
    buf[kStride * lane + 14] = G.ml;
    buf[kStride * lane + 15] = __longlong_as_double(degenerate ? 1ll : 0ll);  // degenerate, pad
    // LDS accesses of one wave complete in issue order; the wavefront-scope
    // fence only keeps the compiler from moving them across the exchange
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    dvec2* dst = reinterpret_cast<dvec2*>(v.geo + (size_t)kGeoDoubles * base);
#pragma unroll
    for (int j = 0; j < kGeoDoubles / 2; ++j) {
        const int p = lane + 64 * j, m = p >> 3, k = p & 7;
        if (m < nw)
            dst[p] = dvec2{buf[kStride * m + 2 * k], buf[kStride * m + 2 * k + 1]};
    }
}

// The CSR rows of one tile of nodes.  The tile's (node, tet) pairs' records
// are staged in LDS by eight lanes each, so that every record is read as one
// whole line, with zeros for inactive tets; then one lane per pair forms its
// diagonal block's 6 values, one lane per off-diagonal row block sums its 9
// values over the block's terms, and six lanes per node sum the diagonal
// block's, all in ascending tet id.  Both blocks (i, j) and (j, i) are formed,
// each by its row's tile: entry (p, q) of one is bitwise entry (q, p) of the
// other, since a product's operands commute, and twice the arithmetic costs
// less than scattering the mirror in 24-byte pieces.  The rows leave through
// LDS as one contiguous range.
//
// Loads past a tile's end take its last element (in range), so that no branch
// or wait separates the loads of a round (with one: 116 us instead of 50 on the
// 384,000-tet cube; summing stored contributions from HBM took 88 to 91).  The
// phases of one workgroup wait for each other, so it takes several on a compute
// unit to keep it busy: with 31,920 bytes of LDS five fit, and it takes 46 us
// (of which 24 are arithmetic); with 34,032, four, 50.
constexpr int kRowThreads = 192;
constexpr int kRowStride = 13;              // doubles per staged record (odd: neighbouring records differ in bank)
constexpr int kDiagStride = kTilePairs + 1;  // diagonal values: value vi of pair p at vi * kDiagStride + p
constexpr int kRowOut = 6 * kDiagStride > 9 * kTileBlocks ? 6 * kDiagStride : 9 * kTileBlocks;
static_assert(kRowThreads == kTileBlocks + 64 && kTileNodes * 6 <= 64, "one wave of diagonal lanes");
static_assert(kTilePairs == kRowThreads, "one lane per pair");
template <bool NT>
__global__ __launch_bounds__(kRowThreads) void k_rows(DevView v)
{
    __shared__ double s_geo[kTilePairs * kRowStride];  // g, lamV
    __shared__ double s_mu[kTilePairs];                // muV
    __shared__ double s_out[kRowOut];  // the diagonal values, then the rows
    __shared__ uint16_t s_term[kTileTerms];
    const RowTile tile = v.tiles[xcd_remap(blockIdx.x, gridDim.x)];
    const int tid = threadIdx.x;
    constexpr int kRounds = kTilePairs * 8 / kRowThreads;
    constexpr int kPerRound = kRowThreads / 8;
    constexpr int kTermRounds = kTileTerms / kRowThreads;
    const int j = tid & 7;
    uint32_t u[kRounds];
#pragma unroll
    for (int k = 0; k < kRounds; ++k)
        u[k] = v.di[tile.pair0 + min(k * kPerRound + (tid >> 3), tile.pairs - 1)];
    uint16_t term[kTermRounds];
#pragma unroll
    for (int k = 0; k < kTermRounds; ++k)
        term[k] = v.terms[tile.term0 + min(k * kRowThreads + tid, tile.terms - 1)];
    const uint32_t own = v.di[tile.pair0 + min(tid, tile.pairs - 1)];  // this lane's pair
    // row block or row node of this lane
    const int dl = tid - kTileBlocks;  // diagonal lane: node dl / 6, value dl % 6
    const bool has_blk = tid < tile.blks, has_node = dl >= 0 && dl < 6 * tile.nodes;
    const uint2 rb = dl < 0 ? v.rowblk[tile.blk0 + min(tid, tile.blks - 1)]
                            : v.rownode[tile.node0 + min(dl / 6, tile.nodes - 1)];
    dvec2 q[kRounds];
    uint8_t on[kRounds];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
        q[k] = reinterpret_cast<const dvec2*>(v.geo + (size_t)kGeoDoubles * (u[k] >> 2))[j];
        on[k] = v.mask[u[k] >> 2];
    }
#pragma unroll
    for (int k = 0; k < kTermRounds; ++k)
        s_term[k * kRowThreads + tid] = term[k];
#pragma unroll
    for (int k = 0; k < kRounds; ++k) {
        const int p = k * kPerRound + (tid >> 3);
        const double x = on[k] ? q[k].x : 0.0, y = on[k] ? q[k].y : 0.0;
        if (j < 7) {  // j = 6: lamV, muV
            s_geo[p * kRowStride + 2 * j] = x;
            *(j < 6 ? s_geo + p * kRowStride + 2 * j + 1 : s_mu + p) = y;
        } else {
            s_out[5 * kDiagStride + p] = x;  // ml, until its lane puts a diagonal value there
        }
    }
    __syncthreads();
    {
        const double* r = s_geo + tid * kRowStride;
        const double* pa = r + 3 * (own & 3u);
        Geo G;
        G.lamV = r[12];
        G.muV = s_mu[tid];
        G.ml = s_out[5 * kDiagStride + tid];
        const double g[3] = {pa[0], pa[1], pa[2]};
        const double s = dot3(g, g);
#pragma unroll
        for (int vi = 0; vi < 6; ++vi) {
            constexpr int P[6] = {0, 0, 0, 1, 1, 2}, Q[6] = {0, 1, 2, 1, 2, 2};
            s_out[vi * kDiagStride + tid] = entry(g, g, s, G, P[vi], Q[vi], true);
        }
    }
    __syncthreads();
    const int rl = (int)(rb.y >> 16), at = (int)(rb.y & 0xffffu);
    const int first = (int)(rb.x & 0xffffu), end = first + (int)(rb.x >> 16);
    double acc[3][3] = {};
    if (dl < 0) {
        for (int k = first; k < end; ++k) {
            const uint32_t t = s_term[k];
            const double* r = s_geo + (t >> 4) * kRowStride;
            const double* pa = r + 3 * ((t >> 2) & 3u);
            const double* pb = r + 3 * (t & 3u);
            Geo G;
            G.lamV = r[12];
            G.muV = s_mu[t >> 4];
            const double ga[3] = {pa[0], pa[1], pa[2]}, gb[3] = {pb[0], pb[1], pb[2]};
            const double s = dot3(ga, gb);
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int c = 0; c < 3; ++c)
                    acc[i][c] = acc[i][c] + entry(ga, gb, s, G, i, c, false);
        }
    } else {
        const double* x = s_out + (dl % 6) * kDiagStride;
        for (int k = first; k < end; k += 8) {
            double t[8];
#pragma unroll
            for (int w = 0; w < 8; ++w)
                t[w] = x[min(k + w, end - 1)];
#pragma unroll
            for (int w = 0; w < 8; ++w)
                acc[0][0] = acc[0][0] + (k + w < end ? t[w] : 0.0);
        }
    }
    __syncthreads();
    if (has_blk && end > first) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                s_out[at + i * rl + c] = acc[i][c];
    } else if (has_node) {
        const int i = kDiagP[dl % 6], c = kDiagQ[dl % 6];
        s_out[at + i * rl + c] = acc[0][0];
        if (i != c)
            s_out[at + c * rl + i] = acc[0][0];
    }
    __syncthreads();
    for (int k = tid; k < 9 * tile.blks; k += kRowThreads) {
        if (NT)
            __builtin_nontemporal_store(s_out[k], v.values + tile.val0 + k);
        else
            v.values[tile.val0 + k] = s_out[k];
    }
}

// ---------------------------------------------------------------------------
// Sums of a few blocks by one wave (streaming, and the rows of nodes too large
// for a tile)
// ---------------------------------------------------------------------------

// A wave sums up to two diagonal blocks or up to six off-diagonal ones: the
// ten blocks of a tet take three waves, two for its diagonal blocks (2 x 24
// incidences each on the structured cube) and one for the others (32).  One
// wave for all ten took 128 terms, two per lane, and two values per lane in
// turn, and the longer instruction stream was the longest link of a frame's
// chain.
template <bool kDiag>
struct Unit {
    static constexpr int kBlocks = kDiag ? 2 : 6;
    static constexpr int kValues = kDiag ? 6 : 9;  // entries formed per term
    static constexpr int kStride = kDiag ? 7 : 9;  // doubles per term in LDS (odd: no bank conflicts)
};
constexpr int kUnits = 3;       // waves for a tet's ten blocks
constexpr int kUnitTerms = 64;  // terms formed at a time, one per lane
// LDS of a wave of either kind, with room to read eight terms past the last,
// and of the three waves of a tet
constexpr int kUnitDoubles = (kUnitTerms + 8) * Unit<false>::kStride;
constexpr int kDiagUnitDoubles = (kUnitTerms + 8) * Unit<true>::kStride;
constexpr int kTetDoubles = 2 * kDiagUnitDoubles + kUnitDoubles;

// The state of a tet is its mask byte unless the frame's own edits say
// otherwise: listed gives 0 or 1 for an edited tet, kUnlisted for any other.
struct MaskState {
    __device__ __forceinline__ uint32_t listed(uint32_t) const { return kUnlisted; }
};

// The wave's blocks laid end to end: the terms before each block's, and for
// this lane's block its terms, their start and the shift to incidences.
template <bool kDiag>
struct UnitTerms {
    int cnt, own, shift;
    int pre[Unit<kDiag>::kBlocks + 1];
    __device__ __forceinline__ int total() const { return pre[Unit<kDiag>::kBlocks]; }
};

template <bool kDiag>
__device__ __forceinline__ UnitTerms<kDiag> unit_terms(const BlockDesc& d)
{
    const int lane = threadIdx.x & 63;
    UnitTerms<kDiag> b;
    b.cnt = lane < Unit<kDiag>::kBlocks && d.kind >= 0 ? d.k1 - d.k0 : 0;
    b.own = 0;
    b.pre[0] = 0;
#pragma unroll
    for (int r = 0; r < Unit<kDiag>::kBlocks; ++r) {
        b.own = lane == r ? b.pre[r] : b.own;
        b.pre[r + 1] = b.pre[r] + __builtin_amdgcn_readlane(b.cnt, r);
    }
    b.shift = d.k0 - b.own;
    return b;
}

// Incidence of term base + lane (of some incidence where there is no such term).
template <bool kDiag>
__device__ __forceinline__ uint32_t load_incidence(const DevView& v, const UnitTerms<kDiag>& b, int base)
{
    const int t = base + (int)(threadIdx.x & 63);
    int r = 0;
#pragma unroll
    for (int w = 1; w < Unit<kDiag>::kBlocks; ++w)
        r += t >= b.pre[w] ? 1 : 0;
    const int k = t + __shfl(b.shift, r, 64);
    return (kDiag ? v.di : v.oi)[t < b.total() ? k : 0];
}

// What one lane needs to form one term's entries.
struct Term {
    uint32_t tet;
    double ga[3], gb[3], lamV, muV, ml;
    uint8_t active;
};

template <bool kDiag>
__device__ __forceinline__ void load_term(const DevView& v, uint32_t u, Term& t)
{
    t.tet = kDiag ? u >> 2 : u >> 4;
    const double* r = v.geo + (size_t)kGeoDoubles * t.tet;
    const double* pa = r + 3 * (kDiag ? u & 3u : (u >> 2) & 3u);
#pragma unroll
    for (int i = 0; i < 3; ++i)
        t.ga[i] = pa[i];
    t.lamV = r[12];
    t.muV = r[13];
    if (kDiag) {
        t.ml = r[14];
    } else {
        const double* pb = r + 3 * (u & 3u);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            t.gb[i] = pb[i];
    }
    t.active = v.mask[t.tet];
}

// Sum the wave's blocks and write their CSR values; u: the incidences of the
// first kUnitTerms terms.  Each lane forms the entries of one term at a time
// from its tet's record into val (LDS, kUnitDoubles per wave); then one lane
// per block value adds its block's entries in ascending order.  Any segment
// length works: a round's incidences are loaded a round ahead, and with kAhead its
// records too (rows of nodes of 20,000 and 5,000 tets 470 -> 397 and 123 -> 109 us;
// in the frames the 20 registers cost a third of the waves).
template <bool kDiag, bool kAhead, class State>
__device__ __forceinline__ void sum_unit(const DevView& v, const BlockDesc& d, const UnitTerms<kDiag>& b, uint32_t u,
                                         double* val, const State& state)
{
    using U = Unit<kDiag>;
    const int lane = threadIdx.x & 63;
    const int total = b.total();
    // the value of this lane: block r0, entry e0 of it, term range
    const bool has = lane < U::kBlocks * U::kValues;
    const int r0 = has ? lane / U::kValues : 0, e0 = has ? lane % U::kValues : 0;
    const int lo = __shfl(b.own, r0, 64), hi = has ? lo + __shfl(b.cnt, r0, 64) : lo;
    double acc = 0.0;
    Term t, next;
    if (kAhead) {
        load_term<kDiag>(v, u, next);
        if (kUnitTerms < total)
            u = load_incidence<kDiag>(v, b, kUnitTerms);
    }
    for (int base = 0; base < total; base += kUnitTerms) {
        constexpr int kLead = (kAhead ? 2 : 1) * kUnitTerms;
        if (kAhead)
            t = next;
        if (!kAhead || base + kUnitTerms < total)
            load_term<kDiag>(v, u, kAhead ? next : t);
        if (base + kLead < total)
            u = load_incidence<kDiag>(v, b, base + kLead);
        Geo G;
        G.lamV = t.lamV;
        G.muV = t.muV;
        if (kDiag)
            G.ml = t.ml;
        const double* ga = t.ga;
        const double* gb = kDiag ? t.ga : t.gb;
        const uint32_t listed = state.listed(t.tet);  // while the record is in flight
        const bool on = listed == kUnlisted ? t.active != 0 : listed != 0u;
        // LDS accesses of one wave complete in issue order; the fences only
        // keep the compiler from moving them
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const double s = dot3(ga, gb);
        double* dst = val + lane * U::kStride;
#pragma unroll
        for (int k = 0; k < U::kValues; ++k) {
            constexpr int P[6] = {0, 0, 0, 1, 1, 2}, Q[6] = {0, 1, 2, 1, 2, 2};
            const double x = entry(ga, gb, s, G, kDiag ? P[k % 6] : k / 3, kDiag ? Q[k % 6] : k % 3, kDiag);
            dst[k] = on ? x : 0.0;
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // eight terms at a time; those past the block's end (the space has
        // room for them) are replaced by +0.0
        const int z = min(hi - base, kUnitTerms);
        for (int k = max(lo - base, 0); k < z; k += 8) {
            const double* p = val + k * U::kStride + e0;
            double x[8];
#pragma unroll
            for (int w = 0; w < 8; ++w)
                x[w] = p[w * U::kStride];
#pragma unroll
            for (int w = 0; w < 8; ++w)
                acc = acc + (k + w < z ? x[w] : 0.0);
        }
    }
    const int up = __shfl(d.up, r0, 64), rl = __shfl(d.rl, r0, 64);
    const int dn = __shfl(d.lo, r0, 64), rj = __shfl(d.rlj, r0, 64);
    if (hi > lo) {
        // entries 00 01 02 11 12 22 of a diagonal block, row by row of another
        const int pc = kDiag ? (int)(0xA65210u >> (4 * e0)) & 15 : 0;
        const int p = kDiag ? pc >> 2 : e0 / 3, c = kDiag ? pc & 3 : e0 % 3;
        v.values[up + p * rl + c] = acc;
        if (!kDiag || p != c)
            v.values[dn + c * rj + p] = acc;
    }
}

// The same from the start, with the states in the mask.
template <bool kDiag, bool kAhead>
__device__ __forceinline__ void sum_unit_masked(const DevView& v, const BlockDesc& d, double* val)
{
    const UnitTerms<kDiag> b = unit_terms<kDiag>(d);
    if (b.total() > 0)
        sum_unit<kDiag, kAhead>(v, d, b, load_incidence<kDiag>(v, b, 0), val, MaskState{});
}

// Rows of nodes too large for a tile: waves of two of their diagonal blocks,
// then waves of six of their off-diagonal ones.  An off-diagonal block is
// written in both its rows; the other node's tile, if it has one, writes the
// same bits.
__global__ __launch_bounds__(kBlock) void k_rows_big(DevView v)
{
    __shared__ double s_val[kBlock / 64][kUnitDoubles];
    const int lane = threadIdx.x & 63;
    const int w = blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wd = (v.n_bigd + Unit<true>::kBlocks - 1) / Unit<true>::kBlocks;
    BlockDesc d = empty_desc();
    if (w < wd) {
        const int k = w * Unit<true>::kBlocks + lane;
        if (lane < Unit<true>::kBlocks && k < v.n_bigd)
            d = load_desc(v.desc + v.bigd[k]);
        sum_unit_masked<true, true>(v, d, s_val[threadIdx.x >> 6]);
    } else {
        const int k = (w - wd) * Unit<false>::kBlocks + lane;
        if (lane < Unit<false>::kBlocks && k < v.n_bigo)
            d = load_desc(v.desc + v.bigo[k]);
        sum_unit_masked<false, true>(v, d, s_val[threadIdx.x >> 6]);
    }
}

// ---------------------------------------------------------------------------
// Streaming update
// ---------------------------------------------------------------------------

__device__ __forceinline__ int tet_vertex(int4 t, int a)
{
    return a == 0 ? t.x : (a == 1 ? t.y : (a == 2 ? t.z : t.w));
}

// Local vertices (A, B) of block slot r: r < 4 diagonal (r, r); 4..9 the
// pairs 01 02 03 12 13 23.  Two bits per slot, packed.
constexpr uint32_t kSlotA = 0u | 1u << 2 | 2u << 4 | 3u << 6 | 0u << 8 | 0u << 10 | 0u << 12 | 1u << 14 | 1u << 16 |
                            2u << 18;
constexpr uint32_t kSlotB = 0u | 1u << 2 | 2u << 4 | 3u << 6 | 1u << 8 | 2u << 10 | 3u << 12 | 2u << 14 | 3u << 16 |
                            3u << 18;

__device__ int32_t kNoTet = -1;
__device__ uint8_t kNoState = 0;

__device__ __forceinline__ bool is_degenerate(const DevView& v, int id)
{
    return reinterpret_cast<const TetGeo*>(v.geo)[id].degenerate != 0;
}

// Edit count of this frame: *n_dev if given and within [0, n_host], else n_host.
__device__ __forceinline__ int frame_count(int32_t n_host, const int32_t* n_dev, bool& bad)
{
    bad = false;
    if (!n_dev)
        return n_host;
    const int n = *n_dev;
    if (n < 0 || n > n_host) {
        bad = true;
        return 0;
    }
    return n;
}

// Phase 1 for lane r of edit i = (tet id, requested state st); 16 lanes per
// edit, lane r < 10 owns block slot r.  Validate the edit; lane 0 takes the
// tet's stamp (a second edit of the same tet in this frame finds it taken:
// duplicate).  If the state changes, each slot lane claims its block (first
// claimant wins; the claim's kind and block descriptor are returned in ckind
// (-1: no claim) and cbd for the wave's compaction) and the owner flips the
// mask bit.  Returns the lane's error bits.  All 16 lanes of the edit must
// call it together.
__device__ __forceinline__ int edit_lane(const DevView& v, int id, unsigned st, int i, int r, int& ckind,
                                         BlockDesc& cbd)
{
    if (id < 0 || id >= v.n_tets || st > 1u) {
        if (r == 0) {
            v.undo[i] = 0xFF;
            return ERR_RANGE;
        }
        return 0;
    }
    const bool slot = r < 10;
    // round trip 1: this lane's block descriptor, the tet's mask bit, its
    // stamp and whether an activation would assemble a degenerate tet
    BlockDesc bd = empty_desc();
    if (slot)
        bd = load_desc(v.trec[id].desc + r);
    const uint8_t prev = v.mask[id];
    const bool degenerate = is_degenerate(v, id);
    unsigned taken = 0u;
    if (r == 0)
        taken = atomicExch(&v.estamp[id], 1u);
    // round trip 2: the block claim
    const bool change = prev != st;
    unsigned claimed = 1u;
    if (slot && change)
        claimed = atomicExch(&v.bstamp[bd.block], 1u);
    const int owner = __shfl(taken, (threadIdx.x & 63) & ~(kEditLanes - 1), 64) == 0u;
    int bits = 0;
    if (!owner) {
        if (r == 0)
            bits = ERR_DUP;
    } else if (change && r == 0) {
        v.mask[id] = (uint8_t)st;
        if (st && degenerate)
            atomicOr(&v.ctl->err, ERR_DEGENERATE);
    }
    if (slot && claimed == 0u) {
        ckind = r < 4 ? 0 : 1;
        cbd = bd;
    }
    if (r == 0)
        v.undo[i] = (owner && change) ? prev : (uint8_t)0xFF;
    return bits;
}

// Phase 2 waves: kDW per claim region for its diagonal records (two at a
// time) and kOW for its off-diagonal ones (six at a time), each going on while
// records are left; then one lane per edit (stamp release, rollback).  A region
// fills from its start and mostly holds 4 to 6 diagonal and 10 to 15
// off-diagonal claims, so four and two waves take one pass or two (of 4 + 2, 4 +
// 4, 5 + 3, 8 + 2 and 8 + 4 waves the first is the fastest for refinement frames of
// 5,778 and 7,344 edits, 12.5 and 14.7 us against 13.2 to 14.9 and 15.7 to 18.0);
// a persistent grid, which cannot have them all resident, takes fewer.
template <int kDW, int kOW>
struct RegionWaves {
    static constexpr int kWaves = kDW + kOW;
    bool diag;
    int blocks, stride, first, k, count;  // k: the record of lane 0 in this pass

    // The claim record of this lane in wave `part` of region w, if there is one.
    __device__ __forceinline__ BlockDesc start(const DevView& v, int w, int part)
    {
        diag = part < kDW;
        blocks = diag ? Unit<true>::kBlocks : Unit<false>::kBlocks;
        stride = blocks * (diag ? kDW : kOW);
        first = w * kRegion + (diag ? 0 : kRegionDiag);
        k = (diag ? part : part - kDW) * blocks;
        count = v.rcount[2 * w + (diag ? 0 : 1)];
        return load(v);
    }
    __device__ __forceinline__ BlockDesc load(const DevView& v) const
    {
        const int lane = threadIdx.x & 63;
        BlockDesc d = empty_desc();
        if (lane < blocks) {
            d = load_desc(v.rec + (size_t)first + k + lane);  // in range, valid or not
            if (k + lane >= count)
                d = empty_desc();
        }
        return d;
    }
    // Re-sum the wave's blocks, first record d, unless the frame has an error,
    // and release their claim stamps either way.
    __device__ __forceinline__ void run(const DevView& v, BlockDesc d, int fe, double* val)
    {
        static_assert(kRegionDiag >= 2 * kDW && kRegionOff >= 6 * kOW, "a wave's first records are in its region");
        while (k < count) {
            if (!fe) {
                if (diag)
                    sum_unit_masked<true, false>(v, d, val);
                else
                    sum_unit_masked<false, false>(v, d, val);
            }
            if ((int)(threadIdx.x & 63) < blocks && d.kind >= 0)
                v.bstamp[d.block] = 0u;
            k += stride;
            if (k < count)
                d = load(v);
        }
    }
};
using TouchedWaves = RegionWaves<4, 2>;  // two-launch frame
using FusedWaves = RegionWaves<2, 2>;    // persistent frame

// Phase 2, edit lane for edit i (tet id, undo byte u): release the tet stamp
// and, if the frame has an error, undo the edit's mask flip.
__device__ __forceinline__ void touched_edit(const DevView& v, int id, uint8_t u, int fe)
{
    if (id < 0 || id >= v.n_tets)
        return;
    v.estamp[id] = 0u;
    if (fe && u != 0xFF)
        v.mask[id] = u;
}

// Workgroup-wide OR of error bits.
__device__ __forceinline__ int block_or(int bits, int* s_bits)
{
    if (threadIdx.x == 0)
        *s_bits = 0;
    __syncthreads();
    if (bits)
        atomicOr(s_bits, bits);
    __syncthreads();
    return *s_bits;
}

// OR of the first g error bytes of the edit phase.
__device__ __forceinline__ int frame_error(const DevView& v, int g, int* s_bits)
{
    int bits = 0;
    for (int w = threadIdx.x; w < g; w += kBlock)
        bits |= v.wg_err[w];
    return block_or(bits, s_bits);
}

__device__ __forceinline__ void publish_frame(const DevView& v, int fe, int n, int regions)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        v.ctl->frame_err = fe;
        v.ctl->last_n = n;
        v.ctl->last_regions = regions;
        if (fe)
            atomicOr(&v.ctl->err, fe);
    }
}

// Compact the wave's claims into claim region `region`: diagonal claims
// first, then off-diagonal ones, each in lane order; lane 0 records the two
// counts.  Called by every lane of the wave (ckind = -1: no claim).
__device__ __forceinline__ void compact_claims(const DevView& v, int64_t region, int ckind, const BlockDesc& cbd)
{
    const uint64_t dm = __ballot(ckind == 0);
    const uint64_t om = __ballot(ckind == 1);
    const uint64_t below = __lanemask_lt();
    BlockDesc* base = v.rec + region * kRegion;
    if (ckind == 0)
        store_desc(base + __popcll(dm & below), cbd);
    else if (ckind == 1)
        store_desc(base + kRegionDiag + __popcll(om & below), cbd);
    if ((threadIdx.x & 63) == 0) {
        v.rcount[2 * region] = __popcll(dm);
        v.rcount[2 * region + 1] = __popcll(om);
    }
}

// Phase 1 as its own kernel: one 16-lane group per edit.  Each workgroup
// writes its error bits to its own byte, so nothing needs resetting.
__global__ __launch_bounds__(kBlock) void k_edits(DevView v, const int32_t* __restrict__ ids,
                                                  const uint8_t* __restrict__ states, int32_t n_host,
                                                  const int32_t* __restrict__ n_dev)
{
    __shared__ int s_bits;
    const int gt = blockIdx.x * kBlock + threadIdx.x;
    const int i = gt / kEditLanes;
    // the edit itself is read while the device-side count is still in flight
    int id = -1;
    unsigned st = 0;
    if (i < n_host) {
        id = ids[i];
        st = states[i];
    }
    bool bad_n;
    const int n = frame_count(n_host, n_dev, bad_n);
    int bits = (bad_n && gt == 0) ? ERR_RANGE : 0;
    int ckind = -1;
    BlockDesc cbd;
    if (i < n)
        bits |= edit_lane(v, id, st, i, gt - i * kEditLanes, ckind, cbd);
    compact_claims(v, gt / 64, ckind, cbd);
    bits = block_or(bits, &s_bits);
    if (threadIdx.x == 0)
        v.wg_err[blockIdx.x] = (uint8_t)bits;
}

// Phase 2 as its own kernel.
__global__ __launch_bounds__(kBlock) void k_touched(DevView v, const int32_t* __restrict__ ids, int32_t n_host,
                                                    const int32_t* __restrict__ n_dev)
{
    __shared__ double s_val[kBlock / 64][kUnitDoubles];
    __shared__ int s_bits;
    // the edit phase ran `edit_wgs` workgroups of kRegionsPerBlock waves, each wave one claim region
    const int edit_wgs = n_host > 0 ? (n_host * kEditLanes + kBlock - 1) / kBlock : 1;
    const int regions = edit_wgs * kRegionsPerBlock;
    const int64_t wave = (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const bool rec_wave = wave < (int64_t)regions * TouchedWaves::kWaves;
    TouchedWaves tw;
    // claim record and count, or the edit's id and undo byte, load together
    // with the error bytes and the device-side count
    BlockDesc d = empty_desc();
    if (rec_wave)
        d = tw.start(v, (int)(wave / TouchedWaves::kWaves), (int)(wave % TouchedWaves::kWaves));
    const int64_t i = (wave - (int64_t)regions * TouchedWaves::kWaves) * 64 + lane;
    const bool edit = !rec_wave && i < n_host;
    const int id = *(edit ? ids + i : &kNoTet);
    const uint8_t u = edit ? v.undo[i] : (uint8_t)0xFF;
    // the error bytes of every workgroup of the edit phase
    int bits = threadIdx.x < edit_wgs ? v.wg_err[threadIdx.x] : 0;
    for (int k = threadIdx.x + kBlock; k < edit_wgs; k += kBlock)
        bits |= v.wg_err[k];
    bool bad_n;
    const int n = frame_count(n_host, n_dev, bad_n);
    const int fe = block_or(bits, &s_bits);
    publish_frame(v, fe, n, regions);
    if (rec_wave)
        tw.run(v, d, fe, s_val[threadIdx.x >> 6]);
    else if (edit && i < n)
        touched_edit(v, id, u, fe);
}

// ---------------------------------------------------------------------------
// +/- delta policy (the paper's streaming_update for element assembly:
// touched entries change by adding or removing the edited elements' local
// contributions, Sec. 3.4 / Sec. 3.5)
// ---------------------------------------------------------------------------

// Add s * (block slot r's values) into the CSR values of block d (and its
// mirror), with hardware FP64 atomics.  The order in which concurrent edits
// land is not fixed, so the result is reproducible only up to rounding.
__device__ __forceinline__ void delta_block(const DevView& v, const BlockDesc& d, const double* x, bool add)
{
    if (d.kind == 0) {
#pragma unroll
        for (int vi = 0; vi < 6; ++vi) {
            const int p = kDiagP[vi], q = kDiagQ[vi];
            const double y = add ? x[vi] : -x[vi];
            unsafeAtomicAdd(v.values + d.up + p * d.rl + q, y);
            if (p != q)
                unsafeAtomicAdd(v.values + d.up + q * d.rl + p, y);
        }
    } else {
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                const double y = add ? x[3 * p + q] : -x[3 * p + q];
                unsafeAtomicAdd(v.values + d.up + p * d.rl + q, y);
                unsafeAtomicAdd(v.values + d.lo + q * d.rlj + p, y);
            }
    }
}

// Lane r of edit i under the delta policy (16 lanes per edit, lane r < 10
// owns block slot r).  A changed tet's block entries, formed from its
// geometry record, are added (activation) or subtracted (deletion); the mask
// stays as the exact policy expects, so either policy may follow.  Invalid
// and duplicate edits are skipped and reported; nothing is rolled back.
__device__ __forceinline__ int delta_lane(const DevView& v, int id, unsigned st, int r)
{
    if (id < 0 || id >= v.n_tets || st > 1u)
        return r == 0 ? ERR_RANGE : 0;
    const bool slot = r < 10;
    const uint8_t prev = v.mask[id];
    unsigned taken = 0u;
    if (r == 0)
        taken = atomicExch(&v.estamp[id], 1u);
    BlockDesc bd = empty_desc();
    Geo G;
    double ga[3], gb[3];
    bool degenerate = false;
    if (slot) {
        bd = load_desc(v.trec[id].desc + r);
        const int4 t = v.T[id];
        int A = (int)(kSlotA >> (2 * r)) & 3, B = (int)(kSlotB >> (2 * r)) & 3;
        const bool swap = tet_vertex(t, A) > tet_vertex(t, B);  // block orientation: the smaller node's row
        const TetGeo* q = reinterpret_cast<const TetGeo*>(v.geo) + id;
        const double* pa = q->g + 3 * (swap ? B : A);
        const double* pb = q->g + 3 * (swap ? A : B);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            ga[i] = pa[i];
            gb[i] = pb[i];
        }
        G.lamV = q->lamV;
        G.muV = q->muV;
        G.ml = q->ml;
        degenerate = q->degenerate != 0;
    }
    const bool owner = __shfl(taken, (threadIdx.x & 63) & ~(kEditLanes - 1), 64) == 0u;
    if (!owner)
        return r == 0 ? ERR_DUP : 0;
    if (prev == st)
        return 0;
    if (r == 0) {
        v.mask[id] = (uint8_t)st;
        if (st && degenerate)
            atomicOr(&v.ctl->err, ERR_DEGENERATE);
    }
    if (!slot)
        return 0;
    const double s = dot3(ga, gb);
    double x[9];
    if (r < 4) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            constexpr int P[6] = {0, 0, 0, 1, 1, 2}, Q[6] = {0, 1, 2, 1, 2, 2};
            x[k] = entry(ga, gb, s, G, P[k], Q[k], true);
        }
#pragma unroll
        for (int k = 6; k < 9; ++k)
            x[k] = 0.0;
    } else {
#pragma unroll
        for (int k = 0; k < 9; ++k)
            x[k] = entry(ga, gb, s, G, k / 3, k % 3, false);
    }
    delta_block(v, bd, x, st != 0u);
    return 0;
}

__global__ __launch_bounds__(kBlock) void k_delta_edits(DevView v, const int32_t* __restrict__ ids,
                                                        const uint8_t* __restrict__ states, int32_t n_host,
                                                        const int32_t* __restrict__ n_dev)
{
    const int gt = blockIdx.x * kBlock + threadIdx.x;
    const int i = gt / kEditLanes;
    int id = -1;
    unsigned st = 0;
    if (i < n_host) {
        id = ids[i];
        st = states[i];
    }
    bool bad_n;
    const int n = frame_count(n_host, n_dev, bad_n);
    int bits = (bad_n && gt == 0) ? ERR_RANGE : 0;
    if (i < n)
        bits |= delta_lane(v, id, st, gt - i * kEditLanes);
    if (bits)
        atomicOr(&v.ctl->err, bits);
    if (gt == 0) {
        v.ctl->last_n = n;
        v.ctl->frame_err = 0;
        v.ctl->last_regions = 0;  // the delta policy claims no blocks
    }
}

// Release the frame's tet stamps (one lane per edit).
__global__ __launch_bounds__(kBlock) void k_delta_clear(DevView v, const int32_t* __restrict__ ids, int32_t n_host,
                                                        const int32_t* __restrict__ n_dev)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    bool bad_n;
    const int n = frame_count(n_host, n_dev, bad_n);
    if (i < n) {
        const int id = ids[i];
        if (id >= 0 && id < v.n_tets)
            v.estamp[id] = 0u;
    }
}

// The whole frame in one persistent launch: phase 1 over the edits, grid
// barrier, phase 2 over the claimed blocks (grid-stride loops; lane groups
// stay aligned because the stride is a multiple of the workgroup size).
__global__ __launch_bounds__(kBlock) void k_frame(DevView v, const int32_t* __restrict__ ids,
                                                  const uint8_t* __restrict__ states, int32_t n_host,
                                                  const int32_t* __restrict__ n_dev, unsigned spin_limit)
{
    __shared__ double s_val[kBlock / 64][kUnitDoubles];
    __shared__ int s_bits;
    __shared__ int s_ok;
    bool bad_n;
    const int n = frame_count(n_host, n_dev, bad_n);
    const int regions = (n_host > 0 ? (n_host * kEditLanes + kBlock - 1) / kBlock : 1) * kRegionsPerBlock;
    int bits = (bad_n && blockIdx.x == 0 && threadIdx.x == 0) ? ERR_RANGE : 0;
    // phase 1 over whole waves (one claim region each), so that every lane of
    // a wave runs the compaction together
    for (int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x; t < (int64_t)regions * 64;
         t += (int64_t)gridDim.x * kBlock) {
        const int i = (int)(t / kEditLanes);
        int ckind = -1;
        BlockDesc cbd;
        if (i < n)
            bits |= edit_lane(v, ids[i], states[i], i, (int)(t - (int64_t)i * kEditLanes), ckind, cbd);
        compact_claims(v, t / 64, ckind, cbd);
    }
    bits = block_or(bits, &s_bits);
    if (threadIdx.x == 0)
        v.wg_err[blockIdx.x] = (uint8_t)bits;
    if (!grid_barrier(v.ctl, gridDim.x, spin_limit, &s_ok))
        return;
    const int fe = frame_error(v, gridDim.x, &s_bits);
    publish_frame(v, fe, n, regions);
    const int lane = threadIdx.x & 63;
    const int64_t rec_waves = (int64_t)regions * FusedWaves::kWaves, waves = rec_waves + (n_host + 63) / 64;
    for (int64_t w = (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); w < waves;
         w += (int64_t)gridDim.x * (kBlock / 64)) {
        if (w < rec_waves) {
            FusedWaves fw;
            const BlockDesc d = fw.start(v, (int)(w / FusedWaves::kWaves), (int)(w % FusedWaves::kWaves));
            fw.run(v, d, fe, s_val[threadIdx.x >> 6]);
        } else {
            const int64_t i = (w - rec_waves) * 64 + lane;
            if (i < n)
                touched_edit(v, ids[i], v.undo[i], fe);
        }
    }
}

// A whole frame in one launch without a grid barrier, for edit lists that fit
// a table in LDS.  Every workgroup reads the whole list into its own table
// (validating it, so that all agree on the frame's error before anything is
// written and nothing needs undoing), and three waves per edit re-sum the ten
// blocks of its tet, taking an edited tet's state from the table and any other
// tet's from the mask; only the edit's own waves use and write its tet's mask
// byte, so no result depends on when it is written.  Blocks shared by several
// edits are summed by each of them to the same bits: cheaper than claiming
// them, which takes a second launch (or a grid barrier) before the claims can
// be used.  What remains is a chain of four dependent round trips: edit, block
// descriptors, incidences, geometry.
//
// kEdits: edits per workgroup; kShare: edits of the list per lane (n_host <=
// 64 kUnits kEdits kShare).
template <int kEdits, int kShare>
__global__ __launch_bounds__(64 * kUnits * kEdits) void k_once(DevView v, const int32_t* __restrict__ ids,
                                                               const uint8_t* __restrict__ states, int32_t n_host,
                                                               const int32_t* __restrict__ n_dev, int log2)
{
    constexpr int kThreads = 64 * kUnits * kEdits;
    // the table's heads, then its edits
    extern __shared__ int4 s_dynamic[];
    __shared__ double s_val[kEdits][kTetDoubles];
    __shared__ int s_bits, s_change[kEdits];
    int32_t* head = reinterpret_cast<int32_t*>(s_dynamic);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int unit = wave % kUnits, own = wave / kUnits, i = blockIdx.x * kEdits + own;
    // the wave's own edit, and this lane's share of the list
    int id = -1;
    unsigned st = 0;
    if (n_host > 0) {
        id = ids[min(i, n_host - 1)];
        st = states[min(i, n_host - 1)];
    }
    EditShare<kThreads, kShare> share;
    share.load(ids, states, n_host, &kNoTet, &kNoState);
    share.clear(s_dynamic, log2);
    if (tid == 0)
        s_bits = 0;
    bool bad_n;
    const int n = frame_count(n_host, n_dev, bad_n);
    const bool mine = i < n && id >= 0 && id < v.n_tets;
    BlockDesc bd = empty_desc();
    uint8_t prev = 0;
    bool degenerate = false;
    if (mine) {  // in flight while the table is built
        if (lane < (unit < 2 ? Unit<true>::kBlocks : Unit<false>::kBlocks))
            bd = load_desc(v.trec[id].desc + 2 * unit + lane);
        if (unit == 0) {
            prev = v.mask[id];
            degenerate = is_degenerate(v, id);
        }
    }
    __syncthreads();
    int bits = bad_n ? ERR_RANGE : 0;
    const EditTable table{head, reinterpret_cast<int2*>(head + (1 << log2) + kTableSpare), log2};
    bits |= share.insert(table, n, v.n_tets);
    __syncthreads();
    // in flight while duplicates are looked for
    UnitTerms<true> bdiag{};
    UnitTerms<false> boff{};
    uint32_t u = 0;
    if (mine) {
        if (unit < 2) {
            bdiag = unit_terms<true>(bd);
            u = load_incidence<true>(v, bdiag, 0);
        } else {
            boff = unit_terms<false>(bd);
            u = load_incidence<false>(v, boff, 0);
        }
    }
    bits |= share.duplicates(table);
    if (bits)
        atomicOr(&s_bits, bits);
    if (unit == 0 && lane == 0)
        s_change[own] = prev != st;
    __syncthreads();
    const int fe = s_bits;
    publish_frame(v, fe, n, -1);
    if (fe || !mine)
        return;
    const bool change = s_change[own] != 0;
    if (unit == 0 && lane == 0) {
        v.undo[i] = change ? prev : (uint8_t)0xFF;
        reinterpret_cast<int32_t*>(v.rec)[i] = id;
        if (change) {
            v.mask[id] = (uint8_t)st;
            if (st && degenerate)
                atomicOr(&v.ctl->err, ERR_DEGENERATE);
        }
    }
    if (!change)
        return;
    if (unit < 2)
        sum_unit<true, false>(v, bd, bdiag, u, s_val[own] + unit * kDiagUnitDoubles, table);
    else
        sum_unit<false, false>(v, bd, boff, u, s_val[own] + 2 * kDiagUnitDoubles, table);
}

// Statistics of a frame of k_once: the distinct blocks of its changed tets
// (claimed through their stamps) and their incidences, diagonal and
// off-diagonal, into count[0..3]; then the stamps are released.  Summed per
// workgroup first: an atomic for each block on the four words took 400 us of the
// call after 2,000 edits (515 -> 61 us).
__global__ __launch_bounds__(kBlock) void k_once_stats(DevView v, int n, unsigned long long* count, int release)
{
    __shared__ unsigned long long s_count[4];
    if (threadIdx.x < 4)
        s_count[threadIdx.x] = 0ull;
    __syncthreads();
    const int t = blockIdx.x * kBlock + threadIdx.x, i = t / kEditLanes, r = t % kEditLanes;
    if (i < n && r < 10 && v.undo[i] != 0xFF) {
        const BlockDesc d = load_desc(v.trec[reinterpret_cast<const int32_t*>(v.rec)[i]].desc + r);
        if (release) {
            v.bstamp[d.block] = 0u;
        } else if (atomicExch(&v.bstamp[d.block], 1u) == 0u) {
            atomicAdd(s_count + (d.kind == 0 ? 0 : 1), 1ull);
            atomicAdd(s_count + (d.kind == 0 ? 2 : 3), (unsigned long long)(d.k1 - d.k0));
        }
    }
    __syncthreads();
    if (threadIdx.x < 4 && s_count[threadIdx.x])
        atomicAdd(count + threadIdx.x, s_count[threadIdx.x]);
}

// Audit: 1 if tet e's stored geometry differs in any bit from what the
// rebuild would store.
__device__ __forceinline__ int audit_element(const DevView& v, int e)
{
    Geo G;
    element_geometry(v, e, v.T[e], G);
    const TetGeo* q = reinterpret_cast<const TetGeo*>(v.geo) + e;
    auto differs = [](double x, double y) { return __double_as_longlong(x) != __double_as_longlong(y); };
    bool bad = differs(q->lamV, G.lamV) || differs(q->muV, G.muV) || differs(q->ml, G.ml);
#pragma unroll
    for (int k = 0; k < 12; ++k)
        bad = bad || differs(q->g[k], G.g[k / 3][k % 3]);
    return bad ? 1 : 0;
}

__global__ __launch_bounds__(kBlock) void k_audit_tets(DevView v, unsigned long long* count)
{
    const int e = blockIdx.x * kBlock + threadIdx.x;
    const int bad = e < v.n_tets ? audit_element(v, e) : 0;
    const uint64_t m = __ballot(bad != 0);
    if ((threadIdx.x & 63) == 0 && m)
        atomicAdd(count, (unsigned long long)__popcll(m));
}

// Audit: values whose bits differ between a and b.
__global__ __launch_bounds__(kBlock) void k_audit_values(const double* __restrict__ a, const double* __restrict__ b,
                                                         int64_t n, unsigned long long* count)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool bad = i < n && __double_as_longlong(a[i]) != __double_as_longlong(b[i]);
    const uint64_t m = __ballot(bad);
    if ((threadIdx.x & 63) == 0 && m)
        atomicAdd(count, (unsigned long long)__popcll(m));
}

// Release every tet and block stamp (after a fused frame whose grid barrier
// gave up, some workgroups left before phase 2 and their stamps stay taken).
__global__ __launch_bounds__(kBlock) void k_clear_stamps(DevView v)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < v.n_tets)
        v.estamp[i] = 0u;
    if (i < v.nd + v.no)
        v.bstamp[i] = 0u;
}

// Every tet's block descriptors, 16 bytes a thread, once per context (filling them
// in on the host and copying took 30 of the 228 ms that the building of 384,000 tets
// took).
__global__ __launch_bounds__(kBlock) void k_records(DevView v, int4* __restrict__ out)
{
    static_assert(sizeof(BlockDesc) == 32 && sizeof(TetRecord) == 320, "20 times 16 bytes");
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < 20 * (int64_t)v.n_tets)
        out[i] = reinterpret_cast<const int4*>(v.desc + v.e2b[i / 2])[i % 2];
}

__global__ __launch_bounds__(kBlock) void k_set_params(int n_nodes, int n_tets, const double* __restrict__ x_aos,
                                                       const double* __restrict__ Ein, double* xs, double* ys,
                                                       double* zs, double* Eout)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (x_aos && i < n_nodes) {
        xs[i] = x_aos[3 * (size_t)i + 0];
        ys[i] = x_aos[3 * (size_t)i + 1];
        zs[i] = x_aos[3 * (size_t)i + 2];
    }
    if (Ein && i < n_tets)
        Eout[i] = Ein[i];
}

inline unsigned blocks_for(int64_t threads)
{
    return (unsigned)((threads + kBlock - 1) / kBlock);
}

}  // namespace

hipError_t launch_records(const DevView& v, TetRecord* trec, hipStream_t s)
{
    if (v.n_tets == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_records, dim3(blocks_for(20 * (int64_t)v.n_tets)), dim3(kBlock), 0, s, v,
                       reinterpret_cast<int4*>(trec));
    return hipGetLastError();
}

hipError_t launch_geometry(const DevView& v, hipStream_t s)
{
    if (v.n_tets == 0)
        return hipSuccess;
    launch_kernel(&k_geometry, dim3(blocks_for(v.n_tets)), dim3(kBlock), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_rows(const DevView& v, bool nt, hipStream_t s)
{
    if (v.n_tiles == 0)
        return hipSuccess;
    if (nt)
        launch_kernel(&k_rows<true>, dim3(v.n_tiles), dim3(kRowThreads), 0, s, v);
    else
        launch_kernel(&k_rows<false>, dim3(v.n_tiles), dim3(kRowThreads), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_rows_big(const DevView& v, bool always, hipStream_t s)
{
    const int waves = (v.n_bigd + Unit<true>::kBlocks - 1) / Unit<true>::kBlocks +
                      (v.n_bigo + Unit<false>::kBlocks - 1) / Unit<false>::kBlocks;
    if (waves == 0 && !always)
        return hipSuccess;
    launch_kernel(&k_rows_big, dim3(waves > 0 ? (waves + kBlock / 64 - 1) / (kBlock / 64) : 1), dim3(kBlock), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_edit_phase(const DevView& v, const int32_t* ids, const uint8_t* states, int32_t n_host,
                             const int32_t* n_dev, hipStream_t s)
{
    // an empty list still runs one workgroup of each phase: they record the frame (count 0)
    launch_kernel(&k_edits, dim3(n_host > 0 ? blocks_for((int64_t)n_host * kEditLanes) : 1u), dim3(kBlock), 0,
                       s, v, ids, states, n_host, n_dev);
    return hipGetLastError();
}

hipError_t launch_delta_frame(const DevView& v, const int32_t* ids, const uint8_t* states, int32_t n_host,
                              const int32_t* n_dev, hipStream_t s)
{
    hipLaunchKernelGGL(k_delta_edits, dim3(n_host > 0 ? blocks_for((int64_t)n_host * kEditLanes) : 1u), dim3(kBlock),
                       0, s, v, ids, states, n_host, n_dev);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_host == 0)
        return e;
    hipLaunchKernelGGL(k_delta_clear, dim3(blocks_for(n_host)), dim3(kBlock), 0, s, v, ids, n_host, n_dev);
    return hipGetLastError();
}

hipError_t launch_once(const DevView& v, const int32_t* ids, const uint8_t* states, int32_t n_host,
                       const int32_t* n_dev, hipStream_t s)
{
    const int log2 = table_log2(n_host);
#define ONCE(E, S)                                                                                           \
    if (n_host <= 64 * kUnits * E * S) {                                                                     \
        launch_kernel(&k_once<E, S>, dim3(n_host > 0 ? (n_host + E - 1) / E : 1), dim3(64 * kUnits * E),     \
                      table_bytes(log2, 64 * kUnits * E, S),                                                 \
                      s, v, ids, states, n_host, n_dev, log2);                                               \
        return hipGetLastError();                                                                            \
    }
    ONCE(1, 1)
    ONCE(2, 2)
    ONCE(4, 3)
#undef ONCE
    return hipErrorInvalidValue;
}
static_assert(kFrameOnceEdits == 64 * kUnits * 4 * 3, "the largest variant covers the largest list");

hipError_t launch_once_stats(const DevView& v, int32_t n, unsigned long long* counts4, hipStream_t s)
{
    hipError_t e = hipMemsetAsync(counts4, 0, 4 * sizeof(unsigned long long), s);
    for (int release = 0; release <= 1 && e == hipSuccess && n > 0; ++release) {
        hipLaunchKernelGGL(k_once_stats, dim3(blocks_for((int64_t)n * kEditLanes)), dim3(kBlock), 0, s, v, n, counts4,
                           release);
        e = hipGetLastError();
    }
    return e;
}

// Lanes of phase 2: the regions' waves, then one lane per edit.
static int64_t touched_lanes(int32_t n_host, int region_waves)
{
    const int64_t regions = (n_host > 0 ? ((int64_t)n_host * kEditLanes + kBlock - 1) / kBlock : 1) * kRegionsPerBlock;
    return regions * region_waves * 64 + n_host;
}

hipError_t launch_touched_phase(const DevView& v, const int32_t* ids, int32_t n_host, const int32_t* n_dev,
                                hipStream_t s)
{
    launch_kernel(&k_touched, dim3(blocks_for(touched_lanes(n_host, TouchedWaves::kWaves))), dim3(kBlock), 0, s, v, ids, n_host, n_dev);
    return hipGetLastError();
}

// The query counts seven workgroups of k_frame on a compute unit, by its 72
// VGPRs and 104 scalar ones, and a grid of so many was not all resident: its
// barrier gave up.  The scalar registers that each wave holds besides its own are
// not in that count, so it takes no more than five, which leave a third of them.
constexpr int kFramePerCu = 5;
hipError_t frame_max_grid(int device, int* max_grid)
{
    int cus = 0, per_cu = 0;
    hipError_t e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e == hipSuccess)
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)&k_frame, kBlock, 0);
    if (e == hipSuccess)
        *max_grid = (per_cu < kFramePerCu ? per_cu : kFramePerCu) * cus;
    return e;
}

int frame_grid_for(int32_t n_host, int max_grid, int grid_cap)
{
    const int64_t want = (touched_lanes(n_host, FusedWaves::kWaves) + kBlock - 1) / kBlock;
    int64_t g = want < max_grid ? want : max_grid;
    if (grid_cap > 0 && g > grid_cap)
        g = grid_cap;
    return (int)(g < 1 ? 1 : g);
}

hipError_t launch_frame(const DevView& v, int grid, const int32_t* ids, const uint8_t* states, int32_t n_host,
                        const int32_t* n_dev, unsigned spin_limit, hipStream_t s)
{
    launch_kernel(&k_frame, dim3(grid), dim3(kBlock), 0, s, v, ids, states, n_host, n_dev, spin_limit);
    return hipGetLastError();
}

hipError_t launch_audit(const DevView& v, double* scratch_values, int64_t nnz, unsigned long long* counts,
                        hipStream_t s)
{
    hipError_t e = hipSuccess;
    if (v.n_tets > 0) {
        hipLaunchKernelGGL(k_audit_tets, dim3(blocks_for(v.n_tets)), dim3(kBlock), 0, s, v, counts + 1);
        e = hipGetLastError();
    }
    if (e != hipSuccess || nnz == 0)
        return e;
    DevView w = v;
    w.values = scratch_values;
    e = launch_rows(w, false, s);
    if (e == hipSuccess)
        e = launch_rows_big(w, false, s);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(k_audit_values, dim3(blocks_for(nnz)), dim3(kBlock), 0, s, v.values, scratch_values, nnz,
                       counts);
    return hipGetLastError();
}

hipError_t launch_clear_stamps(const DevView& v, hipStream_t s)
{
    const int64_t n = v.n_tets > v.nd + v.no ? v.n_tets : v.nd + v.no;
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_clear_stamps, dim3(blocks_for(n)), dim3(kBlock), 0, s, v);
    return hipGetLastError();
}

hipError_t launch_set_params(const DevView& v, const double* x_aos, const double* E, double* xs, double* ys,
                             double* zs, double* Eout, hipStream_t s)
{
    const int64_t n = v.n_nodes > v.n_tets ? v.n_nodes : v.n_tets;
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_set_params, dim3(blocks_for(n)), dim3(kBlock), 0, s, v.n_nodes, v.n_tets, x_aos, E, xs,
                       ys, zs, Eout);
    return hipGetLastError();
}

}  // namespace sta
