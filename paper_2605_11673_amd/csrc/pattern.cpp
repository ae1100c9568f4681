// Host-side construction of the fixed superset pattern and of the maps the
// kernels use (paper Sec. 3.3: "precomputed tetrahedron-to-edge incidence";
// here the elasticity analogue, tet -> 3x3 node blocks).
//
// Blocks.  Every node that lies in some candidate tet owns a diagonal block
// (i,i); every node pair i<j that shares a candidate tet owns an off-diagonal
// block (i,j).  A block's incidence segment lists the candidate tets that
// contribute to it in ascending tet id; this order is the summation order of
// every entry, in the rebuild and in the streaming update alike.
//
// CSR, for node blocks of size bs (3 for elasticity, 1 for the scalar proxy
// operator).  Row bs*i+p has the columns bs*j+q of every neighbour j of i
// (i itself included) in ascending order, so the bs rows of node i share one
// column list of length bs*deg(i).  A block's values therefore sit at
//   up + p*rowlen(i) + q            (upper block, row node i)
//   lo + q*rowlen(j) + p            (its mirror, row node j)
// with up / lo the CSR index of entry (bs*i,bs*j) / (bs*j,bs*i).
#include <algorithm>
#include <cstring>

#include "sta_internal.h"

namespace sta {

namespace {
const int kPairA[6] = {0, 0, 0, 1, 1, 2};
const int kPairB[6] = {1, 2, 3, 2, 3, 3};
}  // namespace

std::string build_host_pattern(int64_t n, const int32_t* tets, int64_t m, HostPattern& P, int bs)
{
    // diagonal blocks: used nodes in ascending id
    std::vector<int32_t> did(n, -1);
    for (int64_t e = 0; e < m; ++e)
        for (int a = 0; a < 4; ++a)
            did[tets[4 * e + a]] = 0;
    int64_t nd = 0;
    for (int64_t i = 0; i < n; ++i)
        if (did[i] == 0)
            did[i] = (int32_t)nd++;

    // off-diagonal blocks: unique (min, max) node pairs in ascending order, the larger nodes of each
    // smaller one sorted by themselves (one sort of all pairs took three times as long)
    std::vector<int64_t> first((size_t)n + 1, 0);
    auto smaller = [&](int64_t e, int p) { return std::min(tets[4 * e + kPairA[p]], tets[4 * e + kPairB[p]]); };
    auto larger = [&](int64_t e, int p) { return std::max(tets[4 * e + kPairA[p]], tets[4 * e + kPairB[p]]); };
    for (int64_t e = 0; e < m; ++e)
        for (int p = 0; p < 6; ++p)
            first[smaller(e, p) + 1]++;
    for (int64_t i = 0; i < n; ++i)
        first[i + 1] += first[i];
    std::vector<int32_t> partner((size_t)m * 6);
    {
        std::vector<int64_t> fill(first.begin(), first.end() - 1);
        for (int64_t e = 0; e < m; ++e)
            for (int p = 0; p < 6; ++p)
                partner[fill[smaller(e, p)]++] = larger(e, p);
    }
    int64_t no = 0;
    for (int64_t i = 0; i < n; ++i) {  // unique ones to the front; first[i] becomes their begin
        const auto b = partner.begin() + first[i], e = partner.begin() + first[i + 1];
        std::sort(b, e);
        const auto u = std::unique(b, e);
        std::copy(b, u, partner.begin() + no);
        first[i] = no;
        no += u - b;
    }
    first[n] = no;
    partner.resize((size_t)no);
    if (nd > INT32_MAX || no > INT32_MAX || 6 * m > INT32_MAX)
        return "mesh too large for 32-bit block indices";

    // element -> block ids, and segment sizes
    P.e2b.assign((size_t)m * 10, 0);
    std::vector<int64_t> dcount(nd + 1, 0), ocount(no + 1, 0);
    for (int64_t e = 0; e < m; ++e) {
        for (int a = 0; a < 4; ++a) {
            int32_t b = did[tets[4 * e + a]];
            P.e2b[10 * e + a] = b;
            dcount[b + 1]++;
        }
        for (int p = 0; p < 6; ++p) {
            const int32_t i = smaller(e, p);
            const int32_t b = (int32_t)(std::lower_bound(partner.begin() + first[i], partner.begin() + first[i + 1],
                                                         larger(e, p)) - partner.begin());
            P.e2b[10 * e + 4 + p] = b;
            ocount[b + 1]++;
        }
    }
    P.dseg.assign(nd + 1, 0);
    P.oseg.assign(no + 1, 0);
    for (int64_t b = 0; b < nd; ++b)
        P.dseg[b + 1] = (int32_t)(P.dseg[b] + dcount[b + 1]);
    for (int64_t b = 0; b < no; ++b)
        P.oseg[b + 1] = (int32_t)(P.oseg[b] + ocount[b + 1]);

    // incidences in ascending element id within each segment (counting sort)
    P.dinc.assign((size_t)m * 4, 0);
    P.oinc.assign((size_t)m * 6, 0);
    P.e2p.assign((size_t)m * 10, 0);
    std::vector<int32_t> dfill(P.dseg.begin(), P.dseg.end() - 1), ofill(P.oseg.begin(), P.oseg.end() - 1);
    for (int64_t e = 0; e < m; ++e) {
        for (int a = 0; a < 4; ++a) {
            int32_t b = P.e2b[10 * e + a];
            int32_t k = dfill[b]++;
            P.dinc[k] = (int32_t)e;
            P.e2p[10 * e + a] = k;
        }
        for (int p = 0; p < 6; ++p) {
            int32_t b = P.e2b[10 * e + 4 + p];
            int32_t k = ofill[b]++;
            P.oinc[k] = (int32_t)e;
            P.e2p[10 * e + 4 + p] = k;
        }
    }

    // node adjacency (self included), ascending
    std::vector<int64_t> deg(n + 1, 0);
    for (int64_t i = 0; i < n; ++i)
        deg[i + 1] = did[i] >= 0 ? 1 : 0;
    for (int64_t i = 0; i < n; ++i)
        for (int64_t b = first[i]; b < first[i + 1]; ++b) {
            deg[i + 1]++;
            deg[partner[b] + 1]++;
        }
    std::vector<int64_t> aoff(n + 1, 0);
    for (int64_t i = 0; i < n; ++i)
        aoff[i + 1] = aoff[i] + deg[i + 1];
    std::vector<int32_t> adj((size_t)aoff[n]);
    std::vector<int64_t> afill(aoff.begin(), aoff.end() - 1);
    for (int64_t i = 0; i < n; ++i)
        if (did[i] >= 0)
            adj[afill[i]++] = (int32_t)i;
    for (int64_t i = 0; i < n; ++i)
        for (int64_t b = first[i]; b < first[i + 1]; ++b) {
            adj[afill[i]++] = partner[b];
            adj[afill[partner[b]]++] = (int32_t)i;
        }
    for (int64_t i = 0; i < n; ++i)
        std::sort(adj.begin() + aoff[i], adj.begin() + aoff[i + 1]);

    // CSR
    int64_t nnz = 0;
    for (int64_t i = 0; i < n; ++i)
        nnz += (int64_t)bs * bs * (aoff[i + 1] - aoff[i]);
    if (nnz > INT32_MAX)
        return "pattern has more than 2^31-1 entries";
    P.nnz = nnz;
    P.rowptr.assign((size_t)bs * n + 1, 0);
    P.colidx.assign((size_t)nnz, 0);
    int64_t at = 0;
    for (int64_t i = 0; i < n; ++i) {
        const int64_t d = aoff[i + 1] - aoff[i];
        for (int p = 0; p < bs; ++p) {
            P.rowptr[bs * i + p] = (int32_t)at;
            for (int64_t s = 0; s < d; ++s)
                for (int q = 0; q < bs; ++q)
                    P.colidx[at++] = bs * adj[aoff[i] + s] + q;
        }
    }
    P.rowptr[bs * n] = (int32_t)at;

    auto pos = [&](int64_t i, int64_t j) -> int64_t {
        auto b = adj.begin() + aoff[i], e = adj.begin() + aoff[i + 1];
        return std::lower_bound(b, e, (int32_t)j) - b;
    };
    P.dmeta.assign((size_t)nd * 2, 0);
    for (int64_t i = 0; i < n; ++i) {
        if (did[i] < 0)
            continue;
        const int64_t b = did[i];
        P.dmeta[2 * b + 0] = (int32_t)(P.rowptr[bs * i] + bs * pos(i, i));
        P.dmeta[2 * b + 1] = (int32_t)(bs * (aoff[i + 1] - aoff[i]));
    }
    P.ometa.assign((size_t)no * 4, 0);
    P.opair.assign((size_t)no * 2, 0);
    for (int64_t b = 0, i = 0; b < no; ++b) {
        while (b >= first[i + 1])
            ++i;
        const int64_t j = partner[b];
        P.opair[2 * b + 0] = (int32_t)i;
        P.opair[2 * b + 1] = (int32_t)j;
        P.ometa[4 * b + 0] = (int32_t)(P.rowptr[bs * i] + bs * pos(i, j));
        P.ometa[4 * b + 1] = (int32_t)(bs * (aoff[i + 1] - aoff[i]));
        P.ometa[4 * b + 2] = (int32_t)(P.rowptr[bs * j] + bs * pos(j, i));
        P.ometa[4 * b + 3] = (int32_t)(bs * (aoff[j + 1] - aoff[j]));
    }
    P.ndiag.assign(did.begin(), did.end());
    P.nd = nd;
    P.no = no;
    return "";
}

void build_row_plan(int64_t n, const int32_t* tets, int64_t m, const HostPattern& P,
                    const std::vector<int64_t>& node_off, RowPlan& R)
{
    // incidences with their local vertices
    R.di.resize((size_t)m * 4);
    R.oi.resize((size_t)m * 6);
    for (int64_t e = 0; e < m; ++e)
        for (int a = 0; a < 4; ++a)
            R.di[P.e2p[10 * e + a]] = (uint32_t)e << 2 | (uint32_t)a;
    for (int64_t e = 0; e < m; ++e)
        for (int p = 0; p < 6; ++p) {  // the pair's smaller node first, as in opair
            const uint32_t a = kPairA[p], b = kPairB[p];
            const bool up = tets[4 * e + a] < tets[4 * e + b];
            R.oi[P.e2p[10 * e + 4 + p]] = (uint32_t)e << 4 | (up ? a << 2 | b : b << 2 | a);
        }
    // per row block (9 CSR values each) its off-diagonal block and whether the row is its upper node
    const int64_t nb = P.nnz / 9;
    std::vector<int32_t> row_off((size_t)nb, -1);
    for (int64_t o = 0; o < P.no; ++o) {
        const int64_t i = P.opair[2 * o], j = P.opair[2 * o + 1];
        row_off[P.rowptr[3 * i] / 9 + (P.ometa[4 * o + 0] - P.rowptr[3 * i]) / 3] = (int32_t)(2 * o);
        row_off[P.rowptr[3 * j] / 9 + (P.ometa[4 * o + 2] - P.rowptr[3 * j]) / 3] = (int32_t)(2 * o + 1);
    }
    R.rowblk.assign((size_t)nb, make_uint2(0, 0));
    R.terms.reserve((size_t)m * 12);
    R.rownode.reserve((size_t)P.nd);
    std::vector<uint8_t> big_off((size_t)P.no, 0);
    size_t mesh = 0;
    bool open = false;
    for (int64_t i = 0; i < n; ++i) {
        while (mesh + 2 < node_off.size() && i >= node_off[mesh + 1]) {
            ++mesh;
            open = false;
        }
        const int32_t d = P.ndiag[i];
        if (d < 0)
            continue;
        const int32_t b0 = P.rowptr[3 * i] / 9, b1 = P.rowptr[3 * i + 3] / 9;
        const int pairs = P.dseg[d + 1] - P.dseg[d];
        int64_t terms = 0;
        for (int32_t b = b0; b < b1; ++b)
            if (row_off[b] >= 0)
                terms += P.oseg[row_off[b] / 2 + 1] - P.oseg[row_off[b] / 2];
        if (pairs > kTilePairs || b1 - b0 > kTileBlocks || terms > kTileTerms) {
            R.bigd.push_back(d);
            R.bigd_mesh.push_back((int32_t)mesh);
            for (int32_t b = b0; b < b1; ++b)
                if (row_off[b] >= 0)
                    big_off[row_off[b] / 2] = 1;
            open = false;
            continue;
        }
        if (open) {
            const RowTile& t = R.tiles.back();
            open = t.pairs + pairs <= kTilePairs && t.blks + (b1 - b0) <= kTileBlocks && t.nodes < kTileNodes &&
                   t.terms + terms <= kTileTerms && t.pair0 + t.pairs == P.dseg[d] && t.blk0 + t.blks == b0;
        }
        if (!open) {
            RowTile t{};
            t.pair0 = P.dseg[d];
            t.blk0 = b0;
            t.term0 = (int32_t)R.terms.size();
            t.val0 = P.rowptr[3 * i];
            t.node0 = (int32_t)R.rownode.size();
            R.tiles.push_back(t);
            R.tile_mesh.push_back((int32_t)mesh);
            open = true;
        }
        RowTile& t = R.tiles.back();
        const uint32_t rl = (uint32_t)(3 * (b1 - b0));
        const uint32_t p0 = (uint32_t)t.pairs, row0 = (uint32_t)(P.rowptr[3 * i] - t.val0);
        for (int32_t b = b0; b < b1; ++b) {
            const uint32_t at = row0 + 3u * (uint32_t)(b - b0), first = (uint32_t)t.terms;
            if (row_off[b] >= 0) {
                const int32_t o = row_off[b] / 2;
                for (int32_t k = P.oseg[o]; k < P.oseg[o + 1]; ++k) {
                    const int64_t e = P.oinc[k];
                    const uint32_t u = R.oi[k] & 15u;
                    const uint32_t a = row_off[b] % 2 ? u & 3u : u >> 2, c = row_off[b] % 2 ? u >> 2 : u & 3u;
                    const uint32_t p = p0 + (uint32_t)(P.e2p[10 * e + a] - P.dseg[d]);
                    R.terms.push_back((uint16_t)(p << 4 | a << 2 | c));
                    ++t.terms;
                }
            }
            R.rowblk[b] = make_uint2(first | ((uint32_t)t.terms - first) << 16, at | rl << 16);
            if (row_off[b] < 0)
                R.rownode.push_back(make_uint2(p0 | (uint32_t)pairs << 16, at | rl << 16));
        }
        t.pairs += pairs;
        t.blks += b1 - b0;
        t.nodes += 1;
    }
    mesh = 0;
    for (int64_t o = 0; o < P.no; ++o) {
        while (mesh + 2 < node_off.size() && P.opair[2 * o] >= node_off[mesh + 1])
            ++mesh;
        if (big_off[o]) {
            R.bigo.push_back((int32_t)(P.nd + o));
            R.bigo_mesh.push_back((int32_t)mesh);
        }
    }
}

}  // namespace sta
