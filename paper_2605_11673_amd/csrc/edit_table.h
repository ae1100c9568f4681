// A frame's edit list as a table in LDS, for kernels that apply a whole frame
// in one launch: every workgroup holds the whole list, so that all of them
// agree on the frame's error before anything is written, and take the state of
// an edited tet from the list, whether or not its mask byte is written yet.
#pragma once

#include <hip/hip_runtime.h>

#include "sta_internal.h"

namespace sta {

constexpr uint32_t kUnlisted = 2u;  // EditTable::listed of a tet that no edit names
constexpr int kTableSpare = 64;     // heads past the buckets, for lanes without an edit

// Chained hash table: head[h] is the last edit of bucket h (-1: none) and
// edit[i] = (tet << 1 | requested state, the next edit of its bucket).
struct EditTable {
    int32_t* head;
    int2* edit;
    int log2;
    __device__ __forceinline__ uint32_t bucket(uint32_t e) const { return (e * 2654435761u) >> (32 - log2); }
    __device__ __forceinline__ uint32_t listed(uint32_t e) const
    {
        uint32_t l = kUnlisted;
        for (int i = head[bucket(e)]; i >= 0;) {
            const int2 t = edit[i];
            l = (uint32_t)t.x >> 1 == e ? (uint32_t)t.x & 1u : l;
            i = t.y;
        }
        return l;
    }
};

// log2 of the buckets for a list: at least the edits, up to 2048.
inline int table_log2(int32_t n)
{
    int log2 = 8;
    while ((1 << log2) < n && log2 < 11)
        ++log2;
    return log2;
}

// Bytes of LDS: the heads, then one edit per thread and share.
inline uint32_t table_bytes(int log2, int threads, int share)
{
    return (uint32_t)(sizeof(int32_t) * ((1 << log2) + kTableSpare) + sizeof(int2) * threads * share);
}

// One thread's share of the list: edits t, t + kThreads, ...  load and clear,
// __syncthreads, insert, __syncthreads, duplicates, __syncthreads.
template <int kThreads, int kShare>
struct EditShare {
    int id[kShare], next[kShare];
    uint8_t state[kShare];
    bool valid[kShare];

    // none_id, none_state: what an empty list reads
    __device__ __forceinline__ void load(const int32_t* ids, const uint8_t* states, int n_host, const int32_t* none_id,
                                         const uint8_t* none_state)
    {
#pragma unroll
        for (int k = 0; k < kShare; ++k) {
            id[k] = *(n_host > 0 ? ids + min((int)threadIdx.x + k * kThreads, n_host - 1) : none_id);
            state[k] = *(n_host > 0 ? states + min((int)threadIdx.x + k * kThreads, n_host - 1) : none_state);
        }
    }
    static __device__ __forceinline__ void clear(int4* heads, int log2)
    {
        for (int h = threadIdx.x; h < 1 << (log2 - 2); h += kThreads)
            heads[h] = make_int4(-1, -1, -1, -1);
    }
    // The first n edits into the table; error bits of those that are not valid.
    __device__ __forceinline__ int insert(const EditTable& table, int n, int n_tets)
    {
        int bits = 0;
#pragma unroll
        for (int k = 0; k < kShare; ++k) {
            const int t = (int)threadIdx.x + k * kThreads;
            const bool in = t < n;
            valid[k] = in && (uint32_t)id[k] < (uint32_t)n_tets && state[k] <= 1;
            bits |= in && !valid[k] ? ERR_RANGE : 0;
            next[k] = atomicExch(table.head + (valid[k] ? table.bucket((uint32_t)id[k])
                                                        : (1u << table.log2) + (threadIdx.x & 63u)),
                                 t);
        }
#pragma unroll
        for (int k = 0; k < kShare; ++k) {
            next[k] = valid[k] ? next[k] : -1;
            table.edit[threadIdx.x + k * kThreads] =
                make_int2((int)((uint32_t)id[k] << 1 | (state[k] & 1u)), next[k]);
        }
        return bits;
    }
    // A duplicate finds its twin further down its own chain.
    __device__ __forceinline__ int duplicates(const EditTable& table)
    {
        int bits = 0;
        bool more = false;
#pragma unroll
        for (int k = 0; k < kShare; ++k)
            more |= next[k] >= 0;
        while (more) {
            int2 t[kShare];
#pragma unroll
            for (int k = 0; k < kShare; ++k)
                t[k] = table.edit[next[k] >= 0 ? next[k] : 0];
            more = false;
#pragma unroll
            for (int k = 0; k < kShare; ++k)
                if (next[k] >= 0) {
                    bits |= (uint32_t)t[k].x >> 1 == (uint32_t)id[k] ? ERR_DUP : 0;
                    next[k] = t[k].y;
                    more |= next[k] >= 0;
                }
        }
        return bits;
    }
};

}  // namespace sta
