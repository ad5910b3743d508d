// TransR: the items of a mini-batch, the (chunk, relation) pairs that occur in it, with their positives.  Formed by extra
// workgroups of the gather launch, one per chunk.
#pragma once
#include "kge_common.h"

constexpr int TRANSR_PB = 32;  // positives per block of an item's positives

// most items of a chunk of g positives, most blocks of positives
inline int transr_max_items(int g, int64_t n_rel) { return g < n_rel ? g : (int)n_rel; }
inline int transr_max_pblocks(int g, int64_t n_rel) { return transr_max_items(g, n_rel) + g / TRANSR_PB; }

#ifdef __HIPCC__
namespace {

constexpr int ITEM_TILE = 2048;  // positives of a chunk whose relation ids and intermediate results stay in LDS

__device__ __forceinline__ int wave_scan(int v) {  // inclusive
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(v, o, 64);
        if (lane >= o) v += u;
    }
    return v;
}

constexpr int ITEM_TABLE = 4096;  // relations that are counted in LDS tables

// Rank of every positive among the positives of the chunk with its relation, and their number.
// Few relations: a table of counts in LDS.  A wave finds its lanes with equal relations from ballots over the bits of the
// id; the first of them adds their number to the table, wave after wave, so that ranks follow the order of the positives.
// (Work linear in g: 2 us at g = 266; comparing every positive with every other took 20.)
// Many relations: brute force over the chunk's relation ids in LDS, four per read, up to 16 threads per positive.
// A scan over the first positives of the items then numbers the items and lays out their positives and blocks of positives.
template <int THREADS>
__device__ void transr_items(const TransrGroups& q, const int64_t* r, int c, int g, int64_t n_rel, int max_pblocks) {
    __shared__ __attribute__((aligned(16))) uint32_t id[ITEM_TILE];
    __shared__ int rank_[ITEM_TILE];
    __shared__ int table[ITEM_TABLE], offset[ITEM_TABLE];
    __shared__ int wsum[3][THREADS / 64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const bool small = g <= ITEM_TILE, few = n_rel <= ITEM_TABLE;
    int* rank = small ? rank_ : q.rank + c * g;  // longer chunks keep it in memory
    int* first = q.first + c * g;                // (many relations only)
    auto key = [&](int p) {
        const int64_t x = r[p];
        return (uint32_t)(x < 0 ? 0 : x >= n_rel ? n_rel - 1 : x);
    };
    auto key_again = [&](int p) { return small ? id[p] : key(p); };
    auto stage = [&](int t0) {
        __syncthreads();
        for (int e = tid; e < ITEM_TILE && t0 + e < ((g + 3) & ~3); e += THREADS)
            id[e] = t0 + e < g ? key(t0 + e) : 0xffffffffu;  // (no relation has that id)
        __syncthreads();
    };
    if (few)
        for (int e = tid; e < n_rel; e += THREADS) table[e] = 0;
    if (small) stage(0);
    else __syncthreads();
    if (few) {
        const int bits = 32 - __builtin_clz((uint32_t)n_rel);
        for (int p0 = 0; p0 < g; p0 += THREADS) {
            const int p = p0 + tid;
            const bool valid = p < g;
            const uint32_t mine = valid ? key_again(p) : 0;
            unsigned long long same = __ballot(valid);
            for (int x = 0; x < bits; ++x) {
                const bool bit = mine >> x & 1;
                const unsigned long long bal = __ballot(bit);
                same &= bit ? bal : ~bal;
            }
            const int leader = __builtin_ctzll(same | 1ull << 63);
            int old = 0;
            for (int w = 0; w < THREADS / 64; ++w) {
                if (wave == w && valid && lane == leader) {
                    old = table[mine];
                    table[mine] = old + __popcll(same);
                }
                __syncthreads();
            }
            old = __shfl(old, leader, 64);
            if (valid) rank[p] = old + __popcll(same & ((1ull << lane) - 1));
        }
    } else {
        int share = 1;  // threads per positive
        while (share < 16 && g * share * 2 <= THREADS) share *= 2;
        for (int p0 = 0; p0 < g; p0 += THREADS / share) {
            const int p = p0 + tid / share, part = tid % share;
            const uint32_t mine = p < g ? key(p) : 0xfffffffeu;
            int fst = g, rnk = 0, cnt = 0;
            for (int t0 = 0; t0 < g; t0 += ITEM_TILE) {
                if (!small) stage(t0);
                const int lim = min(ITEM_TILE, g - t0);
#pragma unroll 2
                for (int e = 4 * part; e < lim; e += 4 * share) {
                    const uint4 v = *reinterpret_cast<const uint4*>(id + e);
                    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const bool eq = w[u] == mine;
                        const int at = t0 + e + u;
                        cnt += eq;
                        rnk += eq && at < p;
                        fst = eq && at < fst ? at : fst;
                    }
                }
            }
            for (int o = share / 2; o > 0; o >>= 1) {
                cnt += __shfl_xor(cnt, o, 64);
                rnk += __shfl_xor(rnk, o, 64);
                fst = min(fst, __shfl_xor(fst, o, 64));
            }
            if (p < g && part == 0) {
                first[p] = fst;
                rank[p] = rnk;
                q.slot_of[c * g + p] = cnt;  // (until the scan)
            }
        }
    }
    __syncthreads();
    int items = 0, members = 0, blocks = 0;  // of earlier rounds
    for (int p0 = 0; p0 < g; p0 += THREADS) {
        const int p = p0 + tid;
        const uint32_t mine = p < g ? key_again(p) : 0;
        const int all = p < g ? (few ? table[mine] : q.slot_of[c * g + p]) : 0;
        const bool rep = p < g && rank[p] == 0;
        const int cnt = rep ? all : 0, nb = (cnt + TRANSR_PB - 1) / TRANSR_PB;
        const int si = wave_scan(rep), sm = wave_scan(cnt), sb = wave_scan(nb);
        if (lane == 63) { wsum[0][wave] = si; wsum[1][wave] = sm; wsum[2][wave] = sb; }
        __syncthreads();
        int bi = items, bm = members, bb = blocks;
        for (int w = 0; w < THREADS / 64; ++w) {
            if (w < wave) { bi += wsum[0][w]; bm += wsum[1][w]; bb += wsum[2][w]; }
            items += wsum[0][w]; members += wsum[1][w]; blocks += wsum[2][w];
        }
        const int slot = c * g + bi + si - 1, off = c * g + bm + sm - cnt;
        if (p < g) q.slot_of[c * g + p] = rep ? slot : -1;
        if (rep) {
            if (few) offset[mine] = off;
            q.items[slot] = {mine, off, cnt};
            for (int x = 0; x < nb; ++x)
                q.pblocks[(int64_t)c * max_pblocks + bb + sb - nb + x] = {slot, mine, off + x * TRANSR_PB, min(TRANSR_PB, cnt - x * TRANSR_PB),
                                                                        x * TRANSR_PB, cnt};
        }
        __syncthreads();
    }
    if (tid == 0) { q.n_items[c] = items; q.n_pblocks[c] = blocks; }
    for (int p = tid; p < g; p += THREADS) {
        int off, all;
        if (few) {
            const uint32_t mine = key_again(p);
            off = offset[mine];
            all = table[mine];
        } else {
            const TransrItem item = q.items[q.slot_of[c * g + first[p]]];
            off = item.off;
            all = item.n;
        }
        q.members[off + rank[p]] = c * g + p;
        q.count[off + rank[p]] = all;
    }
}

}  // namespace
#endif
