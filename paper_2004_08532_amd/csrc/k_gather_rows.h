// Device code of the row gather and of the key ranking, for the launches that hold such workgroups: k_gather.hip (nothing
// else in the launch) and k_front.hip (beside the tiles of the forward product).
#pragma once
#include "kge_common.h"
#include "k_transr_items.h"

namespace {

struct GatherArgs {
    const float* E;
    const float* R;
    StepIds ids;
    int b, n_neg, D, Dr, bf16;
    float gamma;
    int64_t n_ent, n_rel;
    float* O;
    float* Nst;
    uint16_t* Obf;  // bf16 operands: o_i and the corrupting rows as the products read them (row pitch ld_bf);
    uint16_t* Nbf;  // Nst is then not written
    int ld_bf;
    float* fpos;
    float* pos_out;
    float* o_n2;
    float* n_n2;
    float* cpos;      // dL/df+_i = -sigmoid(-f+_i) / b
    float* inv_dpos;  // TransE-L2: 1 / |o_i - c_i| (0 if the distance is 0)
    float* row_loss;  // softplus(-f+_i) / b
    int32_t* rank_out;  // evaluation with ranks counted by the forward launch: set to 1 here (else null)
    int rank_blocks;         // blocks [0, rank_blocks) order the key lists, the others gather rows
    int ent_rank_blocks;     // the first ent_rank_blocks of them order the entity key list, the rest the relation keys
    uint64_t bucket_mul;     // long entity lists: bucket of an id = (id * bucket_mul) >> 32 (0: brute-force blocks)
    KeyList ent, rel;
    // TransR: workgroups that form the items of the chunks, chunks of g positives
    int item_blocks, g, max_pblocks;
    TransrGroups items;
};

// One block size for both kinds of block in a launch: THREADS = 256 for short key lists, 1024 for long ones.  The
// rank blocks keep the whole key list in (dynamic) LDS, and every block of a launch is given the same amount; with
// a long list the blocks are large, so that the LDS of a gather block is spread over 16 row-gathering waves and
// does not limit how many of them a CU holds, and so that fewer blocks load the list.
constexpr int RANK_LONG_LIST = 6144;  // keys from which on the 1024-thread blocks are used (measured: lists of 2,200 and 4,096 keys are 4-5 us faster with the small brute-force blocks)
template <int THREADS> struct RankShape {
    static constexpr int R = THREADS == 256 ? 1 : 2;     // keys ranked by one 32-thread group
    static constexpr int ITEMS = (THREADS / 32) * R;     // keys ranked per block
    static constexpr int LOADS = 4096 / THREADS;         // key loads in flight per thread
};

// Orders a key list by brute-force ranking: rank(i) = #{j : key_j < key_i} + #{j < i : key_j == key_i}.  The lists
// are a few thousand keys, so the n^2 comparisons, spread over n/8 (n/64) blocks that run beside the gather blocks of
// the same launch, cost less than one pass of a single-workgroup sort, need no other kernel and no other stream,
// and give exactly the order a stable sort by id would (equal ids in position order).  Every block holds the whole
// list in LDS.  A group of 32 threads ranks RANK_R consecutive keys: each thread scans every 32nd 16-byte chunk of
// the list and compares it with all RANK_R keys, so a chunk read from LDS serves 4 * RANK_R comparisons.  The tie
// rule costs nothing away from the group's own keys: for entries before them "key_j <= key_i" counts, i.e.
// key_j < key_i + 1, for entries after them key_j < key_i, so the scan is three loops over one comparison each.
template <int THREADS>
__device__ __forceinline__ void rank_block(const KeyList& l, int blk, uint32_t* keys) {
    constexpr int RANK_R = RankShape<THREADS>::R, RANK_ITEMS = RankShape<THREADS>::ITEMS;
    constexpr int RANK_LOADS = RankShape<THREADS>::LOADS, GATHER_THREADS = THREADS;
    const int tid = threadIdx.x, n = l.n;
    const int n4 = (n + 3) & ~3;  // the tail is padded with 0xffffffff, which is larger than any id
    // independent loads are issued before the first is used: one round of memory latency per 4096 keys
    const KeySources ks = key_sources(l);
    for (int base = 0; base < n4; base += RANK_LOADS * GATHER_THREADS) {
        int64_t raw[RANK_LOADS];
#pragma unroll
        for (int u = 0; u < RANK_LOADS; ++u) {
            const int i = base + u * GATHER_THREADS + tid;
            raw[u] = *key_address(l, ks, i < n ? i : 0);  // unconditional: all loads go out together
        }
#pragma unroll
        for (int u = 0; u < RANK_LOADS; ++u) {
            const int i = base + u * GATHER_THREADS + tid;
            if (i < n4) keys[i] = i < n ? clamp_key(l, raw[u]) : 0xffffffffu;
        }
    }
    __syncthreads();
    const int it0 = blk * RANK_ITEMS + (tid >> 5) * RANK_R, t = tid & 31;
    if (it0 >= n) return;
    uint32_t ki[RANK_R];
    int cnt[RANK_R];
#pragma unroll
    for (int r = 0; r < RANK_R; ++r) {
        ki[r] = keys[it0 + r < n4 ? it0 + r : n4 - 1];  // ids are below 2^31, so ki + 1 does not wrap for real keys
        cnt[r] = 0;
    }
    int j = 4 * t;
    // entries wholly before the group's keys: key_j <= key_i
#pragma unroll 2
    for (; j + 3 < it0; j += 128) {
        const uint4 kj = *reinterpret_cast<const uint4*>(keys + j);
#pragma unroll
        for (int r = 0; r < RANK_R; ++r) {
            const uint32_t thr = ki[r] + 1u;
            cnt[r] += (kj.x < thr) + (kj.y < thr) + (kj.z < thr) + (kj.w < thr);
        }
    }
    // the chunk(s) that hold the group's own keys: the full rule
    for (; j < it0 + RANK_R && j < n4; j += 128) {
        const uint4 kj = *reinterpret_cast<const uint4*>(keys + j);
        const uint32_t kv[4] = {kj.x, kj.y, kj.z, kj.w};
#pragma unroll
        for (int r = 0; r < RANK_R; ++r) {
#pragma unroll
            for (int e = 0; e < 4; ++e) cnt[r] += (kv[e] < ki[r] || (kv[e] == ki[r] && j + e < it0 + r)) ? 1 : 0;
        }
    }
    // entries after them: key_j < key_i
#pragma unroll 2
    for (; j < n4; j += 128) {
        const uint4 kj = *reinterpret_cast<const uint4*>(keys + j);
#pragma unroll
        for (int r = 0; r < RANK_R; ++r) cnt[r] += (kj.x < ki[r]) + (kj.y < ki[r]) + (kj.z < ki[r]) + (kj.w < ki[r]);
    }
#pragma unroll
    for (int r = 0; r < RANK_R; ++r) {
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) cnt[r] += __shfl_xor(cnt[r], o, 32);
        if (t == 0 && it0 + r < n) {
            l.key[0][cnt[r]] = ki[r];
            l.pos[0][cnt[r]] = (uint32_t)(it0 + r);
        }
    }
}

// Long lists (RANK_LONG_LIST keys and more): brute force would compare every key with every other (1.5e8 comparisons
// for 12,288 keys, which set the duration of the whole launch).  Here a block of 1024 threads ranks 1024 keys with
// work linear in the list.  The id range [0, n_ids) is cut into RANK_BUCKETS equal slices, so buckets are ordered
// like the ids they hold.  Every block (1) counts the keys per bucket with LDS atomics, (2) turns the counts into
// offsets, (3) drops one word per key into its bucket's stretch of LDS, in whatever order the atomics hand out:
// (id - first id of the bucket) << 14 | position, so that the words of a bucket compare like (id, position) pairs,
// and (4) ranks its own 1024 keys: offset of the key's bucket + the number of smaller words in that bucket.  The
// result does not depend on the order inside the buckets.  Needs positions below 2^14 (lists end at 14,336 keys) and
// buckets narrower than 2^18 ids (tables of up to 134 M rows; larger ones keep the brute-force blocks).
constexpr int RANK_BUCKETS = 512;
constexpr int RANK_POS_BITS = 14;
__host__ __device__ constexpr size_t bucketed_lds_words(int n) { return (size_t)n + 3 * RANK_BUCKETS + 16; }
inline bool bucketed_ranking_fits(int64_t n_ids) { return n_ids / RANK_BUCKETS + 2 < (1 << (32 - RANK_POS_BITS)); }

__device__ __forceinline__ void rank_block_bucketed(const KeyList& l, int blk, uint64_t bucket_mul, uint32_t* lds) {
    constexpr int T = 1024, MAXK = KGE_RANK_MAX_KEYS / T;  // keys per thread: position u * T + tid
    const int tid = threadIdx.x, n = l.n;
    uint32_t* word = lds;                               // [n] one word per key, bucket after bucket
    int* cnt = reinterpret_cast<int*>(lds + n);         // [RANK_BUCKETS]
    int* off = cnt + RANK_BUCKETS;                      // [RANK_BUCKETS] exclusive prefix of cnt
    uint32_t* first = reinterpret_cast<uint32_t*>(off + RANK_BUCKETS);  // [RANK_BUCKETS] smallest id of the bucket
    int* wave_tot = reinterpret_cast<int*>(first + RANK_BUCKETS);       // [8]
    if (tid < RANK_BUCKETS) {
        cnt[tid] = 0;
        // bucket(id) = (id * bucket_mul) >> 32 >= tid  <=>  id >= ceil((tid << 32) / bucket_mul)
        first[tid] = (uint32_t)((((uint64_t)tid << 32) + bucket_mul - 1) / bucket_mul);
    }
    const KeySources ks = key_sources(l);
    int64_t raw[MAXK];
#pragma unroll
    for (int u = 0; u < MAXK; ++u) {
        const int p = u * T + tid;
        raw[u] = *key_address(l, ks, p < n ? p : 0);
    }
    __syncthreads();
    uint32_t key[MAXK];
    int bucket[MAXK], slot[MAXK];
#pragma unroll
    for (int u = 0; u < MAXK; ++u) {
        key[u] = clamp_key(l, raw[u]);
        bucket[u] = (int)(((uint64_t)key[u] * bucket_mul) >> 32);
        slot[u] = u * T + tid < n ? atomicAdd(&cnt[bucket[u]], 1) : 0;
    }
    __syncthreads();
    if (tid < RANK_BUCKETS) {  // exclusive prefix over the bucket counts: scan inside the 8 waves, then across them
        const int c = cnt[tid];
        int inc = c;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int v = __shfl_up(inc, o, 64);
            if ((tid & 63) >= o) inc += v;
        }
        if ((tid & 63) == 63) wave_tot[tid >> 6] = inc;
        off[tid] = inc - c;
    }
    __syncthreads();
    if (tid < RANK_BUCKETS) {
        int before = 0;
        for (int w = 0; w < (tid >> 6); ++w) before += wave_tot[w];
        off[tid] += before;
    }
    __syncthreads();
    uint32_t mine_word = 0;
    int mine_bucket = 0;
#pragma unroll
    for (int u = 0; u < MAXK; ++u) {
        const uint32_t wd = ((key[u] - first[bucket[u]]) << RANK_POS_BITS) | (uint32_t)(u * T + tid);
        if (u * T + tid < n) word[off[bucket[u]] + slot[u]] = wd;
        if (u == blk) { mine_word = wd; mine_bucket = bucket[u]; }  // this block ranks positions blk * T + tid
    }
    __syncthreads();
    const int mine = blk * T + tid;
    if (mine >= n) return;
    const int lo = off[mine_bucket], hi = lo + cnt[mine_bucket];
    int before = lo;
    // a bucket holds 24 words on average, the bucket of a hub entity hundreds, and the wave waits for its longest
    // scan: four words per LDS read once the position is a multiple of four
    int j = lo;
    for (; j < hi && (j & 3) != 0; ++j) before += word[j] < mine_word ? 1 : 0;
#pragma unroll 4
    for (; j + 3 < hi; j += 4) {
        const uint4 w4 = *reinterpret_cast<const uint4*>(word + j);
        before += (w4.x < mine_word) + (w4.y < mine_word) + (w4.z < mine_word) + (w4.w < mine_word);
    }
    for (; j < hi; ++j) before += word[j] < mine_word ? 1 : 0;
    l.key[0][before] = (mine_word >> RANK_POS_BITS) + first[mine_bucket];
    l.pos[0][before] = (uint32_t)mine;
}

// four floats -> four bf16 (round to nearest even), stored as 8 bytes
__device__ __forceinline__ void st4_bf16(uint16_t* p, float x0, float x1, float x2, float x3) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 a, b;
    a[0] = (__bf16)x0; a[1] = (__bf16)x1; b[0] = (__bf16)x2; b[1] = (__bf16)x3;
    *reinterpret_cast<uint2*>(p) = make_uint2(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b));
}

// NV = 16-byte vectors per lane: ceil(D/4/64) for the real models, ceil(D/8/64) (re, im) pairs for the complex ones.
// One row by one wave: a positive (rows 0 .. b - 1) or a corrupting row (behind them).
template <int MODEL, int NV>
__device__ __forceinline__ void gather_row(const GatherArgs& a, int row) {
    const int lane = threadIdx.x & 63;
#include "k_gather_row_body.h"
}

inline void kge_fill_gather_args(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int gsz, float gamma,
                                 float* pos_out, GatherArgs* out) {
    GatherArgs a = {};
    const int b = ids.b, n_neg = ids.n_neg;
    a.E = E; a.R = R; a.ids = ids;
    a.b = b; a.n_neg = n_neg; a.D = c->cfg.ent_dim; a.Dr = c->cfg.rel_dim;
    a.bf16 = c->cfg.gemm_input;
    a.gamma = gamma; a.n_ent = c->cfg.num_entities; a.n_rel = c->cfg.num_relations;
    a.Obf = c->Obf; a.Nbf = c->Nbf; a.ld_bf = c->ld_bf;
    a.O = c->O; a.Nst = c->Nst; a.fpos = c->fpos; a.pos_out = pos_out; a.o_n2 = c->o_n2; a.n_n2 = c->n_n2;
    a.cpos = c->cpos; a.inv_dpos = c->inv_dpos; a.row_loss = c->row_loss; a.rank_out = c->rank_out;
    a.item_blocks = c->cfg.model == KGE_TRANSR ? b / gsz : 0;
    a.g = gsz; a.max_pblocks = transr_max_pblocks(gsz, a.n_rel); a.items = c->tr_groups;
    *out = a;
}

}  // namespace
