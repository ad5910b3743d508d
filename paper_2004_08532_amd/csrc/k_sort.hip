// Duplicate reduction, part 1, for LONG key lists: sort the (row id, position) pairs of a mini-batch.
//
// A mini-batch touches few rows and may touch one row many times (paper Sec. 2); before the optimizer runs,
// all gradient rows of one embedding row have to be added up, so the key lists (2b + (b/g)k entity keys, b
// relation keys) are brought into (id, position) order.  Lists of up to KGE_RANK_MAX_KEYS keys are ordered by the
// rank blocks of the gather launch (k_gather.hip).  Longer lists are sorted here: least-significant-digit radix sort
// over only as many bits as the table's row count needs, ping-ponging through global memory.  A list is cut into slices
// of 2048 keys, one workgroup of 512 threads per slice, and inside a slice every wavefront owns 256 consecutive keys,
// all of them in flight at once.  A pass is two launches:
//   k_sort_count    keys per digit of every slice (LDS atomics)
//   k_sort_scatter  every wavefront ranks its keys inside the slice (equal digits of a 64-key round by ballots), the
//                   workgroup adds up what the earlier slices hold per digit and what all slices hold of the smaller
//                   digits, and the keys go to their places
// and a third one in between, k_sort_offsets, where there are too many slices for every workgroup to walk them.
// The sort is stable, so equal ids end up ordered by position.  Both lists go through the same launches (the entity
// slices first, then the relation slices); they run on their own stream beside the forward / backward kernels.
// The passes are chains of dependent steps, not bound by bytes: digits of up to 10 bits where the list has few slices
// (two passes for a million rows instead of three), 8 otherwise.  31,000 keys of 20 bits: 9 launches of 60 us together
// before (8-bit digits, a wave's rounds of loads one after the other, an offsets launch per pass), now 4.
// This file also holds the export of distinct ids and counts (test hook).
#include "kge_common.h"

namespace {

constexpr int SORT_THREADS = 512;
constexpr int SORT_WAVES = SORT_THREADS / 64;
constexpr int SORT_SLICE = KGE_SORT_SLICE;          // keys per workgroup
constexpr int WAVE_KEYS = SORT_SLICE / SORT_WAVES;  // consecutive keys per wavefront
constexpr int ROUNDS = WAVE_KEYS / 64;
constexpr int MAX_DIGITS = 1 << KGE_SORT_MAX_BITS;

struct SortArgs {
    KeyList list[2];       // entity keys, relation keys
    int slices[2];         // workgroups per list
    uint32_t* slice_tot[2];  // [slices][digits] per list: keys with the digit in the slice
    uint32_t* bases[2];    // with k_sort_offsets: [digits] number of keys with a smaller digit; slice_tot then holds the
                           // keys with the digit in the earlier slices
    int pass;
    // k_sort_offsets has walked the list's slices (8-bit digits).  Not bool: from a byte index that is the same in all lanes
    // the compiler formed a scalar load of bases[which] whose base was off by the index and whose offset made up for it; the
    // hardware drops the low two bits of each, so for list 1 it loaded a pointer from halves of two
    int offsets[2];
};

// the lanes of the wave that hold the same digit as this lane (valid lanes only)
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, bool valid, int bits) {
    uint64_t peers = __ballot(valid);
    for (int bit = 0; bit < bits; ++bit) {
        const bool one = (d >> bit) & 1u;
        const uint64_t bm = __ballot(valid && one);
        peers &= one ? bm : ~bm;
    }
    return peers;
}

// which list and slice this workgroup has
struct SortRange {
    int which, slice, begin, n;
};
__device__ __forceinline__ SortRange sort_range(const SortArgs& a) {
    SortRange r;
    r.which = (int)blockIdx.x >= a.slices[0] ? 1 : 0;
    r.slice = blockIdx.x - (r.which ? a.slices[0] : 0);
    r.n = a.list[r.which].n;
    r.begin = r.slice * SORT_SLICE + (threadIdx.x >> 6) * WAVE_KEYS + (threadIdx.x & 63);  // the lane's first key
    return r;
}

__device__ __forceinline__ bool sort_pass_runs(const SortArgs& a, int which) { return a.pass < a.list[which].passes; }

// the lane's keys of all rounds; every load goes out before the first is used
__device__ __forceinline__ void load_keys(const SortArgs& a, const KeyList& l, const SortRange& r, uint32_t (&key)[ROUNDS]) {
    if (a.pass == 0) {
        const KeySources ks = key_sources(l);
        int64_t raw[ROUNDS];
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u) raw[u] = *key_address(l, ks, r.begin + 64 * u < r.n ? r.begin + 64 * u : 0);
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u) key[u] = clamp_key(l, raw[u]);
    } else {
        const uint32_t* kin = l.key[(a.pass - 1) & 1];
#pragma unroll
        for (int u = 0; u < ROUNDS; ++u) key[u] = kin[r.begin + 64 * u < r.n ? r.begin + 64 * u : 0];
    }
}

__global__ __launch_bounds__(SORT_THREADS) void k_sort_count(SortArgs a) {
    __shared__ uint32_t hist[MAX_DIGITS];
    const SortRange r = sort_range(a);
    if (!sort_pass_runs(a, r.which)) return;  // (a list whose ids need fewer passes is already sorted)
    const KeyList& l = a.list[r.which];
    const int nd = 1 << l.digit_bits, shift = l.digit_bits * a.pass;
    uint32_t key[ROUNDS];
    load_keys(a, l, r, key);
    for (int d = threadIdx.x; d < nd; d += SORT_THREADS) hist[d] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u)
        if (r.begin + 64 * u < r.n) atomicAdd(&hist[(key[u] >> shift) & (nd - 1)], 1u);
    __syncthreads();
    uint32_t* out = a.slice_tot[r.which] + (int64_t)r.slice * nd;
    for (int d = threadIdx.x; d < nd; d += SORT_THREADS) out[d] = hist[d];
}

// exclusive prefix of v over the SORT_THREADS threads of the workgroup
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t* wave_tot) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
    }
    if (lane == 63) wave_tot[w] = incl;
    __syncthreads();
    uint32_t off = incl - v;
    for (int ww = 0; ww < w; ++ww) off += wave_tot[ww];
    return off;
}

// One workgroup per list, thread d = digit d (8-bit digits): the running sum over the slices of the digit's totals
// replaces the totals; the exclusive prefix over the digits' sums goes to bases.
__global__ __launch_bounds__(SORT_THREADS) void k_sort_offsets(SortArgs a) {
    __shared__ uint32_t wave_tot[SORT_WAVES];
    const int which = blockIdx.x;
    if (!sort_pass_runs(a, which) || !a.offsets[which]) return;
    const int d = threadIdx.x, nd = 1 << a.list[which].digit_bits;
    uint32_t* tot = a.slice_tot[which];
    const int slices = a.slices[which];
    uint32_t total = 0;
    if (d < nd) {
        for (int u0 = 0; u0 < slices; u0 += 16) {  // sixteen loads in flight
            uint32_t v[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) v[q] = tot[(int64_t)(u0 + q < slices ? u0 + q : u0) * nd + d];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                if (u0 + q < slices) {
                    tot[(int64_t)(u0 + q) * nd + d] = total;
                    total += v[q];
                }
            }
        }
    }
    const uint32_t base = block_prefix(total, wave_tot);
    if (d < nd) a.bases[which][d] = base;
}

__global__ __launch_bounds__(SORT_THREADS) void k_sort_scatter(SortArgs a) {
    __shared__ volatile uint16_t hist[SORT_WAVES][MAX_DIGITS];  // keys of the digit in the wave, then in the earlier waves
    __shared__ uint32_t start[MAX_DIGITS];                      // where the slice's keys of the digit go
    __shared__ uint32_t part[2][SORT_THREADS];
    __shared__ uint32_t wave_tot[SORT_WAVES];
    const SortRange r = sort_range(a);
    if (!sort_pass_runs(a, r.which)) return;
    const KeyList& l = a.list[r.which];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    const int nd = 1 << l.digit_bits, shift = l.digit_bits * a.pass;
    uint32_t key[ROUNDS], pos[ROUNDS];
    load_keys(a, l, r, key);
    const uint32_t* pin = a.pass == 0 ? nullptr : l.pos[(a.pass - 1) & 1];
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) pos[u] = a.pass == 0 ? (uint32_t)(r.begin + 64 * u) : pin[r.begin + 64 * u < r.n ? r.begin + 64 * u : 0];

    // per digit: keys in the earlier slices, keys in all slices
    const uint32_t* tot = a.slice_tot[r.which];
    if (a.offsets[r.which]) {
        for (int d = tid; d < nd; d += SORT_THREADS) start[d] = tot[(int64_t)r.slice * nd + d] + a.bases[r.which][d];
    } else {
        const int slices = a.slices[r.which];
        const int share = nd < SORT_THREADS ? SORT_THREADS / nd : 1;  // threads per digit
        for (int d0 = 0; d0 < nd; d0 += SORT_THREADS) {
            const int d = d0 + (nd < SORT_THREADS ? tid & (nd - 1) : tid), q0 = nd < SORT_THREADS ? tid / nd : 0;
            uint32_t before = 0, total = 0;
            for (int s0 = q0; s0 < slices; s0 += 16 * share) {
                uint32_t v[16];
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = tot[(int64_t)(s0 + q * share < slices ? s0 + q * share : s0) * nd + d];
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int s = s0 + q * share;
                    total += s < slices ? v[q] : 0u;
                    before += s < r.slice ? v[q] : 0u;
                }
            }
            if (share > 1) {
                part[0][tid] = before;
                part[1][tid] = total;
                __syncthreads();
                if (tid < nd) {
                    for (int q = 1; q < share; ++q) { before += part[0][tid + q * nd]; total += part[1][tid + q * nd]; }
                } else {
                    total = 0;
                }
            }
            const uint32_t carry = d0 == 0 ? 0u : part[1][0];  // keys of the digits before d0
            const uint32_t base = block_prefix(total, wave_tot) + carry;
            if (share == 1 || tid < nd) start[d] = base + before;
            __syncthreads();  // wave_tot and part are free again
            if (d0 + SORT_THREADS < nd && tid == SORT_THREADS - 1) part[1][0] = base + total;
            __syncthreads();
        }
    }
    for (int e = tid; e < SORT_WAVES * nd; e += SORT_THREADS) hist[e / nd][e & (nd - 1)] = 0;
    __syncthreads();
    uint32_t idx[ROUNDS];  // the key's place among the wave's keys of its digit
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
        const bool valid = r.begin + 64 * u < r.n;
        const uint32_t d = (key[u] >> shift) & (nd - 1);
        const uint64_t peers = digit_peers(d, valid, l.digit_bits);
        const uint32_t had = hist[w][d];
        idx[u] = had + (uint32_t)__popcll(peers & lt_mask);
        __builtin_amdgcn_wave_barrier();
        if (valid && (peers & lt_mask) == 0) hist[w][d] = (uint16_t)(had + (uint32_t)__popcll(peers));
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int d = tid; d < nd; d += SORT_THREADS) {
        uint32_t run = 0;
#pragma unroll
        for (int ww = 0; ww < SORT_WAVES; ++ww) {
            const uint32_t v = hist[ww][d];
            hist[ww][d] = (uint16_t)run;
            run += v;
        }
    }
    __syncthreads();
    uint32_t* kout = l.key[a.pass & 1];
    uint32_t* pout = l.pos[a.pass & 1];
#pragma unroll
    for (int u = 0; u < ROUNDS; ++u) {
        if (r.begin + 64 * u >= r.n) continue;
        const uint32_t d = (key[u] >> shift) & (nd - 1);
        const uint32_t dst = start[d] + hist[w][d] + idx[u];
        kout[dst] = key[u];
        pout[dst] = pos[u];
    }
}

// Test hook: distinct ids and their multiplicities from a sorted key list (one workgroup).
__global__ __launch_bounds__(1024) void k_dedup_export(const uint32_t* keys, int n, int64_t* uniq, int32_t* count,
                                                       int64_t* n_unique) {
    __shared__ uint32_t wave_cnt[16];
    __shared__ uint32_t running;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    if (tid == 0) running = 0;
    __syncthreads();
    for (int base = 0; base < n; base += 1024) {
        const int p = base + tid;
        const bool is_head = p < n && (p == 0 || keys[p - 1] != keys[p]);
        const uint64_t bal = __ballot(is_head);
        const uint32_t in_wave = (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) wave_cnt[w] = (uint32_t)__popcll(bal);
        __syncthreads();
        uint32_t off = running;
        for (int ww = 0; ww < w; ++ww) off += wave_cnt[ww];
        if (is_head) {
            const uint32_t key = keys[p];
            int q = p + 1;
            while (q < n && keys[q] == key) ++q;
            uniq[off + in_wave] = (int64_t)key;
            count[off + in_wave] = q - p;
        }
        __syncthreads();
        if (tid == 0) {
            uint32_t s = running;
            for (int ww = 0; ww < 16; ++ww) s += wave_cnt[ww];
            running = s;
        }
        __syncthreads();
    }
    if (tid == 0) *n_unique = (int64_t)running;
}

int bits_for(int64_t n_ids) {
    int bits = 1;
    while (bits < 32 && (((int64_t)1) << bits) < n_ids) ++bits;
    return bits;
}

// Digits of up to 10 bits while every workgroup of the scatter can walk the slices of all its digits cheaply (up to
// KGE_SORT_FEW_SLICES slices), 8 bits otherwise; the passes share the bits evenly.
void set_passes(KeyList& l) {
    const int bits = bits_for(l.n_ids), most = (l.n + SORT_SLICE - 1) / SORT_SLICE <= KGE_SORT_FEW_SLICES ? KGE_SORT_MAX_BITS : 8;
    l.passes = (bits + most - 1) / most;
    l.digit_bits = (bits + l.passes - 1) / l.passes;
}
static_assert(KGE_SORT_FEW_SLICES <= 160, "k_sort_offsets takes 8-bit digits");
constexpr int OFFSETS_SLICES = 160;  // from here on the slices are walked once per pass, by k_sort_offsets

}  // namespace

void kge_make_key_lists(kge_ctx* c, const StepIds& ids, KeyList* ent, KeyList* rel) {
    KeyList e = {}, rl = {};
    const int b = ids.b, n_neg = ids.n_neg;
    e.src[0] = ids.h; e.src[1] = ids.t; e.src[2] = ids.neg;
    e.n_src[0] = b; e.n_src[1] = b; e.n_src[2] = n_neg;
    e.blk = ids.blk; e.which = 0;
    e.n = 2 * b + n_neg;
    e.n_ids = c->cfg.num_entities;
    set_passes(e);
    e.key[0] = c->ekey[0]; e.key[1] = c->ekey[1]; e.pos[0] = c->epos[0]; e.pos[1] = c->epos[1];
    rl.src[0] = ids.r; rl.src[1] = ids.r; rl.src[2] = ids.r;
    rl.n_src[0] = b; rl.n_src[1] = 0; rl.n_src[2] = 0;
    rl.blk = ids.blk; rl.which = 1;
    rl.n = b;
    rl.n_ids = c->cfg.num_relations;
    set_passes(rl);
    rl.key[0] = c->rkey[0]; rl.key[1] = c->rkey[1]; rl.pos[0] = c->rpos[0]; rl.pos[1] = c->rpos[1];
    c->last_ent_keys = e.n;
    c->last_rel_keys = rl.n;
    *ent = e;
    *rel = rl;
}

// Radix sort of both key lists (lists too long for the rank path of the gather launch).
void kge_launch_sort(kge_ctx* c, const StepIds& ids, hipStream_t st) {
    SortArgs a;
    kge_make_key_lists(c, ids, &a.list[0], &a.list[1]);
    c->ebuf = (a.list[0].passes - 1) & 1;
    c->rbuf = (a.list[1].passes - 1) & 1;
    for (int w = 0; w < 2; ++w) a.slices[w] = (a.list[w].n + SORT_SLICE - 1) / SORT_SLICE;
    const size_t digits0 = (size_t)a.slices[0] << a.list[0].digit_bits, digits1 = (size_t)a.slices[1] << a.list[1].digit_bits;
    a.slice_tot[0] = c->sort_counts;
    a.slice_tot[1] = a.slice_tot[0] + digits0;
    a.bases[0] = a.slice_tot[1] + digits1;
    a.bases[1] = a.bases[0] + MAX_DIGITS;
    for (int w = 0; w < 2; ++w) a.offsets[w] = a.slices[w] > OFFSETS_SLICES;
    const int passes = a.list[0].passes > a.list[1].passes ? a.list[0].passes : a.list[1].passes;
    const dim3 grid(a.slices[0] + a.slices[1]);
    // while profiling: the first launch takes the scope's start timestamp, the last one its stop timestamp
    hipEvent_t ev0 = c->launch_ev0, ev1 = c->launch_ev1;
    c->launch_ev0 = nullptr;
    c->launch_ev1 = nullptr;
    for (a.pass = 0; a.pass < passes; ++a.pass) {
        if (a.pass == 0 && ev0) hipExtLaunchKernelGGL(k_sort_count, grid, dim3(SORT_THREADS), 0, st, ev0, nullptr, 0, a);
        else hipLaunchKernelGGL(k_sort_count, grid, dim3(SORT_THREADS), 0, st, a);
        if (a.offsets[0] || a.offsets[1]) hipLaunchKernelGGL(k_sort_offsets, dim3(2), dim3(SORT_THREADS), 0, st, a);
        if (a.pass == passes - 1 && ev1) hipExtLaunchKernelGGL(k_sort_scatter, grid, dim3(SORT_THREADS), 0, st, nullptr, ev1, 0, a);
        else hipLaunchKernelGGL(k_sort_scatter, grid, dim3(SORT_THREADS), 0, st, a);
    }
}

void kge_launch_dedup_export(kge_ctx* c, int which, int64_t* uniq, int32_t* count, int64_t* n_unique,
                             hipStream_t st) {
    const uint32_t* keys = which == 0 ? c->ekey[c->ebuf] : c->rkey[c->rbuf];
    const int n = (int)(which == 0 ? c->last_ent_keys : c->last_rel_keys);
    hipLaunchKernelGGL(k_dedup_export, dim3(1), dim3(1024), 0, st, keys, n, uniq, count, n_unique);
}
