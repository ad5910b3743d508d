// Row gather with fused positive forward (paper Sec. 3.1 step 2 and the first half of step 3).
//
// One wavefront per row.  A wave reads the rows it needs with 16-byte loads (a 1600-byte row is 100 such
// loads, lanes 0..63 then 0..35, so every request is a run of whole cache lines), forms
//     o_i = phi(a_i, r_i)   (Sec. 3.3: o = h + r for TransE; a*r, a*conj(r), rotations for the other models)
// scores the positive pair psi(o_i, c_i) (Table 1) with a shuffle reduction, and writes o_i once into the
// dense staging array that the chunked negative scoring reads.  Waves past the positives copy the k
// corrupting rows of every chunk into staging (the O(bkd/g) rows of Sec. 3.3) and compute |n|^2 for TransE-L2.
// In a training step the same launch carries extra blocks that bring the step's key lists into (id, position)
// order for the duplicate reduction (rank_block in k_gather_rows.h): that work needs only the ids, so it rides along here.
#include "k_gather_rows.h"

namespace {

template <int MODEL, int NV, int THREADS>
__global__ __launch_bounds__(THREADS) void k_gather(GatherArgs a) {
    constexpr int ROWS_PER_BLOCK = THREADS / 64;
    extern __shared__ __attribute__((aligned(16))) uint32_t rank_keys[];  // (read 16 bytes at a time)
    int block = blockIdx.x;
    if constexpr (MODEL == KGE_TRANSR) {
        if (block < a.item_blocks) {
            transr_items<THREADS>(a.items, step_view(a.ids).r + (int64_t)block * a.g, block, a.g, a.n_rel, a.max_pblocks);
            return;
        }
        block -= a.item_blocks;
    }
    // the rank blocks come first: they run longest and need nothing but the ids
    if (block < a.rank_blocks) {
        const int rb = block;
        if (rb < a.ent_rank_blocks) {
            if (THREADS == 1024 && a.bucket_mul != 0) rank_block_bucketed(a.ent, rb, a.bucket_mul, rank_keys);
            else rank_block<THREADS>(a.ent, rb, rank_keys);
        } else {
            rank_block<THREADS>(a.rel, rb - a.ent_rank_blocks, rank_keys);
        }
        return;
    }
    gather_row<MODEL, NV>(a, (block - a.rank_blocks) * ROWS_PER_BLOCK + (threadIdx.x >> 6));
}

template <int MODEL, int THREADS>
void launch_nv(kge_ctx* c, const GatherArgs& a, int nv, dim3 grid, size_t lds, hipStream_t st) {
    switch (nv) {
    case 1: KGE_LAUNCH(c, (k_gather<MODEL, 1, THREADS>), grid, dim3(THREADS), lds, st, a); break;
    case 2: KGE_LAUNCH(c, (k_gather<MODEL, 2, THREADS>), grid, dim3(THREADS), lds, st, a); break;
    case 3: KGE_LAUNCH(c, (k_gather<MODEL, 3, THREADS>), grid, dim3(THREADS), lds, st, a); break;
    default: KGE_LAUNCH(c, (k_gather<MODEL, 4, THREADS>), grid, dim3(THREADS), lds, st, a); break;
    }
}

template <int THREADS>
void launch_model(kge_ctx* c, GatherArgs& a, int nv, int rows, bool with_keys, const StepIds& ids, hipStream_t st) {
    const int gather_blocks = (rows + THREADS / 64 - 1) / (THREADS / 64);
    a.ent_rank_blocks = 0;
    int rank_blocks = 0;
    size_t lds = 0;
    if (with_keys) {
        constexpr int ITEMS = RankShape<THREADS>::ITEMS;
        kge_make_key_lists(c, ids, &a.ent, &a.rel);
        a.bucket_mul = 0;
        if (THREADS == 1024 && bucketed_ranking_fits(a.ent.n_ids)) {  // long entity list: 1024 keys per block
            a.ent_rank_blocks = (a.ent.n + 1023) / 1024;
            a.bucket_mul = ((uint64_t)RANK_BUCKETS << 32) / (uint64_t)a.ent.n_ids;
            lds = sizeof(uint32_t) * bucketed_lds_words(a.ent.n);
            const size_t rel_lds = sizeof(uint32_t) * (size_t)((a.rel.n + 3) & ~3);
            if (rel_lds > lds) lds = rel_lds;
        } else {
            a.ent_rank_blocks = (a.ent.n + ITEMS - 1) / ITEMS;
            lds = sizeof(uint32_t) * (size_t)((a.ent.n + 3) & ~3);  // the entity list is the longer one
        }
        rank_blocks = a.ent_rank_blocks + (a.rel.n + ITEMS - 1) / ITEMS;
        c->ebuf = 0;
        c->rbuf = 0;
    }
    a.rank_blocks = rank_blocks;
    const dim3 grid(gather_blocks + rank_blocks + a.item_blocks);
    switch (c->cfg.model) {
    case KGE_TRANSE_L2: launch_nv<KGE_TRANSE_L2, THREADS>(c, a, nv, grid, lds, st); break;
    case KGE_TRANSE_L1: launch_nv<KGE_TRANSE_L1, THREADS>(c, a, nv, grid, lds, st); break;
    case KGE_DISTMULT: launch_nv<KGE_DISTMULT, THREADS>(c, a, nv, grid, lds, st); break;
    case KGE_COMPLEX: launch_nv<KGE_COMPLEX, THREADS>(c, a, nv, grid, lds, st); break;
    case KGE_RESCAL: launch_nv<KGE_RESCAL, THREADS>(c, a, nv, grid, lds, st); break;
    case KGE_TRANSR: launch_nv<KGE_TRANSR, THREADS>(c, a, nv, grid, lds, st); break;
    default: launch_nv<KGE_ROTATE, THREADS>(c, a, nv, grid, lds, st); break;
    }
}

}  // namespace

void kge_launch_gather(kge_ctx* c, const float* E, const float* R, const StepIds& ids, int gsz, float gamma, float* pos_out,
                       bool with_keys, hipStream_t st) {
    GatherArgs a;
    kge_fill_gather_args(c, E, R, ids, gsz, gamma, pos_out, &a);
    const int rows = ids.b + ids.n_neg, model = c->cfg.model;
    const bool cplx = model == KGE_COMPLEX || model == KGE_ROTATE;
    const int nvec = cplx ? a.D / 8 : a.D / 4;
    const int nv = (nvec + 63) / 64;
    if (with_keys && ids.b + rows >= RANK_LONG_LIST) launch_model<1024>(c, a, nv, rows, with_keys, ids, st);
    else launch_model<256>(c, a, nv, rows, with_keys, ids, st);
}

void kge_launch_key_order(kge_ctx* c, const StepIds& ids, hipStream_t st) {
    GatherArgs a = {};
    a.ids = ids;
    if (2 * ids.b + ids.n_neg >= RANK_LONG_LIST) launch_model<1024>(c, a, 1, 0, true, ids, st);
    else launch_model<256>(c, a, 1, 0, true, ids, st);
}
