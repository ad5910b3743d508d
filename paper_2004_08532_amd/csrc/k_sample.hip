// Step 1 of the mini-batch loop (paper Sec. 3.1) on the device: positive triples and the jointly sampled
// corrupting entities of Sec. 3.3, for any range of steps at once, as id arrays that kge_train_steps consumes.
//
// Every id is a function of (seed, stream tag, step, chunk, slot) alone:
//     key = mix(mix(mix(mix(seed + GOLDEN * tag) + step) + a) + j),   id = floor(key * n / 2^64)
// with `mix` a 64-bit xor-shift / multiply finaliser, so any step can be generated without the ones before it and
// one launch fills thousands of steps.  Streams (tags):
//   1  positives: position j of the mini-batch = triple number floor(key * n_triples / 2^64) of the triple list
//   2  uniform corrupting entities: slot j of chunk a = entity floor(key * num_entities / 2^64)
//   3  degree-proportional corrupting entities (Sec. 3.3): slot j of chunk a = the tail (head, when heads are
//      corrupted) of position floor(key * b / 2^64) of the SAME mini-batch; entities are then drawn in proportion
//      to how often they occur in the batch
// Of the k slots of a chunk the first n_degree use stream 3, the others stream 2.
#include "kge_common.h"

namespace {

constexpr uint64_t GOLDEN = 0x9E3779B97F4A7C15ull;

__host__ __device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// floor(key * n / 2^64)
__device__ __forceinline__ int64_t scale_to(uint64_t key, uint64_t n) { return (int64_t)__umul64hi(key, n); }

struct SampleArgs {
    kge_sampler s;
    uint64_t base[4];  // mix(seed + GOLDEN * tag) per tag, formed on the host
    int64_t first_step, n_steps;
    int waves_per_step;  // waves of 64 consecutive items (positives, then corrupting slots) that one step takes
    int64_t* h;
    int64_t* r;
    int64_t* t;
    int64_t* neg;
    int32_t* sides;
};

__device__ __forceinline__ int side_of(int mode, int64_t step) { return mode == 2 ? (int)(step & 1) : mode; }

// A wave owns 64 consecutive items of one step, so the step, its side and the first rounds of the key chain are the
// same in all lanes, and no lane divides by the items per step (one 64-bit division per id took longer than the
// rest).  Bound by the random 24-byte reads of the triple list (a list of millions of triples lies in the Infinity
// Cache, and every read pulls a whole line): a triple is read with two requests (16 + 8 bytes) instead of three, and
// the ids are stored past the caches so that the list keeps them (2 % faster).  1000 steps of 3,200 ids from a list of
// 1 M triples: 30.8 -> 23.1 us, about 146 MB of list lines at 6.3 TB/s.
__global__ __launch_bounds__(256) void k_sample(SampleArgs a) {
    typedef long long i64x2 __attribute__((ext_vector_type(2), aligned(8)));
    const int b = a.s.batch, k = a.s.neg_per_chunk, n_neg = a.s.n_chunks * k, lane = threadIdx.x & 63;
    const float inv_k = 1.f / (float)(k > 0 ? k : 1);
    const int64_t waves = a.n_steps * a.waves_per_step, stride = (int64_t)gridDim.x * 4;
    for (int64_t w = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); w < waves; w += stride) {
        const int64_t si = w >> 32 ? w / a.waves_per_step : (int64_t)((uint32_t)w / (uint32_t)a.waves_per_step);
        const int64_t item = (w - si * a.waves_per_step) * 64 + lane;
        const int64_t step = a.first_step + si;
        const int side = side_of(a.s.side_mode, step);
        const uint64_t zpos = mix64(mix64(a.base[1] + (uint64_t)step));  // positives use a = 0
        if (item < b) {
            const int64_t p = scale_to(mix64(zpos + (uint64_t)item), (uint64_t)a.s.n_triples);
            const i64x2 hr = *reinterpret_cast<const i64x2*>(a.s.triples + 3 * p);
            const int64_t t = a.s.triples[3 * p + 2];
            __builtin_nontemporal_store(hr.x, (long long*)a.h + si * b + item);
            __builtin_nontemporal_store(hr.y, (long long*)a.r + si * b + item);
            __builtin_nontemporal_store(t, a.t + si * b + item);
            if (item == 0 && a.sides) a.sides[si] = side;
        } else if (item - b < n_neg) {
            const uint32_t q = (uint32_t)(item - b);
            uint32_t c = (uint32_t)((float)q * inv_k);  // q / k: the float quotient is off by a few at most
            while (c * (uint32_t)k > q) --c;
            while (q - c * (uint32_t)k >= (uint32_t)k) ++c;
            const uint32_t j = q - c * (uint32_t)k;
            int64_t id;
            if ((int)j < a.s.n_degree) {
                const uint64_t key = mix64(mix64(mix64(a.base[3] + (uint64_t)step) + (uint64_t)c) + (uint64_t)j);
                const int64_t pick = scale_to(key, (uint64_t)b);
                const int64_t p = scale_to(mix64(zpos + (uint64_t)pick), (uint64_t)a.s.n_triples);
                id = a.s.triples[3 * p + (side == KGE_NEG_HEAD ? 0 : 2)];
            } else {
                const uint64_t key = mix64(mix64(mix64(a.base[2] + (uint64_t)step) + (uint64_t)c) + (uint64_t)j);
                id = scale_to(key, (uint64_t)a.s.num_entities);
            }
            __builtin_nontemporal_store(id, a.neg + si * (int64_t)n_neg + q);
        }
    }
}

}  // namespace

int kge_sample_launch(const kge_sampler* s, int64_t first_step, int64_t n_steps, int64_t* h, int64_t* r, int64_t* t,
                      int64_t* neg, int32_t* sides, hipStream_t st) {
    SampleArgs a;
    a.s = *s;
    for (int tag = 0; tag < 4; ++tag) a.base[tag] = mix64(s->seed + GOLDEN * (uint64_t)tag);
    a.first_step = first_step; a.n_steps = n_steps;
    a.h = h; a.r = r; a.t = t; a.neg = neg; a.sides = sides;
    const int64_t per_step = (int64_t)s->batch + (int64_t)s->n_chunks * s->neg_per_chunk;
    a.waves_per_step = (int)((per_step + 63) / 64);
    int64_t blocks = (n_steps * a.waves_per_step + 3) / 4;
    if (blocks > 65536) blocks = 65536;
    hipLaunchKernelGGL(k_sample, dim3((unsigned)blocks), dim3(256), 0, st, a);
    return hipGetLastError() == hipSuccess ? KGE_OK : KGE_ERR_DEVICE;
}
