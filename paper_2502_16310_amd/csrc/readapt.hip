// Re-adaptation bookkeeping for a moving body.  The paper refines once,
// before the solver, and names moving geometry as the case where the cost of
// rebuilding the bins every step decides the bin density (Results
// discussion); refinement and coarsening of the blocks themselves come from
// the forest-of-octrees scheme it builds on (Sec. II-C-1).  Here a step of a
// moving body is: import the moved faces, bin them, refine from the roots (the
// re-adapted forest is the near-wall forest of the new geometry), then relate
// the new forest to the previous one level by level, which is what a solver
// needs to carry its data over: per new block its index in the old level (or
// none) and whether it was kept, created, refined (a leaf that gained
// children) or coarsened (children removed); per old block whether it was
// removed.
//
// Both key lists of a level are sorted, so every lookup is a binary search;
// the 64 lanes of a wave look up 64 consecutive keys, whose search paths
// share their upper levels in the cache.  Counts per level and state are
// reduced per workgroup and added once per workgroup.
#include <algorithm>
#include <cstring>

#include "agal_internal.hpp"
#include "device.hpp"

struct agal_forest_diff_t {
    agal_context ctx = nullptr;
    hipStream_t stream = nullptr;
    int L = 0;
    int64_t n_new[agal::kMaxLevels + 1] = {};
    int64_t n_old[agal::kMaxLevels + 1] = {};
    void *base = nullptr;   // owns the arrays below
    int32_t *old_index[agal::kMaxLevels + 1] = {};
    uint8_t *state[agal::kMaxLevels + 1] = {};
    uint8_t *removed[agal::kMaxLevels + 1] = {};
    unsigned long long counts[agal::kMaxLevels + 1][4] = {};   // created, refined, coarsened, removed
};

namespace agal {
namespace {

constexpr int kDiffThreads = 256;

__device__ __forceinline__ int64_t find_key(const uint32_t *keys, int64_t n, uint32_t k) {
    int64_t lo = 0, hi = n - 1;
    while (lo <= hi) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        const uint32_t v = keys[mid];
        if (v == k) return mid;
        if (v < k) lo = mid + 1;
        else hi = mid - 1;
    }
    return -1;
}

// One level's new blocks (old index, state; created / refined / coarsened
// counts) and old blocks (removed flag and count).
struct DiffLevel {
    const uint32_t *nkeys, *okeys;
    const uint8_t *nleaf, *oleaf;
    int64_t nn, no;
    int32_t *old_index;
    uint8_t *state, *removed;
};
struct DiffArgs {
    DiffLevel lev[kMaxLevels + 1];
    uint32_t wg0[2 * (kMaxLevels + 1) + 1];   // first workgroup: level l's new blocks at 2 l, its old ones at 2 l + 1
    unsigned long long *counts;   // four per level, zeroed
};

// Every level in one launch: a level is one chain of dependent loads per thread
// (a binary search), 5 to 9 us whatever its size, and eight launches ran one
// after the other.  Four levels of a moving body, both ways: 58 us, together 19.
__global__ __launch_bounds__(kDiffThreads) void k_diff(DiffArgs A) {
    __shared__ uint32_t s_acc[3];
    int seg = 0;
    while (blockIdx.x >= A.wg0[seg + 1]) ++seg;
    const DiffLevel &V = A.lev[seg >> 1];
    const int64_t first = (int64_t)(blockIdx.x - A.wg0[seg]) * kDiffThreads + threadIdx.x;
    const int64_t stride = (int64_t)(A.wg0[seg + 1] - A.wg0[seg]) * kDiffThreads;
    uint32_t c[3] = {0u, 0u, 0u};
    if (seg & 1) {
        for (int64_t j = first; j < V.no; j += stride) {
            const bool gone = find_key(V.nkeys, V.nn, V.okeys[j]) < 0;
            V.removed[j] = gone ? 1 : 0;
            c[0] += gone ? 1u : 0u;
        }
    } else {
        for (int64_t i = first; i < V.nn; i += stride) {
            const int64_t j = find_key(V.okeys, V.no, V.nkeys[i]);
            uint8_t st = 0;
            if (j < 0) st = 1;
            else if (V.oleaf[j] && !V.nleaf[i]) st = 2;
            else if (!V.oleaf[j] && V.nleaf[i]) st = 3;
            V.old_index[i] = (int32_t)j;
            V.state[i] = st;
#pragma unroll
            for (int k = 0; k < 3; ++k) c[k] += st == k + 1 ? 1u : 0u;
        }
    }
    if (threadIdx.x < 3) s_acc[threadIdx.x] = 0u;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        // wave sums by shuffles, one LDS atomic per wave
        uint32_t v = c[k];
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, dev::kWave);
        if (dev::lane_id() == 0 && v) atomicAdd(&s_acc[k], v);
    }
    __syncthreads();
    if (threadIdx.x < 3 && s_acc[threadIdx.x])
        atomicAdd(&A.counts[4 * (seg >> 1) + ((seg & 1) ? 3 : threadIdx.x)], (unsigned long long)s_acc[threadIdx.x]);
}

bool same_grid(agal_forest a, agal_forest b) {
    if (a->dim != b->dim || a->L != b->L) return false;
    for (int k = 0; k < 3; ++k)
        if (a->roots[k] != b->roots[k] || std::memcmp(&a->lo[k], &b->lo[k], 4) || std::memcmp(&a->hi[k], &b->hi[k], 4))
            return false;
    return true;
}

}  // namespace
}  // namespace agal

using namespace agal;

extern "C" {

agal_status agal_forest_diff_create(agal_forest old_f, agal_forest new_f, void *stream, agal_forest_diff *out) {
    if (!old_f || !new_f || !out) return fail(AGAL_EINVAL, "agal_forest_diff_create: NULL argument");
    if (!same_grid(old_f, new_f))
        return fail(AGAL_EINVAL, "agal_forest_diff_create: forests over different root grids, domains or level counts");
    hipStream_t s = (hipStream_t)stream;
    agal_context ctx = new_f->ctx;
    auto *d = new agal_forest_diff_t;
    d->ctx = ctx;
    d->stream = s;
    d->L = new_f->L;
    unsigned long long *counts = nullptr;
    const int nl = d->L + 1;
    Slab arrays;
    arrays.add(&counts, (size_t)nl * 4);
    for (int l = 0; l < nl; ++l) {
        arrays.add(&d->old_index[l], (size_t)new_f->lev[l].n);
        arrays.add(&d->state[l], (size_t)new_f->lev[l].n);
        arrays.add(&d->removed[l], (size_t)old_f->lev[l].n);
    }
    agal_status st = arrays.get(ctx->mem, &d->base, s);
    if (st != AGAL_OK) {
        delete d;
        return st;
    }
    fill_u64(reinterpret_cast<uint64_t *>(counts), 0ull, (int64_t)nl * 4, s);
    {
        ProfScope prof(ctx, "forest_diff", s);
        DiffArgs D{};
        D.counts = counts;
        for (int l = 0; l < nl; ++l) {
            const Level &A = old_f->lev[l], &B = new_f->lev[l];
            d->n_new[l] = B.n;
            d->n_old[l] = A.n;
            D.lev[l] = {B.keys, A.keys, B.leaf, A.leaf, B.n, A.n, d->old_index[l], d->state[l], d->removed[l]};
            auto wgs = [](int64_t n) { return (uint32_t)std::min<int64_t>((n + kDiffThreads - 1) / kDiffThreads, 2048); };
            D.wg0[2 * l + 1] = D.wg0[2 * l] + wgs(B.n);
            D.wg0[2 * l + 2] = D.wg0[2 * l + 1] + wgs(A.n);
        }
        if (D.wg0[2 * nl])
            hipLaunchKernelGGL(k_diff, dim3(D.wg0[2 * nl]), dim3(kDiffThreads), 0, s, D);
    }
    if (st == AGAL_OK) {
        const hipError_t e1 = hipGetLastError();
        const hipError_t e2 = e1 == hipSuccess ? hipMemcpyAsync(d->counts, counts, (size_t)nl * 4 * 8,
                                                                hipMemcpyDeviceToHost, s)
                                               : e1;
        const hipError_t e3 = e2 == hipSuccess ? hipStreamSynchronize(s) : e2;
        if (e3 != hipSuccess) st = fail(AGAL_EHIP, "agal_forest_diff_create: %s", hipGetErrorString(e3));
    }
    if (st != AGAL_OK) {
        agal_destroy_forest_diff(d);
        return st;
    }
    *out = d;
    return AGAL_OK;
}

agal_status agal_forest_diff_view(agal_forest_diff d, int level, const int32_t **d_old_index, const uint8_t **d_state,
                                  const uint8_t **d_removed, int64_t *n_new, int64_t *n_old, int64_t counts[4]) {
    if (!d) return fail(AGAL_EINVAL, "agal_forest_diff_view: NULL diff");
    if (level < 0 || level > d->L) return fail(AGAL_EINVAL, "agal_forest_diff_view: level %d outside [0, %d]", level, d->L);
    if (d_old_index) *d_old_index = d->old_index[level];
    if (d_state) *d_state = d->state[level];
    if (d_removed) *d_removed = d->removed[level];
    if (n_new) *n_new = d->n_new[level];
    if (n_old) *n_old = d->n_old[level];
    if (counts)
        for (int k = 0; k < 4; ++k) counts[k] = (int64_t)d->counts[level][k];
    return AGAL_OK;
}

void agal_destroy_forest_diff(agal_forest_diff d) {
    if (!d) return;
    dev_free(d->ctx->mem, d->base, d->stream);
    delete d;
}

}  // extern "C"
