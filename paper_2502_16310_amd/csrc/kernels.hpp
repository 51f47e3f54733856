// Per-item device code of every kernel of the path: one wave's blocks for the
// flag and link kernels, one thread's item for the balance and merge steps,
// one workgroup's node tile for the adjoint, one face / bin group for the
// binning.  The single-body kernels (refine.hip, links.hip, bins.hip) and the
// batched persistent kernels (batch.hip) are thin loops around these, so both
// forms compute bit-identical flags and link fractions.
#pragma once
#pragma clang fp contract(off)

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdint>

#include "device.hpp"

namespace agal {
namespace kern {

// ===========================================================================
// Import (paper Sec. II-B)
// ===========================================================================
// Face f: validate its indices, gather its corners into the structure-of-arrays
// coordinate list, the bounding-box rows and the per-face record, and copy
// its indices.  Returns error bits: 2 for an index outside [0, Nv) (the face
// is then written as zeros).
template <int D>
__device__ __forceinline__ uint32_t import_face(const float *verts, int64_t Nv, const int32_t *faces, int64_t F,
                                                float *coords, float *aabb, float *rec, int32_t *fidx, int64_t f,
                                                float *ext = nullptr) {
    float v[D][D];
    bool ok = true;
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const int64_t vi = faces ? (int64_t)faces[f * D + k] : f * D + k;
        ok = ok && vi >= 0 && vi < Nv;
        fidx[f * D + k] = (vi >= 0 && vi < Nv) ? (int32_t)vi : 0;
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        const int64_t vi = faces ? (int64_t)faces[f * D + k] : f * D + k;
#pragma unroll
        for (int a = 0; a < D; ++a) v[k][a] = ok ? verts[vi * D + a] : 0.0f;
    }
    float r[dev::kRecFloats<D>];
#pragma unroll
    for (int k = 0; k < D; ++k)
#pragma unroll
        for (int a = 0; a < D; ++a) {
            coords[(int64_t)(k * D + a) * F + f] = v[k][a];
            r[k * D + a] = v[k][a];
        }
#pragma unroll
    for (int a = 0; a < D; ++a) {
        float mn = v[0][a], mx = v[0][a];
#pragma unroll
        for (int k = 1; k < D; ++k) {
            mn = dev::fminf_(mn, v[k][a]);
            mx = dev::fmaxf_(mx, v[k][a]);
        }
        aabb[(int64_t)a * F + f] = mn;
        aabb[(int64_t)(D + a) * F + f] = mx;
        r[D * D + a] = mn;
        r[D * D + D + a] = mx;
        if (ext) ext[a] = fmaxf(ext[a], mx - mn);   // largest box extent per axis (NaN ignored)
    }
    if constexpr (D == 3) r[15] = 0.0f;
    float4 *out = reinterpret_cast<float4 *>(rec) + f * (dev::kRecFloats<D> / 4);
#pragma unroll
    for (int i = 0; i < dev::kRecFloats<D> / 4; ++i)
        out[i] = make_float4(r[4 * i], r[4 * i + 1], r[4 * i + 2], r[4 * i + 3]);
    return ok ? 0u : 2u;
}

// ===========================================================================
// Spatial binning (paper Sec. II-C-3)
// ===========================================================================
constexpr int kCanonCap = 2048;      // ids per LDS segment of the canonical sorts
constexpr int kBigThreads = 1024;

template <int D>
__device__ __forceinline__ void face_bin_range(const float *aabb, int64_t F, int64_t f, const dev::BinGrid &g,
                                               int lo[3], int hi[3]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) { lo[a] = 0; hi[a] = 0; }
#pragma unroll
    for (int a = 0; a < D; ++a) {
        lo[a] = dev::bin_of(aabb[(int64_t)a * F + f], g.lo[a], g.s[a], g.B);
        hi[a] = dev::bin_of(aabb[(int64_t)(D + a) * F + f], g.lo[a], g.s[a], g.B);
    }
}

// atomicAdd(p, 1) for every active lane, returning its old value, with the
// lanes whose counter is the first active lane's combined into one atomic (up
// to four such rounds; the rest add alone).  With few bins many faces of a
// wave share one, and same-address atomics from every face would serialise.
// Lanes are matched by address, so lanes of different arrays never combine.
// Slots of combined lanes follow the lane order.
__device__ __forceinline__ uint32_t add_one_combined(uint32_t *p) {
    const int lane = dev::lane_id();
    const uint64_t a = (uint64_t)(uintptr_t)p;
    bool pending = true;
    uint32_t slot = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint64_t act = __ballot(pending);
        if (!act) break;
        const int leader = __builtin_ctzll(act);
        const uint64_t la = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(a >> 32), leader) << 32) |
                            (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a, leader);
        const bool mine = pending && a == la;
        const uint64_t m = __ballot(mine);
        uint32_t base = 0;
        if (lane == leader) base = atomicAdd(p, (uint32_t)__popcll(m));
        base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
        if (mine) {
            slot = base + (uint32_t)dev::lanes_below(m);
            pending = false;
        }
    }
    if (pending) slot = atomicAdd(p, 1u);
    return slot;
}

// Count and scatter: one workgroup per nf consecutive faces (nf a power of two
// up to kPairThreads).  The (face, bin) pairs of its faces are taken
// kPairThreads x kPairRounds at a time, one per thread and round, and first
// meet in an LDS hash table of their bins: each pair takes its rank among the
// chunk's pairs of its bin there, and each distinct bin then goes out as one
// device atomic, all of a chunk's in flight together.  What bounds the passes is
// those atomics, performed past the per-XCD L2: neighbouring faces share their
// bins, so a chunk sends a fifth of its pairs.  A thread per face looping over
// its bins, equal bins of a wave combined in up to four rounds, took 33 us to
// count and 38 us to scatter 327,680 faces over 128^3 bins and 18 and 68 us for
// 320 faces of ~20 bins each.
constexpr int kPairThreads = 256;
constexpr int kPairRounds = 4;
constexpr int kPairTable = 2048;   // slots, twice a chunk's pairs

struct PairLds {
    uint4 key4[kPairTable / 4];   // bin index, ~0 empty (as uint4 for the clearing stores)
    uint4 val4[kPairTable / 4];   // pairs of the chunk in the bin, then (scatter) the chunk's first slot there
    uint32_t pre[kPairThreads], bin0[kPairThreads], nx[kPairThreads], ny[kPairThreads];
    uint32_t wsum[kPairThreads / dev::kWave];
};

// The total pairs of the nf faces of the workgroup's table (kOne: of its face k0 alone), a chunk of kPairThreads x
// kPairRounds at a time.
template <bool kScatter, bool kOne>
__device__ __forceinline__ void bin_pair_chunks(const dev::BinGrid &g, int64_t f0, int nf, int k0, uint32_t total,
                                                uint32_t *count, const uint32_t *off, int32_t *ids, PairLds &S) {
    const int tid = threadIdx.x;
    uint32_t *key = reinterpret_cast<uint32_t *>(S.key4), *val = reinterpret_cast<uint32_t *>(S.val4);
    constexpr uint32_t kChunk = kPairThreads * kPairRounds;
    for (uint64_t c0 = 0; c0 < total; c0 += kChunk) {
#pragma unroll
        for (int k = 0; k < kPairTable / 4 / kPairThreads; ++k) {
            S.key4[tid + k * kPairThreads] = make_uint4(~0u, ~0u, ~0u, ~0u);
            S.val4[tid + k * kPairThreads] = make_uint4(0u, 0u, 0u, 0u);
        }
        __syncthreads();
        uint32_t slot[kPairRounds], rank[kPairRounds];
        int32_t face[kPairRounds];
#pragma unroll
        for (int r = 0; r < kPairRounds; ++r) {
            const uint64_t v64 = c0 + (uint32_t)(r * kPairThreads + tid);
            const uint32_t v = (uint32_t)v64;
            face[r] = -1;
            if (v64 < total) {
                int k = kOne ? k0 : 0;   // the last face whose pairs start at or before v (the faces with none end the list)
#pragma unroll
                for (int step = kOne ? 0 : kPairThreads / 2; step >= 1; step >>= 1)
                    if (k + step < nf && S.pre[k + step] <= v) k += step;
                const uint32_t u = v - (kOne ? 0u : S.pre[k]), nx = S.nx[k], ny = S.ny[k];
                const uint32_t q = u / nx, z = q / ny;
                const uint32_t b = S.bin0[k] + (z * (uint32_t)g.B + (q - z * ny)) * (uint32_t)g.B + (u - q * nx);
                uint32_t h = (b * 2654435761u) >> 21;   // 11 bits: kPairTable slots
                while (true) {   // at most kChunk of kPairTable slots are taken
                    const uint32_t prev = atomicCAS(&key[h], ~0u, b);
                    if (prev == ~0u || prev == b) break;
                    h = (h + 1) & (kPairTable - 1);
                }
                face[r] = (int32_t)(f0 + k);
                slot[r] = h;
                rank[r] = atomicAdd(&val[h], 1u);
            }
        }
        __syncthreads();
        uint32_t base[kPairTable / kPairThreads];
#pragma unroll
        for (int k = 0; k < kPairTable / kPairThreads; ++k) {
            const int h = tid + k * kPairThreads;
            const uint32_t b = key[h];
            if (b == ~0u) continue;
            const uint32_t c = val[h];
            if constexpr (kScatter) base[k] = off[b] + (atomicSub(count + b, c) - c);
            else atomicAdd(count + b, c);
        }
        if constexpr (kScatter) {
#pragma unroll
            for (int k = 0; k < kPairTable / kPairThreads; ++k) {
                const int h = tid + k * kPairThreads;
                if (key[h] != ~0u) val[h] = base[k];
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kPairRounds; ++r)
                if (face[r] >= 0) ids[val[slot[r]] + rank[r]] = face[r];
        }
        __syncthreads();
    }
}

// kScatter false: count[bin] += the faces' pairs.  true: count holds the totals
// of the count pass and is used up (down to zero) as the cursor; the pairs go
// to ids at off[bin] + the place taken.  The faces' sum has to fit 32 bits:
// bin_pair_faces gives nf > 1 to faces of at most 512 bins.  A batch keeps its
// plan's nf while its faces may grow (kPlanned): with a face above kPairFaceMax
// the workgroup takes its faces one by one.
constexpr uint32_t kPairFaceMax = UINT32_MAX / kPairThreads;
template <int D, bool kScatter, bool kPlanned>
__device__ __forceinline__ void bin_pairs(const float *aabb, int64_t F, const dev::BinGrid &g, int64_t f0, int nf,
                                          uint32_t *count, const uint32_t *off, int32_t *ids, PairLds &S) {
    const int tid = threadIdx.x, lane = dev::lane_id(), w = tid / dev::kWave;
    uint32_t n = 0;
    if (tid < nf && f0 + tid < F) {
        int lo[3], hi[3];
        face_bin_range<D>(aabb, F, f0 + tid, g, lo, hi);
        uint32_t m[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) m[a] = (uint32_t)max(0, hi[a] - lo[a] + 1);
        n = m[0] * m[1] * m[2];   // at most B^D <= 2^31
        S.bin0[tid] = ((uint32_t)lo[2] * (uint32_t)g.B + (uint32_t)lo[1]) * (uint32_t)g.B + (uint32_t)lo[0];
        S.nx[tid] = m[0];
        S.ny[tid] = m[1];
    }
    const uint32_t incl = dev::wave_inclusive_sum(n);
    const bool wide = kPlanned && nf > 1 && __ballot(n > kPairFaceMax) != 0ull;
    if (lane == dev::kWave - 1) S.wsum[w] = wide ? UINT32_MAX : incl;   // (a sum is at most 2^31)
    __syncthreads();
    uint32_t before = 0, total = 0;
    bool single = false;
#pragma unroll
    for (int j = 0; j < kPairThreads / dev::kWave; ++j) {
        if (kPlanned) single = single || S.wsum[j] == UINT32_MAX;
        before += j < w ? S.wsum[j] : 0u;
        total += S.wsum[j];
    }
    if (!single) {
        S.pre[tid] = before + incl - n;   // faces past nf: the total
        bin_pair_chunks<kScatter, false>(g, f0, nf, 0, total, count, off, ids, S);
    } else {
        S.pre[tid] = n;
        __syncthreads();
        for (int k0 = 0; k0 < nf; ++k0)
            bin_pair_chunks<kScatter, true>(g, f0, nf, k0, S.pre[k0], count, off, ids, S);
    }
    __syncthreads();   // before the next faces' sums
}

// Faces per workgroup of the above: as many as give every CU two workgroups,
// and no more than fill one chunk when every face has the bins of the largest
// (per_face).  With few bins (nb) and many faces to each, the atomics of all
// workgroups meet on a few cache lines, and a workgroup sends at most one per
// bin however many faces it takes: then it takes as many as fill two such chunks.
// Whole binning of faces in random order, by the first rule / by both (and in
// the form with a thread per face): 20,000 segments in 9^2 bins 192 / 107 us
// (168), 5,120 triangles in 4^3 104 / 67 (82) and in 1 bin 72 / 59 (56), 81,920
// in 10^3 153 / 143 (146).  Below eight faces to a bin fewer workgroups cost
// more than the atomics saved: 1,280 segments in 22^2 bins 46 / 49.
constexpr int64_t kFewBins = 2048;
inline int bin_pair_faces(int64_t F, double per_face, int64_t nb, int n_cu) {
    const bool few = nb <= kFewBins && F / 8 >= nb;
    int nf = kPairThreads;
    while (nf > 1 && ((!few && F / nf < 2 * (int64_t)n_cu) ||
                      nf * per_face > (few ? 2.0 : 1.0) * (kPairThreads * kPairRounds)))
        nf >>= 1;
    return nf;
}

// Canonical order of one bin of at most kRankCap ids costs each id a pass over
// the bin's ids in LDS; a larger bin is sorted by a network, whose steps grow
// with log^2 instead of with the bin.  Measured, small + medium kernel, against
// ranks alone by one wave per group: 81,920 faces over 16^3 box bins (~170 ids in
// a bin) 833 -> 26 us, sampled-point bins 190 -> 25 us; 327,680 faces over 128^3
// bins (~34 ids in an occupied bin) 60 -> 36 us, 40,500 over 50^3 47 -> 16 us.
constexpr int kRankCap = 64;
constexpr int kCanonThreads = 256;
constexpr int kCanonWaves = kCanonThreads / dev::kWave;
constexpr int kWaveCap = 128;   // ids of a group that one wave sorts by itself (two a lane)

// LDS of one group of 64 bins: bounds and ids.
struct CanonLds {
    uint32_t off[kCanonWaves][dev::kWave + 1];
    int32_t val[kCanonCap];
};

// Sort ids[s0, s1) (64 bins whose offsets are in s_off) by rank: each id's
// position inside its bin is the number of smaller ids there.  Bins of at most
// kLaneRank ids: an id per lane, which reads its bin's ids from LDS.  Up to
// kRankCap: a bin per wave, an id per lane, every id broadcast to the wave from
// its register (a bin of 50 took each of its ids 50 LDS reads before).  Larger
// bins are left as they are.  NT threads (a wave, or the workgroup), t of them
// the caller; a thread's ids are loaded together.  kLaneRank 8 / 16 / 32, small and
// medium kernel: 327,680 faces in bins of ~21 ids 29 / 30 / 30 us, of ~15 36 / 35 /
// 27, of ~8 64 / 50 / 48; 20,480 faces in bins of ~8 13 / 10 / 9.
constexpr int kLaneRank = 16;
template <int NT, class Sync>
__device__ __forceinline__ void rank_sort_segment(int32_t *ids, const uint32_t *s_off, uint32_t s0, uint32_t s1,
                                                  int32_t *s_val, int t, Sync &&sync) {
    constexpr int PER = (NT == dev::kWave ? kWaveCap : kCanonCap) / NT;
    const int n = (int)(s1 - s0), lane = dev::lane_id(), wv = t / dev::kWave;
    int32_t own[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) own[k] = t + k * NT < n ? ids[s0 + t + k * NT] : 0;
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (t + k * NT < n) s_val[t + k * NT] = own[k];
    sync();
    const int l = (int)(s_off[lane + 1] - s_off[lane]);   // of bin `lane`
    if (__ballot(l > 1 && l <= kLaneRank)) {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = t + k * NT;
            if (e >= n) continue;
            // bin of entry e: the last one starting at or before it
            const uint32_t pos = s0 + (uint32_t)e;
            int bin = 0;
#pragma unroll
            for (int step = dev::kWave / 2; step >= 1; step >>= 1) bin += s_off[bin + step] <= pos ? step : 0;
            const int bs = (int)(s_off[bin] - s0), be = (int)(s_off[bin + 1] - s0);
            if (be - bs > kLaneRank) continue;
            const int32_t v = own[k];
            int rank = 0;
            // four ids in flight (past the end: the entry's own id, which counts 0)
            for (int j = bs; j < be; j += 4) {
                int32_t x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = s_val[j + u < be ? j + u : e];
#pragma unroll
                for (int u = 0; u < 4; ++u) rank += x[u] < v ? 1 : 0;
            }
            ids[s0 + bs + rank] = v;
        }
    }
    int k = 0;
    for (uint64_t m = __ballot(l > kLaneRank && l <= kRankCap); m; m &= m - 1ull, ++k) {
        if (k % (NT / dev::kWave) != wv) continue;
        const int bin = __builtin_ctzll(m);
        const int bs = (int)(s_off[bin] - s0), len = __builtin_amdgcn_readlane(l, bin);
        const int32_t v = lane < len ? s_val[bs + lane] : INT32_MAX;
        int rank = 0;
        for (int j = 0; j < len; ++j) rank += __builtin_amdgcn_readlane(v, j) < v ? 1 : 0;
        if (lane < len) ids[s0 + bs + rank] = v;
    }
}

// The group of 64 consecutive bins starting at b0, by NT threads (t of them the
// caller; s_off and s_val their LDS).  A group whose ids fit the LDS segment
// has its bins of at most kRankCap ids rank-sorted here in one go.  Every other
// bin with more than one id goes to a list: the medium list (at most kCanonCap
// ids: sorted by a workgroup per bin) or, tagged with big_tag, the big list
// (rebuilt by an ordered sweep).  Lists are appended through counters
// (counts[0], counts[1] = medium and big counts).
template <int NT, class Sync>
__device__ __forceinline__ void bin_canon_group(int32_t *ids, const uint32_t *off, int64_t nb, int64_t b0,
                                                uint32_t *med_list, uint32_t *big_list, uint32_t *counts,
                                                uint32_t big_tag, uint32_t *s_off, int32_t *s_val, int t,
                                                Sync &&sync) {
    const int nbins = (int)std::min<int64_t>(dev::kWave, nb - b0);
    for (int i = t; i <= dev::kWave; i += NT) s_off[i] = off[b0 + min(i, nbins)];   // bins past the last: empty
    sync();
    const uint32_t g0 = s_off[0], g1 = s_off[nbins];
    const bool fits = g1 - g0 <= (uint32_t)kCanonCap;
    if (t < nbins) {
        const uint32_t a0 = s_off[t], a1 = s_off[t + 1];
        if (a1 - a0 > (uint32_t)kCanonCap) big_list[atomicAdd(counts + 1, 1u)] = big_tag + (uint32_t)(b0 + t);
        else if (a1 - a0 > (fits ? (uint32_t)kRankCap : 1u)) med_list[atomicAdd(counts, 1u)] = (uint32_t)(b0 + t);
    }
    if (fits) rank_sort_segment<NT>(ids, s_off, g0, g1, s_val, t, sync);
    sync();   // before the next group's offsets and ids
}

// Workgroup w of nw: the groups w, w + nw, ... of 64 bins each.  Only the groups
// that hold at least two ids are opened, found 64 at a time from one load of
// their bounds: of a body's bins at a fine density most groups are empty (2^21
// bins over 327,680 faces: 87 % hold at most one id).  The full ones lie next to
// each other, along the body, so a workgroup's groups are nw apart.  Groups of at
// most kWaveCap ids are sorted by a wave each, side by side; the others by the
// whole workgroup, one after the other.
__device__ __forceinline__ void bin_canon_groups(int32_t *ids, const uint32_t *off, int64_t nb, int64_t w, int64_t nw,
                                                 uint32_t *med_list, uint32_t *big_list, uint32_t *counts,
                                                 uint32_t big_tag) {
    __shared__ CanonLds S;
    const int lane = dev::lane_id(), wv = (int)threadIdx.x / dev::kWave;
    const int64_t groups = (nb + dev::kWave - 1) / dev::kWave;
    for (int64_t i0 = w; i0 < groups; i0 += nw * dev::kWave) {
        const int64_t g = i0 + lane * nw;
        uint32_t n = 0;
        if (g < groups) n = off[std::min<int64_t>((g + 1) * dev::kWave, nb)] - off[g * dev::kWave];
        // the same in every wave of the workgroup
        const uint64_t small = __ballot(n > 1u && n <= (uint32_t)kWaveCap);
        int k = 0;
        for (uint64_t open = small; open; open &= open - 1ull, ++k)
            if (k % kCanonWaves == wv)
                bin_canon_group<dev::kWave>(ids, off, nb, (i0 + __builtin_ctzll(open) * nw) * dev::kWave, med_list,
                                            big_list, counts, big_tag, S.off[wv], S.val + wv * kWaveCap, lane,
                                            [] { dev::wave_sync(); });
        const uint64_t large = __ballot(n > (uint32_t)kWaveCap);
        if (!large) continue;
        __syncthreads();
        for (uint64_t open = large; open; open &= open - 1ull)
            bin_canon_group<kCanonThreads>(ids, off, nb, (i0 + __builtin_ctzll(open) * nw) * dev::kWave, med_list,
                                           big_list, counts, big_tag, S.off[0], S.val, (int)threadIdx.x,
                                           [] { __syncthreads(); });
    }
}

// Workgroups of the above for nb bins: one per group, at most as many as are
// resident at once (eight of 256 threads per CU).
inline unsigned canon_grid(int64_t nb, int n_cu) {
    return (unsigned)std::min<int64_t>((nb + dev::kWave - 1) / dev::kWave, 8 * (int64_t)n_cu);
}

// One workgroup of kMedThreads threads: bin b's segment (at most kCanonCap
// ids) sorted in LDS by a bitonic network over the next power of two.  A step
// of distance d <= 64 stays inside the 128 values of a wave's 64 pairs, so
// only the longer ones wait for the whole workgroup.
constexpr int kMedThreads = 256;
__device__ __forceinline__ void bin_canon_medium(int32_t *ids, const uint32_t *off, int64_t b) {
    __shared__ int32_t s_val[kCanonCap];
    const uint32_t s0 = off[b], s1 = off[b + 1];
    const int n = (int)(s1 - s0);
    int m = 2;
    while (m < n) m <<= 1;
    for (int e = threadIdx.x; e < m; e += kMedThreads) s_val[e] = e < n ? ids[s0 + e] : INT32_MAX;
    __syncthreads();
    for (int k = 2; k <= m; k <<= 1)
        for (int d = k >> 1; d >= 1; d >>= 1) {
            for (int i = threadIdx.x; i < m / 2; i += kMedThreads) {
                const int p = 2 * i - (i & (d - 1)), q = p + d;
                const int32_t x = s_val[p], y = s_val[q];
                if ((x > y) == ((p & k) == 0)) {
                    s_val[p] = y;
                    s_val[q] = x;
                }
            }
            // the next step's distance: d / 2, or k at the end of a stage
            if (d > 64 || (d == 1 && k > 64)) __syncthreads();
            else dev::wave_sync();
        }
    __syncthreads();
    for (int e = threadIdx.x; e < n; e += kMedThreads) ids[s0 + e] = s_val[e];
    __syncthreads();
}

// Bins with more than kCanonCap ids: rewrite the segment by an ordered sweep
// over all faces (membership recomputed from the bounding boxes).
// One workgroup of kBigThreads threads rebuilds bin b's segment.
template <int D>
__device__ __forceinline__ void bin_canon_big_bin(const float *aabb, int64_t F, const dev::BinGrid &g,
                                                  const uint32_t *off, int32_t *ids, int64_t b) {
    __shared__ uint32_t s_wsum[kBigThreads / dev::kWave];
    const int w = threadIdx.x / dev::kWave, lane = threadIdx.x % dev::kWave;
    {
        const int bx = (int)(b % g.B);
        const int by = (int)((b / g.B) % g.B);
        const int bz = D == 3 ? (int)(b / ((int64_t)g.B * g.B)) : 0;
        uint32_t run = off[b];
        for (int64_t f0 = 0; f0 < F; f0 += kBigThreads) {
            const int64_t f = f0 + threadIdx.x;
            uint32_t mem = 0;
            if (f < F) {
                int lo[3], hi[3];
                face_bin_range<D>(aabb, F, f, g, lo, hi);
                mem = (bx >= lo[0] && bx <= hi[0] && by >= lo[1] && by <= hi[1] && bz >= lo[2] && bz <= hi[2]) ? 1u : 0u;
            }
            uint32_t incl = dev::wave_inclusive_sum(mem);
            if (lane == dev::kWave - 1) s_wsum[w] = incl;
            __syncthreads();
            uint32_t pre = 0, tot = 0;
            for (int j = 0; j < kBigThreads / dev::kWave; ++j) {
                if (j < w) pre += s_wsum[j];
                tot += s_wsum[j];
            }
            if (mem) ids[run + pre + incl - 1] = (int32_t)f;
            run += tot;
            __syncthreads();
        }
    }
}


// ===========================================================================
// Candidate faces of a box (shared by the flag and q kernels)
// ===========================================================================
// Walks the face ids of bins [ilo, ihi] (inclusive, per axis) in rounds of 64,
// one candidate per lane: round(has, f, cur) is called by the whole wave, with
// `cur` the bin coordinates of the lane's candidate, and returns false to stop.
// Up to 64 bins are opened at once (one lane per bin, offsets loaded together;
// a wave prefix of their sizes makes one list), so small bins share rounds,
// and the ids of the next round are loaded while the current round runs:
// about one memory latency per 64 candidates instead of two per bin.
template <class Round>
__device__ __forceinline__ void for_candidates(const dev::BinGrid &g, const int ilo[3], const int ihi[3],
                                               Round &&round) {
    const int lane = dev::lane_id();
    const int nx = ihi[0] - ilo[0] + 1, ny = ihi[1] - ilo[1] + 1, nz = ihi[2] - ilo[2] + 1;
    const int nbins = nx * ny * nz;
    for (int bg = 0; bg < nbins; bg += dev::kWave) {
        const int bi = bg + lane;
        uint32_t s0 = 0, cnt = 0;
        if (bi < nbins) {
            const int bx = ilo[0] + bi % nx, by = ilo[1] + (bi / nx) % ny, bz = ilo[2] + bi / (nx * ny);
            const int64_t b = ((int64_t)bz * g.B + by) * g.B + bx;
            s0 = g.off[b];
            cnt = g.off[b + 1] - s0;
        }
        const uint32_t incl = dev::wave_inclusive_sum(cnt);
        const uint32_t pre = incl - cnt;
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, dev::kWave - 1);   // scalar
        const uint64_t nonempty = __ballot(cnt > 0);
        // id of list entry c0 + lane (or -1) and the lane holding its bin.  The
        // cross-lane reads run with every lane active: a lane reading from an
        // inactive lane gets 0, not that lane's value.
        auto fetch = [&](uint32_t c0, int &k) -> int32_t {
            const uint32_t v = c0 + lane;
            k = 0;
            for (uint64_t m = nonempty; m; m &= m - 1ull) {
                const int kk = __builtin_ctzll(m);
                k = __builtin_amdgcn_readlane(pre, kk) <= v ? kk : k;
            }
            const uint32_t s0k = __shfl(s0, k, dev::kWave);
            const uint32_t prek = __shfl(pre, k, dev::kWave);
            if (v >= total) return -1;
            const int32_t id = g.ids[s0k + (v - prek)];
            return id >= 0 && (int64_t)id < g.F ? id : -1;
        };
        int k = 0;
        int32_t f = fetch(0, k);
        for (uint32_t c0 = 0; c0 < total; c0 += dev::kWave) {
            int kn = 0;
            const int32_t fn = c0 + dev::kWave < total ? fetch(c0 + dev::kWave, kn) : -1;   // next round, in flight
            const int bk = bg + k;
            const int cur[3] = {ilo[0] + bk % nx, ilo[1] + (bk / nx) % ny, ilo[2] + bk / (nx * ny)};
            if (!round(f >= 0, f, cur)) return;
            f = fn;
            k = kn;
        }
    }
}

// Each face of bins [ilo, ihi] once, for boxes that span many bins (the flag
// pass): ids are read four rounds of 64 at a time (one memory latency per 256
// list entries), an LDS hash set of face ids drops the repeats of a face that
// lies in several bins, and the records of the faces that remain are loaded
// 64 at a time.  stage(has, f, r) is called by the whole wave with up to 64
// such faces (r the lane's face record) and returns false to stop.  A face
// that finds no free slot within kSeenProbes tries is passed on as new, so a
// crowded set can let a repeat through; stage() must tolerate that.
constexpr int kSeen = 1024;             // hash-set slots (power of two)
constexpr int kSeenProbes = 16;         // slots tried before a face is let through as new
constexpr int kUniqCap = 5 * 64;        // faces waiting for their records

template <int D, class Stage>
__device__ __forceinline__ void for_unique_candidates(const dev::BinGrid &g, const float *rec, const int ilo[3],
                                                      const int ihi[3], int32_t *s_seen, int32_t *s_list,
                                                      uint32_t *s_bpre, uint32_t *s_bs0, Stage &&stage) {
    constexpr int RF = dev::kRecFloats<D>;
    const int lane = dev::lane_id();
    const int nx = ihi[0] - ilo[0] + 1, ny = ihi[1] - ilo[1] + 1, nz = ihi[2] - ilo[2] + 1;
    const int nbins = nx * ny * nz;
    __syncthreads();
    for (int i = lane; i < kSeen; i += dev::kWave) s_seen[i] = -1;
    int nl = 0;   // wave-uniform list length
    // records of list entries 0 .. t-1, one per lane, to stage(); the rest moves to the front
    auto flush = [&](int t) -> bool {
        __syncthreads();
        const int32_t f = lane < t ? s_list[lane] : -1;
        __syncthreads();
        for (int i = lane; i < nl - t; i += dev::kWave) s_list[i] = s_list[t + i];   // up to 4 x 64 remain
        nl -= t;
        float r[RF];
        if (f >= 0) dev::load_rec<D>(rec, f, r);
        return stage(f >= 0, f, (const float *)r);
    };
    for (int bg = 0; bg < nbins; bg += dev::kWave) {
        const int bi = bg + lane;
        uint32_t s0 = 0, cnt = 0;
        if (bi < nbins) {
            const int bx = ilo[0] + bi % nx, by = ilo[1] + (bi / nx) % ny, bz = ilo[2] + bi / (nx * ny);
            const int64_t b = ((int64_t)bz * g.B + by) * g.B + bx;
            s0 = g.off[b];
            cnt = g.off[b + 1] - s0;
        }
        const uint32_t incl = dev::wave_inclusive_sum(cnt);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, dev::kWave - 1);   // scalar
        if (total == 0) continue;
        // the non-empty bins in list order, for a binary search per list entry
        const uint64_t ne = __ballot(cnt > 0);
        const int nne = __popcll(ne);
        __syncthreads();
        if (cnt > 0) {
            const int k = dev::lanes_below(ne);
            s_bpre[k] = incl - cnt;
            s_bs0[k] = s0;
        }
        __syncthreads();
        for (uint32_t c0 = 0; c0 < total; c0 += 4 * dev::kWave) {
            int32_t id[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t v = c0 + q * dev::kWave + lane;
                id[q] = -1;
                if (v < total) {
                    int lo = 0, hi = nne - 1;   // last non-empty bin starting at or before v
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (s_bpre[mid] <= v) lo = mid;
                        else hi = mid - 1;
                    }
                    const int32_t f = g.ids[s_bs0[lo] + (v - s_bpre[lo])];
                    id[q] = f >= 0 && (int64_t)f < g.F ? f : -1;
                }
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bool fresh = false;
                if (id[q] >= 0) {
                    uint32_t h = ((uint32_t)id[q] * 2654435761u) >> 22;   // 10 bits: kSeen slots
                    fresh = true;   // a crowded set lets the face through
                    for (int probe = 0; probe < kSeenProbes; ++probe) {
                        const int32_t prev = atomicCAS(&s_seen[h], -1, id[q]);
                        if (prev == -1) break;
                        if (prev == id[q]) {
                            fresh = false;
                            break;
                        }
                        h = (h + 1) & (kSeen - 1);
                    }
                }
                const uint64_t m = __ballot(fresh);
                if (fresh) s_list[nl + dev::lanes_below(m)] = id[q];
                nl += __popcll(m);
            }
            while (nl >= dev::kWave)
                if (!flush(dev::kWave)) return;
        }
    }
    if (nl > 0) (void)flush(nl);
}

// ===========================================================================
// Near-wall refinement (paper Sec. II-C-1, II-C-2)
// ===========================================================================
constexpr int kFlagCap = 128;  // staged candidate faces per wave

template <int D>
struct FlagArgs {
    dev::Faces faces;
    dev::BinGrid bins;
    const uint32_t *keys;
    int64_t n;
    int level;
    int R[3];
    float lo[3];
    float dx[3];
    float eps[3];
    float h;
    uint8_t *cf;     // n * 4^D
    uint8_t *pmark;  // n
};

// One wave: blocks first .. first + 64/4^D - 1 of A (one lane per cell).
template <int D, bool kDedup = false>
__device__ __forceinline__ void flag_wave(const FlagArgs<D> &A, int64_t first) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    constexpr int BPW = 64 / CELLS;
    constexpr int NF = D * D;   // staged corner coordinates
    __shared__ float s_f[NF][kFlagCap];
    __shared__ __align__(16) uint32_t s_code[kFlagCap];
    const int lane = threadIdx.x;
    const int64_t blk = first + lane / CELLS;
    const bool valid = blk < A.n;
    const int cell = lane % CELLS;
    const int sub = lane / CELLS;

    int bc[3] = {0, 0, 0};
    if (valid) dev::decode_key<D>(A.keys[blk], A.level, A.R[0], A.R[1], bc);
    const int pos3[3] = {cell & 3, (cell >> 2) & 3, cell >> 4};
    float m[3];
    m[0] = dev::cell_centre(A.lo[0], 4 * bc[0] + pos3[0], A.dx[0]);
    m[1] = dev::cell_centre(A.lo[1], 4 * bc[1] + pos3[1], A.dx[1]);
    m[2] = D == 3 ? dev::cell_centre(A.lo[2], 4 * bc[2] + pos3[2], A.dx[2]) : 0.0f;
    const float h = A.h;
    bool flagged = !valid;

    // The box-axis part of the separating-axis test is separable: cell (i0,i1,i2)
    // of a block is not separated from a face along axis a exactly when position
    // i_a passes the axis-a test, so a staged face carries one bit per (axis,
    // position) of the block it was staged for, computed with the same FP32
    // expressions every lane would use (min_k fl(v_k - m) = fl(min_k v_k - m)),
    // and a lane tests a face with one AND against its own D bits.  (In 2D the
    // four blocks of a wave take bits 8t..8t+7; a face near a cell of block t
    // lies in block t's query box, so it is staged, and coded, for block t.)
    uint32_t lbits = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) lbits |= 1u << (sub * 4 * D + 4 * a + pos3[a]);
    float mc[D][4];   // cell centres along each axis of the block being staged
    auto face_code = [&](int t, const float *bb) -> uint32_t {   // bb: min[D], max[D]
        uint32_t c = 0;
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float lo_a = bb[a] - mc[a][i], hi_a = bb[D + a] - mc[a][i];
                c |= (!(lo_a > h) && !(hi_a < -h)) ? (1u << (4 * a + i)) : 0u;
            }
        return c << (t * 4 * D);
    };

    int count = 0;  // staged faces (wave-uniform)
    // The full tests wait in a queue of (lane, staged face) pairs and are taken
    // 64 at a time, one per lane, whichever lane queued them: a cell near many
    // faces does not hold the wave while the other lanes idle.  A pair whose
    // cell is flagged meanwhile is dropped.
    constexpr int TCAP = 128;   // below 64 after a take, at most 64 added per step
    __shared__ uint32_t s_q[TCAP];
    __shared__ float s_m[64][3];
    __shared__ int s_fl[64];
#pragma unroll
    for (int a = 0; a < 3; ++a) s_m[lane][a] = m[a];
    s_fl[lane] = flagged ? 1 : 0;
    int nq = 0;   // wave-uniform
    auto take = [&](int t) {
        __syncthreads();
        const uint32_t item = lane < t ? s_q[lane] : 0u;
        __syncthreads();
        if (lane < nq - t) s_q[lane] = s_q[t + lane];
        nq -= t;
        const int l = (int)(item >> 7), j = (int)(item & 127u);
        if (lane < t && !s_fl[l]) {
            float v[D * D];
#pragma unroll
            for (int k = 0; k < D * D; ++k) v[k] = s_f[k][j];
            const float ml[3] = {s_m[l][0], s_m[l][1], s_m[l][2]};
            bool hit;
            if constexpr (D == 3) hit = dev::sat_triangle(v, ml, h);
            else hit = dev::sat_segment(v, ml, h);
            if (hit) s_fl[l] = 1;
        }
    };
    // Batches of 64 staged faces: each lane marks the faces its cube's box axes do
    // not separate from it and queues them for the full test, until flagged.
    auto test_staged = [&](int n) {
        __syncthreads();
        for (int j0 = 0; j0 < n; j0 += 64) {
            flagged = s_fl[lane] != 0;
            if (__ballot(!flagged) == 0) break;
            const int jn = min(64, n - j0);
            uint64_t nm = 0;
            if (!flagged)
                for (int jj = 0; jj < jn; jj += 4) {
                    // four codes per step, read as the uint32_t objects they are
                    const uint32_t cs[4] = {s_code[j0 + jj], s_code[j0 + jj + 1], s_code[j0 + jj + 2],
                                            s_code[j0 + jj + 3]};
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        nm |= ((cs[u] & lbits) == lbits && jj + u < jn) ? (1ull << (jj + u)) : 0ull;
                }
            while (__ballot(nm != 0)) {
                int j = 0;
                const bool has = nm != 0;
                if (has) {
                    j = j0 + __builtin_ctzll(nm);
                    nm &= nm - 1ull;
                }
                const uint64_t want = __ballot(has);
                if (has) s_q[nq + dev::lanes_below(want)] = ((uint32_t)lane << 7) | (uint32_t)j;
                nq += __popcll(want);
                if (nq >= 64) {
                    take(64);
                    __syncthreads();
                    if (s_fl[lane]) nm = 0;   // flagged meanwhile: nothing more to queue
                }
            }
        }
        if (nq > 0) take(nq);
        __syncthreads();
        flagged = s_fl[lane] != 0;
    };

    __shared__ int32_t s_seen[kDedup ? kSeen : 1];
    __shared__ int32_t s_list[kDedup ? kUniqCap : 1];
    __shared__ uint32_t s_bpre[kDedup ? 64 : 1], s_bs0[kDedup ? 64 : 1];
    bool done = __ballot(!flagged) == 0;
    for (int sb = 0; sb < BPW && !done; ++sb) {
        if (first + sb >= A.n) break;
        // block coordinates of sub-block sb (from its first lane)
        int sc[3];
        sc[0] = __shfl(bc[0], sb * CELLS, 64);
        sc[1] = __shfl(bc[1], sb * CELLS, 64);
        sc[2] = __shfl(bc[2], sb * CELLS, 64);
        float qlo[3] = {0, 0, 0}, qhi[3] = {0, 0, 0};
        int ilo[3] = {0, 0, 0}, ihi[3] = {0, 0, 0};
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i) mc[a][i] = dev::uniform(dev::cell_centre(A.lo[a], 4 * sc[a] + i, A.dx[a]));
#pragma unroll
        for (int a = 0; a < D; ++a) {
            qlo[a] = (dev::cell_centre(A.lo[a], 4 * sc[a], A.dx[a]) - h) - A.eps[a];
            qhi[a] = (dev::cell_centre(A.lo[a], 4 * sc[a] + 3, A.dx[a]) + h) + A.eps[a];
            ilo[a] = dev::bin_of(qlo[a], A.bins.lo[a], A.bins.s[a], A.bins.B);
            ihi[a] = dev::bin_of(qhi[a], A.bins.lo[a], A.bins.s[a], A.bins.B);
        }
        // stage the faces whose box meets the query box (r: the lane's face record)
        auto stage = [&](bool has, int32_t f, const float *r) -> bool {
            bool keep = has;
#pragma unroll
            for (int a = 0; a < D; ++a) keep = keep && r[D * D + a] <= qhi[a] && r[D * D + D + a] >= qlo[a];
            const uint64_t mask = __ballot(keep);
            const int nk = __popcll(mask);
            if (nk == 0) return true;
            if (count + nk > kFlagCap) {
                test_staged(count);
                count = 0;
                done = __ballot(!flagged) == 0;
                if (done) return false;
            }
            if (keep) {
                const int pos = count + dev::lanes_below(mask);
#pragma unroll
                for (int k = 0; k < NF; ++k) s_f[k][pos] = r[k];
                s_code[pos] = face_code(sb, r + D * D);
            }
            count += nk;
            return true;
        };
        if constexpr (kDedup) {
            for_unique_candidates<D>(A.bins, A.faces.rec, ilo, ihi, s_seen, s_list, s_bpre, s_bs0, stage);
        } else {
            for_candidates(A.bins, ilo, ihi, [&](bool has, int32_t f, const int cur[3]) -> bool {
                // visit each face once: in the first bin of (its bins) x (query bins)
                float r[dev::kRecFloats<D>];
                bool first_bin = has;
                if (has) {
                    dev::load_rec<D>(A.faces.rec, f, r);
#pragma unroll
                    for (int a = 0; a < D; ++a)
                        first_bin = first_bin &&
                                    max(dev::bin_of(r[D * D + a], A.bins.lo[a], A.bins.s[a], A.bins.B), ilo[a]) == cur[a];
                }
                return stage(first_bin, f, (const float *)r);
            });
        }
    }
    if (!done && count > 0) test_staged(count);

    if (valid) A.cf[blk * CELLS + cell] = flagged ? 1 : 0;
    // block mark: OR over the block's cells
    const uint64_t fm = __ballot(valid && flagged);
    if (valid && cell == 0) {
        uint64_t bm = fm;
        if constexpr (CELLS < 64) bm = (fm >> (lane & ~(CELLS - 1))) & ((1ull << CELLS) - 1);
        A.pmark[blk] = bm ? 1 : 0;
    }
}

// How far from its bounding box a face can be near_l2 at distance R, squared
// (+inf: no bound is claimed).  near_l2 decides on rounded sums, so it may call
// a point near that is a little beyond R: on an edge of length l the rounded
// cross and dot products move the distance by at most 2^-19 (R + l); on the
// face itself the normal's rounding tilts the plane and moves the three sides
// by up to 2^-20 of the point's distance, at a corner that over the sine of its
// angle.  With |n| >= 1e-2 l_max^2 (every angle's sine is at least that) all of
// it stays below 1e-3 (R + l_max), which the bound adds.  Slivers below that,
// edges too short or too long for their squares' and fourth powers' range, and
// huge R get no bound.  Where it is finite, near_l2 also accepts every point
// within R (1 - 2^-15) of the first corner: the first edge's test comes down to
// that corner, to the other end when that is nearer, or to the line between,
// which is nearer still.  r: the face's record.
template <int D>
AGAL_HD float near_reach2(const float *r, float R) {
    float m2 = 0.0f;
    bool fine = R <= 1e8f;
#pragma unroll
    for (int k = 0; k < (D == 3 ? 3 : 1); ++k) {
        const float *a = r + D * k, *b = r + D * ((k + 1) % D);
        float e2 = 0.0f;
#pragma unroll
        for (int j = 0; j < D; ++j) e2 += (b[j] - a[j]) * (b[j] - a[j]);
        m2 = fmaxf(m2, e2);
    }
    fine = fine && m2 >= 1e-10f && m2 <= 1e10f;
    if constexpr (D == 3) {
        float e1[3], e2[3], n[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            e1[a] = r[3 + a] - r[a];
            e2[a] = r[6 + a] - r[a];
        }
        dev::cross3_(e1, e2, n);
        fine = fine && dev::dot3_(n, n) >= 1e-4f * (m2 * m2);
    }
    const float reach = 1.002f * R + 0.002f * sqrtf(m2);
    return fine ? reach * reach : __builtin_inff();   // a NaN coordinate: not fine
}

// The two short tests of the own-bin pass for the face of record r (reach2: its near_reach2) and the point m: true
// where near_l2 certainly accepts (sure2: 0.9999 R^2); maybe: false where it certainly refuses.
template <int D>
AGAL_HD bool own_short(const float *r, const float *m, float reach2, float sure2, bool &maybe) {
    float d2 = 0.0f, w2 = 0.0f;
#pragma unroll
    for (int a = 0; a < D; ++a) {
        const float d = fmaxf(fmaxf(r[D * D + a] - m[a], m[a] - r[D * D + D + a]), 0.0f);
        d2 += d * d;
        const float w = m[a] - r[a];
        w2 += w * w;
    }
    maybe = !(d2 > reach2);                             // (a NaN on either side keeps the face)
    return reach2 < __builtin_inff() && w2 <= sure2;   // the short acceptance holds where the bound does
}

// Own-bin flag pass, the paper's face detection as printed (Sec. II-C-2 with
// Algorithm 1, bins of Sec. II-C-3): a cell looks only at the faces of the one
// bin that holds its centre (bin index function of the binning) and is
// flagged when its centre lies within Euclidean distance h of one of them
// (near_l2).  One wave: blocks first .. first + 64/4^D - 1 (one lane per
// cell).  The wave takes the distinct own bins of its lanes one after the
// other and each bin's faces 64 at a time, a face per lane (the next 64
// records and the ids after those in flight), and goes through the bin's cells
// that are not flagged yet.  What bounds the pass is VALU issue in the tests:
// near_l2 takes ~200 instructions, and a wave has to try every face of its bin
// for a cell that is near none.  So kOwnCells cells at a time take two short
// tests first: a face whose first corner is clearly within h flags the cell
// (near_l2 accepts it), a face whose box is beyond near_reach2 is out (near_l2
// would refuse it), and near_l2 runs only for a cell where neither settles it.
// 81,920 faces in 16^3 bins (up to 1,000 a bin), h = 0.05, two passes: 1,121 us
// with a cell per lane and near_l2 for every face; 366 with the box test before
// it; 136 with a face per lane; 121 with the corner test.
// A bin of at most as many faces as the wave has cells there leaves lanes idle
// that way: it takes a cell per lane, with the same tests for each of its faces.
// Whole calls over 32^3 roots, two passes, one cell length: 320 faces in 16^3
// bins 325 us with near_l2 for every face, 663 with a face per lane, 267 with the
// rule; 80 faces in 4^3 bins 425, 821, 325; 5,120 faces in 16^3 bins 471, 495, 352
// (411 with the line at half as many faces, 353 at twice as many).
// Faces without a bound (slivers, specks) need near_l2 for every cell.  By face,
// the lanes take its branches each their own way; by cell, the cells of a block
// mostly go together: so they too go by cell, from LDS, unless few cells are left
// (in 2D, where near_l2 costs no more than the short tests, with the others of
// their 64).  4,000 slivers in one bin, 16^3 roots: 19.7 ms with near_l2 for every
// face by cell, 28.6 by face, 22.2 by the rule; with a third of the faces flat
// 19.5, 20.1, 12.5.
// Writes every cell flag and the block's pass mark (0 or 1).
constexpr int kOwnCells = 4;
template <int D>
__device__ __forceinline__ void flag_own_bin_wave(const FlagArgs<D> &A, int64_t first) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    constexpr int RF = dev::kRecFloats<D>;
    __shared__ float s_v[64][D * D];
    const int lane = dev::lane_id();
    const int64_t blk = first + lane / CELLS;
    const bool valid = blk < A.n;
    const int cell = lane % CELLS;
    int bc[3] = {0, 0, 0};
    if (valid) dev::decode_key<D>(A.keys[blk], A.level, A.R[0], A.R[1], bc);
    float m[3] = {0.0f, 0.0f, 0.0f};
    m[0] = dev::cell_centre(A.lo[0], 4 * bc[0] + (cell & 3), A.dx[0]);
    m[1] = dev::cell_centre(A.lo[1], 4 * bc[1] + ((cell >> 2) & 3), A.dx[1]);
    if constexpr (D == 3) m[2] = dev::cell_centre(A.lo[2], 4 * bc[2] + (cell >> 4), A.dx[2]);
    int ib[3] = {0, 0, 0};
#pragma unroll
    for (int a = 0; a < D; ++a) ib[a] = dev::bin_of(m[a], A.bins.lo[a], A.bins.s[a], A.bins.B);
    const int mybin = (ib[2] * A.bins.B + ib[1]) * A.bins.B + ib[0];   // B^D < 2^31 (checked when binning)
    const float sure2 = 0.9999f * (A.h * A.h);
    uint64_t flagged = 0;   // lanes (cells) flagged, wave-uniform
    for (uint64_t open = __ballot(valid); open;) {
        const int bin = __builtin_amdgcn_readlane(mybin, __builtin_ctzll(open));
        uint64_t cells = __ballot(mybin == bin) & open;   // this bin's cells not flagged yet
        open &= ~cells;
        const uint32_t s0 = A.bins.off[bin], s1 = A.bins.off[bin + 1];
        // id of list entry e (-1 past the bin's end, and for an id that is no face), and its record (NaN: never near)
        auto id_at = [&](uint64_t e) -> int32_t {
            if (e >= s1) return -1;
            const int32_t f = A.bins.ids[e];
            return f >= 0 && (int64_t)f < A.bins.F ? f : -1;
        };
        auto rec_at = [&](int32_t f, float (&r)[RF]) {
            if (f >= 0) {
                dev::load_rec<D>(A.faces.rec, f, r);
            } else {
#pragma unroll
                for (int k = 0; k < RF; ++k) r[k] = __builtin_nanf("");
            }
        };
        // a cell per lane: the faces held by the lanes of `faces`, one after the other
        auto by_cell = [&](uint64_t faces, const float (&rl)[RF]) {
            bool todo = ((cells >> lane) & 1ull) != 0ull;
            dev::wave_sync();
#pragma unroll
            for (int k = 0; k < D * D; ++k) s_v[lane][k] = rl[k];
            dev::wave_sync();
            for (; faces && __ballot(todo); faces &= faces - 1ull) {
                const int j = __builtin_ctzll(faces);
                float v[D * D];
#pragma unroll
                for (int k = 0; k < D * D; ++k) v[k] = s_v[j][k];
                if (todo && dev::near_l2<D>(v, m, A.h)) todo = false;
            }
            flagged |= cells & ~__ballot(todo);
            cells &= ~flagged;
        };
        // the same for faces with a bound, by the short tests first
        auto by_cell_bounded = [&](uint64_t faces, const float (&rl)[RF], float reach2l) {
            bool todo = ((cells >> lane) & 1ull) != 0ull;
            for (; faces && __ballot(todo); faces &= faces - 1ull) {
                const int j = __builtin_ctzll(faces);
                auto of_face = [&](float x) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), j)); };
                float r[RF];
#pragma unroll
                for (int k = 0; k < D * D + 2 * D; ++k) r[k] = of_face(rl[k]);
                const float reach2 = of_face(reach2l);   // (with the whole wave: the face's lane may be done)
                if (todo) {
                    bool maybe;
                    if (own_short<D>(r, m, reach2, sure2, maybe)) todo = false;
                    else if (maybe && dev::near_l2<D>(r, m, A.h)) todo = false;
                }
            }
            flagged |= cells & ~__ballot(todo);
            cells &= ~flagged;
        };
        float rn[RF];
        int32_t f = id_at((uint64_t)s0 + (uint32_t)lane);
        rec_at(f, rn);
        if (s1 - s0 <= (uint32_t)__popcll(cells)) {
            const float reach2 = near_reach2<D>(rn, A.h);
            const bool bounded = reach2 < __builtin_inff();
            by_cell_bounded(__ballot(f >= 0 && bounded), rn, reach2);
            const uint64_t wide = __ballot(f >= 0 && !bounded);
            if (wide) by_cell(wide, rn);
            continue;
        }
        int32_t fn = id_at((uint64_t)s0 + dev::kWave + (uint32_t)lane);
        for (uint64_t c0 = s0; c0 < s1 && cells; c0 += dev::kWave) {
            float r[RF];
#pragma unroll
            for (int k = 0; k < RF; ++k) r[k] = rn[k];
            bool has = f >= 0;
            f = fn;
            rec_at(f, rn);
            fn = id_at(c0 + 2 * dev::kWave + (uint32_t)lane);
            const float reach2 = near_reach2<D>(r, A.h);
            const uint64_t wide = __ballot(has && !(reach2 < __builtin_inff()));
            if (wide) {
                const uint64_t faces = D == 3 ? wide : __ballot(has);
                if (5 * __popcll(faces) <= 8 * __popcll(cells)) {
                    by_cell(faces, r);
                    has = has && !((faces >> lane) & 1ull);
                    if (!__ballot(has)) continue;
                }
            }
            for (uint64_t left = cells; left;) {
                int c[kOwnCells];
                bool sure[kOwnCells], maybe[kOwnCells];
                float mc[kOwnCells][3];
#pragma unroll
                for (int u = 0; u < kOwnCells; ++u) {
                    c[u] = left ? __builtin_ctzll(left) : c[0];   // the last few: one cell several times
                    left &= left - 1ull;
                    mc[u][2] = 0.0f;
#pragma unroll
                    for (int a = 0; a < D; ++a)
                        mc[u][a] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(m[a]), c[u]));
                    sure[u] = own_short<D>(r, mc[u], reach2, sure2, maybe[u]) && has;
                    maybe[u] = maybe[u] && has;
                }
#pragma unroll
                for (int u = 0; u < kOwnCells; ++u) {
                    bool near = __ballot(sure[u]) != 0ull;
                    if (!near && __ballot(maybe[u])) {
                        bool hit = false;
                        if (maybe[u]) hit = dev::near_l2<D>(r, mc[u], A.h);
                        near = __ballot(hit) != 0ull;
                    }
                    if (near) flagged |= 1ull << c[u];
                }
            }
            cells &= ~flagged;
        }
    }
    if (valid) A.cf[blk * CELLS + cell] = (flagged >> lane) & 1ull ? 1 : 0;
    if (valid && cell == 0) {
        uint64_t bm = flagged;
        if constexpr (CELLS < 64) bm = (flagged >> (lane & ~(CELLS - 1))) & ((1ull << CELLS) - 1);
        A.pmark[blk] = bm ? 1 : 0;
    }
}

// Mark propagation of the own-bin pass (Sec. II-C-3), one step in two
// launches so that a step grows the marked set by exactly one ring whatever
// the order of the threads: (1) every unmarked level-l neighbour (faces,
// edges, corners; inside the domain; present at level l) of a block whose
// pass mark is 1 (flagged) or 3 (propagated) gets the intermediate value 4;
// (2) every 4 becomes 3.  One thread per (block, neighbour position).
template <int D>
__device__ __forceinline__ void prop_spread_item(const uint32_t *keys, int64_t n, uint8_t *pm, int l, int R0, int R1,
                                                 int R2, int64_t t) {
    constexpr int NNB = D == 3 ? 26 : 8;
    const int64_t i = t / NNB;
    const uint8_t p = pm[i];
    if (p != 1 && p != 3) return;
    int k = (int)(t % NNB);
    k += k >= NNB / 2 ? 1 : 0;   // skip the centre of the 3^D stencil
    const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = D == 3 ? k / 9 - 1 : 0;
    int c[3];
    dev::decode_key<D>(keys[i], l, R0, R1, c);
    const int ext[3] = {R0 << l, R1 << l, R2 << l};
    int nc[3] = {c[0] + dx, c[1] + dy, c[2] + dz};
    if (nc[0] < 0 || nc[0] >= ext[0] || nc[1] < 0 || nc[1] >= ext[1]) return;
    if (D == 3 && (nc[2] < 0 || nc[2] >= ext[2])) return;
    const uint32_t kn = dev::encode_key<D>(nc, l, R0, R1);
    const int64_t j = dev::lower_bound_u32(keys, n, kn);
    if (j < n && keys[j] == kn && pm[j] == 0) pm[j] = 4;
}

// Face-centric flag pass.  A cell's flag is an OR over faces of one FP32 test
// (sat_triangle / sat_segment at the cell centre, half-width h), so it can be
// gathered from the faces' side as well: each face visits the cells whose
// centre lies within h + eps of its box on every axis (a superset of the cells
// whose box-axis tests it passes) and sets the flag of each cell it is not
// separated from.  The work is a few cells per face, spread over every lane of
// the chip, where the cell-centric pass is as long as its busiest block's wave
// (a coarse block's query box spans hundreds of bins).  Cells of blocks that
// do not exist at the level are skipped: a dense table over the level's block
// grid holds each block's index; an entry counts only when it is below n and
// the level's key at that index is the key of the grid position, so the table
// is never cleared and stale entries read as absent.  At level 0 every block
// exists and the index is the linear one.  Cell flags and block marks must
// start at zero; only ones are stored, so faces that meet the same cell race
// harmlessly.
// The pass is bound by vector instructions: ~300 of the full test for 64 pairs,
// ~110 to find the pairs, their blocks and flags, and ~60 to queue those that
// need the test.  With the short form of the test (below) before the block is
// looked up, no queue: 327,680 faces over four levels 298 -> 195 us, 81,920
// faces over three 101 -> 70, 20,480 faces 44 -> 34.  A face's set-up by four
// lanes (a quarter of its record, an axis of its FP64 cell range, an edge's axes
// each) instead of one: ~350 of a wave's 1,370 instructions less, 199 -> 177, 71 ->
// 63, 35 -> 30.
// Faces per wave G (4, 8 or 16) is picked per launch: small face counts take
// small G so that the pass still has several waves per SIMD to hide the table
// and flag reads.  All levels of a call with G = 4 / 8 / 16: 20,480 faces 29 / 32 /
// 43 us, 40,500 38.5 / 34 / 41, 81,920 68 / 61 / 59, 327,680 255 / 195 / 176; six
// bodies in a batch, whose faces have more cells each, 136 / 149 / 203.  (So the
// step from 4 to 8 could come at half as many faces for one body, for ~4 us; the
// batch's, which counts the faces of all bodies, would lose more.)
constexpr int kFaceFlagWaves = 4;   // waves per workgroup
constexpr int kFaceFlagInts = 10;   // per-face words of the wave's face table
inline int face_flag_g(int64_t faces, int n_cu) {
    const int64_t want = 8 * 4 * (int64_t)n_cu;   // waves: eight per SIMD
    return faces >= 16 * want ? 16 : (faces >= 8 * want ? 8 : 4);
}

template <int D>
struct FaceFlagArgs {
    const float *rec;         // F x kRecFloats<D>
    int64_t F;
    int NB[3];                // blocks per axis at this level (roots << level)
    const uint32_t *table;    // NB0 NB1 NB2 entries, x fastest; null at level 0
    const uint32_t *keys;     // the level's keys (n), to validate table entries
    int64_t n;
    int level;
    int R[2];                 // roots along x and y (key encoding)
    float lo[3];
    float dx[3];              // cell size at this level
    float eps[3];
    float h;
    uint8_t *cf;              // n x 4^D, zeroed
    uint8_t *pmark;           // n, zeroed
};

// Inclusive sum over the wave on DPP (every lane active): row shifts by 1, 2,
// 4 and 8, then lane 15 of the previous row into rows 1 and 3 and lane 31
// into rows 2 and 3; lanes without a source add 0.
__device__ __forceinline__ uint32_t dpp_inclusive_sum(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);
    return v;
}

// Short form of sat_triangle for one face and many cells of half-width h: the
// 13 axes are set up once per face (sat_axes: axes of edge `part`, or with part
// 3 the plane and the box), and a cell costs ~50 operations instead of ~300.
// With m the cell's centre and every axis a, its separation is |a . (m - v0) -
// c| - w, w = half the triangle's extent along a plus the cell's; sat_gap
// returns the largest of the 13.  Where R bounds the distance of a corner to the
// centre on each axis and u = 2^-24, sat_triangle's rounded comparison of an
// edge axis is off by at most 22 u R^2, its plane's (here over R) by 136 u R^2,
// and the ones here by at most 36 and 75; so a gap beyond 2^-15 R^2 = 512 u R^2
// (delta) decides: above, sat_triangle finds a separating axis, below -delta it
// finds none.  In between, and where R is so small or large that R^3 leaves
// FP32's range (beyond 1e-12 .. 1e12: delta = inf), the test itself is run.  An
// axis that is zero (edge along a coordinate axis) separates nothing there either.
constexpr int kSatWords = 13;   // float4 per face: 9 edge axes (a, c, w), normal, v0, box

AGAL_HD void sat_axes(const float *r, float h, const float eps[3], int part, float4 *out) {
    const float b[3] = {r[3] - r[0], r[4] - r[1], r[5] - r[2]}, c[3] = {r[6] - r[0], r[7] - r[1], r[8] - r[2]};
    float R = 0.0f;
#pragma unroll
    for (int a = 0; a < 3; ++a) R = fmaxf(R, (r[12 + a] - r[9 + a]) + (fabsf(h) + eps[a]));
    R *= 1.0001f;
    const float R2 = R * R;
    if (part < 3) {
        float e[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) e[a] = part == 0 ? b[a] : (part == 1 ? r[6 + a] - r[3 + a] : -c[a]);
#pragma unroll
        for (int x = 0; x < 3; ++x) {   // on components (y, z), (x, z), (x, y)
            const int i = x == 0 ? 1 : 0, j = x == 2 ? 1 : 2;
            const float au = x == 1 ? e[j] : -e[j], av = x == 1 ? -e[i] : e[i];
            const float p1 = au * b[i] + av * b[j], p2 = au * c[i] + av * c[j];
            const float mn = fminf(fminf(p1, p2), 0.0f), mx = fmaxf(fmaxf(p1, p2), 0.0f);
            const bool none = au == 0.0f && av == 0.0f;
            out[3 * part + x] = make_float4(au, av, -0.5f * (mn + mx),
                                            none ? R2 : 0.5f * (mx - mn) + h * (fabsf(au) + fabsf(av)));
        }
    } else {
        const float inv = 1.0f / R;
        const float n[3] = {(b[1] * c[2] - b[2] * c[1]) * inv, (b[2] * c[0] - b[0] * c[2]) * inv,
                            (b[0] * c[1] - b[1] * c[0]) * inv};
        out[9] = make_float4(n[0], n[1], n[2], h * ((fabsf(n[0]) + fabsf(n[1])) + fabsf(n[2])));
        out[10] = make_float4(r[0], r[1], r[2], R);
        float bc[3], bw[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            bc[a] = 0.5f * ((r[9 + a] - r[a]) + (r[12 + a] - r[a]));
            bw[a] = 0.5f * (r[12 + a] - r[9 + a]) + h;
        }
        const bool fits = R2 >= 1e-24f && R2 <= 1e24f;
        out[11] = make_float4(bc[0], bc[1], bc[2], fits ? 3.0517578125e-05f * R2 : INFINITY);
        out[12] = make_float4(bw[0], bw[1], bw[2], 0.0f);
    }
}

AGAL_HD float sat_gap(const float4 *ax, const float m[3], float &delta) {
    const float4 v = ax[10], n = ax[9], bc = ax[11], bw = ax[12];
    const float p[3] = {m[0] - v.x, m[1] - v.y, m[2] - v.z};
    const float box = fmaxf(fmaxf(fabsf(p[0] - bc.x) - bw.x, fabsf(p[1] - bc.y) - bw.y), fabsf(p[2] - bc.z) - bw.z);
    float gap = fmaxf(box * v.w, fabsf(fmaf(n.x, p[0], fmaf(n.y, p[1], n.z * p[2]))) - n.w);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const float4 a = ax[k];
        const int i = k % 3 == 0 ? 1 : 0, j = k % 3 == 2 ? 1 : 2;
        gap = fmaxf(gap, fabsf(fmaf(a.x, p[i], fmaf(a.y, p[j], a.z))) - a.w);
    }
    delta = bc.w;
    return gap;
}

// One wave: faces face0 .. face0 + G - 1.  The (face, cell) pairs of
// its faces are listed in face order and taken 64 at a time, one per lane.  A
// face with a non-finite coordinate has no pairs (its input is rejected
// anyway; the batched form reports it after the run).  Pair counts are 64-bit:
// a face much larger than the level's cells can have more than 2^32 / 16
// pairs; index arithmetic stays 32-bit while the wave's total fits.
template <int D, int G>
__device__ __forceinline__ void flag_faces_wave(const FaceFlagArgs<D> &A, int64_t face0,
                                                float (*s_rec)[dev::kRecFloats<D>], int (*s_i)[kFaceFlagInts]) {
    constexpr int RF = dev::kRecFloats<D>;
    constexpr int CELLS = D == 3 ? 64 : 16;
    static_assert(G >= 2 && 4 * G <= 64 && (G & (G - 1)) == 0, "face search takes log2(G) steps; four lanes per face");
    const int lane = dev::lane_id();
    // four lanes per face: a quarter of its record each, then an axis of its cell range each
    const int k4 = lane >> 2, q4 = lane & 3;
    const bool own = k4 < G, live = own && face0 + k4 < A.F;
    constexpr int RQ = RF / 4;
    float4 part = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (live && q4 < RQ) part = reinterpret_cast<const float4 *>(A.rec)[(face0 + k4) * RQ + q4];
    if (own && q4 < RQ) *reinterpret_cast<float4 *>(&s_rec[k4][4 * q4]) = part;
    // (3D: the last word of a record is none of the face's)
    const bool fine = isfinite(part.x) && isfinite(part.y) && isfinite(part.z) && ((D == 3 && q4 == 3) || isfinite(part.w));
    const bool finite = ((__ballot(fine) >> (lane & ~3)) & 15ull) == 15ull;
    dev::wave_sync();
    int i0 = 0, n = 1;
    if (own && q4 < D) {
        // cells i with centre lo + (i + 1/2) dx in [min - h - eps, max + h + eps]
        auto axis = [&](auto x, auto y, auto z) { return q4 == 0 ? x : (q4 == 1 ? y : z); };
        const int nc = 4 * axis(A.NB[0], A.NB[1], A.NB[2]);
        const double lo = axis(A.lo[0], A.lo[1], A.lo[2]), inv = 1.0 / (double)axis(A.dx[0], A.dx[1], A.dx[2]);
        const double reach = (double)A.h + (double)axis(A.eps[0], A.eps[1], A.eps[2]);
        const double mn = s_rec[k4][D * D + q4], mx = s_rec[k4][D * D + D + q4];
        const double xl = fmin(fmax((mn - reach - lo) * inv - 0.5, -1.0), (double)nc);
        const double xh = fmax(fmin((mx + reach - lo) * inv - 0.5, (double)nc), -1.0);
        i0 = max(0, (int)ceil(xl));
        const int i1 = min(nc - 1, (int)floor(xh));
        n = live && finite ? max(0, i1 - i0 + 1) : 0;
    }
    uint64_t cnt = (uint64_t)(uint32_t)n * (uint32_t)__shfl_xor(n, 1, dev::kWave);
    cnt *= __shfl_xor(cnt, 2, dev::kWave);
    if (!own || q4 != 0) cnt = 0;   // a face's pairs count at its first lane
    if (own && q4 < 3) {
        s_i[k4][q4] = i0;
        s_i[k4][3 + q4] = n;
        if (q4 < 2) s_i[k4][8 + q4] = n > 1 ? (int)(0xFFFFFFFFu / (uint32_t)n + 1u) : 0;   // ceil(2^32 / n)
    }
    // pair indices below 2^16 (every face of the wave): quotients by the
    // per-axis cell counts as multiply-high by ceil(2^32 / n), exact there
    const bool small = __ballot(cnt > 65536u) == 0ull;
    // inclusive wave prefix of the pair counts: 32 bits hold 64 counts of 2^16
    uint64_t incl = cnt;
    if (small) {
        incl = dpp_inclusive_sum((uint32_t)cnt);
    } else {
#pragma unroll
        for (int d = 1; d < dev::kWave; d <<= 1) {
            const uint64_t y = __shfl_up(incl, d, dev::kWave);
            if (lane >= d) incl += y;
        }
    }
    const uint64_t total = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(incl >> 32), dev::kWave - 1) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)incl, dev::kWave - 1);
    if (own && q4 == 0) {
        const uint64_t pre = incl - cnt;
        s_i[k4][6] = (int)(uint32_t)pre;
        s_i[k4][7] = (int)(uint32_t)(pre >> 32);
    }
    constexpr int NAX = D == 3 ? kSatWords : 1;
    __shared__ float4 s_ax[kFaceFlagWaves][G][NAX];
    float4(*ax)[NAX] = s_ax[threadIdx.x / dev::kWave];
    if constexpr (D == 3)
        if (own) sat_axes(s_rec[k4], A.h, A.eps, q4, ax[k4]);
    dev::wave_sync();
    // pair v: its cell is tested, and flagged if its block exists at the level
    auto pair = [&](auto v) {
        using T = decltype(v);
        auto pre_of = [&](int k) -> T {
            return (T)(((uint64_t)(uint32_t)s_i[k][7] << 32) | (uint32_t)s_i[k][6]);
        };
        int k = 0;   // the last face whose pairs start at or before v
#pragma unroll
        for (int step = G / 2; step >= 1; step >>= 1)
            if (pre_of(k + step) <= v) k += step;
        const T u = v - pre_of(k);
        int g[3] = {0, 0, 0};
        const T n0 = (T)s_i[k][3], n1 = (T)s_i[k][4];
        T q0, q1;
        if (sizeof(T) == 4 && small) {
            q0 = n0 > 1 ? (T)__umulhi((uint32_t)u, (uint32_t)s_i[k][8]) : u;
            q1 = n1 > 1 ? (T)__umulhi((uint32_t)q0, (uint32_t)s_i[k][9]) : q0;
        } else {
            q0 = u / n0;
            q1 = q0 / n1;
        }
        g[0] = s_i[k][0] + (int)(u - q0 * n0);
        if constexpr (D == 3) {
            g[1] = s_i[k][1] + (int)(q0 - q1 * n1);
            g[2] = s_i[k][2] + (int)q1;
        } else {
            g[1] = s_i[k][1] + (int)q0;
        }
        float m[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int a = 0; a < D; ++a) m[a] = dev::cell_centre(A.lo[a], g[a], A.dx[a]);
        float acc = 0.0f, delta = 1.0f;   // 2D: undecided
        if constexpr (D == 3) acc = sat_gap(ax[k], m, delta);
        if (acc > delta) return;   // certainly separated
        int64_t blk = (int64_t)(g[1] >> 2) * A.NB[0] + (g[0] >> 2);
        int cell = (g[0] & 3) | ((g[1] & 3) << 2);
        if constexpr (D == 3) {
            blk += (int64_t)(g[2] >> 2) * A.NB[0] * A.NB[1];
            cell |= (g[2] & 3) << 4;
        }
        if (A.table) {
            const uint32_t t = A.table[blk];
            const int bc[3] = {g[0] >> 2, g[1] >> 2, D == 3 ? g[2] >> 2 : 0};
            if ((int64_t)t >= A.n || A.keys[t] != dev::encode_key<D>(bc, A.level, A.R[0], A.R[1]))
                return;   // no such block at this level
            blk = t;
        }
        uint8_t *cf = A.cf + (blk * CELLS + cell);
        if (*cf) return;   // flagged already
        if (!(acc < -delta)) {
            float vv[D * D];
#pragma unroll
            for (int j = 0; j < D * D; ++j) vv[j] = s_rec[k][j];
            if constexpr (D == 3) {
                if (!dev::sat_triangle(vv, m, A.h)) return;
            } else {
                if (!dev::sat_segment(vv, m, A.h)) return;
            }
        }
        *cf = 1;
        A.pmark[blk] = 1;
    };
    if (total <= 0xFFFFFFFFull) {
        const uint32_t tot = (uint32_t)total;
        for (uint32_t c0 = 0; c0 < tot; c0 += dev::kWave)
            if (c0 + lane < tot) pair((uint32_t)(c0 + lane));
    } else {
        for (uint64_t c0 = 0; c0 < total; c0 += dev::kWave)
            if (c0 + lane < total) pair((uint64_t)(c0 + lane));
    }
}

// 2:1 balance: a block of level m marked in this pass needs every neighbour
// position (faces, edges, corners) inside the domain to exist at level m;
// where it does not, the covering level-(m-1) leaf is marked.  One thread per
// (block, neighbour position).  Blocks are created as whole sibling groups,
// the children of a refined parent, so a level-m position exists exactly when
// its level-(m-1) parent exists and is not a leaf: a neighbour with the
// block's own parent exists, and any other takes one binary search, for its
// parent in level m-1 (refined: it exists; a leaf: marked; missing: the 2:1
// rule was broken below, an error).
template <int D>
__device__ __forceinline__ void ripple_item(const uint32_t *keys_m, int64_t n_m, const uint8_t *pm_m, int m,
                                            const uint32_t *keys_p, int64_t n_p, const uint8_t *leaf_p, uint8_t *pm_p,
                                            int R0, int R1, int R2, uint32_t *err, int64_t t) {
    constexpr int NNB = D == 3 ? 26 : 8;
    {
        const int64_t i = t / NNB;
        if (!pm_m[i]) return;
        int k = (int)(t % NNB);
        k += k >= NNB / 2 ? 1 : 0;   // skip the centre of the 3^D stencil
        const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = D == 3 ? k / 9 - 1 : 0;
        int c[3];
        dev::decode_key<D>(keys_m[i], m, R0, R1, c);
        const int ext[3] = {R0 << m, R1 << m, R2 << m};
        int nc[3] = {c[0] + dx, c[1] + dy, c[2] + dz};
        if (nc[0] < 0 || nc[0] >= ext[0] || nc[1] < 0 || nc[1] >= ext[1]) return;
        if (D == 3 && (nc[2] < 0 || nc[2] >= ext[2])) return;
        int pc[3] = {nc[0] >> 1, nc[1] >> 1, D == 3 ? nc[2] >> 1 : 0};
        if (pc[0] == c[0] >> 1 && pc[1] == c[1] >> 1 && (D == 2 || pc[2] == c[2] >> 1)) return;   // a sibling
        const uint32_t kp = dev::encode_key<D>(pc, m - 1, R0, R1);
        const int64_t jp = dev::lower_bound_u32(keys_p, n_p, kp);
        if (jp < n_p && keys_p[jp] == kp) {
            if (leaf_p[jp]) pm_p[jp] = 2;
        } else {
            atomicOr(err, 1u);
        }
    }
}

// Child generation of one pass (single body), for every parent level m with
// marks at once.  With pos the exclusive prefix of the level's marks, an
// existing block of level m + 1 moves up by the children of the marked parents
// before its own, pos[its parent] 2^D, and the children of marked parent i go
// where the level holds its smaller keys, plus pos[i] 2^D: no list of the
// marked keys is needed, and the parents' own bytes (leaf 0, export mark) are
// set in the same launch.
struct GrowSeg {
    const uint32_t *pkeys;   // parent level m
    const uint8_t *pm;
    const uint32_t *pos;
    uint8_t *pleaf, *pmark;  // set in place; null when the level is rebuilt in this launch (as a child level)
    int64_t pn;
    const uint32_t *ckeys;   // child level m + 1 before the pass
    const uint8_t *cleaf, *cmark, *ccf;
    const uint8_t *cpm;      // its pass marks (null: it was not tested)
    int64_t cn;
    uint32_t *nkeys;         // child level m + 1 after the pass
    uint8_t *nleaf, *nmark, *ncf;   // ncf null: no cell flags to carry or clear
};

template <int D>
__device__ __forceinline__ void grow_old_item(const GrowSeg &g, int64_t j) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    const uint32_t k = g.ckeys[j];
    const uint8_t mk = g.cpm ? g.cpm[j] : 0;
    const int64_t p = j + ((int64_t)g.pos[dev::lower_bound_u32(g.pkeys, g.pn, k >> D)] << D);
    g.nkeys[p] = k;
    g.nleaf[p] = mk ? 0 : g.cleaf[j];
    g.nmark[p] = mk ? mk : g.cmark[j];
    if (g.ncf)   // one 16- or 64-byte row: 16-byte moves
#pragma unroll
        for (int c = 0; c < CELLS / 16; ++c)
            reinterpret_cast<uint4 *>(g.ncf + p * CELLS)[c] = reinterpret_cast<const uint4 *>(g.ccf + j * CELLS)[c];
}

// Child t & (2^D - 1) of parent t >> D: its place, or -1 (the parent is not
// marked); key_out: its key.
template <int D>
__device__ __forceinline__ int64_t grow_child_item(const GrowSeg &g, int64_t t, uint32_t &key_out) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    const int64_t i = t >> D;
    const uint8_t mk = g.pm[i];
    if (!mk) return -1;
    const uint32_t ci = (uint32_t)(t & ((1 << D) - 1)), key = g.pkeys[i];
    if (ci == 0 && g.pleaf) {
        g.pleaf[i] = 0;
        g.pmark[i] = mk;
    }
    const int64_t p = dev::lower_bound_u32(g.ckeys, g.cn, key << D) + ((int64_t)g.pos[i] << D) + ci;
    key_out = (key << D) | ci;
    g.nkeys[p] = key_out;
    g.nleaf[p] = 1;
    g.nmark[p] = 0;
    if (g.ncf)
#pragma unroll
        for (int c = 0; c < CELLS / 16; ++c) reinterpret_cast<uint4 *>(g.ncf + p * CELLS)[c] = make_uint4(0u, 0u, 0u, 0u);
    return p;
}

// Marked blocks of level m: become parents (leaf 0, export mark = pass mark)
// and their keys are compacted in order into mk.
__device__ __forceinline__ void mark_parents_item(const uint32_t *keys, const uint8_t *pm, const uint32_t *pos,
                                                  uint8_t *leaf, uint8_t *mark, uint32_t *mk, int64_t i) {
    {
        const uint8_t p = pm[i];
        if (!p) return;
        leaf[i] = 0;
        mark[i] = p;
        mk[pos[i]] = keys[i];
    }
}

// Existing blocks of level m+1 move to their place in the merged list.
template <int CELLS>
__device__ __forceinline__ void merge_old_item(const uint32_t *keys, const uint8_t *leaf, const uint8_t *mark,
                                               const uint8_t *cf, const uint32_t *mk, int64_t n_mk, int D,
                                               uint32_t *nkeys, uint8_t *nleaf, uint8_t *nmark, uint8_t *ncf,
                                               int64_t i, int64_t cap = INT64_MAX) {
    {
        const uint32_t k = keys[i];
        const int64_t r = dev::lower_bound_u32(mk, n_mk, k >> D);
        const int64_t p = i + (r << D);
        if (p >= cap) return;   // batched plans: out of planned capacity (reported by the count step)
        nkeys[p] = k;
        nleaf[p] = leaf[i];
        nmark[p] = mark[i];
        if (ncf) {   // one 16- or 64-byte row: 16-byte moves
#pragma unroll
            for (int c = 0; c < CELLS / 16; ++c) {
                uint4 x;
                __builtin_memcpy(&x, cf + i * CELLS + 16 * c, 16);
                __builtin_memcpy(ncf + p * CELLS + 16 * c, &x, 16);
            }
        }
    }
}

// Children of the marked parents, placed after the existing keys below them.
template <int CELLS>
__device__ __forceinline__ void children_item(const uint32_t *mk, const uint32_t *keys_old, int64_t n_old, int D,
                                              uint32_t *nkeys, uint8_t *nleaf, uint8_t *nmark, uint8_t *ncf,
                                              int64_t t, int64_t cap = INT64_MAX) {
    {
        const int64_t pi = t >> D;
        const uint32_t ci = (uint32_t)(t & ((1 << D) - 1));
        const uint32_t parent = mk[pi];
        const int64_t below = dev::lower_bound_u32(keys_old, n_old, parent << D);
        const int64_t p = below + t;
        if (p >= cap) return;
        nkeys[p] = (parent << D) | ci;
        nleaf[p] = 1;
        nmark[p] = 0;
        if (ncf) {
            const uint4 z = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int c = 0; c < CELLS / 16; ++c) __builtin_memcpy(ncf + p * CELLS + 16 * c, &z, 16);
        }
    }
}



// ===========================================================================
// Link fractions and their adjoint (paper Sec. II-C-1)
// ===========================================================================
constexpr int kLinkCap = 32;   // staged faces per wave (LDS per wave bounds occupancy)

template <int D, int Q>
struct LinkArgs {
    dev::Faces faces;
    dev::BinGrid bins;
    const uint32_t *keys;
    int64_t n;
    int level;
    int R[3];
    float lo[3];
    float dx[3];
    float eps[3];
    // Candidate faces per block (list mode): the faces of block b are
    // list[loff[b] .. loff[b + 1]).  Null: the wave walks the bins under the
    // block instead.
    const uint32_t *loff;
    const int32_t *list;
    uint32_t list_cap;     // entries allocated for the lists (reads stay below it)
    uint64_t *node_key;    // node rows (staging rows in walk mode)
    float *q;
    int32_t *face;
};

// Candidate faces staged in LDS by one link wave: vertices (3D: and the FP32
// normal n = (b - a) x (c - a), and the two numbers of the reach test below),
// the face id and the face's near code (one bit per (axis, cell position) of
// the block it was staged for).
// With kNorms (3D) the face's L1 norms |E1|_1 and |E2|_1 are staged too (f[14],
// f[15]); without them the filter forms them again from the staged corners, with
// the same expressions, so the results are the same and the staging area is
// smaller.  That form, the row pass's, has the node pass's mask of the block's
// cells that reach the face in place of the near code and the reach test.
template <int D, int CAP = kLinkCap, bool kNorms = true>
struct LinkStaged {
    static constexpr int NF = D == 3 ? (kNorms ? 16 : 12) : 4;
    float f[NF][CAP];
    int32_t id[CAP];
    uint32_t code[kNorms ? CAP : 2 * CAP];   // (cells 0 .. 31, then 32 .. 63)
};

// Corners (3D: and normal) of record r at place pos.
template <int D, int CAP, bool kN>
AGAL_HD void link_stage_face(LinkStaged<D, CAP, kN> &S, int pos, int32_t f, const float *r) {
    S.id[pos] = f;
#pragma unroll
    for (int k = 0; k < D * D; ++k) S.f[k][pos] = r[k];
    if constexpr (D == 3) {
        const float e10 = r[3] - r[0], e11 = r[4] - r[1], e12 = r[5] - r[2];
        const float e20 = r[6] - r[0], e21 = r[7] - r[1], e22 = r[8] - r[2];
        S.f[9][pos] = e11 * e22 - e12 * e21;
        S.f[10][pos] = e12 * e20 - e10 * e22;
        S.f[11][pos] = e10 * e21 - e11 * e20;
    }
}

// c0: centre of cell (0, 0, 0) of the block the face is staged for.
//
// The reach test (link_reach) asks whether any direction's segment from a cell
// of that block can meet the face's plane: |T . n| <= S = sum_a |n_a dx_a| within
// rounding, T = o - v0.  T . n is taken as base + sum_a i_a (n_a dx_a) from cell
// (0, 0, 0)'s value, i_a the cell's position: ten operations for a pair instead of
// ~45.  It has to pass every pair that link_filter can pass, so the bound adds to
// S and to the filter's own margins MD and MT (|T|_1 at most nT over the block)
// what the two sums may differ by: the cells' centres are rounded each on its
// own (by less than eps / 2 per axis), and the two sums carry at most 2^-20 nT
// |E1|_1 |E2|_1 of rounding together (|n_a| <= |E1|_1 |E2|_1), and a few of the
// smallest denormal numbers.  A refined star of 7.3 M nodes: the pass
// that finds nodes 395 -> 390 us; with the row pass's two lanes per node, rows 966 -> 920.
template <int D, int CAP>
AGAL_HD void link_stage(LinkStaged<D, CAP, true> &S, int pos, int32_t f, const float *r,
                                           const float dx[3], const float eps[3], const float c0[3], uint32_t code) {
    link_stage_face<D>(S, pos, f, r);
    if constexpr (D == 3) {
        const float e10 = r[3] - r[0], e11 = r[4] - r[1], e12 = r[5] - r[2];
        const float e20 = r[6] - r[0], e21 = r[7] - r[1], e22 = r[8] - r[2];
        const float n0 = e11 * e22 - e12 * e21;
        const float n1 = e12 * e20 - e10 * e22;
        const float n2 = e10 * e21 - e11 * e20;
        const float n1n = fabsf(e10) + fabsf(e11) + fabsf(e12), n2n = fabsf(e20) + fabsf(e21) + fabsf(e22);
        const float T0 = c0[0] - r[0], T1 = c0[1] - r[1], T2 = c0[2] - r[2];
        const float nT = ((fabsf(T0) + fabsf(T1)) + fabsf(T2)) + 3.0f * ((dx[0] + dx[1]) + dx[2]);
        const float Sn = (fabsf(n0 * dx[0]) + fabsf(n1 * dx[1])) + fabsf(n2 * dx[2]);
        const float Se = (fabsf(n0 * eps[0]) + fabsf(n1 * eps[1])) + fabsf(n2 * eps[2]);
        const float mx = fmaxf(fmaxf(dx[0], dx[1]), dx[2]);
        // MD + MT and the two sums' rounding: 2^-20 (max dx + 2 nT) |E1| |E2|, a quarter more for their own roundings
        const float slack = 1.1920928955078125e-06f * (mx + 2.0f * nT) * (n1n * n2n);
        S.f[12][pos] = (T0 * n0 + T1 * n1) + T2 * n2;
        S.f[13][pos] = ((Sn * 1.00001f + Se) + slack) + 1e-43f;
        S.f[14][pos] = n1n;
        S.f[15][pos] = n2n;
    }
    S.code[pos] = code;
}

// x, negated when by is negative.
AGAL_HD double flip_sign(double x, double by) {
    return __builtin_bit_cast(double, __builtin_bit_cast(int64_t, x) ^ (__builtin_bit_cast(int64_t, by) & INT64_MIN));
}
AGAL_HD float flip_sign(float x, float by) {
    return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) ^ (__builtin_bit_cast(uint32_t, by) & 0x80000000u));
}
// The smaller of two numbers, NaN if one is (v_minimum3_f32).
AGAL_HD float min_nan(float a, float b) { return __builtin_elementwise_minimum(a, b); }

// FP32 filter of staged face j for a link origin o over all direction pairs.
// With T = o - a, E1 = b - a, E2 = c - a the solution of o + t D = a + u E1 +
// v E2 is det = D.n, u = D.(T x E2)/det, v = D.(E1 x T)/det, t = -(T.n)/det;
// T x E2, E1 x T and T.n do not depend on D, and D = c_i dx has entries in
// {-dx, 0, dx}, so a direction costs a few additions, and the opposite
// direction has the same u, v and t of the opposite sign; NP direction pairs
// (directions 1 + 2p, p < NP).  Each quantity carries an absolute rounding
// error bounded by 2^-21 times the product of the L1 norms of its factors
// (the direction counted as its largest cell size); margins of 2^-20 times
// those products are applied.  Returns the pairs that may meet the face (every true hit passes:
// |t| <= 1 on the face's plane and barycentrics inside).  With kSure, *sure tells whether some pair
// certainly meets it (the same tests narrowed by the margins: the exact u, v,
// 1 - u - v and 1 - |t| are then positive by at least half a margin, so the
// FP64 decision finds a hit for one of the pair's two directions).
//
// The three barycentrics, scaled by |D.n|, are held against one margin M = MU +
// MV + 2 MD through their minimum.  M also covers a D.n within MD of zero, whose
// computed sign may be wrong: a hit has |u D.n|, |v D.n| and |(u + v) D.n| <=
// |D.n| <= 2 MD, so none of the three is below -M whatever the sign; and all
// three above M means |D.n| > 3 M.  The minimum is the one that passes a NaN
// on (overflow), which fails both tests; where D.n itself may overflow (2^24 MD
// does) Ms, M for the certain pairs, is NaN.  Before, with separate comparisons,
// margins of their own and one for |D.n| <= MD (~18 instructions a pair, now ~14,
// and 17 fewer registers in the node pass): node pass of a refined star 380 us,
// now 301; row pass 787, now 756; large faces (walk mode, 768 faces on 192^3
// cells) 294, now 284.
template <int D, int NP, bool kSure, int CAP, bool kN>
AGAL_HD uint32_t link_filter(const LinkStaged<D, CAP, kN> &S, int j, const float o[3], const float dx[3],
                                                bool *sure) {
    // The pair-independent sums of margins are formed once: comparing
    // atn - (MD + MT) <= ad instead of atn <= (ad + MD) + MT (and so on) moves
    // each bound by a rounding of at most a sixteenth of a margin, within the
    // half margin the error bounds leave free.
    uint32_t cm = 0;
    bool cs = false;
    if constexpr (D == 3) {
        const float T0 = o[0] - S.f[0][j], T1 = o[1] - S.f[1][j], T2 = o[2] - S.f[2][j];
        const float e10 = S.f[3][j] - S.f[0][j], e11 = S.f[4][j] - S.f[1][j], e12 = S.f[5][j] - S.f[2][j];
        const float e20 = S.f[6][j] - S.f[0][j], e21 = S.f[7][j] - S.f[1][j], e22 = S.f[8][j] - S.f[2][j];
        const float n0 = S.f[9][j], n1 = S.f[10][j], n2 = S.f[11][j];
        float n1n, n2n;
        if constexpr (kN) {
            n1n = S.f[14][j];
            n2n = S.f[15][j];
        } else {
            n1n = fabsf(e10) + fabsf(e11) + fabsf(e12);
            n2n = fabsf(e20) + fabsf(e21) + fabsf(e22);
        }
        const float nT = fabsf(T0) + fabsf(T1) + fabsf(T2);
        const float mx_ = fmaxf(fmaxf(dx[0], dx[1]), dx[2]) * 9.5367431640625e-07f;  // dx * 2^-20
        const float MU = mx_ * nT * n2n;
        const float MV = mx_ * n1n * nT;
        const float MD = mx_ * n1n * n2n;
        const float MT = 9.5367431640625e-07f * nT * n1n * n2n;
        const float p10 = (T1 * e22 - T2 * e21) * dx[0];
        const float p11 = (T2 * e20 - T0 * e22) * dx[1];
        const float p12 = (T0 * e21 - T1 * e20) * dx[2];
        const float p20 = (e11 * T2 - e12 * T1) * dx[0];
        const float p21 = (e12 * T0 - e10 * T2) * dx[1];
        const float p22 = (e10 * T1 - e11 * T0) * dx[2];
        const float d0 = n0 * dx[0], d1 = n1 * dx[1], d2 = n2 * dx[2];
        const float atn = fabsf((T0 * n0 + T1 * n1) + T2 * n2);
        const float MDT = MD + MT, M = (MU + MV) + 2.0f * MD;
        const float Ms = M + 0.0f * (MD * 16777216.0f);
        const float t_lo = atn - MDT;   // |t| <= 1 possible: t_lo <= |D.n|
        const float t_hi = atn + MDT;   // |t| < 1 certain: t_hi <= |D.n|
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int i = 1 + 2 * p;
            const int c0 = dir_c<D>(i, 0), c1 = dir_c<D>(i, 1), c2 = dir_c<D>(i, 2);
            // signed sums over the direction's non-zero components, started at the first of them (an
            // addition to 0.0f would stay in the code: it only changes the sign of a zero, which no
            // comparison below sees)
            float den = 0.0f, nu = 0.0f, nv = 0.0f;
            bool started = false;
            auto term = [&](int c, float d, float pu, float pv) {
                if (!c) return;
                const float sd = c > 0 ? d : -d, su_ = c > 0 ? pu : -pu, sv_ = c > 0 ? pv : -pv;
                if (started) {
                    den += sd;
                    nu += su_;
                    nv += sv_;
                } else {
                    den = sd;
                    nu = su_;
                    nv = sv_;
                    started = true;
                }
            };
            term(c0, d0, p10, p20);
            term(c1, d1, p11, p21);
            term(c2, d2, p12, p22);
            const float ad = fabsf(den);
            const float su = flip_sign(nu, den);
            const float sv = flip_sign(nv, den);
            const float mn = min_nan(min_nan(su, sv), (ad - su) - sv);
            cm |= ((t_lo <= ad) & (mn >= -M)) ? (1u << p) : 0u;
            if constexpr (kSure) cs = cs | ((t_hi <= ad) & (mn > Ms));
        }
    } else {
        const float w0 = S.f[0][j] - o[0], w1 = S.f[1][j] - o[1];
        const float e0 = S.f[2][j] - S.f[0][j], e1 = S.f[3][j] - S.f[1][j];
        const float nw = fabsf(w0) + fabsf(w1), ne = fabsf(e0) + fabsf(e1);
        const float mx_ = fmaxf(dx[0], dx[1]) * 9.5367431640625e-07f;
        const float MD = mx_ * ne, MS = mx_ * nw, MW = 9.5367431640625e-07f * nw * ne;
        const float awxe = fabsf(w0 * e1 - w1 * e0);
        const float MDW = MD + MW, M = MS + 2.0f * MD;
        const float Ms = M + 0.0f * (MD * 16777216.0f);
        const float t_lo = awxe - MDW, t_hi = awxe + MDW;
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int i = 1 + 2 * p;
            const float D0 = (float)dir_c<D>(i, 0) * dx[0], D1 = (float)dir_c<D>(i, 1) * dx[1];
            const float den = D0 * e1 - D1 * e0;
            const float ad = fabsf(den);
            const float sn = w0 * D1 - w1 * D0;
            const float ss = flip_sign(sn, den);
            const float mn = min_nan(ss, ad - ss);
            cm |= ((t_lo <= ad) & (mn >= -M)) ? (1u << p) : 0u;
            if constexpr (kSure) cs = cs | ((t_hi <= ad) & (mn > Ms));
        }
    }
    if constexpr (kSure) *sure = cs;
    return cm;
}

// Whether any direction pair can pass the filter for staged face j and the cell
// at position i of the block it was staged for (3D; always in 2D).
template <int D, int CAP>
AGAL_HD bool link_reach(const LinkStaged<D, CAP, true> &S, int j, const float i[3], const float dx[3]) {
    if constexpr (D == 3) {
        const float s = ((S.f[12][j] + i[0] * (S.f[9][j] * dx[0])) + i[1] * (S.f[10][j] * dx[1])) +
                        i[2] * (S.f[11][j] * dx[2]);
        return !(fabsf(s) > S.f[13][j]);   // a NaN stays for the filter
    } else {
        return true;
    }
}

// FP64 decision for staged face j, direction Dv (the first direction of a
// pair) and origin o: the segment-triangle test (Moller-Trumbore, two-sided,
// closed) in the same expression order as the definition; returns t of Dv,
// or NaN when the line misses the face or det = 0.  The opposite direction
// hits at -t (negating D negates P, det and t exactly), so the pair has a
// link in direction Dv when t is in [0, 1] and in -Dv when -t is.
//
// The definition asks for u = un / det >= 0, u <= 1, v >= 0 and u + v <= 1, each
// rounded.  Only t is divided here; the answers are the same.  No quotient
// underflows (un and det are sums of products of FP32 numbers), so u and v have
// the signs of un and vn once det's is taken out; un / |det| rounds to more than
// 1 exactly when un > |det|; and fl(u + v) is off by at most 2^-52 near 1, so
// beyond 2^-50 |det| from un + vn = |det| the sum decides, and within it the two
// quotients are formed as the definition has them.  A division is ~14 of the
// ~130 instructions of a decision: the row pass of a refined star's 7.3 M nodes
// 838 -> 811 us, of 1.7 M nodes of D3Q19 168 -> 162.
template <int D, int CAP, bool kN>
AGAL_HD double link_decide(const LinkStaged<D, CAP, kN> &S, int j, const double o[3], const float dir[3]) {
    const double nan = __builtin_nan("");
    if constexpr (D == 3) {
        const double a0 = S.f[0][j], a1 = S.f[1][j], a2 = S.f[2][j];
        const double E1[3] = {(double)S.f[3][j] - a0, (double)S.f[4][j] - a1, (double)S.f[5][j] - a2};
        const double E2[3] = {(double)S.f[6][j] - a0, (double)S.f[7][j] - a1, (double)S.f[8][j] - a2};
        const double T[3] = {o[0] - a0, o[1] - a1, o[2] - a2};
        const double Dv[3] = {(double)dir[0], (double)dir[1], (double)dir[2]};
        const double P[3] = {Dv[1] * E2[2] - Dv[2] * E2[1], Dv[2] * E2[0] - Dv[0] * E2[2],
                             Dv[0] * E2[1] - Dv[1] * E2[0]};
        const double det = E1[0] * P[0] + E1[1] * P[1] + E1[2] * P[2];
        if (det == 0.0) return nan;
        const double ad = fabs(det);
        const double un = flip_sign(T[0] * P[0] + T[1] * P[1] + T[2] * P[2], det);
        if (un < 0.0 || un > ad) return nan;
        const double Qv[3] = {T[1] * E1[2] - T[2] * E1[1], T[2] * E1[0] - T[0] * E1[2], T[0] * E1[1] - T[1] * E1[0]};
        const double vn = flip_sign(Dv[0] * Qv[0] + Dv[1] * Qv[1] + Dv[2] * Qv[2], det);
        const double over = (un + vn) - ad, m = ad * 0x1p-50;
        if (vn < 0.0 || over > m) return nan;
        if (over >= -m && un / ad + vn / ad > 1.0) return nan;
        return (E2[0] * Qv[0] + E2[1] * Qv[1] + E2[2] * Qv[2]) / det;
    } else {
        const double a0 = S.f[0][j], a1 = S.f[1][j];
        const double e0 = (double)S.f[2][j] - a0, e1 = (double)S.f[3][j] - a1;
        const double D0 = (double)dir[0], D1 = (double)dir[1];
        const double den = D0 * e1 - D1 * e0;
        if (den == 0.0) return nan;
        const double w0 = a0 - o[0], w1 = a1 - o[1];
        const double sn = flip_sign(w0 * D1 - w1 * D0, den);
        if (!(sn >= 0.0 && sn <= fabs(den))) return nan;
        return (w0 * e1 - w1 * e0) / den;
    }
}

// Link box of sub-block sb of a wave (block coordinates sc): per axis the
// bounds of each cell position's link box (cell +- one cell, widened by eps;
// wave-uniform, kept in scalar registers), the block's link box [qlo, qhi]
// and the bins under it.
template <int D>
struct LinkBox {
    float mlo[D][4], mhi[D][4];
    float c0[3];   // centre of cell (0, 0, 0)
    float qlo[3], qhi[3];
    int ilo[3], ihi[3];
};

template <int D, int Q>
__device__ __forceinline__ void link_box(const LinkArgs<D, Q> &A, const int sc[3], LinkBox<D> &bx) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        bx.qlo[a] = bx.qhi[a] = 0.0f;
        bx.ilo[a] = bx.ihi[a] = 0;
        bx.c0[a] = a < D ? dev::uniform(dev::cell_centre(A.lo[a], 4 * sc[a], A.dx[a])) : 0.0f;
    }
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float c = dev::cell_centre(A.lo[a], 4 * sc[a] + i, A.dx[a]);
            bx.mlo[a][i] = dev::uniform((c - A.dx[a]) - A.eps[a]);
            bx.mhi[a][i] = dev::uniform((c + A.dx[a]) + A.eps[a]);
        }
#pragma unroll
    for (int a = 0; a < D; ++a) {
        bx.qlo[a] = (dev::cell_centre(A.lo[a], 4 * sc[a], A.dx[a]) - A.dx[a]) - A.eps[a];
        bx.qhi[a] = (dev::cell_centre(A.lo[a], 4 * sc[a] + 3, A.dx[a]) + A.dx[a]) + A.eps[a];
        bx.ilo[a] = dev::bin_of(bx.qlo[a], A.bins.lo[a], A.bins.s[a], A.bins.B);
        bx.ihi[a] = dev::bin_of(bx.qhi[a], A.bins.lo[a], A.bins.s[a], A.bins.B);
    }
}

// Offers the candidate faces of block blk (sub-block sb of the wave, link box
// bx) to the staging area: the faces whose bounding box meets the block's link
// box, from the block's candidate list (list mode) or from the bins under the
// box (each face once, in the first bin of (its bins) x (the box's bins)).  A
// round of 64 candidates can keep more faces than the area holds: they are
// staged in pieces that fit, flush(count) testing and emptying the area
// between pieces (whole wave).  Returns the number of faces left staged.
template <int D, int Q, class Flush>
__device__ __forceinline__ int link_gather(const LinkArgs<D, Q> &A, int64_t blk, int sb, const LinkBox<D> &bx,
                                           LinkStaged<D> &S, int count, Flush &&flush) {
    const int lane = dev::lane_id();
    auto face_code = [&](const float *bb) -> uint32_t {   // bb: min[D], max[D]
        uint32_t c = 0;
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                c |= (bb[a] <= bx.mhi[a][i] && bb[D + a] >= bx.mlo[a][i]) ? (1u << (4 * a + i)) : 0u;
        return c << (sb * 4 * D);
    };
    auto round = [&](bool has, int32_t f, const int *cur) {
        bool keep = false;
        float r[dev::kRecFloats<D>];
        const float *bb = r + D * D;   // min then max
        if (has) {
            dev::load_rec<D>(A.faces.rec, f, r);
            keep = true;
#pragma unroll
            for (int a = 0; a < D; ++a) {
                if (cur) {
                    const int fb = max(dev::bin_of(bb[a], A.bins.lo[a], A.bins.s[a], A.bins.B), bx.ilo[a]);
                    keep = keep && fb == cur[a];
                }
                keep = keep && bb[a] <= bx.qhi[a] && bb[D + a] >= bx.qlo[a];
            }
        }
        uint64_t rest = __ballot(keep);
        while (rest) {
            if (count > 0 && count + __popcll(rest) > kLinkCap) {
                flush(count);
                count = 0;
            }
            const bool now = ((rest >> lane) & 1ull) && dev::lanes_below(rest) < kLinkCap - count;
            const uint64_t part = __ballot(now);
            rest &= ~part;
            const int pos = count + dev::lanes_below(part);
            count += __popcll(part);
            if (now) link_stage<D>(S, pos, f, r, A.dx, A.eps, bx.c0, face_code(bb));
        }
    };
    if (A.list) {
        const uint32_t s0 = A.loff[blk], s1 = min(A.loff[blk + 1], A.list_cap);   // wave-uniform
        for (uint32_t c0 = s0; c0 < s1; c0 += dev::kWave) {
            const uint32_t e = c0 + (uint32_t)lane;
            const int32_t f = e < s1 ? A.list[e] : -1;
            round(f >= 0 && f < A.faces.F, f, nullptr);
        }
    } else {
        for_candidates(A.bins, bx.ilo, bx.ihi, [&](bool has, int32_t f, const int cur[3]) -> bool {
            round(has, f, cur);
            return true;
        });
    }
    return count;
}

// One wave: finest-level blocks first .. first + 64/4^D - 1 of A; best hit
// per (cell, direction) and the node rows.  out.rows(blk, count) places each
// block's nodes: it returns the first row for them (and records the count),
// or -1 when it has no room; rows are written in cell order.
template <int D, int Q, class Out>
__device__ __forceinline__ void links_wave(const LinkArgs<D, Q> &A, int64_t first, Out &out) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    constexpr int BPW = 64 / CELLS;
    constexpr int NP = (Q - 1) / 2;            // direction pairs
    __shared__ LinkStaged<D> S;
    __shared__ float s_dir[NP][3];   // D = c * dx of each direction pair's first direction
    const int lane = threadIdx.x;
    if (lane < NP)
        for (int a = 0; a < 3; ++a) s_dir[lane][a] = (float)dir_c<D>(1 + 2 * lane, a) * A.dx[a];
    const int64_t blk = first + lane / CELLS;
    const bool valid = blk < A.n;
    const int cell = lane % CELLS;
    const int sub = lane / CELLS;
    int bc[3] = {0, 0, 0};
    uint32_t key = 0;
    if (valid) {
        key = A.keys[blk];
        dev::decode_key<D>(key, A.level, A.R[0], A.R[1], bc);
    }
    float o[3];
    o[0] = dev::cell_centre(A.lo[0], 4 * bc[0] + (cell & 3), A.dx[0]);
    o[1] = dev::cell_centre(A.lo[1], 4 * bc[1] + ((cell >> 2) & 3), A.dx[1]);
    o[2] = D == 3 ? dev::cell_centre(A.lo[2], 4 * bc[2] + (cell >> 4), A.dx[2]) : 0.0f;
    // Near test of a staged face against the lane's link box (cell +- one cell
    // per axis), separable by axis: a staged face carries one bit per (axis,
    // position) of the block it was staged for, from the same FP32 expressions
    // every lane would use, and a lane tests it with one AND against its own D
    // bits.  (2D: block t of the wave uses bits 8t..8t+7; a face near a cell of
    // block t lies in block t's link box, so it is staged, and coded, for t.)
    const int pos3[3] = {cell & 3, (cell >> 2) & 3, cell >> 4};
    const float fpos[3] = {(float)pos3[0], (float)pos3[1], (float)pos3[2]};
    uint32_t lbits = 0;
#pragma unroll
    for (int a = 0; a < D; ++a) lbits |= 1u << (sub * 4 * D + 4 * a + pos3[a]);

    // Best hit per (lane, direction) as one 64-bit key: the FP32 bits of t
    // (t >= 0, so they order like t) above the face id, so the smaller key is
    // the smaller t and, between equal t, the lower face id.
    __shared__ unsigned long long s_best[Q - 1][64];
    __shared__ float s_o[64][3];
    // Work waits in two queues and is taken 64 at a time, one item per lane,
    // whichever lanes queued it: (lane, staged face) pairs for the FP32
    // filter, then (lane, staged face, direction pair) for the FP64 decision.
    constexpr int TCAP = 128;   // below 64 after a take, at most 64 added per step
    __shared__ uint32_t s_qa[TCAP];
    __shared__ uint32_t s_qb[TCAP];
#pragma unroll
    for (int i = 0; i < Q - 1; ++i) s_best[i][lane] = ~0ull;
#pragma unroll
    for (int a = 0; a < 3; ++a) s_o[lane][a] = o[a];
    int na = 0, nb = 0;   // wave-uniform queue lengths

    // A hit at t64 for direction i of lane l.  t is decided in FP64 and kept
    // rounded to FP32 (a negative zero as zero).
    auto consider = [&](int i, int l, double t64, int32_t f) {
        if (!(t64 >= 0.0 && t64 <= 1.0)) return;
        const float t = (float)t64 + 0.0f;
        const unsigned long long k = ((unsigned long long)__float_as_uint(t) << 32) | (uint32_t)f;
        atomicMin(&s_best[i][l], k);
    };
    auto take_b = [&](int take) {   // wave-uniform
        __syncthreads();
        const uint32_t item = lane < take ? s_qb[lane] : 0u;
        __syncthreads();
        if (lane < nb - take) s_qb[lane] = s_qb[take + lane];
        nb -= take;
        if (lane < take) {
            const int l = (int)(item >> 20);
            const int j = (int)((item >> 13) & 127u);
            const int p = (int)(item & 31u);
            const double ol[3] = {s_o[l][0], s_o[l][1], s_o[l][2]};
            const double t = link_decide<D>(S, j, ol, s_dir[p]);
            consider(2 * p, l, t, S.id[j]);        // direction 1 + 2p
            consider(2 * p + 1, l, -t, S.id[j]);   // its opposite
        }
    };
    auto take_a = [&](int take) {   // wave-uniform
        __syncthreads();
        const uint32_t item = lane < take ? s_qa[lane] : 0u;
        __syncthreads();
        if (lane < na - take) s_qa[lane] = s_qa[take + lane];
        na -= take;
        const int l = (int)(item >> 7), j = (int)(item & 127u);
        uint32_t cm = 0;
        if (lane < take) {
            const float ol[3] = {s_o[l][0], s_o[l][1], s_o[l][2]};
            cm = link_filter<D, NP, false, kLinkCap>(S, j, ol, A.dx, nullptr);
        }
        while (__ballot(cm != 0)) {
            const bool has = cm != 0;
            int p = 0;
            if (has) {
                p = __builtin_ctz(cm);
                cm &= cm - 1u;
            }
            const uint64_t m = __ballot(has);
            if (has) s_qb[nb + dev::lanes_below(m)] = ((uint32_t)l << 20) | ((uint32_t)j << 13) | (uint32_t)p;
            nb += __popcll(m);
            if (nb >= 64) take_b(64);
        }
    };

    // Staged faces are visited in batches of 64: each lane marks the faces
    // whose box meets its link box (broadcast LDS reads), then queues its own
    // marked faces that its links can reach.  Both queues are emptied before
    // the staging area is refilled.
    auto test_staged = [&](int n) {
        __syncthreads();
        for (int j0 = 0; j0 < n; j0 += 64) {
            const int jn = min(64, n - j0);
            uint64_t nm = 0;
            if (valid)
            for (int jj = 0; jj < jn; jj += 4) {
                const uint32_t cs[4] = {S.code[j0 + jj], S.code[j0 + jj + 1], S.code[j0 + jj + 2],
                                        S.code[j0 + jj + 3]};
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    nm |= ((cs[u] & lbits) == lbits && jj + u < jn) ? (1ull << (jj + u)) : 0ull;
            }
            while (__ballot(nm != 0)) {
                bool pass = false;
                int j = 0;
                if (nm) {
                    j = j0 + __builtin_ctzll(nm);
                    nm &= nm - 1ull;
                    pass = link_reach<D>(S, j, fpos, A.dx);
                }
                const uint64_t m = __ballot(pass);
                if (pass) s_qa[na + dev::lanes_below(m)] = ((uint32_t)lane << 7) | (uint32_t)j;
                na += __popcll(m);
                if (na >= 64) take_a(64);
            }
        }
        if (na > 0) take_a(na);
        if (nb > 0) take_b(nb);
        __syncthreads();
    };

    int count = 0;
    for (int sb = 0; sb < BPW; ++sb) {
        if (first + sb >= A.n) break;
        int sc[3];
        sc[0] = __shfl(bc[0], sb * CELLS, 64);
        sc[1] = __shfl(bc[1], sb * CELLS, 64);
        sc[2] = __shfl(bc[2], sb * CELLS, 64);
        LinkBox<D> bx;
        link_box<D, Q>(A, sc, bx);
        count = link_gather<D, Q>(A, first + sb, sb, bx, S, count, test_staged);
    }
    if (count > 0) test_staged(count);

    uint64_t best[Q - 1];
    bool has = false;
#pragma unroll
    for (int i = 0; i < Q - 1; ++i) {
        best[i] = s_best[i][lane];
        has = has || best[i] != ~0ull;
    }
    // ordered compaction of the cells that have a link
    has = has && valid;
    const uint64_t hm = __ballot(has);
    // rank inside the block: lanes of this block below this lane that have a link
    uint64_t bm = hm;
    if constexpr (CELLS < 64) bm = (hm >> (sub * CELLS)) & ((1ull << CELLS) - 1);
    int64_t row0 = 0;
    if (valid && cell == 0) row0 = out.rows(blk, (uint32_t)__popcll(bm));
    row0 = __shfl(row0, sub * CELLS, 64);
    // a negative first row: the output policy ran out of capacity
    const int64_t node = has && row0 >= 0 ? row0 + __popcll(bm & ((1ull << cell) - 1)) : -1;
    if (node >= 0) {
        A.node_key[node] = (uint64_t)key * CELLS + (uint64_t)cell;
        float *qr = A.q + node * Q;
        int32_t *fr = A.face + node * Q;
        qr[0] = -1.0f;
        fr[0] = -1;
#pragma unroll
        for (int i = 0; i < Q - 1; ++i) {
            const bool hit = best[i] != ~0ull;
            qr[i + 1] = hit ? __uint_as_float((uint32_t)(best[i] >> 32)) : -1.0f;
            fr[i + 1] = hit ? (int32_t)(uint32_t)best[i] : -1;
        }
    }
}

// Near code of a face box bb (min[D], max[D]) for the block at block
// coordinates bc: bit 4a + i is set when the link box of cell position i along
// axis a (centre +- one cell, widened by eps) meets the box along a -- the
// same FP32 expressions as link_box.  Per lane (the block need not be
// wave-uniform).
template <int D, int Q>
AGAL_HD uint32_t link_code_at(const LinkArgs<D, Q> &A, const int bc[3], const float *bb) {
    uint32_t c = 0;
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float m = dev::cell_centre(A.lo[a], 4 * bc[a] + i, A.dx[a]);
            const float lo_ = (m - A.dx[a]) - A.eps[a], hi_ = (m + A.dx[a]) + A.eps[a];
            c |= (bb[a] <= hi_ && bb[D + a] >= lo_) ? (1u << (4 * a + i)) : 0u;
        }
    return c;
}

// Cells (bit x + 4 y + 16 z) of a block that a face's near code covers.
template <int D>
AGAL_HD uint64_t code_cells(uint32_t c) {
    const uint32_t y = (c >> 4) & 15u, z = (c >> 8) & 15u;
    const uint32_t rows = ((y & 1u) | ((y & 2u) << 3) | ((y & 4u) << 6) | ((y & 8u) << 9)) * (c & 15u);   // 16 bits
    if constexpr (D == 2) return rows;
    const uint32_t lo = ((z & 1u) | ((z & 2u) << 15)) * rows, hi = (((z >> 2) & 1u) | ((z >> 2) & 2u) << 15) * rows;
    return ((uint64_t)hi << 32) | lo;
}

// Cells of its block that staged face j passes link_reach for (3D; all in 2D):
// the same sums, each formed once for the cells that share it.
template <int D, int CAP>
AGAL_HD uint64_t reach_cells(const LinkStaged<D, CAP, true> &S, int j, const float dx[3]) {
    if constexpr (D == 2) {
        return ~0ull;
    } else {
        const float a = S.f[9][j] * dx[0], b = S.f[10][j] * dx[1], c = S.f[11][j] * dx[2], bound = S.f[13][j];
        uint32_t m[2] = {0u, 0u};
#pragma unroll
        for (int x = 0; x < 4; ++x) {
            const float sx = S.f[12][j] + (float)x * a;
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                const float sy = sx + (float)y * b;
#pragma unroll
                for (int z = 0; z < 4; ++z)
                    m[z / 2] |= fabsf(sy + (float)z * c) > bound ? 0u : 1u << (x + 4 * y + 16 * (z & 1));
            }
        }
        return ((uint64_t)m[1] << 32) | m[0];
    }
}

// Node pass of list mode: which finest-level cells have at least one link.
// Work is taken from the candidate lists 64 (face, block) entries at a time
// (persistent loop over the entries), one per lane: a lane finds the cells of
// its block whose link box meets its face's box and from which a direction can
// reach its plane -- exactly the pairs the row pass filters -- as a 64-bit mask,
// and the lanes give up a cell each in turn, without those known to have a link
// already, to a queue.  (Listing every near pair, 64 at a time and one per lane,
// took ~80 instructions for 64 pairs, of which most reach no plane; the masks take
// ~280 for a window's 64 entries: a refined star 295 -> 254 us, six bodies 306 ->
// 238, a moving sphere 76 -> 67.)
// 64 pairs at a time go from the queue to the FP32 filter narrowed and widened by
// its margins: a certain hit sets the cell's bit in its block's mask, a
// possible one is decided in FP64 exactly as the row pass decides it.  So a
// block's mask is the set of its cells for which the row pass finds a hit.
// The 64 entries of a window belong to a few blocks (the lists are in block
// order): each block's mask is read once into LDS, hits are ORed there, and
// the new bits go out with one device atomic per block at the window's end
// (device-scope atomics are performed past the per-XCD L2, so one per hit
// costs memory-side traffic).
// mask: one 64-bit word per block, zeroed.  lword: on entry each entry's block
// (high half) and face, on return its mask of cells, 0 for an entry without a face
// or block; list (written): its face.
template <int D, int Q>
__device__ __forceinline__ void links_nodes_entries(const LinkArgs<D, Q> &A, int32_t *list, uint64_t *lword,
                                                    unsigned long long *mask, int64_t wg, int64_t nwg) {
    constexpr int NP = (Q - 1) / 2;
    constexpr int RF = dev::kRecFloats<D>;
    __shared__ LinkStaged<D, 64> S;
    __shared__ float s_dir[NP][3];
    __shared__ int s_bc[64][3];        // its block coordinates
    __shared__ uint32_t s_head[64];    // first entry of the window with the same block
    __shared__ unsigned long long s_m[64];   // at a block's first entry: its mask as known to the wave
    constexpr int QCAP = 128;
    __shared__ uint32_t s_q[QCAP];     // queued pairs: entry << 8 | cell
    const int lane = dev::lane_id();
    if (lane < NP)
        for (int a = 0; a < 3; ++a) s_dir[lane][a] = (float)dir_c<D>(1 + 2 * lane, a) * A.dx[a];
    const uint32_t total = min(A.loff[A.n], A.list_cap);
    int nq = 0;   // wave-uniform queue length

    for (int64_t w = wg; w * 64 < (int64_t)total; w += nwg) {
        const uint32_t e = (uint32_t)(w * 64) + (uint32_t)lane;
        uint32_t bits = 0, b = 0;
        bool known = false;   // its block is one of the level
        unsigned long long cells = 0ull;   // of this lane's entry, not given up yet
        int bc[3] = {0, 0, 0};
        if (e < total) {
            const uint64_t word = lword[e];
            const int32_t f = (int32_t)(uint32_t)word;
            b = (uint32_t)(word >> 32);
            known = (int64_t)b < A.n;
            if (f >= 0 && f < A.faces.F && known) {
                float r[RF];
                dev::load_rec<D>(A.faces.rec, f, r);
                dev::decode_key<D>(A.keys[b], A.level, A.R[0], A.R[1], bc);
                bits = link_code_at<D, Q>(A, bc, r + D * D);
                float c0[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int a = 0; a < D; ++a) c0[a] = dev::cell_centre(A.lo[a], 4 * bc[a], A.dx[a]);
                link_stage<D>(S, lane, f, r, A.dx, A.eps, c0, bits);
                cells = code_cells<D>(bits) & reach_cells<D>(S, lane, A.dx);
            }
            list[e] = f;
            lword[e] = cells;
        }
        s_bc[lane][0] = bc[0];
        s_bc[lane][1] = bc[1];
        s_bc[lane][2] = bc[2];
        const bool live = known;
        const uint32_t prev_b = (uint32_t)__shfl_up((int)b, 1, dev::kWave);
        const bool head = live && (lane == 0 || prev_b != b);
        const uint64_t heads = __ballot(head);
        const uint64_t upto = lane == dev::kWave - 1 ? ~0ull : ((2ull << lane) - 1ull);
        const uint64_t hb = heads & upto;
        const int my_head = hb ? 63 - __clzll((long long)hb) : lane;
        s_head[lane] = (uint32_t)my_head;
        const unsigned long long m0 = head ? mask[b] : 0ull;
        s_m[lane] = m0;
        dev::wave_sync();
        // one work loop: queue a cell of every lane that has one still open, and
        // decide 64 queued pairs whenever the queue holds that many (or the
        // cells are exhausted); each step has one place in the code
        while (true) {
            const bool more = __ballot(cells != 0ull) != 0ull;
            if (nq >= 64 || (nq > 0 && !more)) {
                const int ntake = min(nq, 64);
                dev::wave_sync();
                const uint32_t item = lane < ntake ? s_q[lane] : 0u;
                dev::wave_sync();
                if (lane < nq - ntake) s_q[lane] = s_q[ntake + lane];
                nq -= ntake;
                if (lane < ntake) {
                    const int j = (int)(item >> 8), cell = (int)(item & 255u);
                    float o[3] = {0.0f, 0.0f, 0.0f};
                    o[0] = dev::cell_centre(A.lo[0], 4 * s_bc[j][0] + (cell & 3), A.dx[0]);
                    o[1] = dev::cell_centre(A.lo[1], 4 * s_bc[j][1] + ((cell >> 2) & 3), A.dx[1]);
                    if constexpr (D == 3) o[2] = dev::cell_centre(A.lo[2], 4 * s_bc[j][2] + (cell >> 4), A.dx[2]);
                    bool hit = false;
                    uint32_t maybe = link_filter<D, NP, true, 64>(S, j, o, A.dx, &hit);
                    if (!hit && maybe) {
                        const double o64[3] = {o[0], o[1], o[2]};
                        while (maybe) {
                            const int p = __builtin_ctz(maybe);
                            maybe &= maybe - 1u;
                            const double t = link_decide<D>(S, j, o64, s_dir[p]);
                            if (t >= -1.0 && t <= 1.0) {
                                hit = true;
                                break;
                            }
                        }
                    }
                    if (hit) atomicOr(&s_m[s_head[j]], 1ull << cell);
                }
            } else if (more) {
                cells &= ~s_m[my_head];
                const bool want = cells != 0ull;
                const uint32_t item = ((uint32_t)lane << 8) | (uint32_t)(want ? __builtin_ctzll(cells) : 0);
                cells &= cells - 1ull;
                const uint64_t wm = __ballot(want);
                if (want) s_q[nq + dev::lanes_below(wm)] = item;
                nq += __popcll(wm);
            } else {
                break;
            }
        }
        dev::wave_sync();
        if (head) {
            const unsigned long long m1 = s_m[lane];
            if (m1 != m0) atomicOr(&mask[b], m1 & ~m0);
        }
        dev::wave_sync();
    }
}

// Row pass of list mode: one wave per row_nodes(Q) consecutive nodes (node k:
// block nblk[k], node key written beforehand), two lanes per node.  28 nodes
// per wave keep the best-key table at 6 KB and the wave's LDS at 8.6 KB, so
// that 18 waves fit a CU.  With the node map, a refined star's 7.3 M nodes of
// D3Q27 take 730 us with 24 nodes per wave (the same entries staged more often),
// 667 with 28 and 697 with 32 (fewer waves); D3Q19 and D2Q9 rows leave room for
// the 32 nodes that two lanes each allow: 1.7 M nodes of D3Q19 141 -> 137.5.
// Runs of 32 consecutive waves go to one XCD, as neighbours share faces and list entries:
// -> 142.8 us, a refined star 750 -> 741 (runs of 128 and 512 the same).
// row_nodes(Q) * Q words stay a multiple of four for the 16-byte row stores.  The wave stages
// the candidate entries of its blocks -- one contiguous range of the lists,
// blocks being in node order -- and every lane queues the staged faces of its
// own block that its cell reaches; the best hit per direction is kept as in
// links_wave, in a node-major table from which the wave writes its rows of q
// and face ids as flat coalesced runs.
// Bound by vector instructions (2,300 per wave with the rows' words put together
// element by element from a table without the rest direction, whose key for no
// hit needed a select; ~2,000 with the table laid out and keyed as the rows are
// written): a refined star's 7.3 M nodes 920 -> 860 us, 1.7 M nodes of D3Q19
// 182 -> 172; six bodies in one launch 720 -> 677 (there with five waves a SIMD).
// Which cells of its block an entry's face reaches comes from the node pass, a
// 64-bit mask an entry.  The near code formed here took ~190 instructions of a wave
// that has ~20 entries on its 64 lanes (star 823 -> 788 us, with 2 B an entry); the
// reach test and what is staged for it ~140 more, run for twice the pairs (star
// 732 -> 675, moving sphere 142.5 -> 130, batch 594 -> 559; the node pass 250 -> 258).
// The entries are staged at their places in the lists, so a node's are found from
// its block's offsets instead of by two binary searches in LDS (star 676 -> 644,
// moving sphere 130 -> 122, batch 543 -> 526).
constexpr int row_nodes(int q) { return q > 19 ? 28 : 32; }   // nodes per wave of the row pass
constexpr int kRowTiles = 32;   // consecutive waves of the row pass on one XCD

template <int D, int Q>
__device__ __forceinline__ void links_rows_nodes(const LinkArgs<D, Q> &A, const uint64_t *lword, const uint32_t *nblk,
                                                 const uint64_t *node_key, uint32_t nn, int64_t chunk) {
    constexpr int kRowNodes = row_nodes(Q);
    constexpr int CELLS = D == 3 ? 64 : 16;
    constexpr int NP = (Q - 1) / 2;
    constexpr int RF = dev::kRecFloats<D>;
    __shared__ LinkStaged<D, kLinkCap, false> S;
    __shared__ float s_dir[NP][3];
    static_assert(kLinkCap <= 32 && kRowNodes <= 32 && NP <= 32, "near masks are 32-bit; queue items 16-bit");
    const int lane = dev::lane_id();
    if (lane < NP)
        for (int a = 0; a < 3; ++a) s_dir[lane][a] = (float)dir_c<D>(1 + 2 * lane, a) * A.dx[a];
    const int64_t k0 = chunk * kRowNodes;
    const int nnodes = (int)min<int64_t>(kRowNodes, (int64_t)nn - k0);
    // two lanes per node while the staged faces are looked through: lane l and l + 32 have node l, and each
    // half of its faces
    const int node = lane & 31, half = lane >> 5;
    const bool valid = node < nnodes;
    const uint32_t myb = valid ? nblk[k0 + node] : 0u;
    const uint64_t nkey = valid ? node_key[k0 + node] : 0ull;
    const int cell = (int)(nkey % CELLS);
    int bc[3] = {0, 0, 0};
    if (valid) dev::decode_key<D>((uint32_t)(nkey / CELLS), A.level, A.R[0], A.R[1], bc);
    float o[3];
    o[0] = dev::cell_centre(A.lo[0], 4 * bc[0] + (cell & 3), A.dx[0]);
    o[1] = dev::cell_centre(A.lo[1], 4 * bc[1] + ((cell >> 2) & 3), A.dx[1]);
    o[2] = D == 3 ? dev::cell_centre(A.lo[2], 4 * bc[2] + (cell >> 4), A.dx[2]) : 0.0f;
    const uint32_t *node_cells = S.code + (cell >> 5) * kLinkCap;   // the staged faces' words with this cell's bit
    // the list entries of the node's block
    const uint32_t own0 = valid ? A.loff[myb] : 0u, own1 = valid ? min(A.loff[myb + 1], A.list_cap) : 0u;
    // node-major best keys (t's bits, face), a row of Q per node: the wave's rows of q and face ids as they are
    // written.  A key without a hit is (-1.0f, -1), above every hit's as unsigned numbers.
    constexpr unsigned long long kNoHit = 0xBF800000FFFFFFFFull;
    __shared__ alignas(16) unsigned long long s_best[kRowNodes * Q];
    constexpr int TCAP = 128;
    __shared__ uint16_t s_qa[TCAP];   // (node, staged entry) pairs to filter: l << 5 | j
    __shared__ uint16_t s_qb[TCAP];   // direction pairs to decide: l << 10 | j << 5 | p
    static_assert(kRowNodes % 4 == 0 && kRowNodes <= 32, "16-byte row stores, two lanes per node");
    for (int i = 2 * lane; i < kRowNodes * Q; i += 2 * dev::kWave)
        *reinterpret_cast<ulonglong2 *>(s_best + i) = make_ulonglong2(kNoHit, kNoHit);
    int na = 0, nb = 0;

    auto consider = [&](int i, int l, double t64, int32_t f) {
        if (!(t64 >= 0.0 && t64 <= 1.0)) return;
        const float t = (float)t64 + 0.0f;
        const unsigned long long key = ((unsigned long long)__float_as_uint(t) << 32) | (uint32_t)f;
        atomicMin(&s_best[l * Q + i], key);
    };
    auto take_b = [&](int take) {
        dev::wave_sync();
        const uint32_t item = lane < take ? (uint32_t)s_qb[lane] : 0u;
        dev::wave_sync();
        if (lane < nb - take) s_qb[lane] = s_qb[take + lane];
        nb -= take;
        const int l = (int)(item >> 10);   // lane l has node l's centre
        const double ol[3] = {__shfl(o[0], l, dev::kWave), __shfl(o[1], l, dev::kWave), __shfl(o[2], l, dev::kWave)};
        if (lane < take) {
            const int j = (int)((item >> 5) & 31u);
            const int p = (int)(item & 31u);
            const double t = link_decide<D>(S, j, ol, s_dir[p]);
            consider(1 + 2 * p, l, t, S.id[j]);
            consider(2 + 2 * p, l, -t, S.id[j]);
        }
    };
    auto take_a = [&](int take) {
        dev::wave_sync();
        const uint32_t item = lane < take ? (uint32_t)s_qa[lane] : 0u;
        dev::wave_sync();
        if (lane < na - take) s_qa[lane] = s_qa[take + lane];
        na -= take;
        const int l = (int)(item >> 5), j = (int)(item & 31u);
        const float ol[3] = {__shfl(o[0], l, dev::kWave), __shfl(o[1], l, dev::kWave), __shfl(o[2], l, dev::kWave)};
        uint32_t cm = 0;
        if (lane < take) cm = link_filter<D, NP, false, kLinkCap>(S, j, ol, A.dx, nullptr);
        while (__ballot(cm != 0)) {
            const bool has = cm != 0;
            int p = 0;
            if (has) {
                p = __builtin_ctz(cm);
                cm &= cm - 1u;
            }
            const uint64_t m = __ballot(has);
            if (has) s_qb[nb + dev::lanes_below(m)] = (uint16_t)((l << 10) | (j << 5) | p);
            nb += __popcll(m);
            if (nb >= 64) take_b(64);
        }
    };
    // staged entries that the lane's cell reaches (same block, its bit of their
    // masks), queued; both queues emptied before the staging area is refilled
    auto test_staged = [&](uint32_t c0, int n) {
        dev::wave_sync();
        uint32_t nm = 0;
        // the staged entries are the lists' entries c0 .. c0 + n - 1: those of the lane's block are one range of them
        const int lo = (int)max<int64_t>((int64_t)own0 - c0, 0), hi = (int)min<int64_t>((int64_t)own1 - c0, n);
        for (int j = lo + half; j < hi; j += 2) nm |= ((node_cells[j] >> (cell & 31)) & 1u) << j;
        while (__ballot(nm != 0)) {
            const bool has = nm != 0;
            const int j = has ? __builtin_ctz(nm) : 0;
            nm &= nm - 1u;
            const uint64_t m = __ballot(has);
            if (has) s_qa[na + dev::lanes_below(m)] = (uint16_t)((node << 5) | j);
            na += __popcll(m);
            if (na >= 64) take_a(64);
        }
        if (na > 0) take_a(na);
        if (nb > 0) take_b(nb);
        dev::wave_sync();
    };

    // the wave's entries: lists of blocks nblk[k0] .. nblk[k0 + nnodes - 1]
    const uint32_t b_first = (uint32_t)__builtin_amdgcn_readfirstlane((int)nblk[k0]);
    const uint32_t b_last = (uint32_t)__builtin_amdgcn_readfirstlane((int)nblk[k0 + nnodes - 1]);
    const uint32_t e0 = A.loff[b_first], e1 = min(A.loff[b_last + 1], A.list_cap);
    for (uint64_t c0 = e0; c0 < e1; c0 += kLinkCap) {
        const int n = (int)min<uint64_t>(kLinkCap, e1 - c0);
        if (lane < n) {
            const uint64_t cells = lword[c0 + lane];   // 0: not a face and block, or none of the cells reaches the face
            S.code[lane] = (uint32_t)cells;
            S.code[kLinkCap + lane] = (uint32_t)(cells >> 32);
            if (cells) {
                const int32_t f = A.list[c0 + lane];
                float r[RF];
                dev::load_rec<D>(A.faces.rec, f, r);
                link_stage_face<D>(S, lane, f, r);
            }
        }
        test_staged((uint32_t)c0, n);
    }
    dev::wave_sync();

    // rows k0 .. k0 + nnodes - 1 of q and face ids: element e of the span is
    // node e / Q, direction e % Q.  Each lane writes four consecutive elements
    // with 16-byte stores (the span starts on a 16-byte boundary: kRowNodes Q
    // words per wave), the last few elements one at a time.
    float *qd = A.q + k0 * Q;
    int32_t *fd = A.face + k0 * Q;
    const int total = nnodes * Q, total4 = total & ~3;
    for (int e = 4 * lane; e < total4; e += 256) {
        const uint4 k01 = *reinterpret_cast<const uint4 *>(s_best + e), k23 = *reinterpret_cast<const uint4 *>(s_best + e + 2);
        // rows are not read again by this pass: stored past the caches' keep policy
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        __builtin_nontemporal_store(u4{k01.y, k01.w, k23.y, k23.w}, reinterpret_cast<u4 *>(qd + e));
        __builtin_nontemporal_store(u4{k01.x, k01.z, k23.x, k23.z}, reinterpret_cast<u4 *>(fd + e));
    }
    if (lane < total - total4) {
        const int e = total4 + lane;
        qd[e] = __uint_as_float((uint32_t)(s_best[e] >> 32));
        fd[e] = (int32_t)(uint32_t)s_best[e];
    }
}

// ---------------------------------------------------------------------------
// Adjoint: a queue of live links per tile of nodes, one link per thread.
// ---------------------------------------------------------------------------
template <int D, int Q>
struct AdjArgs {
    const float *rec;      // face records (F x kRecFloats<D>)
    int64_t F;
    const int32_t *fidx;
    const uint64_t *node_key;
    const int32_t *face;
    const float *gq;
    int64_t n;
    int level;
    int R[3];
    float lo[3];
    float dx[3];
    float *grad;
};

constexpr int kAdjThreads = 256;   // nodes per tile = threads per workgroup
constexpr int kAdjWaves = kAdjThreads / 64;
constexpr int kAdjGroup = 4;      // slots per lane per wave step (queued between takes: up to 64 x this)
constexpr int kAdjHashBits = 9;
constexpr int kAdjHash = 1 << kAdjHashBits;   // per-workgroup face accumulators

// Gradient of one link's t with respect to the D vertices of its face, scaled
// by the link's weight w: out[k][a] = s_k n_a with s_k = w lambda_k / (D . n),
// lambda the barycentric coordinates of the hit and n = E1 x E2 (2D: the edge
// normal).  n belongs to the face, so the links of one face are summed as the
// D scalars s_k and multiplied by n once.
//
// face_normal is the one expression of n (per link and at the final scatter).
// link_setup sets up what depends on the face and the node only (edges,
// normal, cross products with T = o - v0); link_scalars adds the direction.
// A grazing link (|D . n| below 2^-10 of |D| |E1| |E2|) takes its barycentrics
// and denominator in FP64 from the FP32 data.
template <int D>
__device__ __forceinline__ void face_normal(const float *v, float n[3]) {
    if constexpr (D == 3) {
        const float e1[3] = {v[3] - v[0], v[4] - v[1], v[5] - v[2]};
        const float e2[3] = {v[6] - v[0], v[7] - v[1], v[8] - v[2]};
        n[0] = e1[1] * e2[2] - e1[2] * e2[1];
        n[1] = e1[2] * e2[0] - e1[0] * e2[2];
        n[2] = e1[0] * e2[1] - e1[1] * e2[0];
    } else {
        n[0] = -(v[3] - v[1]);
        n[1] = v[2] - v[0];
        n[2] = 0.0f;
    }
}

template <int D>
struct LinkFace {
    float v[dev::kRecFloats<D>];               // the face record
    float e1[3], e2[3], n[3], p1[3], p2[3];   // 3D: edges, normal, T x E2, E1 x T   (T = o - v0)
    float ee;                                  // |E1| |E2| (2D: |E|)
};

template <int D>
__device__ __forceinline__ void link_setup(const float *rec, int32_t f, const float o[3], LinkFace<D> &R) {
    dev::load_rec<D>(rec, f, R.v);
    const float *v = R.v;
    face_normal<D>(v, R.n);
    if constexpr (D == 3) {
        const float e1[3] = {v[3] - v[0], v[4] - v[1], v[5] - v[2]};
        const float e2[3] = {v[6] - v[0], v[7] - v[1], v[8] - v[2]};
        const float T[3] = {o[0] - v[0], o[1] - v[1], o[2] - v[2]};
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            R.e1[a] = e1[a];
            R.e2[a] = e2[a];
        }
        R.p1[0] = T[1] * e2[2] - T[2] * e2[1];
        R.p1[1] = T[2] * e2[0] - T[0] * e2[2];
        R.p1[2] = T[0] * e2[1] - T[1] * e2[0];
        R.p2[0] = e1[1] * T[2] - e1[2] * T[1];
        R.p2[1] = e1[2] * T[0] - e1[0] * T[2];
        R.p2[2] = e1[0] * T[1] - e1[1] * T[0];
        R.ee = sqrtf((e1[0] * e1[0] + e1[1] * e1[1]) + e1[2] * e1[2]) *
               sqrtf((e2[0] * e2[0] + e2[1] * e2[1]) + e2[2] * e2[2]);
    } else {
        const float e0 = v[2] - v[0], e1 = v[3] - v[1];
        R.e1[0] = e0;
        R.e1[1] = e1;
        R.p1[0] = v[0] - o[0];   // w = a - o
        R.p1[1] = v[1] - o[1];
        R.ee = sqrtf(e0 * e0 + e1 * e1);
    }
}

// Link of direction Dv (length dd) with weight w: s[k] = w * lambda_k / (D . n).
template <int D>
__device__ __forceinline__ void link_scalars(const float o[3], const LinkFace<D> &R, const float Dv[3], float dd,
                                             float w, float s[D]) {
    float lam[D], inv;
    const float *v = R.v;
    if constexpr (D == 3) {
        const float den = (Dv[0] * R.n[0] + Dv[1] * R.n[1]) + Dv[2] * R.n[2];
        float u, vv;
        if (fabsf(den) < 0.0009765625f * dd * R.ee) {
            double E1[3], E2[3], N[3], TT[3];
            for (int a = 0; a < 3; ++a) {
                E1[a] = (double)v[3 + a] - (double)v[a];
                E2[a] = (double)v[6 + a] - (double)v[a];
                TT[a] = (double)o[a] - (double)v[a];
            }
            N[0] = E1[1] * E2[2] - E1[2] * E2[1];
            N[1] = E1[2] * E2[0] - E1[0] * E2[2];
            N[2] = E1[0] * E2[1] - E1[1] * E2[0];
            const double den64 = (double)Dv[0] * N[0] + (double)Dv[1] * N[1] + (double)Dv[2] * N[2];
            const double P1[3] = {TT[1] * E2[2] - TT[2] * E2[1], TT[2] * E2[0] - TT[0] * E2[2],
                                  TT[0] * E2[1] - TT[1] * E2[0]};
            const double P2[3] = {E1[1] * TT[2] - E1[2] * TT[1], E1[2] * TT[0] - E1[0] * TT[2],
                                  E1[0] * TT[1] - E1[1] * TT[0]};
            u = (float)(((double)Dv[0] * P1[0] + (double)Dv[1] * P1[1] + (double)Dv[2] * P1[2]) / den64);
            vv = (float)(((double)Dv[0] * P2[0] + (double)Dv[1] * P2[1] + (double)Dv[2] * P2[2]) / den64);
            inv = (float)(1.0 / den64);
        } else {
            inv = 1.0f / den;
            u = ((Dv[0] * R.p1[0] + Dv[1] * R.p1[1]) + Dv[2] * R.p1[2]) * inv;
            vv = ((Dv[0] * R.p2[0] + Dv[1] * R.p2[1]) + Dv[2] * R.p2[2]) * inv;
        }
        lam[0] = 1.0f - u - vv;
        lam[1] = u;
        lam[2] = vv;
    } else {
        const float e0 = R.e1[0], e1 = R.e1[1];
        const float w0 = R.p1[0], w1 = R.p1[1];
        const float den = Dv[0] * R.n[0] + Dv[1] * R.n[1];
        float sp;
        if (fabsf(den) < 0.0009765625f * dd * R.ee) {
            const double E0 = (double)v[2] - (double)v[0], E1 = (double)v[3] - (double)v[1];
            const double W0 = (double)v[0] - (double)o[0], W1 = (double)v[1] - (double)o[1];
            const double dxe = (double)Dv[0] * E1 - (double)Dv[1] * E0;   // D x e
            sp = (float)((W0 * (double)Dv[1] - W1 * (double)Dv[0]) / dxe);
            inv = (float)(1.0 / ((double)Dv[0] * -E1 + (double)Dv[1] * E0));
        } else {
            const float dxe = Dv[0] * e1 - Dv[1] * e0;
            sp = (w0 * Dv[1] - w1 * Dv[0]) / dxe;
            inv = 1.0f / den;
        }
        lam[0] = 1.0f - sp;
        lam[1] = sp;
    }
#pragma unroll
    for (int k = 0; k < D; ++k) s[k] = w * lam[k] * inv;
}

// s += the DPP-moved s (control CTRL: row_shr:n = 0x110 + n, row_bcast:15 =
// 0x142, row_bcast:31 = 0x143; ROWS: the rows written) on the lanes with use;
// lanes without a source, or in rows not written, move 0.  Every lane active.
template <int CTRL, int ROWS, int N>
__device__ __forceinline__ void dpp_add(float (&s)[N], bool use) {
    float up[N];
#pragma unroll
    for (int k = 0; k < N; ++k)
        up[k] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(s[k]), CTRL, ROWS, 0xF, false));
    if (use)
#pragma unroll
        for (int k = 0; k < N; ++k) s[k] += up[k];
}

// The links of a tile of kAdjThreads nodes: the tile's face and weight rows
// are one contiguous span, read kAdjGroup slots per lane with 16-byte loads,
// the waves taking every kAdjWaves-th step of 64 kAdjGroup slots with the
// next step's loads in flight.  Each wave appends the live slots it reads (a
// face and a non-zero weight) to a queue of its own and takes 64 at a time,
// one link per lane, whatever the per-node link counts.  Queue order is slot
// order, so the links of one face tend to sit in neighbouring lanes: a
// segmented sum over runs of equal face ids leaves one lane per run, which
// adds the run's D scalars to the face's entry of the workgroup's LDS hash
// table (neighbouring nodes in key order hit few distinct faces).  At the end
// each face's sums, times its normal, are added per vertex in a second LDS hash
// table (a tile's faces share most of their vertices), and each vertex's sum
// goes out with one float atomic per coordinate: about a sixth of the global
// atomics of sending every face's share straight to its vertices.  One
// workgroup of kAdjThreads threads: nodes node0 .. node0 + kAdjThreads - 1 of A.
template <int D, int Q>
__device__ __forceinline__ void adjoint_tile(const AdjArgs<D, Q> &A, int64_t node0) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    constexpr int QCAP = (kAdjGroup + 1) * dev::kWave;   // below 64 after the takes, 64 kAdjGroup per step added
    static_assert(Q <= 32, "direction index packed in 5 bits");
    __shared__ int32_t s_key[kAdjHash];
    __shared__ float s_acc[kAdjHash][D];
    __shared__ float s_D[Q][4];   // c_i * dx per axis, then its length
    __shared__ float s_o[kAdjThreads][3];
    // the link queues (tile-local node * 32 + direction, face), reused at the
    // end for the vertex table
    __shared__ uint32_t s_qraw[2 * kAdjWaves * QCAP];
    uint32_t(*s_meta)[QCAP] = reinterpret_cast<uint32_t(*)[QCAP]>(s_qraw);
    int32_t(*s_qf)[QCAP] = reinterpret_cast<int32_t(*)[QCAP]>(s_qraw + kAdjWaves * QCAP);
    constexpr int kVHash = 512;   // vertex accumulators (power of two)
    static_assert(kVHash * (1 + D) <= 2 * kAdjWaves * QCAP, "vertex table fits in the queues");
    int32_t *v_key = reinterpret_cast<int32_t *>(s_qraw);
    float(*v_acc)[D] = reinterpret_cast<float(*)[D]>(s_qraw + kVHash);
    const int tid = threadIdx.x;
    const int lane = dev::lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(tid / dev::kWave);
    for (int i = tid; i < kAdjHash; i += kAdjThreads) {
        s_key[i] = -1;
#pragma unroll
        for (int k = 0; k < D; ++k) s_acc[i][k] = 0.0f;
    }
    if (tid < Q) {
        float d[3];
        for (int a = 0; a < 3; ++a) d[a] = (float)dir_c<D>(tid, a) * A.dx[a];
        for (int a = 0; a < 3; ++a) s_D[tid][a] = d[a];
        s_D[tid][3] = D == 3 ? sqrtf((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]) : sqrtf(d[0] * d[0] + d[1] * d[1]);
    }
    const int nn = (int)min((int64_t)kAdjThreads, A.n - node0);
    if (tid < nn) {
        const uint64_t nk = A.node_key[node0 + tid];
        const uint32_t key = (uint32_t)(nk / CELLS);
        const int cell = (int)(nk % CELLS);
        int bc[3];
        dev::decode_key<D>(key, A.level, A.R[0], A.R[1], bc);
        s_o[tid][0] = dev::cell_centre(A.lo[0], 4 * bc[0] + (cell & 3), A.dx[0]);
        s_o[tid][1] = dev::cell_centre(A.lo[1], 4 * bc[1] + ((cell >> 2) & 3), A.dx[1]);
        s_o[tid][2] = D == 3 ? dev::cell_centre(A.lo[2], 4 * bc[2] + (cell >> 4), A.dx[2]) : 0.0f;
    }
    __syncthreads();

    // Scalars s of face f (normal n) into the hash table; a full table sends
    // s_k n straight to the vertices.
    auto to_lds = [&](int32_t f, const float (&s)[D], const float (&n)[3]) {
        uint32_t h = ((uint32_t)f * 2654435761u) >> (32 - kAdjHashBits);
        for (int probe = 0; probe < kAdjHash; ++probe) {
            const int32_t prev = atomicCAS(&s_key[h], -1, f);
            if (prev == -1 || prev == f) {
#pragma unroll
                for (int k = 0; k < D; ++k) atomicAdd(&s_acc[h][k], s[k]);
                return;
            }
            h = (h + 1) & (kAdjHash - 1);
        }
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const int64_t vk = A.fidx[(int64_t)f * D + k];
#pragma unroll
            for (int a = 0; a < D; ++a) unsafeAtomicAdd(&A.grad[vk * D + a], s[k] * n[a]);
        }
    };
    uint32_t *qm = s_meta[wv];
    int32_t *qf = s_qf[wv];
    const int64_t base = node0 * Q;
    int qn = 0;   // wave-uniform queue length
    // Takes queue entries 0 .. take-1 (one per lane), moves the rest to the
    // front, computes the taken links and sums them per run of equal faces.
    auto take = [&](int cnt) {
        dev::wave_sync();
        const int t = min(cnt, dev::kWave);
        uint32_t meta = 0;
        int32_t f = -1;
        if (lane < t) {
            meta = qm[lane];
            f = qf[lane];
        }
        dev::wave_sync();
        // up to 4 x 64 entries remain: every lane moves several, in order (a
        // read of entry t + i precedes the write of entry i + 64 over it)
        for (int i = lane; i < cnt - t; i += dev::kWave) {
            qm[i] = qm[t + i];
            qf[i] = qf[t + i];
        }
        qn = cnt - t;
        float s[D], n[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int k = 0; k < D; ++k) s[k] = 0.0f;
        if (lane < t) {
            const int nl = (int)(meta >> 5), i = (int)(meta & 31u);
            const float w = A.gq[base + nl * Q + i];   // read again (just fetched): keeps queue entries at 8 B
            const float o[3] = {s_o[nl][0], s_o[nl][1], s_o[nl][2]};
            const float Dv[3] = {s_D[i][0], s_D[i][1], s_D[i][2]};
            LinkFace<D> R;
            link_setup<D>(A.rec, f, o, R);
            link_scalars<D>(o, R, Dv, s_D[i][3], w, s);
#pragma unroll
            for (int a = 0; a < 3; ++a) n[a] = R.n[a];
        }
        // segmented inclusive sum over runs of equal f (every lane active
        // here), on DPP: within each row of 16 lanes by row shifts, then
        // lane 15 of the previous row to rows 1 and 3, then lane 31 to rows 2
        // and 3, each step taken by the lanes whose run reaches its source
        const int32_t fp = __shfl_up(f, 1, dev::kWave);
        const uint64_t heads = __ballot(lane == 0 || fp != f);
        const uint64_t upto = (2ull << lane) - 1ull;   // lanes 0 .. lane (all 64 at lane 63)
        const int start = 63 - __clzll(heads & upto);
        const int rl = lane & 15;
        // within rows (row_shr:d); once no lane can use a shift, no longer one can
        if (__ballot(rl >= 1 && lane - 1 >= start)) {
            dpp_add<0x111, 0xF>(s, rl >= 1 && lane - 1 >= start);
            if (__ballot(rl >= 2 && lane - 2 >= start)) {
                dpp_add<0x112, 0xF>(s, rl >= 2 && lane - 2 >= start);
                if (__ballot(rl >= 4 && lane - 4 >= start)) {
                    dpp_add<0x114, 0xF>(s, rl >= 4 && lane - 4 >= start);
                    if (__ballot(rl >= 8 && lane - 8 >= start)) dpp_add<0x118, 0xF>(s, rl >= 8 && lane - 8 >= start);
                }
            }
        }
        const bool b15 = (lane & 16) && (lane & ~15) - 1 >= start;   // row_bcast:15 into rows 1 and 3
        if (__ballot(b15)) dpp_add<0x142, 0xA>(s, b15);
        const bool b31 = lane >= 32 && start <= 31;   // row_bcast:31 into rows 2 and 3
        if (__ballot(b31)) dpp_add<0x143, 0xC>(s, b31);
        const bool tail = lane == dev::kWave - 1 || (((heads >> lane) >> 1) & 1ull);
        if (tail && f >= 0) to_lds(f, s, n);
    };

    const int span = nn * Q;
    // Slots are read four per lane (16-byte loads of face ids and weights,
    // 256 slots per wave step; the tile's span starts on a 16-byte boundary
    // as kAdjThreads * Q is a multiple of four), the waves taking every
    // kAdjWaves-th step with the next step's loads in flight; a partial step at
    // the span's end, or rows not 16-byte aligned, go slot by slot.  Live
    // slots are queued in slot order (a lane's at its prefix of the wave's
    // live counts).
    constexpr int kV = kAdjGroup;
    static_assert(kV == 4, "int4 / float4 loads");
    static_assert((kAdjThreads * Q) % kV == 0, "tile spans start on 16-byte boundaries");
    const bool vec = ((reinterpret_cast<uintptr_t>(A.gq) | reinterpret_cast<uintptr_t>(A.face)) & 15u) == 0;
    const int nst = (span + kV * dev::kWave - 1) / (kV * dev::kWave);
    int4 nf;
    float4 nw;
    auto load = [&](int st) {
        const int s0 = st * kV * dev::kWave + kV * lane;
        if (vec && s0 + kV <= span) {
            nf = *reinterpret_cast<const int4 *>(A.face + base + s0);
            nw = *reinterpret_cast<const float4 *>(A.gq + base + s0);
        } else {
            int32_t lf[kV];
            float lw[kV];
#pragma unroll
            for (int k = 0; k < kV; ++k) {
                lf[k] = -1;
                lw[k] = 0.0f;
                if (s0 + k < span) {
                    lf[k] = A.face[base + s0 + k];
                    lw[k] = A.gq[base + s0 + k];
                }
            }
            nf = make_int4(lf[0], lf[1], lf[2], lf[3]);
            nw = make_float4(lw[0], lw[1], lw[2], lw[3]);
        }
    };
    if (wv < nst) load(wv);
    for (int st = wv; st < nst; st += kAdjWaves) {
        const int32_t f[kV] = {nf.x, nf.y, nf.z, nf.w};
        const float w[kV] = {nw.x, nw.y, nw.z, nw.w};
        if (st + kAdjWaves < nst) load(st + kAdjWaves);
        const int s0 = st * kV * dev::kWave + kV * lane;
        int nl = s0 / Q, i = s0 - nl * Q;
        uint32_t meta[kV], live = 0;
#pragma unroll
        for (int k = 0; k < kV; ++k) {
            // false past the span (f = -1)
            live |= (i != 0 && f[k] >= 0 && w[k] != 0.0f) ? 1u << k : 0u;
            meta[k] = ((uint32_t)nl << 5) | (uint32_t)i;
            if (++i == Q) {
                i = 0;
                ++nl;
            }
        }
        const uint32_t cnt = (uint32_t)__popc(live);
        const uint32_t incl = dpp_inclusive_sum(cnt);
        int at = qn + (int)(incl - cnt);
#pragma unroll
        for (int k = 0; k < kV; ++k)
            if ((live >> k) & 1u) {
                qm[at] = meta[k];
                qf[at] = f[k];
                ++at;
            }
        qn += __builtin_amdgcn_readlane((int)incl, dev::kWave - 1);
        while (qn >= dev::kWave) take(qn);
    }
    if (qn > 0) take(qn);
    __syncthreads();

    // the queues are free: vertex table
    for (int i = tid; i < kVHash; i += kAdjThreads) {
        v_key[i] = -1;
#pragma unroll
        for (int a = 0; a < D; ++a) v_acc[i][a] = 0.0f;
    }
    __syncthreads();
    for (int sl = tid; sl < kAdjHash; sl += kAdjThreads) {
        const int32_t f = s_key[sl];
        if (f < 0) continue;
        float v[dev::kRecFloats<D>], n[3];
        dev::load_rec<D>(A.rec, f, v);
        face_normal<D>(v, n);
#pragma unroll
        for (int k = 0; k < D; ++k) {
            const int32_t vk = A.fidx[(int64_t)f * D + k];
            const float sk = s_acc[sl][k];
            uint32_t h = ((uint32_t)vk * 2654435761u) >> 23;   // 9 bits: kVHash slots
            bool placed = false;
            for (int probe = 0; probe < 32; ++probe) {
                const int32_t prev = atomicCAS(&v_key[h], -1, vk);
                if (prev == -1 || prev == vk) {
#pragma unroll
                    for (int a = 0; a < D; ++a) atomicAdd(&v_acc[h][a], sk * n[a]);
                    placed = true;
                    break;
                }
                h = (h + 1) & (kVHash - 1);
            }
            if (!placed)
#pragma unroll
                for (int a = 0; a < D; ++a) unsafeAtomicAdd(&A.grad[(int64_t)vk * D + a], sk * n[a]);
        }
    }
    __syncthreads();
    for (int i = tid; i < kVHash; i += kAdjThreads) {
        const int32_t vk = v_key[i];
        if (vk < 0) continue;
#pragma unroll
        for (int a = 0; a < D; ++a) unsafeAtomicAdd(&A.grad[(int64_t)vk * D + a], v_acc[i][a]);
    }
    __syncthreads();
}

// Copy c staged node rows (key, q row, face row) from row src to row dst, as
// flat coalesced runs over one wave.
template <int Q>
__device__ __forceinline__ void compact_block(int c, int64_t src, int64_t dst, const uint64_t *__restrict__ skey,
                                              const float *__restrict__ sq, const int32_t *__restrict__ sface,
                                              uint64_t *__restrict__ key, float *__restrict__ q,
                                              int32_t *__restrict__ face) {
    if (c == 0) return;
    for (int r = threadIdx.x; r < c; r += 64) key[dst + r] = skey[src + r];
    const float *__restrict__ qs = sq + src * Q;
    const int32_t *__restrict__ fs = sface + src * Q;
    float *__restrict__ qd = q + dst * Q;
    int32_t *__restrict__ fd = face + dst * Q;
    const int n = c * Q;
    // four loads per array in flight before the stores
    int e = threadIdx.x;
    for (; e + 3 * 64 < n; e += 4 * 64) {
        float a[4];
        int32_t b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            a[u] = qs[e + u * 64];
            b[u] = fs[e + u * 64];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            qd[e + u * 64] = a[u];
            fd[e + u * 64] = b[u];
        }
    }
    for (; e < n; e += 64) {
        qd[e] = qs[e];
        fd[e] = fs[e];
    }
}


// ---- link fractions, list mode: candidate blocks per face ------------------
// Finest-level block of integer block coordinates c: at level 0 the root's
// linear index; above, the parent's first child plus the child index.  The
// parent is found in a dense table over the parents' grid (index of its first
// child; never cleared, the block found is checked against its key) or, where
// that grid is too large, in a hash table of parent keys (linear probing; slot =
// parent key << 32 | index of its first child, ~0 empty).  -1: no such block.
// The dense table needs no clearing launch and one load per probe: blocks, count
// and scatter 27 -> 20 us for 64^3 parents (20,480 faces), 130 -> 119 for 256^3
// (327,680 faces, 64 MiB of which the body touches a few); the limit is the flag
// step's own for its tables.
constexpr int64_t kParentTable = int64_t(1) << 24;   // positions

struct BlockFind {
    const uint32_t *table;    // null: the hash table
    const unsigned long long *hash;
    uint32_t hmask;   // slots - 1
    int hshift;       // 32 - log2(slots)
    int level;
    int R[3];
    const uint32_t *keys;   // the level's sorted keys (a found index is checked against them)
    int64_t n;
};

__device__ __forceinline__ uint32_t hash_slot(uint32_t key, int shift) { return (key * 2654435761u) >> shift; }

// Place of the block at coordinates p in the dense table over level m.
__device__ __forceinline__ int64_t parent_slot(const int p[3], int m, const int R[3]) {
    return ((int64_t)p[2] * (R[1] << m) + p[1]) * (R[0] << m) + p[0];
}

template <int D>
__device__ __forceinline__ int64_t find_block(const BlockFind &B, const int c[3]) {
    if (B.level == 0) {
        const int64_t i = ((int64_t)c[2] * B.R[1] + c[1]) * B.R[0] + c[0];
        return i < B.n ? i : -1;
    }
    const int p[3] = {c[0] >> 1, c[1] >> 1, D == 3 ? c[2] >> 1 : 0};
    const uint32_t pk = dev::encode_key<D>(p, B.level - 1, B.R[0], B.R[1]);
    uint32_t ci = (uint32_t)(c[0] & 1) | ((uint32_t)(c[1] & 1) << 1);
    if (D == 3) ci |= (uint32_t)(c[2] & 1) << 2;
    if (B.table) {
        const int64_t i = (int64_t)B.table[parent_slot(p, B.level - 1, B.R)] + ci;
        return i < B.n && B.keys[i] == ((pk << D) | ci) ? i : -1;
    }
    uint32_t s = hash_slot(pk, B.hshift);
    for (uint32_t probe = 0; probe <= B.hmask; ++probe) {
        const unsigned long long v = B.hash[s];
        if (v == ~0ull) return -1;
        if ((uint32_t)(v >> 32) == pk) {
            const int64_t i = (int64_t)(uint32_t)v + ci;
            return i < B.n && B.keys[i] == ((pk << D) | ci) ? i : -1;
        }
        s = (s + 1) & B.hmask;
    }
    return -1;
}

// Block i of the level: its node mask zeroed and, above level 0, the parent of
// every first child (child index 0) entered into the dense or the hash table.
template <int D>
__device__ __forceinline__ void link_block_item(const uint32_t *keys, int64_t i, uint32_t *table, int level,
                                                const int R[3], unsigned long long *hash, uint32_t hmask, int hshift,
                                                unsigned long long *mask) {
    mask[i] = 0ull;
    if (!table && !hash) return;
    const uint32_t key = keys[i];
    if (key & ((1u << D) - 1u)) return;
    const uint32_t pk = key >> D;
    if (table) {
        int p[3];
        dev::decode_key<D>(pk, level - 1, R[0], R[1], p);
        table[parent_slot(p, level - 1, R)] = (uint32_t)i;
        return;
    }
    const unsigned long long v = ((unsigned long long)pk << 32) | (uint32_t)i;
    uint32_t s = hash_slot(pk, hshift);
    for (uint32_t probe = 0; probe <= hmask; ++probe) {
        if (atomicCAS(&hash[s], ~0ull, v) == ~0ull) break;
        s = (s + 1) & hmask;
    }
}

// Block ranges of a face's candidate blocks, per axis in FP64: block b is a
// candidate when its link box [lo + (4b - 0.5) dx - eps, lo + (4b + 4.5) dx +
// eps] (FP32 in the link kernels) meets the face box widened by m = 2 eps,
// a margin above the FP32 rounding of those bounds, so the list holds every
// face the kernels' own FP32 box test keeps (and a few more, which it drops).
struct LinkFaceGrid {
    double lo[3], dx[3], m[3];
    int NB[3];
};

// One wave per kLinkFaceG faces: count (kScatter false) or write (true) each
// face into the list of every existing candidate block.  The (face, block
// position) pairs of the wave's faces are taken 64 at a time, one per lane,
// so the hash probes of many pairs are in flight together.  A face with more
// than max_coords candidate positions is skipped by both passes (the bound
// the list was sized with makes that impossible for the geometry it was
// measured on; the test keeps the writes inside the list whatever happens, and
// `over`, when given, records the skip), and so is a write at or past cap.
constexpr int kLinkFaceG = 16;

template <int D, bool kScatter>
__device__ __forceinline__ void link_faces_wave(const float *aabb, int64_t F, const LinkFaceGrid &G,
                                                const BlockFind &B, int64_t max_coords, uint32_t *cnt,
                                                const uint32_t *loff, uint32_t *cursor, uint64_t *lword,
                                                uint32_t cap, int64_t f0, uint32_t *over = nullptr) {
    __shared__ int s_i[kLinkFaceG][8];   // per face: first block per axis, positions per axis, pair prefix
    const int lane = dev::lane_id();
    uint32_t npos = 0;
    if (lane < kLinkFaceG) {
        const int64_t f = f0 + lane;
        int b0[3] = {0, 0, 0}, nb[3] = {1, 1, 1};
        bool any = f < F;
#pragma unroll
        for (int a = 0; a < D; ++a) {
            if (!any) break;
            const double mn = aabb[(int64_t)a * F + f], mx = aabb[(int64_t)(D + a) * F + f];
            double l = ceil((mn - G.lo[a] - G.m[a] - 4.5 * G.dx[a]) / (4.0 * G.dx[a]));
            double h = floor((mx - G.lo[a] + G.m[a] + 0.5 * G.dx[a]) / (4.0 * G.dx[a]));
            l = l < 0.0 ? 0.0 : l;
            h = h > (double)(G.NB[a] - 1) ? (double)(G.NB[a] - 1) : h;
            if (!(l <= h)) {   // outside the grid, or a non-finite coordinate
                any = false;
                break;
            }
            b0[a] = (int)l;
            nb[a] = (int)(h - l) + 1;
        }
        if (any && (int64_t)nb[0] * nb[1] * nb[2] <= max_coords) npos = (uint32_t)(nb[0] * nb[1] * nb[2]);
        else if (any && over) atomicOr(over, 8u);   // beyond the bound the lists were sized with
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            s_i[lane][a] = b0[a];
            s_i[lane][3 + a] = nb[a];
        }
    }
    const uint32_t incl = dev::wave_inclusive_sum(npos);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, dev::kWave - 1);
    if (lane < kLinkFaceG) s_i[lane][6] = (int)(incl - npos);
    dev::wave_sync();
    for (uint32_t c0 = 0; c0 < total; c0 += dev::kWave) {
        const uint32_t v = c0 + (uint32_t)lane;
        if (v >= total) break;
        int k = 0;   // the last face whose pairs start at or before v
#pragma unroll
        for (int step = kLinkFaceG / 2; step >= 1; step >>= 1)
            if ((uint32_t)s_i[k + step][6] <= v) k += step;
        uint32_t u = v - (uint32_t)s_i[k][6];
        int c[3];
        c[0] = s_i[k][0] + (int)(u % (uint32_t)s_i[k][3]);
        u /= (uint32_t)s_i[k][3];
        c[1] = s_i[k][1] + (int)(u % (uint32_t)s_i[k][4]);
        c[2] = s_i[k][2] + (int)(u / (uint32_t)s_i[k][4]);
        const int64_t idx = find_block<D>(B, c);
        if (idx < 0) continue;
        if constexpr (kScatter) {
            const uint32_t pos = loff[idx] + atomicAdd(&cursor[idx], 1u);
            if (pos < cap) lword[pos] = ((uint64_t)idx << 32) | (uint32_t)(f0 + k);   // one store of scattered 8 B
        } else {
            atomicAdd(&cnt[idx], 1u);
        }
    }
}

// Nodes of blocks b0 .. b0 + 63 (below n; b0 wave-uniform): every lane loads
// one block's mask, first node index and key, then the wave writes the
// blocks' nodes block by block, lane i writing cell i when it is set at
// noff + (set cells below i), so each block's nodes go out as one coalesced
// run of keys and block indices.
template <int D>
__device__ __forceinline__ void node_map_chunk(const unsigned long long *mask, const uint32_t *noff,
                                               const uint32_t *keys, int64_t b0, int64_t n, uint32_t *nblk,
                                               uint64_t *node_key) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    const int lane = dev::lane_id();
    const int64_t b = b0 + lane;
    unsigned long long m = 0ull;
    uint32_t off = 0, key = 0;
    if (b < n) {
        m = mask[b];
        off = noff[b];
        key = keys[b];
    }
    for (uint64_t live = __ballot(m != 0ull); live; live &= live - 1ull) {
        const int j = __builtin_ctzll(live);
        const unsigned long long mj = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(m >> 32), j) << 32) |
                                      (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)m, j);
        const uint32_t oj = (uint32_t)__builtin_amdgcn_readlane((int)off, j);
        const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)key, j);
        if (lane < CELLS && ((mj >> lane) & 1ull)) {
            const int64_t k = (int64_t)oj + dev::lanes_below(mj);
            nblk[k] = (uint32_t)(b0 + j);
            node_key[k] = (uint64_t)kj * CELLS + (uint64_t)lane;
        }
    }
}

}  // namespace kern
}  // namespace agal
