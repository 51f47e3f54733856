// Near-wall refinement (paper Sec. II-C-1, II-C-2; forest layout Sec. II-A).
//
// Level by level (the paper's "primary mode of access"): every cell of every
// block of the tested level that a face comes within the distance of is flagged;
// a block with a flagged cell is marked, 2:1 balance marks the coarser
// neighbours that must follow, and marked blocks are replaced by 2^D children
// merged into the next level's sorted key list.
//
// Mapping on CDNA, picked per level:
//  * face-centric, where the level's block grid fits a dense table and no face
//    spans too many cells: a wave64 takes 4 to 16 faces, their axes set up in
//    LDS, and one (face, nearby cell) pair per lane at a time; a short form of
//    the separating-axis test decides all but the pairs within its rounding,
//    and the table gives the block.
//  * cell-centric: one wave64 per 4x4x4 block (one lane per cell; four 4x4
//    blocks per wave in 2D).  The wave walks the bins under the block's query
//    box, culls each face against the box by its bounding box (lane-parallel,
//    one face per lane), compacts the survivors with a ballot into LDS, then
//    every lane runs the separating-axis test of its cell against the staged
//    faces (LDS broadcast reads) and stops once flagged.
//  * own-bin (the paper's printed form): a cell looks at its own bin's faces.
#include <algorithm>
#include <cmath>

#include "agal_internal.hpp"
#include "device.hpp"
#include "kernels.hpp"

namespace agal {
namespace {

using namespace kern;

#define AGAL_GRID_STRIDE(i, n) \
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += (int64_t)gridDim.x * blockDim.x)

template <int D, bool kDedup>
__global__ __launch_bounds__(64) void k_flag(FlagArgs<D> A) {
    flag_wave<D, kDedup>(A, (int64_t)blockIdx.x * (D == 3 ? 1 : 4));
}

template <int D>
__global__ __launch_bounds__(64) void k_flag_own_bin(FlagArgs<D> A) {
    flag_own_bin_wave<D>(A, (int64_t)blockIdx.x * (D == 3 ? 1 : 4));
}

template <int D>
__global__ void k_prop_spread(const uint32_t *keys, int64_t n, uint8_t *pm, int l, int R0, int R1, int R2) {
    AGAL_GRID_STRIDE(t, n * (D == 3 ? 26 : 8)) prop_spread_item<D>(keys, n, pm, l, R0, R1, R2, t);
}

__global__ void k_prop_commit(uint8_t *pm, int64_t n) {
    AGAL_GRID_STRIDE(i, n) if (pm[i] == 4) pm[i] = 3;
}

template <int D, int G>
__global__ __launch_bounds__(64 * kFaceFlagWaves) void k_flag_faces(FaceFlagArgs<D> A) {
    __shared__ alignas(16) float s_rec[kFaceFlagWaves][G][dev::kRecFloats<D>];
    __shared__ int s_i[kFaceFlagWaves][G][kFaceFlagInts];
    const int w = (int)threadIdx.x / dev::kWave;
    flag_faces_wave<D, G>(A, ((int64_t)blockIdx.x * kFaceFlagWaves + w) * G, s_rec[w], s_i[w]);
}

template <int D, int G>
void launch_flag_faces(const FaceFlagArgs<D> &A, hipStream_t s) {
    const int64_t per_wg = (int64_t)kFaceFlagWaves * G;
    hipLaunchKernelGGL((k_flag_faces<D, G>), dim3((unsigned)((A.F + per_wg - 1) / per_wg)), dim3(64 * kFaceFlagWaves),
                       0, s, A);
}

template <int D>
__global__ void k_ripple(const uint32_t *keys_m, int64_t n_m, const uint8_t *pm_m, int m, const uint32_t *keys_p,
                         int64_t n_p, const uint8_t *leaf_p, uint8_t *pm_p, int R0, int R1, int R2, uint32_t *err) {
    AGAL_GRID_STRIDE(t, n_m * (D == 3 ? 26 : 8))
    ripple_item<D>(keys_m, n_m, pm_m, m, keys_p, n_p, leaf_p, pm_p, R0, R1, R2, err, t);
}

// Level 0 (every root, key = x-fastest linear index, all leaves, no marks) and
// the error word, in one launch.
// (cf: the roots' cell flags to zero, cf_vec 16-byte words per root, or null;
// zero[0 .. nzero): the first pass's zeroed scratch)
__global__ void k_init_roots(uint32_t *keys, uint8_t *leaf, uint8_t *mark, int64_t n, uint32_t *err, uint4 *cf,
                             int cf_vec, uint32_t *zero, int64_t nzero) {
    AGAL_GRID_STRIDE(i, n) {
        keys[i] = (uint32_t)i;
        leaf[i] = 1;
        mark[i] = 0;
        if (cf)
            for (int j = 0; j < cf_vec; ++j) cf[i * cf_vec + j] = make_uint4(0u, 0u, 0u, 0u);
    }
    AGAL_GRID_STRIDE(i, nzero) zero[i] = 0u;
    if (blockIdx.x == 0 && threadIdx.x == 0) *err = 0u;
}

// Child generation of one pass, all parent levels in one launch (items are
// numbered across the segments by the host-made prefix: a segment's existing
// children, then its parents times 2^D), and what the next pass starts from: its
// zeroed scratch and, for the face-centric step, the block table of the level
// it tests (table[block grid position] = block index; ncf of that level's
// segment clears the cell flags).  What bounds it is the searches' chains of
// loads and, on small bodies, the launches: a thread per (parent, child), the
// unmarked ones leaving at once, in place of a launch that listed the marked
// keys, one that placed their children and one for the table (20,480 faces, 3
// passes: 33 us in 8 launches, 20 us in 3; 327,680 faces, 4 passes: 69 -> 60).
// Where most of many parents are unmarked, as in a large root grid around a small
// body, a thread per (parent, child) is mostly threads that leave: a level of more
// than kGrowByChild parents takes a thread per parent, and a wave then goes through
// the children of its marked ones (whole calls, 1,280 faces: 200^3 roots, two
// passes 834 -> 644 us, 128^3 383 -> 348; 5,000^2 roots 9,231 -> 9,048; lines at 2^14,
// 2^16 and 2^20 parents within 2 % of one another, those above 2^18 being the rarer).
constexpr int64_t kGrowByChild = int64_t(1) << 18;
__host__ __device__ inline int64_t whole_waves(int64_t n) { return (n + dev::kWave - 1) & ~int64_t(dev::kWave - 1); }
// Threads of a segment; its parts start at whole waves.
template <int D>
int64_t grow_threads(const GrowSeg &g) {
    return whole_waves(g.cn) + whole_waves(g.pn > kGrowByChild ? g.pn : g.pn << D);
}
struct GrowArgs {
    GrowSeg seg[kMaxLevels + 1];
    int64_t pre[kMaxLevels + 2];   // prefix of the segments' threads (grow_threads)
    int nseg;
    uint32_t *table;               // of segment 0's child level (null: none)
    int tlevel, R0, R1;
    uint32_t *zero;
    int64_t nzero;
};

template <int D>
__global__ void k_grow(GrowArgs a) {
    AGAL_GRID_STRIDE(i, a.pre[a.nseg]) {
        int k = 0;
        while (k + 1 < a.nseg && a.pre[k + 1] <= i) ++k;
        const GrowSeg &g = a.seg[k];
        const int64_t j = i - a.pre[k], t = j - whole_waves(g.cn);
        if (t < 0) {
            if (j < g.cn) grow_old_item<D>(g, j);
            continue;
        }
        auto child = [&](int64_t u) {
            uint32_t key = 0;
            const int64_t p = grow_child_item<D>(g, u, key);
            if (p >= 0 && k == 0 && a.table) {
                int c[3];
                dev::decode_key<D>(key, a.tlevel, a.R0, a.R1, c);
                a.table[((int64_t)c[2] * (a.R1 << a.tlevel) + c[1]) * (a.R0 << a.tlevel) + c[0]] = (uint32_t)p;
            }
        };
        if (g.pn <= kGrowByChild) {
            if (t < g.pn << D) child(t);
            continue;
        }
        // 64 parents a wave: the marked ones' lanes in order, then 64 >> D of them at a time
        const int lane = dev::lane_id();
        const bool marked = t < g.pn && g.pm[t] != 0;
        const uint64_t mm = __ballot(marked);
        const int n = __popcll(mm), below = dev::lanes_below(mm);
        const int order = __builtin_amdgcn_ds_permute((marked ? below : n + lane - below) << 2, lane);
        for (int w0 = 0; w0 < n; w0 += dev::kWave >> D) {
            const int w = w0 + (lane >> D), src = __shfl(order, w & (dev::kWave - 1), dev::kWave);
            if (w < n) child(((t - lane + src) << D) | (lane & ((1 << D) - 1)));
        }
    }
    AGAL_GRID_STRIDE(i, a.nzero) a.zero[i] = 0u;
}

unsigned grid_for(int64_t n, int threads = 256, int64_t cap = 16384) {
    int64_t b = (n + threads - 1) / threads;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

// One block of device memory, released at the end of its scope (stream ordered).
struct Scratch {
    agal_context ctx;
    hipStream_t s;
    void *base = nullptr;
    agal_status get(Slab &arrays) { return arrays.get(ctx->mem, &base, s); }
    void release() { dev_free(ctx->mem, base, s); }
    ~Scratch() { release(); }
};

// A level's arrays (n blocks; cells flags per block, 0: none) in one block.
void add_level(Slab &arrays, agal::Level &v, int64_t n, int cells) {
    v.n = n;
    arrays.add(&v.keys, (size_t)n);
    arrays.add(&v.leaf, (size_t)n);
    arrays.add(&v.mark, (size_t)n);
    if (cells) arrays.add(&v.cf, (size_t)n * cells);
}

// Which candidate walker the flag pass of n blocks takes at cell size dx and
// distance h.  The deduplicating one (many list entries per memory latency,
// repeats dropped by a hash set before any record is read) shortens the waves
// of blocks whose query box (4 dx + 2 h per axis) spans many bins; it pays for
// clearing the set and for more LDS per wave.  Measured on MI355X: it wins
// when the pass is bound by its longest waves (few blocks: the two coarsest
// levels over a 20,480-face sphere, 4096 and 3776 blocks, 80 -> 60 and
// 40 -> 27 us) and loses when the pass has blocks enough to fill the GPU many
// times (32768 blocks over a 327,680-face body: 285 -> 375 us).
template <int D>
bool flag_dedup(const agal_bins_t *bn, const float dx[3], float h, int64_t n_blocks, int n_cu) {
    double nbins = 1.0;
    for (int a = 0; a < D; ++a) nbins *= std::min((double)bn->B, std::floor((4.0 * dx[a] + 2.0 * h) * bn->s[a]) + 2.0);
    return nbins > 64.0 && n_blocks < 32 * (int64_t)n_cu;
}

// The flag pass of level l runs face-centric (one lane per (face, cell) pair
// near the face) while the level's block grid has at most the context's
// flag_table_max positions (the table is needed above level 0 only) and the
// largest face has at most kFaceFlagMaxPairs candidate cells, else
// cell-centric (one wave per block).  Measured on MI355X, face-centric wins at
// every level tried: flags 127 -> 74 us over a 20,480-face sphere (3 levels)
// and 875 -> 272 us over a 327,680-face body (4 levels), most at the coarse
// levels, whose few blocks each span hundreds of bins.
template <int D>
int64_t block_grid_size(const agal_forest_t *fo, int l) {
    int64_t e = 1;
    for (int a = 0; a < D; ++a) e *= (int64_t)fo->roots[a] << l;
    return e;
}

// Propagation steps of an own-bin pass (Sec. II-C-3): one more than the whole
// number of block lengths in the distance, 1 + floor(d / (4 dx)) with the
// smallest cell size over the axes (FP32); none with one bin, where every cell
// sees every face.  n_prop >= 0 overrides the rule.
inline int prop_steps(const agal_forest_t *fo, int l, int B, int n_prop) {
    if (n_prop >= 0) return n_prop;
    if (B <= 1) return 0;
    float dxm = fo->dx[l][0];
    for (int a = 1; a < fo->dim; ++a) dxm = std::min(dxm, fo->dx[l][a]);
    return 1 + (int)std::floor(fo->d[l] / (4.0f * dxm));
}

template <int D>
agal_status refine_impl(agal_geom g, agal_bins bn, agal_forest fo, hipStream_t s, bool own_bin = false,
                        int n_prop = -1) {
    constexpr int CELLS = D == 3 ? 64 : 16;
    constexpr int BPW = 64 / CELLS;
    agal_context ctx = g->ctx;
    const auto &mem = ctx->mem;
    uint32_t *err = nullptr;

    // level 0: every root, key = x-fastest linear index
    agal::Level &L0 = fo->lev[0];
    {
        Slab arrays;
        add_level(arrays, L0, (int64_t)fo->roots[0] * fo->roots[1] * fo->roots[2], fo->L > 0 ? CELLS : 0);
        arrays.add(&err, 1);
        AGAL_TRY(arrays.get(mem, &L0.base, s));
    }
    // Scratch of pass l, in one block: a zeroed buffer (the look-back status
    // words of the pass's scan of the marks, then the pass marks of every level
    // l' <= l), the block table for the face-centric step above level 0 (never
    // cleared: its entries are checked against the level's keys), and per level
    // l' <= l the marks' prefix.
    struct PassBuf {
        uint8_t *buf = nullptr;
        int64_t words = 0, status_bytes = 0;
        bool by_face = false;
        uint32_t *table = nullptr, *pos[kMaxLevels + 1] = {};
    };
    auto pass_buf = [&](Scratch &sc, int l, PassBuf &pb) -> agal_status {
        pb = PassBuf{};
        float eps[3];
        for (int a = 0; a < 3; ++a) eps[a] = dev::kEps * std::max(1.0f, std::max(std::fabs(fo->lo[a]), std::fabs(fo->hi[a])));
        pb.by_face = !own_bin && block_grid_size<D>(fo, l) <= ctx->flag_table_max &&
                     face_flag_pairs(D, g->max_extent, fo->d[l], fo->dx[l], eps) <= kFaceFlagMaxPairs;
        int64_t ns[kMaxLevels + 1], tot = 0;
        Slab arrays;
        for (int m = 0; m <= l; ++m) {
            ns[m] = fo->lev[m].n;
            tot += ns[m];
            arrays.add(&pb.pos[m], (size_t)ns[m] + 1);
        }
        pb.status_bytes = 8 * (scan_flags_u8_multi_tiles(ns, l + 1) + 1);
        pb.words = (pb.status_bytes + tot + 3) / 4;
        arrays.add(&pb.buf, (size_t)(4 * pb.words));
        if (l > 0 && pb.by_face && ns[l] > 0) arrays.add(&pb.table, (size_t)block_grid_size<D>(fo, l));
        return sc.get(arrays);
    };
    // the level-0 cell flags (for the face-centric step) and the first pass's
    // zeroed scratch are cleared by the root-init launch
    Scratch scratch[2] = {{ctx, s}, {ctx, s}};   // pass l's is scratch[l & 1]
    PassBuf pb;
    if (fo->L > 0) AGAL_TRY(pass_buf(scratch[0], 0, pb));
    hipLaunchKernelGGL(k_init_roots, dim3(grid_for(L0.n)), dim3(256), 0, s, L0.keys, L0.leaf, L0.mark, L0.n, err,
                       reinterpret_cast<uint4 *>(L0.cf), CELLS / 16, reinterpret_cast<uint32_t *>(pb.buf),
                       pb.words);

    dev::BinGrid bins{};
    bins.off = bn->off;
    bins.ids = bn->ids;
    bins.B = bn->B;
    bins.F = g->F;
    for (int a = 0; a < 3; ++a) {
        bins.lo[a] = bn->lo[a];
        bins.s[a] = bn->s[a];
    }
    dev::Faces faces{g->coords, g->aabb, g->rec, g->F};

    for (int l = 0; l < fo->L; ++l) {
        // the pass's zeroed scratch, block table and cell flags were prepared by
        // the launch before it (the roots' or the previous pass's children)
        agal::Level &Ll = fo->lev[l];
        uint8_t *pm[kMaxLevels + 1] = {};
        uint64_t *scan_status = reinterpret_cast<uint64_t *>(pb.buf);
        {
            int64_t at = pb.status_bytes;
            for (int m = 0; m <= l; ++m) {
                pm[m] = pb.buf + at;
                at += fo->lev[m].n;
            }
        }
        // (i) flag every cell of every level-l block
        if (Ll.n > 0) {
            FlagArgs<D> A{};
            A.faces = faces;
            A.bins = bins;
            A.keys = Ll.keys;
            A.n = Ll.n;
            A.level = l;
            for (int a = 0; a < 3; ++a) {
                A.R[a] = fo->roots[a];
                A.lo[a] = fo->lo[a];
                A.dx[a] = fo->dx[l][a];
                float sc = std::max(1.0f, std::max(std::fabs(fo->lo[a]), std::fabs(fo->hi[a])));
                A.eps[a] = dev::kEps * sc;
            }
            A.h = fo->d[l];
            A.cf = Ll.cf;
            A.pmark = pm[l];
            const int64_t waves = (Ll.n + BPW - 1) / BPW;
            ProfScope prof(ctx, "flag_sat", s);
            const bool dedup = flag_dedup<D>(bn, fo->dx[l], A.h, Ll.n, ctx->n_cu);
            if (own_bin) {
                hipLaunchKernelGGL((k_flag_own_bin<D>), dim3((unsigned)waves), dim3(64), 0, s, A);
            } else if (pb.by_face) {
                FaceFlagArgs<D> B{};
                B.rec = g->rec;
                B.F = g->F;
                for (int a = 0; a < 3; ++a) {
                    B.NB[a] = a < D ? fo->roots[a] << l : 1;
                    B.lo[a] = A.lo[a];
                    B.dx[a] = A.dx[a];
                    B.eps[a] = A.eps[a];
                }
                B.table = pb.table;
                B.keys = Ll.keys;
                B.n = Ll.n;
                B.level = l;
                B.R[0] = fo->roots[0];
                B.R[1] = fo->roots[1];
                B.h = A.h;
                B.cf = Ll.cf;
                B.pmark = pm[l];
                if (g->F > 0) {
                    const int G = face_flag_g(g->F, ctx->n_cu);
                    if (G == 16) launch_flag_faces<D, 16>(B, s);
                    else if (G == 8) launch_flag_faces<D, 8>(B, s);
                    else launch_flag_faces<D, 4>(B, s);
                }
            } else if (dedup) {
                hipLaunchKernelGGL((k_flag<D, true>), dim3((unsigned)waves), dim3(64), 0, s, A);
            } else {
                hipLaunchKernelGGL((k_flag<D, false>), dim3((unsigned)waves), dim3(64), 0, s, A);
            }
        }
        // (i') own-bin pass: the marks spread over prop_steps rings of level-l blocks
        if (own_bin && Ll.n > 0) {
            const int steps = prop_steps(fo, l, bn->B, n_prop);
            ProfScope prof(ctx, "mark_propagation", s);
            for (int st = 0; st < steps; ++st) {
                hipLaunchKernelGGL(k_prop_spread<D>, dim3(grid_for(Ll.n * (D == 3 ? 26 : 8))), dim3(256), 0, s,
                                   Ll.keys, Ll.n, pm[l], l, fo->roots[0], fo->roots[1], fo->roots[2]);
                hipLaunchKernelGGL(k_prop_commit, dim3(grid_for(Ll.n)), dim3(256), 0, s, pm[l], Ll.n);
            }
        }
        // (ii) balance ripple, level l down to 1
        for (int m = l; m >= 1; --m) {
            const agal::Level &M = fo->lev[m], &P = fo->lev[m - 1];
            if (M.n == 0) continue;
            ProfScope prof(ctx, "balance_ripple", s);
            hipLaunchKernelGGL(k_ripple<D>, dim3(grid_for(M.n * (D == 3 ? 26 : 8))), dim3(256), 0, s,
                               M.keys, M.n, pm[m], m, P.keys, P.n, P.leaf, pm[m - 1],
                               fo->roots[0], fo->roots[1], fo->roots[2], err);
        }
        // (iii) children: count marks per level, then merge level by level
        uint32_t nmark[kMaxLevels + 2] = {};
        {
            const uint8_t *ins[kMaxLevels + 1];
            int64_t ns[kMaxLevels + 1];
            for (int m = 0; m <= l; ++m) {
                ins[m] = pm[m];
                ns[m] = fo->lev[m].n;
            }
            // marks per level and the balance error word, back through mapped host memory
            AGAL_TRY(scan_flags_u8_multi(ctx, ins, pb.pos, ns, l + 1, err, nmark, s, scan_status));
        }
        if (nmark[l + 1] != 0) return fail(AGAL_ESTATE, "agal_near_wall_refine: forest lost 2:1 balance");
        // every parent level with marks at once: the new child levels are fresh
        // arrays, and a level that is both a parent (m) and a child (of m - 1)
        // takes its marks while it is copied.  The old arrays go back after the
        // launch that reads them.
        GrowArgs ga{};
        void *gone[kMaxLevels + 1] = {};
        const bool next_by_face = l + 1 < fo->L && !own_bin;   // (its cell flags are cleared; other steps write them all)
        for (int m = l; m >= 0; --m) {
            const int64_t c = nmark[m];
            agal::Level &P = fo->lev[m];
            agal::Level &C = fo->lev[m + 1];
            if (c == 0) {
                if (m + 1 == l + 1 && C.keys == nullptr) {
                    // no child level yet: an empty one keeps views valid
                    Slab arrays;
                    add_level(arrays, C, 0, m + 1 < fo->L ? CELLS : 0);
                    AGAL_TRY(arrays.get(mem, &C.base, s));
                }
                continue;
            }
            GrowSeg &gs = ga.seg[ga.nseg];
            agal::Level N;
            Slab arrays;
            add_level(arrays, N, C.n + (c << D), m + 1 < fo->L ? CELLS : 0);
            const agal_status got = arrays.get(mem, &N.base, s);
            if (got != AGAL_OK) {
                for (int k = 0; k < ga.nseg; ++k) dev_free(mem, gone[k], s);
                return got;
            }
            gs.pkeys = P.keys;
            gs.pm = pm[m];
            gs.pos = pb.pos[m];
            const bool rebuilt = m > 0 && nmark[m - 1] != 0;   // by the next segment
            gs.pleaf = rebuilt ? nullptr : P.leaf;
            gs.pmark = rebuilt ? nullptr : P.mark;
            gs.pn = P.n;
            gs.cpm = m < l ? pm[m + 1] : nullptr;
            gs.ckeys = C.keys;
            gs.cleaf = C.leaf;
            gs.cmark = C.mark;
            gs.ccf = C.cf;
            gs.cn = C.n;
            gs.nkeys = N.keys;
            gs.nleaf = N.leaf;
            gs.nmark = N.mark;
            gs.ncf = m < l || next_by_face ? N.cf : nullptr;
            ga.pre[ga.nseg + 1] = ga.pre[ga.nseg] + grow_threads<D>(gs);
            gone[ga.nseg++] = C.base;
            C = N;
        }
        agal_status st = AGAL_OK;
        PassBuf next;
        if (l + 1 < fo->L) {
            st = pass_buf(scratch[(l + 1) & 1], l + 1, next);
            ga.zero = reinterpret_cast<uint32_t *>(next.buf);
            ga.nzero = next.words;
        }
        // (marks at level l, the first segment, whenever there are any: balance marks come from flagged blocks)
        ga.table = next.table;
        ga.tlevel = l + 1;
        ga.R0 = fo->roots[0];
        ga.R1 = fo->roots[1];
        if (st == AGAL_OK && (ga.nseg > 0 || ga.nzero > 0)) {
            ProfScope prof(ctx, "child_gen", s);
            hipLaunchKernelGGL(k_grow<D>, dim3(grid_for(std::max(ga.pre[ga.nseg], ga.nzero))), dim3(256), 0, s, ga);
        }
        for (int k = 0; k < ga.nseg; ++k) dev_free(mem, gone[k], s);
        scratch[l & 1].release();
        pb = next;
        AGAL_TRY(st);
        AGAL_TRY_HIP(hipGetLastError());
    }
    return AGAL_OK;
}

}  // namespace
}  // namespace agal

using namespace agal;

extern "C" {

static agal_status near_wall_refine(agal_geom g, agal_bins b, const agal_forest_desc *desc, void *stream,
                                    agal_forest *out, bool own_bin, int n_prop) {
    if (!g || !b || !desc || !out) return fail(AGAL_EINVAL, "agal_near_wall_refine: NULL argument");
    if (b->geom_id != g->id) return fail(AGAL_ESTATE, "agal_near_wall_refine: bins were built from another geometry");
    if (b->discrete && !own_bin)
        return fail(AGAL_EINVAL, "agal_near_wall_refine: the box test needs bins by bounding box (sampled-point bins "
                                 "can miss a face that crosses a bin between its points); use the own-bin form");
    const int D = desc->dim;
    if (D != g->dim) return fail(AGAL_EINVAL, "agal_near_wall_refine: desc->dim %d != geometry dim %d", D, g->dim);
    if (desc->n_levels < 0 || desc->n_levels > kMaxLevels)
        return fail(AGAL_EINVAL, "agal_near_wall_refine: n_levels must be in [0, %d]", kMaxLevels);
    if (desc->n_levels > 0 && !desc->d_spec) return fail(AGAL_EINVAL, "agal_near_wall_refine: d_spec is NULL");
    uint64_t nroots = 1;
    for (int a = 0; a < D; ++a) {
        if (desc->roots[a] < 1) return fail(AGAL_EINVAL, "agal_near_wall_refine: roots must be >= 1");
        if (!(desc->hi[a] > desc->lo[a])) return fail(AGAL_EINVAL, "agal_near_wall_refine: hi must exceed lo");
        nroots *= (uint64_t)desc->roots[a];
    }
    if ((nroots << (D * desc->n_levels)) > ((uint64_t)1 << 32) || nroots > ((uint64_t)1 << 32))
        return fail(AGAL_EINVAL, "agal_near_wall_refine: roots * 2^(D*n_levels) exceeds the 32-bit key space");
    for (int l = 0; l < desc->n_levels; ++l)
        if (!(desc->d_spec[l] >= 0.0f) || !std::isfinite(desc->d_spec[l]))
            return fail(AGAL_EINVAL, "agal_near_wall_refine: d_spec[%d] must be finite and >= 0", l);

    auto *fo = new (std::nothrow) agal_forest_t();
    if (!fo) return fail(AGAL_ENOMEM, "agal_near_wall_refine: host allocation failed");
    fo->ctx = g->ctx;
    fo->geom_id = g->id;
    fo->stream = (hipStream_t)stream;
    fo->dim = D;
    fo->L = desc->n_levels;
    for (int a = 0; a < 3; ++a) {
        fo->roots[a] = a < D ? desc->roots[a] : 1;
        fo->lo[a] = a < D ? desc->lo[a] : 0.0f;
        fo->hi[a] = a < D ? desc->hi[a] : 1.0f;
    }
    for (int l = 0; l <= fo->L; ++l)
        for (int a = 0; a < 3; ++a) fo->dx[l][a] = (fo->hi[a] - fo->lo[a]) / (float)(4 * fo->roots[a] * (1 << l));
    for (int l = 0; l < fo->L; ++l) fo->d[l] = desc->d_spec[l];
    agal_status st = D == 3 ? refine_impl<3>(g, b, fo, (hipStream_t)stream, own_bin, n_prop)
                            : refine_impl<2>(g, b, fo, (hipStream_t)stream, own_bin, n_prop);
    if (st != AGAL_OK) {
        agal_destroy_forest(fo);
        return st;
    }
    *out = fo;
    return AGAL_OK;
}

agal_status agal_near_wall_refine(agal_geom g, agal_bins b, const agal_forest_desc *desc, void *stream,
                                  agal_forest *out) {
    return near_wall_refine(g, b, desc, stream, out, false, -1);
}

agal_status agal_near_wall_refine_own_bin(agal_geom g, agal_bins b, const agal_forest_desc *desc, int n_prop,
                                          void *stream, agal_forest *out) {
    return near_wall_refine(g, b, desc, stream, out, true, n_prop);
}

agal_status agal_forest_level_view(agal_forest f, int level, const uint32_t **d_keys, const uint8_t **d_leaf,
                                   const uint8_t **d_mark, const uint8_t **d_cell_flag, int64_t *n_blocks) {
    if (!f) return fail(AGAL_EINVAL, "agal_forest_level_view: NULL forest");
    if (level < 0 || level > f->L) return fail(AGAL_EINVAL, "agal_forest_level_view: level %d outside [0, %d]", level, f->L);
    const agal::Level &L = f->lev[level];
    if (d_keys) *d_keys = L.keys;
    if (d_leaf) *d_leaf = L.leaf;
    if (d_mark) *d_mark = L.mark;
    if (d_cell_flag) *d_cell_flag = level < f->L ? L.cf : nullptr;
    if (n_blocks) *n_blocks = L.n;
    return AGAL_OK;
}

agal_status agal_forest_info(agal_forest f, int *dim, int *n_levels) {
    if (!f) return fail(AGAL_EINVAL, "agal_forest_info: NULL forest");
    if (dim) *dim = f->dim;
    if (n_levels) *n_levels = f->L;
    return AGAL_OK;
}

void agal_destroy_forest(agal_forest f) {
    if (!f) return;
    for (int l = 0; l <= kMaxLevels; ++l) dev_free(f->ctx->mem, f->lev[l].base, f->stream);
    delete f;
}

}  // extern "C"
