// The link, flag and own-bin arithmetic of kernels.hpp and device.hpp compiled
// for the host, called case by case from test_host_arithmetic.py.
#include "kernels.hpp"

using namespace agal;
using namespace agal::kern;

namespace {

// One face against all cells of one block, as the link passes take them.
template <int D>
void link_case(const float *v, const float *lo, const float *dx, const float *eps, const int *block, uint64_t *near,
               uint64_t *reach, uint64_t *reach_each, uint32_t *may, uint32_t *may_rows, uint8_t *sure, float *centre,
               double *t) {
    constexpr int Q = D == 3 ? 27 : 9, NP = (Q - 1) / 2, CELLS = D == 3 ? 64 : 16;
    LinkArgs<D, Q> A{};
    float d3[3] = {0.0f, 0.0f, 0.0f}, e3[3] = {0.0f, 0.0f, 0.0f}, c0[3] = {0.0f, 0.0f, 0.0f};
    int bc[3] = {0, 0, 0};
    float r[dev::kRecFloats<D>] = {};
    for (int k = 0; k < D * D; ++k) r[k] = v[k];
    for (int a = 0; a < D; ++a) {
        A.lo[a] = lo[a];
        A.dx[a] = d3[a] = dx[a];
        A.eps[a] = e3[a] = eps[a];
        bc[a] = block[a];
        c0[a] = dev::cell_centre(lo[a], 4 * block[a], dx[a]);
        r[D * D + a] = r[D * D + D + a] = v[a];
        for (int k = 1; k < D; ++k) {
            r[D * D + a] = fminf(r[D * D + a], v[D * k + a]);
            r[D * D + D + a] = fmaxf(r[D * D + D + a], v[D * k + a]);
        }
    }
    LinkStaged<D, 1, true> S{};
    LinkStaged<D, 1, false> R{};
    const uint32_t code = link_code_at<D, Q>(A, bc, r + D * D);
    link_stage<D>(S, 0, 0, r, d3, e3, c0, code);
    link_stage_face<D>(R, 0, 0, r);
    *near = code_cells<D>(code);
    *reach = reach_cells<D>(S, 0, d3);
    *reach_each = 0;
    for (int c = 0; c < CELLS; ++c) {
        const int pos[3] = {c & 3, (c >> 2) & 3, c >> 4};
        float o[3] = {0.0f, 0.0f, 0.0f}, fpos[3] = {0.0f, 0.0f, 0.0f};
        for (int a = 0; a < D; ++a) {
            fpos[a] = (float)pos[a];
            centre[c * D + a] = o[a] = dev::cell_centre(lo[a], 4 * block[a] + pos[a], dx[a]);
        }
        *reach_each |= link_reach<D>(S, 0, fpos, d3) ? 1ull << c : 0ull;
        bool certain = false;
        may[c] = link_filter<D, NP, true>(S, 0, o, d3, &certain);
        may_rows[c] = link_filter<D, NP, false>(R, 0, o, d3, (bool *)nullptr);
        sure[c] = certain;
        const double o64[3] = {o[0], o[1], o[2]};
        for (int p = 0; p < NP; ++p) {
            float dir[3];
            for (int a = 0; a < 3; ++a) dir[a] = (float)dir_c<D>(1 + 2 * p, a) * d3[a];
            t[c * NP + p] = link_decide<D>(S, 0, o64, dir);
        }
    }
}

template <int D>
void links_of(int64_t n, const float *v, const float *lo, const float *dx, const float *eps, const int *block,
              uint64_t *near, uint64_t *reach, uint64_t *reach_each, uint32_t *may, uint32_t *may_rows, uint8_t *sure,
              float *centre, double *t) {
    constexpr int CELLS = D == 3 ? 64 : 16, NP = D == 3 ? 13 : 4;
    for (int64_t i = 0; i < n; ++i)
        link_case<D>(v + i * D * D, lo + i * D, dx + i * D, eps + i * D, block + i * D, near + i, reach + i,
                     reach_each + i, may + i * CELLS, may_rows + i * CELLS, sure + i * CELLS, centre + i * CELLS * D,
                     t + i * CELLS * NP);
}

template <int D>
void own_of(int64_t n, const float *v, const float *p, const float *R, uint8_t *near, float *reach2, uint8_t *sure,
            uint8_t *maybe) {
    for (int64_t i = 0; i < n; ++i) {
        float r[dev::kRecFloats<D>] = {};
        for (int k = 0; k < D * D; ++k) r[k] = v[i * D * D + k];
        for (int a = 0; a < D; ++a) {
            r[D * D + a] = r[D * D + D + a] = r[a];
            for (int k = 1; k < D; ++k) {
                r[D * D + a] = fminf(r[D * D + a], r[D * k + a]);
                r[D * D + D + a] = fmaxf(r[D * D + D + a], r[D * k + a]);
            }
        }
        float m[3] = {0.0f, 0.0f, 0.0f};
        for (int a = 0; a < D; ++a) m[a] = p[i * D + a];
        near[i] = dev::near_l2<D>(r, m, R[i]);
        reach2[i] = near_reach2<D>(r, R[i]);
        bool mb = false;
        sure[i] = own_short<D>(r, m, reach2[i], 0.9999f * (R[i] * R[i]), mb);
        maybe[i] = mb;
    }
}

}  // namespace

#define EXPORT extern "C" __attribute__((visibility("default")))

EXPORT void links(int dim, int64_t n, const float *v, const float *lo, const float *dx, const float *eps,
                  const int *block, uint64_t *near, uint64_t *reach, uint64_t *reach_each, uint32_t *may,
                  uint32_t *may_rows, uint8_t *sure, float *centre, double *t) {
    if (dim == 3) links_of<3>(n, v, lo, dx, eps, block, near, reach, reach_each, may, may_rows, sure, centre, t);
    else links_of<2>(n, v, lo, dx, eps, block, near, reach, reach_each, may, may_rows, sure, centre, t);
}

EXPORT void own(int dim, int64_t n, const float *v, const float *p, const float *R, uint8_t *near, float *reach2,
                uint8_t *sure, uint8_t *maybe) {
    if (dim == 3) own_of<3>(n, v, p, R, near, reach2, sure, maybe);
    else own_of<2>(n, v, p, R, near, reach2, sure, maybe);
}

EXPORT void sat(int64_t n, const float *v, const float *m, const float *h, const float *eps, uint8_t *full, float *gap,
                float *delta) {
    for (int64_t i = 0; i < n; ++i) {
        float r[16] = {};
        for (int k = 0; k < 9; ++k) r[k] = v[9 * i + k];
        for (int a = 0; a < 3; ++a) {
            r[9 + a] = fminf(fminf(r[a], r[3 + a]), r[6 + a]);
            r[12 + a] = fmaxf(fmaxf(r[a], r[3 + a]), r[6 + a]);
        }
        float4 ax[kSatWords];
        const float e[3] = {eps[i], eps[i], eps[i]};
        for (int part = 0; part < 4; ++part) sat_axes(r, h[i], e, part, ax);
        full[i] = dev::sat_triangle(r, m + 3 * i, h[i]);
        gap[i] = sat_gap(ax, m + 3 * i, delta[i]);
    }
}

EXPORT uint64_t cells_of_code(int dim, uint32_t code) { return dim == 3 ? code_cells<3>(code) : code_cells<2>(code); }
