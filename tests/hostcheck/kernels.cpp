// Host-compiled runs of the per-tetrahedron code in the kernels' own split of
// it: the edge form's setup in two passes (k_setup marks what it leaves,
// k_setup_rest sets the marked up one by one), and depth slabs deposited as
// values, a wavefront's lanes to a pair, alone and as a stack.  Test code only.
#include "tess_tet.h"

#include <cstring>
#include <vector>

using namespace tess;

namespace {
struct Scene {
    LatticeParams L;
    ViewParams V;
    BinParams B;
};

Scene scene(const float *const xyz[3], const int32_t dims[3], int32_t periodic, const double rot[9],
            const double extent[2], int32_t W, int32_t H, int32_t wrap, int32_t qpow, double bound) {
    Scene S;
    std::memset((void *)&S, 0, sizeof(S));
    LatticeParams &L = S.L;
    L.x = xyz[0]; L.y = xyz[1]; L.z = xyz[2];
    for (int a = 0; a < 3; ++a) {
        L.d[a] = dims[a];
        L.c[a] = periodic ? dims[a] : dims[a] - 1;
        L.box[a] = 1.0;
    }
    L.ncubes = (int64_t)L.c[0] * L.c[1] * L.c[2];
    L.periodic = periodic;
    L.tet_mass = 1.0 / (6.0 * (double)L.ncubes);
    L.v0 = 1.0 / (6.0 * (double)L.ncubes);
    L.det_v0_frac = 1e-6;
    L.det_cond_k = qpow != 1 ? -1.0 : 1e3;
    ViewParams &V = S.V;
    for (int i = 0; i < 9; ++i) V.rot[i] = rot[i];
    for (int i = 0; i < 3; ++i) V.center[i] = 0.5;
    V.u_left = -0.5 * extent[0];
    V.v_bottom = -0.5 * extent[1];
    V.inv_du = W / extent[0];
    V.inv_dv = H / extent[1];
    V.inv_W = 1.0 / W;
    V.inv_H = 1.0 / H;
    V.mass_px = 6.0 * L.tet_mass * V.inv_du * V.inv_dv;
    V.crease_bmax = V.mass_px * (double)L.ncubes / ((double)W * H) * (bound / W);
    V.W = W; V.H = H; V.wrap = wrap; V.qpow = qpow;
    BinParams &B = S.B;
    B.W = W; B.H = H; B.wrap = wrap;
    B.ext_u = extent[0];
    B.ext_v = extent[1];
    return S;
}
}  // namespace

// The setup in one pass and in the kernels' two: counts of words that differ
// in out[0..3]: slope changes, silhouette kinds, own records, counters; the
// tetrahedra left to the second pass and with own records in out[4], out[5]
extern "C" void hk_setup(const float *x, const float *y, const float *z, const int32_t dims[3], int32_t periodic,
                         const double rot[9], const double extent[2], int32_t W, int32_t H, int32_t wrap, int32_t qpow,
                         double bound, long long out[6]) {
    const float *const xyz[3] = {x, y, z};
    Scene S = scene(xyz, dims, periodic, rot, extent, W, H, wrap, qpow, bound);
    const LatticeParams &L = S.L;
    const int64_t nvert = (int64_t)dims[0] * dims[1] * dims[2], ntet = 6 * L.ncubes;
    std::vector<double> kinks[2];
    std::vector<uint8_t> sil[2];
    std::vector<Payload> rec[2];
    CubeCounts cnt[2];
    long long rest = 0;
    for (int p = 0; p < 2; ++p) {
        kinks[p].assign(36 * nvert, -7.0);
        sil[p].assign(36 * nvert, 255);
        rec[p].resize(ntet);
        std::memset((void *)rec[p].data(), 0, sizeof(Payload) * ntet);
        ViewParams V = S.V;
        V.edges = 1;
        V.kinks = kinks[p].data();
        V.sil = sil[p].data();
        V.own_cap = (uint64_t)ntet;
        std::vector<uint32_t> left(L.ncubes, 0u);
        for (int64_t cube = 0; cube < L.ncubes; ++cube) {
            auto own = [&](int t, const RecHead &R, const Payload &P) {
                if (R.flags & REC_VALID) rec[p][6 * cube + t] = P;
            };
            if (p == 0)
                setup_cube<kFormPyramid, true>(L, V, cube, own, cnt[p]);
            else
                setup_cube<kFormPyramid, true, 1>(L, V, cube, [](int, const RecHead &, const Payload &) {}, cnt[p],
                                                  &left[cube]);
        }
        for (int64_t cube = 0; p == 1 && cube < L.ncubes; ++cube)
            for (int t = 0; t < 6; ++t) {
                uint32_t one = left[cube] & (1u << t);
                if (!one) continue;
                ++rest;
                setup_cube<kFormPyramid, true, 3>(
                    L, V, cube,
                    [&](int k, const RecHead &R, const Payload &P) {
                        if (R.flags & REC_VALID) rec[p][6 * cube + k] = P;
                    },
                    cnt[p], &one);
            }
    }
    for (int k = 0; k < 6; ++k) out[k] = 0;
    for (int64_t i = 0; i < 36 * nvert; ++i) {
        out[0] += std::memcmp(&kinks[0][i], &kinks[1][i], sizeof(double)) != 0;
        out[1] += sil[0][i] != sil[1][i];
    }
    for (int64_t i = 0; i < ntet; ++i) {
        out[2] += std::memcmp((const void *)&rec[0][i], (const void *)&rec[1][i], sizeof(Payload)) != 0;
        out[5] += (rec[0][i].h.flags & REC_VALID) != 0u;
    }
    out[3] = (cnt[0].n_tets != cnt[1].n_tets) + (cnt[0].n_zero != cnt[1].n_zero) + (cnt[0].n_inv != cnt[1].n_inv) +
             (cnt[0].n_dets != cnt[1].n_dets) + (cnt[0].n_deg != cnt[1].n_deg);
    out[4] = rest;
}

// n_slab slabs (t0, t1 each) as values in tiles of rows x cols, `lanes` lanes
// to a pair: set up one by one, or (stack) once for all; images out[n_slab][H][W]
extern "C" long long hk_slabs(const float *x, const float *y, const float *z, const int32_t dims[3], int32_t periodic,
                              const double rot[9], const double extent[2], int32_t W, int32_t H, int32_t wrap,
                              int32_t qpow, const double *slabs, int32_t n_slab, int32_t stack, int32_t rows,
                              int32_t cols, int32_t lanes, double *out) {
    const float *const xyz[3] = {x, y, z};
    Scene S = scene(xyz, dims, periodic, rot, extent, W, H, wrap, qpow, 64.0);
    const LatticeParams &L = S.L;
    S.L.det_cond_k = -1.0;
    BinParams &B = S.B;
    B.Th = rows;
    B.Tw = cols;
    B.ntx = (W + cols - 1) / cols;
    B.nty = (H + rows - 1) / rows;
    B.direct = 1;
    long long frags = 0;
    auto draw = [&](const RecHead &h, const Payload &P, int k) {
        B.slab_t[0] = slabs[2 * k];
        B.slab_t[1] = slabs[2 * k + 1];
        const TileRange tr = tet_tiles(h, B);
        for (int s = 0; s < tr.count; ++s) {
            const int tile = tet_tile(B, tr, s), tx0 = tile % B.ntx * cols, ty0 = tile / B.ntx * rows;
            const int n = cols < W - tx0 ? cols : W - tx0, r = rows < H - ty0 ? rows : H - ty0;
            for (int lane = 0; lane < lanes; ++lane) {
                uint32_t spans = 0, kinks = 0;
                frags += slab_pair(h, P.c, B, tx0, ty0, n, r, lane, lanes,
                                   [&](int row, int u, double v) {
                                       if (row < 0 || row >= r || u < 0 || u >= n) throw 1;
                                       out[((size_t)k * H + ty0 + row) * W + tx0 + u] += v;
                                   },
                                   spans, kinks);
            }
        }
    };
    CubeCounts cnt;
    ViewParams V = S.V;
    V.slab = 1;
    if (stack) {
        V.slab_t[0] = slabs[0];
        V.slab_t[1] = slabs[2 * n_slab - 1];
        V.stack = slabs;
        V.nstack = n_slab;
        for (int64_t cube = 0; cube < L.ncubes; ++cube)
            setup_cube<kFormStack>(L, V, cube, [&](int, const RecHead &R, const Payload &P) {
                if (R.flags & REC_VALID)
                    for (uint32_t k = R.spare & 0xffffu; k <= R.spare >> 16; ++k) draw(R, P, (int)k);
            }, cnt);
    } else {
        for (int k = 0; k < n_slab; ++k) {
            V.slab_t[0] = slabs[2 * k];
            V.slab_t[1] = slabs[2 * k + 1];
            for (int64_t cube = 0; cube < L.ncubes; ++cube)
                setup_cube<kFormFace>(L, V, cube, [&](int, const RecHead &R, const Payload &P) {
                    if (R.flags & REC_VALID) draw(R, P, k);
                }, cnt);
        }
    }
    return frags;
}
