// RWG functions of a planar element and the EFIE interaction blocks of a lattice of them.
//
// The paper represents its elements with Rao-Wilton-Glisson functions (Sec. I,
// Sec. II-B) and leaves the fill rules open.  This fill: one function per
// interior edge of the element mesh, f = +-(l / 2A)(r - v) on the edge's two
// triangles (v the vertex opposite the edge, + on the lower-index triangle),
// Galerkin entries Z_mn = j k eta <<f_m . f_n, G>> - j (eta / k) <<div f_m,
// div f_n, G>> with G = exp(-jkR) / (4 pi R), Radon's seven-point (degree 5)
// rule on test and source triangles, and for elements at most one lattice step
// apart in x and y the static part 1/(4 pi R) of the source integral taken in
// closed form at each test point (coplanar potential integrals of Wilton et al.,
// IEEE TAP 1984), the remainder (exp(-jkR) - 1)/(4 pi R) by the rule.
//
// Workgroups per lattice offset and share of its test triangles, which are
// taken in chunks of U (the chunk's moments fill at most 64 KB of LDS).  Phase 1: a thread per
// (test triangle t, source triangle u) integrates over the 7 x 7 point pairs
// the six moments, taken about the test triangle's centroid c_t,
//   m0 = <<G>>, mr = <<(r - c_t) G>> (two components), mp = <<r' G>> (two
//   components) and mrp = <<(r - c_t) . r' G>>,
// once per triangle pair (a triangle carries up to three RWG functions, so
// moments per function would repeat this work about 2.6 times on the bowtie).
// Phase 2: a thread per (edge m of a triangle t of the chunk, source basis q) combines
// the moments of t and q's two triangles (v_m and v_q the free vertices,
// d_m = v_m - c_t):
//   <<(r - v_m) . (r' - v_q) G>> = mrp - d_m . mp - v_q . (mr - d_m m0),
// and adds t's share of the entry to a zeroed block: two shares an entry (m's two
// triangles), whose sum does not depend on their order, so the block is deterministic.
// Blocks two or more lattice steps apart use the same rule on test and source
// side, so T[-d] = T[d]^T for them (Galerkin reciprocity of the discrete
// operator): only one of each such pair is integrated and the other is its
// transpose; the nearer blocks, whose static part is integrated one-sidedly,
// are all integrated.
#include <algorithm>
#include <cmath>
#include <map>
#include <utility>

#include "rwg.h"
#include "runtime.h"

namespace mbt {

namespace {

constexpr double kEta = 376.730313668;   // free-space wave impedance, ohm
constexpr double kInv4Pi = 0.25 / M_PI;

struct RwgDev {
    const double2* qp;
    const double* qw;
    const double2* tv;
    const double* area;
    const double2* tcen;   // nt: triangle centroids
    const int* btri;
    const int* tedge;      // 3 per triangle: 2m + (0: T+ of basis m, 1: T-), -1: no basis
    const double2* bfree;
    const double2* bdel;   // 2M: free vertex minus the centroid of its triangle
    const double* blen;
};

constexpr int kPairVals = 6;                      // m0, mr (x, y), mp (x, y), mrp per triangle pair
constexpr int kPairLdsBytes = 64 * 1024;          // LDS for one chunk of pair moments

// sqrt(x) = root + tail and half its reciprocal (to a few last bits) for normal x:
// Goldschmidt's coupled iteration from the hardware's reciprocal root; the tail is the
// residual step that would round into the root.
__device__ __forceinline__ void sqrt_half(double x, double& root, double& tail, double& half) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double r = fma(-h, g, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
    }
    tail = fma(-g, g, x) * h;
    root = g;
    half = h;
}

// exp(-jkR)/(4 pi R), R2 = R^2 > 0, k / pi = kp + kl.  The phase is reduced in half
// turns, exactly; what R, the product kp R and kp itself leave out of it enters to first
// order, beside the sine and cosine.  1/R is taken of R with its tail, in one rounding.
// Three roundings reach the result (sine or cosine, 1/R, their product).  Its rms error is
// 0.97 to 1.03e-16 at every distance; with a rounded square root, sincos(k R) and a
// division it is 1.00e-16 below kR = 0.6, 2.0e-16 at 2 to 6 and 5.8e-15 at 60 to 200.
__device__ __forceinline__ double2 green_full(double kp, double kl, double R2) {
    double R, e, h, s, c;
    sqrt_half(R2, R, e, h);
    const double x = kp * R;
    const double d = M_PI * fma(kl, R, fma(kp, e, fma(kp, R, -x)));
    sincospi(x, &s, &c);
    const double z = h + h;
    double f = kInv4Pi * z;
    f = fma(fma(-f, e, fma(-f, R, kInv4Pi)), z, f);
    const double t = d * f;
    return make_double2(fma(c, f, -s * t), -fma(s, f, c * t));
}

// (exp(-jkR) - 1)/(4 pi R) = -(k / 4 pi) (sin x / x)(sin x + j cos x), x = kR/2 (finite at R = 0)
__device__ __forceinline__ double2 green_rem(double k, double R) {
    const double x = 0.5 * k * R;
    double s, c;
    sincos(x, &s, &c);
    const double f = -k * kInv4Pi * (x > 0.0 ? s / x : 1.0);
    return make_double2(f * s, f * c);
}

// Closed-form S0 = int_T dS'/|r' - rho| and S1 = int_T (r' - rho)/|r' - rho| dS' for
// rho in the plane of triangle v[0..2]: over the edges (p-, p+), with unit direction t,
// outward normal u, P = (p - rho).u, l+- = (p+- - rho).t, R+- = |p+- - rho| and
// L = ln((R+ + l+)/(R- + l-)):  S0 = sum P L,  S1 = 1/2 sum u (P^2 L + l+ R+ - l- R-).
__device__ void static_potentials(const double2* v, double2 rho, double& S0, double2& S1) {
    const double cx = (v[0].x + v[1].x + v[2].x) / 3.0, cy = (v[0].y + v[1].y + v[2].y) / 3.0;
    S0 = 0.0;
    S1 = make_double2(0.0, 0.0);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const double2 pm = v[i], pp = v[(i + 1) % 3];
        const double ex = pp.x - pm.x, ey = pp.y - pm.y;
        const double len = sqrt(ex * ex + ey * ey);
        const double tx = ex / len, ty = ey / len;
        double ux = ty, uy = -tx;
        if ((pm.x - cx) * ux + (pm.y - cy) * uy < 0.0) {
            ux = -ux;
            uy = -uy;
        }
        const double dmx = pm.x - rho.x, dmy = pm.y - rho.y;
        const double dpx = pp.x - rho.x, dpy = pp.y - rho.y;
        const double P = dmx * ux + dmy * uy;
        const double lp = dpx * tx + dpy * ty, lm = dmx * tx + dmy * ty;
        const double Rp = sqrt(dpx * dpx + dpy * dpy), Rm = sqrt(dmx * dmx + dmy * dmy);
        double c1 = lp * Rp - lm * Rm;
        if (P != 0.0) {
            // R + l = P^2 / (R - l) where l < 0 avoids the cancellation
            double L;
            if (lp < 0.0 && lm < 0.0) {
                L = log((Rm - lm) / (Rp - lp));
            } else {
                const double num = lp < 0.0 ? P * P / (Rp - lp) : Rp + lp;
                const double den = lm < 0.0 ? P * P / (Rm - lm) : Rm + lm;
                L = log(num / den);
            }
            S0 += P * L;
            c1 += P * P * L;
        }
        S1.x += 0.5 * c1 * ux;
        S1.y += 0.5 * c1 * uy;
    }
}

// NEAR: the offsets at most one step away (a launch of its own: the closed forms take
// twice the registers), else the others that are integrated.  blockIdx.y takes every
// gridDim.y-th chunk.  FP64 arithmetic bounds it.  On a 64x64 lattice of the bowtie (96
// functions) the far launch takes 8.0 ms; with the library's sincos, square root and
// division, every chunk looking through all M^2 entries and both kinds of offsets in one
// kernel of 231 registers the fill took 16.9, and 0.98 instead of 0.18 ms on 8x8, where
// one workgroup per offset left the chip idle.
constexpr int kFillT = 512;
template <bool NEAR>
__global__ __launch_bounds__(kFillT, NEAR ? 2 : 4) void rwg_fill_kernel(RwgDev d, int nt, int M, int U, int nx, int ny, double ldx,
                                                          double ldy, double k, double kp, double kl,
                                                          double2* __restrict__ T) {
    extern __shared__ double2 pm[];   // [t - t0][u][kPairVals]
    const int nox = 2 * nx - 1;
    // near: the offsets -1..1 of each axis that the lattice has
    const int nnx = min(nx, 2) * 2 - 1, nny = min(ny, 2) * 2 - 1;
    const int ox = NEAR ? (int)blockIdx.x % nnx - nnx / 2 : (int)blockIdx.x % nox - (nx - 1);
    const int oy = NEAR ? (int)blockIdx.x / nnx - nny / 2 : (int)blockIdx.x / nox - (ny - 1);
    const int off = (oy + ny - 1) * nox + ox + nx - 1;
    // the test element sits at lattice offset (ox, oy) from the source element at the origin
    const double sx = ox * ldx, sy = oy * ldy;
    if (!NEAR) {
        if (ox >= -1 && ox <= 1 && oy >= -1 && oy <= 1) return;
        if (oy < 0 || (oy == 0 && ox < 0)) return;   // the transpose of T[-d], filled afterwards
    }
    double2* Tb = T + (int64_t)off * M * M;
    for (int t0 = blockIdx.y * U; t0 < nt; t0 += gridDim.y * U) {
        const int nu = min(U, nt - t0);
        for (int task = threadIdx.x; task < nt * nu; task += blockDim.x) {
            const int u = task % nt, t = t0 + task / nt;
            const double2 ct = d.tcen[t];
            double2 rs[kRwgQ];
            double ws[kRwgQ];
#pragma unroll
            for (int j = 0; j < kRwgQ; ++j) {
                rs[j] = d.qp[u * kRwgQ + j];
                ws[j] = d.qw[u * kRwgQ + j];
            }
            double2 tvu[3];
            if (NEAR) {
#pragma unroll
                for (int j = 0; j < 3; ++j) tvu[j] = d.tv[u * 3 + j];
            }
            double2 m0 = make_double2(0, 0), mrx = m0, mry = m0, mpx = m0, mpy = m0, mrp = m0;
            for (int i = 0; i < kRwgQ; ++i) {
                const double2 q = d.qp[t * kRwgQ + i];
                const double rox = q.x + sx, roy = q.y + sy;
                const double wo = d.qw[t * kRwgQ + i];
                double2 g0 = make_double2(0, 0), g1x = make_double2(0, 0), g1y = make_double2(0, 0);
#pragma unroll
                for (int j = 0; j < kRwgQ; ++j) {
                    const double dx = rox - rs[j].x, dy = roy - rs[j].y;
                    const double R2 = dx * dx + dy * dy;
                    const double2 G = NEAR ? green_rem(k, sqrt(R2)) : green_full(kp, kl, R2);
                    const double2 wg = make_double2(ws[j] * G.x, ws[j] * G.y);
                    g0 = cadd(g0, wg);
                    g1x = cadd(g1x, make_double2(rs[j].x * wg.x, rs[j].x * wg.y));
                    g1y = cadd(g1y, make_double2(rs[j].y * wg.x, rs[j].y * wg.y));
                }
                if (NEAR) {
                    double S0;
                    double2 S1;
                    static_potentials(tvu, make_double2(rox, roy), S0, S1);
                    g0.x += S0 * kInv4Pi;
                    g1x.x += (S1.x + rox * S0) * kInv4Pi;
                    g1y.x += (S1.y + roy * S0) * kInv4Pi;
                }
                // about the centroid in the element frame: the lattice shift cancels exactly
                const double ax = q.x - ct.x, ay = q.y - ct.y;
                m0 = cadd(m0, make_double2(wo * g0.x, wo * g0.y));
                mrx = cadd(mrx, make_double2(wo * ax * g0.x, wo * ax * g0.y));
                mry = cadd(mry, make_double2(wo * ay * g0.x, wo * ay * g0.y));
                mpx = cadd(mpx, make_double2(wo * g1x.x, wo * g1x.y));
                mpy = cadd(mpy, make_double2(wo * g1y.x, wo * g1y.y));
                mrp = cadd(mrp, make_double2(wo * (ax * g1x.x + ay * g1y.x), wo * (ax * g1x.y + ay * g1y.y)));
            }
            double2* a = pm + (int64_t)task * kPairVals;
            a[0] = m0;
            a[1] = mrx;
            a[2] = mry;
            a[3] = mpx;
            a[4] = mpy;
            a[5] = mrp;
        }
        __syncthreads();
        for (int e = threadIdx.x; e < nu * 3 * M; e += blockDim.x) {
            const int q = e % M, tl = e / M / 3;
            const int me = d.tedge[3 * t0 + e / M];
            if (me < 0) continue;
            const int m = me >> 1, side = me & 1;
            const double lmq = d.blen[m] * d.blen[q];
            const double At = d.area[t0 + tl];
            const double2 dm = d.bdel[me];
            double2 sum = make_double2(0, 0);
#pragma unroll
            for (int tau = 0; tau < 2; ++tau) {
                const int u = d.btri[2 * q + tau];
                const double Au = d.area[u];
                const double2 vq = d.bfree[2 * q + tau];
                const double2* a = pm + ((int64_t)tl * nt + u) * kPairVals;
                const double2 hvx = csub(a[1], make_double2(dm.x * a[0].x, dm.x * a[0].y));
                const double2 hvy = csub(a[2], make_double2(dm.y * a[0].x, dm.y * a[0].y));
                const double2 hw = make_double2(a[5].x - (dm.x * a[3].x + dm.y * a[4].x),
                                                a[5].y - (dm.x * a[3].y + dm.y * a[4].y));
                const double2 A = make_double2(hw.x - (vq.x * hvx.x + vq.y * hvy.x),
                                               hw.y - (vq.x * hvx.y + vq.y * hvy.y));
                // j k eta A / (4 At Au) - j (eta / k) m0 / (At Au)
                const double cv = k * kEta / (4.0 * At * Au), cs = kEta / (k * At * Au);
                const double re = -(cv * A.y - cs * a[0].y);
                const double im = cv * A.x - cs * a[0].x;
                const double sg = (side == tau) ? lmq : -lmq;
                sum.x += sg * re;
                sum.y += sg * im;
            }
            atomicAdd(&Tb[(int64_t)m * M + q].x, sum.x);
            atomicAdd(&Tb[(int64_t)m * M + q].y, sum.y);
        }
        __syncthreads();
    }
}

// T[d] = T[-d]^T for the far offsets that the fill kernel skipped, a tile of the block per
// workgroup through LDS (read straight down the columns it took 1.6 ms
// at 64x64 elements, 0.45 so)
constexpr int kMirT = 32;
__global__ __launch_bounds__(256) void rwg_mirror_kernel(int M, int nx, int ny, double2* __restrict__ T) {
    __shared__ double2 tile[kMirT][kMirT + 1];
    const int nox = 2 * nx - 1;
    const int off = blockIdx.x;
    const int ox = off % nox - (nx - 1), oy = off / nox - (ny - 1);
    const bool near = ox >= -1 && ox <= 1 && oy >= -1 && oy <= 1;
    if (near || !(oy < 0 || (oy == 0 && ox < 0))) return;
    const int mirror = (-oy + (ny - 1)) * nox + (-ox + (nx - 1));
    const int nm = (M + kMirT - 1) / kMirT;
    const int p0 = (int)blockIdx.y / nm * kMirT, q0 = (int)blockIdx.y % nm * kMirT;
    const int tx = threadIdx.x % kMirT, ty = threadIdx.x / kMirT;
    for (int j = ty; j < kMirT; j += 256 / kMirT)
        if (q0 + j < M && p0 + tx < M) tile[j][tx] = T[((int64_t)mirror * M + q0 + j) * M + p0 + tx];
    __syncthreads();
    for (int j = ty; j < kMirT; j += 256 / kMirT)
        if (p0 + j < M && q0 + tx < M) T[((int64_t)off * M + p0 + j) * M + q0 + tx] = tile[tx][j];
}

}  // namespace

RwgMesh rwg_from_mesh(const mbt_rwg_mesh& ms) {
    MBT_REQUIRE(ms.vert && ms.tri && ms.port_edges, "NULL mesh array");
    MBT_REQUIRE(ms.nvert >= 3 && ms.nvert <= 4096, "nvert must be within 3..4096");
    MBT_REQUIRE(ms.ntri >= 2 && ms.ntri <= kRwgMaxTri, "ntri must be within 2..256");
    MBT_REQUIRE(ms.nport_edges >= 1 && ms.nport_edges <= kMaxPortBases, "nport_edges must be within 1..8");
    MBT_REQUIRE(std::isfinite(ms.port_dir[0]) && std::isfinite(ms.port_dir[1]) &&
                    (ms.port_dir[0] != 0.0 || ms.port_dir[1] != 0.0),
                "port_dir must be a finite nonzero vector");
    const int nv = ms.nvert, nt = ms.ntri;
    std::vector<double2> v(nv);
    for (int i = 0; i < nv; ++i) {
        v[i] = make_double2(ms.vert[2 * i], ms.vert[2 * i + 1]);
        MBT_REQUIRE(std::isfinite(v[i].x) && std::isfinite(v[i].y), "mesh vertices must be finite");
    }
    RwgMesh h;
    h.nt = nt;
    h.area.resize(nt);
    h.tv.resize((size_t)nt * 3);
    std::map<std::pair<int, int>, std::vector<int>> owners;
    for (int t = 0; t < nt; ++t) {
        int id[3];
        for (int j = 0; j < 3; ++j) {
            id[j] = ms.tri[3 * t + j];
            MBT_REQUIRE(id[j] >= 0 && id[j] < nv, "triangle vertex index out of range");
            h.tv[3 * t + j] = v[id[j]];
        }
        MBT_REQUIRE(id[0] != id[1] && id[1] != id[2] && id[0] != id[2], "triangle with a repeated vertex");
        const double2 a = v[id[0]], b = v[id[1]], c = v[id[2]];
        h.area[t] = 0.5 * std::fabs((b.x - a.x) * (c.y - a.y) - (b.y - a.y) * (c.x - a.x));
        MBT_REQUIRE(h.area[t] > 0.0, "degenerate (zero-area) triangle");
        for (int j = 0; j < 3; ++j) {
            const int p = id[j], q = id[(j + 1) % 3];
            owners[{std::min(p, q), std::max(p, q)}].push_back(t);
        }
    }
    // interior edges in increasing (smaller vertex, larger vertex) order (std::map order)
    std::map<std::pair<int, int>, int> index;
    for (const auto& kv : owners) {
        MBT_REQUIRE(kv.second.size() <= 2, "mesh edge shared by more than two triangles");
        if (kv.second.size() != 2) continue;
        const int m = h.M++;
        index[kv.first] = m;
        const int tp = std::min(kv.second[0], kv.second[1]), tm = std::max(kv.second[0], kv.second[1]);
        MBT_REQUIRE(tp != tm, "triangle listed twice");
        auto opposite = [&](int t) {
            for (int j = 0; j < 3; ++j) {
                const int w = ms.tri[3 * t + j];
                if (w != kv.first.first && w != kv.first.second) return w;
            }
            throw Error(-1, "invalid triangle");
        };
        h.btri.push_back(tp);
        h.btri.push_back(tm);
        h.bfree.push_back(v[opposite(tp)]);
        h.bfree.push_back(v[opposite(tm)]);
        const double2 a = v[kv.first.first], b = v[kv.first.second];
        h.blen.push_back(std::sqrt((b.x - a.x) * (b.x - a.x) + (b.y - a.y) * (b.y - a.y)));
    }
    MBT_REQUIRE(h.M >= 1 && h.M <= kMaxBlockM, "the mesh must have 1..128 interior edges (RWG functions)");
    // gap bases: weight sign * length, the sign from the T+ -> T- direction along port_dir
    auto centroid = [&](int t) {
        return make_double2((h.tv[3 * t].x + h.tv[3 * t + 1].x + h.tv[3 * t + 2].x) / 3.0,
                            (h.tv[3 * t].y + h.tv[3 * t + 1].y + h.tv[3 * t + 2].y) / 3.0);
    };
    h.port.n = ms.nport_edges;
    for (int i = 0; i < ms.nport_edges; ++i) {
        const int a = ms.port_edges[2 * i], b = ms.port_edges[2 * i + 1];
        auto it = index.find({std::min(a, b), std::max(a, b)});
        MBT_REQUIRE(it != index.end(), "port edge is not an interior edge of the mesh");
        const int m = it->second;
        for (int j = 0; j < i; ++j) MBT_REQUIRE(h.port.idx[j] != m, "port edge listed twice");
        const double2 cp = centroid(h.btri[2 * m]), cm = centroid(h.btri[2 * m + 1]);
        const double proj = (cm.x - cp.x) * ms.port_dir[0] + (cm.y - cp.y) * ms.port_dir[1];
        MBT_REQUIRE(proj != 0.0, "port edge parallel to port_dir");
        h.port.idx[i] = m;
        h.port.w[i] = (proj > 0 ? 1.0 : -1.0) * h.blen[m];
    }
    // Radon's seven-point rule: the centroid and two orbits of three points
    const double r15 = std::sqrt(15.0);
    const double a1 = (6.0 - r15) / 21.0, a2 = (6.0 + r15) / 21.0;
    const double w0 = 9.0 / 40.0, w1 = (155.0 - r15) / 1200.0, w2 = (155.0 + r15) / 1200.0;
    const double bary[kRwgQ][3] = {{1.0 / 3.0, 1.0 / 3.0, 1.0 / 3.0},
                                   {1.0 - 2.0 * a1, a1, a1}, {a1, 1.0 - 2.0 * a1, a1}, {a1, a1, 1.0 - 2.0 * a1},
                                   {1.0 - 2.0 * a2, a2, a2}, {a2, 1.0 - 2.0 * a2, a2}, {a2, a2, 1.0 - 2.0 * a2}};
    const double wts[kRwgQ] = {w0, w1, w1, w1, w2, w2, w2};
    h.qp.resize((size_t)nt * kRwgQ);
    h.qw.resize((size_t)nt * kRwgQ);
    for (int t = 0; t < nt; ++t)
        for (int i = 0; i < kRwgQ; ++i) {
            double x = 0, y = 0;
            for (int j = 0; j < 3; ++j) {
                x += bary[i][j] * h.tv[3 * t + j].x;
                y += bary[i][j] * h.tv[3 * t + j].y;
            }
            h.qp[(size_t)t * kRwgQ + i] = make_double2(x, y);
            h.qw[(size_t)t * kRwgQ + i] = wts[i] * h.area[t];
        }
    return h;
}

static void split_phase(double k, double& kp, double& kl) {
    kp = k / M_PI;
    kl = (double)((long double)k / 3.14159265358979323846264338327950288L - (long double)kp);
}

static __global__ void green_kernel(double kp, double kl, const double* __restrict__ R2, int64_t n,
                                    double2* __restrict__ G) {
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) G[i] = green_full(kp, kl, R2[i]);
}

void rwg_green(double k, const double* R2, int64_t n, double2* G, hipStream_t s) {
    double kp, kl;
    split_phase(k, kp, kl);
    hipLaunchKernelGGL(green_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, kp, kl, R2, n, G);
    MBT_LAUNCH_CHECK();
}

void rwg_fill_blocks(const Geom& g, const RwgMesh& h, double k, double2* T, hipStream_t s) {
    const int nt = h.nt, M = h.M;
    MBT_REQUIRE(M == g.M, "mesh and geometry disagree on the number of bases");
    // triangle centroids and each free vertex relative to its triangle's centroid
    std::vector<double2> tcen(nt), bdel(2 * (size_t)M);
    for (int t = 0; t < nt; ++t)
        tcen[t] = make_double2((h.tv[3 * t].x + h.tv[3 * t + 1].x + h.tv[3 * t + 2].x) / 3.0,
                               (h.tv[3 * t].y + h.tv[3 * t + 1].y + h.tv[3 * t + 2].y) / 3.0);
    for (int i = 0; i < 2 * M; ++i)
        bdel[i] = make_double2(h.bfree[i].x - tcen[h.btri[i]].x, h.bfree[i].y - tcen[h.btri[i]].y);
    // one upload of the mesh tables, laid out back to back
    const size_t b_qp = sizeof(double2) * h.qp.size(), b_qw = sizeof(double) * h.qw.size();
    const size_t b_tv = sizeof(double2) * h.tv.size(), b_ar = sizeof(double) * h.area.size();
    const size_t b_tc = sizeof(double2) * tcen.size(), b_bt = sizeof(int) * h.btri.size();
    const size_t b_bf = sizeof(double2) * h.bfree.size(), b_bd = sizeof(double2) * bdel.size();
    const size_t b_bl = sizeof(double) * h.blen.size();
    std::vector<int> tedge(3 * (size_t)nt, -1);
    for (int i = 0; i < 2 * M; ++i) {
        int* e = tedge.data() + 3 * (size_t)h.btri[i];
        while (*e >= 0) ++e;   // a triangle has three edges, each of one basis at most
        *e = i;
    }
    const size_t b_te = sizeof(int) * tedge.size();
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    DBuf buf;
    buf.alloc(up(b_qp) + up(b_qw) + up(b_tv) + up(b_ar) + up(b_tc) + up(b_bt) + up(b_bf) + up(b_bd) + up(b_bl) + up(b_te));
    char* p = buf.as<char>();
    RwgDev d;
    auto put = [&](const void* src, size_t b) {
        char* dst = p;
        MBT_HIP(hipMemcpyAsync(dst, src, b, hipMemcpyHostToDevice, s));
        p += up(b);
        return dst;
    };
    d.qp = reinterpret_cast<const double2*>(put(h.qp.data(), b_qp));
    d.qw = reinterpret_cast<const double*>(put(h.qw.data(), b_qw));
    d.tv = reinterpret_cast<const double2*>(put(h.tv.data(), b_tv));
    d.area = reinterpret_cast<const double*>(put(h.area.data(), b_ar));
    d.tcen = reinterpret_cast<const double2*>(put(tcen.data(), b_tc));
    d.btri = reinterpret_cast<const int*>(put(h.btri.data(), b_bt));
    d.bfree = reinterpret_cast<const double2*>(put(h.bfree.data(), b_bf));
    d.bdel = reinterpret_cast<const double2*>(put(bdel.data(), b_bd));
    d.blen = reinterpret_cast<const double*>(put(h.blen.data(), b_bl));
    d.tedge = reinterpret_cast<const int*>(put(tedge.data(), b_te));
    // test triangles per chunk: the chunk's pair moments fit the LDS allowance, and the passes of
    // the workgroup over the pairs are as few as they can be
    const int most = std::max(1, std::min(nt, kPairLdsBytes / (nt * kPairVals * (int)sizeof(double2))));
    auto passes = [&](int u) {
        auto of = [&](int n) { return (nt * n + kFillT - 1) / kFillT; };
        return nt / u * of(u) + of(nt % u);
    };
    int U = most;
    for (int u = most - 1; u >= 1; --u)
        if (passes(u) < passes(U)) U = u;
    const int nchunk = (nt + U - 1) / U;
    const size_t lds = sizeof(double2) * (size_t)nt * U * kPairVals;
    double kp, kl;
    split_phase(k, kp, kl);
    // four workgroups per CU or more: fewer, and the fill waits for one workgroup's chain of points
    const int64_t half = g.noff() / 2 + 1;
    const int share = (int)std::min<int64_t>(nchunk, (1023 + half) / half);
    const int near = (2 * std::min(g.nx, 2) - 1) * (2 * std::min(g.ny, 2) - 1);
    zero_d(T, (int64_t)g.noff() * M * M, s);
    hipLaunchKernelGGL((rwg_fill_kernel<true>), dim3((unsigned)near, (unsigned)nchunk), dim3(kFillT), lds, s, d, nt, M, U,
                       g.nx, g.ny, g.dx, g.dy, k, kp, kl, T);
    hipLaunchKernelGGL((rwg_fill_kernel<false>), dim3((unsigned)g.noff(), (unsigned)share), dim3(kFillT), lds, s, d, nt, M,
                       U, g.nx, g.ny, g.dx, g.dy, k, kp, kl, T);
    MBT_LAUNCH_CHECK();
    const int nm = (M + kMirT - 1) / kMirT;
    hipLaunchKernelGGL(rwg_mirror_kernel, dim3((unsigned)g.noff(), (unsigned)(nm * nm)), dim3(256), 0, s, M, g.nx, g.ny,
                       T);
    MBT_LAUNCH_CHECK();
    // the tables are freed when this returns: wait for the kernel
    MBT_HIP(hipStreamSynchronize(s));
}

}  // namespace mbt
