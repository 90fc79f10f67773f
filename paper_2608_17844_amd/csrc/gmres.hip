// Batched restarted GMRES(m): one independent Krylov solve per right-hand side,
// all sharing the batched operator (the paper's "new M1" GMRES with the
// normal-equation strategy, or GMRES with the element-block preconditioner).
//
// The paper uses MATLAB's GMRES and states no details; this solver fixes them:
// x0 = 0; Arnoldi by classical Gram-Schmidt with delayed reorthogonalisation
// (DCGS2, Swirydowicz et al. 2021: the second projection of step k-1 is folded
// into the dot sweep of step k, so each step sweeps the basis twice), or by
// plain CGS2 in three sweeps on request; complex Givens rotations (c real,
// s complex, c = 0 and s = 1 when the pivot is zero); stop as soon as the
// least-squares residual |g_{j+1}| <= tol * ||b||; the explicit residual
// b - A x is recomputed at every restart, and a RHS counts as converged only
// on that explicit residual: <= tol * ||b||, or <= 2 tol * ||b|| after a cycle
// whose least-squares residual met the tolerance (the two residuals differ by
// rounding; a larger gap means the recurrence lost its Arnoldi relation, e.g.
// at a breakdown, and the RHS restarts from the explicit residual).  In DCGS2 a
// step whose reorthogonalised norm nu^2 = ||u||^2 - ||s||^2 has cancelled to
// below 1e-12 ||u||^2 is a breakdown (nu = 0): the cycle ends there.
//
// Vectors are RHS-innermost, v[n][r]: a lane owns one RHS and walks rows, so
// every per-RHS dot product is accumulated in a fixed order that does not
// depend on how many other RHS share the batch (bit-identical results alone or
// batched).  Rows are split into fixed chunks (a function of N only) whose
// partial sums are reduced by a second kernel in a fixed order (groups of 64
// chunks, then the groups).
//
// HBM traffic per Arnoldi step is dominated by the basis reads.  DCGS2 step k
// reads V_{0..k-1}, the candidate u and w = A u once for all dot products
// (s = V^H u, z = V^H w, u^H u, u^H w) and once more for the update that
// writes the normalised v_k and the next candidate.  CGS2 is fused into three
// passes: (1) h = V^H w; (2) w <- w - V h together with h2 = V^H w; (3)
// w <- w - V h2 together with ||w||^2.  In the dot sweeps the waves of a
// workgroup share rows and RHS and split the basis vectors; the DCGS2 update
// gives each wave its own rows and all vectors.
// The reduced-precision inner solves keep the basis packed (FP32 components
// rounded to 24 bits, two RHS per 12-byte word) or in FP32, with FP32 work
// vectors; all dot products, norms and the Hessenberg/Givens recurrences stay
// FP64.  The file also holds the batched PCG on the normal equations (Sec.
// II-C), which reuses the chunked reductions.
#include "common.h"
#include "gmres.h"

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

namespace mbt {

namespace {

constexpr int kMaxVec = 64;            // basis vectors per pass -> restart <= 63

// Accumulations written as explicit fused multiply-adds in a fixed order.  The
// kernels have variants that move one or two RHS per lane; leaving the fusion of
// products and sums to the compiler lets it differ between variants, and a RHS's
// result would then depend on the parity of the batch size.
// acc + a b
__device__ __forceinline__ double2 cfma(double2 acc, double2 a, double2 b) {
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(-a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(a.y, b.x, acc.y);
    return acc;
}
// acc + conj(a) b
__device__ __forceinline__ double2 cfmac(double2 acc, double2 a, double2 b) {
    acc.x = fma(a.x, b.x, acc.x);
    acc.x = fma(a.y, b.y, acc.x);
    acc.y = fma(a.x, b.y, acc.y);
    acc.y = fma(-a.y, b.x, acc.y);
    return acc;
}
// w s - c - k v  (the DCGS2 candidate update)
__device__ __forceinline__ double2 next_candidate(double2 w, double s, double2 c, double2 k, double2 v) {
    double2 t;
    t.x = fma(w.x, s, -c.x);
    t.y = fma(w.y, s, -c.y);
    t.x = fma(-k.x, v.x, t.x);
    t.x = fma(k.y, v.y, t.x);
    t.y = fma(-k.x, v.y, t.y);
    t.y = fma(-k.y, v.x, t.y);
    return t;
}
// acc + |a|^2
__device__ __forceinline__ double nfma(double acc, double2 a) { return fma(a.y, a.y, fma(a.x, a.x, acc)); }

__device__ __forceinline__ double2 ld2(const double2* p) { return *p; }
__device__ __forceinline__ double2 ld2(const float2* p) { float2 v = *p; return make_double2(v.x, v.y); }
__device__ __forceinline__ void st2(double2* p, double2 v) { *p = v; }
__device__ __forceinline__ void st2(float2* p, double2 v) { *p = make_float2((float)v.x, (float)v.y); }

// RPL consecutive complex values (RHS columns) per lane, widened to FP64.
// FP32 pairs are moved with one 16-byte access.
template <int RPL> __device__ __forceinline__ void ldp(const double2* p, double2 (&o)[RPL]) {
#pragma unroll
    for (int k = 0; k < RPL; ++k) o[k] = p[k];
}
template <int RPL> __device__ __forceinline__ void ldp(const float2* p, double2 (&o)[RPL]) {
    if constexpr (RPL == 2) {
        const float4 v = *reinterpret_cast<const float4*>(p);
        o[0] = make_double2(v.x, v.y);
        o[1] = make_double2(v.z, v.w);
    } else {
#pragma unroll
        for (int k = 0; k < RPL; ++k) o[k] = ld2(p + k);
    }
}
template <int RPL> __device__ __forceinline__ void stp(double2* p, const double2 (&v)[RPL]) {
#pragma unroll
    for (int k = 0; k < RPL; ++k) p[k] = v[k];
}
template <int RPL> __device__ __forceinline__ void stp(float2* p, const double2 (&v)[RPL]) {
    if constexpr (RPL == 2) {
        *reinterpret_cast<float4*>(p) = make_float4((float)v[0].x, (float)v[0].y, (float)v[1].x, (float)v[1].y);
    } else {
#pragma unroll
        for (int k = 0; k < RPL; ++k) st2(p + k, v[k]);
    }
}

// Raw (storage-format) pack of RPL adjacent complex values, kept in registers
// between the load of the next row and its use; widened to FP64 at use.
template <typename T, int RPL> struct Raw;
template <> struct Raw<double2, 1> {
    double2 v;
    __device__ __forceinline__ void load(const double2* p) { v = *p; }
    __device__ __forceinline__ void zero() { v = make_double2(0, 0); }
    __device__ __forceinline__ double2 get(int) const { return v; }
};
template <> struct Raw<double2, 2> {
    double2 v[2];
    __device__ __forceinline__ void load(const double2* p) { v[0] = p[0]; v[1] = p[1]; }
    __device__ __forceinline__ void zero() { v[0] = v[1] = make_double2(0, 0); }
    __device__ __forceinline__ double2 get(int k) const { return v[k]; }
};
template <> struct Raw<float2, 1> {
    float2 v;
    __device__ __forceinline__ void load(const float2* p) { v = *p; }
    __device__ __forceinline__ void zero() { v = make_float2(0, 0); }
    __device__ __forceinline__ double2 get(int) const { return make_double2(v.x, v.y); }
};
template <> struct Raw<float2, 2> {
    float4 v;
    __device__ __forceinline__ void load(const float2* p) { v = *reinterpret_cast<const float4*>(p); }
    __device__ __forceinline__ void zero() { v = make_float4(0, 0, 0, 0); }
    __device__ __forceinline__ double2 get(int k) const { return k ? make_double2(v.z, v.w) : make_double2(v.x, v.y); }
};

// ------------------------------------------------------------------ packed 24-bit basis storage
// The mixed path may keep its Krylov basis with the low byte of each FP32
// component rounded away (sign, 8-bit exponent, 15-bit mantissa; unit roundoff
// 2^-16), three quarters of the FP32 bytes.  Two complex values of adjacent RHS
// columns (four components) form one 12-byte word, so a basis vector of N x R
// values (R even) is N x R/2 words.  The work vectors (the candidate and A times
// it) stay FP32.
struct p24x2 {
    uint32_t w[3];
};
template <typename T> struct PerWord { static constexpr int v = 1; };
template <> struct PerWord<p24x2> { static constexpr int v = 2; };
// element offset n*R + r (r even for packed words) -> offset in storage words
template <typename T> __device__ __forceinline__ int64_t vofs(int64_t off) { return off / PerWord<T>::v; }

__device__ __forceinline__ uint32_t to24(double x) {
    const uint32_t u = __float_as_uint((float)x);
    return (u + 0x7Fu + ((u >> 8) & 1u)) >> 8;   // nearest, ties to even, on the dropped byte
}
__device__ __forceinline__ double from24(uint32_t t) { return (double)__uint_as_float(t << 8); }
__device__ __forceinline__ double2 round24(double2 v) { return make_double2(from24(to24(v.x)), from24(to24(v.y))); }

template <> struct Raw<p24x2, 2> {
    uint32_t a, b, c;
    __device__ __forceinline__ void load(const p24x2* p) {
        const uint3 t = *reinterpret_cast<const uint3*>(p);
        a = t.x;
        b = t.y;
        c = t.z;
    }
    __device__ __forceinline__ void zero() { a = b = c = 0; }
    __device__ __forceinline__ double2 get(int k) const {
        if (k == 0) return make_double2(from24(a & 0xFFFFFFu), from24((a >> 24) | ((b & 0xFFFFu) << 8)));
        return make_double2(from24((b >> 16) | ((c & 0xFFu) << 16)), from24(c >> 8));
    }
};
__device__ __forceinline__ void st24(p24x2* p, double2 v0, double2 v1) {
    const uint32_t t0 = to24(v0.x), t1 = to24(v0.y), t2 = to24(v1.x), t3 = to24(v1.y);
    uint3 o;
    o.x = t0 | (t1 << 24);
    o.y = (t1 >> 8) | (t2 << 16);
    o.z = (t2 >> 16) | (t3 << 8);
    *reinterpret_cast<uint3*>(p) = o;
}

// One pass over the basis V_0..V_{nvec-1} (rows of one chunk, 64*RPL RHS columns
// per workgroup).  The NW waves of a workgroup read the same rows and columns
// and split the basis vectors (wave w takes i = w, w+NW, ..., G per wave); a
// lane owns RPL adjacent RHS columns.
// MODE 0: h[i] = sum_n conj(V_i[n]) w[n]                         (partials per chunk)
// MODE 1: w <- w - sum_i coef_i V_i ; h2[i] = sum_n conj(V_i) w   (partials per chunk)
// MODE 2: w <- w - sum_i coef_i V_i ; ||w||^2                      (partials per chunk)
template <typename TB, typename TO, int MODE, int NW, int G, int RPL>
__global__ __launch_bounds__(NW * 64) void arnoldi_kernel(const TB* __restrict__ V, int64_t vstride, int nvec,
                                                          const double2* __restrict__ coef, TO* w, int64_t N, int R,
                                                          int64_t rows_per_chunk, double2* __restrict__ partial) {
    __shared__ double2 xch[2][NW][64 * RPL];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int r0 = (blockIdx.x * 64 + lane) * RPL;
    const bool live = r0 < R;            // R is a multiple of RPL
    const int64_t chunk = blockIdx.y;
    const int64_t n0 = chunk * rows_per_chunk;
    const int64_t n1 = min(N, n0 + rows_per_chunk);

    double2 acc[G][RPL];
    double2 cf[G][RPL];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int i = wave + NW * g;
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            acc[g][k] = make_double2(0, 0);
            cf[g][k] = (MODE != 0 && live && i < nvec) ? coef[(int64_t)i * R + r0 + k] : make_double2(0, 0);
        }
    }
    double nrm[RPL];
#pragma unroll
    for (int k = 0; k < RPL; ++k) nrm[k] = 0.0;
    int buf = 0;
    // rows are software-pipelined: the loads of row n+1 are issued before the
    // arithmetic (and the cross-wave exchange) of row n
    Raw<TB, RPL> cur[G], nxt[G];
    Raw<TO, RPL> cw, nw_raw;
    auto load_row = [&](int64_t n, Raw<TB, RPL>(&v)[G], Raw<TO, RPL>& wr) {
        const int64_t off = n * R + r0;
        wr.load(w + off);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = wave + NW * g;
            if (i < nvec) v[g].load(V + i * vstride + vofs<TB>(off));
            else v[g].zero();
        }
    };
    if (live && n0 < n1) load_row(n0, cur, cw);
    for (int64_t n = n0; n < n1; ++n) {
        const int64_t off = n * R + r0;
        if (live && n + 1 < n1) load_row(n + 1, nxt, nw_raw);
        // values are widened at each use from the raw registers (no widened copies live across the barrier)
        double2 wv[RPL];
#pragma unroll
        for (int k = 0; k < RPL; ++k) wv[k] = cw.get(k);
        if constexpr (MODE == 0) {
            if (live) {
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int k = 0; k < RPL; ++k) acc[g][k] = cfmac(acc[g][k], cur[g].get(k), wv[k]);
            }
        } else {
            double2 u[RPL];
#pragma unroll
            for (int k = 0; k < RPL; ++k) u[k] = make_double2(0, 0);
            if (live) {
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int k = 0; k < RPL; ++k) u[k] = cfma(u[k], cf[g][k], cur[g].get(k));
            }
#pragma unroll
            for (int k = 0; k < RPL; ++k) xch[buf][wave][lane * RPL + k] = u[k];
            __syncthreads();
            double2 nw[RPL];
#pragma unroll
            for (int k = 0; k < RPL; ++k) {
                double2 tot = xch[buf][0][lane * RPL + k];
#pragma unroll
                for (int q = 1; q < NW; ++q) tot = cadd(tot, xch[buf][q][lane * RPL + k]);
                nw[k] = csub(wv[k], tot);
            }
            buf ^= 1;
            if (live) {
                if constexpr (MODE == 1) {
#pragma unroll
                    for (int g = 0; g < G; ++g)
#pragma unroll
                        for (int k = 0; k < RPL; ++k) acc[g][k] = cfmac(acc[g][k], cur[g].get(k), nw[k]);
                } else if constexpr (MODE == 2) {
#pragma unroll
                    for (int k = 0; k < RPL; ++k) nrm[k] = nfma(nrm[k], nw[k]);
                }
                if (wave == 0) stp<RPL>(w + off, nw);
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) cur[g] = nxt[g];
        cw = nw_raw;
    }
    if (!live) return;
    if constexpr (MODE == 0 || MODE == 1) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int i = wave + NW * g;
            if (i < nvec)
#pragma unroll
                for (int k = 0; k < RPL; ++k) partial[(chunk * nvec + i) * R + r0 + k] = acc[g][k];
        }
    } else if constexpr (MODE == 2) {
        if (wave == 0)
#pragma unroll
            for (int k = 0; k < RPL; ++k) partial[chunk * R + r0 + k] = make_double2(nrm[k], 0.0);
    }
}

// ------------------------------------------------------------------ delayed reorthogonalisation (DCGS2)
constexpr int kDotRows = 8;   // rows of u and w staged in LDS per step of the dot sweep

// Dot sweep: with u the candidate (slot k) and w = A u (slot k+1),
//   s_i = V_i^H u, z_i = V_i^H w (i < k), alpha = u^H u, beta = u^H w.
// Partials per chunk: [s_0..s_{k-1}, z_0..z_{k-1}, alpha, beta].  One launch
// covers the vectors i0 .. i0+nv-1 (the sweep may be split into launches of at
// most NW*G vectors); alpha and beta come from the launch with i0 = 0.
//
// Every wave of the workgroup needs the same rows of u and w: they are staged in
// LDS kDotRows rows at a time by all threads, so each value is read from memory
// once per workgroup (waves reading them independently drift apart over the
// chunk and re-fetch lines that the basis stream has evicted).  The next rows
// are fetched into registers while the staged ones are used, into the other
// half of the stage.  A wave loads RU rows of its G vectors before it uses any:
// RU * G loads in flight cover the memory latency, which bounds the sweep when
// a short batch leaves few workgroups on the chip.
template <typename TB, typename TV, int NW, int G, int RPL, bool HASW, int RU>
__global__ __launch_bounds__(NW * 64, (std::is_same<TV, p24x2>::value && G <= 4 ? 4 : 1)) void dcgs2_dots_kernel(const TV* __restrict__ V, int64_t vstride, int k,
                                                             int i0, int nv, const TB* __restrict__ u,
                                                             const TB* __restrict__ w, int64_t N, int R,
                                                             int64_t rows_per_chunk, double2* __restrict__ partial) {
    static_assert(kDotRows % RU == 0, "the stage holds whole groups of rows");
    // The next rows of V are loaded while these are used, but where the registers are short:
    // the packed basis with two vectors a wave or more, eight vectors.  Sweeps of 17 to 32 vectors
    // without it: FP32 pairs (7,936 folded rows of 1,024 RHS) 2,190 instead of 1,317 us, single
    // FP32 columns (8,959 of 289) 254 instead of 135, FP64 (11,625 of 258) 271 instead of 263.
    constexpr bool PF = G * RPL <= 2 || (sizeof(TV) == 8 && RPL == 2) || (!std::is_same<TV, p24x2>::value && G == 4);
    // blockIdx.z takes NW * G vectors of the launch's nv
    i0 += blockIdx.z * NW * G;
    nv = min(nv - (int)blockIdx.z * NW * G, NW * G);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: scalar branches and bases
    const int r0 = (blockIdx.x * 64 + lane) * RPL;
    const bool live = r0 < R;
    const unsigned rv = (unsigned)vofs<TV>(r0);   // this lane's word of a row
    const int64_t chunk = blockIdx.y;
    const int64_t n0 = chunk * rows_per_chunk;
    const int64_t n1 = min(N, n0 + rows_per_chunk);
    const int nred = 2 * k + 2;
    double2 as[G][RPL], az[G][RPL], aa[RPL], ab[RPL];
#pragma unroll
    for (int k2 = 0; k2 < RPL; ++k2) {
        aa[k2] = ab[k2] = make_double2(0, 0);
#pragma unroll
        for (int g = 0; g < G; ++g) as[g][k2] = az[g][k2] = make_double2(0, 0);
    }
    constexpr int NST = (kDotRows * 64 + NW * 64 - 1) / (NW * 64);   // staged values per thread
    __shared__ Raw<TB, RPL> su[2][kDotRows][64];
    __shared__ Raw<TB, RPL> sw[HASW ? 2 : 1][HASW ? kDotRows : 1][64];
    const bool ab_here = (i0 == 0) && (wave == 0);
    Raw<TB, RPL> pu[NST], pw[HASW ? NST : 1];
    auto fetch = [&](int64_t nb) {
#pragma unroll
        for (int j = 0; j < NST; ++j) {
            const int i = threadIdx.x + j * NW * 64;
            const int64_t n = nb + (i >> 6);
            const int c = (blockIdx.x * 64 + (i & 63)) * RPL;
            if (i < kDotRows * 64 && n < n1 && c < R) {
                pu[j].load(u + n * R + c);
                if (HASW) pw[j].load(w + n * R + c);
            } else {
                pu[j].zero();
                if (HASW) pw[j].zero();
            }
        }
    };
    // the RU rows of this wave's vectors from row n on; rows past the chunk are zero here
    // and in the stage: they add exact zeros
    Raw<TV, RPL> cur[RU][G], nxt[PF ? RU : 1][G];
    auto load_v = [&](int64_t n, Raw<TV, RPL>(&v)[RU][G]) {
#pragma unroll
        for (int q = 0; q < RU; ++q) {
            const int64_t off = vofs<TV>((n + q) * R);   // uniform: the row's offset
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int j = wave + NW * g;
                if (j < nv && (n + q < n1 || (RU == 1 && !PF))) v[q][g].load(V + (int64_t)(i0 + j) * vstride + off + rv);
                else v[q][g].zero();
            }
        }
    };
    fetch(n0);
    if (PF && live) load_v(n0, cur);
    int buf = 0;
    for (int64_t nb = n0; nb < n1; nb += kDotRows, buf ^= 1) {
        const int nrow = (int)min((int64_t)kDotRows, n1 - nb);
#pragma unroll
        for (int j = 0; j < NST; ++j) {
            const int i = threadIdx.x + j * NW * 64;
            if (i < kDotRows * 64) {
                su[buf][i >> 6][i & 63] = pu[j];
                if (HASW) sw[buf][i >> 6][i & 63] = pw[j];
            }
        }
        __syncthreads();
        if (nb + kDotRows < n1) fetch(nb + kDotRows);
        if (!live) continue;
        auto use_rows = [&](int rr) {
            if constexpr (!PF) load_v(nb + rr, cur);
            else load_v(nb + rr + RU, nxt);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < RU; ++q) {
#pragma unroll
                for (int k2 = 0; k2 < RPL; ++k2) {
                    // one value's widening at a time: hoisted above the others' it would spill
                    __builtin_amdgcn_sched_barrier(0);
                    const double2 uv = su[buf][rr + q][lane].get(k2);
                    const double2 wv = HASW ? sw[buf][rr + q][lane].get(k2) : make_double2(0, 0);
#pragma unroll
                    for (int g = 0; g < G; ++g) {
                        const double2 vv = cur[q][g].get(k2);
                        as[g][k2] = cfmac(as[g][k2], vv, uv);
                        if (HASW) az[g][k2] = cfmac(az[g][k2], vv, wv);
                    }
                }
            }
            if constexpr (PF)
#pragma unroll
                for (int q = 0; q < RU; ++q)
#pragma unroll
                    for (int g = 0; g < G; ++g) cur[q][g] = nxt[q][g];
        };
        if constexpr (PF) {
#pragma unroll
            for (int rr = 0; rr < kDotRows; rr += RU)
                if (rr < nrow) use_rows(rr);
        } else {
            for (int rr = 0; rr < nrow; rr += RU) use_rows(rr);
        }
        if (ab_here)
            for (int rr = 0; rr < nrow; ++rr) {
#pragma unroll
                for (int k2 = 0; k2 < RPL; ++k2) {
                    const double2 uv = su[buf][rr][lane].get(k2);
                    aa[k2].x = nfma(aa[k2].x, uv);
                    if (HASW) ab[k2] = cfmac(ab[k2], uv, sw[buf][rr][lane].get(k2));
                }
            }
    }
    if (!live) return;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const int j = wave + NW * g;
        if (j < nv)
#pragma unroll
            for (int k2 = 0; k2 < RPL; ++k2) {
                partial[(chunk * nred + i0 + j) * R + r0 + k2] = as[g][k2];
                partial[(chunk * nred + k + i0 + j) * R + r0 + k2] = az[g][k2];
            }
    }
    if (ab_here)
#pragma unroll
        for (int k2 = 0; k2 < RPL; ++k2) {
            partial[(chunk * nred + 2 * k) * R + r0 + k2] = aa[k2];
            partial[(chunk * nred + 2 * k + 1) * R + r0 + k2] = ab[k2];
        }
}

// Adds a workgroup's share of the RHS that still iterate to *counter (low half: the
// sum, high half: workgroups that have added theirs); the last of nwg workgroups
// reports the total to the host, tagged with the cycle's generation.
__device__ __forceinline__ void report_count(unsigned long long* counter, unsigned n, unsigned nwg,
                                             unsigned long long* host_slot, uint32_t gen) {
    const unsigned long long old =
        __hip_atomic_fetch_add(counter, (1ull << 32) | n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((unsigned)(old >> 32) == nwg - 1)
        __hip_atomic_store(host_slot, ((unsigned long long)gen << 32) | (uint32_t)((uint32_t)old + n), __ATOMIC_RELEASE,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

// Bookkeeping of DCGS2 step k (red: reduced [s, z, alpha, beta]) and the
// coefficients of its update sweep, one workgroup per kStepR right-hand sides.
// Completes Hessenberg column k-1 (raw and rotated), Givens, convergence;
// inv_nu[r] = 1/nu for a RHS that takes another step, 0 for one that stops.  Then
// t = Hbar_{k-1} s (rows 0..k), h = projections of A v_k (raw column k of H),
// c = t/nu + h; the coefficients of a RHS that stops are zero (coef = 0: no
// update follows).  The per-RHS recurrence is a chain of O(k) dependent
// operations, which bounds the kernel: its inputs are staged in LDS by all
// threads with the recurrence's scalars under way beside them, and one thread per RHS
// runs it from there while the other waves sum the coefficients' rows.  At 128 RHS and
// up to 32 vectors it takes 9.2 us on average (11.8 with the loads where they are
// needed and the sums at the end), where a thread per RHS walking global memory, a
// second kernel for the coefficients and a third for the count took 24 + 8 + 5 us and
// the host waited for a copy before the update could start.
constexpr int kStepR = 16;
constexpr int kStepRows = 32;                  // row threads per RHS
constexpr int kStepSum = kStepRows - 64 / kStepR;   // those outside wave 0
constexpr int kStepOwn = (kMaxVec + kStepSum - 1) / kStepSum;
__global__ __launch_bounds__(kStepR * kStepRows) void dcgs2_step_kernel(GmresState st, double2* __restrict__ Hraw,
                                                                       const double2* __restrict__ red, int R, int k,
                                                                       int m, int coef, double* __restrict__ inv_nu,
                                                                       double2* __restrict__ cs_out,
                                                                       double2* __restrict__ cc_out,
                                                                       unsigned long long* counter,
                                                                       unsigned long long* host_slot, uint32_t gen) {
    __shared__ double2 S[kMaxVec][kStepR], Z[kMaxVec][kStepR];
    __shared__ double2 HC[kMaxVec][kStepR], HJ[kMaxVec][kStepR];   // column k-1: raw, rotated
    __shared__ double2 sn[kMaxVec][kStepR];
    __shared__ double cs[kMaxVec][kStepR];
    __shared__ double inus[kStepR];
    const int rr = threadIdx.x % kStepR, ti = threadIdx.x / kStepR;
    const int r = blockIdx.x * kStepR + rr;
    const bool valid = r < R;
    const bool act = valid && st.active[r] != 0;
    const int64_t ldH = (int64_t)(m + 1) * R;
    double2* Hc = Hraw + (int64_t)(k > 0 ? k - 1 : 0) * ldH;
    // the scalars of the recurrence, under way with the column
    double alpha = 0, beta0 = 0, bnorm = 0;
    double2 gj = make_double2(0, 0);
    int iters = 0;
    if (ti == 0 && valid) {
        alpha = red[(int64_t)(2 * k) * R + r].x;
        if (k == 0) beta0 = st.beta[r];
        else gj = st.g[(int64_t)(k - 1) * R + r];
        bnorm = st.bnorm[r];
        iters = st.iters[r];
    }
    if (valid)
        for (int i = ti; i < k; i += kStepRows) {
            const double2 s = red[(int64_t)i * R + r];
            const double2 z = red[(int64_t)(k + i) * R + r];
            const double2 h = cadd(Hc[(int64_t)i * R + r], s);
            if (i < k - 1) {
                cs[i][rr] = st.cs[(int64_t)i * R + r];
                sn[i][rr] = st.sn[(int64_t)i * R + r];
            }
            S[i][rr] = s;
            Z[i][rr] = z;
            if (act) Hc[(int64_t)i * R + r] = h;
            HC[i][rr] = h;
            HJ[i][rr] = h;
        }
    __syncthreads();
    // Wave 0 runs the recurrence; the rows of t (all but its last term, which needs the
    // recurrence's nu) are summed by the others meanwhile: row i by row thread 4 + i mod kStepSum.
    const int own = ti - 64 / kStepR;
    double2 t[kStepOwn], sz = make_double2(0, 0);
    if (own >= 0 && valid && coef) {
#pragma unroll
        for (int e = 0; e < kStepOwn; ++e) {
            const int i = own + e * kStepSum;
            t[e] = make_double2(0, 0);
            if (i > k) continue;
            const double2* Hi = Hraw + (int64_t)i * R + r;
#pragma unroll 8
            for (int l = (i > 0 ? i - 1 : 0); l < k - 1; ++l)   // Hbar is upper Hessenberg: H[i][l] = 0 for l < i-1
                t[e] = cadd(t[e], cmul(Hi[(int64_t)l * ldH], S[l][rr]));
            if (i == k) {
                for (int l = 0; l < k; ++l) sz = cadd(sz, cmulc(S[l][rr], Z[l][rr]));
                sz = csub(red[(int64_t)(2 * k + 1) * R + r], sz);
            }
        }
    }
    if (ti == 0) {
        double inu = 0.0;
        if (act) {
            double ss = 0;
            for (int i = 0; i < k; ++i) {
                const double2 s = S[i][rr];
                ss += s.x * s.x + s.y * s.y;
            }
            // nu^2 by Pythagoras loses its relative accuracy as ss -> alpha: below
            // 1e-12 alpha the candidate lies in the span of the basis (breakdown)
            const double nu = (alpha - ss > 1e-12 * alpha) ? sqrt(alpha - ss) : 0.0;
            bool stop = false;
            if (k == 0) {
                st.g[r] = make_double2(beta0 * nu, 0.0);
            } else {
                HC[k][rr] = make_double2(nu, 0.0);
                Hc[(int64_t)k * R + r] = make_double2(nu, 0.0);
                const int j = k - 1;
                double2 a = HJ[0][rr];
                for (int i = 0; i < j; ++i) {
                    const double c = cs[i][rr];
                    const double2 sv = sn[i][rr];
                    const double2 b = HJ[i + 1][rr];
                    HJ[i][rr] = cadd(make_double2(c * a.x, c * a.y), cmul(sv, b));
                    a = csub(make_double2(c * b.x, c * b.y), cmulc(sv, a));
                }
                const double2 h1v = a;
                double c;
                double2 sv;
                const double a1 = hypot(h1v.x, h1v.y);
                if (a1 == 0.0) {
                    c = 0.0;
                    sv = make_double2(1.0, 0.0);
                } else {
                    const double d = hypot(a1, nu);
                    c = a1 / d;
                    sv = make_double2(h1v.x / a1 * nu / d, h1v.y / a1 * nu / d);
                }
                st.cs[(int64_t)j * R + r] = c;
                st.sn[(int64_t)j * R + r] = sv;
                HJ[j][rr] = cadd(make_double2(c * h1v.x, c * h1v.y), make_double2(sv.x * nu, sv.y * nu));
                HJ[k][rr] = make_double2(0, 0);
                const double2 gn = make_double2(-(sv.x * gj.x + sv.y * gj.y), -(sv.x * gj.y - sv.y * gj.x));
                st.g[(int64_t)j * R + r] = make_double2(c * gj.x, c * gj.y);
                st.g[(int64_t)(j + 1) * R + r] = gn;
                st.iters[r] = iters + 1;
                st.kcyc[r] = k;
                const double res = hypot(gn.x, gn.y);
                if (!(nu == nu) || isinf(nu) || !(res == res)) {
                    st.flag[r] = 1;
                    stop = true;
                } else if (res <= st.tol * bnorm || nu == 0.0 || k == m) {
                    stop = true;
                }
            }
            if (stop || k == m || nu == 0.0) st.active[r] = 0;
            else inu = 1.0 / nu;
        }
        inus[rr] = inu;
        if (valid) inv_nu[r] = inu;
    }
    __syncthreads();
    if (act && k > 0)
        for (int i = ti; i <= k; i += kStepRows) st.H[(int64_t)(k - 1) * ldH + (int64_t)i * R + r] = HJ[i][rr];
    if (threadIdx.x == 0) {
        unsigned n = 0;
        for (int q = 0; q < kStepR; ++q) n += inus[q] != 0.0 ? 1 : 0;
        report_count(counter, n, gridDim.x, host_slot, gen);
    }
    if (!coef || !valid || own < 0) return;
    const double in = inus[rr];
#pragma unroll
    for (int e = 0; e < kStepOwn; ++e) {
        const int i = own + e * kStepSum;
        if (i > k) continue;
        if (in == 0.0) {
            if (i < k) cs_out[(int64_t)i * R + r] = make_double2(0, 0);
            cc_out[(int64_t)i * R + r] = make_double2(0, 0);
            continue;
        }
        if (k > 0) t[e] = cadd(t[e], cmul(HC[i][rr], S[k - 1][rr]));
        double2 h;
        if (i < k) {
            const double2 d = csub(Z[i][rr], t[e]);
            h = make_double2(d.x * in, d.y * in);
            cs_out[(int64_t)i * R + r] = S[i][rr];
        } else {
            h = make_double2((sz.x * in - t[e].x) * in, (sz.y * in - t[e].y) * in);
        }
        Hraw[(int64_t)k * ldH + (int64_t)i * R + r] = h;
        cc_out[(int64_t)i * R + r] = make_double2(t[e].x * in + h.x, t[e].y * in + h.y);
    }
}

// Whether a sweep of `groups` workgroups spreads its vectors over several workgroups of
// eight (each stages u and w again, from cache).  It does where whole ones leave CUs idle or
// leave a few CUs with two: there a sweep waits for its loads rather than for memory
// bandwidth.  Packed basis, split against whole: 124 workgroups 59 against 92 us, 248 114
// against 117, 320 31 against 36, 343 20 against 19.  FP64: 124 94 against 107, 273 98
// against 114; but one workgroup a CU is as fast whole there (132: 23 against 22.5) or faster
// (240: 33 against 31; 248: 179 against 162).
template <typename TB> bool dots_split(int64_t groups) {
    return groups <= 330 && !(sizeof(TB) == 16 && groups > 192 && groups <= 256);
}

// rows whose loads a wave of G vectors issues together: eight loads in flight, or as many as
// fit beside the accumulators (two RHS per lane) and the rows loaded ahead without spilling
template <typename TV, int NW, int G, int RPL> constexpr int dot_ru() {
    if (sizeof(TV) == 8 && RPL == 2 && G > 1) return G == 2 ? 2 : 1;
    if (sizeof(TV) == 16 && G == 4) return 1;
    return G * RPL >= 8 ? 1 : (RPL == 2 && NW == 4) ? 2 : (RPL == 2 && G == 1) ? 4 : 8 / G;
}

template <typename TB, typename TV, int NW, int G, int RPL, bool HASW>
void launch_dcgs2_dots_cfg(const TV* V, int64_t vs, int k, int i0, int nv, const TB* u, const TB* w, int64_t N, int R,
                           int64_t rpc, int nchunk, double2* partial, hipStream_t s) {
    const dim3 grid((unsigned)((R / RPL + 63) / 64), (unsigned)nchunk, (unsigned)std::max(1, (nv + NW * G - 1) / (NW * G)));
    hipLaunchKernelGGL((dcgs2_dots_kernel<TB, TV, NW, G, RPL, HASW, dot_ru<TV, NW, G, RPL>()>), grid, dim3(NW * 64), 0, s, V, vs, k,
                       i0, nv, u, w, N, R, rpc, partial);
    MBT_LAUNCH_CHECK();
}

template <typename TB, typename TV, int RPL, bool HASW>
void launch_dcgs2_dots_rpl(const TV* V, int64_t vs, int k, int i0, int nv, const TB* u, const TB* w, int64_t N, int R,
                           int64_t rpc, int nchunk, double2* partial, hipStream_t s) {
    const int64_t groups = (int64_t)((R / RPL + 63) / 64) * nchunk;
    if (nv <= 4)
        launch_dcgs2_dots_cfg<TB, TV, 4, 1, RPL, HASW>(V, vs, k, i0, nv, u, w, N, R, rpc, nchunk, partial, s);
    else if (nv <= 8 || dots_split<TB>(groups))
        launch_dcgs2_dots_cfg<TB, TV, 8, 1, RPL, HASW>(V, vs, k, i0, nv, u, w, N, R, rpc, nchunk, partial, s);
    else if (nv <= 16)
        launch_dcgs2_dots_cfg<TB, TV, 8, 2, RPL, HASW>(V, vs, k, i0, nv, u, w, N, R, rpc, nchunk, partial, s);
    else if (nv <= 32)
        launch_dcgs2_dots_cfg<TB, TV, 8, 4, RPL, HASW>(V, vs, k, i0, nv, u, w, N, R, rpc, nchunk, partial, s);
    else
        launch_dcgs2_dots_cfg<TB, TV, 8, 8, RPL, HASW>(V, vs, k, i0, nv, u, w, N, R, rpc, nchunk, partial, s);
}

// The dot sweep of a short row (R <= 64 columns): a lane per column leaves most of a
// wave idle, so here a wave takes GV = 64 / 2^lgc vectors at once (2^lgc >= R lanes
// each), and the rows of a stage are GV times as many.  Per (vector, column) it adds
// the rows of the chunk in order as dcgs2_dots_kernel does, so the sums are the same.
// The rows come one group of loads after another, which bounds it.  Packed basis, up
// to 50 vectors: 11,625 rows of 8 columns in 23 us (58 with a lane per two columns), 3,072
// of 32 in 8.7 (13); 16 rows a group measured the same.
constexpr int kNarW = 4;          // waves
constexpr int kNarStage = 512;    // staged values of u and of w
constexpr int kNarRows = 8;       // rows whose loads a lane issues together
template <typename T> struct NarRaw { using type = Raw<T, 1>; };
template <> struct NarRaw<p24x2> { using type = Raw<p24x2, 2>; };
template <typename TB, typename TV, bool HASW>
__global__ __launch_bounds__(kNarW * 64) void dcgs2_dots_narrow_kernel(const TV* __restrict__ V, int64_t vstride, int k,
                                                                      const TB* __restrict__ u,
                                                                      const TB* __restrict__ w, int64_t N, int R,
                                                                      int lgc, int64_t rows_per_chunk,
                                                                      double2* __restrict__ partial) {
    using RV = typename NarRaw<TV>::type;
    constexpr int NST = kNarStage / (kNarW * 64);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & ((1 << lgc) - 1);
    const int j = (((int)blockIdx.y * kNarW + wave) << (6 - lgc)) + (lane >> lgc);   // this lane's vector
    const int64_t chunk = blockIdx.x;
    const int64_t n0 = chunk * rows_per_chunk;
    const int64_t n1 = min(N, n0 + rows_per_chunk);
    const int nred = 2 * k + 2;
    const int srows = kNarStage >> lgc;   // rows of a stage
    const bool live = c < R && j < k;
    const bool ab_here = blockIdx.y == 0 && wave == 0 && c < R && (lane >> lgc) == 0;
    double2 as = make_double2(0, 0), az = as, aa = as, ab = as;
    __shared__ Raw<TB, 1> su[2][kNarStage];
    __shared__ Raw<TB, 1> sw[HASW ? 2 : 1][HASW ? kNarStage : 1];
    Raw<TB, 1> pu[NST], pw[HASW ? NST : 1];
    auto fetch = [&](int64_t nb) {
#pragma unroll
        for (int q = 0; q < NST; ++q) {
            const int i = threadIdx.x + q * kNarW * 64;
            const int64_t n = nb + (i >> lgc);
            const int col = i & ((1 << lgc) - 1);
            if (n < n1 && col < R) {
                pu[q].load(u + n * R + col);
                if (HASW) pw[q].load(w + n * R + col);
            } else {
                pu[q].zero();
                if (HASW) pw[q].zero();
            }
        }
    };
    RV va[kNarRows], vb[kNarRows];
    const TV* Vj = V + (int64_t)j * vstride;
    auto load_v = [&](int64_t n, RV(&v)[kNarRows]) {
#pragma unroll
        for (int q = 0; q < kNarRows; ++q) {
            if (live && n + q < n1) v[q].load(Vj + vofs<TV>((n + q) * R + c));
            else v[q].zero();
        }
    };
    // the group of rows from n on (row rr of its stage), in cur, while the next one's loads go to nxt
    auto group = [&](int64_t n, RV(&cur)[kNarRows], RV(&nxt)[kNarRows]) {
        const int rr = (int)(n - n0) % srows;
        const int buf = (int)((n - n0) / srows) & 1;
        if (rr == 0) {
#pragma unroll
            for (int q = 0; q < NST; ++q) {
                const int i = threadIdx.x + q * kNarW * 64;
                su[buf][i] = pu[q];
                if (HASW) sw[buf][i] = pw[q];
            }
            __syncthreads();
            fetch(n + srows);
        }
        load_v(n + kNarRows, nxt);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int q = 0; q < kNarRows; ++q) {
            const int i = ((rr + q) << lgc) + c;
            const double2 vv = cur[q].get(c & 1);
            as = cfmac(as, vv, su[buf][i].get(0));
            if (HASW) az = cfmac(az, vv, sw[buf][i].get(0));
        }
        if (ab_here)
#pragma unroll
            for (int q = 0; q < kNarRows; ++q) {
                const int i = ((rr + q) << lgc) + c;
                const double2 uv = su[buf][i].get(0);
                aa.x = nfma(aa.x, uv);
                if (HASW) ab = cfmac(ab, uv, sw[buf][i].get(0));
            }
    };
    fetch(n0);
    load_v(n0, va);
    for (int64_t n = n0; n < n1; n += 2 * kNarRows) {
        group(n, va, vb);
        if (n + kNarRows < n1) group(n + kNarRows, vb, va);
    }
    if (live) {
        partial[(chunk * nred + j) * R + c] = as;
        partial[(chunk * nred + k + j) * R + c] = az;
    }
    if (ab_here) {
        partial[(chunk * nred + 2 * k) * R + c] = aa;
        partial[(chunk * nred + 2 * k + 1) * R + c] = ab;
    }
}

template <typename TB, typename TV, bool HASW>
void launch_dcgs2_dots_narrow(const TV* V, int64_t vs, int k, const TB* u, const TB* w, int64_t N, int R, int64_t rpc,
                              int nchunk, double2* partial, hipStream_t s) {
    int lgc = 0;
    while ((1 << lgc) < R) ++lgc;
    // a stage has a multiple of kNarRows rows
    MBT_REQUIRE(lgc <= 6 && (kNarStage >> lgc) % kNarRows == 0, "narrow dot sweep: row too long");
    const int per = kNarW << (6 - lgc);   // vectors of a workgroup
    hipLaunchKernelGGL((dcgs2_dots_narrow_kernel<TB, TV, HASW>),
                       dim3((unsigned)nchunk, (unsigned)std::max(1, (k + per - 1) / per)), dim3(kNarW * 64), 0, s, V, vs, k,
                       u, w, N, R, lgc, rpc, partial);
    MBT_LAUNCH_CHECK();
}

// Row-split update sweep: each wave owns RB consecutive rows of 64 RHS columns
// and walks all k basis vectors itself, so there is no cross-wave reduction and
// no workgroup barrier; the per-RHS coefficients are re-read (from L2) for each
// block of rows.  The next VU vectors' rows are loaded while the current ones are
// accumulated.  Summation over i is sequential per (row, RHS), whatever RB and VU.
template <typename TB, int RB, int VU>
__global__ __launch_bounds__(256) void dcgs2_update_rows_kernel(const TB* __restrict__ V, int64_t vstride, int k,
                                                                TB* u, TB* w, const double2* __restrict__ cs_,
                                                                const double2* __restrict__ cc_,
                                                                const double* __restrict__ inv_nu_, int64_t total,
                                                                int R, int Rt,
                                                                const unsigned long long* __restrict__ live) {
    if ((uint32_t)*live == 0) return;   // every RHS has stopped (the host may not know yet)
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int r = blockIdx.x * 64 + lane;
    const int64_t n0 = ((int64_t)blockIdx.y * 4 + wave) * RB;
    if (r >= R || n0 * R + r >= total) return;
    // folded rows (R = F * Rt columns per row): column r is RHS r mod Rt
    const int rt = r % Rt;
    const double2* cs = cs_ + rt;
    const double2* cc = cc_ + rt;
    const double* inv_nu = inv_nu_ + rt;
    int nr = RB;   // rows that have this column (the last row may be shorter)
    while ((n0 + nr - 1) * R + r >= total) --nr;
    double2 a[RB], c[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) a[j] = c[j] = make_double2(0, 0);
    const TB* base = V + n0 * R + r;
    Raw<TB, 1> cur[VU][RB], nxt[VU][RB];
    double2 fs[VU], fc[VU], fs_n[VU], fc_n[VU];
    auto load = [&](int i0, Raw<TB, 1>(&v)[VU][RB], double2(&s)[VU], double2(&t)[VU]) {
#pragma unroll
        for (int q = 0; q < VU; ++q) {
            const int i = i0 + q;
            s[q] = t[q] = make_double2(0, 0);
            if (i < k) {
                s[q] = cs[(int64_t)i * Rt];
                t[q] = cc[(int64_t)i * Rt];
            }
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                if (i < k && j < nr) v[q][j].load(base + i * vstride + (int64_t)j * R);
                else v[q][j].zero();
            }
        }
    };
    load(0, cur, fs, fc);
    for (int i = 0; i < k; i += VU) {
        load(i + VU, nxt, fs_n, fc_n);
#pragma unroll
        for (int q = 0; q < VU; ++q) {
            if (VU > 1 && i + q >= k) break;
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                const double2 vv = cur[q][j].get(0);
                a[j] = cfma(a[j], fs[q], vv);
                c[j] = cfma(c[j], fc[q], vv);
            }
        }
#pragma unroll
        for (int q = 0; q < VU; ++q) {
#pragma unroll
            for (int j = 0; j < RB; ++j) cur[q][j] = nxt[q][j];
            fs[q] = fs_n[q];
            fc[q] = fc_n[q];
        }
    }
    const double inu = inv_nu[0];
    const double2 ckv = cc[(int64_t)k * Rt];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        if (j < nr) {
            const int64_t off = (n0 + j) * R + r;
            const double2 d = csub(ld2(u + off), a[j]);
            const double2 vk = make_double2(d.x * inu, d.y * inu);
            const double2 wv = ld2(w + off);
            const double2 un = next_candidate(wv, inu, c[j], ckv, vk);
            st2(u + off, vk);
            st2(w + off, un);
        }
    }
}

// Row-split update sweep into the packed basis: as dcgs2_update_rows_kernel,
// with a lane owning two adjacent RHS columns (one packed word per row).  v_k
// goes to its own slot vk (rounded to the packed format, and the rounded value
// is the one removed from u_{k+1}); u_{k+1} overwrites u.
template <int RB, int VU>
__global__ __launch_bounds__(256) void dcgs2_update_rows24_kernel(const p24x2* __restrict__ V, int64_t vstride, int k,
                                                                  float2* u, const float2* __restrict__ w,
                                                                  p24x2* __restrict__ vk, const double2* __restrict__ cs_,
                                                                  const double2* __restrict__ cc_,
                                                                  const double* __restrict__ inv_nu_, int64_t total,
                                                                  int R, int Rt,
                                                                  const unsigned long long* __restrict__ live) {
    if ((uint32_t)*live == 0) return;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int r0 = 2 * (blockIdx.x * 64 + lane);
    const int64_t n0 = ((int64_t)blockIdx.y * 4 + wave) * RB;
    if (r0 >= R || n0 * R + r0 >= total) return;
    // folded rows (R = F * Rt columns per row, Rt even): columns r0, r0+1 are RHS r0 mod Rt and the next
    const int rt = r0 % Rt;
    const double2* cs = cs_ + rt;
    const double2* cc = cc_ + rt;
    const double* inv_nu = inv_nu_ + rt;
    int nr = RB;   // rows that have this column (the last row may be shorter)
    while ((n0 + nr - 1) * R + r0 >= total) --nr;
    const int64_t rw = R / 2;   // packed words per row
    double2 a[RB][2], c[RB][2];
#pragma unroll
    for (int j = 0; j < RB; ++j)
#pragma unroll
        for (int q = 0; q < 2; ++q) a[j][q] = c[j][q] = make_double2(0, 0);
    const p24x2* base = V + (n0 * R + r0) / 2;
    Raw<p24x2, 2> cur[VU][RB], nxt[VU][RB];
    double2 fs[VU][2], fc[VU][2], fs_n[VU][2], fc_n[VU][2];
    auto load = [&](int i0, Raw<p24x2, 2>(&v)[VU][RB], double2(&s)[VU][2], double2(&t)[VU][2]) {
#pragma unroll
        for (int e = 0; e < VU; ++e) {
            const int i = i0 + e;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                s[e][q] = t[e][q] = make_double2(0, 0);
                if (i < k) {
                    s[e][q] = cs[(int64_t)i * Rt + q];
                    t[e][q] = cc[(int64_t)i * Rt + q];
                }
            }
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                if (i < k && j < nr) v[e][j].load(base + i * vstride + (int64_t)j * rw);
                else v[e][j].zero();
            }
        }
    };
    load(0, cur, fs, fc);
    for (int i = 0; i < k; i += VU) {
        load(i + VU, nxt, fs_n, fc_n);
#pragma unroll
        for (int e = 0; e < VU; ++e) {
            if (VU > 1 && i + e >= k) break;
#pragma unroll
            for (int j = 0; j < RB; ++j)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const double2 vv = cur[e][j].get(q);
                    a[j][q] = cfma(a[j][q], fs[e][q], vv);
                    c[j][q] = cfma(c[j][q], fc[e][q], vv);
                }
        }
#pragma unroll
        for (int e = 0; e < VU; ++e) {
#pragma unroll
            for (int j = 0; j < RB; ++j) cur[e][j] = nxt[e][j];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                fs[e][q] = fs_n[e][q];
                fc[e][q] = fc_n[e][q];
            }
        }
    }
    double inu[2];
    double2 ckv[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        inu[q] = inv_nu[q];
        ckv[q] = cc[(int64_t)k * Rt + q];
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        if (j < nr) {
            const int64_t off = (n0 + j) * R + r0;
            double2 uv[2], wv[2], v[2], un[2];
            ldp<2>(u + off, uv);
            ldp<2>(w + off, wv);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const double2 d = csub(uv[q], a[j][q]);
                v[q] = round24(make_double2(d.x * inu[q], d.y * inu[q]));
                un[q] = next_candidate(wv[q], inu[q], c[j][q], ckv[q], v[q]);
            }
            st24(vk + off / 2, v[0], v[1]);
            stp<2>(u + off, un);
        }
    }
}

// Rows per wave of the row-split sweeps.  Eight rows amortise the coefficients
// over the basis traffic once the waves fill the chip; a short batch leaves each
// wave alone on its CU, waiting one memory latency per vector, so below kFewWaves
// waves of eight rows it takes two rows and four vectors at a time instead.  Update
// sweep, two rows against eight: packed basis 992 waves 23 against 25 us, 1,052 26
// against 48, 1,841 42 against 32, 1,984 49 against 38; FP64 526 24 against 26, 951 30 against
// 32, 1,274 52 against 52, 1,841 74 against 67, 1,984 73 against 70.
constexpr int64_t kFewWaves = 1280;

// These sweeps treat every column of a row alike and know a column's RHS by its place
// mod Rt, so rows shorter than half a wave (lanes of them: a column or a packed word
// each) are joined: `join` rows make one, the last of which may be shorter.  At 11,625
// rows of 8 columns the packed update takes 8 instead of 33 us.
inline int join_rows(int64_t lanes) { return lanes > 32 ? 1 : (int)(64 / lanes); }
inline bool few_waves(int64_t N, int64_t lanes) {
    const int join = join_rows(lanes);
    N = (N + join - 1) / join;
    return ((N + 7) / 8) * ((lanes * join + 63) / 64) < kFewWaves;
}

template <int RB, int VU>
void launch_dcgs2_update24_rb(const p24x2* V, int64_t vs, int k, float2* u, const float2* w, p24x2* vk,
                              const double2* cs, const double2* cc, const double* inv_nu, int64_t N, int R, int Rt,
                              const unsigned long long* live, hipStream_t s) {
    const int64_t total = N * R;
    const int join = join_rows(R / 2);
    N = (N + join - 1) / join;
    R *= join;
    const int64_t gy = (N + 4 * RB - 1) / (4 * RB);
    MBT_REQUIRE(gy < 65536, "dcgs2 update: too many row blocks");
    hipLaunchKernelGGL((dcgs2_update_rows24_kernel<RB, VU>), dim3((unsigned)((R / 2 + 63) / 64), (unsigned)gy), dim3(256),
                       0, s, V, vs, k, u, w, vk, cs, cc, inv_nu, total, R, Rt, live);
    MBT_LAUNCH_CHECK();
}

void launch_dcgs2_update24(const p24x2* V, int64_t vs, int k, float2* u, const float2* w, p24x2* vk,
                           const double2* cs, const double2* cc, const double* inv_nu, int64_t N, int R, int Rt,
                           const unsigned long long* live, hipStream_t s) {
    MBT_REQUIRE(R % 2 == 0, "packed basis needs an even number of RHS");
    MBT_REQUIRE(Rt % 2 == 0 && R % Rt == 0, "packed basis: folded width must be a multiple of the even RHS count");
    if (few_waves(N, R / 2)) launch_dcgs2_update24_rb<2, 4>(V, vs, k, u, w, vk, cs, cc, inv_nu, N, R, Rt, live, s);
    else launch_dcgs2_update24_rb<8, 1>(V, vs, k, u, w, vk, cs, cc, inv_nu, N, R, Rt, live, s);
}

// End of a cycle: x += sum_{i < steps} y_i V_i.  Each wave owns RB rows of 64
// lanes (RPL adjacent RHS per lane) and walks the vectors in order, so a
// RHS's sum has the same order whatever the batch and however long the cycle
// of the other RHS ran.
template <typename TV, int RPL, int RB, int VU>
__global__ __launch_bounds__(256) void solution_update_kernel(const TV* __restrict__ V, int64_t vstride, int steps,
                                                              const double2* __restrict__ y_, double2* __restrict__ x,
                                                              int64_t total, int R, int Rt) {
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int r0 = (blockIdx.x * 64 + lane) * RPL;
    const int64_t n0 = ((int64_t)blockIdx.y * 4 + wave) * RB;
    if (r0 >= R || n0 * R + r0 >= total) return;
    const double2* y = y_ + r0 % Rt;   // folded rows: column r0 is RHS r0 mod Rt
    int nr = RB;   // rows that have this column (the last row may be shorter)
    while ((n0 + nr - 1) * R + r0 >= total) --nr;
    double2 acc[RB][RPL];
#pragma unroll
    for (int j = 0; j < RB; ++j)
#pragma unroll
        for (int q = 0; q < RPL; ++q) acc[j][q] = make_double2(0, 0);
    Raw<TV, RPL> cur[VU][RB], nxt[VU][RB];
    double2 yc[VU][RPL], yn[VU][RPL];
    auto load = [&](int i0, Raw<TV, RPL>(&v)[VU][RB], double2(&c)[VU][RPL]) {
#pragma unroll
        for (int e = 0; e < VU; ++e) {
            const int i = i0 + e;
#pragma unroll
            for (int q = 0; q < RPL; ++q) c[e][q] = i < steps ? y[(int64_t)i * Rt + q] : make_double2(0, 0);
#pragma unroll
            for (int j = 0; j < RB; ++j) {
                if (i < steps && j < nr) v[e][j].load(V + i * vstride + vofs<TV>((n0 + j) * R + r0));
                else v[e][j].zero();
            }
        }
    };
    load(0, cur, yc);
    for (int i = 0; i < steps; i += VU) {
        load(i + VU, nxt, yn);
#pragma unroll
        for (int e = 0; e < VU; ++e) {
            if (VU > 1 && i + e >= steps) break;
#pragma unroll
            for (int j = 0; j < RB; ++j)
#pragma unroll
                for (int q = 0; q < RPL; ++q) acc[j][q] = cfma(acc[j][q], yc[e][q], cur[e][j].get(q));
        }
#pragma unroll
        for (int e = 0; e < VU; ++e) {
#pragma unroll
            for (int j = 0; j < RB; ++j) cur[e][j] = nxt[e][j];
#pragma unroll
            for (int q = 0; q < RPL; ++q) yc[e][q] = yn[e][q];
        }
    }
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        if (j < nr) {
            const int64_t off = (n0 + j) * R + r0;
#pragma unroll
            for (int q = 0; q < RPL; ++q) x[off + q] = cadd(x[off + q], acc[j][q]);
        }
    }
}

template <typename TV, int RPL, int RB, int VU>
void launch_solution_update_rb(const TV* V, int64_t vs, int steps, const double2* y, double2* x, int64_t N, int R,
                               int Rt, hipStream_t s) {
    const int64_t total = N * R;
    const int join = join_rows(R / RPL);
    N = (N + join - 1) / join;
    R *= join;
    const int64_t gy = (N + 4 * RB - 1) / (4 * RB);
    MBT_REQUIRE(gy < 65536, "solution update: too many row blocks");
    hipLaunchKernelGGL((solution_update_kernel<TV, RPL, RB, VU>), dim3((unsigned)((R / RPL + 63) / 64), (unsigned)gy),
                       dim3(256), 0, s, V, vs, steps, y, x, total, R, Rt);
    MBT_LAUNCH_CHECK();
}

template <typename TV>
void launch_solution_update(const TV* V, int64_t vs, int steps, const double2* y, double2* x, int64_t N, int R,
                            int Rt, hipStream_t s) {
    MBT_REQUIRE(R % Rt == 0, "folded width must be a multiple of the RHS count");
    constexpr int RPL = PerWord<TV>::v;
    MBT_REQUIRE(R % RPL == 0, "packed basis needs an even number of RHS");
    if (few_waves(N, R / RPL)) launch_solution_update_rb<TV, RPL, 2, 4>(V, vs, steps, y, x, N, R, Rt, s);
    else launch_solution_update_rb<TV, RPL, 8, 1>(V, vs, steps, y, x, N, R, Rt, s);
}

template <typename TB, typename TV>
void launch_dcgs2_dots(const TV* V, int64_t vs, int k, const TB* u, const TB* w, int64_t N, int R, int64_t rpc,
                       int nchunk, double2* partial, hipStream_t s) {
    // half a wave's lanes or fewer in use (a lane owns two columns where FP32 rows are even)
    const bool pairs = sizeof(TB) == 8 && R % 2 == 0;
    if (R <= (pairs ? 64 : 32) && (pairs || std::is_same<TV, TB>::value)) {
        if (w) launch_dcgs2_dots_narrow<TB, TV, true>(V, vs, k, u, w, N, R, rpc, nchunk, partial, s);
        else launch_dcgs2_dots_narrow<TB, TV, false>(V, vs, k, u, w, N, R, rpc, nchunk, partial, s);
        return;
    }
    if constexpr (sizeof(TB) == 8) {
        if (R % 2 == 0) {
            // FP32 pairs of RHS per lane (16-byte accesses) fit the register budget up to 32
            // vectors per launch: longer sweeps are split, re-reading u and w once more
            for (int i0 = 0; i0 == 0 || i0 < k; i0 += 32) {
                const int nv = std::min(32, k - i0);
                if (w) launch_dcgs2_dots_rpl<TB, TV, 2, true>(V, vs, k, i0, nv, u, w, N, R, rpc, nchunk, partial, s);
                else launch_dcgs2_dots_rpl<TB, TV, 2, false>(V, vs, k, i0, nv, u, w, N, R, rpc, nchunk, partial, s);
            }
            return;
        }
    }
    if constexpr (std::is_same<TV, TB>::value) {
        if (w) launch_dcgs2_dots_rpl<TB, TV, 1, true>(V, vs, k, 0, k, u, w, N, R, rpc, nchunk, partial, s);
        else launch_dcgs2_dots_rpl<TB, TV, 1, false>(V, vs, k, 0, k, u, w, N, R, rpc, nchunk, partial, s);
    } else {
        throw Error(-1, "packed basis needs an even number of RHS");
    }
}

template <typename TB, int RB, int VU>
void launch_dcgs2_update_rb(const TB* V, int64_t vs, int k, TB* u, TB* w, const double2* cs, const double2* cc,
                            const double* inv_nu, int64_t N, int R, int Rt, const unsigned long long* live,
                            hipStream_t s) {
    const int64_t total = N * R;
    const int join = join_rows(R);
    N = (N + join - 1) / join;
    R *= join;
    const int64_t gy = (N + 4 * RB - 1) / (4 * RB);
    MBT_REQUIRE(gy < 65536, "dcgs2 update: too many row blocks");
    hipLaunchKernelGGL((dcgs2_update_rows_kernel<TB, RB, VU>), dim3((unsigned)((R + 63) / 64), (unsigned)gy), dim3(256), 0,
                       s, V, vs, k, u, w, cs, cc, inv_nu, total, R, Rt, live);
    MBT_LAUNCH_CHECK();
}

template <typename TB>
void launch_dcgs2_update(const TB* V, int64_t vs, int k, TB* u, TB* w, const double2* cs, const double2* cc,
                         const double* inv_nu, int64_t N, int R, int Rt, const unsigned long long* live,
                         hipStream_t s) {
    MBT_REQUIRE(R % Rt == 0, "folded width must be a multiple of the RHS count");
    if (few_waves(N, R)) launch_dcgs2_update_rb<TB, 2, 4>(V, vs, k, u, w, cs, cc, inv_nu, N, R, Rt, live, s);
    else launch_dcgs2_update_rb<TB, 8, 1>(V, vs, k, u, w, cs, cc, inv_nu, N, R, Rt, live, s);
}

template <typename TB, typename TO, int MODE, int RPL>
void launch_pass_rpl(const TB* V, int64_t vs, int nvec, const double2* coef, TO* w, int64_t N, int R, int64_t rpc,
                     int nchunk, double2* partial, hipStream_t s, int cfg_n) {
    const dim3 grid((unsigned)((R / RPL + 63) / 64), (unsigned)nchunk);
    if (cfg_n <= 4)
        hipLaunchKernelGGL((arnoldi_kernel<TB, TO, MODE, 4, 1, RPL>), grid, dim3(256), 0, s, V, vs, nvec, coef, w, N, R, rpc, partial);
    else if (cfg_n <= 8)
        hipLaunchKernelGGL((arnoldi_kernel<TB, TO, MODE, 4, 2, RPL>), grid, dim3(256), 0, s, V, vs, nvec, coef, w, N, R, rpc, partial);
    else if (cfg_n <= 16)
        hipLaunchKernelGGL((arnoldi_kernel<TB, TO, MODE, 4, 4, RPL>), grid, dim3(256), 0, s, V, vs, nvec, coef, w, N, R, rpc, partial);
    else if (cfg_n <= 32)
        hipLaunchKernelGGL((arnoldi_kernel<TB, TO, MODE, 8, 4, RPL>), grid, dim3(512), 0, s, V, vs, nvec, coef, w, N, R, rpc, partial);
    else
        hipLaunchKernelGGL((arnoldi_kernel<TB, TO, MODE, 8, 8, RPL>), grid, dim3(512), 0, s, V, vs, nvec, coef, w, N, R, rpc, partial);
    MBT_LAUNCH_CHECK();
}

// FP32 bases with an even number of columns move two RHS per 16-byte access.
// The kernel configuration follows nvec (the classical CGS2 sweeps).
template <typename TB, typename TO, int MODE>
void launch_pass(const TB* V, int64_t vs, int nvec, const double2* coef, TO* w, int64_t N, int R, int64_t rpc,
                 int nchunk, double2* partial, hipStream_t s) {
    const int cfg_n = nvec;
    if constexpr (sizeof(TB) == 8) {
        // the update-and-dot pass over more than 32 vectors keeps one RHS per lane (register budget)
        if (R % 2 == 0 && !(MODE == 1 && cfg_n > 32)) {
            launch_pass_rpl<TB, TO, MODE, 2>(V, vs, nvec, coef, w, N, R, rpc, nchunk, partial, s, cfg_n);
            return;
        }
    }
    launch_pass_rpl<TB, TO, MODE, 1>(V, vs, nvec, coef, w, N, R, rpc, nchunk, partial, s, cfg_n);
}

// out[i][r] = sum over the chunks c and the folded copies f < F of
// partial[c][i][f * R + r], in an order fixed by nchunk and F alone: the terms
// j = f * nchunk + c are dealt to kRedSub running sums (sum q takes j = q,
// q + kRedSub, ...), which are then added in order.  A workgroup owns kRedOut
// adjacent outputs (whole cache lines of every chunk), so a short batch still
// spreads its terms over many loads in flight: at 768 chunks of 4 x 32 columns
// (64x64 elements, 32 RHS) the sums of a sweep take 43 us when each is one
// thread's walk over 64 chunks; at 62 chunks of 4 x 128 columns 20 us, and 6.6 us
// so.
constexpr int kRedOut = 16;
constexpr int kRedWaves = 8;
constexpr int kRedSub = kRedWaves * 64 / kRedOut;
constexpr int kMaxChunks = 2048;
__global__ __launch_bounds__(64 * kRedWaves) void reduce_partials_kernel(const double2* __restrict__ partial,
                                                                         int nchunk, int nvec, int R, int F,
                                                                         double2* __restrict__ out) {
    __shared__ double2 gs[kRedSub][kRedOut];
    const int o = threadIdx.x % kRedOut, q = threadIdx.x / kRedOut;
    const int64_t t = (int64_t)blockIdx.x * kRedOut + o;
    double2 sum = make_double2(0, 0);
    if (t < (int64_t)nvec * R) {
        const int64_t i = t / R, r = t % R;
        const int64_t row = (int64_t)R * F;
        const double2* p = partial + i * row + r;
        int f = 0, c = q;
        while (c >= nchunk && f < F) {
            c -= nchunk;
            ++f;
        }
#pragma unroll 4
        while (f < F) {
            sum = cadd(sum, p[(int64_t)c * nvec * row + (int64_t)f * R]);
            c += kRedSub;
            while (c >= nchunk && f < F) {
                c -= nchunk;
                ++f;
            }
        }
    }
    gs[q][o] = sum;
    __syncthreads();
    if (q == 0 && t < (int64_t)nvec * R) {
#pragma unroll 8
        for (int g = 1; g < kRedSub; ++g) sum = cadd(sum, gs[g][o]);
        out[t] = sum;
    }
}

// partial holds nvec rows of F * R columns per chunk; out nvec rows of R
void launch_reduce_partials(const double2* partial, int nchunk, int nvec, int R, int F, double2* out, hipStream_t s) {
    MBT_REQUIRE(nchunk >= 1 && nchunk <= kMaxChunks, "reduction: too many chunks");
    const int64_t nout = (int64_t)nvec * R;
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((unsigned)((nout + kRedOut - 1) / kRedOut)), dim3(64 * kRedWaves), 0,
                       s, partial, nchunk, nvec, R, F, out);
    MBT_LAUNCH_CHECK();
}

// partial[chunk][r] = sum over the chunk's rows of |X[n][r]|^2: the rows are dealt to
// kNormWaves running sums (row n0 + j to sum j mod kNormWaves), added in order
constexpr int kNormWaves = 8;
template <typename TB>
__global__ __launch_bounds__(64 * kNormWaves) void colnorm2_kernel(const TB* __restrict__ X, int64_t N, int R,
                                                                   int64_t rows_per_chunk,
                                                                   double2* __restrict__ partial) {
    __shared__ double gs[kNormWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = blockIdx.x * 64 + lane;
    const int64_t chunk = blockIdx.y;
    const int64_t n0 = chunk * rows_per_chunk, n1 = min(N, n0 + rows_per_chunk);
    double s = 0;
    if (r < R) {
#pragma unroll 4
        for (int64_t n = n0 + wave; n < n1; n += kNormWaves) s = nfma(s, ld2(X + n * R + r));
    }
    gs[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && r < R) {
        for (int q = 1; q < kNormWaves; ++q) s += gs[q][lane];
        partial[chunk * R + r] = make_double2(s, 0.0);
    }
}

__device__ __forceinline__ double sum_norm_partials(const double2* partial, int nchunk, int R, int r) {
    double s = 0;
    for (int c = 0; c < nchunk; ++c) s += partial[(int64_t)c * R + r].x;
    return sqrt(s);
}

// One RHS at the start of a restart cycle: whether it goes on.
__device__ int cycle_init_rhs(GmresState st, const double2* __restrict__ nrm2, int r, int first) {
    const double beta = sqrt(nrm2[r].x);
    if (first) {
        st.bnorm[r] = beta;
        st.conv[r] = (beta == 0.0) ? 1 : 0;
        st.cand[r] = 0;
        st.iters[r] = 0;
        st.flag[r] = 0;
    }
    st.beta[r] = beta;
    st.kcyc[r] = 0;
    int act = 0;
    if (!st.conv[r] && !st.flag[r]) {
        if (!(beta == beta) || isinf(beta)) {
            st.flag[r] = 1;
        } else if (beta <= st.tol * st.bnorm[r] || (st.cand[r] && beta <= 2.0 * st.tol * st.bnorm[r])) {
            st.conv[r] = 1;
        } else {
            act = 1;
        }
    }
    st.cand[r] = 0;
    st.active[r] = act;
    st.scale[r] = act ? 1.0 / beta : 0.0;
    st.g[r] = make_double2(act ? beta : 0.0, 0.0);
    return act;
}

// Start of a restart cycle: beta = ||r|| (nrm2: the reduced squared norms);
// decide convergence at restart; reports how many RHS go on.
__global__ __launch_bounds__(256) void cycle_init_kernel(GmresState st, const double2* __restrict__ nrm2, int R,
                                                         int first, unsigned long long* counter,
                                                         unsigned long long* host_slot, uint32_t gen) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    int act = 0;
    if (r < R) act = cycle_init_rhs(st, nrm2, r, first);
    const int n = __syncthreads_count(act);
    if (threadIdx.x == 0) report_count(counter, (unsigned)n, gridDim.x, host_slot, gen);
}

// Arnoldi step j bookkeeping: Hessenberg column, Givens rotations, residual
// estimate, per-RHS stop decision and the normalisation factor of v_{j+1}.
__global__ void finalize_kernel(GmresState st, const double2* __restrict__ h1, const double2* __restrict__ h2,
                                const double2* __restrict__ npart, int nchunk, int R, int j, int m) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= R) return;
    if (!st.active[r]) {
        st.scale[r] = 0.0;
        return;
    }
    const double hn = sum_norm_partials(npart, nchunk, R, r);
    const int64_t ldH = (int64_t)(m + 1) * R;   // H[j][i][r]: column j, row i
    double2* Hj = st.H + (int64_t)j * ldH;
    for (int i = 0; i <= j; ++i) Hj[(int64_t)i * R + r] = cadd(h1[(int64_t)i * R + r], h2[(int64_t)i * R + r]);
    // previous rotations
    for (int i = 0; i < j; ++i) {
        const double c = st.cs[(int64_t)i * R + r];
        const double2 s = st.sn[(int64_t)i * R + r];
        const double2 a = Hj[(int64_t)i * R + r], b = Hj[(int64_t)(i + 1) * R + r];
        Hj[(int64_t)i * R + r] = cadd(make_double2(c * a.x, c * a.y), cmul(s, b));
        Hj[(int64_t)(i + 1) * R + r] = csub(make_double2(c * b.x, c * b.y), cmulc(s, a));
    }
    const double2 h1v = Hj[(int64_t)j * R + r];
    double c;
    double2 s;
    const double a1 = hypot(h1v.x, h1v.y);
    if (a1 == 0.0) {
        c = 0.0;
        s = make_double2(1.0, 0.0);
    } else {
        const double t = hypot(a1, hn);
        c = a1 / t;
        // s = (h1/|h1|) * conj(hn) / t, hn real
        s = make_double2(h1v.x / a1 * hn / t, h1v.y / a1 * hn / t);
    }
    st.cs[(int64_t)j * R + r] = c;
    st.sn[(int64_t)j * R + r] = s;
    Hj[(int64_t)j * R + r] = cadd(make_double2(c * h1v.x, c * h1v.y), make_double2(s.x * hn, s.y * hn));
    Hj[(int64_t)(j + 1) * R + r] = make_double2(0, 0);
    const double2 gj = st.g[(int64_t)j * R + r];
    const double2 gn = make_double2(-(s.x * gj.x + s.y * gj.y), -(s.x * gj.y - s.y * gj.x));  // -conj(s) g_j
    st.g[(int64_t)j * R + r] = make_double2(c * gj.x, c * gj.y);
    st.g[(int64_t)(j + 1) * R + r] = gn;
    st.iters[r] += 1;
    st.kcyc[r] = j + 1;
    const double res = hypot(gn.x, gn.y);
    const bool bad = !(hn == hn) || isinf(hn) || !(res == res);
    if (bad) {
        st.flag[r] = 1;
        st.active[r] = 0;
        st.scale[r] = 0.0;
        return;
    }
    if (res <= st.tol * st.bnorm[r] || hn == 0.0 || j == m - 1) {
        st.active[r] = 0;
        st.scale[r] = 0.0;
    } else {
        st.scale[r] = 1.0 / hn;
    }
}

template <typename TB>
__global__ void scale_cols_kernel(TB* __restrict__ v, const double* __restrict__ scale, int64_t N, int R) {
    const int64_t total = N * R;
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < total; t += (int64_t)gridDim.x * blockDim.x) {
        const double sc = scale[t % R];
        const double2 x = ld2(v + t);
        st2(v + t, make_double2(x.x * sc, x.y * sc));
    }
}

// End of cycle: y = R_k^{-1} g_k per RHS (k = steps done this cycle); |g_k|
// meeting the tolerance makes the RHS a candidate, which the explicit residual
// of the next restart confirms.  The back substitution is a chain of k steps: a
// wave owns one RHS with row l of the triangle in lane l (k <= 63), the triangle
// staged in LDS with all its loads in flight (a thread per RHS that reads it
// entry by entry takes 160 us at k = 32 and 455 us at k = 50, 128 RHS).
// Launched with at least m + 2 threads.
constexpr int kSolveR = 4;
__global__ __launch_bounds__(64 * kSolveR) void cycle_solve_kernel(GmresState st, int R, int m, double2* __restrict__ y,
                                                                   unsigned long long* __restrict__ counters) {
    __shared__ double2 tri[kSolveR][kMaxVec * (kMaxVec - 1) / 2];   // column i at i (i + 1) / 2, rows 0..i
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (blockIdx.x == 0 && threadIdx.x <= m + 1) counters[threadIdx.x] = 0;   // for the next cycle
    const int rb = blockIdx.x * kSolveR;
    const int64_t ldH = (int64_t)(m + 1) * R;
    {
        // adjacent threads load the same entry of the workgroup's adjacent RHS
        const int q = threadIdx.x % kSolveR, e0 = threadIdx.x / kSolveR;
        const int r = rb + q;
        const int kq = r < R && !st.flag[r] ? st.kcyc[r] : 0;
        const double2* Hl = st.H + (int64_t)e0 * R + r;
#pragma unroll 8
        for (int i = 0; i < kq; ++i)
            if (e0 <= i) tri[q][i * (i + 1) / 2 + e0] = Hl[(int64_t)i * ldH];
    }
    __syncthreads();
    const int r = rb + wave;
    if (r >= R) return;
    const int k = st.flag[r] ? 0 : st.kcyc[r];
    double2 acc = lane < k ? st.g[(int64_t)lane * R + r] : make_double2(0, 0);
    double2 mine = make_double2(0, 0);
    for (int i = k - 1; i >= 0; --i) {
        const double2 d = tri[wave][i * (i + 1) / 2 + i];
        const double2 a = make_double2(__shfl(acc.x, i), __shfl(acc.y, i));
        const double den = d.x * d.x + d.y * d.y;
        const double2 yi = make_double2((a.x * d.x + a.y * d.y) / den, (a.y * d.x - a.x * d.y) / den);
        if (lane == i) mine = yi;
        if (lane < i) acc = csub(acc, cmul(tri[wave][i * (i + 1) / 2 + lane], yi));
    }
    if (lane < m) y[(int64_t)lane * R + r] = mine;
    if (lane == 0 && k > 0) {
        const double2 gk = st.g[(int64_t)k * R + r];
        st.cand[r] = hypot(gk.x, gk.y) <= st.tol * st.bnorm[r] ? 1 : 0;
    }
}

// sum of active flags into one int (single workgroup)
__global__ void count_kernel(const int* __restrict__ a, int R, int* __restrict__ out) {
    __shared__ int s[256];
    int v = 0;
    for (int r = threadIdx.x; r < R; r += 256) v += a[r];
    s[threadIdx.x] = v;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) s[threadIdx.x] += s[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = s[0];
}

// r = b - Ax (in place on Ax), both of the basis type
template <typename TB>
__global__ void residual_kernel(const TB* __restrict__ b, TB* __restrict__ ax, int64_t n) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        st2(ax + t, csub(ld2(b + t), ld2(ax + t)));
}

template <typename TB>
__global__ void copy_kernel(const TB* __restrict__ src, TB* __restrict__ dst, int64_t n) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        dst[t] = src[t];
}

template <typename TB>
__global__ void from_f64_kernel(const double2* __restrict__ src, TB* __restrict__ dst, int64_t n) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        st2(dst + t, src[t]);
}

__global__ void zero_kernel(double2* __restrict__ p, int64_t n) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
        p[t] = make_double2(0, 0);
}

// Waits until the device has reported a count of generation gen into the pinned
// slot.  The kernel that reports it is already enqueued on s, so the wait ends:
// with the value, or with an error once the stream has run dry or failed.
int wait_count(const unsigned long long* slot, uint32_t gen, hipStream_t s) {
    auto seen = [&](int& n) {
        const unsigned long long v = __atomic_load_n(slot, __ATOMIC_ACQUIRE);
        n = (int)(uint32_t)v;
        return (uint32_t)(v >> 32) == gen;
    };
    int n = 0;
    for (;;) {
        for (int spin = 0; spin < 4096; ++spin) {
            if (seen(n)) return n;
            __builtin_ia32_pause();
        }
        const hipError_t e = hipStreamQuery(s);
        if (e == hipErrorNotReady) {
            (void)hipGetLastError();   // not an error
            continue;
        }
        MBT_HIP(e);
        if (seen(n)) return n;
        throw Error(-4, "the step count was not reported");
    }
}

inline unsigned ew_grid(int64_t n) {
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 65536));
}

}  // namespace

// Chunks of the row range for the reduction sweeps: a function of N alone, so a
// right-hand side's sums do not depend on how many others share the batch.  Up
// to 2048 chunks keep a few-RHS batch spread over the whole chip while the
// partial sums stay small next to one basis vector.  A workgroup walks its
// chunk's rows one after the other, so on a small system the chunk length is the
// length of the sweep: the 32-vector sweep of a 12x10 lattice of 15 bases (450
// folded rows, 120 RHS) takes 98 us in chunks of 128 rows and 10.6 us in chunks
// of 16.  The partial sums are written and read once per sweep, so the chunk grows with N.
// N alone decides, so each line weighs narrow batches, which short chunks serve, against
// wide ones.  Sweep and its reduction, us per step, FP64 and packed, at 10 / 100 / 600 RHS on
// 4 folded rows:
//   450 rows (120 RHS), 16 against 32: 19.8 20.1; packed 14.2 17.5
//   1,183 rows, 16 against 32: 13.6 14.4, 54.8 48.8, 308 281; packed 12.6 13.6, 25.1 24.4, 99 88
//   2,535 rows, 32 against 64: 17.7 21.4, 115 110, 582 551; packed 16.7 20.1, 37.5 39.0, 164 155
//   5,250 rows, 32, 64, 128: 30 28 35, 215 207 214, 1182 1090 1042; packed 26 25 33, 74 70 75, 353 328 319
//   6,975 rows, 64 against 128: 35.6 38.4, 267 265, 1429 1346; packed 29.8 35.6, 87 98, 431 426
//   7,936 rows, 64 against 128: 36.9 40.3, 309 285, 1632 1540; packed 31.3 35.6, 94 104, 487 461
// (128 throughout: 33, 58, 293 at 1,183 rows and 33, 115, 502 at 2,535, packed 31, 62, 99 and
// 32, 57, 171: wide FP64 batches of 2,000 to 7,000 rows pay 8 to 16 % of the sweep for it, and the
// update after it up to 8 %, as more partial sums pass through the last-level cache.)
int64_t gmres_rows_per_chunk(int64_t N) {
    const int64_t least = N < 1024 ? 16 : N < 4096 ? 32 : N < 7000 ? 64 : 128;
    return std::max<int64_t>(least, (N + 2047) / 2048);
}
int gmres_nchunk(int64_t N) { return (int)((N + gmres_rows_per_chunk(N) - 1) / gmres_rows_per_chunk(N)); }

// Row folding: the DCGS2 sweeps give each lane one RHS column (two with the
// packed basis) of a row, so batches narrower than 64 (128) columns would leave
// lanes idle.  F consecutive rows of an N x R vector are the same memory as one
// row of F*R columns; the sweeps run on N/F rows of F*R columns, index the
// per-RHS coefficients by column mod R, and the dot partials of the F copies of
// a RHS are summed afterwards in a fixed order.  F depends on N only, so a
// RHS's sums have the same order whatever the width of its batch.
int gmres_fold(int64_t N) { return N % 4 == 0 ? 4 : (N % 2 == 0 ? 2 : 1); }

size_t krylov_partial_values(int64_t N, int R, int m) {
    const int F = gmres_fold(N);
    return std::max((size_t)gmres_nchunk(N) * (2 * m + 2) * R,            // unfolded (CGS2; PCG and COCG take two)
                    (size_t)gmres_nchunk(N / F) * (2 * m + 2) * R * F);   // folded (DCGS2)
}

size_t gmres_state_bytes(int R, int m) {
    size_t s = 0;
    s += sizeof(double2) * (size_t)(m + 1) * (m + 1) * R;      // H (column j has m+1 rows, one spare)
    s += sizeof(double) * (size_t)m * R;                       // cs
    s += sizeof(double2) * (size_t)m * R;                      // sn
    s += sizeof(double2) * (size_t)(m + 1) * R;                // g
    s += sizeof(double2) * (size_t)(m + 1) * R * 2;            // h1, h2
    s += sizeof(double2) * (size_t)m * R;                      // y
    s += sizeof(unsigned long long) * (size_t)(m + 3) + 256;   // counters
    s += sizeof(double2) * (size_t)R + 256;                    // reduced squared norms
    s += sizeof(double) * (size_t)R * 4 + sizeof(int) * (size_t)R * 7 + 12 * 256;
    // delayed reorthogonalisation: unrotated Hessenberg, reduced sweep, coefficients, 1/nu
    s += sizeof(double2) * (size_t)(m + 1) * (m + 1) * R + sizeof(double2) * (size_t)(2 * m + 2) * R +
         sizeof(double2) * (size_t)(2 * m + 1) * R + sizeof(double) * (size_t)R + 4 * 256;
    return s;
}

template <typename TB>
GmresResult gmres_batched(const std::function<void(const TB*, TB*)>& apply, const TB* b, double2* x, TB* Vbasis,
                          int64_t N, int R, const GmresParams& prm, DevArena& arena, hipStream_t s) {
    const int m = prm.restart;
    MBT_REQUIRE(m >= 1 && m + 1 <= kMaxVec, "gmres: restart must be in 1..63");
    const int64_t rpc = gmres_rows_per_chunk(N);
    const size_t arena_mark = arena.off;   // the recurrence state is released on return
    const int nchunk = gmres_nchunk(N);
    const int64_t vs = N * R;   // basis vector stride

    GmresState st;
    st.tol = prm.tol;
    st.H = arena.get<double2>((size_t)(m + 1) * (m + 1) * R);
    st.cs = arena.get<double>((size_t)m * R);
    st.sn = arena.get<double2>((size_t)m * R);
    st.g = arena.get<double2>((size_t)(m + 1) * R);
    st.bnorm = arena.get<double>(R);
    st.beta = arena.get<double>(R);
    st.scale = arena.get<double>(R);
    st.active = arena.get<int>(R);
    st.conv = arena.get<int>(R);
    st.cand = arena.get<int>(R);
    st.flag = arena.get<int>(R);
    st.kcyc = arena.get<int>(R);
    st.iters = arena.get<int>(R);
    int* d_count = arena.get<int>(16);
    double2* h1 = arena.get<double2>((size_t)(m + 1) * R);
    double2* h2 = arena.get<double2>((size_t)(m + 1) * R);
    double2* y = arena.get<double2>((size_t)m * R);
    double2* partial = prm.partial;
    unsigned long long* counters = arena.get<unsigned long long>(m + 3);   // RHS still iterating, per step
    double2* nrm2 = arena.get<double2>(R);
    double2* Hraw = nullptr;
    double2* red = nullptr;
    double2* coef_s = nullptr;
    double2* coef_c = nullptr;
    double* inv_nu = nullptr;
    if (prm.dcgs2) {
        Hraw = arena.get<double2>((size_t)(m + 1) * (m + 1) * R);
        red = arena.get<double2>((size_t)(2 * m + 2) * R);
        coef_s = arena.get<double2>((size_t)m * R);
        coef_c = arena.get<double2>((size_t)(m + 1) * R);
        inv_nu = arena.get<double>(R);
    }

    GmresResult res;
    res.iters.assign(R, 0);
    res.conv.assign(R, 0);
    res.flag.assign(R, 0);

    const dim3 gR((R + 255) / 256), bR(256);
    int* h_count = prm.host_count;

    auto count_active = [&]() -> int {
        hipLaunchKernelGGL(count_kernel, dim3(1), dim3(256), 0, s, st.active, R, d_count);
        MBT_LAUNCH_CHECK();
        MBT_HIP(hipMemcpyAsync(h_count, d_count, sizeof(int), hipMemcpyDeviceToHost, s));
        MBT_HIP(hipStreamSynchronize(s));
        return *h_count;
    };

    // Packed basis (FP32 work vectors, even R, m >= 4): the candidate u and w = A u
    // live in two work vectors and the basis vectors in m packed slots, which
    // together take no more than the m+1 FP32 slots of the plain layout.  Plain
    // layout: slot k holds the candidate u_k, slot k+1 receives w = A u_k.
    bool packed = false;
    if constexpr (std::is_same<TB, float2>::value) packed = prm.packed_basis && prm.dcgs2 && R % 2 == 0 && m >= 4;
    TB* U = Vbasis;                                   // packed: candidate, residual
    TB* Wv = Vbasis + vs;                             // packed: A u, iterate copy
    p24x2* V24 = reinterpret_cast<p24x2*>(Vbasis + 2 * vs);
    const int64_t vs24 = vs / 2;
    TB* r0v = Vbasis;                                 // residual / first candidate (both layouts)
    TB* xb = Vbasis + vs;                             // iterate in the basis type (both layouts)
    // the DCGS2 sweeps and the solution update run on folded rows
    const int F = prm.dcgs2 ? gmres_fold(N) : 1;
    const int64_t Nf = N / F;
    const int Rf = R * F;
    const int64_t rpcf = gmres_rows_per_chunk(Nf);
    const int nchunkf = gmres_nchunk(Nf);

    unsigned long long* slots = prm.host.slots;
    // x = 0, r0 = b
    hipLaunchKernelGGL(zero_kernel, dim3(ew_grid(vs)), dim3(256), 0, s, x, vs);
    hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(256), 0, s, reinterpret_cast<double2*>(counters), (m + 3) / 2);
    hipLaunchKernelGGL((copy_kernel<TB>), dim3(ew_grid(vs)), dim3(256), 0, s, b, r0v, vs);
    MBT_LAUNCH_CHECK();
    bool first = true;
    for (int cycle = 0;; ++cycle) {
        // beta = ||r|| (r sits in V_0, or in the candidate vector when packed);
        // the convergence verdict of the previous cycle is taken on it
        hipLaunchKernelGGL((colnorm2_kernel<TB>), dim3((R + 63) / 64, nchunk), dim3(64 * kNormWaves), 0, s, r0v, N, R, rpc, partial);
        launch_reduce_partials(partial, nchunk, 1, R, 1, nrm2, s);
        const uint32_t gen = (uint32_t)++*prm.host.gen;
        hipLaunchKernelGGL(cycle_init_kernel, gR, bR, 0, s, st, nrm2, R, first ? 1 : 0, counters + m + 1, slots + m + 1,
                           gen);
        MBT_LAUNCH_CHECK();
        first = false;
        if (wait_count(slots + m + 1, gen, s) == 0 || cycle == prm.max_cycles) break;
        res.cycles++;
        hipLaunchKernelGGL((scale_cols_kernel<TB>), dim3(ew_grid(vs)), dim3(256), 0, s, r0v, st.scale, N, R);
        MBT_LAUNCH_CHECK();
        int steps = 0;
        // delayed reorthogonalisation: one dot sweep and one update sweep per step
        // (the last step needs only the dots of u_m)
        for (int k = 0; prm.dcgs2 && k <= m; ++k) {
            const bool hasw = k < m;
            TB* u = packed ? U : Vbasis + (int64_t)k * vs;
            TB* w = hasw ? (packed ? Wv : Vbasis + (int64_t)(k + 1) * vs) : nullptr;
            if (hasw) {
                apply(u, w);
                res.matvecs += prm.matvecs_per_apply;
            }
            const double vbytes = (double)vs * sizeof(TB);
            const double bbytes = packed ? (double)vs * 6.0 : vbytes;   // one basis vector
            {
                ProfScope ps(kKArnoldiDots, k * bbytes + (hasw ? 2 : 1) * vbytes, 8.0 * (2 * k + 2) * vs, s);
                if (packed) {
                    if constexpr (std::is_same<TB, float2>::value)
                        launch_dcgs2_dots<TB, p24x2>(V24, vs24, k, u, w, Nf, Rf, rpcf, nchunkf, partial, s);
                } else {
                    launch_dcgs2_dots<TB, TB>(Vbasis, vs, k, u, w, Nf, Rf, rpcf, nchunkf, partial, s);
                }
            }
            launch_reduce_partials(partial, nchunkf, 2 * k + 2, R, F, red, s);
            hipLaunchKernelGGL(dcgs2_step_kernel, dim3((R + kStepR - 1) / kStepR), dim3(kStepR * kStepRows), 0, s, st,
                               Hraw, red, R, k, m, hasw ? 1 : 0, inv_nu, coef_s, coef_c, counters + k, slots + k, gen);
            MBT_LAUNCH_CHECK();
            steps = k;
            if (k == m) break;
            {
                // k basis vectors, u and w read; v_k and u_{k+1} written
                ProfScope ps(kKArnoldiUpdateDots, (k + 1) * bbytes + 3 * vbytes, 16.0 * k * vs, s);
                if (packed) {
                    if constexpr (std::is_same<TB, float2>::value)
                        launch_dcgs2_update24(V24, vs24, k, U, Wv, V24 + (int64_t)k * vs24, coef_s, coef_c, inv_nu, Nf,
                                              Rf, R, counters + k, s);
                } else {
                    launch_dcgs2_update<TB>(Vbasis, vs, k, u, w, coef_s, coef_c, inv_nu, Nf, Rf, R, counters + k, s);
                }
            }
            // the update is under way (or has nothing to do) while the host learns whether any RHS goes on
            if (wait_count(slots + k, gen, s) == 0) break;
        }
        for (int j = 0; !prm.dcgs2 && j < m; ++j) {
            steps = j + 1;
            TB* vj = Vbasis + (int64_t)j * vs;
            TB* w = Vbasis + (int64_t)(j + 1) * vs;
            apply(vj, w);
            res.matvecs += prm.matvecs_per_apply;
            const int nvec = j + 1;
            // algorithmic traffic of a pass: nvec basis vectors and w read (+ w written by the updates)
            const double vbytes = (double)vs * sizeof(TB);
            {
                ProfScope ps(kKArnoldiDots, (nvec + 1) * vbytes, 8.0 * nvec * vs, s);
                launch_pass<TB, TB, 0>(Vbasis, vs, nvec, nullptr, w, N, R, rpc, nchunk, partial, s);
            }
            launch_reduce_partials(partial, nchunk, nvec, R, 1, h1, s);
            {
                ProfScope ps(kKArnoldiUpdateDots, (nvec + 2) * vbytes, 16.0 * nvec * vs, s);
                launch_pass<TB, TB, 1>(Vbasis, vs, nvec, h1, w, N, R, rpc, nchunk, partial, s);
            }
            launch_reduce_partials(partial, nchunk, nvec, R, 1, h2, s);
            {
                ProfScope ps(kKArnoldiUpdateNorm, (nvec + 2) * vbytes, 8.0 * nvec * vs, s);
                launch_pass<TB, TB, 2>(Vbasis, vs, nvec, h2, w, N, R, rpc, nchunk, partial, s);
            }
            hipLaunchKernelGGL(finalize_kernel, gR, bR, 0, s, st, h1, h2, partial, nchunk, R, j, m);
            hipLaunchKernelGGL((scale_cols_kernel<TB>), dim3(ew_grid(vs)), dim3(256), 0, s, w, st.scale, N, R);
            MBT_LAUNCH_CHECK();
            if (count_active() == 0) break;
        }
        // y = R^{-1} g ; x += V y
        hipLaunchKernelGGL(cycle_solve_kernel, dim3((R + kSolveR - 1) / kSolveR), dim3(64 * kSolveR), 0, s, st, R, m, y,
                           counters);
        MBT_LAUNCH_CHECK();
        // configuration fixed by m: a RHS's update x += V y does not depend on how long
        // the other RHS of the batch kept the cycle going
        if (packed)
            launch_solution_update<p24x2>(V24, vs24, steps, y, x, Nf, Rf, R, s);
        else
            launch_solution_update<TB>(Vbasis, vs, steps, y, x, Nf, Rf, R, s);
        // explicit residual r = b - A x into V_0 (x cast to the basis type into V_1 first)
        hipLaunchKernelGGL((from_f64_kernel<TB>), dim3(ew_grid(vs)), dim3(256), 0, s, x, xb, vs);
        MBT_LAUNCH_CHECK();
        apply(xb, r0v);
        res.matvecs += prm.matvecs_per_apply;
        hipLaunchKernelGGL((residual_kernel<TB>), dim3(ew_grid(vs)), dim3(256), 0, s, b, r0v, vs);
        MBT_LAUNCH_CHECK();
    }
    MBT_HIP(hipMemcpyAsync(res.iters.data(), st.iters, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipMemcpyAsync(res.conv.data(), st.conv, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipMemcpyAsync(res.flag.data(), st.flag, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipStreamSynchronize(s));
    arena.off = arena_mark;
    return res;
}

// ------------------------------------------------------------------ short recurrences (PCG, COCG)
// Both need two per-RHS dot products per step, each followed by a per-RHS scalar
// update.  A dot sweep writes chunk partials; the kernel that adds them also runs
// the scalar update and, where the step's verdict falls, reports how many RHS go
// on.
namespace {

constexpr int kDotSums = 8;
// MODE 0: sum conj(a) b; 1: sum a b; 2: sum a b and sum |a|^2.  Partials
// [chunk][v][r]; a chunk's rows are dealt to kDotSums running sums (row n0 + j to sum
// j mod kDotSums), which are added in order.  NW waves hold kDotSums / NW of them each.
// One wave per chunk that walks its rows one by one takes 61 us for 29,760 rows of 64 RHS
// in FP64 (31 MB per vector).
template <typename TB, int MODE, int NW>
__global__ __launch_bounds__(64 * NW) void krylov_dot_kernel(const TB* __restrict__ a, const TB* __restrict__ b,
                                                             int64_t N, int R, int64_t rows_per_chunk,
                                                             double2* __restrict__ partial) {
    static_assert(NW == 1 || NW == kDotSums, "a wave has all sums or one");
    constexpr int S = kDotSums / NW;
    __shared__ double2 gs[NW][64];
    __shared__ double gn[MODE == 2 ? NW : 1][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r = blockIdx.x * 64 + lane;
    const int64_t chunk = blockIdx.y;
    const int64_t n0 = chunk * rows_per_chunk, n1 = min(N, n0 + rows_per_chunk);
    double2 ab[S];
    double aa[S];
#pragma unroll
    for (int q = 0; q < S; ++q) {
        ab[q] = make_double2(0, 0);
        aa[q] = 0.0;
    }
    auto add = [&](int q, int64_t n) {
        const double2 av = ld2(a + n * R + r), bv = ld2(b + n * R + r);
        ab[q] = MODE == 0 ? cfmac(ab[q], av, bv) : cfma(ab[q], av, bv);
        if (MODE == 2) aa[q] = nfma(aa[q], av);
    };
    if (r < R) {
        if constexpr (S == 1) {
#pragma unroll 4
            for (int64_t n = n0 + wave; n < n1; n += kDotSums) add(0, n);
        } else {
            int64_t n = n0;
            for (; n + S <= n1; n += S)
#pragma unroll
                for (int q = 0; q < S; ++q) add(q, n + q);
#pragma unroll
            for (int q = 0; q < S; ++q)
                if (n + q < n1) add(q, n + q);
        }
    }
    if constexpr (S == 1) {
        gs[wave][lane] = ab[0];
        if (MODE == 2) gn[wave][lane] = aa[0];
        __syncthreads();
        if (wave != 0) return;
    }
    if (r >= R) return;
#pragma unroll
    for (int q = 1; q < kDotSums; ++q) {
        ab[0] = cadd(ab[0], S == 1 ? gs[q % NW][lane] : ab[q % S]);
        if (MODE == 2) aa[0] += S == 1 ? gn[q % NW][lane] : aa[q % S];
    }
    constexpr int nv = MODE == 2 ? 2 : 1;
    partial[chunk * nv * R + r] = ab[0];
    if (MODE == 2) partial[(chunk * nv + 1) * R + r] = make_double2(aa[0], 0.0);
}

// The chunk partials of NV dots added per RHS (in the order of
// reduce_partials_kernel) and handed to op(r, sums), which updates the RHS's
// scalars and says whether it goes on.  COUNT: reports the number that do; else
// the counter is cleared for the step's report.
template <int NV, bool COUNT, typename Op>
__global__ __launch_bounds__(64 * kRedWaves) void krylov_scalar_kernel(const double2* __restrict__ partial, int nchunk,
                                                                       int R, Op op, unsigned long long* counter,
                                                                       unsigned long long* host_slot, uint32_t gen) {
    __shared__ double2 gs[NV][kRedSub][kRedOut];
    const int o = threadIdx.x % kRedOut, q = threadIdx.x / kRedOut;
    const int r = blockIdx.x * kRedOut + o;
    double2 sum[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        sum[v] = make_double2(0, 0);
        if (r < R) {
#pragma unroll 4
            for (int c = q; c < nchunk; c += kRedSub) sum[v] = cadd(sum[v], partial[((int64_t)c * NV + v) * R + r]);
        }
        gs[v][q][o] = sum[v];
    }
    __syncthreads();
    int act = 0;
    if (q == 0 && r < R) {
#pragma unroll
        for (int v = 0; v < NV; ++v)
#pragma unroll 8
            for (int g = 1; g < kRedSub; ++g) sum[v] = cadd(sum[v], gs[v][g][o]);
        act = op(r, sum);
    }
    if (COUNT) {
        const int n = __syncthreads_count(act);
        if (threadIdx.x == 0) report_count(counter, (unsigned)n, gridDim.x, host_slot, gen);
    } else if (blockIdx.x == 0 && threadIdx.x == 0) {
        *counter = 0;
    }
}

template <typename TB, int MODE, bool COUNT, typename Op>
void krylov_dot(const TB* a, const TB* b, int64_t N, int R, double2* partial, const Op& op, unsigned long long* counter,
                unsigned long long* host_slot, uint32_t gen, hipStream_t s) {
    const int64_t rpc = gmres_rows_per_chunk(N);
    const int nchunk = gmres_nchunk(N);
    const dim3 grid((R + 63) / 64, nchunk);
    // A wave for each running sum; from 3,072 workgroups on one wave for all eight, which then keeps the
    // chip as busy with fewer of them waiting for each other (31,744 rows of 1,024 RHS in FP64, 3,968
    // workgroups: 184 against 195 us, of two products 208 against 212; 512 RHS: 102 against 94,
    // 64 RHS 46 against 12).  FP32 moves half the bytes, and its single products stay with a wave each
    // (1,024 RHS: 118 against 110 us; of two products 120 against 124).
    if ((int64_t)grid.x * nchunk >= 3072 && (sizeof(TB) == 16 || MODE == 2))
        hipLaunchKernelGGL((krylov_dot_kernel<TB, MODE, 1>), grid, dim3(64), 0, s, a, b, N, R, rpc, partial);
    else
        hipLaunchKernelGGL((krylov_dot_kernel<TB, MODE, kDotSums>), grid, dim3(64 * kDotSums), 0, s, a, b, N, R, rpc,
                           partial);
    hipLaunchKernelGGL((krylov_scalar_kernel<MODE == 2 ? 2 : 1, COUNT, Op>), dim3((R + kRedOut - 1) / kRedOut),
                       dim3(64 * kRedWaves), 0, s, partial, nchunk, R, op, counter, host_slot, gen);
    MBT_LAUNCH_CHECK();
}

}  // namespace

// ------------------------------------------------------------------ batched PCG (Sec. II-C)
// Conjugate gradients on N x = b (N = Z^H Z, Hermitian positive definite) with
// the preconditioner P applied as P^{-1}; one independent recurrence per RHS
// column, FP64 coefficients and dots, vectors of type TB.  With P = L L^H the
// iterates are those of plain CG on the split system of eq. (precond), and the
// stop test is that system's relative residual sqrt(r^H P^{-1} r / b^H P^{-1} b).
namespace {

struct PcgState {
    double tol;
    double *rho, *rho0, *alpha, *beta;
    int *active, *conv, *flag, *iters;
};

// rho of the initial residual
struct PcgInit {
    PcgState st;
    __device__ int operator()(int r, const double2* rz) const {
        const double rho = rz[0].x;
        st.rho[r] = rho;
        st.rho0[r] = rho;
        st.iters[r] = 0;
        st.flag[r] = !(rho == rho) || isinf(rho) || rho < 0.0;
        st.conv[r] = !st.flag[r] && rho == 0.0;
        st.active[r] = !st.flag[r] && !st.conv[r];
        st.alpha[r] = 0.0;
        st.beta[r] = 0.0;
        return st.active[r];
    }
};

// alpha = rho / p^H q for the RHS still iterating
struct PcgAlpha {
    PcgState st;
    __device__ int operator()(int r, const double2* pq) const {
        double a = 0.0;
        if (st.active[r]) {
            a = st.rho[r] / pq[0].x;
            if (!(a == a) || isinf(a)) {
                st.flag[r] = 1;
                st.active[r] = 0;
                a = 0.0;
            }
        }
        st.alpha[r] = a;
        return st.active[r];
    }
};

// x += alpha p (x in FP64), r -= alpha q
template <typename TB>
__global__ void pcg_xr_kernel(double2* __restrict__ x, TB* __restrict__ rv, const TB* __restrict__ p,
                              const TB* __restrict__ q, const double* __restrict__ alpha, int64_t NR, int R) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < NR; t += (int64_t)gridDim.x * blockDim.x) {
        const double a = alpha[t % R];
        const double2 pv = ld2(p + t), qv = ld2(q + t), xv = x[t], rr = ld2(rv + t);
        x[t] = make_double2(fma(a, pv.x, xv.x), fma(a, pv.y, xv.y));
        st2(rv + t, make_double2(fma(-a, qv.x, rr.x), fma(-a, qv.y, rr.y)));
    }
}

// rho_new = r^H z: stop test on the split-system residual, then beta
struct PcgBeta {
    PcgState st;
    __device__ int operator()(int r, const double2* rz) const {
        double b = 0.0;
        if (st.active[r]) {
            const double rn = rz[0].x;
            st.iters[r] += 1;
            if (!(rn == rn) || isinf(rn)) {
                st.flag[r] = 1;
                st.active[r] = 0;
            } else if (sqrt(fmax(rn, 0.0) / st.rho0[r]) <= st.tol) {
                st.conv[r] = 1;
                st.active[r] = 0;
            } else {
                b = rn / st.rho[r];
                st.rho[r] = rn;
            }
        }
        st.beta[r] = b;
        return st.active[r];
    }
};

// p = z + beta p
template <typename TB>
__global__ void pcg_p_kernel(TB* __restrict__ p, const TB* __restrict__ z, const double* __restrict__ beta, int64_t NR,
                             int R) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < NR; t += (int64_t)gridDim.x * blockDim.x) {
        const double b = beta[t % R];
        const double2 zv = ld2(z + t), pv = ld2(p + t);
        st2(p + t, make_double2(fma(b, pv.x, zv.x), fma(b, pv.y, zv.y)));
    }
}

}  // namespace

size_t pcg_state_bytes(int R) {
    return 2 * sizeof(double2) * (size_t)R + 4 * sizeof(double) * (size_t)R + 4 * sizeof(int) * (size_t)R + 16 * 256;
}

template <typename TB>
GmresResult pcg_batched(const std::function<void(const TB*, TB*)>& applyN,
                        const std::function<void(const TB*, TB*)>& applyPinv, const TB* b, double2* x, TB* work,
                        int64_t N, int R, double tol, int maxit, double2* partial, const HostReport& host,
                        DevArena& arena, hipStream_t s) {
    const size_t mark = arena.off;
    const int64_t NR = N * R;
    TB* rv = work;
    TB* z = work + NR;
    TB* p = work + 2 * NR;
    TB* q = work + 3 * NR;
    PcgState st;
    st.tol = tol;
    st.rho = arena.get<double>(R);
    st.rho0 = arena.get<double>(R);
    st.alpha = arena.get<double>(R);
    st.beta = arena.get<double>(R);
    st.active = arena.get<int>(R);
    st.conv = arena.get<int>(R);
    st.flag = arena.get<int>(R);
    st.iters = arena.get<int>(R);
    unsigned long long* counter = arena.get<unsigned long long>(2);
    GmresResult res;
    // x = 0, r = b, z = P^{-1} r, p = z, rho = r^H z
    hipLaunchKernelGGL(zero_kernel, dim3(ew_grid(NR)), dim3(256), 0, s, x, NR);
    hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(256), 0, s, reinterpret_cast<double2*>(counter), 1);
    hipLaunchKernelGGL((copy_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, b, rv, NR);
    MBT_LAUNCH_CHECK();
    applyPinv(rv, z);
    hipLaunchKernelGGL((copy_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, z, p, NR);
    MBT_LAUNCH_CHECK();
    uint32_t gen = (uint32_t)++*host.gen;
    krylov_dot<TB, 0, true>(rv, z, N, R, partial, PcgInit{st}, counter, host.slots, gen, s);
    res.cycles = 1;
    for (int it = 0; it < maxit && wait_count(host.slots, gen, s) > 0; ++it) {
        applyN(p, q);
        krylov_dot<TB, 0, false>(p, q, N, R, partial, PcgAlpha{st}, counter, host.slots, 0, s);
        hipLaunchKernelGGL((pcg_xr_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, x, rv, p, q, st.alpha, NR, R);
        MBT_LAUNCH_CHECK();
        applyPinv(rv, z);
        gen = (uint32_t)++*host.gen;
        krylov_dot<TB, 0, true>(rv, z, N, R, partial, PcgBeta{st}, counter, host.slots, gen, s);
        // the new direction is formed while the host learns whether any RHS goes on
        hipLaunchKernelGGL((pcg_p_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, p, z, st.beta, NR, R);
        MBT_LAUNCH_CHECK();
        res.matvecs += 2;
    }
    res.iters.assign(R, 0);
    res.conv.assign(R, 0);
    res.flag.assign(R, 0);
    MBT_HIP(hipMemcpyAsync(res.iters.data(), st.iters, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipMemcpyAsync(res.conv.data(), st.conv, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipMemcpyAsync(res.flag.data(), st.flag, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipStreamSynchronize(s));
    arena.off = mark;
    return res;
}

// ------------------------------------------------------------------ batched COCG
// Conjugate orthogonal conjugate gradients (van der Vorst and Melissen, 1990)
// on Z x = b for complex symmetric Z with a complex symmetric preconditioner M
// applied as M^{-1}: the CG recurrences with the bilinear form a^T b in place
// of a^H b.  One operator application and one preconditioner application per
// step, no Krylov basis.  Stop test: ||r|| <= tol ||b||.  The element-block
// P_K is symmetric (Galerkin self block), so M = P_K keeps the recurrence
// valid.  One independent recurrence per RHS column, FP64 coefficients.
namespace {

struct CocgState {
    double tol;
    double2 *rho, *alpha, *beta;
    double* bnorm2;
    int *active, *conv, *flag, *iters;
};

__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
    const double d = b.x * b.x + b.y * b.y;
    return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}

// red = [r^T z, |r|^2] of the initial residual r = b
struct CocgInit {
    CocgState st;
    __device__ int operator()(int r, const double2* red) const {
        const double2 rho = red[0];
        const double bb = red[1].x;
        st.rho[r] = rho;
        st.bnorm2[r] = bb;
        st.iters[r] = 0;
        st.flag[r] = !(bb == bb) || isinf(bb) || !(rho.x == rho.x) || !(rho.y == rho.y);
        st.conv[r] = !st.flag[r] && bb == 0.0;
        st.active[r] = !st.flag[r] && !st.conv[r];
        st.alpha[r] = make_double2(0, 0);
        st.beta[r] = make_double2(0, 0);
        return st.active[r];
    }
};

// alpha = rho / p^T q for the RHS still iterating (a vanishing p^T q is a breakdown)
struct CocgAlpha {
    CocgState st;
    __device__ int operator()(int r, const double2* pq) const {
        double2 a = make_double2(0, 0);
        if (st.active[r]) {
            a = cdiv(st.rho[r], pq[0]);
            if (!(a.x == a.x) || !(a.y == a.y) || isinf(a.x) || isinf(a.y)) {
                st.flag[r] = 1;
                st.active[r] = 0;
                a = make_double2(0, 0);
            }
        }
        st.alpha[r] = a;
        return st.active[r];
    }
};

// x += alpha p (x in FP64), r -= alpha q
template <typename TB>
__global__ void cocg_xr_kernel(double2* __restrict__ x, TB* __restrict__ rv, const TB* __restrict__ p,
                               const TB* __restrict__ q, const double2* __restrict__ alpha, int64_t NR, int R) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < NR; t += (int64_t)gridDim.x * blockDim.x) {
        const double2 a = alpha[t % R];
        const double2 na = make_double2(-a.x, -a.y);
        x[t] = cfma(x[t], a, ld2(p + t));
        st2(rv + t, cfma(ld2(rv + t), na, ld2(q + t)));
    }
}

// red = [r^T z, |r|^2]: stop test on ||r|| / ||b||, then beta = rho_new / rho
struct CocgBeta {
    CocgState st;
    __device__ int operator()(int r, const double2* red) const {
        double2 b = make_double2(0, 0);
        if (st.active[r]) {
            const double2 rz = red[0];
            const double rr = red[1].x;
            st.iters[r] += 1;
            if (!(rr == rr) || isinf(rr) || !(rz.x == rz.x) || !(rz.y == rz.y)) {
                st.flag[r] = 1;
                st.active[r] = 0;
            } else if (sqrt(rr / st.bnorm2[r]) <= st.tol) {
                st.conv[r] = 1;
                st.active[r] = 0;
            } else if (rr > 1e12 * st.bnorm2[r]) {
                // a residual a million times the right-hand side: the recurrence has run away
                // (the FP32 short recurrence does so on a few RHS); stop it unconverged
                st.active[r] = 0;
            } else {
                b = cdiv(rz, st.rho[r]);
                st.rho[r] = rz;
            }
        }
        st.beta[r] = b;
        return st.active[r];
    }
};

// p = z + beta p
template <typename TB>
__global__ void cocg_p_kernel(TB* __restrict__ p, const TB* __restrict__ z, const double2* __restrict__ beta,
                              int64_t NR, int R) {
    for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < NR; t += (int64_t)gridDim.x * blockDim.x)
        st2(p + t, cfma(ld2(z + t), beta[t % R], ld2(p + t)));
}

}  // namespace

size_t cocg_state_bytes(int R) {
    return 5 * sizeof(double2) * (size_t)R + sizeof(double) * (size_t)R + 4 * sizeof(int) * (size_t)R + 16 * 256;
}

template <typename TB>
GmresResult cocg_batched(const std::function<void(const TB*, TB*)>& applyZ,
                         const std::function<void(const TB*, TB*)>& applyMinv, const TB* b, double2* x, TB* work,
                         int64_t N, int R, double tol, int maxit, double2* partial, const HostReport& host,
                        DevArena& arena, hipStream_t s) {
    const size_t mark = arena.off;
    const int64_t NR = N * R;
    TB* rv = work;
    TB* z = work + NR;
    TB* p = work + 2 * NR;
    TB* q = work + 3 * NR;
    CocgState st;
    st.tol = tol;
    st.rho = arena.get<double2>(R);
    st.alpha = arena.get<double2>(R);
    st.beta = arena.get<double2>(R);
    st.bnorm2 = arena.get<double>(R);
    st.active = arena.get<int>(R);
    st.conv = arena.get<int>(R);
    st.flag = arena.get<int>(R);
    st.iters = arena.get<int>(R);
    unsigned long long* counter = arena.get<unsigned long long>(2);
    GmresResult res;
    // x = 0, r = b, z = M^{-1} r, p = z, rho = r^T z
    hipLaunchKernelGGL(zero_kernel, dim3(ew_grid(NR)), dim3(256), 0, s, x, NR);
    hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(256), 0, s, reinterpret_cast<double2*>(counter), 1);
    hipLaunchKernelGGL((copy_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, b, rv, NR);
    MBT_LAUNCH_CHECK();
    applyMinv(rv, z);
    hipLaunchKernelGGL((copy_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, z, p, NR);
    MBT_LAUNCH_CHECK();
    uint32_t gen = (uint32_t)++*host.gen;
    krylov_dot<TB, 2, true>(rv, z, N, R, partial, CocgInit{st}, counter, host.slots, gen, s);
    res.cycles = 1;
    for (int it = 0; it < maxit && wait_count(host.slots, gen, s) > 0; ++it) {
        applyZ(p, q);
        krylov_dot<TB, 1, false>(p, q, N, R, partial, CocgAlpha{st}, counter, host.slots, 0, s);
        hipLaunchKernelGGL((cocg_xr_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, x, rv, p, q, st.alpha, NR, R);
        MBT_LAUNCH_CHECK();
        applyMinv(rv, z);
        gen = (uint32_t)++*host.gen;
        krylov_dot<TB, 2, true>(rv, z, N, R, partial, CocgBeta{st}, counter, host.slots, gen, s);
        // the new direction is formed while the host learns whether any RHS goes on
        hipLaunchKernelGGL((cocg_p_kernel<TB>), dim3(ew_grid(NR)), dim3(256), 0, s, p, z, st.beta, NR, R);
        MBT_LAUNCH_CHECK();
        res.matvecs += 1;
    }
    res.iters.assign(R, 0);
    res.conv.assign(R, 0);
    res.flag.assign(R, 0);
    MBT_HIP(hipMemcpyAsync(res.iters.data(), st.iters, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipMemcpyAsync(res.conv.data(), st.conv, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipMemcpyAsync(res.flag.data(), st.flag, sizeof(int) * R, hipMemcpyDeviceToHost, s));
    MBT_HIP(hipStreamSynchronize(s));
    arena.off = mark;
    return res;
}

template GmresResult cocg_batched<double2>(const std::function<void(const double2*, double2*)>&,
                                           const std::function<void(const double2*, double2*)>&, const double2*,
                                           double2*, double2*, int64_t, int, double, int, double2*, const HostReport&,
                                           DevArena&, hipStream_t);
template GmresResult cocg_batched<float2>(const std::function<void(const float2*, float2*)>&,
                                          const std::function<void(const float2*, float2*)>&, const float2*, double2*,
                                          float2*, int64_t, int, double, int, double2*, const HostReport&,
                                           DevArena&, hipStream_t);

template GmresResult pcg_batched<double2>(const std::function<void(const double2*, double2*)>&,
                                          const std::function<void(const double2*, double2*)>&, const double2*,
                                          double2*, double2*, int64_t, int, double, int, double2*, const HostReport&,
                                           DevArena&, hipStream_t);
template GmresResult pcg_batched<float2>(const std::function<void(const float2*, float2*)>&,
                                         const std::function<void(const float2*, float2*)>&, const float2*, double2*,
                                         float2*, int64_t, int, double, int, double2*, const HostReport&,
                                           DevArena&, hipStream_t);

template GmresResult gmres_batched<double2>(const std::function<void(const double2*, double2*)>&, const double2*,
                                            double2*, double2*, int64_t, int, const GmresParams&, DevArena&, hipStream_t);
template GmresResult gmres_batched<float2>(const std::function<void(const float2*, float2*)>&, const float2*, double2*,
                                           float2*, int64_t, int, const GmresParams&, DevArena&, hipStream_t);

}  // namespace mbt
