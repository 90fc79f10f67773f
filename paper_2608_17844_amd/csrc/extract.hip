// Port quantities on the device, FP64.
//
// * Z_p = Y_p^{-1}: the open-circuit port impedance (paper eq. (passZ)) from
//   the short-circuit admittance that unit delta-gap excitations give;
// * S = (Z_p - z0)(Z_p + z0)^{-1} = I - 2 z0 (Z_p + z0)^{-1}, eq. (S2Z) solved
//   for S;
// * the center element's active impedance for port currents phased to steer
//   the main beam at (theta, phi) (Sec. II-E), I_j = exp(-j k (x_j u + y_j v))
//   under the e^{-jkR} kernel of the fill (eqs. (actZ), (actZmat)), its ARC
//   (eq. (ARC)), and the wave-excited reflection coefficient, the phased S-sum
//   of Sec. II-E;
// * for a phased voltage excitation of every gap, V_j = exp(-j k (x_j u + y_j v))
//   on the same beam-steering convention, the right-hand sides and, from the
//   gap currents the solve returns, the center element's active impedance
//   Z_a,c = V_c / I_p,c (eq. (actZ) with those port currents) and its ARC.
//
// The dense inverses use Gauss-Jordan elimination with partial pivoting: up to 64
// rows in one workgroup's registers, up to 4,096 in panels of eight (four) columns,
// each launch factoring the next panel while it applies the current one, so the
// matrix is streamed once per panel.  Larger sizes use one pivot kernel and one
// rank-1 elimination kernel per column.
#include "common.h"
#include "extract.h"

#include <algorithm>
#include <vector>

namespace mbt {

namespace {

constexpr int kPivT = 1024;

// argmax |A[i][k]| over i >= k (ties -> smallest i), swap rows k and p, scale
// row k by 1/A[k][k] (with A[k][k] replaced by 1), save column k multipliers.
__global__ __launch_bounds__(kPivT) void gj_pivot_kernel(double2* __restrict__ A, int n, int k, double2* __restrict__ colbuf,
                                                         int* __restrict__ piv, int* __restrict__ singular) {
    __shared__ double sv[kPivT];
    __shared__ int si[kPivT];
    const int tid = threadIdx.x;
    double best = -1.0;
    int bi = n;
    for (int i = k + tid; i < n; i += kPivT) {
        const double2 v = A[(int64_t)i * n + k];
        const double m = v.x * v.x + v.y * v.y;
        if (m > best) { best = m; bi = i; }
    }
    sv[tid] = best;
    si[tid] = bi;
    __syncthreads();
    for (int s = kPivT / 2; s > 0; s >>= 1) {
        if (tid < s) {
            const double o = sv[tid + s];
            const int oi = si[tid + s];
            if (o > sv[tid] || (o == sv[tid] && oi < si[tid])) { sv[tid] = o; si[tid] = oi; }
        }
        __syncthreads();
    }
    const int p = si[0];
    if (tid == 0) {
        piv[k] = p;
        if (!(sv[0] > 0.0)) singular[0] = 1;
    }
    if (p != k && p < n)
        for (int j = tid; j < n; j += kPivT) {
            const double2 t = A[(int64_t)k * n + j];
            A[(int64_t)k * n + j] = A[(int64_t)p * n + j];
            A[(int64_t)p * n + j] = t;
        }
    __syncthreads();
    const double2 d = A[(int64_t)k * n + k];
    const double den = d.x * d.x + d.y * d.y;
    const double2 dinv = den > 0.0 ? make_double2(d.x / den, -d.y / den) : make_double2(0, 0);
    for (int i = tid; i < n; i += kPivT) colbuf[i] = (i == k) ? make_double2(0, 0) : A[(int64_t)i * n + k];
    __syncthreads();
    for (int j = tid; j < n; j += kPivT) {
        const double2 v = (j == k) ? make_double2(1.0, 0.0) : A[(int64_t)k * n + j];
        A[(int64_t)k * n + j] = cmul(v, dinv);
    }
}

__global__ void gj_elim_kernel(double2* __restrict__ A, int n, int k, const double2* __restrict__ colbuf) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const int i = (int)(t / n), j = (int)(t % n);
    if (i == k) return;
    const double2 base = (j == k) ? make_double2(0, 0) : A[t];
    A[t] = csub(base, cmul(colbuf[i], A[(int64_t)k * n + j]));
}

// ---- one-launch and panelled forms
// Both keep the rows where they are: a step's pivot is the unused row of largest
// magnitude in its column, and the elimination ends with the row of step k at row
// p_k.  With B the in-place result, A^{-1}[k][p_j] = B[p_k][j].

// Wave-wide maximum through DPP lane permutations (pairs, quads, eight, sixteen
// lanes) and the four row results read out of lanes 0, 16, 32 and 48.  Called by all
// 64 lanes.
template <int CTRL> __device__ __forceinline__ uint32_t dpp_max(uint32_t key) {
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)key, CTRL, 0xF, 0xF, false);
    return o > key ? o : key;
}
__device__ __forceinline__ uint32_t row_max(uint32_t key) {   // within sixteen lanes
    key = dpp_max<0xB1>(key);    // quad_perm [1,0,3,2]
    key = dpp_max<0x4E>(key);    // quad_perm [2,3,0,1]
    key = dpp_max<0x141>(key);   // row_half_mirror
    return dpp_max<0x140>(key);  // row_mirror
}
__device__ __forceinline__ uint32_t wave_max(uint32_t key) {
    key = row_max(key);
    uint32_t best = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)key, 16 * r);
        best = o > best ? o : best;
    }
    return best;
}

// Pivot keys: |v|^2 in FP64 (positive doubles order as integers), one up; 1 for zero and
// NaN, above the 0 of rows out of the search.
__device__ __forceinline__ uint64_t mag_key(double2 v) {
    const double m = v.x * v.x + v.y * v.y;
    return m > 0.0 ? (uint64_t)__double_as_longlong(m) + 1 : 1;
}
// The lanes that hold the largest key of the wave.  The upper halves decide almost always;
// the lower ones are compared when several lanes share the largest upper half.  Called by
// all 64 lanes.
__device__ __forceinline__ uint64_t wave_best(uint64_t key) {
    const uint32_t hi = (uint32_t)(key >> 32);
    const uint32_t best = wave_max(hi);
    uint64_t at = __ballot(hi == best);
    if (at & (at - 1)) {
        const uint32_t lo = hi == best ? (uint32_t)key : 0u;
        const uint32_t low = wave_max(lo);
        at = __ballot(hi == best && lo == low);
    }
    return at;
}
// The same where lane i holds key i mod NW, NW <= 16 (every sixteen lanes hold them all): the
// keys that are the largest.
template <int NW> __device__ __forceinline__ uint32_t row_best(uint64_t key) {
    static_assert(16 % NW == 0, "sixteen lanes hold whole sets of keys");
    constexpr uint32_t set = (1u << NW) - 1;
    const uint32_t hi = (uint32_t)(key >> 32);
    const uint32_t best = row_max(hi);
    uint32_t at = (uint32_t)__ballot(hi == best) & set;
    if (at & (at - 1)) {
        const uint32_t lo = hi == best ? (uint32_t)key : 0u;
        const uint32_t low = row_max(lo);
        at = (uint32_t)__ballot(hi == best && lo == low) & set;
    }
    return at;
}
__device__ __forceinline__ double2 recip(double2 d) {
    const double den = d.x * d.x + d.y * d.y;
    return den > 0.0 ? make_double2(d.x / den, -d.y / den) : make_double2(0, 0);
}

// n <= ROWS: the whole matrix in the registers of one workgroup, TPR threads per row
// with CPT columns each (column j in thread j mod TPR).  Per step: the column goes
// to LDS, every wave finds the pivot in it, the pivot row goes to LDS, all rows
// update; two barriers.  Writes the inverse.  The chain of n steps bounds it: 0.078 ms
// at n = 25 and 0.181 ms at n = 64 with the copies to and from the host, where a launch
// per pivot search and per rank-1 pass took 0.250 and two-launch panels 0.398 ms.
// More columns per thread in fewer waves (2 and 4 threads a row) took 0.10 and 0.40 ms.
template <int ROWS, int TPR, int CPT>
__global__ __launch_bounds__(ROWS * TPR) void gj_small_kernel(const double2* __restrict__ A, int n,
                                                             double2* __restrict__ out, int* __restrict__ singular) {
    static_assert(TPR * CPT >= ROWS && ROWS <= 64, "a wave looks at one row per lane");
    __shared__ double2 col[2][ROWS], prow[2][TPR * CPT];
    __shared__ int piv[ROWS], pos[ROWS];
    const int lane = threadIdx.x & 63;
    const int i = threadIdx.x / TPR, tt = threadIdx.x % TPR;
    double2 a[CPT];
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        const int j = q * TPR + tt;
        a[q] = (i < n && j < n) ? A[(int64_t)i * n + j] : make_double2(0, 0);
    }
    bool open = lane < n;   // row `lane` is still in the search (the same in every wave)
    int par = 0;
    bool bad = false;
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
        for (int t = 0; t < TPR; ++t, par ^= 1) {
            const int k = q * TPR + t;
            if (k >= n) break;
            if (tt == t) col[par][i] = a[q];
            __syncthreads();
            const double2 cv = open ? col[par][lane] : make_double2(0, 0);
            const int p = __ffsll((unsigned long long)wave_best(open ? mag_key(cv) : 0)) - 1;
            if (lane == p) open = false;
            if (i == p) {
#pragma unroll
                for (int e = 0; e < CPT; ++e) prow[par][e * TPR + tt] = a[e];
                if (tt == 0) {
                    piv[k] = p;
                    pos[p] = k;
                }
            }
            __syncthreads();
            const double2 d = col[par][p];
            const double2 di = recip(d);
            bad = bad || !(d.x * d.x + d.y * d.y > 0.0);
            const double2 l = col[par][i];
#pragma unroll
            for (int e = 0; e < CPT; ++e) {
                const bool kc = e == q && tt == t;
                const double2 rk = cmul(kc ? make_double2(1.0, 0.0) : prow[par][e * TPR + tt], di);
                a[e] = i == p ? rk : csub(kc ? make_double2(0, 0) : a[e], cmul(l, rk));
            }
        }
    }
    if (threadIdx.x == 0 && bad) *singular = 1;
    __syncthreads();
    if (i >= n) return;
#pragma unroll
    for (int e = 0; e < CPT; ++e) {
        const int j = e * TPR + tt;
        if (j < n) out[(int64_t)pos[i] * n + piv[j]] = a[e];
    }
}

// Larger n: panels of NB columns.  One launch per panel: workgroup 0 brings the next
// panel's columns up to date and factors it (thread t owns rows t, t + PT, ..., RPT
// of them, with their panel values in registers), while the others apply the current
// panel to SW columns each.  The chain of pivot steps in workgroup 0 bounds it:
// per step each wave puts its best row in LDS and one barrier later all read the
// winner.  What workgroup 0 reads and writes is compact and column by column (column
// pieces n rows apart would cost a cache line per value): the columns that it
// factors are handed over by the launch before, and the factored ones are copied
// into the matrix by the launch after.  A launch takes 12.1 us at n = 120, 16.0 at 512
// and 25 at 1000 and 1024, all but 0.5 to 3 us of it workgroup 0's chain; factoring
// and update in launches of their own took 23 and 42 us at 120 and 1024.  A CU holds one
// such workgroup: strips of four columns keep all of a launch resident up to 1024
// rows (eight took 19.8 against 17.7 us at 512 rows, half the chip idle; a 257th workgroup, the next
// panel's strips among them, 30 us at 1024), strips of eight up to 2048.
template <int NB> struct GjPanel {
    double2* L;    // [NB][n]: multiplier of row i at step c, 0 for the step's pivot row
    double2* P;    // [NB][n]: the panel's columns before its factorisation, up to date with the panel before the last
    double2* F;    // [NB][n]: and after it
    double2* dv;   // [NB]: reciprocal pivots
};

// One launch: k0: the current panel's first column (nb0 columns, 0: none yet), k1: the
// next one's (nb1 columns, 0: none left), after it nb2 columns of the one that the
// launch after factors.  from_p: the next panel's columns are in nxt.P (else in A).
template <int NB, int PT, int RPT, int SW>
__global__ __launch_bounds__(PT) void gj_step_kernel(double2* __restrict__ A, int n, int k0, int nb0, int k1, int nb1,
                                                     int nb2, int from_p, GjPanel<NB> cur, GjPanel<NB> nxt,
                                                     int* __restrict__ piv, int* __restrict__ used,
                                                     int* __restrict__ singular) {
    constexpr int NW = PT / 64;
    constexpr bool PRE = RPT <= 2;                      // the multipliers fit the registers beside the rows
    constexpr int CW = NB;                              // columns that the pivot-row wave works on
    static_assert(NB * CW <= 64 && NB % SW == 0, "one wave works out the pivot rows; panels are whole strips");
    __shared__ double2 rks[NB][CW], rfin[NB][CW];
    __shared__ signed char prank[PT * RPT];             // which pivot of the current panel a row is, -1: none
    const int tid = threadIdx.x;
    const bool factor = blockIdx.x == 0;
    if (factor && nb1 == 0) return;
    // strips in a cache line's pairs eight workgroups apart, which share an XCD and its L2;
    // those of the next panel are left out
    const int sb = (int)blockIdx.x - 1;
    int strip = SW == 4 ? (sb & ~15) + 2 * (sb & 7) + ((sb >> 3) & 1) : sb;
    if (strip >= k1 / SW) strip += (nb1 + SW - 1) / SW;
    const int j0 = factor ? k1 : strip * SW;
    const int cw = tid % SW, js = j0 + cw;              // the strip column of this thread
    if (!factor && j0 >= n) return;
    if (!factor && j0 >= k0 && j0 < k0 + nb0) {
        // the current panel's own columns (whole strips)
        if (js < k0 + nb0)
            for (int i = tid / SW; i < n; i += PT / SW) A[(int64_t)i * n + js] = cur.F[(int64_t)(js - k0) * n + i];
        return;
    }
    // the factoring workgroup's rows, and the first of a strip's, are on their way while the pivot
    // rows are worked out (strips: 1500 rows 18.4 -> 16.5 ms, 2304 90 -> 80, copies included)
    constexpr int VPRE = RPT <= 2 ? RPT * SW : 4;
    double2 vpre[VPRE];
    if (!factor && js < n)
#pragma unroll
        for (int e = 0; e < VPRE; ++e) {
            const int i = tid / SW + e * (PT / SW);
            vpre[e] = i < n ? A[(int64_t)i * n + js] : make_double2(0, 0);
        }
    double2 rowv[RPT][NB], lown[PRE ? RPT : 1][NB];
    if (factor) {
#pragma unroll
        for (int e = 0; e < RPT; ++e) {
            const int i = tid + e * PT;
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                rowv[e][c] = (i < n && c < nb1) ? (from_p ? nxt.P[(int64_t)c * n + i] : A[(int64_t)i * n + k1 + c])
                                                : make_double2(0, 0);
                if (PRE) lown[e][c] = (i < n && c < nb0) ? cur.L[(int64_t)c * n + i] : make_double2(0, 0);
            }
        }
    }
    for (int i = tid; i < n; i += PT) prank[i] = -1;
    __syncthreads();
    if (tid < 64) {
        // Lane (q, t): pivot row q in this workgroup's column t.  rks: row c right after its
        // scaling (the value the other rows are eliminated with); rfin: its final entries.
        const int q = tid / CW, t = tid % CW;
        const bool on = q < nb0;
        const int pq = on ? piv[k0 + q] : 0;
        if (on && t == 0) prank[pq] = (signed char)q;
        double2 r = make_double2(0, 0);
        if (on) {
            if (!factor) r = (t < SW && j0 + t < n) ? A[(int64_t)pq * n + j0 + t] : r;
            else if (t < nb1) r = from_p ? nxt.P[(int64_t)t * n + pq] : A[(int64_t)pq * n + k1 + t];
        }
        double2 lq[NB];   // multipliers of pivot row q
#pragma unroll
        for (int c = 0; c < NB; ++c) lq[c] = (on && c < nb0) ? cur.L[(int64_t)c * n + pq] : make_double2(0, 0);
        double2 d = on ? cur.dv[q] : make_double2(0, 0);
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            const double2 sc = cmul(r, d);
            const double2 rc = make_double2(__shfl(sc.x, c * CW + t), __shfl(sc.y, c * CW + t));
            if (c < nb0) {
                if (q == c) {
                    r = rc;
                    rks[c][t] = rc;
                } else {
                    r = csub(r, cmul(lq[c], rc));
                }
            }
        }
        if (on) rfin[q][t] = r;
    }
    __syncthreads();
    if (!factor) {
        const int k2 = k1 + nb1;
        if (js >= n) return;
        const bool ahead = js >= k2 && js < k2 + nb2;   // the columns that the launch after this one factors
        double2* dst = ahead ? cur.P + (int64_t)(js - k2) * n : A + js;
        const int64_t ds = ahead ? 1 : n;
        double2 rk[NB];
#pragma unroll
        for (int c = 0; c < NB; ++c) rk[c] = c < nb0 ? rks[c][cw] : make_double2(0, 0);
        auto put = [&](int i, double2 v) {
            const int pr = prank[i];
            double2 l[NB];
#pragma unroll
            for (int c = 0; c < NB; ++c) l[c] = c < nb0 ? cur.L[(int64_t)c * n + i] : make_double2(0, 0);
#pragma unroll
            for (int c = 0; c < NB; ++c) v = csub(v, cmul(l[c], rk[c]));
            dst[(int64_t)i * ds] = pr >= 0 ? rfin[pr][cw] : v;
        };
#pragma unroll
        for (int e = 0; e < VPRE; ++e)
            if (tid / SW + e * (PT / SW) < n) put(tid / SW + e * (PT / SW), vpre[e]);
        if constexpr (VPRE < RPT * SW)
#pragma unroll 4
            for (int i = tid / SW + VPRE * (PT / SW); i < n; i += PT / SW) put(i, A[(int64_t)i * n + js]);
        return;
    }
    // the next panel: bring it up to date ...
    bool open[RPT];   // rows still in the pivot search
#pragma unroll
    for (int e = 0; e < RPT; ++e) {
        const int i = tid + e * PT;
        open[e] = i < n && (nb0 == 0 || used[i] == 0);
        if (nb0 > 0 && i < n) {
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                if (c < nb0) {
                    const double2 l = PRE ? lown[PRE ? e : 0][c] : cur.L[(int64_t)c * n + i];
#pragma unroll
                    for (int q = 0; q < NB; ++q) rowv[e][q] = csub(rowv[e][q], cmul(l, rks[c][q]));
                }
            }
            const int pr = prank[i];
            if (pr >= 0)
#pragma unroll
                for (int q = 0; q < NB; ++q) rowv[e][q] = rfin[pr][q];
        }
    }
    // ... and factor it
    __shared__ uint64_t wkey[2][NW];
    __shared__ int wrow[2][NW];
    __shared__ double2 wval[2][NW][NB];
    const int lane = tid & 63, wave = tid >> 6;
    bool bad = false;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        if (c < nb1) {
            uint64_t key = 0;
            int sel = 0;
#pragma unroll
            for (int e = 0; e < RPT; ++e) {
                const uint64_t ke = open[e] ? mag_key(rowv[e][c]) : 0;
                if (ke > key) {
                    key = ke;
                    sel = e;
                }
            }
            const int first = __ffsll((unsigned long long)wave_best(key)) - 1;
            if (lane == first) {
                wkey[c & 1][wave] = key;
                wrow[c & 1][wave] = tid + sel * PT;
#pragma unroll
                for (int e = 0; e < RPT; ++e)
                    if (e == sel)
#pragma unroll
                        for (int q = 0; q < NB; ++q) wval[c & 1][wave][q] = rowv[e][q];
            }
            __syncthreads();
            const int bw = __ffs((int)row_best<NW>(wkey[c & 1][lane % NW])) - 1;
            const int p = __builtin_amdgcn_readfirstlane(wrow[c & 1][bw]);
            const double2 d = wval[c & 1][bw][c];
            const double2 di = recip(d);
            bad = bad || !(d.x * d.x + d.y * d.y > 0.0);
            double2 rk[NB];
#pragma unroll
            for (int q = 0; q < NB; ++q) rk[q] = cmul(q == c ? make_double2(1.0, 0.0) : wval[c & 1][bw][q], di);
#pragma unroll
            for (int e = 0; e < RPT; ++e) {
                const int i = tid + e * PT;
                const double2 l = i == p ? make_double2(0, 0) : rowv[e][c];
                if (i < n) nxt.L[(int64_t)c * n + i] = l;
#pragma unroll
                for (int q = 0; q < NB; ++q)
                    rowv[e][q] = csub(q == c ? make_double2(0, 0) : rowv[e][q], cmul(l, rk[q]));
                if (i == p) {
                    open[e] = false;
#pragma unroll
                    for (int q = 0; q < NB; ++q) rowv[e][q] = rk[q];
                }
            }
            if (tid == 0) {
                piv[k1 + c] = p;
                nxt.dv[c] = di;
            }
        }
    }
#pragma unroll
    for (int e = 0; e < RPT; ++e) {
        const int i = tid + e * PT;
        if (i < n) {
            used[i] = open[e] ? 0 : 1;
#pragma unroll
            for (int c = 0; c < NB; ++c)
                if (c < nb1) nxt.F[(int64_t)c * n + i] = rowv[e][c];
        }
    }
    if (tid == 0 && bad) *singular = 1;
}

// out[k][p_j] = in[p_k][j]
__global__ void gj_unscramble_kernel(const double2* __restrict__ in, double2* __restrict__ out, int n,
                                     const int* __restrict__ piv) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const int k = (int)(t / n), j = (int)(t % n);
    out[(int64_t)k * n + piv[j]] = in[(int64_t)piv[k] * n + j];
}

// out[i][j] = in[i][src[j]]
__global__ void permute_cols_kernel(const double2* __restrict__ in, double2* __restrict__ out, int n,
                                    const int* __restrict__ src) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const int i = (int)(t / n), j = (int)(t % n);
    out[t] = in[(int64_t)i * n + src[j]];
}

// The row interchanges of the elimination become column interchanges of the
// inverse, last first; one thread, n swaps (a small part of the n launches before it).
// An out-of-range pivot marks the matrix singular.
__global__ void perm_from_pivots_kernel(const int* __restrict__ piv, int* __restrict__ src, int n,
                                        int* __restrict__ flag) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    for (int j = 0; j < n; ++j) src[j] = j;
    for (int k = n - 1; k >= 0; --k) {
        const int p = piv[k];
        if (p < 0 || p >= n) {
            *flag = 1;
            return;
        }
        const int t = src[k];
        src[k] = src[p];
        src[p] = t;
    }
}

__global__ void clear_flag_kernel(int* flag) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *flag = 0;
}

__global__ void add_diag_kernel(const double2* __restrict__ in, double2* __restrict__ out, int n, double z) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    double2 v = in[t];
    if (t / n == t % n) v.x += z;
    out[t] = v;
}

// S = I - 2 z0 B
__global__ void s_from_inv_kernel(const double2* __restrict__ B, double2* __restrict__ S, int n, double z0) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const double2 b = B[t];
    S[t] = make_double2(((t / n == t % n) ? 1.0 : 0.0) - 2.0 * z0 * b.x, -2.0 * z0 * b.y);
}

// One workgroup per scan direction.  Zp and S are column-major P x P.
__global__ __launch_bounds__(256) void scan_kernel(const double2* __restrict__ Zp, const double2* __restrict__ S, int nx,
                                                   int ny, double dx, double dy, double k, int c,
                                                   const double* __restrict__ theta, const double* __restrict__ phi,
                                                   double z0, double2* __restrict__ Za, double2* __restrict__ G,
                                                   double2* __restrict__ Gw) {
    __shared__ double2 sz[256], ss[256];
    const int sidx = blockIdx.x;
    const int P = nx * ny;
    const double u = sin(theta[sidx]) * cos(phi[sidx]);
    const double v = sin(theta[sidx]) * sin(phi[sidx]);
    double2 az = make_double2(0, 0), as = make_double2(0, 0);
    for (int j = threadIdx.x; j < P; j += 256) {
        const double xj = (j % nx) * dx, yj = (j / nx) * dy;
        double sn, cs;
        sincos(k * (xj * u + yj * v), &sn, &cs);
        const double2 ph = make_double2(cs, -sn);   // I_j = exp(-j k (x_j u + y_j v))
        az = cadd(az, cmul(Zp[(int64_t)j * P + c], ph));
        if (S) as = cadd(as, cmul(S[(int64_t)j * P + c], ph));
    }
    sz[threadIdx.x] = az;
    ss[threadIdx.x] = as;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            sz[threadIdx.x] = cadd(sz[threadIdx.x], sz[threadIdx.x + s]);
            ss[threadIdx.x] = cadd(ss[threadIdx.x], ss[threadIdx.x + s]);
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double xc = (c % nx) * dx, yc = (c / nx) * dy;
        double sn, cs;
        sincos(k * (xc * u + yc * v), &sn, &cs);
        const double2 pc = make_double2(cs, sn);    // 1 / I_c
        const double2 za = cmul(sz[0], pc);
        Za[sidx] = za;
        const double2 num = make_double2(za.x - z0, za.y), den = make_double2(za.x + z0, za.y);
        const double dd = den.x * den.x + den.y * den.y;
        G[sidx] = make_double2((num.x * den.x + num.y * den.y) / dd, (num.y * den.x - num.x * den.y) / dd);
        if (Gw) Gw[sidx] = cmul(ss[0], pc);
    }
}

inline unsigned g1(int64_t n) { return (unsigned)((n + 255) / 256); }

// Rows up to PT * RPT.  Workspace in out (n > 64): two panels' multipliers, columns
// and reciprocal pivots, the used-row marks.
template <int NB, int PT, int RPT, int SW>
void gj_panels(double2* A, double2* out, int n, int* piv, int* flag, hipStream_t s) {
    MBT_REQUIRE(n > 64 && n <= PT * RPT, "panelled inverse: size out of range");
    GjPanel<NB> pan[2];
    const size_t pn = (size_t)NB * n;
    for (int h = 0; h < 2; ++h) {
        pan[h].L = out + h * pn;
        pan[h].P = out + (2 + h) * pn;
        pan[h].F = out + (4 + h) * pn;
        pan[h].dv = out + 6 * pn + h * NB;
    }
    int* used = reinterpret_cast<int*>(out + 6 * pn + 2 * NB);
    auto step = [&](int k0, int nb0) {
        const int k1 = k0 + nb0, nb1 = std::min(NB, n - k1), nb2 = std::min(NB, n - k1 - nb1);
        const int h = nb0 ? (k0 / NB) & 1 : 1;   // the current panel's buffers
        const int strips = nb0 ? (n + SW - 1) / SW - (nb1 + SW - 1) / SW : 0;
        hipLaunchKernelGGL((gj_step_kernel<NB, PT, RPT, SW>), dim3(1 + (SW == 4 ? (strips + 15) / 16 * 16 : strips)),
                           dim3(PT), 0, s, A, n, k0, nb0, k1, nb1, nb2, k1 >= 2 * NB ? 1 : 0, pan[h], pan[h ^ 1], piv,
                           used, flag);
    };
    step(0, 0);
    for (int k0 = 0; k0 < n; k0 += NB) step(k0, std::min(NB, n - k0));
}

}  // namespace

namespace {

// The elimination and the inverse into out, all on the device; flag receives 1 if a
// pivot's squared magnitude is zero or NaN (an infinite one passes, as its reciprocal 0 or NaN).
// Each form takes what its registers hold (64 rows x 4 columns a thread; panel rows per
// thread: one to 512, two to 1024, four beyond, so that the factoring workgroup has no
// more waves to gather per step than it needs; with the copies 512 rows take 2.98 ms at
// two rows a thread and 2.80 at one, 1024 the same with 1,024 threads).  Lattices have up to
// 4,096 ports; above, only callers of the bare inverse get there.
void gj_on_device(double2* A, double2* out, int n, double2* colbuf, int* piv, int* flag, hipStream_t s) {
    hipLaunchKernelGGL(clear_flag_kernel, dim3(1), dim3(64), 0, s, flag);
    if (n <= 32) {
        hipLaunchKernelGGL((gj_small_kernel<32, 8, 4>), dim3(1), dim3(256), 0, s, A, n, out, flag);
    } else if (n <= 64) {
        hipLaunchKernelGGL((gj_small_kernel<64, 16, 4>), dim3(1), dim3(1024), 0, s, A, n, out, flag);
    } else if (n <= 4096) {
        if (n <= 256) gj_panels<8, 256, 1, 4>(A, out, n, piv, flag, s);
        else if (n <= 512) gj_panels<8, 512, 1, 4>(A, out, n, piv, flag, s);
        else if (n <= 1024) gj_panels<8, 512, 2, 4>(A, out, n, piv, flag, s);
        else if (n <= 2048) gj_panels<8, 512, 4, 8>(A, out, n, piv, flag, s);
        else gj_panels<4, 1024, 4, 4>(A, out, n, piv, flag, s);
        hipLaunchKernelGGL(gj_unscramble_kernel, dim3(g1((int64_t)n * n)), dim3(256), 0, s, A, out, n, piv);
    } else {
        for (int k = 0; k < n; ++k) {
            hipLaunchKernelGGL(gj_pivot_kernel, dim3(1), dim3(kPivT), 0, s, A, n, k, colbuf, piv, flag);
            hipLaunchKernelGGL(gj_elim_kernel, dim3(g1((int64_t)n * n)), dim3(256), 0, s, A, n, k, colbuf);
        }
        int* src = reinterpret_cast<int*>(colbuf);
        hipLaunchKernelGGL(perm_from_pivots_kernel, dim3(1), dim3(64), 0, s, piv, src, n, flag);
        hipLaunchKernelGGL(permute_cols_kernel, dim3(g1((int64_t)n * n)), dim3(256), 0, s, A, out, n, src);
    }
    MBT_LAUNCH_CHECK();
}

}  // namespace

// Gauss-Jordan inverse of A (n x n, any consistent layout: the inverse of the stored
// array is returned in the same layout) into out, which must not overlap A; A is
// overwritten.  Workspace: colbuf n complex, piv n ints, flag one int.
void gj_inverse(double2* A, double2* out, int n, double2* colbuf, int* piv, int* flag, hipStream_t s) {
    gj_on_device(A, out, n, colbuf, piv, flag, s);
    int hflag = 0;
    MBT_HIP(hipMemcpyAsync(&hflag, flag, sizeof(int), hipMemcpyDeviceToHost, s));
    MBT_HIP(hipStreamSynchronize(s));
    if (hflag) throw Error(-1, "port matrix is singular");
}

// The same with no pageable host memory: one 4-byte readback of the singularity
// flag into pinned host memory.
static void gj_inverse_dev_perm(double2* A, double2* out, int n, double2* colbuf, int* piv, int* flag, int* host_flag,
                                hipStream_t s) {
    gj_on_device(A, out, n, colbuf, piv, flag, s);
    MBT_HIP(hipMemcpyAsync(host_flag, flag, sizeof(int), hipMemcpyDeviceToHost, s));
    MBT_HIP(hipStreamSynchronize(s));
    if (*host_flag) throw Error(-1, "port matrix is singular");
}

void s_matrix_dev_perm(const double2* Zp, double2* S, double2* work, int n, double z0, double2* colbuf, int* piv,
                       int* flag, int* host_flag, hipStream_t s) {
    hipLaunchKernelGGL(add_diag_kernel, dim3(g1((int64_t)n * n)), dim3(256), 0, s, Zp, work, n, z0);
    MBT_LAUNCH_CHECK();
    gj_inverse_dev_perm(work, S, n, colbuf, piv, flag, host_flag, s);   // S holds (Zp + z0)^{-1}
    hipLaunchKernelGGL(s_from_inv_kernel, dim3(g1((int64_t)n * n)), dim3(256), 0, s, S, S, n, z0);
    MBT_LAUNCH_CHECK();
}

void s_matrix(const double2* Zp, double2* S, double2* work, int n, double z0, double2* colbuf, int* piv, int* flag,
              hipStream_t s) {
    hipLaunchKernelGGL(add_diag_kernel, dim3(g1((int64_t)n * n)), dim3(256), 0, s, Zp, work, n, z0);
    MBT_LAUNCH_CHECK();
    gj_inverse(work, S, n, colbuf, piv, flag, s);        // S holds (Zp + z0)^{-1}
    hipLaunchKernelGGL(s_from_inv_kernel, dim3(g1((int64_t)n * n)), dim3(256), 0, s, S, S, n, z0);
    MBT_LAUNCH_CHECK();
}

void scans(const Geom& g, double k, const double2* Zp, const double2* S, int c, const double* theta, const double* phi,
           int nscan, double z0, double2* Za, double2* G, double2* Gw, hipStream_t s) {
    if (nscan <= 0) return;
    hipLaunchKernelGGL(scan_kernel, dim3(nscan), dim3(256), 0, s, Zp, S, g.nx, g.ny, g.dx, g.dy, k, c, theta, phi, z0,
                       Za, G, Gw);
    MBT_LAUNCH_CHECK();
}

__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
    const double d = b.x * b.x + b.y * b.y;
    return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}

// V[(e*M + idx_i)][r] = w_i exp(-j k (x_e u_r + y_e v_r)) for every element e (V pre-zeroed)
__global__ void scan_voltages_kernel(int nx, int P, double dx, double dy, double k, const double* __restrict__ theta,
                                     const double* __restrict__ phi, int R, int M, PortDef pd,
                                     double2* __restrict__ V) {
    const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (t >= (int64_t)P * R) return;
    const int r = (int)(t % R);
    const int e = (int)(t / R);
    const double u = sin(theta[r]) * cos(phi[r]), v = sin(theta[r]) * sin(phi[r]);
    double sn, cs;
    sincos(k * ((e % nx) * dx * u + (e / nx) * dy * v), &sn, &cs);
    for (int i = 0; i < pd.n; ++i) V[((int64_t)e * M + pd.idx[i]) * R + r] = make_double2(pd.w[i] * cs, -pd.w[i] * sn);
}

// Za[r] = V_c,r / Ip[c + P r], G[r] = (Za - z0)/(Za + z0)
__global__ void scan_active_kernel(const double2* __restrict__ Ip, int P, int nscan, int c, int nx, double dx,
                                   double dy, double k, const double* __restrict__ theta,
                                   const double* __restrict__ phi, double z0, double2* __restrict__ Za,
                                   double2* __restrict__ G) {
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= nscan) return;
    const double u = sin(theta[r]) * cos(phi[r]), v = sin(theta[r]) * sin(phi[r]);
    double sn, cs;
    sincos(k * ((c % nx) * dx * u + (c / nx) * dy * v), &sn, &cs);
    const double2 za = cdiv(make_double2(cs, -sn), Ip[(int64_t)c + (int64_t)P * r]);
    Za[r] = za;
    G[r] = cdiv(make_double2(za.x - z0, za.y), make_double2(za.x + z0, za.y));
}

void scan_voltages(const Geom& g, double k, const double* theta, const double* phi, int R, double2* V,
                   hipStream_t s) {
    zero_d(V, g.N * R, s);
    const int64_t n = (int64_t)g.P * R;
    hipLaunchKernelGGL(scan_voltages_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, g.nx, g.P, g.dx, g.dy,
                       k, theta, phi, R, g.M, g.port, V);
    MBT_LAUNCH_CHECK();
}

void scan_active(const Geom& g, double k, const double2* Ip, int nscan, int c, const double* theta,
                 const double* phi, double z0, double2* Za, double2* G, hipStream_t s) {
    hipLaunchKernelGGL(scan_active_kernel, dim3((nscan + 63) / 64), dim3(64), 0, s, Ip, g.P, nscan, c, g.nx, g.dx,
                       g.dy, k, theta, phi, z0, Za, G);
    MBT_LAUNCH_CHECK();
}

}  // namespace mbt
