// Binary64 residual R = B - A X and the norms of the backward error
// (Algorithm 1's residual steps, the ones it carries out in high precision).
//
// A is symmetric with only its lower triangle stored.  One or two right-hand
// sides: one pass over the lower triangle, every stored element serving its
// row and its column (k_resid_sym).  More: the whole symmetric matrix on
// binary64 MFMA, the part right of the diagonal read from the lower
// triangle's columns (k_resid_mfma).  Both leave partial sums that a second
// kernel adds in a fixed order, so results are bitwise reproducible run to
// run.  The same pass can accumulate sum_j |a_ij| for ||A||_inf.
#include "common.h"
#include "internal.h"
#include <algorithm>

// The whole symmetric matrix times X for up to 16 NT right-hand sides on
// v_mfma_f64_16x16x4f64.  Workgroup (I, s): rows [128 I, 128 I + 128), the
// 64-column tiles J = s, s + S, ...; each wave owns 32 rows.  The k-slots of
// the MFMA are a free summation order: lane (r = lane % 16, u = lane / 16)
// takes columns 16 g + 8 e + 2 u + q of a tile at step (e, q) of group g.  Left of the
// diagonal its values are then 128-byte runs of rows (lanes r), right of it
// -- the transpose, stored as columns -- 16-byte loads that cover 64-byte runs
// of a column (lanes u): A goes from memory to the MFMA's registers without shared memory,
// the next tile's values in flight while the current one is multiplied.  X's
// tile is shared by the four waves through LDS (two buffers, one barrier per
// tile; pitch 66 doubles: 16-byte reads of 16 columns without bank
// conflicts).  Operands are given as (X, A), so that register v of a lane is
// right-hand side 4 v + u, row r: partials are stored along rows.
// The products of two tiles (128 columns) make one sum, added to those before,
// and the slices are added in pairs: the rounding error, in units of
// u |a||x| sqrt(n), is 0.92, 1.6 and 2.0 at n = 1300, 6000 and 12000.  One sum
// over a workgroup's whole slice, and the slices one after the other, gave
// 1.5, 5.7 and 13.6 (and 1.5, 3.4 and 9.1 with twice the slices).  At 17 and
// more columns the sums of the tiles before stay in shared memory, a thread's
// own places: in registers 45 values would spill (n = 12000: 531 us a call).
// Bound by reading the symmetric A once per chunk of 32 right-hand sides, and
// by the binary64 MFMA rate at 17..32 columns.  Staging A's 64 x 64 tiles
// through shared memory (two barriers per tile, X re-read for every 64 rows)
// took 256 us at n = 10000 with 32 columns and 362 at n = 12000, without the
// reduction; with it this takes 221 and 296 us (3.9 TB/s).  With 5 columns at
// n = 6000, and 8 at 16384, 69 and 382 us.
typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));  // 16-byte load, 8-byte aligned
template <int NT>
__global__ __launch_bounds__(256, 2) void k_resid_mfma(const double *__restrict__ A, int64_t lda, int64_t n,
                                                       const double *__restrict__ X, int64_t ldx, int m, int c0,
                                                       int S, double *__restrict__ P, double *__restrict__ Pabs,
                                                       int want_abs)
{
    constexpr int MC = 16 * NT, PX = 66, XU = MC * 64 / 256;
    __shared__ __align__(16) double Xs[2][MC * PX];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r = lane & 15, u = lane >> 4;
    const int s = blockIdx.y;
    const int64_t iw = (int64_t)blockIdx.x * 128 + 32 * w;  // the wave's first row
    const int njt = (int)((n + 63) / 64);
    doublex4 acc[2][NT];  // of one or two tiles; tot of those before, a thread's own places where registers are short
    __shared__ __align__(16) double2 tots[NT > 1 ? 4 * NT : 1][256];
    doublex4 tot[2][NT];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            tot[h][t] = doublex4{0.0, 0.0, 0.0, 0.0};
            if constexpr (NT > 1)
                tots[2 * (NT * h + t)][tid] = tots[2 * (NT * h + t) + 1][tid] = double2{0.0, 0.0};
        }
    double aabs[2] = {0.0, 0.0};
    // a[h][g][2 e + q]: row iw + 16 h + r, column 64 J + 16 g + 8 e + 2 u + q
    auto fetch = [&](double (&a)[2][4][4], int J) {
        const int64_t j0 = (int64_t)J * 64;
        if (iw + 32 <= n && j0 + 64 <= iw) {
            const double *p = A + iw + r + (j0 + 2 * u) * lda;
#pragma unroll
            for (int g = 0; g < 4; ++g)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int h = 0; h < 2; ++h) a[h][g][q] = p[16 * h + (int64_t)(16 * g + 8 * (q >> 1) + (q & 1)) * lda];
        } else if (j0 + 64 <= n && j0 >= iw + 32) {
            const double *p = A + j0 + 2 * u + (iw + r) * lda;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int q = 0; q < 4; q += 2) {
                        const double2u v = *(const double2u *)(p + 16 * h * lda + 16 * g + 4 * q);
                        a[h][g][q] = v.x;
                        a[h][g][q + 1] = v.y;
                    }
        } else {  // on the diagonal, or at the matrix's edge
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int64_t gi = iw + 16 * h + r, gj = j0 + 16 * g + 8 * (q >> 1) + 2 * u + (q & 1);
                        a[h][g][q] = (gi < n && gj < n) ? (gi >= gj ? A[gi + gj * lda] : A[gj + gi * lda]) : 0.0;
                    }
        }
    };
    double xv[XU];
    auto fetch_x = [&](int J) {
        const int64_t gj = (int64_t)J * 64 + (tid & 63);
#pragma unroll
        for (int e = 0; e < XU; ++e) {
            const int c = c0 + (tid >> 6) + 4 * e;
            xv[e] = (gj < n && c < m) ? X[gj + (int64_t)c * ldx] : 0.0;
        }
    };
    auto stage_x = [&](int buf) {
#pragma unroll
        for (int e = 0; e < XU; ++e) Xs[buf][((tid >> 6) + 4 * e) * PX + (tid & 63)] = xv[e];
    };
    auto multiply = [&](const double (&a)[2][4][4], int buf) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            double2 x[NT][2];
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    x[t][e] = *(const double2 *)&Xs[buf][(16 * t + r) * PX + 16 * g + 8 * e + 2 * u];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        acc[h][t] = __builtin_amdgcn_mfma_f64_16x16x4f64((q & 1) ? x[t][q >> 1].y : x[t][q >> 1].x,
                                                                         a[h][g][q], acc[h][t], 0, 0, 0);
        }
        if (want_abs)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int q = 0; q < 4; ++q) aabs[h] += fabs(a[h][g][q]);
    };
    auto fold = [&]() {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (NT > 1) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        double2 &p = tots[2 * (NT * h + t) + e][tid];
                        const double2 v = p;
                        p = double2{v.x + acc[h][t][2 * e], v.y + acc[h][t][2 * e + 1]};
                    }
                } else {
                    tot[h][t] += acc[h][t];
                }
            }
    };
    double a0[2][4][4], a1[2][4][4];
    if (s < njt) {
        fetch_x(s);
        fetch(a0, s);
        stage_x(0);
    }
    __syncthreads();
    for (int J = s; J < njt; J += 2 * S) {
        if (J + S < njt) {
            fetch_x(J + S);
            fetch(a1, J + S);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[h][t] = doublex4{0.0, 0.0, 0.0, 0.0};
        multiply(a0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (J + S < njt)
            stage_x(1);
        __syncthreads();
        if (J + S >= njt) {
            fold();
            break;
        }
        if (J + 2 * S < njt) {
            fetch_x(J + 2 * S);
            fetch(a0, J + 2 * S);
        }
        __builtin_amdgcn_sched_barrier(0);
        multiply(a1, 1);
        fold();
        __builtin_amdgcn_sched_barrier(0);
        if (J + 2 * S < njt)
            stage_x(0);
        __syncthreads();
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int64_t gi = iw + 16 * h + r;
        if constexpr (NT > 1)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; v += 2) {
                    const double2 p = tots[2 * (NT * h + t) + v / 2][tid];
                    tot[h][t][v] = p.x;
                    tot[h][t][v + 1] = p.y;
                }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int c = c0 + 16 * t + 4 * v + u;
                if (gi < n && c < m) P[((int64_t)s * m + c) * n + gi] = tot[h][t][v];
            }
        if (want_abs) {  // the four k-slots of a row, in a fixed order
            double v = aabs[h];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (u == 0 && gi < n) Pabs[(int64_t)s * n + gi] = v;
        }
    }
}

// Single pass over the lower triangle for one or two right-hand sides.
// Workgroup (J, q) walks tiles I = J + q ch .. of the 64-column strip J
// (contiguous in memory); wave w holds columns 16 w .. 16 w + 15 of the tile,
// lane l its row l.  Each stored a_ij (i > j) serves twice: a_ij x_j for row i
// (a row partial per tile, RP[I][J]) and a_ij x_i for row j (accumulated over
// the chunk in registers, CP[J][q]); a diagonal tile uses its lower triangle
// only (the diagonal once).  k_resid_sym_reduce then sums, per row of block I,
// RP[I][0..I] (as four interleaved sums) and CP[I][.], in a fixed order.  With
// WA an extra "column" c = MC carries |a_ij| (row sums of |A|).
// Bound by reading the triangle (224 us, 4.8 TB/s, at n = 16384).  ch tiles
// per workgroup: 16 where that leaves 512 workgroups, fewer on smaller
// matrices, whose chunks of 16 tiles in sequence left the chip idle, and the
// column sums reduced 16 at a time (a lane keeps half of its sums at each
// exchange: 17 exchanges instead of 96).  n = 300: 12.2 us before, 7.0 now;
// n = 3000: 26.0 and 16.9 us.  (More column partials then: the reduction sums
// them apart from the row partials, or they would cost accuracy: n = 2500
// 1.05 u |a||x| sqrt(n), and 1.23 behind the rows'.)
#define RSYM_CH 16
template <int MC, bool WA>
__global__ __launch_bounds__(256) void k_resid_sym(const double *__restrict__ A, int64_t lda, int64_t n,
                                                   const double *__restrict__ X, int64_t ldx, int m, int ch, int Q,
                                                   double *__restrict__ RP, double *__restrict__ CP)
{
    constexpr int NC = MC + 1;  // partial "columns" in the layout: MC right-hand sides + |A|
    constexpr int NA = WA ? NC : MC;  // the ones this variant computes
    constexpr int CW = 16;
    __shared__ double xs[MC][64];
    __shared__ double red[2][4][NA][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int J = blockIdx.x, q = blockIdx.y;
    const int nrb = (int)((n + 63) / 64);
    const int I0 = J + q * ch, I1 = min(I0 + ch, nrb);
    if (I0 >= nrb)
        return;
    const int64_t j0 = (int64_t)J * 64;
    // x of the strip's columns, for the row partials
    for (int idx = threadIdx.x; idx < MC * 64; idx += 256) {
        const int c = idx / 64, j = idx % 64;
        xs[c][j] = (j0 + j < n && c < m) ? X[(j0 + j) + (int64_t)c * ldx] : 0.0;
    }
    __syncthreads();
    double cacc[CW][NA];
#pragma unroll
    for (int jj = 0; jj < CW; ++jj)
#pragma unroll
        for (int c = 0; c < NA; ++c) cacc[jj][c] = 0.0;
    // tile loads run one tile ahead of the arithmetic
    double an[CW];
    auto load_tile = [&](int I) {
        const int64_t gi = (int64_t)I * 64 + lane;
#pragma unroll
        for (int jj = 0; jj < CW; ++jj) {
            const int64_t gj = j0 + CW * w + jj;
            an[jj] = (gi < n && gj < n) ? A[gi + gj * lda] : 0.0;
        }
    };
    if (I0 == J) {  // the tile on the diagonal, always a chunk's first: its lower triangle
#pragma unroll
        for (int jj = 0; jj < CW; ++jj) {
            const int64_t gi = j0 + lane, gj = j0 + CW * w + jj;
            an[jj] = (gi < n && gj <= gi) ? A[gi + gj * lda] : 0.0;
        }
    } else {
        load_tile(I0);
    }
    for (int I = I0; I < I1; ++I) {
        const int64_t gi = (int64_t)I * 64 + lane;
        double a[CW];
#pragma unroll
        for (int jj = 0; jj < CW; ++jj) a[jj] = an[jj];
        if (I + 1 < I1)
            load_tile(I + 1);
        const int dj = lane - CW * w;  // on the diagonal tile: row minus the wave's first column
        double xi[MC];
#pragma unroll
        for (int c = 0; c < MC; ++c) xi[c] = (gi < n && c < m) ? X[gi + (int64_t)c * ldx] : 0.0;
        double racc[NA];
#pragma unroll
        for (int c = 0; c < NA; ++c) racc[c] = 0.0;
#pragma unroll
        for (int jj = 0; jj < CW; ++jj) {
            const bool strict = (I != J) || (dj > jj);
#pragma unroll
            for (int c = 0; c < MC; ++c) {
                racc[c] = fma(a[jj], xs[c][CW * w + jj], racc[c]);
                if (strict)
                    cacc[jj][c] = fma(a[jj], xi[c], cacc[jj][c]);
            }
            if constexpr (WA) {
                racc[NA - 1] += fabs(a[jj]);
                if (strict)
                    cacc[jj][NA - 1] += fabs(a[jj]);
            }
        }
        // row partial of tile (I, J): sum over the 4 waves in order (the two
        // buffers alternate, so one barrier per tile)
        double(*rd)[NA][64] = red[I & 1];
#pragma unroll
        for (int c = 0; c < NA; ++c) rd[w][c][lane] = racc[c];
        __syncthreads();
        for (int idx = threadIdx.x; idx < NA * 64; idx += 256) {
            const int c = idx / 64, i = idx % 64;
            RP[(((int64_t)I * nrb + J) * NC + c) * 64 + i] = ((rd[0][c][i] + rd[1][c][i]) + rd[2][c][i]) + rd[3][c][i];
        }
    }
    // column partials: the 64 lanes of all 16 columns together, in a fixed
    // order -- at each exchange a lane hands over half of its sums and adds
    // its partner's to the half it keeps; lane l ends with column l / 4
#pragma unroll
    for (int c = 0; c < NA; ++c) {
#pragma unroll
        for (int h = CW / 2, off = 32; h >= 1; h /= 2, off /= 2) {
            const bool up = (lane & off) != 0;
#pragma unroll
            for (int k = 0; k < h; ++k) {
                const double give = up ? cacc[k][c] : cacc[k + h][c];
                const double keep = up ? cacc[k + h][c] : cacc[k][c];
                cacc[k][c] = keep + __shfl_xor(give, off);
            }
        }
        double v = cacc[0][c];
        v += __shfl_xor(v, 2);
        v += __shfl_xor(v, 1);
        if ((lane & 3) == 0)
            CP[(((int64_t)J * Q + q) * NC + c) * 64 + CW * w + (lane >> 2)] = v;
    }
}

SPD_DEV double nanmax2(double a, double b) { return (a > b || a != a) ? a : b; }
SPD_DEV double wave_max2(double v)
{
    for (int off = 32; off > 0; off >>= 1)
        v = nanmax2(v, __shfl_xor(v, off));
    return v;
}

__global__ __launch_bounds__(256) void k_resid_reduce(const double *__restrict__ B, int64_t ldb,
                                                      const double *__restrict__ X, int64_t ldx, int64_t n, int m,
                                                      int S, const double *__restrict__ P,
                                                      const double *__restrict__ Pabs, int want_abs,
                                                      const double *__restrict__ d, double *__restrict__ R,
                                                      int64_t ldr, double *norms)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int c = blockIdx.y;
    double vr = 0.0, vx = 0.0, vb = 0.0, vd = 0.0, va = 0.0;
    if (i < n) {
        // eight slices at a time, added in pairs (their loads in flight: one at
        // a time they cost a memory round trip each, 10.6 us for the 21 slices
        // of n = 1300)
        auto total = [&](const double *p, int64_t st) {
            double sum = 0.0;
            for (int s0 = 0; s0 < S; s0 += 8) {
                double v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = (s0 + k < S) ? p[(s0 + k) * st] : 0.0;
                sum += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            }
            return sum;
        };
        const double sum = total(P + (int64_t)c * n + i, (int64_t)m * n);
        const double b = B[i + c * ldb];
        const double r = b - sum;
        R[i + c * ldr] = r;
        vr = fabs(r);
        vx = fabs(X[i + c * ldx]);
        vb = fabs(b);
        vd = d ? fabs(d[i] * r) : vr;
        if (want_abs && c == 0)
            va = total(Pabs + i, n);
    }
    vr = wave_max2(vr);
    vx = wave_max2(vx);
    vb = wave_max2(vb);
    vd = wave_max2(vd);
    if (want_abs && c == 0)
        va = wave_max2(va);
    if ((threadIdx.x & 63) == 0) {
        atomic_max_nonneg(norms + 1 + c, vr);
        atomic_max_nonneg(norms + 1 + m + c, vx);
        atomic_max_nonneg(norms + 1 + 2 * m + c, vb);
        atomic_max_nonneg(norms + 1 + 3 * m + c, vd);
        if (want_abs && c == 0)
            atomic_max_nonneg(norms, va);
    }
}

// R = B - (sum_J RP[I][J] + sum_q CP[I][q]) and the norms (as k_resid_reduce).
// Workgroup (I, c): 64 rows of block I, four waves; wave p sums the row
// partials J = p, p + 4, ... and the column partials q = p, p + 4, ... (four
// at a time: their loads in flight, and added in pairs), each kind to a sum of
// its own, and the four waves' sums are added in the fixed order
// (s0 + s1) + (s2 + s3).
template <int MC>
__global__ __launch_bounds__(256) void k_resid_sym_reduce(const double *__restrict__ B, int64_t ldb,
                                                          const double *__restrict__ X, int64_t ldx, int64_t n, int m,
                                                          int ch, int Q, const double *__restrict__ RP,
                                                          const double *__restrict__ CP, int want_abs,
                                                          const double *__restrict__ d, double *__restrict__ R,
                                                          int64_t ldr, double *norms)
{
    constexpr int NC = MC + 1;
    __shared__ double part[2][4][64];
    const int il = threadIdx.x & 63, p = threadIdx.x >> 6;
    const int I = blockIdx.x, c = blockIdx.y;
    const int nrb = (int)((n + 63) / 64);
    const bool wa = want_abs && c == 0;
    {
        // v = p, p + 4, ... < cnt, consecutive ones st doubles apart
        auto sum = [&](const double *rp, const double *ra, int64_t st, int cnt, double &y, double &ya) {
            int v = p;
            for (; v + 12 < cnt; v += 16) {
                const double v0 = rp[v * st], v1 = rp[(v + 4) * st], v2 = rp[(v + 8) * st], v3 = rp[(v + 12) * st];
                if (wa) {
                    const double a0 = ra[v * st], a1 = ra[(v + 4) * st], a2 = ra[(v + 8) * st], a3 = ra[(v + 12) * st];
                    ya += (a0 + a1) + (a2 + a3);
                }
                y += (v0 + v1) + (v2 + v3);
            }
            for (; v < cnt; v += 4) {
                y += rp[v * st];
                if (wa)
                    ya += ra[v * st];
            }
        };
        const double *rp = RP + (int64_t)I * nrb * NC * 64 + il, *cp = CP + (int64_t)I * Q * NC * 64 + il;
        double y = 0.0, ya = 0.0, yc = 0.0, yca = 0.0;
        sum(rp + c * 64, rp + MC * 64, (int64_t)NC * 64, I + 1, y, ya);
        sum(cp + c * 64, cp + MC * 64, (int64_t)NC * 64, (nrb - I + ch - 1) / ch, yc, yca);
        y += yc;
        ya += yca;
        part[0][p][il] = y;
        part[1][p][il] = ya;
    }
    __syncthreads();
    if (p != 0)
        return;
    const int64_t i = (int64_t)I * 64 + il;
    double vr = 0.0, vx = 0.0, vb = 0.0, vd = 0.0, va = 0.0;
    if (i < n) {
        const double y = (part[0][0][il] + part[0][1][il]) + (part[0][2][il] + part[0][3][il]);
        const double ya = (part[1][0][il] + part[1][1][il]) + (part[1][2][il] + part[1][3][il]);
        const double b = B[i + c * ldb];
        const double r = b - y;
        R[i + c * ldr] = r;
        vr = fabs(r);
        vx = fabs(X[i + c * ldx]);
        vb = fabs(b);
        vd = d ? fabs(d[i] * r) : vr;
        va = ya;
    }
    vr = wave_max2(vr);
    vx = wave_max2(vx);
    vb = wave_max2(vb);
    vd = wave_max2(vd);
    if (wa)
        va = wave_max2(va);
    if (il == 0) {
        atomic_max_nonneg(norms + 1 + c, vr);
        atomic_max_nonneg(norms + 1 + m + c, vx);
        atomic_max_nonneg(norms + 1 + 2 * m + c, vb);
        atomic_max_nonneg(norms + 1 + 3 * m + c, vd);
        if (wa)
            atomic_max_nonneg(norms, va);
    }
}

namespace spd {

// column slices of the MFMA residual: two workgroups per compute unit (512)
// in one round, at most 64
static int resid_splits(int64_t n)
{
    const int64_t nb = (n + 127) / 128, nj = (n + 63) / 64;
    int64_t S = 512 / (nb > 0 ? nb : 1);
    S = std::min<int64_t>(std::min<int64_t>(S, nj), 64);
    return (int)std::max<int64_t>(S, 1);
}

// Shape of the single pass over the triangle (one or two right-hand sides)
#define RSYM_MAX_M 2
struct RsymShape {
    int nrb, ch, Q;
    int64_t rp, cp;  // doubles of the row and column partials
};
static RsymShape rsym_shape(int64_t n, int m)
{
    RsymShape h;
    const int64_t nrb = (n + 63) / 64;
    h.nrb = (int)nrb;
    h.ch = (int)std::max<int64_t>(1, std::min<int64_t>(RSYM_CH, nrb * nrb / 2 / 512));
    h.Q = (int)((nrb + h.ch - 1) / h.ch);
    h.rp = nrb * nrb * ((m <= 1 ? 1 : 2) + 1) * 64;
    h.cp = nrb * h.Q * ((m <= 1 ? 1 : 2) + 1) * 64;
    return h;
}

// With more than two right-hand sides at least the layout of 64-row blocks
// times up to 2048 / blocks slices, the size that spd_residual_noalloc's
// limits are stated for.
int64_t resid_scratch(int64_t n, int m)
{
    const int64_t nrb = (n + 63) / 64;
    const int64_t S = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(2048 / std::max<int64_t>(nrb, 1), nrb), 64));
    int64_t need = std::max<int64_t>(S, resid_splits(n)) * n * (m + 1);
    if (m <= RSYM_MAX_M) {
        const RsymShape h = rsym_shape(n, m);
        need = std::max<int64_t>(need, h.rp + h.cp);
    }
    return need;
}

// eta[c] = ||r_c|| / (||A|| ||x_c|| + ||b_c||) from the residual's norms
// (norms[0] = ||A||, then max|r|, max|x|, max|b| per column), rounded as the
// host formula rounds it (no fused multiply-add)
__global__ void k_eta_from_norms(const double *__restrict__ norms, int m, double *__restrict__ eta)
{
#pragma clang fp contract(off)
    const int c = blockIdx.x * 64 + threadIdx.x;
    if (c >= m)
        return;
    const double an = norms[0], rn = norms[1 + c], xn = norms[1 + m + c], bn = norms[1 + 2 * m + c];
    const double den = an * xn + bn;
    double v = (den > 0.0) ? rn / den : (rn > 0.0 ? __builtin_inf() : 0.0);
    if (!(rn == rn) || !(xn == xn) || !(an == an))
        v = __builtin_nan("");
    eta[c] = v;
}

template <int MC>
static void launch_sym(const RsymShape &h, const double *A, int64_t lda, int64_t n, const double *X, int64_t ldx,
                       const double *B, int64_t ldb, int m, double *R, int64_t ldr, const double *d, double *norms,
                       int want_anorm, double *RP, double *CP, hipStream_t st)
{
    const dim3 g((unsigned)h.nrb, (unsigned)h.Q), gr((unsigned)h.nrb, (unsigned)m);
    if (want_anorm)
        hipLaunchKernelGGL((k_resid_sym<MC, true>), g, dim3(256), 0, st, A, lda, n, X, ldx, m, h.ch, h.Q, RP, CP);
    else
        hipLaunchKernelGGL((k_resid_sym<MC, false>), g, dim3(256), 0, st, A, lda, n, X, ldx, m, h.ch, h.Q, RP, CP);
    hipLaunchKernelGGL((k_resid_sym_reduce<MC>), gr, dim3(256), 0, st, B, ldb, X, ldx, n, m, h.ch, h.Q, RP, CP,
                       want_anorm, d, R, ldr, norms);
}

void launch_eta_from_norms(const double *norms, int m, double *eta, hipStream_t st)
{
    if (m <= 0) return;
    hipLaunchKernelGGL(k_eta_from_norms, dim3((unsigned)((m + 63) / 64)), dim3(64), 0, st, norms, m, eta);
}

void launch_residual(const double *A, int64_t lda, int64_t n, const double *X, int64_t ldx, const double *B,
                     int64_t ldb, int m, double *R, int64_t ldr, const double *d, double *norms, int want_anorm,
                     double *P, hipStream_t st)
{
    if (n <= 0 || m <= 0) return;
    if (m <= RSYM_MAX_M) {
        const RsymShape h = rsym_shape(n, m);
        auto go = [&](auto f) { f(h, A, lda, n, X, ldx, B, ldb, m, R, ldr, d, norms, want_anorm, P, P + h.rp, st); };
        if (m <= 1)
            go(launch_sym<1>);
        else
            go(launch_sym<2>);
        return;
    }
    const int S = resid_splits(n);
    double *Pabs = P + (int64_t)S * n * m;
    const dim3 g((unsigned)((n + 127) / 128), (unsigned)S);
    for (int c0 = 0; c0 < m; c0 += 32) {
        const int wa = (want_anorm && c0 == 0) ? 1 : 0;
        if (m - c0 <= 16)
            hipLaunchKernelGGL(k_resid_mfma<1>, g, dim3(256), 0, st, A, lda, n, X, ldx, m, c0, S, P, Pabs, wa);
        else
            hipLaunchKernelGGL(k_resid_mfma<2>, g, dim3(256), 0, st, A, lda, n, X, ldx, m, c0, S, P, Pabs, wa);
    }
    hipLaunchKernelGGL(k_resid_reduce, dim3((unsigned)((n + 255) / 256), (unsigned)m), dim3(256), 0, st, B, ldb, X,
                       ldx, n, m, S, P, Pabs, want_anorm, d, R, ldr, norms);
}

}  // namespace spd
