// Half-precision requests (BF16, FP16) of the batched solver, included by
// k_batch.hip.  A factor with rounded products is good for a few bits per
// correction, and for about one system in a thousand the last bits of its
// factor, solves and residuals decide whether the corrections end within the
// iteration limit -- the request's outcome, half precision or the fallback.
// So this path keeps its order of operations: right-looking over a
// column-major factor, the residual by whole rows from A and a mirror of its
// lower triangle, the solves on the VALU (in the order of the other paths 2 to
// 12 of 4096 requests ended otherwise than here).
#pragma once

namespace half_path {
using T = float;

// shared state of the workgroup
struct SolveSmem {
    double ys[SPD_BATCH_MAXRHS * SPD_BATCH_NMAX];  // solve vectors (factor type)
    double Lk[BNB * (BNB + 1)];                    // inverse of the diagonal block
    double ts[SPD_BATCH_MAXRHS * BNB];
    double red[16][4 * SPD_BATCH_MAXRHS + 1];
    double norms[1 + 4 * SPD_BATCH_MAXRHS];
    double smax[SPD_BATCH_MAXRHS];
    unsigned long long zmax[SPD_BATCH_MAXRHS];  // max |z| per column of the last solve (binary64 bits)
    double arow[SPD_BATCH_NMAX];  // row sums of |A|
    double part[4][SPD_BATCH_MAXRHS + 1][64];  // the residual's per-wave partial row sums (+ |A|)
    int info;
};
// ---------------------------------------------------------------------------
// H = round(mu D A D) (lower), identity padding up to np; d (binary64); and
// Am, A's strict lower triangle mirrored into the strict upper triangle of an
// np x np array, so that the residual can stream whole rows of A with
// coalesced loads while A itself is read only in its lower triangle.  32 x 32
// tiles of the lower triangle, one per wave at a time: the tile is loaded
// once (lane = row, 16 columns per lane), converted into L, and transposed
// through the wave's buffer in shared memory (element (c, r) at
// c * 32 + (r ^ c)) for the mirror's coalesced stores.
template <int WAVES>
__device__ __attribute__((noinline)) void b_convert(const double *A, int n, int np, double *d, double mu, int equil,
                                                    T *L, double *Am, SolveSmem &sm)
{
    // global memory (see gmem): the parameters re-derived as global pointers
    A = (const double *)gmem(A);
    d = (double *)gmem(d);
    L = (T *)gmem(L);
    Am = (double *)gmem(Am);
    constexpr int NT = WAVES * 64;
    static_assert(WAVES * BNB * BNB * 8 <= (int)sizeof(sm.ys), "tile buffers");
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double *dsh = sm.arow;
    for (int i = tid; i < n; i += NT) {
        const double a = A[i + (int64_t)i * n];
        const double di = (equil && a > 0.0) ? 1.0 / sqrt(a) : 1.0;
        d[i] = di;
        dsh[i] = di;
    }
    __syncthreads();
    const int r = lane & 31, h = lane >> 5;
    const int nb = np / BNB, ntiles = nb * (nb + 1) / 2;
    double *tb = sm.ys + wave * BNB * BNB;
    for (int q = wave; q < ntiles; q += WAVES) {
        int I = (int)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);  // q = I (I + 1) / 2 + J, J <= I
        while (I * (I + 1) / 2 > q) --I;
        while ((I + 1) * (I + 2) / 2 <= q) ++I;
        const int J = q - I * (I + 1) / 2;
        const int i = I * BNB + r;
        double a[BNB / 2];
#pragma unroll
        for (int u = 0; u < BNB / 2; ++u) {
            const int j = J * BNB + 2 * u + h;
            a[u] = (i < n && j < n && j <= i) ? A[i + (int64_t)j * n] : 0.0;
        }
        const double di = (i < n) ? dsh[i] : 0.0;
#pragma unroll
        for (int u = 0; u < BNB / 2; ++u) {
            const int c = 2 * u + h, j = J * BNB + c;
            if (j <= i) {
                T v;
                if (i < n && j < n)
                    v = (T)(((mu * di) * a[u]) * dsh[j]);
                else
                    v = (i == j) ? (T)1 : (T)0;
                L[i + (int64_t)j * np] = v;
            }
            tb[c * BNB + (r ^ c)] = a[u];
        }
        __builtin_amdgcn_wave_barrier();
        // Am (row J*32 + c, column I*32 + rr) = a (I*32 + rr, J*32 + c), c = lane % 32, strictly above the diagonal
        double *dst = Am + (int64_t)J * BNB + (int64_t)I * BNB * np;
#pragma unroll
        for (int u = 0; u < BNB / 2; ++u) {
            const int rr = 2 * u + h;
            if (I > J || r < rr)
                dst[r + (int64_t)rr * np] = tb[r * BNB + (rr ^ r)];
        }
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
}

// Factor the 32 x 32 diagonal block at (k0, k0) in one wavefront and form
// its inverse W, left-looking: lane r holds row r; at column j every lane
// forms a_rj - sum_{q<j} L[r][q] L[j][q] with row j of L read from shared
// memory (Lr, row-major, every lane the same address: a broadcast, four
// values per read), lane j's value is the pivot (one readlane), and each lane
// publishes its new L[r][j] to Lr.  W follows by forward substitution
// L W = I, lane c building column c (W[r][c] = (delta_rc -
// sum_{q<r} L[r][q] W[q][c]) / L[r][r]) from the same rows.  Lanes 32..63
// mirror lanes 0..31 and store nothing.  Outputs: the block in L, W in Ws
// (Ws[c * 33 + r]) and Wg (column-major).  Returns the 1-based failing
// column of the block, 0 on success.
inline __device__ __attribute__((noinline)) int b_diag(T *L, int np, int k0, T *Ws, T *Wg, T *Lr)
{
    L = (T *)gmem(L);  // global memory (see gmem)
    Wg = (T *)gmem(Wg);
    constexpr int S = 36;  // Lr row stride (16-byte aligned rows)
    const int lane = threadIdx.x & 63, r = lane & 31;
    const bool store = lane < BNB;
    T row[BNB];
#pragma unroll
    for (int c = 0; c < BNB; ++c)
        row[c] = (c <= r) ? L[(k0 + r) + (int64_t)(k0 + c) * np] : (T)0;
    int bad = 0;
#pragma unroll
    for (int j = 0; j < BNB; ++j) {
        T p[4] = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
        for (int q = 0; q < j; ++q) p[q & 3] = fma(row[q], Lr[j * S + q], p[q & 3]);
        const T sv = row[j] - ((p[0] + p[1]) + (p[2] + p[3]));
        const T piv = rl(sv, j);
        if (!(piv > (T)0)) {
            bad = j + 1;
            break;
        }
        const T ljj = sqrt(piv);
        row[j] = (r == j) ? ljj : ((r > j) ? sv / ljj : (T)0);
        if (store)
            Lr[r * S + j] = row[j];
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_sched_barrier(0);
    }
    if (bad)
        return bad;
    // W: each new row of W goes to Ws as it is formed
    T w[BNB];
#pragma unroll
    for (int i = 0; i < BNB; ++i) {
        T p[4] = {(T)0, (T)0, (T)0, (T)0};
#pragma unroll
        for (int q = 0; q < i; ++q) p[q & 3] = fma(Lr[i * S + q], w[q], p[q & 3]);
        const T rhs = ((r == i) ? (T)1 : (T)0) - ((p[0] + p[1]) + (p[2] + p[3]));
        w[i] = (i < r) ? (T)0 : rhs / Lr[i * S + i];
        if (store)
            Ws[r * (BNB + 1) + i] = w[i];  // lane r = column r of W
        __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_wave_barrier();
    // the block of L and W (column-major) to global memory, column by column
    for (int e = lane; e < BNB * BNB; e += 64) {
        const int rr = e % BNB, cc = e / BNB;
        if (cc <= rr)
            L[(k0 + rr) + (int64_t)(k0 + cc) * np] = Lr[rr * S + cc];
        Wg[e] = Ws[cc * (BNB + 1) + rr];
    }
    return 0;
}

// ---------------------------------------------------------------------------
// Blocked right-looking Cholesky of the np x np lower matrix in L.  Returns
// the 1-based failing column (0 on success); Winv receives the inverses of
// the 32 x 32 diagonal blocks.  The trailing-update operands are rounded to
// the format half (binary32 accumulation).
template <int WAVES>
__device__ __attribute__((noinline)) int b_factor(T *L, int np, T *Winv, int half, SolveSmem &sm)
{
    L = (T *)gmem(L);  // global memory (see gmem)
    Winv = (T *)gmem(Winv);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nb = np / BNB;
    T *Ws = (T *)sm.Lk;  // inverse of the diagonal block: Ws[c * 33 + r] = W[r][c]
    for (int kb = 0; kb < nb; ++kb) {
        const int k0 = kb * BNB;
        if (wave == 0) {
            const int bad = b_diag(L, np, k0, Ws, Winv + (int64_t)kb * BNB * BNB, (T *)sm.ys);
            if (lane == 0)
                sm.info = bad ? k0 + bad : 0;
        }
        __syncthreads();
        if (sm.info)
            return sm.info;
        // panel: L_ik = H_ik W^T for the row blocks below, one 32 x 32 block per
        // wave.  The blocks also go, transposed, to U = L^T in the strict upper
        // triangle of the same array (for the backward substitutions, three or
        // more of them on average), through the wave's 32 x 32 buffer in shared memory
        // (element (c, r) at c * 32 + (r ^ c): both sides conflict-free) so
        // that both global stores are coalesced.  The buffers overlap b_diag's
        // rows, which are no longer needed.
        T *tb = (T *)sm.ys + wave * BNB * BNB;
        for (int I = kb + 1 + wave; I < nb; I += WAVES) {
            Acc32<T> acc;
            acc.zero();
            // D[c][r] = sum_q W[c][q] H[r][q]
            mma_tile(acc, Ws, BNB + 1, L + (int64_t)I * BNB + (int64_t)k0 * np, np, BNB, lane);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int c = Acc32<T>::row(j, lane), r = Acc32<T>::col(j, lane);
                L[((int64_t)I * BNB + r) + (int64_t)(k0 + c) * np] = acc.get(j);
                tb[c * BNB + (r ^ c)] = acc.get(j);
            }
            __builtin_amdgcn_wave_barrier();
            // U (row k0 + c, column I*32 + rr) = L (I*32 + rr, k0 + c), c = lane % 32
            const int cc = lane & 31, h = lane >> 5;
            T *dst = L + k0 + (int64_t)I * BNB * np;
#pragma unroll
            for (int u = 0; u < BNB / 2; ++u) {
                const int rr = 2 * u + h;
                dst[cc + (int64_t)rr * np] = tb[cc * BNB + (rr ^ cc)];
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // trailing update of the lower tiles (I, J), kb < J <= I; a wave's
        // next tile's C values and this tile's operands are loaded before
        // this tile's MFMAs
        const int t = nb - kb - 1, ntile = t * (t + 1) / 2;
        auto tile_of = [&](int q, int &gI, int &gJ) {
            int I = (int)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);
            while (I * (I + 1) / 2 > q) --I;
            while ((I + 1) * (I + 2) / 2 <= q) ++I;
            gI = kb + 1 + I;
            gJ = kb + 1 + q - I * (I + 1) / 2;
        };
        auto load_c = [&](Acc32<T> &acc, const T *C) {
            // register j: column Acc32::row(j) of the tile, row Acc32::col(j)
#pragma unroll
            for (int j = 0; j < 16; ++j)
                acc.set(j, C[Acc32<T>::col(j, lane) + (int64_t)Acc32<T>::row(j, lane) * np]);
        };
        int gI = 0, gJ = 0;
        Acc32<T> nxt;
        if (wave < ntile) {
            tile_of(wave, gI, gJ);
            load_c(nxt, L + (int64_t)gI * BNB + (int64_t)gJ * BNB * np);
        }
        for (int q = wave; q < ntile; q += WAVES) {
            T *C = L + (int64_t)gI * BNB + (int64_t)gJ * BNB * np;
            const T *pJ = L + (int64_t)gJ * BNB + (int64_t)k0 * np;
            const T *pI = L + (int64_t)gI * BNB + (int64_t)k0 * np;
            Acc32<T> acc = nxt;
            Frag fa[BNB / Frag::K], fb[BNB / Frag::K];
#pragma unroll
            for (int s2 = 0; s2 < BNB / Frag::K; ++s2) {
                fa[s2].load(pJ + (int64_t)s2 * Frag::K * np, np, lane);
                fb[s2].load(pI + (int64_t)s2 * Frag::K * np, np, lane);
            }
            if (q + WAVES < ntile) {
                tile_of(q + WAVES, gI, gJ);
                load_c(nxt, L + (int64_t)gI * BNB + (int64_t)gJ * BNB * np);
            }
#pragma unroll
            for (int s2 = 0; s2 < BNB / Frag::K; ++s2) {
                fa[s2].v = round_half(fa[s2].v, half);
                fb[s2].v = round_half(fb[s2].v, half);
                fa[s2].negate();
                mma(acc, fa[s2], fb[s2]);
            }
#pragma unroll
            for (int j = 0; j < 16; ++j)
                C[Acc32<T>::col(j, lane) + (int64_t)Acc32<T>::row(j, lane) * np] = acc.get(j);
        }
        __syncthreads();
    }
    return 0;
}

// ---------------------------------------------------------------------------
// X (+)= s mu D L^{-T} L^{-1} round(D R / s) for m right-hand sides; the
// scales s_c = pow2_ceil(smax[c]) (smax in shared memory).  Every global
// read is coalesced across lanes and issued in batches (no loop carries a
// load-to-use dependency).
template <int WAVES>
__device__ __attribute__((noinline)) void b_solve(const T *L, const T *Winv, int n, int np, int m, const double *R, const double *d, double mu,
                     double *X, int accumulate, SolveSmem &sm)
{
    constexpr int NT = WAVES * 64, MR = SPD_BATCH_MAXRHS;
    const int tid = threadIdx.x;
    const int nb = np / BNB;
    const auto gL = gmem(L), gW = gmem(Winv);
    const auto gR = gmem(R), gd = gmem(d);
    const auto gX = gmem(X);
    T *ys = (T *)sm.ys;  // ys[c * NMAX + i]
    constexpr int NM = SPD_BATCH_NMAX;
    for (int idx = tid; idx < m * np; idx += NT) {
        const int c = idx / np, i = idx % np;
        const double s = pow2_ceil(sm.smax[c]);
        ys[c * NM + i] = (i < n) ? (T)(gd[i] * gR[i + (int64_t)c * n] / s) : (T)0;
    }
    __syncthreads();
    // Each step first issues the loads it needs -- the W block (staged in
    // shared memory, Wl[q * 33 + r] = W[r][q]) and the matrix values of the
    // step -- so that their latencies overlap; sums keep the same order.
    constexpr int WPT = BNB * BNB / NT;  // W values staged per thread
    static_assert(WPT * NT == BNB * BNB, "W staging");
    T *Wl = (T *)sm.Lk;
    T *zs = (T *)sm.ts;  // the block just solved, zs[c * BNB + r]
    // forward: z_k = W_k y_k, then y_below -= L_below,k z_k
    for (int kb = 0; kb < nb; ++kb) {
        const int k0 = kb * BNB;
        const auto W = gW + (int64_t)kb * BNB * BNB;
        T wt[WPT];
#pragma unroll
        for (int u = 0; u < WPT; ++u) wt[u] = W[tid + u * NT];
        const int i1 = k0 + BNB + tid;
        T lv[BNB];
        if (i1 < np) {
#pragma unroll
            for (int q = 0; q < BNB; ++q) lv[q] = gL[i1 + (int64_t)(k0 + q) * np];
        }
#pragma unroll
        for (int u = 0; u < WPT; ++u) {
            const int e = tid + u * NT;
            Wl[(e / BNB) * (BNB + 1) + e % BNB] = wt[u];
        }
        __syncthreads();
        if (tid < BNB * m) {
            const int r = tid % BNB, c = tid / BNB;
            T z = (T)0;
#pragma unroll
            for (int q = 0; q < BNB; ++q) z += Wl[q * (BNB + 1) + r] * ys[c * NM + k0 + q];  // W is zero above its diagonal
            zs[tid] = z;
        }
        __syncthreads();
        if (tid < BNB * m)
            ys[(tid / BNB) * NM + k0 + tid % BNB] = zs[tid];
        if (i1 < np) {
#pragma unroll
            for (int c = 0; c < MR; ++c) {
                if (c < m) {
                    T sacc = (T)0;
#pragma unroll
                    for (int q = 0; q < BNB; ++q) sacc += lv[q] * zs[c * BNB + q];
                    ys[c * NM + i1] -= sacc;
                }
            }
        }
        for (int i = i1 + NT; i < np; i += NT) {
            T lw[BNB];
#pragma unroll
            for (int q = 0; q < BNB; ++q) lw[q] = gL[i + (int64_t)(k0 + q) * np];
#pragma unroll
            for (int c = 0; c < MR; ++c) {
                if (c < m) {
                    T sacc = (T)0;
#pragma unroll
                    for (int q = 0; q < BNB; ++q) sacc += lw[q] * zs[c * BNB + q];
                    ys[c * NM + i] -= sacc;
                }
            }
        }
        __syncthreads();
    }
    // backward, right-looking on U = L^T (held in the strict upper triangle
    // of the same array, written by the factorisation's panel steps):
    // x_k = W_k^T y_k, then
    // y_above -= U_above,k x_k -- the forward sweep's mirror, each row's
    // values of a step one coalesced load per column of the block
    for (int kb = nb - 1; kb >= 0; --kb) {
        const int k0 = kb * BNB;
        const auto W = gW + (int64_t)kb * BNB * BNB;
        T wt[WPT];
#pragma unroll
        for (int u = 0; u < WPT; ++u) wt[u] = W[tid + u * NT];
        const int i1 = tid;  // rows above the block: 0 .. k0 - 1
        T lv[BNB];
        if (i1 < k0) {
#pragma unroll
            for (int q = 0; q < BNB; ++q) lv[q] = gL[i1 + (int64_t)(k0 + q) * np];
        }
#pragma unroll
        for (int u = 0; u < WPT; ++u) {
            const int e = tid + u * NT;
            Wl[(e / BNB) * (BNB + 1) + e % BNB] = wt[u];
        }
        __syncthreads();
        if (tid < BNB * m) {
            const int r = tid % BNB, c = tid / BNB;
            T x = (T)0;
#pragma unroll
            for (int q = 0; q < BNB; ++q) x += Wl[r * (BNB + 1) + q] * ys[c * NM + k0 + q];  // W^T: zero below
            zs[tid] = x;
        }
        __syncthreads();
        if (tid < BNB * m)
            ys[(tid / BNB) * NM + k0 + tid % BNB] = zs[tid];
        if (i1 < k0) {
#pragma unroll
            for (int c = 0; c < MR; ++c) {
                if (c < m) {
                    T sacc = (T)0;
#pragma unroll
                    for (int q = 0; q < BNB; ++q) sacc += lv[q] * zs[c * BNB + q];
                    ys[c * NM + i1] -= sacc;
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        for (int i = i1 + NT; i < k0; i += NT) {
            T lw[BNB];
#pragma unroll
            for (int q = 0; q < BNB; ++q) lw[q] = gL[i + (int64_t)(k0 + q) * np];
#pragma unroll
            for (int c = 0; c < MR; ++c) {
                if (c < m) {
                    T sacc = (T)0;
#pragma unroll
                    for (int q = 0; q < BNB; ++q) sacc += lw[q] * zs[c * BNB + q];
                    ys[c * NM + i] -= sacc;
                }
            }
        }
        __syncthreads();
    }
    if (tid < m)
        sm.zmax[tid] = 0ull;
    __syncthreads();
    for (int idx = tid; idx < m * n; idx += NT) {
        const int c = idx / n, i = idx % n;
        const double s = pow2_ceil(sm.smax[c]);
        const double z = ((s * mu) * gd[i]) * (double)ys[c * NM + i];
        const auto px = gX + i + (int64_t)c * n;
        *px = accumulate ? *px + z : z;
        atomicMax(&sm.zmax[c], (unsigned long long)__double_as_longlong(fabs(z)));
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// R = B - A X (binary64) and the norms: norms[1 + k m + c], k = 0..3:
// max|r|, max|x|, max|b|, max|d r|; with want_anorm also norms[0] =
// ||A||_inf.  X is staged in shared memory.  Rows in passes of 64 (lane =
// row), the columns split among the waves in whole batches of CH: a_ij from
// A for j <= i and from the mirror Am (written by b_convert) for j > i, so
// each load is coalesced (reading the lower triangle alone would need a
// second, column-wise pass whose loads touch a cache line per lane), with the
// next batch in flight.  Each row's four wave partials are added in a fixed
// order, so the result does not depend on timing.  Splitting the columns
// rather than the rows keeps the waves level for every n (rows per wave
// left one wave a second full pass whenever n was just above 256).
// Bound by latency with 512 systems in flight.  4096 systems that all
// converge take 10.2 (FP16) and 13.2 ms (BF16); 11.0 and 14.4 with a choice
// between A and the mirror at every element (most batches lie on one side of
// the diagonal), bounds looked at for every column, and the maxima one kind
// after the other.
template <int WAVES>
__device__ __attribute__((noinline)) void b_residual(const double *A, const double *Am, int n, int np, int m,
                                                     const double *X, const double *B, const double *d, double *R,
                                                     int want_anorm, SolveSmem &sm)
{
    constexpr int NT = WAVES * 64, NM = SPD_BATCH_NMAX;
    static_assert(WAVES == 4, "partial sums are laid out for four waves");
    n = uni(n);
    np = uni(np);
    m = uni(m);
    const auto gA = gmem(uni(A)), gAm = gmem(uni(Am)), gX = gmem(X), gB = gmem(B);
    const auto gR = gmem(R);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int MR = SPD_BATCH_MAXRHS;
    double *xs = sm.ys;  // xs[c * NMAX + j]
    double *abs_rows = sm.arow;
    // (past the last element it is repeated, up to a whole batch: those
    // products are with zeros)
    constexpr int CH = 16;
    const int nx = (n + CH - 1) / CH * CH;
    for (int idx = tid; idx < m * nx; idx += NT) {
        const int c = idx / nx, j = idx % nx;
        xs[c * NM + j] = gX[min(j, n - 1) + c * n];
    }
    __syncthreads();
    const int nch = (n + CH - 1) / CH, cpw = (nch + WAVES - 1) / WAVES;
    const int jlo = wave * cpw * CH, jhi = min(n, (wave + 1) * cpw * CH);
    for (int i0 = 0; i0 < n; i0 += 64) {
        const int i = i0 + lane;
        double acc[MR], aa = 0.0;
#pragma unroll
        for (int c = 0; c < MR; ++c) acc[c] = 0.0;
        double a[CH], an[CH];
        // (rows past the last one repeat it; their sums are dropped)
        const unsigned ic = (unsigned)min(i, n - 1);
        auto load = [&](double *dst, int j0) {
            auto from = [&](auto p, int ld) {
#pragma unroll
                for (int u = 0; u < CH; ++u) dst[u] = p[ic + (unsigned)(min(j0 + u, n - 1) * ld)];
            };
            if (j0 + CH - 1 <= i0)  // every j <= i
                from(gA, n);
            else if (j0 > i0 + 63)  // every j > i
                from(gAm, np);
            else
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    const unsigned j = (unsigned)min(j0 + u, n - 1);
                    dst[u] = (j <= ic) ? gA[ic + j * (unsigned)n] : gAm[ic + j * (unsigned)np];
                }
            if (j0 + CH > jhi)
#pragma unroll
                for (int u = 0; u < CH; ++u) dst[u] = (j0 + u < jhi) ? dst[u] : 0.0;
        };
        if (jlo < jhi)
            load(a, jlo);
        for (int j0 = jlo; j0 < jhi; j0 += CH) {
            if (j0 + CH < jhi)
                load(an, j0 + CH);
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                const int j = j0 + u;
#pragma unroll
                for (int c = 0; c < MR; ++c)
                    if (c < m)
                        acc[c] = fma(a[u], xs[c * NM + j], acc[c]);
                if (want_anorm)
                    aa += fabs(a[u]);
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) a[u] = an[u];
        }
#pragma unroll
        for (int c = 0; c < MR; ++c)
            if (c < m)
                sm.part[wave][c][lane] = acc[c];
        sm.part[wave][MR][lane] = aa;
        __syncthreads();
        for (int idx = tid; idx < (m + 1) * 64; idx += NT) {
            const int c = idx / 64, l = idx % 64, r = i0 + l;
            const int slot = (c < m) ? c : MR;
            if (r < n && (c < m || want_anorm)) {
                const double s = ((sm.part[0][slot][l] + sm.part[1][slot][l]) + sm.part[2][slot][l]) + sm.part[3][slot][l];
                if (c < m)
                    gR[r + (int64_t)c * n] = gB[r + (int64_t)c * n] - s;
                else
                    abs_rows[r] = s;
            }
        }
        __syncthreads();
    }
    // maxima (NaN propagates): a wave takes whole columns, four rows a lane at a time
    for (int c = wave; c < m; c += WAVES) {
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (int q0 = lane; q0 < n; q0 += 4 * 64) {
            double rv[4], bv[4], dv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int q = min(q0 + 64 * k, n - 1);
                rv[k] = gR[q + c * n];
                bv[k] = gB[q + c * n];
                dv[k] = gmem(d)[q];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int q = q0 + 64 * k;
                if (q < n) {
                    v[0] = b_nanmax(v[0], fabs(rv[k]));
                    v[1] = b_nanmax(v[1], fabs(xs[c * NM + q]));
                    v[2] = b_nanmax(v[2], fabs(bv[k]));
                    v[3] = b_nanmax(v[3], fabs(dv[k] * rv[k]));
                }
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v[k] = b_nanmax(v[k], __shfl_xor(v[k], off));
            if (lane == 0)
                sm.norms[1 + k * m + c] = v[k];
        }
    }
    if (want_anorm) {
        double x = 0.0;
        for (int i = tid; i < n; i += NT) x = b_nanmax(x, abs_rows[i]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x = b_nanmax(x, __shfl_xor(x, off));
        if (lane == 0)
            sm.red[wave][0] = x;
        __syncthreads();
        if (tid == 0) {
            double y = 0.0;
            for (int w = 0; w < WAVES; ++w) y = b_nanmax(y, sm.red[w][0]);
            sm.norms[0] = y;
        }
    }
    __syncthreads();
}

}  // namespace half_path
