// Batched solver: many independent SPD systems A_s X_s = B_s (Eq. (2) per
// system) in one persistent launch, each system taken through all of
// Algorithm 1 by one workgroup:
//   equilibrate and round (mu D A D), left-looking blocked Cholesky in the
//   factor's precision (32-wide panels on MFMA; half-precision requests:
//   k_batch_half.h), triangular solves on MFMA with
//   the 32 x 32 diagonal-block inverses, binary64 residual and backward error,
//   correction loop with the same stopping, divergence and fallback rules as
//   the single-system path (BF16/FP16 -> FP32 -> FP64).
// Systems are handed out by an atomic counter in decreasing order of n
// (counting sort on the device), so the largest start first.  Each workgroup
// owns a fixed slice of workspace (factor, inverses, d, residual): a call
// allocates nothing once the workspace exists, and never synchronises the
// host, so it can be captured in a graph.  Only the lower triangle of each
// A_s is read.
#include <spd.h>

#include <type_traits>

#include "common.h"
#include "internal.h"
#include "sym_rows.h"

#define BNB 32  // panel and tile width
#define BDIAG_S 36  // row stride of a diagonal block in shared memory
#define BDIAG_P 4   // row stride of its panels' buffer
// precision picker: 16 features -> 64 -> 64 -> 4 classes (BF16, FP16, FP32, FP64)
#define PICK_NFEAT 16
#define PICK_NH 64
#define PICK_NCLS 4
#define PICK_LANCZOS 4

struct BatchArgs {
    int64_t batch;
    const int32_t *n, *nrhs;
    const int64_t *a_off, *b_off;
    const double *A, *B;
    double *X;
    int32_t *prec;
    spd_report *reps;
    double tol, mu16;
    int max_iter, fallback, equilibrate;
    const int32_t *order;
    int *queue;
    char *ws;
    int64_t ws_stride;
    const float *picker;  // perceptron parameters for SPD_AUTO (NULL: binary32)
    int64_t *ticks;       // optional: wall-clock ticks of each system's solve
};

// workspace slice of one workgroup
struct BatchWs {
    void *L;      // the factor's 32 x 32 tiles below the diagonal (binary32 or binary64), see BTile
    void *Winv;   // the inverses of its diagonal tiles, in the same layout
    double *d;    // equilibration
    double *R;    // n x m residual
    double *Am;   // half-precision requests: A's strict lower triangle mirrored into the strict upper of an np x np array
};

SPD_DEV BatchWs batch_ws(const BatchArgs &a)
{
    char *p = a.ws + (int64_t)blockIdx.x * a.ws_stride;
    BatchWs w;
    w.L = p;
    p += (int64_t)SPD_BATCH_NMAX * SPD_BATCH_NMAX * 8;
    w.Winv = p;
    p += (int64_t)SPD_BATCH_NMAX * BNB * 8;
    w.d = (double *)p;
    p += (int64_t)SPD_BATCH_NMAX * 8;
    w.R = (double *)p;
    p += (int64_t)SPD_BATCH_NMAX * SPD_BATCH_MAXRHS * 8;
    w.Am = (double *)p;
    return w;
}

// Arguments of a function that is not inlined arrive in vector registers; the
// workgroup's own n, pointers and so on as scalars again (addresses are then a
// scalar base plus a 32-bit lane offset)
SPD_DEV int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <typename P>
SPD_DEV P *uni(P *p)
{
    const unsigned long long b = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffull));
    const unsigned hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return (P *)gmem((P *)(((unsigned long long)hi << 32) | lo));
}

SPD_DEV double b_nanmax(double a, double b) { return (a > b || a != a) ? a : b; }

// pitch of a binary64 vector array in shared memory (16 of them read side by
// side without bank conflicts)
#define BPITCH (SPD_BATCH_NMAX + 2)

// a wave's buffer in the symmetric product: a 16 x 16 quarter tile, then its
// sums over a strip's 32 columns for 8 vectors and |A|
#define BSYM_TB ((SPD_BATCH_MAXRHS + 1) * BNB)

// shared state of the workgroup (two workgroups per compute unit: at most 80 KB)
struct SolveSmem {
    double ys[SPD_BATCH_MAXRHS * BPITCH];  // solve vectors (factor type); x of the residual
    double yo[SPD_BATCH_MAXRHS * BPITCH];  // A x of the residual
    double tb[4 * BSYM_TB];                // the symmetric product's buffers; inverse of the diagonal block
    double arow[SPD_BATCH_NMAX];           // row sums of |A|; d of the factorisation
    double red[4][4 * SPD_BATCH_MAXRHS];
    double norms[1 + 4 * SPD_BATCH_MAXRHS];
    double smax[SPD_BATCH_MAXRHS];
    unsigned long long zmax[SPD_BATCH_MAXRHS];  // max |z| per column of the last solve (binary64 bits)
    int info;
};
// the picker's features and perceptron (about 35 KB: several workgroups per CU)
struct PickSmem {
    double d[BPITCH];   // d_i = a_ii^{-1/2}
    double v[SPD_BATCH_NMAX];   // Lanczos vectors v_j, v_{j-1}, w
    double vp[SPD_BATCH_NMAX];
    double w[BPITCH];
    double x[BPITCH];   // D v
    double rs[SPD_BATCH_NMAX];  // Gershgorin radii of H
    double tb[4 * BSYM_TB];
    double red[4][8];
    double ab[2][PICK_LANCZOS];  // Lanczos alpha, beta
    double th[PICK_LANCZOS];     // Ritz values
    float feat[PICK_NFEAT];
    float hid[2][PICK_NH];
    float logit[PICK_NCLS];
};

SPD_DEV float round_half(float v, int half)
{
    return half == HALF_F16 ? (float)(_Float16)v : (float)(__bf16)v;
}

// value of v in lane src (src uniform); binary64 as two 32-bit halves
SPD_DEV float rl(float v, int src) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src)); }
SPD_DEV double rl(double v, int src)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), src);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), src);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

#include "k_batch_half.h"

// ---------------------------------------------------------------------------
// The factor is stored as 32 x 32 tiles, tile (I, J) at 1024 (I (I + 1)/2 + J),
// each in the order in which an MFMA accumulator holds it (transposed:
// Acc32 register j of a lane is column row(j), row col(j) of the tile), four
// registers next to each other: a solved tile is stored straight from its
// accumulator, and loaded with 16-byte loads, contiguous across the wave, as
// the operand of a later product -- the MFMA's k-slots are a free summation
// order, and an accumulator's columns fall on them.
//   binary32: column c, row r at ((c / 4) 32 + r) 4 + c % 4
//   binary64: at ((4 (c / 16) + c % 4) 32 + r) 4 + (c / 4) % 4
template <typename T> struct BTile;
template <> struct BTile<float> {
    using V = floatx4;
    float v[16];  // lane (r = l % 32, h = l / 32): column 8 (j / 4) + 4 h + j % 4 in v[j]
    static SPD_DEV int pos(int r, int c) { return ((c >> 2) * 32 + r) * 4 + (c & 3); }
    SPD_DEV void load(const float *t, int lane)
    {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const V x = *(const V *)(gmem(t) + (unsigned)((2 * g * 32 + lane) * 4));
#pragma unroll
            for (int i = 0; i < 4; ++i) v[4 * g + i] = x[i];
        }
    }
    static SPD_DEV void store(float *t, const Acc32<float> &a, int lane)
    {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(__attribute__((address_space(1))) V *)(gmem(t) + (unsigned)((2 * g * 32 + lane) * 4)) =
                V{a.v[4 * g], a.v[4 * g + 1], a.v[4 * g + 2], a.v[4 * g + 3]};
    }
    SPD_DEV void store(float *t, int lane) const
    {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(__attribute__((address_space(1))) V *)(gmem(t) + (unsigned)((2 * g * 32 + lane) * 4)) =
                V{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
    }
    // acc += (this as rows of D) (b as columns of D)^T, this negated
    static SPD_DEV void submul(Acc32<float> &acc, const BTile &a, const BTile &b)
    {
#pragma unroll
        for (int j = 0; j < 16; ++j) acc.mma(-a.v[j], b.v[j]);
    }
};
template <> struct BTile<double> {
    typedef double V __attribute__((ext_vector_type(2)));
    double v[2][2][4];  // lane (r = l % 16, u = l / 16): row 16 b + r, column 16 a + 4 q + u in v[b][a][q]
    static SPD_DEV int pos(int r, int c) { return ((4 * (c >> 4) + (c & 3)) * 32 + r) * 4 + ((c >> 2) & 3); }
    // columns 16 a .. 16 a + 15
    static SPD_DEV void load_half(double (&x)[2][4], const double *t, int a, int lane)
    {
        const int r = lane & 15, u = lane >> 4;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const V p = *(const V *)(gmem(t) + (unsigned)(((4 * a + u) * 32 + 16 * b + r) * 4 + q));
                x[b][q] = p[0];
                x[b][q + 1] = p[1];
            }
    }
    SPD_DEV void load(const double *t, int lane)
    {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
            double x[2][4];
            load_half(x, t, a, lane);
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) v[b][a][q] = x[b][q];
        }
    }
    static SPD_DEV void store(double *t, const Acc32<double> &acc, int lane)
    {
        const int r = lane & 15, u = lane >> 4;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; q += 2)
                    *(__attribute__((address_space(1))) V *)(gmem(t) + (unsigned)(((4 * a + u) * 32 + 16 * b + r) * 4 + q)) =
                        V{acc.v[a][b][q], acc.v[a][b][q + 1]};
    }
    SPD_DEV void store(double *t, int lane) const
    {
        const int r = lane & 15, u = lane >> 4;
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int q = 0; q < 4; q += 2)
                    *(__attribute__((address_space(1))) V *)(gmem(t) + (unsigned)(((4 * a + u) * 32 + 16 * b + r) * 4 + q)) =
                        V{v[b][a][q], v[b][a][q + 1]};
    }
    // acc += (the half tile x as rows of D) (the half tile y as columns of D)^T, x negated
    static SPD_DEV void submul_half(Acc32<double> &acc, const double (&x)[2][4], const double (&y)[2][4])
    {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const double fx[2] = {-x[0][q], -x[1][q]}, fy[2] = {y[0][q], y[1][q]};
            acc.mma(fx, fy);
        }
    }
};
template <typename T>
SPD_DEV T *b_tile(T *L, int I, int J)
{
    return L + (int64_t)(I * (I + 1) / 2 + J) * (BNB * BNB);
}

// Factor a 32 x 32 diagonal block, given row-major in Lr (its lower triangle),
// in one wavefront and form its inverse W: column operations that take A to L
// take the identity below it to L^{-T}, so lane l < 32 works on row l of
// [A; I] and lane 32 + c on the identity's row c, column c of W, with the same
// instructions.  Panels of 4 columns: a lane has its 4 elements in registers
// (pivot and multipliers by readlane); the columns to the right take the
// panel's product on MFMA, kept in 16 x 16 accumulators (transposed: a
// register's row is a column of [A; I]) from where the next panel's columns
// go to the lanes through buf.  Output: W in Ws (Ws[c * 33 + r]); nothing
// reads the block of L itself again.  Returns the 1-based failing column of
// the block, 0 on success.
// A serial chain, on the path of the whole factorisation: 8.4 blocks per
// system.  32 column steps with row j read back from shared memory, and a
// 32-deep substitution, took 16 us (binary32) and 20 us (binary64) a block;
// 16 columns in registers at a time, unrolled (29 KB of code, which took
// longer to fetch than to run), 11 and 16; this took 8.6 and 11.4 with the
// products straight off A's values.
// A panel's products are summed by themselves and come off what is left of A's
// values once (and in b_factor eight columns' off the diagonal tile):
// products taken off the values one by one each round at the values' size, and
// one sum over all of them rounds at the size of A where little is left of it.
// First solve, binary64, error / u for n = 33..64 and 65..128 at cond 10: 4.8
// and 5.7 one by one, 3.5 and 3.9 with one sum, 3.7 and 4.1 this way; error /
// (u cond) at cond 1e6: 0.133 and 0.095, 0.140 and 0.107, 0.131 and 0.092.
// 4096 mixed systems take 3.87 ms (binary64) and 4.64 (binary32), one by one
// 3.97 and 4.71.
template <typename T>
SPD_DEV int b_diag_body(T *Ws, T *Lr, T *buf)
{
    constexpr int S = BDIAG_S;  // Lr row stride (16-byte aligned rows)
    constexpr int H = BNB / 2;
    constexpr int P = BDIAG_P;  // row stride of the panel's buffer
    const int lane = threadIdx.x & 63, r16 = lane & 15, u = lane >> 4;
    auto mma = [](T a, T b, auto c) {
        if constexpr (sizeof(T) == 4)
            return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    };
    using acc_t = typename std::conditional<sizeof(T) == 4, floatx4, doublex4>::type;
    // row of accumulator register q
    auto arow = [&](int q) { return sizeof(T) == 4 ? 4 * u + q : 4 * q + u; };
    // columns 16 c .. 16 c + 15: of A's rows (ta: block rows 0 and 1 of column
    // 0, block row 1 of column 1) and of the identity's (ti: block row 0 of
    // columns 0 and 1, block row 1 of column 1; zero where products come off)
    const acc_t zero = {0, 0, 0, 0};
    acc_t ta[3], ti[3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        ta[0][q] = Lr[r16 * S + arow(q)];
        ta[1][q] = Lr[(H + r16) * S + arow(q)];
        ta[2][q] = Lr[(H + r16) * S + H + arow(q)];
        ti[0][q] = ti[2][q] = (r16 == arow(q)) ? (T)1 : (T)0;
        ti[1][q] = (T)0;
    }
    // the 4 columns of accumulator t from 4 pc into rows r0 .. r0 + 15 of the buffer
    auto put = [&](const acc_t &t, int pc, int r0) {
        if constexpr (sizeof(T) == 4) {
            if (u == pc)
                *(floatx4 *)&buf[(r0 + r16) * P] = t;
        } else {
            buf[(r0 + r16) * P + u] = pc < 2 ? (pc == 0 ? t[0] : t[1]) : (pc == 2 ? t[2] : t[3]);
        }
    };
    int bad = 0;
#pragma unroll 1
    for (int p = 0; p < BNB / 4; ++p) {
        const int c0 = 4 * p, pc = p & 3;
        if (p < 4) {
            put(ta[0], pc, 0);
            put(ta[1], pc, H);
            put(ti[0], pc, 2 * H);
        } else {
            put(ta[2], pc, H);
            put(ti[1], pc, 2 * H);
            put(ti[2], pc, 3 * H);
        }
        __builtin_amdgcn_wave_barrier();
        T v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (p < 4 && lane >= 3 * H) ? (T)0 : buf[lane * P + j];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const T piv = rl(v[j], c0 + j);
            bad = (bad == 0 && !(piv > (T)0)) ? c0 + j + 1 : bad;
            const T ljj = sqrt(piv);
            const T q = v[j] / ljj;  // by every lane: no branch around the division
            const T l = (lane == c0 + j) ? ljj : ((lane > c0 + j) ? q : (T)0);
            v[j] = l;
#pragma unroll
            for (int k = j + 1; k < 4; ++k) v[k] = fma(-l, rl(l, c0 + k), v[k]);
        }
        if (bad)
            return bad;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 4; ++j) buf[lane * P + j] = v[j];
        if (lane >= BNB)
#pragma unroll
            for (int j = 0; j < 4; ++j) Ws[(lane - BNB) * (BNB + 1) + c0 + j] = v[j];
        __builtin_amdgcn_wave_barrier();
        T o[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) o[t] = buf[(H * t + r16) * P + u];
        if (p < 4) {
            ta[0] -= mma(o[0], o[0], zero);
            ta[1] -= mma(o[0], o[1], zero);
            ti[0] = mma(-o[0], o[2], ti[0]);
        } else {
            ti[2] = mma(-o[1], o[3], ti[2]);
        }
        ta[2] -= mma(o[1], o[1], zero);
        ti[1] = mma(-o[1], o[2], ti[1]);
        __builtin_amdgcn_wave_barrier();
    }
    return 0;
}

// (inlined, binary64's registers would spill in the products)
__device__ __attribute__((noinline)) int b_diag(double *Ws, double *Lr, double *buf)
{
    return b_diag_body<double>(Ws, Lr, buf);
}
SPD_DEV int b_diag(float *Ws, float *Lr, float *buf) { return b_diag_body<float>(Ws, Lr, buf); }

// ---------------------------------------------------------------------------
// Left-looking blocked Cholesky of H = round(mu D A D) (identity padding up
// to np = 32 nb): panel kb's tiles (I, kb) are formed
// from A in the waves' accumulators (d_i = a_ii^{-1/2} also goes to d), take
// the products of the earlier panels, the diagonal one is factored by wave 0,
// and the others become L_Ik = H_Ik W^T, W the diagonal tile's inverse, and
// are stored once.  Returns the 1-based failing column (0 on success).
//
// Bound by memory traffic, with 512 systems in flight.  Right-looking, with H
// written out by a conversion and every trailing tile read and written once
// per panel, 4096 systems of the batched distribution moved 40 GB in binary32
// and 31 GB in binary64, at 4.3 TB/s, a factorisation of 394 and 600 us (mean
// over the systems).  With the residual's mirror of A gone as well (b_sym),
// 20 and 17 GB, 194 and 330 us.
template <typename T, int WAVES, int KERN>
__device__ __attribute__((noinline)) int b_factor(const double *A, int n, int np, double *d, double mu, int equil,
                                                  T *L, T *Winv, SolveSmem &sm)
{
    const auto gA = gmem(uni(A));
    const auto gd = gmem(uni(d));
    L = uni(L);
    Winv = uni(Winv);
    n = uni(n);
    np = uni(np);
    equil = uni(equil);
    constexpr int NT = WAVES * 64;
    static_assert(BNB * (BNB + 1) * 8 <= (int)sizeof(sm.tb), "inverse of the diagonal block");
    static_assert((BNB * BDIAG_S + 2 * BNB * BDIAG_P) * 8 <= (int)sizeof(sm.yo), "diagonal block");
    using A32 = Acc32<T>;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = np / BNB;
    T *Ws = (T *)sm.tb;  // inverse of the diagonal block: Ws[c * 33 + r] = W[r][c]
    T *Lr = (T *)sm.yo;  // the diagonal block, row-major
    double *dsh = sm.arow;
    for (int i = tid; i < n; i += NT) {
        const double a = gA[i + (int64_t)i * n];
        const double di = (equil && a > 0.0) ? 1.0 / sqrt(a) : 1.0;
        gd[i] = di;
        dsh[i] = di;
    }
    __syncthreads();
    // H's tile (I, kb) in the accumulator's layout (register j: column
    // row(j), row col(j)): A's values, past the matrix and above the diagonal
    // the nearest element below it, dropped
    auto init = [&](A32 &acc, int I, int kb) {
        // (the lane number anew for each tile: what follows from it would
        // otherwise be kept in registers across the whole loop)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        double a[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int i = min(I * BNB + A32::col(j, ln), n - 1), c = min(kb * BNB + A32::row(j, ln), i);
            a[j] = gA[(unsigned)(i + c * n)];
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int i = I * BNB + A32::col(j, ln), k = kb * BNB + A32::row(j, ln);
            T v = (T)(((mu * dsh[min(i, n - 1)]) * a[j]) * dsh[min(k, n - 1)]);
            if (i >= n || k >= n)
                v = (i == k) ? (T)1 : (T)0;
            acc.set(j, v);
        }
    };
    // acc[s] -= L_Iq L_kb,q^T for q < kb and I = I0 + step s < nb, s < NS; the
    // next tile (binary64: half a tile, the accumulators take half of the
    // registers) is in flight
    auto products = [&](auto ns, A32 *acc, int I0, int step, int kb) {
        constexpr int NS = decltype(ns)::value;
        if (kb == 0)
            return;
        if constexpr (sizeof(T) == 4) {
            BTile<T> fk, fi, fkn, nx;
            fk.load(b_tile(L, kb, 0), lane);
            fi.load(b_tile(L, I0, 0), lane);
            for (int q = 0; q < kb; ++q) {
                const int qn = min(q + 1, kb - 1);
                fkn.load(b_tile(L, kb, qn), lane);
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const int I = I0 + step * s;
                    if (I >= nb)
                        break;
                    const bool last = s + 1 == NS || I + step >= nb;
                    nx.load(last ? b_tile(L, I0, qn) : b_tile(L, I + step, q), lane);
                    BTile<T>::submul(acc[s], fk, fi);
                    fi = nx;
                }
                fk = fkn;
            }
        } else {
            double k0[2][4], k1[2][4], x0[2][4], x1[2][4];
            BTile<T>::load_half(k0, b_tile(L, kb, 0), 0, lane);
            BTile<T>::load_half(x0, b_tile(L, I0, 0), 0, lane);
            BTile<T>::load_half(k1, b_tile(L, kb, 0), 1, lane);
            for (int q = 0; q < kb; ++q) {
                const int qn = min(q + 1, kb - 1);
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const int I = I0 + step * s;
                    if (I >= nb)
                        break;
                    const bool last = s + 1 == NS || I + step >= nb;
                    BTile<T>::load_half(x1, b_tile(L, I, q), 1, lane);
                    __builtin_amdgcn_sched_barrier(0);
                    BTile<T>::submul_half(acc[s], k0, x0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (last)
                        BTile<T>::load_half(k0, b_tile(L, kb, qn), 0, lane);
                    BTile<T>::load_half(x0, last ? b_tile(L, I0, qn) : b_tile(L, I + step, q), 0, lane);
                    __builtin_amdgcn_sched_barrier(0);
                    BTile<T>::submul_half(acc[s], k1, x1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (last)
                        BTile<T>::load_half(k1, b_tile(L, kb, qn), 1, lane);
                }
            }
        }
    };
    // the same for the diagonal tile, both operands the same tile, the products
    // of 8 columns summed by themselves in t
    auto products_diag = [&](A32 &acc, A32 &t, int kb) {
        if (kb == 0)
            return;
        BTile<T> f, nx;
        f.load(b_tile(L, kb, 0), lane);
        for (int q = 0; q < kb; ++q) {
            nx.load(b_tile(L, kb, min(q + 1, kb - 1)), lane);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < BNB; c += 8) {
                t.zero();
                if constexpr (sizeof(T) == 4) {
#pragma unroll
                    for (int j = c / 2; j < (c + 8) / 2; ++j) t.mma(-f.v[j], f.v[j]);
                } else {
#pragma unroll
                    for (int p = c / 4; p < (c + 8) / 4; ++p) {
                        const double fx[2] = {-f.v[0][p >> 2][p & 3], -f.v[1][p >> 2][p & 3]},
                                     fy[2] = {f.v[0][p >> 2][p & 3], f.v[1][p >> 2][p & 3]};
                        t.mma(fx, fy);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < 16; ++j) acc.set(j, acc.get(j) + t.get(j));
            }
            f = nx;
        }
    };
    // L_Ik = H_Ik W^T: D[c][r] = sum_q W[c][q] H[r][q], H the accumulator itself
    auto solve = [&](const BTile<T> &w, const A32 &h, int I, int kb) {
        A32 y;
        y.zero();
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int j = 0; j < 16; ++j) y.mma(w.v[j], h.v[j]);
        } else {
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const double fw[2] = {w.v[0][a][q], w.v[1][a][q]}, fh[2] = {h.v[a][0][q], h.v[a][1][q]};
                    y.mma(fw, fh);
                }
        }
        BTile<T>::store(b_tile(L, I, kb), y, lane);
    };
    constexpr int OW = WAVES - 1, SLOTS = 4;
    for (int kb = 0; kb < nb; ++kb) {
        // wave 0 has the diagonal tile alone, whose factor takes as long as
        // the other waves' tiles I = kb + wave + OW s
        const int I0 = kb + wave;
        A32 acc[SLOTS];
        if (wave == 0) {
            init(acc[1], kb, kb);  // (in other slots' registers: in acc[0] the loops spill)
            products_diag(acc[1], acc[2], kb);
#pragma unroll
            for (int j = 0; j < 16; ++j) Lr[A32::col(j, lane) * BDIAG_S + A32::row(j, lane)] = acc[1].get(j);
            __builtin_amdgcn_wave_barrier();
            const int bad = b_diag(Ws, Lr, Lr + BNB * BDIAG_S);
            if (lane == 0)
                sm.info = bad ? kb * BNB + bad : 0;
        } else if (I0 < nb) {
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (I0 + OW * s < nb)
                    init(acc[s], I0 + OW * s, kb);
            products(std::integral_constant<int, SLOTS>(), acc, I0, OW, kb);
        }
        __syncthreads();
        if (sm.info)
            return sm.info;
        BTile<T> w;
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int j = 0; j < 16; ++j) w.v[j] = Ws[A32::row(j, lane) * (BNB + 1) + (lane & 31)];
        } else {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        w.v[b][a][q] = Ws[(16 * a + 4 * q + (lane >> 4)) * (BNB + 1) + 16 * b + (lane & 15)];
        }
        if (wave == 0)
            w.store(Winv + (int64_t)kb * BNB * BNB, lane);
        else
#pragma unroll
            for (int s = 0; s < SLOTS; ++s)
                if (I0 + OW * s < nb)
                    solve(w, acc[s], I0 + OW * s, kb);
        // the tiles past the slots (n > 416)
        static_assert(SPD_BATCH_NMAX / BNB <= 1 + OW * SLOTS + WAVES, "a tile per wave is left at most");
        if (const int I = kb + 1 + OW * SLOTS + wave; I < nb) {
            init(acc[0], I, kb);
            products(std::integral_constant<int, 1>(), acc, I, 1, kb);
            solve(w, acc[0], I, kb);
        }
        __syncthreads();
    }
    return 0;
}

// ---------------------------------------------------------------------------
// X (+)= s mu D L^{-T} L^{-1} round(D R / s) for m right-hand sides; the
// scales s_c = pow2_ceil(smax[c]) (smax in shared memory).
//
// Both sweeps are right-looking over the factor's tiles on MFMA (16 x 16 x 4,
// the right-hand sides as the 16 columns): z_k = W_k y_k, then y_I -= L_Ik z_k
// for the tiles below, wave w taking I = k + 1 + w, ... -- wave 0, which has
// the next diagonal tile's rows first, goes on to z_{k+1} at once, so a step
// costs one barrier.  The backward sweep is the mirror on the transposed
// tiles.  ys[c * YS + i] holds right-hand side c (YS: pitch without bank
// conflicts between the 16 columns).  On the VALU, with the vectors read from
// shared memory for every product, a binary32 solve took 62 us (mean n = 270),
// a binary64 one 218 us; here 42 and 75 us.
template <typename T> struct BVec;
template <> struct BVec<float> {
    using acc = floatx4;
    static constexpr int YS = SPD_BATCH_NMAX + 4;
    static SPD_DEV floatx4 mma(float a, float b, floatx4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
    // k index of slot u at step s (0..7): the columns of a tile as 16-byte runs
    static SPD_DEV int k(int s, int u) { return 16 * (s >> 2) + 4 * u + (s & 3); }
    static SPD_DEV int row(int q, int u) { return 4 * u + q; }  // accumulator register q
};
template <> struct BVec<double> {
    using acc = doublex4;
    static constexpr int YS = SPD_BATCH_NMAX + 2;
    static SPD_DEV doublex4 mma(double a, double b, doublex4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
    static SPD_DEV int k(int s, int u) { return 4 * s + u; }
    static SPD_DEV int row(int q, int u) { return 4 * q + u; }
};
// a tile as the left operand of tile times vectors (t[h][s]: row 16 h + r,
// column k(s, u)), or of its transpose (column 16 h + r, row 4 s + u)
template <typename T, bool TR>
struct BOp {
    T v[2][8];
    SPD_DEV void load(const T *t, int lane)
    {
        const int r = lane & 15, u = lane >> 4;
        const auto g = gmem(t);
        using V = typename BTile<T>::V;
        constexpr int VN = 16 / sizeof(T);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (TR) {
#pragma unroll
                for (int s = 0; s < 8; ++s) v[h][s] = g[(unsigned)BTile<T>::pos(4 * s + u, 16 * h + r)];
            } else {
                // k(s, u), s = 4 j .. 4 j + 3, are next to each other
#pragma unroll
                for (int s = 0; s < 8; s += VN) {
                    const V x = *(const __attribute__((address_space(1))) V *)(g + (unsigned)BTile<T>::pos(16 * h + r, BVec<T>::k(s, u)));
#pragma unroll
                    for (int i = 0; i < VN; ++i) v[h][s + i] = x[i];
                }
            }
        }
    }
};

template <typename T, int WAVES, int KERN>
__device__ __attribute__((noinline)) void b_solve(const T *L, const T *Winv, int n, int np, int m, const double *R, const double *d, double mu,
                     double *X, int accumulate, SolveSmem &sm)
{
    constexpr int YS = BVec<T>::YS;
    using acc_t = typename BVec<T>::acc;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, u = lane >> 4;
    L = uni(L);
    Winv = uni(Winv);
    n = uni(n);
    np = uni(np);
    m = uni(m);
    accumulate = uni(accumulate);
    const int nb = np / BNB;
    const auto gR = gmem(uni(R)), gd = gmem(uni(d));
    const auto gX = gmem(uni(X));
    T *ys = (T *)sm.ys;
    static_assert(SPD_BATCH_MAXRHS * YS * sizeof(T) <= sizeof(sm.ys), "solve vectors");
    // a wave takes whole columns here and at the end, four rows a lane at a
    // time (256): their loads are in flight together, and a column's maximum
    // needs no other wave
    for (int c = wave; c < m; c += WAVES) {
        const double s = pow2_ceil(sm.smax[c]);
        for (int i0 = lane; i0 < np; i0 += 4 * 64) {
            double dv[4], rv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = min(i0 + 64 * k, n - 1);
                dv[k] = gd[i];
                rv[k] = gR[i + c * n];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i0 + 64 * k < np)
                    ys[c * YS + i0 + 64 * k] = (i0 + 64 * k < n) ? (T)(dv[k] * rv[k] / s) : (T)0;
        }
    }
    __syncthreads();
    // the lane's right-hand side (lanes past the last one repeat the first;
    // their products are dropped)
    const bool live = r < m;
    T *yc = ys + (live ? r : 0) * YS;
    // block k's vectors as the right operand, and D's rows back
    auto take = [&](T (&z)[8], int k, bool tr) {
#pragma unroll
        for (int s = 0; s < 8; ++s) z[s] = yc[k * BNB + (tr ? 4 * s + u : BVec<T>::k(s, u))];
    };
    auto sweep = [&](auto trc) {
        constexpr bool TR = decltype(trc)::value;
        using Op = BOp<T, TR>;
        auto product = [&](const Op &a, const T (&z)[8], acc_t (&o)[2]) {
#pragma unroll
            for (int h = 0; h < 2; ++h) o[h] = acc_t{0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 8; ++s)
#pragma unroll
                for (int h = 0; h < 2; ++h) o[h] = BVec<T>::mma(a.v[h][s], z[s], o[h]);
        };
        // steps t = 0 .. nb - 1 on block blk(t); wave w's tiles at step t are
        // blocks blk(t + 1 + w), blk(t + 1 + w + WAVES), ...
        auto blk = [&](int t) { return TR ? nb - 1 - t : t; };
        auto tile = [&](int t, int o) { return TR ? b_tile(L, blk(t), blk(o)) : b_tile(L, blk(o), blk(t)); };
        auto diag = [&](const Op &w, int t) {  // wave 0: z_k = W_k y_k in place
            T z[8];
            take(z, blk(t), TR);
            acc_t o[2];
            product(w, z, o);
            if (live)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int q = 0; q < 4; ++q) yc[blk(t) * BNB + 16 * h + BVec<T>::row(q, u)] = o[h][q];
        };
        // wave 0: the next step's W, loaded a step ahead
        auto winv = [&](int t) { return Winv + (int64_t)blk(t) * BNB * BNB; };
        Op cur, w;
        if (wave == 0)
            w.load(winv(0), lane);
        if (1 + wave < nb)
            cur.load(tile(0, 1 + wave), lane);
        if (wave == 0) {
            diag(w, 0);
            if (nb > 1)
                w.load(winv(1), lane);
        }
        __syncthreads();
        for (int t = 0; t + 1 < nb; ++t) {
            T z[8];
            take(z, blk(t), TR);
            for (int o = t + 1 + wave; o < nb; o += WAVES) {
                Op nx;
                const bool more = o + WAVES < nb;
                if (more)
                    nx.load(tile(t, o + WAVES), lane);
                acc_t p[2];
                product(cur, z, p);
                if (live)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int q = 0; q < 4; ++q) yc[blk(o) * BNB + 16 * h + BVec<T>::row(q, u)] -= p[h][q];
                if (wave == 0 && o == t + 1) {
                    __builtin_amdgcn_wave_barrier();
                    diag(w, t + 1);
                    if (t + 2 < nb)
                        w.load(winv(t + 2), lane);
                }
                if (more)
                    cur = nx;
            }
            if (t + 2 + wave < nb)
                cur.load(tile(t + 1, t + 2 + wave), lane);
            __syncthreads();
        }
    };
    sweep(std::false_type());
    sweep(std::true_type());
    for (int c = wave; c < m; c += WAVES) {
        const double sc = pow2_ceil(sm.smax[c]) * mu;
        unsigned long long zm = 0ull;  // of |z|'s bits: NaN above all
        for (int i0 = lane; i0 < n; i0 += 4 * 64) {
            double dv[4], xv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = min(i0 + 64 * k, n - 1);
                dv[k] = gd[i];
                xv[k] = accumulate ? gX[i + c * n] : 0.0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = i0 + 64 * k;
                if (i < n) {
                    const double z = (sc * dv[k]) * (double)ys[c * YS + i];
                    gX[i + c * n] = accumulate ? xv[k] + z : z;
                    zm = max(zm, (unsigned long long)__double_as_longlong(fabs(z)));
                }
            }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) zm = max(zm, __shfl_xor(zm, off));
        if (lane == 0)
            sm.zmax[c] = zm;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// y = A x (binary64) for m <= 4 G vectors in shared memory (pitch BPITCH) and
// the symmetric A given by its lower triangle, in one pass over that triangle
// on v_mfma_f64_4x4x4f64 (four products side by side: 4 vectors times 16
// columns; 16x16x4 would spend a quarter or half of its rows on them).
// 32-column strips J, wave w takes the 32 x 32 blocks I = J + w, J + w + 4,
// ...: a lane (j = l % 16, u = l / 16) holds columns 16 h + j, rows
// 8 s + 2 u + e, loaded 16 bytes at a time with the next block in flight.  As
// they are, these are the operands of the columns' sums (sum_i a_ij x_i, kept
// in the accumulators over the strip); transposed by 16 x 16 quarters through
// the wave's buffer they are those of the rows' (added to y in shared memory:
// a row block has one wave at a time).  After the strip the waves' column sums
// are added in order, so nothing depends on timing.  A diagonal block is its
// lower half with the diagonal halved: the same code as any other.
// With WA also ya_i = sum_j |a_ij| xa_j (xa NULL: ones; excl: j = i left out),
// with HS the largest |h_ij| off the diagonal and the sum of h_ij^2 of
// H = D A D, per thread.
//
// Bound by reading the triangle with 512 (the picker: 768) systems in flight.
// The residual used to read whole rows, the upper half from a mirror that the
// factorisation wrote (557 us for a binary32 system's 3.5 passes); the
// picker's products read the triangle once by rows and once by columns, a
// cache line per lane (3.7 ms for 4096 systems).  One pass with 16x16x4 and
// diagonal blocks loaded as full symmetric ones, each of whose 16 loads fell
// on 64 cache lines, took 377 us; now 195 us.
SPD_DEV int bsym_pos(int r, int c)  // element (r, c) of a quarter tile: written and read without bank conflicts
{
    const int rr = (r & ~3) | ((r & 1) << 1) | ((r >> 1) & 1);
    return rr * 16 + (c ^ (((r & 1) << 2) | ((r & 4) << 1)));
}
template <int WAVES, int G, bool WA, bool HS>
SPD_DEV void b_sym(const double *A, int n, int m, const double *x, double *y, double *tbs, const double *xa,
                   double *ya, bool excl, const double *d, double &hmax, double &fro)
{
    typedef double double2u __attribute__((ext_vector_type(2), aligned(8)));  // 16-byte load, 8-byte aligned
    constexpr int NT = WAVES * 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j16 = lane & 15, u = lane >> 4;
    const int nb = (n + BNB - 1) / BNB;
    const auto gA = gmem(A);
    double *tb = tbs + wave * BSYM_TB;
    const double *xc[G];  // group g: vectors 4 g .. 4 g + 3; past the last one the first again, dropped
#pragma unroll
    for (int g = 0; g < G; ++g) xc[g] = x + (4 * g + (j16 & 3) < m ? 4 * g + (j16 & 3) : 0) * BPITCH;
    for (int idx = tid; idx < m * BPITCH; idx += NT) y[idx] = 0.0;
    if constexpr (WA)
        for (int i = tid; i < n; i += NT) ya[i] = 0.0;
    // a[h][t]: row 32 I + 8 (t / 2) + 2 u + t % 2, column 32 J + 16 h + j16,
    // 16 bytes at a time (sym_rows.h: what is not in the matrix's lower
    // triangle is loaded from there all the same, and dropped by trim)
    auto load = [&](double (&a)[2][8], int I, int J) {
        int cj[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) cj[h] = min(J * BNB + 16 * h + j16, n - 1);
        if (J == nb - 1) {  // the end of the diagonal
#pragma unroll
            for (int t = 0; t < 8; ++t)
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    a[h][t] = gA[(unsigned)(cj[h] * n + sym_row(I * BNB + 8 * (t >> 1) + 2 * u + (t & 1), cj[h], n))];
            return;
        }
#pragma unroll
        for (int t = 0; t < 8; t += 2)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = sym_first(I * BNB + 4 * t + 2 * u, cj[h], n, I == J);
                const double2u v = *(const __attribute__((address_space(1))) double2u *)(gA + (unsigned)(cj[h] * n + i));
                a[h][t] = v.x;
                a[h][t + 1] = v.y;
            }
    };
    // a block at the end of the matrix or on the diagonal: rows past the last
    // one and what is above the diagonal to zero, the diagonal halved (it is
    // in the rows' sums and in the columns')
    auto trim = [&](double (&a)[2][8], int I, int J) {
        const bool end = J == nb - 1;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int t = 0; t < 8; t += 2) {
                const int i = I * BNB + 4 * t + 2 * u, j = J * BNB + 16 * h + j16;
                const double v0 = a[h][t], v1 = a[h][t + 1];
                a[h][t] = sym_even(v0, v1, i, j, n, end);
                a[h][t + 1] = sym_odd(v0, v1, i, j, n, I == J, end);
            }
    };
    double a[2][8], an[2][8];
    if (wave < nb)
        load(a, wave, 0);
    __syncthreads();
    for (int J = 0; J < nb; ++J) {
        double accc[2][G] = {};
        double cs[2] = {0.0, 0.0};
        double xj[G][2][4], xaj[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int j = J * BNB + 16 * h + 4 * s + u;
#pragma unroll
                for (int g = 0; g < G; ++g) xj[g][h][s] = xc[g][j];
                if constexpr (WA)
                    xaj[h][s] = xa ? xa[j] : 1.0;
            }
        for (int I = J + wave; I < nb; I += WAVES) {
            // the wave's next block: in this strip, or its first of the next
            const bool same = I + WAVES < nb;
            const int In = same ? I + WAVES : J + 1 + wave, Jn = same ? J : J + 1;
            if (In < nb)
                load(an, In, Jn);
            __builtin_amdgcn_sched_barrier(0);
            if (I == J || I * BNB + BNB > n)
                trim(a, I, J);
            double xi[G][8];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int t = 0; t < 8; t += 2) {
                    const double2 v = *(const double2 *)(xc[g] + I * BNB + 4 * t + 2 * u);
                    xi[g][t] = v.x;
                    xi[g][t + 1] = v.y;
                }
            double accr[2][G] = {};
            double rs[2] = {0.0, 0.0};
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int t = 0; t < 4; ++t) tb[bsym_pos(8 * (t >> 1) + 2 * u + (t & 1), j16)] = a[h][4 * b + t];
                    __builtin_amdgcn_wave_barrier();
                    double at[4];
#pragma unroll
                    for (int s = 0; s < 4; ++s) at[s] = tb[bsym_pos(j16, 4 * s + u)];
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int g = 0; g < G; ++g)
                            accc[h][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(xi[g][4 * b + t], a[h][4 * b + t], accc[h][g], 0, 0, 0);
#pragma unroll
                    for (int s = 0; s < 4; ++s)
#pragma unroll
                        for (int g = 0; g < G; ++g)
                            accr[b][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(xj[g][h][s], at[s], accr[b][g], 0, 0, 0);
                    if constexpr (WA) {
#pragma unroll
                        for (int s = 0; s < 4; ++s) {
                            const bool drop = excl && I == J && b == h && j16 == 4 * s + u;
                            rs[b] += drop ? 0.0 : fabs(at[s]) * xaj[h][s];
                        }
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int il = 16 * b + 8 * (t >> 1) + 2 * u + (t & 1);
                            const bool drop = excl && I == J && il == 16 * h + j16;
                            cs[h] += drop ? 0.0 : fabs(a[h][4 * b + t]) * (xa ? xa[I * BNB + il] : 1.0);
                        }
                    }
                    if constexpr (HS) {
                        const double dj = d[J * BNB + 16 * h + j16];
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            const int il = 16 * b + 8 * (t >> 1) + 2 * u + (t & 1);
                            const double hv = (d[I * BNB + il] * a[h][4 * b + t]) * dj;
                            const bool dg = I == J && il == 16 * h + j16;  // halved
                            hmax = dg ? hmax : fmax(hmax, fabs(hv));
                            fro += (dg ? 4.0 : 2.0) * hv * hv;
                        }
                    }
                }
            // accumulator of group g: vector 4 g + u, row 16 b + j16
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (4 * g + u < m)
#pragma unroll
                    for (int b = 0; b < 2; ++b) y[(4 * g + u) * BPITCH + I * BNB + 16 * b + j16] += accr[b][g];
            if constexpr (WA)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    double v = rs[b];
                    v += __shfl_xor(v, 16);
                    v += __shfl_xor(v, 32);
                    if (u == 0 && I * BNB + 16 * b + j16 < n)
                        ya[I * BNB + 16 * b + j16] += v;
                }
            if (In < nb)
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int t = 0; t < 8; ++t) a[h][t] = an[h][t];
        }
        // the strip's column sums: the waves' in order
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int g = 0; g < G; ++g)
                if (4 * g + u < m)
                    tb[(4 * g + u) * BNB + 16 * h + j16] = accc[h][g];
            if constexpr (WA) {
                double v = cs[h];
                v += __shfl_xor(v, 16);
                v += __shfl_xor(v, 32);
                if (u == 0)
                    tb[m * BNB + 16 * h + j16] = v;
            }
        }
        __syncthreads();
        for (int idx = tid; idx < (WA ? m + 1 : m) * BNB; idx += NT) {
            const int c = idx / BNB, j = J * BNB + idx % BNB;
            static_assert(WAVES == 4, "partial sums are laid out for four waves");
            const double v = ((tbs[idx] + tbs[BSYM_TB + idx]) + tbs[2 * BSYM_TB + idx]) + tbs[3 * BSYM_TB + idx];
            if (!WA || c < m)
                y[c * BPITCH + j] += v;
            else if (j < n)
                ya[j] += v;
        }
        __syncthreads();
    }
}

// R = B - A X (binary64) and the norms: norms[1 + k m + c], k = 0..3:
// max|r|, max|x|, max|b|, max|d r|; with want_anorm also norms[0] =
// ||A||_inf.
template <int WAVES, int KERN>
__device__ __attribute__((noinline)) void b_residual(const double *A, int n, int m, const double *X, const double *B,
                                                     const double *d, double *R, int want_anorm, SolveSmem &sm)
{
    constexpr int NT = WAVES * 64;
    n = uni(n);
    m = uni(m);
    want_anorm = uni(want_anorm);
    A = uni(A);
    const auto gX = gmem(uni(X)), gB = gmem(uni(B)), gd = gmem(uni(d));
    const auto gR = gmem(uni(R));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    double *xs = sm.ys;
    const int np = (n + BNB - 1) / BNB * BNB;
    // a wave takes whole columns (as in b_solve), four rows a lane at a time
    for (int c = wave; c < m; c += WAVES)
        for (int i0 = lane; i0 < np; i0 += 4 * 64) {
            double xv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) xv[k] = gX[min(i0 + 64 * k, n - 1) + c * n];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i0 + 64 * k < np)
                    xs[c * BPITCH + i0 + 64 * k] = (i0 + 64 * k < n) ? xv[k] : 0.0;
        }
    double h0 = 0.0, h1 = 0.0;
    const auto ax = [&](auto groups) {
        constexpr int G = decltype(groups)::value;
        if (want_anorm)
            b_sym<WAVES, G, true, false>(A, n, m, xs, sm.yo, sm.tb, nullptr, sm.arow, false, nullptr, h0, h1);
        else
            b_sym<WAVES, G, false, false>(A, n, m, xs, sm.yo, sm.tb, nullptr, nullptr, false, nullptr, h0, h1);
    };
    if (m <= 4)
        ax(std::integral_constant<int, 1>());
    else
        ax(std::integral_constant<int, 2>());
    // r and the maxima (NaN propagates), per column
    for (int c = wave; c < m; c += WAVES) {
        double v[4] = {0.0, 0.0, 0.0, 0.0};
        for (int i0 = lane; i0 < n; i0 += 4 * 64) {
            double bv[4], dv[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = min(i0 + 64 * k, n - 1);
                bv[k] = gB[i + c * n];
                dv[k] = gd[i];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = i0 + 64 * k;
                if (i < n) {
                    const double r = bv[k] - sm.yo[c * BPITCH + i];
                    gR[i + c * n] = r;
                    v[0] = b_nanmax(v[0], fabs(r));
                    v[1] = b_nanmax(v[1], fabs(xs[c * BPITCH + i]));
                    v[2] = b_nanmax(v[2], fabs(bv[k]));
                    v[3] = b_nanmax(v[3], fabs(dv[k] * r));
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
        __syncthreads();
        double x = 0.0;
        for (int i = tid; i < n; i += NT) x = b_nanmax(x, sm.arow[i]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) x = b_nanmax(x, __shfl_xor(x, off));
        if (lane == 0)
            sm.red[wave][0] = x;
        __syncthreads();
        if (tid == 0) {
            double z = 0.0;
            for (int w = 0; w < WAVES; ++w) z = b_nanmax(z, sm.red[w][0]);
            sm.norms[0] = z;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Precision picker (a project addition around Algorithm 1: which precision to
// run it in).  Features of one system, in binary64, by the workgroup:
// d_i = a_ii^{-1/2} (1 where a_ii <= 0), H = D A D, r_i = sum_{j != i} |h_ij|;
// four Lanczos steps on H from (1, ..., 1)/sqrt(n) without
// reorthogonalisation (stopping early when beta <= 1e-12 max(|alpha|, 1));
// theta = eigenvalues of the tridiagonal (bisection on Sturm counts).
//   f0 log2(n)/9, f1 m/8, f2..f4 spread/mean/std of log10 a_ii (/6, /6, /3),
//   f5 log10(1 + max r)/3, f6 log10(1 + mean r)/3, f7 share of rows r < 1,
//   f8 clip(1 - max r, -10, 1)/10, f9 log10 theta_max/3,
//   f10 log10 max(theta_min, 1e-16)/6, f11 log10(theta_max/max(theta_min, 1e-16))/6,
//   f12 max off-diagonal |h_ij|, f13 log10(||H||_F/sqrt(n))/3,
//   f14 last beta/theta_max (0 after an early stop),
//   f15 (theta_2 - theta_1)/(theta_max - theta_1) (0 with fewer than 3 values).

// block reduction of NV values per thread, fixed order (wave butterflies,
// then waves in order); op 0 = sum, 1 = max, 2 = min.  Result in every thread.
template <int WAVES, int NV>
SPD_DEV void b_reduce(double v[NV], const int op[NV], PickSmem &sm)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const double o = __shfl_xor(v[k], off);
            v[k] = op[k] == 0 ? v[k] + o : op[k] == 1 ? fmax(v[k], o) : fmin(v[k], o);
        }
        if (lane == 0)
            sm.red[wave][k] = v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        double x = sm.red[0][k];
        for (int w = 1; w < WAVES; ++w) {
            const double o = sm.red[w][k];
            x = op[k] == 0 ? x + o : op[k] == 1 ? fmax(x, o) : fmin(x, o);
        }
        v[k] = x;
    }
    __syncthreads();
}

// y = H v (v, y in shared memory), H = D A D from the lower triangle of A.
// With first: rs[i] = r_i, and per thread the partial max off-diagonal |h|
// and sum of h^2.
template <int WAVES>
SPD_DEV void b_hv(const double *A, int n, const double *v, double *y, bool first, double &hmax, double &fro,
                  PickSmem &sm)
{
    constexpr int NT = WAVES * 64;
    const int tid = threadIdx.x;
    const int np = (n + BNB - 1) / BNB * BNB;
    for (int i = tid; i < np; i += NT) sm.x[i] = (i < n) ? sm.d[i] * v[i] : 0.0;
    if (first)
        b_sym<WAVES, 1, true, true>(A, n, 1, sm.x, y, sm.tb, sm.d, sm.rs, true, sm.d, hmax, fro);
    else
        b_sym<WAVES, 1, false, false>(A, n, 1, sm.x, y, sm.tb, nullptr, nullptr, false, nullptr, hmax, fro);
    for (int i = tid; i < n; i += NT) {
        y[i] *= sm.d[i];
        if (first)
            sm.rs[i] *= sm.d[i];
    }
    __syncthreads();
}

// eigenvalues (ascending) of the k x k symmetric tridiagonal (al, be), k <= 4
SPD_DEV int sturm_below(const double *al, const double *be, int k, double x)
{
    int c = 0;
    double q = al[0] - x;
    if (q < 0)
        ++c;
    for (int i = 1; i < k; ++i) {
        if (q == 0.0)
            q = 1e-300;
        q = (al[i] - x) - be[i - 1] * be[i - 1] / q;
        if (q < 0)
            ++c;
    }
    return c;
}

// Ritz value q (0-based, ascending) of the k x k tridiagonal (al, be) by
// multisection in one wavefront: each step evaluates the Sturm count at 64
// interior points of [lo, hi] and keeps the subinterval where the count
// passes q, until no representable point lies strictly inside.  Every lane
// returns the same value.
SPD_DEV double ritz_multisect(const double *al, const double *be, int k, int q, double lo, double hi)
{
    const int lane = threadIdx.x & 63;
    for (int it = 0; it < 64; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (mid <= lo || mid >= hi)
            break;
        const double x = lo + (hi - lo) * ((double)(lane + 1) / 65.0);
        const bool above = (x > lo && x < hi) ? sturm_below(al, be, k, x) > q : false;
        const unsigned long long mk = __ballot(above);
        // x_l is increasing in l; the count is non-decreasing in x
        const int first = mk ? __builtin_ctzll(mk) : 64;
        const double xlo = __shfl(x, first > 0 ? first - 1 : 0), xhi = __shfl(x, first < 64 ? first : 63);
        const double nlo = (first > 0) ? fmax(lo, xlo) : lo;
        const double nhi = (first < 64) ? fmin(hi, xhi) : hi;
        if (nlo == lo && nhi == hi)
            break;  // the grid collapsed onto the ends: no interior point left
        lo = nlo;
        hi = nhi;
    }
    return 0.5 * (lo + hi);
}

template <int WAVES>
SPD_DEV void b_features(const double *A, int n, int m, PickSmem &sm)
{
    constexpr int NT = WAVES * 64, K = PICK_LANCZOS;
    const int tid = threadIdx.x;
    double *d = sm.d, *v = sm.v, *vp = sm.vp, *w = sm.w;
    // diagonal statistics
    double st[3] = {0.0, -1e300, 1e300};  // sum, max, min of log10|a_ii|
    const int ops3[3] = {0, 1, 2};
    for (int i = tid; i < n; i += NT) {
        const double a = A[i + (int64_t)i * n];
        d[i] = (a > 0.0) ? 1.0 / sqrt(a) : 1.0;
        const double la = log10(fmax(fabs(a), 1e-300));
        st[0] += la;
        st[1] = fmax(st[1], la);
        st[2] = fmin(st[2], la);
        v[i] = 1.0 / sqrt((double)n);
        vp[i] = 0.0;
    }
    for (int i = n + tid; i < (n + BNB - 1) / BNB * BNB; i += NT) d[i] = 0.0;
    b_reduce<WAVES, 3>(st, ops3, sm);
    const double mean_la = st[0] / n;
    double sq[1] = {0.0};
    const int ops1[1] = {0};
    for (int i = tid; i < n; i += NT) {
        const double la = log10(fmax(fabs(A[i + (int64_t)i * n]), 1e-300)) - mean_la;
        sq[0] += la * la;
    }
    b_reduce<WAVES, 1>(sq, ops1, sm);
    // Lanczos; the first product also yields the Gershgorin radii and |H| stats
    double al[K], be[K];
    int k = 0;
    bool early = false;
    double hmax = 0.0, fro = 0.0;
    double bprev = 0.0;
    for (int j = 0; j < K; ++j) {
        b_hv<WAVES>(A, n, v, w, j == 0, hmax, fro, sm);
        double a1[1] = {0.0};
        for (int i = tid; i < n; i += NT) a1[0] += w[i] * v[i];
        b_reduce<WAVES, 1>(a1, ops1, sm);
        const double alpha = a1[0];
        double b2[1] = {0.0};
        for (int i = tid; i < n; i += NT) {
            const double x = (w[i] - alpha * v[i]) - bprev * vp[i];
            w[i] = x;
            b2[0] += x * x;
        }
        b_reduce<WAVES, 1>(b2, ops1, sm);
        const double beta = sqrt(b2[0]);
        al[j] = alpha;
        k = j + 1;
        if (j == K - 1) {
            be[j] = beta;
            break;
        }
        if (beta <= 1e-12 * fmax(fabs(alpha), 1.0)) {
            be[j] = 0.0;
            early = true;
            break;
        }
        be[j] = beta;
        for (int i = tid; i < n; i += NT) {
            vp[i] = v[i];
            v[i] = w[i] / beta;
        }
        bprev = beta;
        __syncthreads();
    }
    // Gershgorin statistics of H and the |H| statistics (first product)
    double gs[5] = {-1e300, 0.0, 0.0, hmax, fro};  // max r, sum r, count r < 1, max |h|, ||H||_F^2
    const int ops5[5] = {1, 0, 0, 1, 0};
    for (int i = tid; i < n; i += NT) {
        gs[0] = fmax(gs[0], sm.rs[i]);
        gs[1] += sm.rs[i];
        gs[2] += (sm.rs[i] < 1.0) ? 1.0 : 0.0;
    }
    b_reduce<WAVES, 5>(gs, ops5, sm);
    // Ritz values: wave q finds the q-th (al, be and k are the same in every thread)
    const int wave = tid >> 6;
    double lo = al[0], hi = al[0];
    for (int i = 0; i < k; ++i) {
        const double r = (i > 0 ? fabs(be[i - 1]) : 0.0) + (i + 1 < k ? fabs(be[i]) : 0.0);
        lo = fmin(lo, al[i] - r);
        hi = fmax(hi, al[i] + r);
    }
    for (int q = wave; q < k; q += WAVES) {
        const double t = ritz_multisect(al, be, k, q, lo, hi);
        if ((tid & 63) == 0)
            sm.th[q] = t;
    }
    __syncthreads();
    if (tid == 0) {
        double th[K];
        for (int q = 0; q < k; ++q) th[q] = sm.th[q];
        const double tmin = th[0], tmax = th[k - 1];
        double f[PICK_NFEAT];
        f[0] = log2((double)n) / 9.0;
        f[1] = m / 8.0;
        f[2] = (st[1] - st[2]) / 6.0;
        f[3] = mean_la / 6.0;
        f[4] = sqrt(sq[0] / n) / 3.0;
        f[5] = log10(1.0 + gs[0]) / 3.0;
        f[6] = log10(1.0 + gs[1] / n) / 3.0;
        f[7] = gs[2] / n;
        f[8] = fmin(fmax(1.0 - gs[0], -10.0), 1.0) / 10.0;
        f[9] = log10(tmax) / 3.0;
        f[10] = log10(fmax(tmin, 1e-16)) / 6.0;
        f[11] = log10(tmax / fmax(tmin, 1e-16)) / 6.0;
        f[12] = (n > 1) ? gs[3] : 0.0;
        f[13] = log10(sqrt(gs[4]) / sqrt((double)n)) / 3.0;
        f[14] = early ? 0.0 : be[k - 1] / tmax;
        f[15] = (k >= 3 && tmax > th[0]) ? (th[1] - th[0]) / (tmax - th[0]) : 0.0;
        for (int q = 0; q < PICK_NFEAT; ++q) sm.feat[q] = (float)f[q];
    }
    __syncthreads();
}

// the perceptron on sm.feat: class with the largest logit (the first on ties)
SPD_DEV int b_pick(const float *P, PickSmem &sm)
{
    const float *W1 = P, *b1 = W1 + PICK_NH * PICK_NFEAT, *W2 = b1 + PICK_NH, *b2 = W2 + PICK_NH * PICK_NH,
                *W3 = b2 + PICK_NH, *b3 = W3 + PICK_NCLS * PICK_NH;
    const int t = threadIdx.x;
    if (t < PICK_NH) {
        float z = b1[t];
        for (int k = 0; k < PICK_NFEAT; ++k) z += W1[t * PICK_NFEAT + k] * sm.feat[k];
        sm.hid[0][t] = fmaxf(z, 0.0f);
    }
    __syncthreads();
    if (t < PICK_NH) {
        float z = b2[t];
        for (int k = 0; k < PICK_NH; ++k) z += W2[t * PICK_NH + k] * sm.hid[0][k];
        sm.hid[1][t] = fmaxf(z, 0.0f);
    }
    __syncthreads();
    if (t < PICK_NCLS) {
        float z = b3[t];
        for (int k = 0; k < PICK_NH; ++k) z += W3[t * PICK_NH + k] * sm.hid[1][k];
        sm.logit[t] = z;
    }
    __syncthreads();
    int best = 0;
    for (int c = 1; c < PICK_NCLS; ++c)
        if (sm.logit[c] > sm.logit[best])
            best = c;
    __syncthreads();
    return best;
}


// Refinement at the precision of the current factor (T), from the iterate in
// X (the first solve); the single-system path's stopping rule: a column is
// done once eta <= tol and its last correction z_k (zeta_k = ||z_k|| /
// ||x_{k+1}||, rho_k = zeta_k / zeta_{k-1}, eta_k the backward error it was
// solved from) shows x accurate to binary64 level -- eta = 0 or
// zeta_k <= 2^-53; rho_k < 1/2 and rho_k/(1-rho_k) eta_k <= 2^-53; or
// rho_k >= 1/2 and eta_k <= 2^-51.  A binary64 factor's first solve is
// accepted at eta <= tol.  Divergence as before; max_iter corrections
// without success: no convergence.  Returns SPD_OK or SPD_ERR_NO_CONVERGENCE
// and fills the iteration counts and eta.
// residual(first, sm) and solve(sm) as in b_residual and b_solve, by the caller
// (the shared memory as an argument: captured, its address would no longer be
// known in the functions that they call).
template <typename T, typename Smem, typename Res, typename Sol>
SPD_DEV int b_refine(double tol, int max_iter, int m, spd_report &rep, Smem &sm, Res residual, Sol solve)
{
    constexpr double U = 0x1p-53, FLOOR = 0x1p-51;
    constexpr bool STABLE = sizeof(T) == 8;
    rep.iters_low = 1;
    rep.iters_high = 0;
    constexpr int MR = SPD_BATCH_MAXRHS;
    double eta0 = 0.0, anorm = 0.0;
    // identical in every thread
    double eta[MR], eprev[MR], zeta[MR], zprev[MR];
    bool done[MR];
#pragma unroll
    for (int c = 0; c < MR; ++c) {
        zeta[c] = zprev[c] = 1.0;
        eprev[c] = 0.0;
        done[c] = false;
    }
    int stalls = 0;
    for (;;) {
        const int first = (rep.iters_high == 0);
        const int k = rep.iters_high;  // corrections applied so far
        residual(first, sm);
        rep.iters_high++;
        if (first)
            anorm = sm.norms[0];
        bool finite = isfinite(anorm), all = true;
        double worst = 0.0;
#pragma unroll
        for (int c = 0; c < MR; ++c) {
            if (c >= m)
                break;
            const double rn = sm.norms[1 + c], xn = sm.norms[1 + m + c], bn = sm.norms[1 + 2 * m + c];
            const double den = anorm * xn + bn;
            double v = (den > 0.0) ? rn / den : (rn > 0.0 ? __builtin_inf() : 0.0);
            if (!(rn == rn) || !(xn == xn))
                v = __builtin_nan("");
            eta[c] = v;
            if (!isfinite(v))
                finite = false;
            if (v > worst)
                worst = v;
            if (k > 0) {
                const double zn = __longlong_as_double((long long)sm.zmax[c]);
                zeta[c] = (zn == 0.0) ? 0.0 : zn / xn;
            }
            if (!done[c] && v <= tol) {
                if (v == 0.0 || zeta[c] <= U) {
                    done[c] = true;
                } else if (k == 0) {
                    done[c] = STABLE;
                } else {
                    const double rho = zeta[c] / zprev[c];
                    done[c] = (rho < 0.5) ? (rho / (1.0 - rho)) * eprev[c] <= U : eprev[c] <= FLOOR;
                }
            }
            all = all && done[c];
        }
        rep.eta = finite ? worst : __builtin_nan("");
        if (!finite)
            return SPD_ERR_NO_CONVERGENCE;
        if (all && worst <= tol)
            return SPD_OK;
        if (k == 0) {
            eta0 = worst;
        } else {
            bool all_slow = true;
#pragma unroll
            for (int c = 0; c < MR; ++c)
                if (c < m && !(eta[c] > 0.9 * eprev[c]))
                    all_slow = false;
            stalls = all_slow ? stalls + 1 : 0;
            if (worst > tol && (worst > eta0 || stalls >= 2))
                return SPD_ERR_NO_CONVERGENCE;
        }
        if (rep.iters_low > max_iter)
            return SPD_ERR_NO_CONVERGENCE;
#pragma unroll
        for (int c = 0; c < MR; ++c) {
            eprev[c] = eta[c];
            zprev[c] = zeta[c];
        }
        __syncthreads();
        if (threadIdx.x < m)
            sm.smax[threadIdx.x] = sm.norms[1 + 3 * m + threadIdx.x];
        __syncthreads();
        solve(sm);
        rep.iters_low++;
    }
}

// smax[c] = max_i |d_i B[i][c]| (the first solve's scaling)
template <int WAVES, typename Smem>
SPD_DEV void b_rhs_max(const double *B, const double *d, int n, int m, Smem &sm)
{
    double v[SPD_BATCH_MAXRHS];
#pragma unroll
    for (int c = 0; c < SPD_BATCH_MAXRHS; ++c) v[c] = 0.0;
    for (int i = threadIdx.x; i < n; i += WAVES * 64)
#pragma unroll
        for (int c = 0; c < SPD_BATCH_MAXRHS; ++c)
            if (c < m)
                v[c] = b_nanmax(v[c], fabs(d[i] * B[i + (int64_t)c * n]));
#pragma unroll
    for (int c = 0; c < SPD_BATCH_MAXRHS; ++c) {
        for (int off = 32; off > 0; off >>= 1) v[c] = b_nanmax(v[c], __shfl_xor(v[c], off));
        if ((threadIdx.x & 63) == 0)
            sm.red[threadIdx.x >> 6][c] = v[c];
    }
    __syncthreads();
    if (threadIdx.x < m) {
        double x = 0.0;
        for (int q = 0; q < WAVES; ++q) x = b_nanmax(x, sm.red[q][threadIdx.x]);
        sm.smax[threadIdx.x] = x;
    }
    __syncthreads();
}

// One system through Algorithm 1 by one workgroup, at the precisions of the
// kernel's factor type: HI = false takes FP32 requests (and, from the
// half-precision kernel, those that fall back), HI = true the FP64 requests
// and every system handed over (a breakdown or non-convergence in binary32
// with fallback on: prec[s] = the next precision, reps[s].fallbacks the count
// so far).  Systems of the other kernels are skipped; the binary32 kernel also
// reports empty systems and invalid sizes.  ticks[s] and reps[s].fallbacks
// (zeroed by the order kernel) accumulate over the kernels.  KERN: the
// functions that are not inlined once more for the half-precision kernel (1);
// shared with it they are slower in the other (4096 binary32 systems: 4.76 ms
// apart, 4.87 shared).
template <int WAVES, bool HI, int KERN>
SPD_DEV void b_system(const BatchArgs &a, int64_t s, SolveSmem &sm)
{
    using T = typename std::conditional<HI, double, float>::type;
    const int n = a.n[s], m = a.nrhs[s];
    int p = a.prec[s];
    if (p == SPD_AUTO)
        p = SPD_FP32;
    const bool valid = n >= 0 && m >= 0 && n <= SPD_BATCH_NMAX && m <= SPD_BATCH_MAXRHS && p >= SPD_BF16 &&
                       p <= SPD_FP64;
    const bool half = valid && p < SPD_FP32 && n > 0 && m > 0;
    if (HI ? (!valid || p != SPD_FP64) : (half || (valid && p == SPD_FP64)))
        return;  // another kernel's system
    if (!HI && KERN == 0 && valid && a.reps[s].fallbacks)
        return;  // a half-precision request that has been through binary32
    const unsigned long long t0 = wall_clock64();
    spd_report rep;
    rep.status = SPD_OK;
    rep.prec_used = p;
    rep.iters_low = rep.iters_high = 0;
    rep.fallbacks = a.reps[s].fallbacks;
    rep.info = 0;
    rep.eta = 0.0;
    bool handover = false;
    if (!valid) {
        rep.status = SPD_ERR_INVALID_ARG;
    } else if (n > 0 && m > 0) {
        const double *A = a.A + a.a_off[s];
        const double *B = a.B + a.b_off[s];
        double *X = a.X + a.b_off[s];
        const int np = ((n + BNB - 1) / BNB) * BNB;
        const BatchWs w = batch_ws(a);
        // a binary32 factor is equilibrated, a binary64 one that of A itself
        T *L = (T *)w.L, *Winv = (T *)w.Winv;
        rep.prec_used = p;
        const int info = b_factor<T, WAVES, KERN>(A, n, np, w.d, 1.0, HI ? 0 : a.equilibrate, L, Winv, sm);
        rep.info = info;
        int r = SPD_ERR_NOT_SPD;
        if (!info) {
            // first solve from B, then refinement
            b_rhs_max<WAVES>(B, w.d, n, m, sm);
            b_solve<T, WAVES, KERN>(L, Winv, n, np, m, B, w.d, 1.0, X, 0, sm);
            r = b_refine<T>(
                a.tol, a.max_iter, m, rep, sm,
                [&](int first, SolveSmem &h) { b_residual<WAVES, KERN>(A, n, m, X, B, w.d, w.R, first, h); },
                [&](SolveSmem &h) { b_solve<T, WAVES, KERN>(L, Winv, n, np, m, w.R, w.d, 1.0, X, 1, h); });
        }
        rep.status = r;
        if (r != SPD_OK && a.fallback && !HI) {  // binary32 goes to the binary64 kernel
            rep.fallbacks++;
            handover = true;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (handover) {
            a.reps[s].fallbacks = rep.fallbacks;
            a.prec[s] = SPD_FP64;
        } else {
            a.reps[s] = rep;
            a.prec[s] = rep.prec_used;
        }
        if (a.ticks)
            a.ticks[s] += (int64_t)(wall_clock64() - t0);
    }
}

// A half-precision request's attempt (k_batch_half.h): reported where it
// converged or may not fall back, else it is a binary32 request from here on
// (prec[s] = FP32, reps[s].fallbacks = 1).  Returns whether it is.
template <int WAVES>
SPD_DEV bool b_half_system(const BatchArgs &a, int64_t s, half_path::SolveSmem &sm)
{
    const int n = a.n[s], m = a.nrhs[s], p = a.prec[s];
    if (n <= 0 || m <= 0 || n > SPD_BATCH_NMAX || m > SPD_BATCH_MAXRHS || p < SPD_BF16 || p >= SPD_FP32)
        return false;
    const unsigned long long t0 = wall_clock64();
    spd_report rep;
    rep.prec_used = p;
    rep.iters_low = rep.iters_high = 0;
    rep.fallbacks = 0;
    rep.eta = 0.0;
    const double *A = a.A + a.a_off[s];
    const double *B = a.B + a.b_off[s];
    double *X = a.X + a.b_off[s];
    const int np = ((n + BNB - 1) / BNB) * BNB;
    const BatchWs w = batch_ws(a);
    float *L = (float *)w.L, *Winv = (float *)w.Winv;
    const double mu = (p == SPD_FP16) ? a.mu16 : 1.0;
    half_path::b_convert<WAVES>(A, n, np, w.d, mu, a.equilibrate, L, w.Am, sm);
    const int info = half_path::b_factor<WAVES>(L, np, Winv, p == SPD_FP16 ? HALF_F16 : HALF_BF16, sm);
    rep.info = info;
    int r = SPD_ERR_NOT_SPD;
    if (!info) {
        b_rhs_max<WAVES>(B, w.d, n, m, sm);
        half_path::b_solve<WAVES>(L, Winv, n, np, m, B, w.d, mu, X, 0, sm);
        r = b_refine<float>(
            a.tol, a.max_iter, m, rep, sm,
            [&](int first, half_path::SolveSmem &h) {
                half_path::b_residual<WAVES>(A, w.Am, n, np, m, X, B, w.d, w.R, first, h);
            },
            [&](half_path::SolveSmem &h) { half_path::b_solve<WAVES>(L, Winv, n, np, m, w.R, w.d, mu, X, 1, h); });
    }
    rep.status = r;
    const bool back = r != SPD_OK && a.fallback;
    __syncthreads();
    if (threadIdx.x == 0) {
        if (!back) {
            a.reps[s] = rep;
        } else {
            a.reps[s].fallbacks = 1;
            a.prec[s] = SPD_FP32;
        }
        if (a.ticks)
            a.ticks[s] += (int64_t)(wall_clock64() - t0);
    }
    __syncthreads();
    return back;
}

// The precision picker for SPD_AUTO systems: features and perceptron by one
// workgroup per system; prec[s] becomes the chosen class.
__global__ __launch_bounds__(256, 2) void k_batch_pick(BatchArgs a)
{
    __shared__ PickSmem sm;
    __shared__ int s_q;
    for (;;) {
        if (threadIdx.x == 0)
            s_q = atomicAdd(a.queue + 0, 1);
        __syncthreads();
        const int64_t q = s_q;
        if (q >= a.batch)
            return;
        const int64_t s = a.order[q];
        const int n = a.n[s], m = a.nrhs[s];
        if (a.prec[s] == SPD_AUTO && n > 0 && m > 0 && n <= SPD_BATCH_NMAX && m <= SPD_BATCH_MAXRHS) {
            const unsigned long long t0 = wall_clock64();
            b_features<4>(a.A + a.a_off[s], n, m, sm);
            const int p = b_pick(a.picker, sm);
            if (threadIdx.x == 0) {
                a.prec[s] = p;
                if (p < SPD_FP32)
                    a.queue[3] = 1;
                if (a.ticks)
                    a.ticks[s] += (int64_t)(wall_clock64() - t0);
            }
        }
        __syncthreads();
    }
}

template <int WAVES, bool HI>
__global__ __launch_bounds__(WAVES * 64, 2) void k_batch(BatchArgs a)
{
    __shared__ SolveSmem sm;
    __shared__ int s_q;
    for (;;) {
        if (threadIdx.x == 0)
            s_q = atomicAdd(a.queue + (HI ? 2 : 1), 1);
        __syncthreads();
        const int64_t q = s_q;
        if (q >= a.batch)
            return;
        b_system<WAVES, HI, 0>(a, a.order[q], sm);
        __syncthreads();
    }
}

// The half-precision requests; nothing where there are none (queue[3], set by
// the order kernel or the picker).  One that falls back goes on in binary32 at
// once: left to the binary32 kernel, it would wait for the slowest attempt of
// the batch (8 FP16 requests of which one falls back: 2.90 ms, and 2.22 so; 600
// of which 267 do: 6.86 and 6.56).  The binary32 kernel, which runs after this
// one, tells it by its count of fallbacks.
template <int WAVES>
__global__ __launch_bounds__(WAVES * 64, 2) void k_batch_half(BatchArgs a)
{
    __shared__ union {
        half_path::SolveSmem half;
        SolveSmem low;
    } sm;
    __shared__ int s_q;
    if (a.queue[3] == 0)
        return;
    for (;;) {
        if (threadIdx.x == 0)
            s_q = atomicAdd(a.queue + 4, 1);
        __syncthreads();
        const int64_t q = s_q;
        if (q >= a.batch)
            return;
        if (b_half_system<WAVES>(a, a.order[q], sm.half))
            b_system<WAVES, false, 1>(a, a.order[q], sm.low);
        __syncthreads();
    }
}

// Features of every system (one workgroup each), for training the picker.
__global__ __launch_bounds__(256, 2) void k_features(int64_t batch, const int32_t *__restrict__ n,
                                                  const int32_t *__restrict__ nrhs, const int64_t *__restrict__ a_off,
                                                  const double *__restrict__ A, float *__restrict__ feat)
{
    __shared__ PickSmem sm;
    for (int64_t s = blockIdx.x; s < batch; s += gridDim.x) {
        const int ns = n[s], ms = nrhs[s];
        if (ns >= 1 && ns <= SPD_BATCH_NMAX) {
            b_features<4>(A + a_off[s], ns, ms, sm);
            if (threadIdx.x < PICK_NFEAT)
                feat[s * PICK_NFEAT + threadIdx.x] = sm.feat[threadIdx.x];
        } else if (threadIdx.x < PICK_NFEAT) {
            feat[s * PICK_NFEAT + threadIdx.x] = 0.0f;
        }
        __syncthreads();
    }
}

// Order of work: systems sorted by decreasing n (counting sort, one
// workgroup); also clears the work-queue counters and the counts that add up
// over the kernels, and notes whether there are half-precision requests.
__global__ __launch_bounds__(1024) void k_batch_order(int64_t batch, const int32_t *__restrict__ n,
                                                      const int32_t *__restrict__ prec, spd_report *reps,
                                                      int32_t *__restrict__ order, int *queue, int64_t *ticks)
{
    constexpr int NBIN = SPD_BATCH_NMAX + 1;
    __shared__ int hist[NBIN], start[NBIN], half;
    const int tid = threadIdx.x;
    for (int b = tid; b < NBIN; b += 1024) hist[b] = 0;
    if (tid == 0)
        half = 0;
    __syncthreads();
    for (int64_t s = tid; s < batch; s += 1024) {
        reps[s].fallbacks = 0;
        if (prec[s] >= SPD_BF16 && prec[s] < SPD_FP32)
            half = 1;  // (by several threads, the same value)
    }
    for (int64_t s = tid; s < batch; s += 1024) {
        int v = n[s];
        v = (v < 0 || v > SPD_BATCH_NMAX) ? 0 : v;
        atomicAdd(&hist[SPD_BATCH_NMAX - v], 1);
    }
    __syncthreads();
    if (tid == 0) {
        int acc = 0;
        for (int b = 0; b < NBIN; ++b) {
            start[b] = acc;
            acc += hist[b];
        }
        queue[0] = queue[1] = queue[2] = queue[4] = 0;
        queue[3] = half;
    }
    if (ticks)
        for (int64_t s = tid; s < batch; s += 1024) ticks[s] = 0;
    __syncthreads();
    for (int64_t s = tid; s < batch; s += 1024) {
        int v = n[s];
        v = (v < 0 || v > SPD_BATCH_NMAX) ? 0 : v;
        const int pos = atomicAdd(&start[SPD_BATCH_NMAX - v], 1);
        order[pos] = (int32_t)s;
    }
}

namespace spd {

int64_t batch_ws_stride()
{
    int64_t b = (int64_t)SPD_BATCH_NMAX * SPD_BATCH_NMAX * 8 + (int64_t)SPD_BATCH_NMAX * BNB * 8 +
                (int64_t)SPD_BATCH_NMAX * 8 + (int64_t)SPD_BATCH_NMAX * SPD_BATCH_MAXRHS * 8 +
                (int64_t)SPD_BATCH_NMAX * SPD_BATCH_NMAX * 8;
    return (b + 255) / 256 * 256;
}

hipError_t launch_batch(const BatchLaunch &l, hipStream_t st)
{
    BatchArgs a;
    a.batch = l.batch;
    a.n = l.n;
    a.nrhs = l.nrhs;
    a.a_off = l.a_off;
    a.b_off = l.b_off;
    a.A = l.A;
    a.B = l.B;
    a.X = l.X;
    a.prec = l.prec;
    a.reps = l.reps;
    a.tol = l.tol;
    a.mu16 = l.mu16;
    a.max_iter = l.max_iter;
    a.fallback = l.fallback;
    a.equilibrate = l.equilibrate;
    a.order = l.order;
    a.queue = l.queue;
    a.ws = (char *)l.ws;
    a.ws_stride = batch_ws_stride();
    a.picker = l.picker;
    a.ticks = l.ticks;
    hipLaunchKernelGGL(k_batch_order, dim3(1), dim3(1024), 0, st, l.batch, l.n, l.prec, l.reps, l.order, l.queue,
                       l.ticks);
    // picker (AUTO systems), then half-precision requests (with their fallback
    // to binary32), binary32 ones, binary64 (requests and hand-overs); four
    // wavefronts per workgroup
    if (l.picker)
        hipLaunchKernelGGL(k_batch_pick, dim3((unsigned)l.grid), dim3(256), 0, st, a);
    hipLaunchKernelGGL(k_batch_half<4>, dim3((unsigned)l.grid), dim3(256), 0, st, a);
    hipLaunchKernelGGL((k_batch<4, false>), dim3((unsigned)l.grid), dim3(256), 0, st, a);
    hipLaunchKernelGGL((k_batch<4, true>), dim3((unsigned)l.grid), dim3(256), 0, st, a);
    return hipGetLastError();
}

void launch_features(int64_t batch, const int32_t *n, const int32_t *nrhs, const int64_t *a_off, const double *A,
                     float *feat, hipStream_t st)
{
    if (batch <= 0) return;
    const unsigned grid = (unsigned)(batch < 2048 ? batch : 2048);
    hipLaunchKernelGGL(k_features, dim3(grid), dim3(256), 0, st, batch, n, nrhs, a_off, A, feat);
}

}  // namespace spd
