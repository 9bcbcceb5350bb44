// Triangular solves with the low-precision factor (Eq. (3): forward L y = b,
// backward L^T x = y), blocked by big diagonal blocks of NBS (1024) rows.
//
// Set-up, once per factorisation: W_k = L_kk^{-1} for every big diagonal
// block, built from the 32-wide block inverses by repeated doubling,
//   [W11 0; W21 W22] with W21 = -W22 (L21 W11),
// two batched MFMA products per doubling level (the first two levels in
// shared memory).
//
// Solve, one persistent launch per direction.  With K big blocks the forward
// solve is z_k = W_k (b_k - sum_{j<k} L_kj z_j).  It is cut into tasks of R
// rows (32 binary32 / 16 binary64):
//   U(j, i, c): P_ij[c] = L_ij[rows c] z_j          (j < i)
//   Z(i, c)   : z_i[c]  = W_i[rows c] (b_i - sum_j P_ij)
// handed out by an atomic counter column by column (Z(j), U(j, j+1), ...,
// U(j, K-1)), which is a topological order: every task waits only on tasks
// handed out before it, so progress never depends on how many workgroups are
// resident, and the bandwidth-bound U tasks run well ahead of the chain.
// A task loads its matrix block into registers before it waits, so the wait
// hides the load.  Z(i) sums the partials of blocks j <= i-2 (finished a step
// earlier) before it waits for the newest ones, U(i-1, i), so the critical
// path per big block is one Z and one U task.  Partials are summed in a fixed
// order: results do not depend on timing.  The backward solve is the mirror
// image with transposed blocks (x_k = W_k^T (y_k - sum_{j>k} L_jk^T x_j)).
//
// Waits are bounded: after ~1 s without progress a workgroup raises the
// error flag and leaves; every other waiter sees the flag and leaves too.
//
// Publishing a task's results: each XCD has its own L2, and a release fence
// at agent scope writes that whole cache back to memory; once per task it
// cuts the kernel's streaming rate about threefold.  Results that other
// workgroups read are therefore written with agent-scope stores (coherent
// across the L2s by themselves), and publishing waits only for those stores
// to complete before the counter is raised.  The waiting side reads them
// with agent-scope loads in turn, so it needs no acquire fence (an L2
// invalidate) either.
#include "common.h"
#include "internal.h"

#include <algorithm>
#include <type_traits>

#define TRSV_NBS 1024                    // big diagonal block
#define TRSV_NCRIT 64                    // workgroups on the chain's tasks
#define TRSV_NBULK 192                   // workgroups streaming the other blocks
#define TRSV_CDEPTH 1                    // U(p, p+d) tasks taken by the chain: d <= this

// thread 0 only: wait until *addr >= want, or give up after `tmo` ticks of
// wall_clock64 (100 MHz on gfx9) or as soon as another wait has given up.
// The polling loads are relaxed agent-scope atomics (coherent loads that do
// not invalidate the caches).
SPD_DEV bool wait_ge(int *addr, int want, int *err, unsigned long long tmo)
{
    const unsigned long long t0 = wall_clock64();
    while (__hip_atomic_load(addr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want) {
        if (__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            return false;
        if (wall_clock64() - t0 > tmo) {
            __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        __builtin_amdgcn_s_sleep(2);
    }
    return true;
}

// a result that other workgroups read (agent-coherent store), and its read
template <typename T>
SPD_DEV void store_shared(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
SPD_DEV T load_shared(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// Big-block inverses.
// WB holds K blocks of nbs x nbs (column-major, leading dimension nbs); block
// k covers rows [k nbs, k nbs + s_k), s_k = min(nbs, npad - k nbs).
//
// Base: the inverse of each 128-wide diagonal block from the inverses of its
// four 32 x 32 diagonal sub-blocks (left by the factorisation), two doubling
// levels in shared memory; one workgroup per block.  Blocks are 32 x 32, held
// as [row][column] with pitch 33, so both operands and the results are read
// and written without bank conflicts; products are formed transposed, so that
// each lane stores contiguous rows.
template <typename T>
struct InvBlk {
    static constexpr int P = SPD_IB + 1, N = SPD_IB * P;
    // acc += (A B)^T for the 32 x 32 blocks A and B
    static SPD_DEV void mul(Acc32<T> &acc, const T *A, const T *B, int lane)
    {
        if constexpr (sizeof(T) == 4) {
            const int r = lane & 31, u = lane >> 5;
#pragma unroll
            for (int k = 0; k < SPD_IB; k += 2) acc.mma(B[(k + u) * P + r], A[r * P + k + u]);
        } else {
            const int r = lane & 15, u = lane >> 4;
#pragma unroll
            for (int k = 0; k < SPD_IB; k += 4) {
                const double b[2] = {B[(k + u) * P + r], B[(k + u) * P + 16 + r]};
                const double a[2] = {A[r * P + k + u], A[(16 + r) * P + k + u]};
                acc.mma(b, a);
            }
        }
    }
    // D = s acc^T, and to global memory (column-major) when given
    static SPD_DEV void put(const Acc32<T> &acc, T s, T *D, T *G, int64_t ldg, int lane)
    {
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int c = Acc32<T>::row(j, lane), r = Acc32<T>::col(j, lane);
            const T v = s * acc.get(j);
            if (D)
                D[r * P + c] = v;
            if (G)
                G[r + c * ldg] = v;
        }
    }
};

template <typename T>
__global__ __launch_bounds__(256) void k_inv_base(const T *__restrict__ L, int64_t ld, const T *__restrict__ Winv,
                                                  int nbs, T *__restrict__ WB)
{
    using IBk = InvBlk<T>;
    constexpr int IB = SPD_IB;
    // blocks: W_00, W_11, W_22, W_33, then L_10, L_20, L_21, L_30, L_31, L_32
    // (row by row of the strict lower triangle); L_10 and L_32 become W_10
    // and W_32, the other four become T = L_21 W_11 of the second level
    __shared__ T S[10][IBk::N];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b = blockIdx.x, g = b * 128, kb = g / nbs, o = g - kb * nbs;
    const T *Lb = L + g + g * ld, *Wi = Winv + b * 4 * IB * IB;
    T *Wb = WB + kb * nbs * nbs + o + o * nbs;
    auto rowof = [](int q) { return q < 1 ? 1 : (q < 3 ? 2 : 3); };  // block row of strict lower block q
    constexpr int U = 20;  // loads in flight per thread
    for (int base = 0; base < 10 * IB * IB; base += 256 * U) {
        T v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = base + u * 256 + tid, blk = e >> 10, r = e & 31, c = (e >> 5) & 31;
            if (blk < 4) {
                v[u] = Wi[e];
            } else {
                const int i = rowof(blk - 4), j = blk - 4 - i * (i - 1) / 2;
                v[u] = Lb[(IB * i + r) + (int64_t)(IB * j + c) * ld];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = base + u * 256 + tid, blk = e >> 10, r = e & 31, c = (e >> 5) & 31;
            S[blk][r * IBk::P + c] = v[u];
            if (blk < 4)
                Wb[(IB * blk + r) + (int64_t)(IB * blk + c) * nbs] = v[u];
        }
    }
    __syncthreads();
    // first level: waves 0 and 1, W_{2p+1,2p} = -W_{2p+1} (L W_{2p})
    if (wave < 2) {
        T *Lq = S[wave == 0 ? 4 : 9];
        const T *W1 = S[2 * wave], *W2 = S[2 * wave + 1];
        Acc32<T> acc;
        acc.zero();
        IBk::mul(acc, Lq, W1, lane);
        __builtin_amdgcn_wave_barrier();
        IBk::put(acc, (T)1, Lq, nullptr, 0, lane);
        __builtin_amdgcn_wave_barrier();
        acc.zero();
        IBk::mul(acc, W2, Lq, lane);
        __builtin_amdgcn_wave_barrier();
        IBk::put(acc, (T)-1, Lq, Wb + (IB * (2 * wave + 1)) + (int64_t)(IB * 2 * wave) * nbs, nbs, lane);
    }
    __syncthreads();
    // second level, one output block (i, j) per wave, i = 2, 3 and j = 0, 1:
    // T = L_21 W_11, then W_21 = -W_22 T
    const int i = 2 + (wave >> 1), j = wave & 1;
    auto Lblk = [&](int ii, int jj) { return S[4 + ii * (ii - 1) / 2 + jj]; };
    Acc32<T> acc;
    acc.zero();
    if (j == 0) {
        IBk::mul(acc, Lblk(i, 0), S[0], lane);
        IBk::mul(acc, Lblk(i, 1), S[4], lane);
    } else {
        IBk::mul(acc, Lblk(i, 1), S[1], lane);
    }
    __syncthreads();
    IBk::put(acc, (T)1, Lblk(i, j), nullptr, 0, lane);
    __syncthreads();
    acc.zero();
    if (i == 3)
        IBk::mul(acc, S[9], Lblk(2, j), lane);
    IBk::mul(acc, S[i], Lblk(i, j), lane);
    IBk::put(acc, (T)-1, nullptr, Wb + IB * i + (int64_t)(IB * j) * nbs, nbs, lane);
}

// One doubling level of width s.  Workgroup (x, y, z): output tile (x, y) of
// pair p of big block kb (z = kb * ppb + p); the pair is [a0, a1) + [a1, b1)
// inside the block.  PHASE 1: Tk = L21 W11 (W11 lower: k >= 64 y);
// PHASE 2: W21 = -W22 Tk (W22 lower: k < 64 (x + 1)).  64 x 64 tiles, one
// 32 x 32 block per wave on MFMA, computed transposed so that each lane
// stores contiguous rows.  The operands go straight from the caches to
// registers, the next 32 values of k in flight while the current ones are
// multiplied: the k-slots of an MFMA are a free summation order, so a lane
// takes its right operand as one 16-byte load of consecutive k and the left
// operand's columns are picked to match.
// Bound by latency for one or two big blocks (n up to 2048: 8 to 64
// workgroups of a 512-deep product).  128 x 128 tiles staged through shared
// memory with no load ahead took 18 us per launch at n = 300 and 35 us at
// n = 1300 and 3000 (average over the levels); these take 7 and 11 us.  At
// n = 16384 (16 big blocks) both fill the chip: 37 us.
template <typename T, int PHASE>
__global__ __launch_bounds__(256) void k_inv_merge(const T *__restrict__ L, int64_t ld, int64_t npad,
                                                   T *__restrict__ WB, int nbs, int s, T *__restrict__ Tb)
{
    constexpr int F32 = sizeof(T) == 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ppb = (nbs + 2 * s - 1) / (2 * s);
    const int kb = blockIdx.z / ppb, p = blockIdx.z % ppb;
    const int64_t o = (int64_t)kb * nbs;
    const int sk = (int)((npad - o) < nbs ? (npad - o) : nbs);
    const int a0 = 2 * p * s, a1 = a0 + s, b1 = (a0 + 2 * s < sk) ? a0 + 2 * s : sk;
    if (a1 >= sk)
        return;
    const int M = b1 - a1;
    const int m0 = blockIdx.x * 64, n0 = blockIdx.y * 64;
    if (m0 >= M)
        return;
    T *Wk = WB + (int64_t)kb * nbs * nbs;
    T *Tk = Tb + (int64_t)blockIdx.z * s * s;
    const T *A, *B;
    T *Cp;
    int64_t lda, ldb, ldc;
    int kbeg, kend;
    T alpha;
    if (PHASE == 1) {
        A = L + (o + a1) + (o + a0) * ld;
        lda = ld;
        B = Wk + a0 + (int64_t)a0 * nbs;
        ldb = nbs;
        Cp = Tk;
        ldc = s;
        kbeg = n0;
        kend = s;
        alpha = (T)1;
    } else {
        A = Wk + a1 + (int64_t)a1 * nbs;
        lda = nbs;
        B = Tk;
        ldb = s;
        Cp = Wk + a1 + (int64_t)a0 * nbs;
        ldc = nbs;
        kbeg = 0;
        kend = m0 + 64;  // M is a multiple of 128
        alpha = (T)-1;
    }
    const int mw = m0 + 32 * (wave & 1), nw = n0 + 32 * (wave >> 1);
    // lane: row r of a 32 (binary32) / 16 (binary64) row block, k-slot u;
    // group g of 8 values of k: slot u takes k = 8 g + V u + q at step q
    constexpr int RB = F32 ? 32 : 16, NRB = 32 / RB, V = F32 ? 4 : 2, G = 4;
    using VT = typename std::conditional<F32, float4, double2>::type;
    const int r = lane & (RB - 1), u = lane / RB;
    const T *pA = A + mw + r + (int64_t)(V * u) * lda;
    const T *pB = B + V * u + (int64_t)(nw + r) * ldb;
    Acc32<T> acc;
    acc.zero();
    T fa[2][G][NRB][V];
    VT fb[2][G][NRB];
    auto load = [&](int st, int k0) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int h = 0; h < NRB; ++h) {
                fb[st][g][h] = *(const VT *)(pB + k0 + 8 * g + (int64_t)(RB * h) * ldb);
#pragma unroll
                for (int q = 0; q < V; ++q) fa[st][g][h][q] = pA[RB * h + (int64_t)(k0 + 8 * g + q) * lda];
            }
    };
    auto mul = [&](int st) {
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int q = 0; q < V; ++q) {
                if constexpr (F32) {
                    const float4 b = fb[st][g][0];
                    acc.mma(q == 0 ? b.x : q == 1 ? b.y : q == 2 ? b.z : b.w, fa[st][g][0][q]);
                } else {
                    const double b[2] = {q == 0 ? fb[st][g][0].x : fb[st][g][0].y,
                                         q == 0 ? fb[st][g][NRB - 1].x : fb[st][g][NRB - 1].y};
                    const double a[2] = {fa[st][g][0][q], fa[st][g][NRB - 1][q]};
                    acc.mma(b, a);
                }
            }
    };
    // kend - kbeg is a multiple of 64
    load(0, kbeg);
    for (int k0 = kbeg; k0 < kend; k0 += 64) {
        load(1, k0 + 32);
        __builtin_amdgcn_sched_barrier(0);
        mul(0);
        __builtin_amdgcn_sched_barrier(0);
        if (k0 + 64 < kend)
            load(0, k0 + 64);
        __builtin_amdgcn_sched_barrier(0);
        mul(1);
        __builtin_amdgcn_sched_barrier(0);
    }
    // register j: n = row(j), m = col(j)
#pragma unroll
    for (int j = 0; j < 16; ++j)
        Cp[(mw + Acc32<T>::col(j, lane)) + (int64_t)(nw + Acc32<T>::row(j, lane)) * ldc] = alpha * acc.get(j);
}

// ---------------------------------------------------------------------------
// Register-resident block times vector.
//   FWD (rows form):  out[r] = sum_c M[r][c] v[c], R rows, columns [0, ncols)
//   BWD (cols form):  out[c] = sum_r M[r][c] v[r0 + r], R columns, rows [0, nrows)
// M is column-major (leading dimension ld).  VEC elements per 16-byte load;
// R = 8 VEC; every thread holds E = NBS / 32 vectors.
template <typename T> struct VecOf;
template <> struct VecOf<float> { using V = float4; static constexpr int N = 4; };
template <> struct VecOf<double> { using V = double2; static constexpr int N = 2; };

template <typename T>
SPD_DEV T vget(const typename VecOf<T>::V &v, int r)
{
    if constexpr (sizeof(T) == 4)
        return r == 0 ? v.x : r == 1 ? v.y : r == 2 ? v.z : v.w;
    else
        return r == 0 ? v.x : v.y;
}

template <typename T, int MC, bool FWD, int NBS>
struct BlockVec {
    using V = typename VecOf<T>::V;
    static constexpr int VEC = VecOf<T>::N;
    static constexpr int R = 8 * VEC;      // rows (FWD) / columns (BWD) per task
    static constexpr int E = NBS / 32;     // vectors per thread
    static constexpr int TPC = 256 / R;    // BWD: threads per column
    V m[E];

    // FWD: thread t covers rows VEC (t % 8) .. +VEC of columns t / 8 + 32 e.
    // BWD: thread t covers column t / TPC, rows VEC (t % TPC) + 32 e .. +VEC.
    SPD_DEV void load(const T *base, int64_t ld, int len, int tid)
    {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if constexpr (FWD) {
                const int col = tid / 8 + 32 * e;
                if (col < len)
                    m[e] = *(const V *)(base + VEC * (tid % 8) + (int64_t)col * ld);
            } else {
                const int row = VEC * (tid % TPC) + 32 * e;
                if (row < len)
                    m[e] = *(const V *)(base + row + (int64_t)(tid / TPC) * ld);
            }
        }
    }

    // out[r][cc] for r < R (valid in thread tid < R * MC as (tid % R, tid / R)
    // for FWD; in the thread with tid % TPC == 0 for column tid / TPC for BWD)
    SPD_DEV void apply(const T (*vs)[NBS], int len, int r0, T (*red)[R][MC], T out[MC], int tid)
    {
        const int lane = tid & 63, wave = tid >> 6;
        if constexpr (FWD) {
            T acc[VEC][MC];
#pragma unroll
            for (int r = 0; r < VEC; ++r)
#pragma unroll
                for (int cc = 0; cc < MC; ++cc) acc[r][cc] = (T)0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int col = tid / 8 + 32 * e;
                if (col < len) {
#pragma unroll
                    for (int cc = 0; cc < MC; ++cc) {
                        const T x = vs[cc][col];
#pragma unroll
                        for (int r = 0; r < VEC; ++r) acc[r][cc] += vget<T>(m[e], r) * x;
                    }
                }
            }
            // sum over the 8 column groups of this wave (lane bits 3..5), then over waves
#pragma unroll
            for (int sh = 8; sh < 64; sh <<= 1)
#pragma unroll
                for (int r = 0; r < VEC; ++r)
#pragma unroll
                    for (int cc = 0; cc < MC; ++cc) acc[r][cc] += __shfl_xor(acc[r][cc], sh);
            if (lane < 8) {
#pragma unroll
                for (int r = 0; r < VEC; ++r)
#pragma unroll
                    for (int cc = 0; cc < MC; ++cc) red[wave][VEC * lane + r][cc] = acc[r][cc];
            }
            __syncthreads();
            if (tid < R * MC) {
                const int r = tid % R, cc = tid / R;
                out[0] = ((red[0][r][cc] + red[1][r][cc]) + red[2][r][cc]) + red[3][r][cc];
            }
        } else {
            T acc[MC];
#pragma unroll
            for (int cc = 0; cc < MC; ++cc) acc[cc] = (T)0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int row = VEC * (tid % TPC) + 32 * e;
                if (row < len) {
#pragma unroll
                    for (int r = 0; r < VEC; ++r) {
                        const T a = vget<T>(m[e], r);
#pragma unroll
                        for (int cc = 0; cc < MC; ++cc) acc[cc] += a * vs[cc][r0 + row + r];
                    }
                }
            }
#pragma unroll
            for (int sh = 1; sh < TPC; sh <<= 1)
#pragma unroll
                for (int cc = 0; cc < MC; ++cc) acc[cc] += __shfl_xor(acc[cc], sh);
#pragma unroll
            for (int cc = 0; cc < MC; ++cc) out[cc] = acc[cc];
        }
    }
};

// geometry of big block k
SPD_DEV void big_block(int64_t npad, int nbs, int k, int64_t &o, int &sz)
{
    o = (int64_t)k * nbs;
    sz = (int)((npad - o) < nbs ? (npad - o) : nbs);
}

template <typename T, int MC, bool FWD>
__global__ __launch_bounds__(256) void k_trsv_blk(const T *__restrict__ L, int64_t ld, const T *__restrict__ WB,
                                                  int64_t npad, int nbs, int K, const T *__restrict__ Yin,
                                                  T *__restrict__ Zout, int64_t ldy, int c0, int m,
                                                  T *__restrict__ P, int *ctl, int *err, int ncrit, int cdepth,
                                                  unsigned long long tmo)
{
    constexpr int NBS = TRSV_NBS;
    using BV = BlockVec<T, MC, FWD, NBS>;
    constexpr int R = BV::R;
    // vector entries per thread, and partials summed per batch of loads
    constexpr int PER = MC * NBS / 256, QB = PER >= 32 ? 1 : 32 / PER;
    __shared__ T vs[MC][NBS];
    __shared__ T red[4][R][MC];
    __shared__ int s_task, s_ok, s_crit;
    const int tid = threadIdx.x;
    int *qcrit = ctl, *qbulk = ctl + 1, *ticket = ctl + 2;
    int *cntA = ctl + 3, *cntB = ctl + 3 + K, *cntZ = ctl + 3 + 2 * K;
    const int mc = min(MC, m - c0);
    BV bv;
    // Blocks in processing order p (FWD: block p; BWD: block K-1-p); only
    // block K-1 may be shorter than nbs.
    const int slast = (int)(npad - (int64_t)(K - 1) * nbs);
    auto proc_size = [&](int p) -> int { return (FWD ? p == K - 1 : p == 0) ? slast : nbs; };
    auto rows_before = [&](int p) -> int64_t {
        return FWD ? (int64_t)p * nbs : (p == 0 ? 0 : slast + (int64_t)(p - 1) * nbs);
    };
    auto proc_locate = [&](int64_t pos, int &p, int &off) {
        if (FWD) {
            p = (int)(pos / nbs);
            off = (int)(pos - (int64_t)p * nbs);
        } else if (pos < slast) {
            p = 0;
            off = (int)pos;
        } else {
            p = 1 + (int)((pos - slast) / nbs);
            off = (int)((pos - slast) % nbs);
        }
    };

    // The first ncrit workgroups to start take the chain's tasks in step
    // order: every Z(p), the U(p, p+1) that feeds the next Z, and the U(p,
    // p+d) for d <= cdepth; the others take the remaining U tasks column by
    // column.  A workgroup that has started is resident, so the chain never
    // waits for a workgroup that cannot run.
    if (tid == 0)
        s_crit = atomicAdd(ticket, 1) < ncrit;
    __syncthreads();
    const bool crit = s_crit != 0;
    for (;;) {
        if (tid == 0)
            s_task = atomicAdd(crit ? qcrit : qbulk, 1);
        __syncthreads();
        int rem = s_task, pi = -1, pj = -1, c = 0;
        if (crit) {
            // step p: Z(p, 0..), then U(p, p+d, 0..) for d = 1 .. cdepth
            for (int p = 0; p < K && pi < 0; ++p) {
                for (int d = 0; d <= cdepth && p + d < K; ++d) {
                    const int nt = proc_size(p + d) / R;
                    if (rem < nt) {
                        pj = p;
                        pi = p + d;
                        c = rem;
                        break;
                    }
                    rem -= nt;
                }
            }
        } else {
            // column q: U(q, pi, 0..) for the blocks pi from q+1+cdepth on
            for (int q = 0; q + 1 + cdepth < K; ++q) {
                const int cnt = (int)((npad - rows_before(q + 1 + cdepth)) / R);
                if (rem < cnt) {
                    int off;
                    proc_locate(rows_before(q + 1 + cdepth) + (int64_t)rem * R, pi, off);
                    pj = q;
                    c = off / R;
                    break;
                }
                rem -= cnt;
            }
        }
        if (pi < 0)
            return;
        const int nc = proc_size(pi) / R;
        const bool ztask = (pj == pi);
        const int ki = FWD ? pi : K - 1 - pi, kj = FWD ? pj : K - 1 - pj;
        int64_t oi, oj;
        int si, sj;
        big_block(npad, nbs, ki, oi, si);
        big_block(npad, nbs, kj, oj, sj);
        T *Pbase = P + ((int64_t)pi * (pi - 1) / 2) * NBS * MC;  // partials of row pi
        const T *Wk = WB + (int64_t)ki * nbs * nbs;

        // The task's matrix block, loaded before any wait:
        //   U: the block of L coupling ki and kj (entries c R .. +R of block ki);
        //   Z: rows (FWD) / columns (BWD) c R .. +R of W_ki.
        // Vector range it needs: U [0, sj); Z FWD [0, (c+1) R), BWD [c R, si).
        const T *mb;
        int64_t mld;
        int lo, hi;
        if (!ztask) {
            mb = FWD ? L + (oi + c * R) + oj * ld : L + oj + (oi + c * R) * ld;
            mld = ld;
            lo = 0;
            hi = sj;
        } else {
            mb = FWD ? Wk + c * R : Wk + c * R + (int64_t)(c * R) * nbs;
            mld = nbs;
            lo = FWD ? 0 : c * R;
            hi = FWD ? (c + 1) * R : si;
        }
        bv.load(mb, mld, hi - lo, tid);

        if (!ztask) {
            if (tid == 0)
                s_ok = wait_ge(&cntZ[pj], sj / R, err, tmo) ? 1 : 0;
            __syncthreads();
            if (!s_ok)
                return;
            // all of this thread's loads issued before the first use
            T zv[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int t = (tid + 256 * k) % NBS, cc = (tid + 256 * k) / NBS;
                zv[k] = (t < sj && cc < mc) ? load_shared(&Zout[(oj + t) + (int64_t)(c0 + cc) * ldy]) : (T)0;
            }
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int t = (tid + 256 * k) % NBS, cc = (tid + 256 * k) / NBS;
                if (t < sj)
                    vs[cc][t] = zv[k];
            }
        } else {
            if (pi >= 2) {
                if (tid == 0)
                    s_ok = wait_ge(&cntA[pi], (pi - 1) * nc, err, tmo) ? 1 : 0;
                __syncthreads();
                if (!s_ok)
                    return;
            }
            // v = y - (sum of the partials of blocks finished a step ago), in
            // order of q; the loads go out QB partials at a time
            T sA[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) sA[k] = (T)0;
            for (int q0 = 0; q0 + 1 < pi; q0 += QB) {
                T pv[QB][PER];
#pragma unroll
                for (int u = 0; u < QB; ++u)
#pragma unroll
                    for (int k = 0; k < PER; ++k) {
                        const int t = (tid + 256 * k) % NBS, cc = (tid + 256 * k) / NBS;
                        pv[u][k] = (q0 + u + 1 < pi && t >= lo && t < hi)
                                       ? load_shared(&Pbase[(int64_t)(q0 + u) * NBS * MC + cc * NBS + t])
                                       : (T)0;
                    }
#pragma unroll
                for (int u = 0; u < QB; ++u)
#pragma unroll
                    for (int k = 0; k < PER; ++k)
                        if (q0 + u + 1 < pi)
                            sA[k] += pv[u][k];
            }
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int t = (tid + 256 * k) % NBS, cc = (tid + 256 * k) / NBS;
                if (t >= lo && t < hi)
                    vs[cc][t] = (cc < mc) ? Yin[(oi + t) + (int64_t)(c0 + cc) * ldy] - sA[k] : (T)0;
            }
            if (pi >= 1) {
                if (tid == 0)
                    s_ok = wait_ge(&cntB[pi], nc, err, tmo) ? 1 : 0;
                __syncthreads();
                if (!s_ok)
                    return;
                const T *pB = Pbase + (int64_t)(pi - 1) * NBS * MC;
                T bv_[PER];
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const int t = (tid + 256 * k) % NBS, cc = (tid + 256 * k) / NBS;
                    bv_[k] = (t >= lo && t < hi) ? load_shared(&pB[cc * NBS + t]) : (T)0;
                }
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const int t = (tid + 256 * k) % NBS, cc = (tid + 256 * k) / NBS;
                    if (t >= lo && t < hi)
                        vs[cc][t] -= bv_[k];
                }
            }
        }
        __syncthreads();
        T out[MC];
        bv.apply(vs, hi - lo, lo, red, out, tid);

        // results: U -> partial P_{pi,pj}; Z -> solution entries of block ki
        T *dst;
        int64_t dcol;
        int nvalid;
        if (!ztask) {
            dst = Pbase + (int64_t)pj * NBS * MC + c * R;
            dcol = NBS;
            nvalid = MC;
        } else {
            dst = Zout + oi + c * R + (int64_t)c0 * ldy;
            dcol = ldy;
            nvalid = mc;
        }
        if (FWD) {
            if (tid < R * MC && tid / R < nvalid)
                store_shared(&dst[tid % R + (tid / R) * dcol], out[0]);
        } else if (tid % BV::TPC == 0) {
#pragma unroll
            for (int cc = 0; cc < MC; ++cc)
                if (cc < nvalid)
                    store_shared(&dst[tid / BV::TPC + cc * dcol], out[cc]);
        }
        // every thread's result stores complete, then one relaxed increment
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0) {
            int *ctr = ztask ? &cntZ[pi] : (pj == pi - 1 ? &cntB[pi] : &cntA[pi]);
            __hip_atomic_fetch_add(ctr, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

// ---------------------------------------------------------------------------
// Three or more right-hand sides: the same block recurrence on MFMA, 16 NT of
// them per launch.  Tasks of R rows (32 binary32 / 16 binary64) of a big block
// in processing order p, handed out by a counter in the order U(p, 0..), Z(p,
// 0..), p = 0, 1, ... (no U at p = 0):
//   U(p, c): v_p[c] = y_p[c] - sum_{q < p} L_pq[rows c] z_q    (q in order)
//   Z(p, c): z_p[c] = W_p[rows c] v_p                          (v_0 = y_0)
// (transposed blocks for the backward solve).  A task waits only for tasks
// handed out before it.  The sum over q stays in the registers of one
// workgroup, so there are no partial products in memory: with 32 columns
// they would be as large as the blocks themselves.
//
// Eight waves split a block's columns (the k of the product) evenly; the
// k-slots of an MFMA are a free summation order, so lane (r = lane % 16,
// u = lane / 16) takes k = 16 g + 4 u + i at step i of group g: its vector
// values are 16 consecutive bytes, and so are its matrix values in the
// backward solve.  Each vector value is needed by one wave only, so neither
// operand goes through shared memory.  The matrix block is loaded before the
// wait, the next one before the product.  The waves' sums are added in pairs
// through shared memory.
//
// A wave's 128 products of a block make four sums of 32, then one, added to
// those of the blocks before: the rounding error of a column does not exceed
// that of BlockVec (binary32, random unit factor, in units of u: 2.5 at
// n = 300 and 2.6 at 16384; BlockVec 2.6 and 4.2).  One sum over all blocks
// gave 3.6 and 6.4; it took 1-2 % less time in binary32 and 5 % in binary64.
//
// Bound by the chain of 2 K tasks, each a poll, the loads of the vector and a
// 1024-deep product.  A solve, forward and backward, in passes of up to 8
// columns on the VALU (BlockVec) and here: n = 10000 with 32 columns 2183 and
// 457 us; n = 6000 with 3 and 8 columns 216 and 159, 306 and 167; n = 16384
// 610 and 584, 919 and 614 (binary64 1025 and 1034, 1499 and 1068); n = 1300
// 56 and 47, 82 and 50.  One or two columns stay on BlockVec, whose 256
// workgroups stream more: n = 16384 450 and 510 us (with 3 columns here 581),
// n = 3000 64 and 75 (83).
#define TRSM_WAVES 8
// raw buffer loads coherent at agent scope (the SC1 cache policy bit)
#define SPD_BUFFER_AGENT 16
typedef double double2v __attribute__((ext_vector_type(2)));
// buffer resource over memory from a workgroup-uniform address on
template <typename T>
SPD_DEV __amdgpu_buffer_rsrc_t uniform_rsrc(const T *p)
{
    const unsigned long long b = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffull));
    const unsigned hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __builtin_amdgcn_make_buffer_rsrc((void *)(((unsigned long long)hi << 32) | lo), (short)0, 0x7fffffff,
                                             SPD_BUFFER_RSRC_WORD3);
}
template <typename T, int NT, bool FWD>
__global__ __launch_bounds__(64 * TRSM_WAVES) void k_trsv_mfma(const T *__restrict__ L, int64_t ld,
                                                               const T *__restrict__ WB, int64_t npad, int nbs, int K,
                                                               const T *__restrict__ Yin, T *__restrict__ Zout,
                                                               int64_t ldy, int c0, int m, T *__restrict__ V,
                                                               int *ctl, int *err, unsigned long long tmo)
{
    constexpr bool F32 = sizeof(T) == 4;
    constexpr int MT = F32 ? 2 : 1, R = 16 * MT, MC = 16 * NT, NW = TRSM_WAVES, NBS = TRSV_NBS,
                  GM = NBS / (16 * NW);
    static_assert(NW == 8 && GM == 8, "the order of the sums below");
    using acc_t = typename std::conditional<F32, floatx4, doublex4>::type;
    __shared__ T red[NW][MC][R + 1];
    __shared__ int s_task, s_ok[2];
    // the wave's number as a scalar: addresses are then a scalar base plus one
    // 32-bit lane offset per operand
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, u = lane >> 4;
    int *ticket = ctl, *cntV = ctl + 3, *cntZ = ctl + 3 + K;
    const int mc = min(MC, m - c0);
    const int slast = (int)(npad - (int64_t)(K - 1) * nbs);
    auto proc_size = [&](int p) -> int { return (FWD ? p == K - 1 : p == 0) ? slast : nbs; };

    // All loads are buffer loads: a scalar base and offset plus one 32-bit
    // lane offset per operand (flat addresses would not fit the registers
    // beside the blocks).  Wave w takes k in [128 w, 128 w + 128); past a short
    // block's end (len) it takes k = 0 again with a zero vector, so that every
    // block runs the same straight-line code.  a[g][i][t]: row tile t.
    constexpr int EB = sizeof(T);
    auto group = [&](int g, int len) -> int {
        const int k = 16 * GM * w + 16 * g;
        return k < len ? k : 0;
    };
    auto load_block = [&](T (&a)[GM][4][MT], const T *base, int mld, int len) {
        // FWD, base the strip's first row: rows MT r + t of column k + i;
        // BWD, base its first column: rows k .. k + 3 of column 16 t + r
        const __amdgpu_buffer_rsrc_t rc = uniform_rsrc(base);
        const int o0 = (FWD ? MT * r + 4 * u * mld : r * mld + 4 * u) * EB, o1 = o0 + 16 * mld * EB;
#pragma unroll
        for (int g = 0; g < GM; ++g) {
            const int k = group(g, len);
            if constexpr (FWD) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b64(rc, o0, (k + i) * mld * EB, 0);
                    if constexpr (F32) {
                        a[g][i][0] = __builtin_bit_cast(float, (unsigned)v[0]);
                        a[g][i][MT - 1] = __builtin_bit_cast(float, (unsigned)v[1]);
                    } else {
                        a[g][i][0] = __builtin_bit_cast(double, v);
                    }
                }
            } else if constexpr (F32) {
#pragma unroll
                for (int t = 0; t < MT; ++t) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rc, t ? o1 : o0, k * EB, 0);
#pragma unroll
                    for (int i = 0; i < 4; ++i) a[g][i][t] = __builtin_bit_cast(float, (unsigned)v[i]);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    const auto v =
                        __builtin_bit_cast(double2v, __builtin_amdgcn_raw_buffer_load_b128(rc, o0, (k + i) * EB, 0));
                    a[g][i][0] = v[0];
                    a[g][i + 1][0] = v[1];
                }
            }
        }
    };
    // acc += block times the vector (columns past the last right-hand side
    // repeat column c0: their products are dropped).  The vector is read with
    // agent-scope loads (SPD_BUFFER_AGENT), like load_shared.
    acc_t acc[MT][NT];
    int oz[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) oz[t] = (4 * u + (16 * t + r < mc ? 16 * t + r : 0) * (int)ldy) * EB;
    auto multiply = [&](const T (&a)[GM][4][MT], const T *vec, int len) {
        const __amdgpu_buffer_rsrc_t rc = uniform_rsrc(vec);
        T z[GM][NT][4];
#pragma unroll
        for (int g = 0; g < GM; ++g) {
            const int k = group(g, len);
            const bool in = 16 * GM * w + 16 * g < len;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                if constexpr (F32) {
                    const auto v = __builtin_amdgcn_raw_buffer_load_b128(rc, oz[t], k * EB, SPD_BUFFER_AGENT);
#pragma unroll
                    for (int i = 0; i < 4; ++i) z[g][t][i] = in ? __builtin_bit_cast(float, (unsigned)v[i]) : 0.0f;
                } else {
#pragma unroll
                    for (int i = 0; i < 4; i += 2) {
                        const auto v = __builtin_bit_cast(
                            double2v, __builtin_amdgcn_raw_buffer_load_b128(rc, oz[t], (k + i) * EB, SPD_BUFFER_AGENT));
                        z[g][t][i] = in ? v[0] : 0.0;
                        z[g][t][i + 1] = in ? v[1] : 0.0;
                    }
                }
            }
        }
        // four sums, by step i, for the block, added in pairs
        acc_t s[4][MT][NT];
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < MT; ++h)
#pragma unroll
                for (int t = 0; t < NT; ++t) s[i][h][t] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int g = 0; g < GM; ++g)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int t = 0; t < NT; ++t)
#pragma unroll
                    for (int h = 0; h < MT; ++h) {
                        if constexpr (F32)
                            s[i][h][t] =
                                __builtin_amdgcn_mfma_f32_16x16x4f32(z[g][t][i], a[g][i][h], s[i][h][t], 0, 0, 0);
                        else
                            s[i][h][t] =
                                __builtin_amdgcn_mfma_f64_16x16x4f64(z[g][t][i], a[g][i][h], s[i][h][t], 0, 0, 0);
                    }
#pragma unroll
        for (int h = 0; h < MT; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[h][t] += (s[0][h][t] + s[1][h][t]) + (s[2][h][t] + s[3][h][t]);
        __builtin_amdgcn_sched_barrier(0);
    };
    int slot = 0;  // s_ok alternates: a slot is rewritten only after the barrier that follows its reading
    auto wait = [&](int *ctr, int want) -> bool {
        slot ^= 1;
        if (tid == 0)
            s_ok[slot] = wait_ge(ctr, want, err, tmo) ? 1 : 0;
        __syncthreads();
        return s_ok[slot] != 0;
    };

    for (;;) {
        if (tid == 0)
            s_task = atomicAdd(ticket, 1);
        __syncthreads();
        int rem = __builtin_amdgcn_readfirstlane(s_task), p = -1, c = 0;
        bool ztask = false;
        for (int q = 0; q < K; ++q) {
            const int nt = proc_size(q) / R;
            if (q > 0) {
                if (rem < nt) {
                    p = q;
                    c = rem;
                    break;
                }
                rem -= nt;
            }
            if (rem < nt) {
                p = q;
                c = rem;
                ztask = true;
                break;
            }
            rem -= nt;
        }
        if (p < 0)
            return;
        const int ki = FWD ? p : K - 1 - p;
        int64_t oi;
        int si;
        big_block(npad, nbs, ki, oi, si);
        const int nc = si / R;
#pragma unroll
        for (int h = 0; h < MT; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[h][t] = acc_t{0, 0, 0, 0};
        if (ztask) {
            // the strip's rows (FWD) or columns (BWD) of W_ki, with its zeros
            const T *Wk = WB + (int64_t)ki * nbs * nbs;
            T a0[GM][4][MT];
            load_block(a0, FWD ? Wk + c * R : Wk + (int64_t)(c * R) * nbs, nbs, si);
            if (p > 0 && !wait(&cntV[p], nc))
                return;
            multiply(a0, p > 0 ? V + oi : Yin + oi + (int64_t)c0 * ldy, si);
        } else {
            T a0[GM][4][MT], a1[GM][4][MT];
            auto fetch = [&](T (&a)[GM][4][MT], int q) {  // past the last block: that one again, unused
                q = q < p ? q : p - 1;
                const int64_t oj = (int64_t)(FWD ? q : K - 1 - q) * nbs;
                load_block(a, FWD ? L + oi + c * R + oj * ld : L + oj + (oi + c * R) * ld, (int)ld, proc_size(q));
            };
            auto step = [&](const T (&a)[GM][4][MT], int q) -> bool {
                if (!wait(&cntZ[q], proc_size(q) / R))
                    return false;
                multiply(a, Zout + (int64_t)(FWD ? q : K - 1 - q) * nbs + (int64_t)c0 * ldy, proc_size(q));
                return true;
            };
            fetch(a0, 0);
            for (int q = 0;;) {
                fetch(a1, q + 1);
                if (!step(a0, q))
                    return;
                if (++q >= p)
                    break;
                fetch(a0, q + 1);
                if (!step(a1, q))
                    return;
                if (++q >= p)
                    break;
            }
        }
        // accumulator register v: right-hand side 4 u + v (binary32) or
        // 4 v + u (binary64) of its tile, strip row MT r + h (FWD) or 16 h + r
#pragma unroll
        for (int h = 0; h < MT; ++h)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    red[w][16 * t + (F32 ? 4 * u + v : 4 * v + u)][FWD ? MT * r + h : 16 * h + r] = acc[h][t][v];
        __syncthreads();
        for (int e = tid; e < R * mc; e += 64 * NW) {
            const int row = e % R, cc = e / R;
            const T s = ((red[0][cc][row] + red[1][cc][row]) + (red[2][cc][row] + red[3][cc][row])) +
                        ((red[4][cc][row] + red[5][cc][row]) + (red[6][cc][row] + red[7][cc][row]));
            const int64_t i = oi + c * R + row;
            if (ztask)
                store_shared(&Zout[i + (int64_t)(c0 + cc) * ldy], s);
            else
                store_shared(&V[i + (int64_t)cc * ldy], Yin[i + (int64_t)(c0 + cc) * ldy] - s);
        }
        // every thread's result stores complete, then one relaxed increment
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (tid == 0)
            __hip_atomic_fetch_add(ztask ? &cntZ[p] : &cntV[p], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

__global__ void k_zero_int(int *p, int count)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < count)
        p[i] = 0;
}

namespace spd {

int solve_nbs(int64_t npad) { return (int)(npad < TRSV_NBS ? npad : TRSV_NBS); }
int solve_nblocks(int64_t npad) { return (int)((npad + solve_nbs(npad) - 1) / solve_nbs(npad)); }

int64_t solve_winv_elems(int64_t npad)
{
    const int64_t nbs = solve_nbs(npad);
    return solve_nblocks(npad) * nbs * nbs;
}

int64_t solve_tmp_elems(int64_t npad)
{
    const int nbs = solve_nbs(npad), K = solve_nblocks(npad);
    int64_t mx = 1;
    for (int s = 128; s < nbs; s *= 2) {
        const int64_t ppb = (nbs + 2 * s - 1) / (2 * s);
        mx = std::max<int64_t>(mx, K * ppb * (int64_t)s * s);
    }
    return mx;
}

int64_t trsv_scratch_elems(int64_t npad)
{
    const int64_t K = solve_nblocks(npad);
    // the partial products of up to TRSV_MC columns, or the updated right-hand
    // sides v of up to 32
    return std::max<int64_t>(std::max<int64_t>(K * (K - 1) / 2, 1) * TRSV_NBS * TRSV_MC, npad * 32);
}

// counters of one direction, padded to 256 bytes (a caller keeping one set
// per direction back to back keeps each on lines of its own)
int trsv_ctl_ints(int64_t npad) { return (3 + 3 * solve_nblocks(npad) + 63) & ~63; }

template <typename T>
void launch_build_winv(const T *L, int64_t ld, int64_t npad, const T *Winv, T *WB, T *Tb, hipStream_t st)
{
    const int nbs = solve_nbs(npad), K = solve_nblocks(npad);
    hipLaunchKernelGGL(k_inv_base<T>, dim3((unsigned)(npad / 128)), dim3(256), 0, st, L, ld, Winv, nbs, WB);
    for (int s = 128; s < nbs; s *= 2) {
        const int ppb = (nbs + 2 * s - 1) / (2 * s);
        const dim3 grid((unsigned)(s / 64), (unsigned)(s / 64), (unsigned)(K * ppb));
        hipLaunchKernelGGL((k_inv_merge<T, 1>), grid, dim3(256), 0, st, L, ld, npad, WB, nbs, s, Tb);
        hipLaunchKernelGGL((k_inv_merge<T, 2>), grid, dim3(256), 0, st, L, ld, npad, WB, nbs, s, Tb);
    }
}
template void launch_build_winv<float>(const float *, int64_t, int64_t, const float *, float *, float *,
                                       hipStream_t);
template void launch_build_winv<double>(const double *, int64_t, int64_t, const double *, double *, double *,
                                        hipStream_t);

template <typename T, bool FWD>
static void launch_dir(const T *L, int64_t ld, const T *WB, int64_t npad, int m, const T *Yin, T *Zout,
                       int64_t ldy, T *P, int *ctl, bool ctl_zeroed, int *err, unsigned long long tmo,
                       hipStream_t st)
{
    const int nbs = solve_nbs(npad), K = solve_nblocks(npad);
    constexpr int R = 8 * VecOf<T>::N;
    // chain tasks: every Z and U(p, p+d), d <= TRSV_CDEPTH; the other U
    // tasks stream
    const int cdepth = TRSV_CDEPTH;
    int64_t ncrit_tasks = 0, nbulk_tasks = 0;
    for (int p = 0; p < K; ++p) {
        const int64_t o = (int64_t)p * nbs, sz = std::min<int64_t>(nbs, npad - o);
        ncrit_tasks += (1 + std::min(p, cdepth)) * (sz / R);
        nbulk_tasks += std::max(p - cdepth, 0) * (sz / R);
    }
    const int ncrit = (int)std::min<int64_t>(ncrit_tasks, TRSV_NCRIT);
    const int grid = ncrit + (int)std::min<int64_t>(nbulk_tasks, TRSV_NBULK);
    const int nctl = trsv_ctl_ints(npad);
    if (m > TRSV_MC) {
        // MFMA: 32 columns per launch (16 in binary64, whose registers hold half as many)
        constexpr int RM = sizeof(T) == 4 ? 32 : 16, STEP = sizeof(T) == 4 ? 32 : 16;
        const int64_t ntask = 2 * (npad / RM) - (FWD ? std::min<int64_t>(nbs, npad) : npad - (int64_t)(K - 1) * nbs) / RM;
        const dim3 grid_m((unsigned)std::min<int64_t>(ntask, TRSV_NCRIT + TRSV_NBULK));
        for (int c0 = 0; c0 < m; c0 += STEP) {
            if (c0 > 0 || !ctl_zeroed)
                hipLaunchKernelGGL(k_zero_int, dim3((nctl + 255) / 256), dim3(256), 0, st, ctl, nctl);
            auto go = [&](auto kern) {
                hipLaunchKernelGGL(kern, grid_m, dim3(64 * TRSM_WAVES), 0, st, L, ld, WB, npad, nbs, K, Yin, Zout, ldy,
                                   c0, m, P, ctl, err, tmo);
            };
            if constexpr (sizeof(T) == 4) {
                if (m - c0 > 16) {
                    go(k_trsv_mfma<T, 2, FWD>);
                    continue;
                }
            }
            go(k_trsv_mfma<T, 1, FWD>);
        }
        return;
    }
    if (!ctl_zeroed)
        hipLaunchKernelGGL(k_zero_int, dim3((nctl + 255) / 256), dim3(256), 0, st, ctl, nctl);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(grid), dim3(256), 0, st, L, ld, WB, npad, nbs, K, Yin, Zout, ldy, 0, m, P, ctl,
                           err, ncrit, cdepth, tmo);
    };
    if (m == 1)
        go(k_trsv_blk<T, 1, FWD>);
    else
        go(k_trsv_blk<T, 2, FWD>);
}

template <typename T>
void launch_trsv(const T *L, int64_t ld, const T *WB, int64_t npad, int m, T *Y, T *Z, int64_t ldy, T *P, int *ctl,
                 bool ctl_zeroed, int *err, unsigned long long wait_ticks, hipStream_t st)
{
    // each direction has its own counters (ctl, ctl + trsv_ctl_ints)
    launch_dir<T, true>(L, ld, WB, npad, m, Y, Z, ldy, P, ctl, ctl_zeroed, err, wait_ticks, st);
    launch_dir<T, false>(L, ld, WB, npad, m, Z, Y, ldy, P, ctl + trsv_ctl_ints(npad), ctl_zeroed, err, wait_ticks,
                         st);
}
template void launch_trsv<float>(const float *, int64_t, const float *, int64_t, int, float *, float *, int64_t,
                                 float *, int *, bool, int *, unsigned long long, hipStream_t);
template void launch_trsv<double>(const double *, int64_t, const double *, int64_t, int, double *, double *, int64_t,
                                  double *, int *, bool, int *, unsigned long long, hipStream_t);

}  // namespace spd
