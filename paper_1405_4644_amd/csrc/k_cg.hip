// Conjugate gradients with iterative refinement (Algorithm 2, Section 3.2):
// the binary32 operator A~ (dense, or the band |i - j| <= k of Section 4),
// its product with the search directions, and the binary64 vector steps.
//
// Storage.  Dense A~: binary32, ldt x ldt (ldt = n rounded up to 256, zero
// outside n x n), both triangles, in MFMA fragment order (below) so
// that each product streams it with fully coalesced loads.  Band A~:
// Bd[(d + k) ldt + i] = A~(i, i + d) for d = -k..k (zero where i + d falls
// outside 0..n-1, and in rows n..ldt-1).  Search directions: P (binary64,
// n x m, ld n) and its binary32 rounding Pf (layout of pf_off, zero in rows
// n..ldt-1 and in the padding columns of the last block).
//
// Reductions are deterministic: every kernel that needs a dot product
// writes one partial per workgroup, and its consumers sum them for each
// column in a fixed order (every workgroup of a consumer the same way).
// One CG iteration is three launches (four for the dense 5..32-column
// product, which adds its slice sum): product, x/r update, p update; a band
// of half-width up to CG_FUSE_MAXK takes the p update inside the next
// product: two launches.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "common.h"
#include "internal.h"

namespace {

constexpr int CG_MAXK_BAND = 4096;  // largest half-bandwidth kept in band storage
constexpr int CG_BAND_COLS = 4;     // right-hand sides per workgroup of the band product
constexpr int CG_FUSE_MAXK = 128;   // widest half-band whose product also takes the p step (halo <= 256 rows)

__device__ inline double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
// fixed-order sum of one value per thread over a 256-thread block
__device__ inline double block_sum256(double v, double *red)
{
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[w] = v;
    __syncthreads();
    return ((red[0] + red[1]) + red[2]) + red[3];
}

// A~(j, i) in the dense fragment order (k_cg_dense): column block I = i / 32,
// row block J = j / 16 (512 values, contiguous, blocks of one column block
// consecutive along J); inside a block, value e of the float4 number s of
// lane l, with l = 32 h + i % 32 and j % 16 = 8 h + 4 s + e.  A wave's float4
// load of one (s) half of a block is then 1 KB contiguous, and lane l holds
// exactly the MFMA operand values of row i % 32 at k-slot h.

// Offset of the binary32 direction value (j, c): right-hand sides in blocks
// of W columns (W = m for m <= 4, else 32), each block ldt x W stored with
// the column index inside groups of four consecutive rows:
// ((j / 4) W + c % W) 4 + j % 4.  A lane's four consecutive rows of one
// column are one float4.
__device__ inline int64_t pf_off(int64_t j, int c, int W, int64_t ldt)
{
    return (int64_t)(c / W) * ldt * W + ((j >> 2) * W + (c % W)) * 4 + (j & 3);
}

// dense A~ = fl32(A) in fragment order, zero outside n x n; one 64 x 64
// tile of the symmetric A per workgroup, read along A's columns
__global__ __launch_bounds__(256) void k_cg_dense(const double *__restrict__ A, int64_t lda, int64_t n,
                                                  float *__restrict__ Af, int64_t ldt)
{
    __shared__ float tile[64][65];  // tile[jl][il] = A~(J0 + jl, I0 + il)
    const int64_t I0 = (int64_t)blockIdx.x * 64, J0 = (int64_t)blockIdx.y * 64;
    const int t = threadIdx.x;
    if (J0 >= I0 + 64) {  // every jj > ii: A[jj + ii lda], contiguous along jj
        for (int r = 0; r < 16; ++r) {
            const int il = (t >> 6) + 4 * r, jl = t & 63;
            const int64_t ii = I0 + il, jj = J0 + jl;
            tile[jl][il] = (ii < n && jj < n) ? (float)A[jj + ii * lda] : 0.0f;
        }
    } else if (I0 >= J0 + 64) {  // every ii > jj: A[ii + jj lda], contiguous along ii
        for (int r = 0; r < 16; ++r) {
            const int jl = (t >> 6) + 4 * r, il = t & 63;
            const int64_t ii = I0 + il, jj = J0 + jl;
            tile[jl][il] = (ii < n && jj < n) ? (float)A[ii + jj * lda] : 0.0f;
        }
    } else {  // diagonal tile
        for (int r = 0; r < 16; ++r) {
            const int il = (t >> 6) + 4 * r, jl = t & 63;
            const int64_t ii = I0 + il, jj = J0 + jl;
            float v = 0.0f;
            if (ii < n && jj < n) v = (float)((jj >= ii) ? A[jj + ii * lda] : A[ii + jj * lda]);
            tile[jl][il] = v;
        }
    }
    __syncthreads();
    // the tile is 2 column blocks x 4 row blocks of 512 values
    const int64_t nJ = ldt / 16;
    for (int r = 0; r < 16; ++r) {
        const int f = t + 256 * r;          // 0..4095
        const int blk = f >> 9, w = f & 511;
        const int bi = blk >> 2, bj = blk & 3;
        const int s = w >> 8, lane = (w >> 2) & 63, e = w & 3;
        const int il = bi * 32 + (lane & 31), jl = bj * 16 + (lane >> 5) * 8 + s * 4 + e;
        const int64_t I = (I0 >> 5) + bi, J = (J0 >> 4) + bj;
        Af[(I * nJ + J) * 512 + w] = tile[jl][il];
    }
}

// band A~: Bd[(d + k) ldt + i] = fl32(A(i, i + d)), zero outside the matrix
__global__ __launch_bounds__(256) void k_cg_band(const double *__restrict__ A, int64_t lda, int64_t n, int64_t k,
                                                 float *__restrict__ Bd, int64_t ldt)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t d = (int64_t)blockIdx.y - k;
    if (i >= ldt) return;
    const int64_t j = i + d;
    float v = 0.0f;
    if (i < n && j >= 0 && j < n) v = (float)((i >= j) ? A[i + j * lda] : A[j + i * lda]);
    Bd[(d + k) * ldt + i] = v;
}

// any column of the block [c0, c0 + cnt) still active?
__device__ inline bool any_active(const int *act, int c0, int cnt)
{
    bool a = false;
    for (int c = 0; c < cnt; ++c) a |= act[c0 + c] != 0;
    return a;
}

// z = A~ p for up to 4 right-hand sides on the VALU.  A workgroup owns the
// 32 rows of z of one column block; its four waves split the block's row
// blocks, every lane accumulates row i % 32 over its k-slot's rows, with the
// direction values loaded as broadcast float4s.  The halves and the waves
// are summed in a fixed order; one binary64 partial of p^T z per column.
template <int MB>
__global__ __launch_bounds__(256) void k_cg_mv_valu(const float *__restrict__ Af, int64_t ldt, int64_t n,
                                                    const float *__restrict__ Pf, const double *__restrict__ P,
                                                    double *__restrict__ Z, double *__restrict__ part, int64_t npart,
                                                    const int *__restrict__ act)
{
    __shared__ float red[3][MB][64];
    if (!any_active(act, 0, MB)) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int h = lane >> 5, l32 = lane & 31;
    const int64_t nJ = ldt / 16, jq = nJ / 4;
    const int64_t I = blockIdx.x;
    const float *ab = Af + (I * nJ + w * jq) * 512 + lane * 4;
    // rows J 16 + 8 h + 0..3 and + 4..7 of right-hand side b: float4 number
    // (4 J + 2 h) W + b and the next group
    const float4 *pb = reinterpret_cast<const float4 *>(Pf) + (w * jq * 4 + 2 * h) * MB;
    float acc[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[b] = 0.0f;
#pragma unroll 4
    for (int64_t J = 0; J < jq; ++J) {
        const float4 a0 = *reinterpret_cast<const float4 *>(ab + J * 512);
        const float4 a1 = *reinterpret_cast<const float4 *>(ab + J * 512 + 256);
#pragma unroll
        for (int b = 0; b < MB; ++b) {
            const float4 p0 = pb[J * 4 * MB + b], p1 = pb[J * 4 * MB + MB + b];
            acc[b] += a0.x * p0.x;
            acc[b] += a0.y * p0.y;
            acc[b] += a0.z * p0.z;
            acc[b] += a0.w * p0.w;
            acc[b] += a1.x * p1.x;
            acc[b] += a1.y * p1.y;
            acc[b] += a1.z * p1.z;
            acc[b] += a1.w * p1.w;
        }
    }
#pragma unroll
    for (int b = 0; b < MB; ++b) acc[b] += __shfl_xor(acc[b], 32, 64);
    if (w > 0)
#pragma unroll
        for (int b = 0; b < MB; ++b) red[w - 1][b][lane] = acc[b];
    __syncthreads();
    if (w != 0) return;
    const int64_t i = I * 32 + l32;
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const float zf = ((acc[b] + red[0][b][lane]) + red[1][b][lane]) + red[2][b][lane];
        double pz = 0.0;
        if (h == 0 && i < n) {
            const double z = (double)zf;
            Z[i + (int64_t)b * n] = z;
            pz = P[i + (int64_t)b * n] * z;
        }
        pz = wave_sum(pz);
        if (lane == 0) part[blockIdx.x + (int64_t)b * npart] = pz;
    }
}

// z = A~ p for one right-hand side from A~'s lower triangle: a workgroup takes
// a 256 x 256 tile (IB, JB), JB <= IB, as it is stored, its waves 64 of the
// columns j each.  With a_ij a lane has both terms: z_i += a_ij p_j, in eight
// accumulators (row i % 32 of the tile's eight column blocks) over the wave's
// columns, and z_j += a_ij p_i, in eight (its columns of one row block) over
// the eight column blocks, then over the 32 lanes by halving exchanges.  A
// diagonal tile is read whole, for z_i only.  The tile's sums go to Zp[JB][i]
// and Zp[IB][j] (k_cg_xr adds a row's nb of them in order); one binary64
// partial of p^T z per tile.
// Bound by reading the triangle.  Reading all of A~ (k_cg_mv_valu), a solve at
// n = 10000 took 16.0 ms (80 us a product, 5.0 TB/s), now 8.8; n = 7000 6.7 and
// 5.2 ms, n = 4000 3.89 and 3.23.  From CG_SYM_MIN on: 3072 3.07 and 2.91 ms;
// below it the tiles are too few (2816 2.92 and 2.95, 1529 1.97 and 2.48).
constexpr int64_t CG_SYM_MIN = 3072;
__global__ __launch_bounds__(256) void k_cg_mv_sym(const float *__restrict__ Af, int64_t ldt, int64_t n,
                                                   const float *__restrict__ Pf, const double *__restrict__ P,
                                                   float *__restrict__ Zp, double *__restrict__ part,
                                                   const int *__restrict__ act)
{
    __shared__ float si[4][256], sj[256];
    __shared__ double red[4];
    if (!act[0]) return;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l32 = lane & 31;
    const int64_t q = blockIdx.x;  // q = IB (IB + 1) / 2 + JB
    int64_t IB = (int64_t)((sqrt(8.0 * (double)q + 1.0) - 1.0) * 0.5);
    while (IB * (IB + 1) / 2 > q) --IB;
    while ((IB + 1) * (IB + 2) / 2 <= q) ++IB;
    const int64_t JB = q - IB * (IB + 1) / 2;
    const int64_t nJ = ldt / 16;
    const bool off = IB != JB;
    const float *ab = Af + (IB * 8 * nJ + JB * 16 + 4 * w) * 512 + lane * 4;
    const float *pj = Pf + JB * 256 + 64 * w + 8 * h;
    float pi[8], zi[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        pi[c] = Pf[IB * 256 + 32 * c + l32];
        zi[c] = 0.0f;
    }
#pragma unroll 1
    for (int J = 0; J < 4; ++J) {
        floatx4 a[8][2];
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int e = 0; e < 2; ++e) a[c][e] = *reinterpret_cast<const floatx4 *>(ab + (c * nJ + J) * 512 + 256 * e);
        const floatx4 p[2] = {*reinterpret_cast<const floatx4 *>(pj + 16 * J),
                              *reinterpret_cast<const floatx4 *>(pj + 16 * J + 4)};
        float zj[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) zj[e] = 0.0f;
#pragma unroll
        for (int c = 0; c < 8; ++c)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                zi[c] = fmaf(a[c][e >> 2][e & 3], p[e >> 2][e & 3], zi[c]);
                zj[e] = fmaf(a[c][e >> 2][e & 3], pi[c], zj[e]);
            }
        // over the 32 lanes: bit 4 of the lane takes columns 4 .. 7 or 0 .. 3,
        // bits 3 and 2 halve again
#pragma unroll
        for (int d = 16, k = 4; d >= 4; d >>= 1, k >>= 1)
#pragma unroll
            for (int e = 0; e < k; ++e) {
                const bool up = (l32 & d) != 0;
                const float keep = up ? zj[e + k] : zj[e], send = up ? zj[e] : zj[e + k];
                zj[e] = keep + __shfl_xor(send, d, 64);
            }
        float z = zj[0];
        z += __shfl_xor(z, 2, 64);
        z += __shfl_xor(z, 1, 64);
        if ((l32 & 3) == 0) sj[64 * w + 16 * J + 8 * h + (l32 >> 2)] = z;
    }
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        zi[c] += __shfl_xor(zi[c], 32, 64);
        if (h == 0) si[w][32 * c + l32] = zi[c];
    }
    __syncthreads();
    const int64_t i = IB * 256 + tid, j = JB * 256 + tid;
    const float vi = ((si[0][tid] + si[1][tid]) + si[2][tid]) + si[3][tid], vj = sj[tid];
    Zp[JB * ldt + i] = vi;
    if (off) Zp[IB * ldt + j] = vj;
    double pz = (i < n) ? P[i] * (double)vi : 0.0;
    if (off) pz += P[j] * (double)vj;  // (j < n: the tile is not a last column's)
    pz = block_sum256(pz, red);
    if (tid == 0) part[q] = pz;
}

// z = A~ p for 5..32 right-hand sides per launch row (blockIdx.y picks the
// block of 32) on v_mfma_f32_32x32x2f32, split along k over CG_KS slices.
// Workgroup b owns the 32 rows of z of column block b / CG_KS and the
// row-block slice b % CG_KS; its four waves split the slice.  Per row block a
// lane loads two float4s of A~ (its MFMA A-operand values for k-slot h) and
// the matching two float4s of the directions (B operand: column c =
// lane % 32, the same eight rows), both fully coalesced.  Workgroups are
// dealt to the eight XCDs round-robin, so with CG_KS = 8 every XCD streams
// one eighth of the binary32 directions, which fits its L2, instead of all
// of them (9 MB at n = 70000, 32 columns).  Each slice writes its binary32
// partial z to Zp[slice][c][i]; k_cg_mv_ksum adds the slices in order.
constexpr int CG_KS = 8;
__global__ __launch_bounds__(256) void k_cg_mv_mfma_ks(const float *__restrict__ Af, int64_t ldt, int64_t n, int m,
                                                       const float *__restrict__ Pf, float *__restrict__ Zp,
                                                       const int *__restrict__ act)
{
    __shared__ float red[3][16][64];
    const int c0 = blockIdx.y * 32;
    const int mc = min(32, m - c0);
    if (!any_active(act, c0, mc)) return;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int h = lane >> 5, l32 = lane & 31;
    const int64_t nJ = ldt / 16;
    const int64_t I = blockIdx.x / CG_KS, sl = blockIdx.x % CG_KS;
    const int64_t js = nJ * sl / CG_KS, je = nJ * (sl + 1) / CG_KS;
    const int64_t jb = js + (je - js) * w / 4, jend = js + (je - js) * (w + 1) / 4;
    const float *ab = Af + (I * nJ) * 512 + lane * 4;
    const float4 *pb = reinterpret_cast<const float4 *>(Pf + (int64_t)blockIdx.y * ldt * 32) + (2 * h) * 32 + l32;
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll 2
    for (int64_t J = jb; J < jend; ++J) {
        const float4 a0 = *reinterpret_cast<const float4 *>(ab + J * 512);
        const float4 a1 = *reinterpret_cast<const float4 *>(ab + J * 512 + 256);
        const float4 b0 = pb[J * 128], b1 = pb[J * 128 + 32];
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, b0.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, b0.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.z, b0.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.w, b0.w, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, b1.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, b1.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.z, b1.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.w, b1.w, acc, 0, 0, 0);
    }
    if (w > 0)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[w - 1][r][lane] = acc[r];
    __syncthreads();
    if (w != 0) return;
    const int c = c0 + l32;
    if (l32 >= mc) return;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float s = ((acc[r] + red[0][r][lane]) + red[1][r][lane]) + red[2][r][lane];
        const int64_t i = I * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (i < n) Zp[(sl * m + c) * n + i] = s;
    }
}

// z = sum of the CG_KS slices (binary32, slice order), widened; one partial
// of p^T z per workgroup and column (blockIdx.y = column)
__global__ __launch_bounds__(256) void k_cg_mv_ksum(int64_t n, int m, const float *__restrict__ Zp,
                                                    const double *__restrict__ P, double *__restrict__ Z,
                                                    double *__restrict__ part, int64_t npart,
                                                    const int *__restrict__ act)
{
    __shared__ double red[4];
    const int c = blockIdx.y;
    if (!act[c]) return;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double pz = 0.0;
    if (i < n) {
        float s = Zp[(int64_t)c * n + i];
#pragma unroll
        for (int q = 1; q < CG_KS; ++q) s += Zp[((int64_t)q * m + c) * n + i];
        const double z = (double)s;
        Z[i + (int64_t)c * n] = z;
        pz = P[i + (int64_t)c * n] * z;
    }
    pz = block_sum256(pz, red);
    if (threadIdx.x == 0) part[blockIdx.x + (int64_t)c * npart] = pz;
}

// z = A~ p on the band, a thread per row, workgroup (x, y) the rows
// [256 x, 256 x + 256) of CB right-hand sides: their directions over those
// rows and the k-wide halo, rounded to binary32, are staged in LDS column by
// column (pitch span + 1), and each band value is applied to all of them.
// With FUSE the step p = r + beta p of the iteration before is taken here
// (each workgroup forms its rows and its halo from R and Pin, and writes its
// rows to Pout, another buffer, since its neighbours still read Pin), and
// block (0, y) advances the columns' scalar state from slot par ^ 1 to slot
// par: one launch less per iteration.  Only for halos up to the tile's own
// rows (CG_FUSE_MAXK); wider ones would form p many times over.
//
// Bound by latency: the product at n = 12000, half-width 16 and 32 columns
// moves 20 MB.  All 32 columns in one workgroup (47 workgroups there, a fifth
// of the chip) took 62.4 us, and the p step 5.5 us of its own; with four
// columns per workgroup and the p step inside, both take 8.9 us together.
template <int CB, bool FUSE>
__global__ __launch_bounds__(256) void k_cg_mv_band(const float *__restrict__ Bd, int64_t ldt, int64_t n, int64_t k,
                                                    int m, const double *__restrict__ R,
                                                    const double *__restrict__ Pin, double *__restrict__ Pout,
                                                    double *__restrict__ Z, double *__restrict__ part, int64_t npart,
                                                    const double *__restrict__ rrp, int64_t nrr,
                                                    double *__restrict__ sc, int par, int *__restrict__ act,
                                                    int *__restrict__ cnt, int max_inner)
{
    extern __shared__ float pl[];  // CB x (span + 1)
    __shared__ double redc[4 * CB];
    __shared__ double beta[CB];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + t;
    const int cb = blockIdx.y * CB, nc = min(CB, m - cb);
    const int pitch = 256 + 2 * (int)k + 1;
    // columns taking part: those active when the iteration's direction was due
    const int *a_cur = act + (int64_t)(FUSE ? par ^ 1 : par) * m;
    bool on[CB], any = false;
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        on[c] = c < nc && a_cur[cb + c] != 0;
        any |= on[c];
    }
    if constexpr (FUSE) {
        const double *rho = sc + (int64_t)(par ^ 1) * m;
        double *rho_next = sc + (int64_t)par * m;
        const double *thr = sc + 2 * (int64_t)m;
        int *a_next = act + (int64_t)par * m;
        // rho' = r^T r from its partials, a wave per column (fixed order)
        for (int c = w; c < nc; c += 4) {
            double rr = 0.0;
            if (a_cur[cb + c])
                for (int64_t q = lane; q < nrr; q += 64) rr += rrp[q + (int64_t)(cb + c) * nrr];
            rr = wave_sum(rr);
            if (lane == 0) {
                const double rc = rho[cb + c];
                beta[c] = rr / rc;
                if (blockIdx.x == 0) {  // the column's state into the next slot
                    if (a_cur[cb + c]) {
                        const int q = cnt[cb + c] + 1;
                        cnt[cb + c] = q;
                        rho_next[cb + c] = rr;
                        a_next[cb + c] = (q < max_inner && rr > thr[cb + c]) ? 1 : 0;
                    } else {
                        rho_next[cb + c] = rc;
                        a_next[cb + c] = 0;
                    }
                }
            }
        }
        if (!any) return;
        __syncthreads();
    } else {
        if (!any) return;
    }
    // own rows, then the halo (k rows on either side)
    double p[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        p[c] = 0.0;
        if (on[c] && i < n) {
            const int64_t o = i + (int64_t)(cb + c) * n;
            p[c] = Pin[o];
            if constexpr (FUSE) {
                p[c] = R[o] + beta[c] * p[c];
                Pout[o] = p[c];
            }
        }
        pl[c * pitch + k + t] = (float)p[c];
    }
    for (int h = t; h < 2 * (int)k; h += 256) {
        const int off = h < k ? h : 256 + h;  // position in the staged rows
        const int64_t j = i0 - k + off;
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            double v = 0.0;
            if (on[c] && j >= 0 && j < n) {
                const int64_t o = j + (int64_t)(cb + c) * n;
                v = Pin[o];
                if constexpr (FUSE) v = R[o] + beta[c] * v;
            }
            pl[c * pitch + off] = (float)v;
        }
    }
    __syncthreads();
    float acc[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) acc[c] = 0.0f;
    if (i < n) {
        const float *bd = Bd + i;
        const float *col = pl + t;
#pragma unroll 16
        for (int d = 0; d <= 2 * (int)k; ++d) {
            const float a = bd[(int64_t)d * ldt];
#pragma unroll
            for (int c = 0; c < CB; ++c) acc[c] += a * col[c * pitch + d];
        }
    }
    // z, and p^T z per column: wave sums, then the four waves in order
#pragma unroll
    for (int c = 0; c < CB; ++c) {
        double pz = 0.0;
        if (on[c] && i < n) {
            const double z = (double)acc[c];
            Z[i + (int64_t)(cb + c) * n] = z;
            pz = p[c] * z;
        }
        pz = wave_sum(pz);
        if (lane == 0) redc[w * CB + c] = pz;
    }
    __syncthreads();
    if (t < nc)
        part[blockIdx.x + (int64_t)(cb + t) * npart] = ((redc[t] + redc[CB + t]) + redc[2 * CB + t]) + redc[3 * CB + t];
}

// P = R, Pf = fl32(R) (dense products) and a partial of r^T r, for the columns starting a
// phase (blockIdx.y = column)
__global__ __launch_bounds__(256) void k_cg_start(int64_t n, int m, int W, const double *__restrict__ R,
                                                  double *__restrict__ P, float *__restrict__ Pf, int64_t ldt,
                                                  double *__restrict__ part, int64_t npart, const int *__restrict__ go)
{
    __shared__ double red[4];
    const int b = blockIdx.y;
    if (!go[b]) return;
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = (int64_t)blockIdx.x * 1024 + u * 256 + threadIdx.x;
        if (i < n) {
            const double r = R[i + (int64_t)b * n];
            P[i + (int64_t)b * n] = r;
            if (Pf) Pf[pf_off(i, b, W, ldt)] = (float)r;
            s += r * r;
        }
    }
    s = block_sum256(s, red);
    if (threadIdx.x == 0) part[blockIdx.x + (int64_t)b * npart] = s;
}

// fixed-order sum of column b's npart partials; the same value in every block
__device__ inline double sum_parts(const double *part, int64_t npart, int b, double *red)
{
    double s = 0.0;
    for (int64_t q = threadIdx.x; q < npart; q += 256) s += part[q + (int64_t)b * npart];
    return block_sum256(s, red);
}

// Scalar state per column, double-buffered by iteration parity `par`:
// rho[par][b] = r^T r of the current iterate, act[par][b] = column still
// iterating; thr[b] = inner_tol^2 rho_0 and cnt[b] = products this phase.
// Iteration `par` reads slot par and its last kernel writes slot par ^ 1, so
// no kernel reads a slot that it also writes.

// alpha = rho / p^T z (from the product's partials, summed identically in
// every block), x += alpha p, r -= alpha z, and a partial of the new r^T r
// (blockIdx.y = column)
template <bool SYM>
__global__ __launch_bounds__(256) void k_cg_xr(int64_t n, int m, const double *__restrict__ pzp, int64_t npz,
                                               const double *__restrict__ rho, const double *__restrict__ P,
                                               const double *__restrict__ Z, const float *__restrict__ Zp, int64_t ldt,
                                               double *__restrict__ X, int64_t ldx,
                                               double *__restrict__ R, double *__restrict__ part, int64_t npart,
                                               const int *__restrict__ act)
{
    __shared__ double red[4];
    const int b = blockIdx.y;
    if (!act[b]) return;
    float zs[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (SYM) {
        // (ldt is a multiple of 256: a thread's last row may be past it, and
        // then takes the last one's)
        const float *zp[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) zp[u] = Zp + min((int64_t)blockIdx.x * 1024 + u * 256 + threadIdx.x, ldt - 1);
        const int64_t nb = ldt / 256;
#pragma unroll 8
        for (int64_t k = 0; k < nb; ++k)
#pragma unroll
            for (int u = 0; u < 4; ++u) zs[u] += zp[u][k * ldt];
    }
    const double al = rho[b] / sum_parts(pzp, npz, b, red);
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = (int64_t)blockIdx.x * 1024 + u * 256 + threadIdx.x;
        if (i < n) {
            X[i + (int64_t)b * ldx] += al * P[i + (int64_t)b * n];
            const double z = SYM ? (double)zs[u] : Z[i + (int64_t)b * n];
            const double r = R[i + (int64_t)b * n] - al * z;
            R[i + (int64_t)b * n] = r;
            s += r * r;
        }
    }
    s = block_sum256(s, red);
    if (threadIdx.x == 0) part[blockIdx.x + (int64_t)b * npart] = s;
}

// rho' = r^T r (partials of k_cg_xr), beta = rho' / rho, p = r + beta p (Pin
// to P, which may be the same buffer), Pf = fl32(p) for dense products
// (blockIdx.y = column); block (0, b) advances the column's
// state into slot par ^ 1: rho', ++cnt, act' = cnt < max_inner && rho' > thr
__global__ __launch_bounds__(256) void k_cg_p(int64_t n, int m, int W, const double *__restrict__ rrp, int64_t nrr,
                                              double *__restrict__ sc, int par, const double *__restrict__ R,
                                              const double *Pin, double *P, float *__restrict__ Pf, int64_t ldt,
                                              int *__restrict__ act, int *__restrict__ cnt, int max_inner)
{
    __shared__ double red[4];
    const int b = blockIdx.y;
    const double *rho = sc + (int64_t)par * m;
    double *rho_next = sc + (int64_t)(par ^ 1) * m;
    const double *thr = sc + 2 * (int64_t)m;
    const int *a_cur = act + (int64_t)par * m;
    int *a_next = act + (int64_t)(par ^ 1) * m;
    const bool lead = blockIdx.x == 0 && threadIdx.x == 0;
    if (!a_cur[b]) {
        if (lead) {
            a_next[b] = 0;
            rho_next[b] = rho[b];
        }
        return;
    }
    const double rr = sum_parts(rrp, nrr, b, red);
    const double be = rr / rho[b];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int64_t i = (int64_t)blockIdx.x * 1024 + u * 256 + threadIdx.x;
        if (i < n) {
            const double p = R[i + (int64_t)b * n] + be * Pin[i + (int64_t)b * n];
            P[i + (int64_t)b * n] = p;
            if (Pf) Pf[pf_off(i, b, W, ldt)] = (float)p;
        }
    }
    if (lead) {
        rho_next[b] = rr;
        const int c = cnt[b] + 1;
        cnt[b] = c;
        a_next[b] = (c < max_inner && rr > thr[b]) ? 1 : 0;
    }
}

// Start of a phase (one block per column): rho = r^T r into slot 0,
// thr = inner_tol^2 rho, cnt = 0, act[0] = go && max_inner > 0 && rho > thr
__global__ __launch_bounds__(256) void k_cg_begin(const double *__restrict__ part, int64_t npart,
                                                  double *__restrict__ sc, int *__restrict__ act,
                                                  const int *__restrict__ go, int *__restrict__ cnt,
                                                  double inner_tol2, int max_inner, int m)
{
    __shared__ double red[4];
    const int b = blockIdx.x;
    if (!go[b]) {
        if (threadIdx.x == 0) {
            act[b] = 0;
            cnt[b] = 0;
        }
        return;
    }
    const double s = sum_parts(part, npart, b, red);
    if (threadIdx.x != 0) return;
    sc[b] = s;
    sc[2 * (int64_t)m + b] = inner_tol2 * s;
    cnt[b] = 0;
    act[b] = (max_inner > 0 && s > inner_tol2 * s) ? 1 : 0;
}

}  // namespace

namespace spd {

int64_t cg_ldt(int64_t n) { return ((std::max<int64_t>(n, 1) + 255) / 256) * 256; }
bool cg_sym(int64_t ldt, int m) { return m == 1 && ldt >= CG_SYM_MIN; }
int cg_band_ok(int64_t k) { return k >= 0 && k <= CG_MAXK_BAND; }

void launch_cg_dense(const double *A, int64_t lda, int64_t n, float *At, int64_t ldt, hipStream_t st)
{
    dim3 g((unsigned)(ldt / 64), (unsigned)(ldt / 64));
    hipLaunchKernelGGL(k_cg_dense, g, dim3(256), 0, st, A, lda, n, At, ldt);
}

void launch_cg_band(const double *A, int64_t lda, int64_t n, int64_t k, float *Bd, int64_t ldt, hipStream_t st)
{
    dim3 g((unsigned)(ldt / 256), (unsigned)(2 * k + 1));
    hipLaunchKernelGGL(k_cg_band, g, dim3(256), 0, st, A, lda, n, k, Bd, ldt);
}

int cg_pf_width(int m) { return (m <= 4) ? std::max(m, 1) : 32; }
int64_t cg_pf_elems(int64_t ldt, int m)
{
    const int W = cg_pf_width(m);
    return (int64_t)((m + W - 1) / W) * W * ldt;
}

int64_t cg_mv_parts(int64_t n, int64_t ldt, int64_t k, int m)
{
    if (k >= 0) return (n + 255) / 256;
    if (cg_sym(ldt, m)) return (ldt / 256) * (ldt / 256 + 1) / 2;
    return (m <= 4) ? ldt / 32 : (n + 255) / 256;
}

// (the products of 1, of 2 to 4 and of more columns have layouts of their own)
int64_t cg_part_elems(int64_t n, int64_t ldt, int64_t k, int m)
{
    int64_t e = 0;
    for (int q : {1, 2, 3, 4, m})
        if (q <= m) e = std::max(e, cg_mv_parts(n, ldt, k, q) * q);
    return e;
}

int64_t cg_zp_elems(int64_t n, int64_t ldt, int m)
{
    return std::max((m > 4) ? (int64_t)CG_KS * m * n : 0, cg_sym(ldt, 1) ? ldt / 256 * ldt : 0);
}

// columns per workgroup of the band product: four, so that a few dozen row
// blocks with several right-hand sides still spread over the chip; one where
// four columns' rows and halo exceed the 64 KB of LDS a launch may ask for
static int cg_band_cols(int64_t k, int m)
{
    return (m > 1 && (256 + 2 * k + 1) * CG_BAND_COLS * (int64_t)sizeof(float) + 1024 <= 65536) ? CG_BAND_COLS : 1;
}

bool cg_band_fused(int64_t k) { return k <= CG_FUSE_MAXK; }

void launch_cg_mv_band(const float *Bd, int64_t ldt, int64_t n, int64_t k, int m, const double *R, const double *Pin,
                       double *Pout, double *Z, double *part, int64_t npart, const double *rrp, int64_t nrr,
                       double *sc, int par, int *act, int *cnt, int max_inner, hipStream_t st)
{
    const int CB = cg_band_cols(k, m);
    const dim3 g((unsigned)((n + 255) / 256), (unsigned)((m + CB - 1) / CB));
    const size_t lds = (size_t)(256 + 2 * k + 1) * CB * sizeof(float);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, g, dim3(256), lds, st, Bd, ldt, n, k, m, R, Pin, Pout, Z, part, npart, rrp, nrr, sc,
                           par, act, cnt, max_inner);
    };
    if (CB == 1)
        Pout ? go(k_cg_mv_band<1, true>) : go(k_cg_mv_band<1, false>);
    else
        Pout ? go(k_cg_mv_band<CG_BAND_COLS, true>) : go(k_cg_mv_band<CG_BAND_COLS, false>);
}

void launch_cg_mv(const float *At, int64_t ldt, int64_t n, int m, const float *Pf, const double *P,
                  double *Z, double *part, int64_t npart, const int *act, float *Zp, hipStream_t st)
{
    const dim3 blk(256), g((unsigned)(ldt / 32));
    if (cg_sym(ldt, m)) {
        hipLaunchKernelGGL(k_cg_mv_sym, dim3((unsigned)npart), blk, 0, st, At, ldt, n, Pf, P, Zp, part, act);
        return;
    }
    switch (m) {
    case 1: hipLaunchKernelGGL(k_cg_mv_valu<1>, g, blk, 0, st, At, ldt, n, Pf, P, Z, part, npart, act); break;
    case 2: hipLaunchKernelGGL(k_cg_mv_valu<2>, g, blk, 0, st, At, ldt, n, Pf, P, Z, part, npart, act); break;
    case 3: hipLaunchKernelGGL(k_cg_mv_valu<3>, g, blk, 0, st, At, ldt, n, Pf, P, Z, part, npart, act); break;
    case 4: hipLaunchKernelGGL(k_cg_mv_valu<4>, g, blk, 0, st, At, ldt, n, Pf, P, Z, part, npart, act); break;
    default:
        hipLaunchKernelGGL(k_cg_mv_mfma_ks, dim3((unsigned)(ldt / 32 * CG_KS), (unsigned)((m + 31) / 32)), blk, 0, st,
                           At, ldt, n, m, Pf, Zp, act);
        hipLaunchKernelGGL(k_cg_mv_ksum, dim3((unsigned)((n + 255) / 256), (unsigned)m), blk, 0, st, n, m, Zp, P, Z,
                           part, npart, act);
    }
}

int64_t cg_vec_parts(int64_t n) { return std::max<int64_t>((n + 1023) / 1024, 1); }

void launch_cg_start(int64_t n, int m, const double *R, double *P, float *Pf, int64_t ldt, double *part,
                     int64_t npart, const int *go, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_start, dim3((unsigned)npart, (unsigned)m), dim3(256), 0, st, n, m, cg_pf_width(m), R, P,
                       Pf, ldt, part, npart, go);
}

void launch_cg_xr(int64_t n, int m, const double *pzp, int64_t npz, const double *sc, int par, const double *P,
                  const double *Z, const float *Zp, int64_t ldt, double *X, int64_t ldx, double *R, double *part,
                  int64_t npart, const int *act, hipStream_t st)
{
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)npart, (unsigned)m), dim3(256), 0, st, n, m, pzp, npz,
                           sc + (int64_t)par * m, P, Z, Zp, ldt, X, ldx, R, part, npart, act + (int64_t)par * m);
    };
    Zp && cg_sym(ldt, m) ? go(k_cg_xr<true>) : go(k_cg_xr<false>);
}

void launch_cg_p(int64_t n, int m, const double *rrp, int64_t nrr, double *sc, int par, const double *R,
                 const double *Pin, double *P, float *Pf, int64_t ldt, int *act, int *cnt, int max_inner,
                 hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_p, dim3((unsigned)cg_vec_parts(n), (unsigned)m), dim3(256), 0, st, n, m, cg_pf_width(m),
                       rrp, nrr, sc, par, R, Pin, P, Pf, ldt, act, cnt, max_inner);
}

void launch_cg_begin(const double *part, int64_t npart, double *sc, int *act, const int *go, int *cnt,
                     double inner_tol2, int max_inner, int m, hipStream_t st)
{
    hipLaunchKernelGGL(k_cg_begin, dim3((unsigned)m), dim3(256), 0, st, part, npart, sc, act, go, cnt, inner_tol2,
                       max_inner, m);
}

}  // namespace spd
