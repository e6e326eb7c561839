// Steps a7-a9 (Eqs. epsGG, Wq):
//   eps_GG'(w)   = delta_GG' - v^1/2_G chi_GG'(w) v^1/2_G',  v^1/2_G = sqrt(4 pi/Omega)/|q+G|
//   eps^-1(w)    by in-place Gauss-Jordan elimination with partial (row)
//                pivoting, blocked, all frequencies of a q-point batched,
//                FP64 throughout
//   W_GG'(w)     = HA * v^1/2_G eps^-1_GG'(w) v^1/2_G'   (eV)
//
// Elimination step c (per matrix): pick the row r >= c of largest |a_rc| (the
// lowest of those within 2^-40 of it), swap rows r and c, scale row c by
// 1/a_cc (leaving 1/a_cc in place), and subtract a_ic * row c from every other
// row i (leaving -a_ic/a_cc in column c).  After the last step the recorded row swaps are undone as column swaps
// in reverse order, which leaves A^-1 in place.
//
// Blocked form: the steps of a panel of columns K = [c0, c0 + nb) are run on
// the panel's columns only (after the full-row swaps), and the other columns
// R are brought up to date afterwards in one pass.  The steps on K act on the
// matrix as the sweep on block K: with P the panel columns after the panel
// steps (rows K: A_KK^-1, other rows: -A_OK A_KK^-1) and A_KR the pivot rows
// of R before the panel, the updated R columns are
//     A[:, R] = P A_KR + (rows outside K: A[:, R] as they were),
// a complex matrix product with an inner dimension of nb, run on the FP64
// matrix cores.  The arithmetic is that of the unblocked steps regrouped, and
// the pivots are the same.
//
// eps is dimensionless with a unit-scale diagonal, so a pivot below
// kPivotFloor (a condition number beyond ~1e13, where an FP64 inverse has no
// correct digits left) is reported as singular; a non-finite pivot as a
// non-finite input.
#include <cmath>

#include "fft_lds.h"

namespace rp {

namespace {

constexpr double kPivotFloor = 1e-13;

// vs[i] = sqrt(4 pi / Omega) / |q + G_i|; with head set, the q -> 0 form:
// |q + G| = 0 (G = 0) takes sqrt(4 pi / Omega), the q factor being in chi
__global__ void k_vsqrt(int ng, const int *g, double r0, double r1, double r2, double r3, double r4,
                        double r5, double r6, double r7, double r8, double q1, double q2, double q3,
                        double pref, int head, double *vs, int *flag)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ng) return;
    const double f1 = q1 + g[3 * i], f2 = q2 + g[3 * i + 1], f3 = q3 + g[3 * i + 2];
    const double x = f1 * r0 + f2 * r3 + f3 * r6;
    const double y = f1 * r1 + f2 * r4 + f3 * r7;
    const double z = f1 * r2 + f2 * r5 + f3 * r8;
    const double qg = sqrt(x * x + y * y + z * z);
    if (head && qg == 0.0) {
        vs[i] = pref;
        return;
    }
    vs[i] = pref / qg;
    if (!(qg > 0.0)) atomicOr(flag, kFlagNonFinite);
}

__global__ void k_eps(int nfreq, int ng, const double *vs, const double2 *chi, double2 *eps, int *flag)
{
    const long n2 = (long)ng * ng;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n2 * nfreq) return;
    const long e = t % n2;
    const int g = (int)(e / ng), h = (int)(e - (long)g * ng);
    const double s = vs[g] * vs[h];
    const double2 c = chi[t];
    if (!isfinite(c.x) || !isfinite(c.y)) atomicOr(flag, kFlagNonFinite);
    eps[t] = make_double2((g == h ? 1.0 : 0.0) - s * c.x, -s * c.y);
}

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kGjNb = 64;            // panel width

// The panel being worked on sits in a buffer of its own, column by column:
// pb [f][64][ng] (column c0 + j, row i at j ng + i).  Its steps go down columns,
// and in the row-major matrix each element of a column is a line (and, for
// N = 1500, a page) of its own.

// Panel [0, nb) of the matrices into pb; one workgroup per 64 rows.
__global__ void __launch_bounds__(256)
k_gj_first(int ng, int nb, const double2 *a, double2 *pb)
{
    __shared__ double2 t[16][64 + 1];
    const int f = blockIdx.y, tid = threadIdx.x, r0 = blockIdx.x * 64;
    const double2 *A = a + (long)f * ng * ng;
    double2 *B = pb + (long)f * kGjNb * ng;
    for (int k0 = 0; k0 < nb; k0 += 16) {
        for (int e = tid; e < 64 * 16; e += 256) {
            const int r = e >> 4, k = e & 15;
            if (r0 + r < ng && k0 + k < nb) t[k][r] = A[(long)(r0 + r) * ng + k0 + k];
        }
        __syncthreads();
        for (int e = tid; e < 64 * 16; e += 256) {
            const int k = e >> 6, r = e & 63;
            if (r0 + r < ng && k0 + k < nb) B[(long)(k0 + k) * ng + r0 + r] = t[k][r];
        }
        __syncthreads();
    }
}

// Columns [cs, cs + wc) of panel [c0, c0 + nb), wc <= W: the pivoted steps, one
// workgroup per matrix with the N x wc block in registers (thread t holds rows
// t + NT q, q < R).  Then the steps' row swaps on the panel's other columns,
// whose pivot rows go to rkp [f][W][64] for the update of those columns
// (k_gj_inner).
//
// What bounds it is the chain of N steps on one CU per matrix, each a search
// over a column, a workgroup barrier and one row update: about 2 us a step for
// N = 1500, against 16 us for a search launch and an elimination launch over
// the whole panel per step.  More columns per call mean fewer calls (each also
// reads and writes its columns and updates the panel's others, about 15 us
// together), as many as the registers hold: see launch_invert.  Inversions:
// 20 x 1500: 38.2 -> 20.9 ms, 4 x 6000: 258 -> 206 ms, 16 x 300: 3.2 -> 1.1 ms,
// 10 x 89: 0.92 -> 0.35 ms (eps and W included).
//
// The pivot is the row of largest modulus: its square with the last 13 bits
// replaced by 8191 - row is a key whose maximum is the pivot, the lower row on a
// tie of the others (a non-finite entry, or one beyond 1e154, counts as the
// largest double; a non-finite one is reported when it is used).  |re| + |im|
// as the key saves an operation per row and step (1500 x 20: 17.92 against
// 17.97 ms), but can take a pivot below the floor where another row holds one
// above it.
template <int CTRL, int ROWS> __device__ __forceinline__ double dpp_max(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
    return fmax(v, __longlong_as_double((long long)hi << 32 | (unsigned)lo));
}

// largest of a row of 16 lanes' non-negative keys, in its last lane
__device__ __forceinline__ double row_max(double v)
{
    v = dpp_max<0x111, 0xf>(v);   // row_shr 1, 2, 4, 8
    v = dpp_max<0x112, 0xf>(v);
    v = dpp_max<0x114, 0xf>(v);
    return dpp_max<0x118, 0xf>(v);
}

template <int LANE> __device__ __forceinline__ double read_lane(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, LANE), hi = __builtin_amdgcn_readlane((int)(b >> 32), LANE);
    return __longlong_as_double((long long)hi << 32 | (unsigned)lo);
}

__device__ __forceinline__ int key_row(double key) { return 8191 - (int)(__double_as_longlong(key) & 8191); }

template <int R, int W, int NT>
__global__ void __launch_bounds__(NT)
k_gj_panel(int ng, int c0, int nb, int cs, int wc, double2 *pb, double2 *rkp, int *piv, int *flag)
{
    constexpr int NW = NT / 64;
    // two sets, used in turn: a step needs one barrier
    __shared__ double sKey[2][NW];
    __shared__ double2 sCand[2][NW][W], sC[2][W];   // each wave's candidate row, and row c
    __shared__ int sPiv[W];
    const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double2 *B = pb + (long)f * kGjNb * ng;
    double2 v[R][W];
#pragma unroll
    for (int j = 0; j < W; j++)
#pragma unroll
        for (int q = 0; q < R; q++) {
            const int i = tid + q * NT;
            v[q][j] = i < ng && j < wc ? B[(long)(cs - c0 + j) * ng + i] : make_double2(0.0, 0.0);
        }
    // One loop body for every step (unrolled, the code is fetched as slowly as
    // the steps run): the step's column is always v[.][0], and the columns move
    // down by one with each step, so that W of them leave every one in place.
#pragma unroll 1
    for (int s = 0; s < W; s++) {
        if (s >= wc) {
#pragma unroll
            for (int q = 0; q < R; q++) {
                const double2 first = v[q][0];
#pragma unroll
                for (int j = 0; j + 1 < W; j++) v[q][j] = v[q][j + 1];
                v[q][W - 1] = first;
            }
            continue;
        }
        const int c = cs + s, set = s & 1;
        double key = 0.0;
#pragma unroll
        for (int q = 0; q < R; q++) {
            const int i = tid + q * NT;
            const double m = fmin(v[q][0].x * v[q][0].x + v[q][0].y * v[q][0].y, 1.79e308);   // NaN and infinity: 1.79e308
            const double k = __longlong_as_double((__double_as_longlong(m) & ~8191ll) | (8191 - i));
            key = fmax(key, i >= c && i < ng ? k : 0.0);
        }
        key = dpp_max<0x142, 0xa>(row_max(key));   // row_bcast 15 and 31: across the rows
        key = read_lane<63>(dpp_max<0x143, 0xc>(key));
        const int mine = key_row(key);
#pragma unroll
        for (int q = 0; q < R; q++) {
            if (tid + q * NT == mine)
#pragma unroll
                for (int j = 0; j < W; j++) sCand[set][wave][j] = v[q][j];
            if (tid + q * NT == c)
#pragma unroll
                for (int j = 0; j < W; j++) sC[set][j] = v[q][j];
        }
        if (lane == 0) sKey[set][wave] = key;
        __syncthreads();
        const int r = key_row(read_lane<15>(row_max(sKey[set][lane % NW])));
        const double2 *sP = sCand[set][(r % NT) >> 6];
        const double2 p = sP[0];
        const double den = p.x * p.x + p.y * p.y, rd = 1.0 / den;
        const double2 ip = make_double2(p.x * rd, -p.y * rd);
        if (tid == 0) {
            sPiv[s] = r;
            piv[(long)f * ng + c] = r;
            if (!(den > 4.0 * kPivotFloor * kPivotFloor) || !isfinite(den)) {
                const double m = hypot(p.x, p.y);
                if (!isfinite(m)) atomicOr(flag, kFlagNonFinite);
                else if (!(m > kPivotFloor)) atomicOr(flag, kFlagZeroPivot);
            }
        }
        // row c takes the pivot row times 1/p (1/p itself in column c); the
        // others, row r now holding the former row c, lose their multiple of it
#pragma unroll
        for (int q = 0; q < R; q++) {
            const int i = tid + q * NT;
            if (i == r && r != c)
#pragma unroll
                for (int j = 0; j < W; j++) v[q][j] = sC[set][j];
            if (i == c) {
#pragma unroll
                for (int j = 1; j < W; j++) v[q][j - 1] = cmul(sP[j], ip);
                v[q][W - 1] = ip;
            } else {
                const double2 m = cmul(v[q][0], ip);
#pragma unroll
                for (int j = 1; j < W; j++) v[q][j - 1] = csub(v[q][j], cmul(m, sP[j]));
                v[q][W - 1] = make_double2(-m.x, -m.y);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < W; j++)
#pragma unroll
        for (int q = 0; q < R; q++) {
            const int i = tid + q * NT;
            if (i < ng && j < wc) B[(long)(cs - c0 + j) * ng + i] = v[q][j];
        }
    __syncthreads();
    // the swaps on the panel's other columns: rows cs + s and sPiv[s] (some
    // twice, with the same values), each read where the swaps took it from
    constexpr int PER = (2 * W * kGjNb + NT - 1) / NT;
    double2 x[PER];
    int dst[PER];
    const int slot = tid % (2 * W);
    int row = slot < W ? cs + slot : cs;
    if (slot >= W && slot - W < wc) row = sPiv[slot - W];
    // past the last step, or a pivot from the block's own rows
    const bool moves = slot < W ? slot < wc : row >= cs + wc;
    int src = row;
    for (int s = wc - 1; s >= 0; s--) {
        const int r = sPiv[s];
        src = src == cs + s ? r : src == r ? cs + s : src;
    }
#pragma unroll
    for (int e = 0; e < PER; e++) {
        const int j = (tid + e * NT) / (2 * W), col = c0 + j;
        dst[e] = -1;
        if (!moves || j >= nb || (col >= cs && col < cs + wc)) continue;
        dst[e] = row;
        x[e] = B[(long)j * ng + src];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; e++) {
        const int j = (tid + e * NT) / (2 * W);
        if (dst[e] < 0) continue;
        if (dst[e] < cs + wc) rkp[((long)f * W + dst[e] - cs) * kGjNb + j] = x[e];
        else B[(long)j * ng + dst[e]] = x[e];
    }
}

// After panel [c0, c0 + nb): its row swaps on the columns outside it, 32
// columns per workgroup (all their rows are read before any is written).  The
// pivot rows go to rk [f][64][ng] for the update of those columns.
__global__ void __launch_bounds__(256)
k_gj_rows(int ng, int c0, int nb, double2 *a, const int *piv, double2 *rk)
{
    constexpr int COLS = 32, PER = 2 * kGjNb * COLS / 256;
    __shared__ int sPiv[kGjNb], sDst[2 * kGjNb], sSrc[2 * kGjNb];
    const int f = blockIdx.y, tid = threadIdx.x;
    double2 *A = a + (long)f * ng * ng;
    if (tid < nb) sPiv[tid] = piv[(long)f * ng + c0 + tid];
    __syncthreads();
    if (tid < 2 * kGjNb) {
        const int s0 = tid % kGjNb;
        int row = -1, src = -1;
        if (s0 < nb) {
            row = tid < kGjNb ? c0 + s0 : sPiv[s0];
            if (tid >= kGjNb && row < c0 + nb) row = -1;
            src = row;
            for (int s = nb - 1; s >= 0; s--) src = src == c0 + s ? sPiv[s] : src == sPiv[s] ? c0 + s : src;
        }
        sDst[tid] = row;
        sSrc[tid] = src;
    }
    __syncthreads();
    const int j = blockIdx.x * COLS + tid % COLS;
    const bool on = j < ng && !(j >= c0 && j < c0 + nb);
    double2 x[PER];
#pragma unroll
    for (int e = 0; e < PER; e++) {
        const int slot = tid / COLS + e * (256 / COLS);
        if (on && sDst[slot] >= 0) x[e] = A[(long)sSrc[slot] * ng + j];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; e++) {
        const int slot = tid / COLS + e * (256 / COLS);
        if (!on || sDst[slot] < 0) continue;
        if (slot < kGjNb) rk[((long)f * kGjNb + slot) * ng + j] = x[e];
        else A[(long)sDst[slot] * ng + j] = x[e];
    }
}

__device__ __forceinline__ d4 mfma64(double x, double y, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
}

// After the steps of columns [cs, cs + wc) of panel [c0, c0 + nb): the panel's
// other columns,
//   x_ij = sum_k x_i,cs+k rkp[k][j] + (i outside rows [cs, cs + wc) ? x_ij : 0).
// One workgroup per 64 rows; the product runs transposed (matrix rows: columns
// j of the panel, matrix columns: rows i), so that the results of 16 lanes are
// 16 neighbours of a column.  wc <= KC: one chunk, bound by the loads' latency.
template <int W, int KC>
__global__ void __launch_bounds__(256)
k_gj_inner(int ng, int c0, int nb, int cs, int wc, double2 *pb, const double2 *rkp)
{
    __shared__ double2 sR[KC][64];
    __shared__ double2 sP[KC][64];
    const int f = blockIdx.y, tid = threadIdx.x, rt0 = blockIdx.x * 64;
    double2 *B = pb + (long)f * kGjNb * ng;
    const double2 *R = rkp + (long)f * W * kGjNb;
    const int wave = tid >> 6, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wr = (wave >> 1) * 32, wc0 = (wave & 1) * 32;
    double2 x0[2][2][4];
#pragma unroll
    for (int rb = 0; rb < 2; rb++)
#pragma unroll
        for (int bc = 0; bc < 2; bc++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int j = wr + rb * 16 + lk + 4 * r, i = rt0 + wc0 + bc * 16 + li;
                x0[rb][bc][r] = make_double2(0.0, 0.0);
                if (j < nb && i < ng && (i < cs || i >= cs + wc)) x0[rb][bc][r] = B[(long)j * ng + i];
            }
#pragma unroll
    for (int e = tid; e < KC * 64; e += 256) {
        const int k = e >> 6, x = e & 63;
        sR[k][x] = k < wc && x < nb ? R[k * kGjNb + x] : make_double2(0.0, 0.0);
        sP[k][x] = k < wc && rt0 + x < ng ? B[(long)(cs - c0 + k) * ng + rt0 + x] : make_double2(0.0, 0.0);
    }
    __syncthreads();
    d4 accR[2][2], accI[2][2];
#pragma unroll
    for (int rb = 0; rb < 2; rb++)
#pragma unroll
        for (int bc = 0; bc < 2; bc++) {
            accR[rb][bc] = d4{0.0, 0.0, 0.0, 0.0};
            accI[rb][bc] = d4{0.0, 0.0, 0.0, 0.0};
        }
#pragma unroll
    for (int k0 = 0; k0 < KC; k0 += 4) {
        double2 x[2], y[2];
#pragma unroll
        for (int rb = 0; rb < 2; rb++) x[rb] = sR[k0 + lk][wr + rb * 16 + li];
#pragma unroll
        for (int bc = 0; bc < 2; bc++) y[bc] = sP[k0 + lk][wc0 + bc * 16 + li];
#pragma unroll
        for (int rb = 0; rb < 2; rb++)
#pragma unroll
            for (int bc = 0; bc < 2; bc++) {
                accR[rb][bc] = mfma64(x[rb].x, y[bc].x, accR[rb][bc]);
                accR[rb][bc] = mfma64(-x[rb].y, y[bc].y, accR[rb][bc]);
                accI[rb][bc] = mfma64(x[rb].x, y[bc].y, accI[rb][bc]);
                accI[rb][bc] = mfma64(x[rb].y, y[bc].x, accI[rb][bc]);
            }
    }
#pragma unroll
    for (int rb = 0; rb < 2; rb++)
#pragma unroll
        for (int bc = 0; bc < 2; bc++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int j = wr + rb * 16 + lk + 4 * r, i = rt0 + wc0 + bc * 16 + li;
                if (j >= nb || i >= ng || (c0 + j >= cs && c0 + j < cs + wc)) continue;
                B[(long)j * ng + i] = cadd(x0[rb][bc][r], make_double2(accR[rb][bc][r], accI[rb][bc][r]));
            }
}

typedef unsigned int u4 __attribute__((ext_vector_type(4)));

// `bytes` from p on: past them a buffer load gives zeros and a store does
// nothing.  The whole offset goes into the checked vector part (the scalar
// offset would be taken off the size first, and wrap).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t window(const double2 *p, long bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)(unsigned)min(bytes, 0xffffffffL), 0x00020000);
}

__device__ __forceinline__ double2 load16(__amdgpu_buffer_rsrc_t r, int v)
{
    return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, v, 0, 0));
}

__device__ __forceinline__ void store16(__amdgpu_buffer_rsrc_t r, int v, double2 x)
{
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, x), r, v, 0, 0);
}

// Update of the columns outside panel [c0, c0 + nb) (see the header), P in pb:
//   A[i][j] = sum_k pb[k][i] rk[k][j] + (i outside the panel rows ? A[i][j] : 0)
// A 256-thread block owns 64 columns and `run` tiles of 64 rows of one matrix:
// the 64 pivot rows of its columns stay in LDS (64 KB, two blocks per CU), and
// wave w takes rows 16 w .. + 15 of each tile (4 blocks of 16x16) on
// v_mfma_f64_16x16x4f64 (A operand lane i + 16k, B operand lane j + 16k,
// result register r of lane l at row l / 16 + 4 r, column l % 16).  The waves
// run without barriers: each reads its own panel rows straight into the
// operand layout four steps ahead and, in a tile's first steps, the old values
// it will add.  The tiles of the next panel's columns go to its buffer pbn
// instead of A, those of this panel's columns copy it back.
// Bound by the matrix cores with gaps: 20 matrices of 1500, 64 columns: 418 us
// = 53 TFLOP/s and 3.4 TB/s of A (542 us while 32x32 sub-tiles of a wave read
// both operands from chunks in LDS between barriers; 470 us with this form on
// plain loads, whose 64-bit addresses cost the instructions that the bounded
// buffer loads' 32-bit offsets save; without any memory traffic 386 us); 4
// matrices of 6000: 1.28 ms (1.56 ms).
__global__ void __launch_bounds__(256, 2)
k_gj_update(int ng, int c0, int nb, int run, double2 *a, const double2 *pb, double2 *pbn, const double2 *rk)
{
    constexpr int KC = 16, D = 4, STEPS = kGjNb / 4, NT = 256;
    __shared__ double2 sR[kGjNb * 64];
    const int f = blockIdx.z, tid = threadIdx.x;
    const int rt0 = blockIdx.y * run * 64, rt1 = min(ng, rt0 + run * 64), ct0 = blockIdx.x * 64;
    double2 *A = a + (long)f * ng * ng;
    const double2 *B = pb + (long)f * kGjNb * ng;
    if (ct0 == c0) {
        for (int r0 = rt0; r0 < rt1; r0 += 64)
            for (int k0 = 0; k0 < nb; k0 += KC) {
                for (int e = tid; e < KC * 64; e += NT) {
                    const int k = e >> 6, r = e & 63;
                    if (r0 + r < ng && k0 + k < nb) sR[k * 65 + r] = B[(long)(k0 + k) * ng + r0 + r];
                }
                __syncthreads();
                for (int e = tid; e < KC * 64; e += NT) {
                    const int r = e / KC, k = e % KC;
                    if (r0 + r < ng && k0 + k < nb) A[(long)(r0 + r) * ng + c0 + k0 + k] = sR[k * 65 + r];
                }
                __syncthreads();
            }
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const auto rB = window(B, (long)nb * ng * 16);
    const auto rR = window(rk + (long)f * kGjNb * ng, (long)nb * ng * 16);
    // of rows or columns past ng these are other elements, not used
    const int vp = (lk * ng + li) * 16;
    auto fetch = [&](int i0, int ks) { return load16(rB, vp + (4 * ks * ng + i0) * 16); };
    double2 p[D];
#pragma unroll
    for (int d = 0; d < D; d++) p[d] = fetch(rt0 + wave * 16, d);
    {
        double2 t[kGjNb * 64 / NT];
#pragma unroll
        for (int q = 0; q < kGjNb * 64 / NT; q++) t[q] = load16(rR, (tid & 63) * 16 + ((q * (NT / 64) + wave) * ng + ct0) * 16);
#pragma unroll
        for (int q = 0; q < kGjNb * 64 / NT; q++) sR[tid + q * NT] = t[q];
    }
    __syncthreads();
    const bool next = ct0 == c0 + kGjNb;
    double2 *N = pbn + (long)f * kGjNb * ng;
    // the next step's rows of sR are read before a step's matrix work
    double2 yn[4];
#pragma unroll
    for (int bc = 0; bc < 4; bc++) yn[bc] = sR[lk * 64 + bc * 16 + li];
    for (int i0 = rt0 + wave * 16; i0 < rt1; i0 += NT / 4) {
        const auto rA = window(A + (long)i0 * ng + ct0, ((long)(ng - i0) * ng - ct0) * 16);
        d4 accR[4], accI[4];
        double2 old[4][4];
        auto prev = [&](int e) { old[e % 4][e / 4] = load16(rA, vp + (e / 4 * 4 * ng + e % 4 * 16) * 16); };
#pragma unroll
        for (int bc = 0; bc < 4; bc++) {
            accR[bc] = d4{0.0, 0.0, 0.0, 0.0};
            accI[bc] = d4{0.0, 0.0, 0.0, 0.0};
        }
#pragma unroll
        for (int ks = 0; ks < STEPS; ks++) {
            const double2 x = p[ks % D];
            p[ks % D] = ks + D < STEPS ? fetch(i0, ks + D) : fetch(i0 + NT / 4, ks + D - STEPS);
            if (ks < 8) {
                prev(2 * ks);
                prev(2 * ks + 1);
            }
            double2 y[4];
#pragma unroll
            for (int bc = 0; bc < 4; bc++) {
                y[bc] = yn[bc];
                yn[bc] = sR[(4 * ((ks + 1) % STEPS) + lk) * 64 + bc * 16 + li];
            }
#pragma unroll
            for (int bc = 0; bc < 4; bc++) accR[bc] = mfma64(x.x, y[bc].x, accR[bc]);
#pragma unroll
            for (int bc = 0; bc < 4; bc++) accI[bc] = mfma64(x.x, y[bc].y, accI[bc]);
#pragma unroll
            for (int bc = 0; bc < 4; bc++) accR[bc] = mfma64(-x.y, y[bc].y, accR[bc]);
#pragma unroll
            for (int bc = 0; bc < 4; bc++) accI[bc] = mfma64(x.y, y[bc].x, accI[bc]);
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool keep = i0 < c0 || i0 >= c0 + kGjNb;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const int i = i0 + lk + 4 * r;
#pragma unroll
            for (int bc = 0; bc < 4; bc++) {
                const int x = bc * 16 + li;
                double2 v = make_double2(accR[bc][r], accI[bc][r]);
                if (keep) v = cadd(v, old[bc][r]);
                if (next) {
                    if (i < ng && ct0 + x < ng) N[(long)x * ng + i] = v;
                } else if (ct0 + x < ng) {
                    store16(rA, vp + (r * 4 * ng + bc * 16) * 16, v);
                }
            }
        }
    }
}

// undo the row swaps as column swaps in reverse order; one thread per row
__global__ void k_gj_unswap(int nfreq, int ng, double2 *a, const int *piv)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)nfreq * ng) return;
    const int f = (int)(t / ng);
    double2 *row = a + t * ng;
    const int *pv = piv + (long)f * ng;
    for (int c = ng - 1; c >= 0; c--) {
        const int r = pv[c];
        if (r != c) {
            const double2 x = row[c];
            row[c] = row[r];
            row[r] = x;
        }
    }
}

__global__ void k_W(int nfreq, int ng, const double *vs, const double2 *einv, double2 *W)
{
    const long n2 = (long)ng * ng;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n2 * nfreq) return;
    const long e = t % n2;
    const int g = (int)(e / ng), h = (int)(e - (long)g * ng);
    W[t] = cscale(einv[t], kHartreeEv * vs[g] * vs[h]);
}

}  // namespace

void launch_vsqrt(hipStream_t s, const Geometry &g, int ng, const int *gsph, double *vs, int *flag, bool head)
{
    const double pref = sqrt(4.0 * kPi / g.volume);
    hipLaunchKernelGGL(k_vsqrt, dim3((ng + 255) / 256), dim3(256), 0, s, ng, gsph, g.rec[0], g.rec[1],
                       g.rec[2], g.rec[3], g.rec[4], g.rec[5], g.rec[6], g.rec[7], g.rec[8],
                       (double)g.iq[0] / g.kmesh[0], (double)g.iq[1] / g.kmesh[1],
                       (double)g.iq[2] / g.kmesh[2], pref, (int)head, vs, flag);
}

void launch_eps(hipStream_t s, int nfreq, int ng, const double *vs, const double2 *chi, double2 *eps,
                int *flag)
{
    const long tot = (long)nfreq * ng * ng;
    hipLaunchKernelGGL(k_eps, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, nfreq, ng, vs, chi,
                       eps, flag);
}

// two panels and the pivot rows of one, [nfreq][64][ng] each, then the pivot
// rows of a few columns [nfreq][<= 16][64]
size_t invert_scratch_bytes(int ng, int nfreq)
{
    return sizeof(double2) * (size_t)kGjNb * (3 * ng + 16) * nfreq;
}

// Row tiles per workgroup of the update.  A CU's time is about 7 us per tile
// (its matrix work) and 6 us per round of its two workgroups (the pivot rows'
// latency): 8 matrices of 777, 1 .. 4 tiles: model 53, 54, 48, 62 us (and a
// constant), measured 69.9 (2), 62.9 (3), 74.5 (4).  Large grids hardly differ
// (1500 x 20: 418, 420, 425 us for 2, 3, 4; 6000 x 4: 1280, 1296, 1261).
static int update_run(int nfreq, int t)
{
    int best = 1;
    double least = 0.0;
    for (int run = 1; run <= 4; run++) {
        const double blocks = (double)nfreq * std::max(t - 1, 1) * ((t + run - 1) / run);
        const double n = std::ceil(blocks / 256.0), cost = 7.0 * n * run + 6.0 * std::ceil(n / 2.0);
        if (run == 1 || cost < least) best = run, least = cost;
    }
    return best;
}

template <int R, int W, int NT>
static void panel_steps(hipStream_t s, int nfreq, int ng, int c0, int nb, double2 *pb, double2 *rkp, int *piv,
                        int *flag)
{
    for (int cs = c0; cs < c0 + nb; cs += W) {
        const int wc = std::min(W, c0 + nb - cs);
        hipLaunchKernelGGL((k_gj_panel<R, W, NT>), dim3(nfreq), dim3(NT), 0, s, ng, c0, nb, cs, wc, pb, rkp, piv, flag);
        if (nb > wc)
            hipLaunchKernelGGL((k_gj_inner<W, (W > 4 ? W : 4)>), dim3((unsigned)((ng + 63) / 64), nfreq), dim3(256), 0,
                               s, ng, c0, nb, cs, wc, pb, rkp);
    }
}

// the panels of nfreq matrices (see launch_invert)
static void invert_steps(hipStream_t s, int nfreq, int ng, double2 *a, double2 *scratch, int *piv, int *flag)
{
    const unsigned t = (unsigned)((ng + 63) / 64);
    const size_t panel = (size_t)kGjNb * ng * nfreq;
    double2 *pb = scratch, *pbn = scratch + panel, *rk = scratch + 2 * panel, *rkp = scratch + 3 * panel;
    const int run = update_run(nfreq, (int)t);
    hipLaunchKernelGGL(k_gj_first, dim3(t, nfreq), dim3(256), 0, s, ng, std::min(kGjNb, ng), a, pb);
    for (int c0 = 0; c0 < ng; c0 += kGjNb) {
        const int nb = std::min(kGjNb, ng - c0);
        // rows per thread x columns x threads: R W double2 values in registers
        // without spilling; measured against the neighbouring choices at 300,
        // 777, 1500, 2048, 3000 and 6000 (e.g. 6000: <6, 3, 1024> 203 ms,
        // <12, 3, 512> 204, <6, 2, 1024> 205; 1500: <3, 16, 512> 21.5 ms, taken
        // 20.9: whole calls, with the update at 1.56 and 0.54 ms a panel)
        if (ng <= 256) panel_steps<1, 16, 256>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        else if (ng <= 512) panel_steps<1, 16, 512>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        else if (ng <= 1024) panel_steps<2, 8, 512>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        else if (ng <= 1536) panel_steps<3, 8, 512>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        else if (ng <= 2048) panel_steps<2, 8, 1024>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        else if (ng <= 3072) panel_steps<3, 4, 1024>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        else if (ng <= 4096) panel_steps<4, 4, 1024>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        else panel_steps<6, 3, 1024>(s, nfreq, ng, c0, nb, pb, rkp, piv, flag);
        if (ng > nb)
            hipLaunchKernelGGL(k_gj_rows, dim3((unsigned)((ng + 31) / 32), nfreq), dim3(256), 0, s, ng, c0, nb, a, piv,
                               rk);
        hipLaunchKernelGGL(k_gj_update, dim3(t, (t + run - 1) / run, nfreq), dim3(256), 0, s, ng, c0, nb, run, a, pb,
                           pbn, rk);
        std::swap(pb, pbn);
    }
}

void launch_invert(hipStream_t s, int nfreq, int ng, double2 *a, double2 *scratch, size_t scratch_bytes, int *piv,
                   int *flag)
{
    const int per = (int)std::min<size_t>(nfreq, scratch_bytes / invert_scratch_bytes(ng, 1));
    for (int f = 0; f < nfreq; f += per)
        invert_steps(s, std::min(per, nfreq - f), ng, a + (long)f * ng * ng, scratch, piv + (long)f * ng, flag);
    const long rows = (long)nfreq * ng;
    hipLaunchKernelGGL(k_gj_unswap, dim3((unsigned)((rows + 127) / 128)), dim3(128), 0, s, nfreq, ng, a,
                       piv);
}

void launch_W(hipStream_t s, int nfreq, int ng, const double *vs, const double2 *einv, double2 *W)
{
    const long tot = (long)nfreq * ng * ng;
    hipLaunchKernelGGL(k_W, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, nfreq, ng, vs, einv, W);
}

}  // namespace rp
