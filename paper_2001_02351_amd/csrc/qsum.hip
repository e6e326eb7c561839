// One q-point's term of the q-mesh sums of the interaction parameters
// (Eqs. W, Wq, matrix_U, rhoiqG, matrix_V, matrix_J, matrix_X):
//
//   U_i0jR(w) += e^{-iq.R} pre [ sum_{G,G' in S_eps} rho_i(G) eps^-1_GG'(w) conj(rho_j(G'))
//                                + sum_{G in tail} rho_i conj(rho_j) + head ]
//   V_i0jR    += e^{-iq.R} pre [ sum_{G in S_eps + tail} rho_i conj(rho_j) + head ]
//   J_i0jR(w) += pre [ sum_{G,G'} rho_v(G) eps^-1_GG'(w) conj(rho_v(G')) + tail + head ]
//   X_i0jR    += pre [ sum_{G in S_eps + tail} |rho_v(G)|^2 + head ]
//
// with pre = HA 4 pi / (Omega N_q), rho = ntilde(q+G)/|q+G|, the direct
// densities rho_i of the orbitals' own densities and the exchange densities
// rho_v, v = (R, i, j), of the overlap densities phi_i0 phi_jR.  The overlap
// density is taken on the images of the grid points nearest the midpoint
// (c_i + c_j + R)/2, phi_i0 where the image lies within half a cell of c_i
// and phi_jR within half a cell of c_j + R (each orbital is stored folded
// into one cell and stands for a function localized within half a cell of
// its centre).
//
// At q = 0 the first G is G = 0: its density is stored as ntilde(0) (not
// divided by |q|) and enters only through the head term
// A eps^-1_00 ntilde_a(0) conj(ntilde_b(0)) (eps^-1_00 -> 1 for V, X), A the
// mean of 1/|q|^2 over the q-cell around Gamma; the wings are dropped (odd
// in q to leading order).
//
// The exchange quadratic forms run as T = eps^-1 conj(P)^T on the FP64 matrix
// cores (k_wquad: 64 rows G x 80 or 32 densities per workgroup), each tile
// reduced against P in place; those of the orbital pairs are k_wbody's
// (wannier.hip), the densities k_density's (density.hip) on the edges it takes.
#include <type_traits>

#include "fft_lds.h"

namespace rp {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma64(double x, double y, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
}

// Overlap-density grids of the vectors vec[0 .. nvc) (v = (r nwan + i) nwan
// + j), each times e^{iq.rt}; one thread per (vector, grid point).
__global__ void k_xdens(int nwan, int N1, int N2, int N3, const double *__restrict__ phi,
                        const double *__restrict__ centre, const int *__restrict__ R, const int *__restrict__ vec, int nvc,
                        double q1, double q2, double q3, double2 *__restrict__ f)
{
    const long nr = (long)N1 * N2 * N3;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nr * nvc) return;
    const long lv = t / nr, p = t - lv * nr;
    const int v = vec[lv];
    const int j = v % nwan, i = (v / nwan) % nwan, r = v / (nwan * nwan);
    const int p1 = (int)(p / ((long)N2 * N3)), p2 = (int)((p / N3) % N2), p3 = (int)(p % N3);
    const double x[3] = {(double)p1 / N1, (double)p2 / N2, (double)p3 / N3};
    const double qf[3] = {q1, q2, q3};
    const double *ci = centre + 3 * i, *cj = centre + 3 * j;
    const int *Rv = R + 3 * r;
    bool in = true;
    double ph = 0.0;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const double m = 0.5 * (ci[a] + cj[a] + (double)Rv[a]);
        double d = x[a] - m;
        d -= floor(d + 0.5);
        const double rt = m + d;
        const double di = rt - ci[a], dj = rt - (double)Rv[a] - cj[a];
        in = in && di >= -0.5 && di < 0.5 && dj >= -0.5 && dj < 0.5;
        ph += qf[a] * rt;
    }
    const double val = in ? phi[(long)i * nr + p] * phi[(long)j * nr + p] : 0.0;
    double s, c;
    sincospi(2.0 * ph, &s, &c);
    f[t] = make_double2(val * c, val * s);
}

__device__ __forceinline__ void dma16(const void *src, void *lds)
{
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}

// Quadratic forms of many vectors: per 64 rows G (grid y) and frequency (z),
//   out[row tile][f][v] = sum_G P[v][G] sum_G' E[f][G][G'] conj(P[v][G'])
// over G, G' in [klo, ng).  T = E conj(P)^T runs on the FP64 matrix cores, 64
// rows x 16 CB vectors per workgroup (wave w: 16 rows x all vectors), and its
// tile is reduced against P at once.  Bound by the matrix cores: two waves per
// SIMD with the accumulators in ordinary registers, the operands' chunks of 16
// columns streamed into two LDS buffers (global_load_lds; slot k of row r holds
// column k ^ (r & 15), so that the 16 rows of an operand read fall on all
// banks).  2700 vectors, N_G = 1500, 20 frequencies: 25.4 ms at 38.7 TFLOP/s
// with operands staged through registers and 64 accumulators in AGPRs; 58
// TFLOP/s here (8.4 ms for the 1355 that need computing).
template <int CB>
__global__ void __launch_bounds__(256, 2)
k_wquad(int ng, int klo, int nv, int nfreq, const double2 *__restrict__ P, long ldp, const double2 *__restrict__ E,
        double2 *__restrict__ out)
{
    constexpr int KC = 16, TC = 16 * CB;
    __shared__ double2 sE[2][64][KC];
    __shared__ double2 sP[2][TC][KC];
    __shared__ double2 red[4][TC];
    const int f = blockIdx.z, tid = threadIdx.x;
    const int rt0 = blockIdx.y * 64, v0 = blockIdx.x * TC;
    const double2 *Ef = E + (long)f * ng * ng;
    const int wave = tid >> 6, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int wr = wave * 16;
    // DMA: a wave-load fills four rows of 16 slots; wave w loads rows 16 w ..
    // of E and every fourth group of four rows of P
    auto issue = [&](int stg, int kc) {
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int r = wr + 4 * t + lk, k = kc + (li ^ (r & 15));
            dma16(Ef + (long)min(rt0 + r, ng - 1) * ng + min(k, ng - 1), &sE[stg][wr + 4 * t][0]);
        }
#pragma unroll
        for (int t = 0; t < CB; t++) {
            const int b = 4 * (wave + 4 * t), r = b + lk, k = kc + (li ^ (r & 15));
            dma16(P + (long)min(v0 + r, nv - 1) * ldp + min(k, ng - 1), &sP[stg][b][0]);
        }
    };
    d4 accR[CB], accI[CB];
#pragma unroll
    for (int c = 0; c < CB; c++) {
        accR[c] = d4{0.0, 0.0, 0.0, 0.0};
        accI[c] = d4{0.0, 0.0, 0.0, 0.0};
    }
    auto work = [&](int stg, int kc, auto edge) {
#pragma unroll
        for (int k0 = 0; k0 < KC; k0 += 4) {
            const int slot = (k0 + lk) ^ li;
            double2 x = sE[stg][wr + li][slot], y[CB];
#pragma unroll
            for (int c = 0; c < CB; c++) y[c] = sP[stg][c * 16 + li][slot];
            if constexpr (decltype(edge)::value) {
                const int k = kc + k0 + lk;
                if (k < klo || k >= ng) {
                    x = make_double2(0.0, 0.0);
#pragma unroll
                    for (int c = 0; c < CB; c++) y[c] = x;
                }
            }
#pragma unroll
            for (int c = 0; c < CB; c++) {
                accR[c] = mfma64(x.x, y[c].x, accR[c]);
                accI[c] = mfma64(x.y, y[c].x, accI[c]);
            }
#pragma unroll
            for (int c = 0; c < CB; c++) {
                accR[c] = mfma64(x.y, y[c].y, accR[c]);
                accI[c] = mfma64(-x.x, y[c].y, accI[c]);
            }
        }
    };
    issue(0, 0);
    for (int kc = 0, stg = 0; kc < ng; kc += KC, stg ^= 1) {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (kc + KC < ng) issue(stg ^ 1, kc + KC);
        if (kc < klo || kc + KC > ng) work(stg, kc, std::true_type{});
        else work(stg, kc, std::false_type{});
    }
    // result register r of lane (li, lk) holds row lk + 4 r, column li of a 16x16 block
#pragma unroll
    for (int c = 0; c < CB; c++) {
        const int j = v0 + c * 16 + li;
        double2 s = make_double2(0.0, 0.0);
        if (j < nv) {
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int i = rt0 + wr + lk + 4 * r;
                if (i >= klo && i < ng) s = cadd(s, cmul(P[(long)j * ldp + i], make_double2(accR[c][r], accI[c][r])));
            }
        }
        // the four lanes of column li (lk = 0..3) hold disjoint rows
        s.x += __shfl_xor(s.x, 16);
        s.y += __shfl_xor(s.y, 16);
        s.x += __shfl_xor(s.x, 32);
        s.y += __shfl_xor(s.y, 32);
        if (lk == 0) red[wave][c * 16 + li] = s;
    }
    __syncthreads();
    if (tid < TC && v0 + tid < nv)
        out[((long)blockIdx.y * nfreq + f) * nv + v0 + tid] =
            cadd(cadd(red[0][tid], red[1][tid]), cadd(red[2][tid], red[3][tid]));
}

__device__ __forceinline__ double2 block_sum(double2 s, double2 *red)
{
    const int tid = threadIdx.x;
    red[tid] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (tid < h) red[tid] = cadd(red[tid], red[tid + h]);
        __syncthreads();
    }
    return red[0];
}

// Gram sums of the densities: for output o (pair (a, b) = (o / nb, o % nb),
// or a = b = o when diag) bare[o] = sum_{G in [klo, ng)} P[a][G] conj(P[b][G])
// and tail[o] = the same over [ng, ng + ntail).
__global__ void __launch_bounds__(256) k_wgram(int nb, int diag, int ng, int klo, int ntail,
                                               const double2 *__restrict__ P, long ldp,
                                               double2 *__restrict__ bare, double2 *__restrict__ tail)
{
    __shared__ double2 red[256];
    const int o = blockIdx.x;
    const int a = diag ? o : o / nb, b = diag ? o : o % nb;
    const double2 *pa = P + (long)a * ldp, *pb = P + (long)b * ldp;
    double2 s = make_double2(0.0, 0.0), t = make_double2(0.0, 0.0);
    for (int G = klo + threadIdx.x; G < ng; G += 256) s = cadd(s, cmulc(pb[G], pa[G]));
    for (int G = ng + threadIdx.x; G < ng + ntail; G += 256) t = cadd(t, cmulc(pb[G], pa[G]));
    s = block_sum(s, red);
    __syncthreads();
    t = block_sum(t, red);
    if (threadIdx.x == 0) {
        tail[o] = t;
        bare[o] = cadd(s, t);
    }
}

// U[f][r][i][j], V[r][i][j] (+)= e^{-iq.R_r} pre (...); one thread per
// (f, r, i, j) of U, the f = 0 threads also write V
__global__ void k_wsum_u(int nfreq, int nR, int nwan, int ng, const int *__restrict__ R, double q1, double q2,
                         double q3, double pre, int head, double avg, const double2 *__restrict__ E,
                         const double2 *__restrict__ P, long ldp, const double2 *__restrict__ body,
                         const double2 *__restrict__ bare, const double2 *__restrict__ tail, int accumulate,
                         double2 *__restrict__ U, double2 *__restrict__ V)
{
    const long n2 = (long)nwan * nwan;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)nfreq * nR * n2) return;
    const int f = (int)(t / (nR * n2));
    const long rem = t - (long)f * nR * n2;
    const int r = (int)(rem / n2);
    const int ij = (int)(rem - (long)r * n2), i = ij / nwan, j = ij % nwan;
    double s, c;
    sincospi(-2.0 * (q1 * R[3 * r] + q2 * R[3 * r + 1] + q3 * R[3 * r + 2]), &s, &c);
    const double2 ph = make_double2(pre * c, pre * s);
    double2 h = make_double2(0.0, 0.0);
    if (head) h = cscale(cmulc(P[(long)j * ldp], P[(long)i * ldp]), avg);   // A n_i(0) conj(n_j(0))
    if (U) {
        const double2 e00 = E[(long)f * ng * ng];
        double2 x = cadd(cadd(body[(long)f * n2 + ij], tail[ij]), cmul(e00, h));
        x = cmul(ph, x);
        U[t] = accumulate ? cadd(U[t], x) : x;
    }
    if (V && f == 0) {
        const double2 x = cmul(ph, cadd(bare[ij], h));
        const long o = (long)r * n2 + ij;
        V[o] = accumulate ? cadd(V[o], x) : x;
    }
}

// J[f][v], X[v] (+)= pre (...) for the densities of one pass (one thread per
// (f, density)): density lv is that of vector vec[lv] and, where
// vec[nvc + lv] >= 0, of that vector too; part [nrt][nfreq][nvc]
__global__ void k_wsum_x(int nfreq, long nvt, const int *__restrict__ vec, int nvc, int nrt, int ng, double pre,
                         int head, double avg, const double2 *__restrict__ E, const double2 *__restrict__ P, long ldp,
                         const double2 *__restrict__ part, const double2 *__restrict__ bare,
                         const double2 *__restrict__ tail, int accumulate, double2 *__restrict__ J,
                         double2 *__restrict__ X)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)nfreq * nvc) return;
    const int f = (int)(t / nvc), lv = (int)(t - (long)f * nvc);
    double hv = 0.0;
    if (head) {
        const double2 n0 = P[(long)lv * ldp];
        hv = avg * (n0.x * n0.x + n0.y * n0.y);
    }
    const int v = vec[lv], twin = vec[nvc + lv];
    auto put = [&](double2 *o, double2 x) { *o = accumulate ? cadd(*o, x) : x; };
    if (J) {
        double2 s = tail[lv];
        for (int rt = 0; rt < nrt; rt++) s = cadd(s, part[((long)rt * nfreq + f) * nvc + lv]);
        s = cadd(s, cscale(E[(long)f * ng * ng], hv));
        s = cscale(s, pre);
        put(J + (long)f * nvt + v, s);
        if (twin >= 0) put(J + (long)f * nvt + twin, s);
    }
    if (X && f == 0) {
        const double2 x = cscale(make_double2(bare[lv].x + hv, bare[lv].y), pre);
        put(X + v, x);
        if (twin >= 0) put(X + twin, x);
    }
}

unsigned blocks_for(long n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

void launch_xdens(hipStream_t s, const Geometry &g, const FftPlan plans[3], int nwan, const double *phi,
                  const double *centre_dev, const int *R_dev, const int *vec_dev, int nvc, double2 *grids)
{
    const long nr = (long)g.fft[0] * g.fft[1] * g.fft[2];
    hipLaunchKernelGGL(k_xdens, dim3(blocks_for(nr * nvc, 256)), dim3(256), 0, s, nwan, g.fft[0], g.fft[1],
                       g.fft[2], phi, centre_dev, R_dev, vec_dev, nvc, (double)g.iq[0] / g.kmesh[0],
                       (double)g.iq[1] / g.kmesh[1], (double)g.iq[2] / g.kmesh[2], grids);
    launch_fft3d(s, plans, g.fft, nvc, grids);
}

int wquad_row_tiles(int ng) { return (ng + 63) / 64; }

void launch_wquad(hipStream_t s, int nfreq, int ng, int klo, int nv, const double2 *P, long ldp, const double2 *E,
                  double2 *out)
{
    if (nv == 0) return;
    // 80 vectors per workgroup, or 32 where there are no more
    const int tc = nv <= 32 ? 32 : 80;
    const dim3 grid(blocks_for(nv, tc), (unsigned)wquad_row_tiles(ng), (unsigned)nfreq);
    if (tc == 32) hipLaunchKernelGGL(k_wquad<2>, grid, dim3(256), 0, s, ng, klo, nv, nfreq, P, ldp, E, out);
    else hipLaunchKernelGGL(k_wquad<5>, grid, dim3(256), 0, s, ng, klo, nv, nfreq, P, ldp, E, out);
}

void launch_wgram(hipStream_t s, int nout, int nb, bool diag, int ng, int klo, int ntail, const double2 *P,
                  long ldp, double2 *bare, double2 *tail)
{
    if (nout == 0) return;
    hipLaunchKernelGGL(k_wgram, dim3((unsigned)nout), dim3(256), 0, s, nb, (int)diag, ng, klo, ntail, P, ldp, bare,
                       tail);
}

void launch_wsum_u(hipStream_t s, const Geometry &g, int nfreq, int nR, int nwan, int ng, const int *R_dev,
                   double pre, bool head, double avg, const double2 *E, const double2 *P, long ldp,
                   const double2 *body, const double2 *bare, const double2 *tail, int accumulate, double2 *U,
                   double2 *V)
{
    const long n = (long)nfreq * nR * nwan * nwan;
    hipLaunchKernelGGL(k_wsum_u, dim3(blocks_for(n, 128)), dim3(128), 0, s, nfreq, nR, nwan, ng, R_dev,
                       (double)g.iq[0] / g.kmesh[0], (double)g.iq[1] / g.kmesh[1], (double)g.iq[2] / g.kmesh[2], pre,
                       (int)head, avg, E, P, ldp, body, bare, tail, accumulate, U, V);
}

void launch_wsum_x(hipStream_t s, int nfreq, long nvt, const int *vec_dev, int nvc, int ng, double pre, bool head,
                   double avg, const double2 *E, const double2 *P, long ldp, const double2 *part, const double2 *bare,
                   const double2 *tail, int accumulate, double2 *J, double2 *X)
{
    const long n = (long)nfreq * nvc;
    hipLaunchKernelGGL(k_wsum_x, dim3(blocks_for(n, 128)), dim3(128), 0, s, nfreq, nvt, vec_dev, nvc,
                       wquad_row_tiles(ng), ng, pre, (int)head, avg, E, P, ldp, part, bare, tail, accumulate, J, X);
}

}  // namespace rp
