// Step a10 (Eqs. matrix_U, rhoiqG): Wannier densities and the projected
// screened interaction of one q-point.
//
//   f_i(r_j)  = phi_i(r_j)^2 e^{i q.rt_ij},  rt_ij = R_i + minimum image of (r_j - R_i)
//   rho_i(G)  = (Omega/N_r) [sum_j f_i(r_j) e^{iG.r_j}] / |q+G|
//   W_ij(w)   = pre * ( sum_{G,G'} rho_i(G) eps^-1_GG'(w) conj(rho_j(G'))
//                      + sum_{G in tail} rho_i(G) conj(rho_j(G)) ),  pre = HA 4 pi/(Omega Nq)
//
// The e^{iq.rt} factor carries the Bloch phase of the orbital's true position,
// since the home-cell orbital is stored folded into one cell.
#include "fft_lds.h"

namespace rp {

namespace {

__global__ void k_wdens(int nwan, int N1, int N2, int N3, const double *phi, const double *centre,
                        double q1, double q2, double q3, double2 *f)
{
    const long nr = (long)N1 * N2 * N3;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nr * nwan) return;
    const int i = (int)(t / nr);
    const long j = t - (long)i * nr;
    const int j1 = (int)(j / ((long)N2 * N3)), j2 = (int)((j / N3) % N2), j3 = (int)(j % N3);
    const double c1 = centre[3 * i], c2 = centre[3 * i + 1], c3 = centre[3 * i + 2];
    double d1 = (double)j1 / N1 - c1, d2 = (double)j2 / N2 - c2, d3 = (double)j3 / N3 - c3;
    d1 -= floor(d1 + 0.5);
    d2 -= floor(d2 + 0.5);
    d3 -= floor(d3 + 0.5);
    // q.rt = 2 pi sum_a qf_a rtf_a in fractional coordinates
    const double ph = 2.0 * (q1 * (c1 + d1) + q2 * (c2 + d2) + q3 * (c3 + d3));
    double s, c;
    sincospi(ph, &s, &c);
    const double n = phi[t] * phi[t];
    f[t] = make_double2(n * c, n * s);
}

__global__ void k_wgather(int nwan, int N1, int N2, int N3, int nlist, const int *g, double r0,
                          double r1, double r2, double r3, double r4, double r5, double r6, double r7,
                          double r8, double q1, double q2, double q3, double scale, const double2 *fg,
                          double2 *rho, int *flag, int zero_ok)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)nlist * nwan) return;
    const int i = (int)(t / nlist), gi = (int)(t - (long)i * nlist);
    const int m1 = g[3 * gi], m2 = g[3 * gi + 1], m3 = g[3 * gi + 2];
    const double f1 = q1 + m1, f2 = q2 + m2, f3 = q3 + m3;
    const double x = f1 * r0 + f2 * r3 + f3 * r6;
    const double y = f1 * r1 + f2 * r4 + f3 * r7;
    const double z = f1 * r2 + f2 * r5 + f3 * r8;
    const double qg = sqrt(x * x + y * y + z * z);
    const long nr = (long)N1 * N2 * N3;
    const double2 v = fg[(long)i * nr + ((long)pmod(m1, N1) * N2 + pmod(m2, N2)) * N3 + pmod(m3, N3)];
    if (qg > 0.0) {
        rho[t] = cscale(v, scale / qg);
    } else if (zero_ok) {
        rho[t] = cscale(v, scale);   // q + G = 0: ntilde(0) itself
    } else {
        atomicOr(flag, kFlagNonFinite);
        rho[t] = cscale(v, scale / qg);
    }
}

// rows of eps^-1 per workgroup of k_wbody: what the registers hold beside 16 or 32 orbitals
int body_rows(int nwan) { return nwan <= 16 ? 32 : 16; }

typedef double d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ d4 mfma64(double x, double y, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, c, 0, 0, 0);
}

// Quadratic forms of all orbital pairs: over the rows of one workgroup,
//   part[f][row block][i][j] = sum_G P[i][G] sum_G' eps^-1[f][G][G'] conj(P[j][G'])
// with G, G' in [klo, ng).  Bound by reading eps^-1 once.  A workgroup owns 16 RB
// rows G (32, or 16 beside 32 orbitals), each of its four waves a quarter of the
// columns G', so that enough loads are in flight: the four lanes of a row read
// 64 contiguous bytes of it (and of their orbital) straight into a matrix
// operand; 16 NC orbitals.  The product with P over the rows follows in LDS.
// 20 x 1500^2, ten orbitals: 0.62 ms with one workgroup per row and a reduction
// through LDS per orbital, 0.20 here (3.6 TB/s).
//
// A column quarter in one accumulator is a chain of hundreds of additions: W_ij
// of 777 to 1200 vectors was off by 9e-16, against 3.5e-16 for sums by halves.
// So the products of 16 columns start from zero, four columns each, are added
// by halves and join the total with its rounding errors kept, as do the rows:
// 3.3e-16.  That costs no time up to 16 orbitals (ten: 306 us a call either
// way), 10% above (20 x 1500^2, 32 orbitals: 479 -> 517 us, the rows halved).
template <int NC, int RB>
__global__ void __launch_bounds__(256, 2)
k_wbody(int nwan, int ng, int klo, const double2 *__restrict__ P, long ldp, const double2 *__restrict__ einv,
        double2 *__restrict__ part)
{
    constexpr int LD = 16 * NC + 1;
    __shared__ double2 sT[4][16 * RB][LD];
    const int f = blockIdx.y, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const int r0 = blockIdx.x * 16 * RB;
    const double2 *E = einv + (long)f * ng * ng;
    const int steps = (ng + 15) / 16, s0 = steps * wave / 4, s1 = steps * (wave + 1) / 4;
    const double2 *row[RB];
    const double2 *orb[NC];
#pragma unroll
    for (int rb = 0; rb < RB; rb++) row[rb] = E + (long)min(r0 + rb * 16 + li, ng - 1) * ng;
#pragma unroll
    for (int c = 0; c < NC; c++) orb[c] = P + (long)min(c * 16 + li, nwan - 1) * ldp;
    d4 accR[RB][NC], accI[RB][NC], errR[RB][NC], errI[RB][NC];
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
        for (int c = 0; c < NC; c++)
            accR[rb][c] = accI[rb][c] = errR[rb][c] = errI[rb][c] = d4{0.0, 0.0, 0.0, 0.0};
    double2 e[RB][4], o[NC][4];
    auto load = [&](int st) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            const int k = st * 16 + 4 * q + lk;
            const bool in = k >= klo && k < ng;
            const int kc = min(k, ng - 1);
#pragma unroll
            for (int rb = 0; rb < RB; rb++) {
                const double2 v = row[rb][kc];
                e[rb][q] = in ? v : make_double2(0.0, 0.0);
            }
#pragma unroll
            for (int c = 0; c < NC; c++) {
                const double2 v = orb[c][kc];
                o[c][q] = in ? v : make_double2(0.0, 0.0);
            }
        }
    };
    if (s0 < s1) load(s0);
    for (int st = s0; st < s1; st++) {
        double2 x[RB][4], y[NC][4];
#pragma unroll
        for (int q = 0; q < 4; q++) {
#pragma unroll
            for (int rb = 0; rb < RB; rb++) x[rb][q] = e[rb][q];
#pragma unroll
            for (int c = 0; c < NC; c++) y[c][q] = o[c][q];
        }
        if (st + 1 < s1) load(st + 1);
#pragma unroll
        for (int rb = 0; rb < RB; rb++)
#pragma unroll
            for (int c = 0; c < NC; c++) {
                d4 pR[4], pI[4];
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    pR[q] = mfma64(x[rb][q].x, y[c][q].x, d4{0.0, 0.0, 0.0, 0.0});
                    pI[q] = mfma64(x[rb][q].y, y[c][q].x, d4{0.0, 0.0, 0.0, 0.0});
                }
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    pR[q] = mfma64(x[rb][q].y, y[c][q].y, pR[q]);
                    pI[q] = mfma64(-x[rb][q].x, y[c][q].y, pI[q]);
                }
                const d4 sR = (pR[0] + pR[1]) + (pR[2] + pR[3]), sI = (pI[0] + pI[1]) + (pI[2] + pI[3]);
                add_kept(accR[rb][c], errR[rb][c], sR);
                add_kept(accI[rb][c], errI[rb][c], sI);
            }
    }
    // result register r of lane (li, lk) holds row lk + 4 r, column li of a 16x16 block
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
        for (int c = 0; c < NC; c++)
#pragma unroll
            for (int r = 0; r < 4; r++)
                sT[wave][rb * 16 + lk + 4 * r][c * 16 + li] = make_double2(kept(accR[rb][c][r], errR[rb][c][r]), kept(accI[rb][c][r], errI[rb][c][r]));
    __syncthreads();
    for (int t = tid; t < 256 * RB * NC; t += 256) {
        const int r = t / (16 * NC), c = t % (16 * NC);
        sT[0][r][c] = cadd(cadd(sT[0][r][c], sT[1][r][c]), cadd(sT[2][r][c], sT[3][r][c]));
    }
    __syncthreads();
    for (int t = tid; t < nwan * nwan; t += 256) {
        const int i = t / nwan, j = t - i * nwan;
        double2 s = make_double2(0.0, 0.0), d = s;
        for (int r = 0; r < 16 * RB; r++) {
            const int G = r0 + r;
            if (G < klo || G >= ng) continue;
            const double2 v = cmul(P[(long)i * ldp + G], sT[0][r][j]);
            add_kept(s.x, d.x, v.x);
            add_kept(s.y, d.y, v.y);
        }
        part[((long)f * gridDim.x + blockIdx.x) * nwan * nwan + t] = make_double2(kept(s.x, d.x), kept(s.y, d.y));
    }
}

// out[f][ij] = pre (sum of the row blocks' parts + tail[ij]), one wave per
// (ij, f): the lanes take row blocks in turn
__global__ void __launch_bounds__(256)
k_wbody_sum(int n2, int nfreq, int nblk, const double2 *__restrict__ part, const double2 *__restrict__ tail, double pre,
            double2 *__restrict__ out)
{
    const long t = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (t >= (long)n2 * nfreq) return;
    const int f = (int)(t / n2), ij = (int)(t - (long)f * n2);
    double2 s = make_double2(0.0, 0.0);
    for (int b = lane; b < nblk; b += 64) s = cadd(s, part[((long)f * nblk + b) * n2 + ij]);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        s.x += __shfl_xor(s.x, o);
        s.y += __shfl_xor(s.y, o);
    }
    if (lane == 0) out[t] = cscale(tail ? cadd(s, tail[ij]) : s, pre);
}

}  // namespace

void launch_wannier_density(hipStream_t s, const Geometry &g, const FftPlan plans[3], int nwan,
                            const double *phi, const double *centre_frac_dev, double2 *f)
{
    const long tot = (long)g.fft[0] * g.fft[1] * g.fft[2] * nwan;
    hipLaunchKernelGGL(k_wdens, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, nwan, g.fft[0],
                       g.fft[1], g.fft[2], phi, centre_frac_dev, (double)g.iq[0] / g.kmesh[0],
                       (double)g.iq[1] / g.kmesh[1], (double)g.iq[2] / g.kmesh[2], f);
    launch_fft3d(s, plans, g.fft, nwan, f);
}

void launch_wannier_gather(hipStream_t s, const Geometry &g, int nwan, int nlist, const int *glist,
                           const double2 *fgrid, double2 *rho, int *flag, bool zero_ok)
{
    const long tot = (long)nlist * nwan;
    if (tot == 0) return;
    const double scale = g.volume / ((double)g.fft[0] * g.fft[1] * g.fft[2]);
    hipLaunchKernelGGL(k_wgather, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, nwan, g.fft[0],
                       g.fft[1], g.fft[2], nlist, glist, g.rec[0], g.rec[1], g.rec[2], g.rec[3], g.rec[4],
                       g.rec[5], g.rec[6], g.rec[7], g.rec[8], (double)g.iq[0] / g.kmesh[0],
                       (double)g.iq[1] / g.kmesh[1], (double)g.iq[2] / g.kmesh[2], scale, fgrid, rho, flag,
                       (int)zero_ok);
}

size_t wbody_part(int nfreq, int nwan, int ng)
{
    return (size_t)nfreq * ((ng + body_rows(nwan) - 1) / body_rows(nwan)) * nwan * nwan;
}

void launch_wbody(hipStream_t s, int nfreq, int nwan, int ng, int klo, const double2 *P, long ldp, const double2 *einv,
                  const double2 *tail, double pre, double2 *part, double2 *out)
{
    const int rows = body_rows(nwan);
    const dim3 grid((unsigned)((ng + rows - 1) / rows), (unsigned)nfreq);
    if (nwan <= 16) hipLaunchKernelGGL((k_wbody<1, 2>), grid, dim3(256), 0, s, nwan, ng, klo, P, ldp, einv, part);
    else hipLaunchKernelGGL((k_wbody<2, 1>), grid, dim3(256), 0, s, nwan, ng, klo, P, ldp, einv, part);
    const long n = (long)nwan * nwan * nfreq;
    hipLaunchKernelGGL(k_wbody_sum, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, nwan * nwan, nfreq, (int)grid.x,
                       part, tail, pre, out);
}

}  // namespace rp
