// Direct and exchange densities of Wannier orbitals at the vectors of a list
// (Eq. rhoiqG and its exchange form), without a transformed grid in memory:
//
//   rho_v(G) = (Omega/N_r) sum_p f_v(p) e^{iG.r_p} / |q+G|
//   f_v(p)   = phi_i(p) phi_j(p) c1(p1) c2(p2) c3(p3),   v = (R, i, j)
//
// with c_a(p_a) = e^{2 pi i q_a rt_a} where the image rt of p (nearest the
// midpoint (c_i + c_j + R)/2) lies within half a cell of both orbitals along
// axis a, else 0; direct densities are i = j, R = 0, without the cut.  Phase
// and cut are products over the axes, so a density needs two grid values and
// three table entries per point.
//
// One workgroup of NT threads per density (and NT MAXG vectors of the list;
// a few densities spread their planes over several workgroups each)
// walks the grid two or four planes p1 at a time: each quad of lanes transforms a row along axis 3,
// keeping the list's m3 window in LDS, then the window's columns along axis 2;
// the list's vectors, a few per thread, add their axis-1 phase in registers: a
// group's planes from zero, then the group's sum to the total, up to five
// vectors per thread with its rounding errors kept (one addition per plane put
// V and X 4.4e-16 off on 256 x 16 x 16, 1.9e-16 through whole grids and here).
// Planes and rows outside the cut are skipped.  Bound by FP64 arithmetic and
// LDS.  Through whole grids in memory (overlap grids written, three transform
// passes, a gather) the 2700 exchange densities of the 48^3 workload's 27 cells
// took 14.3 ms of device time, here (1355 of them, see exchange_vectors) 0.5.
#include "fft_lds.h"

namespace rp {

namespace {

struct DensityArgs {
    int N1, nwan, nlist, lo3, L3, zero_ok;
    double q[3], rec[9], scale;
    const double *phi, *centre;
    const int *R, *vec, *g;   // R, vec null: direct densities
    long ldp;
    double2 *P, *part;   // part: partial sums of the workgroups z of a density, or null
    int *flag;
};

// The factor of vector gi: (Omega/N_r) / |q+G|
__device__ __forceinline__ double density_scale(const DensityArgs &d, int gi)
{
    const int *m = d.g + 3 * gi;
    const double f1 = d.q[0] + m[0], f2 = d.q[1] + m[1], f3 = d.q[2] + m[2];
    const double x = f1 * d.rec[0] + f2 * d.rec[3] + f3 * d.rec[6];
    const double y = f1 * d.rec[1] + f2 * d.rec[4] + f3 * d.rec[7];
    const double z = f1 * d.rec[2] + f2 * d.rec[5] + f3 * d.rec[8];
    const double qg = sqrt(x * x + y * y + z * z);
    if (!(qg > 0.0)) {
        if (d.zero_ok) return d.scale;   // q + G = 0: ntilde(0) itself
        atomicOr(d.flag, kFlagNonFinite);
    }
    return d.scale / qg;
}

// P[v][g] from the partial sums of nz workgroups per density
__global__ void __launch_bounds__(256) k_density_sum(DensityArgs d, int nv, int nz)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x, n = (long)nv * d.nlist;
    if (t >= n) return;
    const long v = t / d.nlist;
    const int gi = (int)(t - v * d.nlist);
    double2 s = make_double2(0.0, 0.0), e = s;
    for (int z0 = 0; z0 < nz; z0 += 4) {
        double2 x[4];
#pragma unroll
        for (int z = 0; z < 4; z++) x[z] = z0 + z < nz ? d.part[(z0 + z) * n + t] : make_double2(0.0, 0.0);
        const double2 y = cadd(cadd(x[0], x[1]), cadd(x[2], x[3]));
        add_kept(s.x, e.x, y.x);
        add_kept(s.y, e.y, y.y);
    }
    d.P[v * d.ldp + gi] = cscale(make_double2(kept(s.x, e.x), kept(s.y, e.y)), density_scale(d, gi));
}

__device__ __forceinline__ void lds_sync()
{
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <int N, int MAXG, int NT>
__global__ void __launch_bounds__(NT, 512 / NT) k_density(DensityArgs d)
{
    constexpr int Q = N / 4, NGRP = NT / 4, PL = NT / 128;
    extern __shared__ double2 win_dyn[];   // PL windows [N][L3]
    __shared__ double2 tw1[256], twN[N], twQ[Q], c1[256], c2[N], c3[N];
    __shared__ int act[256], nact;
    const int tid = threadIdx.x, s = tid & 3, grp = tid >> 2, res = quad_row(s);
    const int N1 = d.N1, L3 = d.L3;
    const int wsize = N * L3;
    int i = blockIdx.x, j = i, Rv[3] = {0, 0, 0};
    if (d.R) {
        const int v = d.vec[blockIdx.x], nw = d.nwan, r = v / (nw * nw);
        i = (v / nw) % nw;
        j = v % nw;
        for (int a = 0; a < 3; a++) Rv[a] = d.R[3 * r + a];
    }
    fill_twiddles(tw1, N1, tid, NT);
    fill_twiddles(twN, N, tid, NT);
    fill_twiddles(twQ, Q, tid, NT);
    for (int t = tid; t < N1 + 2 * N; t += NT) {
        const int a = t < N1 ? 0 : (t < N1 + N ? 1 : 2), p = t - (a == 0 ? 0 : (a == 1 ? N1 : N1 + N));
        const double ci = d.centre[3 * i + a], cj = d.centre[3 * j + a], Ra = (double)Rv[a];
        const double m = 0.5 * (ci + cj + Ra);
        double x = (double)p / (a == 0 ? N1 : N) - m;
        x -= floor(x + 0.5);
        const double rt = m + x, di = rt - ci, dj = rt - Ra - cj;
        const bool in = !d.R || (di >= -0.5 && di < 0.5 && dj >= -0.5 && dj < 0.5);
        double sn, cs;
        sincospi(2.0 * d.q[a] * rt, &sn, &cs);
        (a == 0 ? c1 : (a == 1 ? c2 : c3))[p] = in ? make_double2(cs, sn) : make_double2(0.0, 0.0);
    }
    // the sums of up to five vectors per thread keep their rounding errors
    constexpr bool KEPT = MAXG <= 5;
    double2 acc[MAXG], err[KEPT ? MAXG : 1];
    // per vector: bits 0-13 the window index, 14-21 m1 mod N1
    unsigned pk[MAXG];
    const int gbase = blockIdx.y * NT * MAXG + tid;
#pragma unroll
    for (int t = 0; t < MAXG; t++) {
        const int gi = gbase + t * NT;
        acc[t] = make_double2(0.0, 0.0);
        if constexpr (KEPT) err[t] = make_double2(0.0, 0.0);
        pk[t] = 0;
        if (gi < d.nlist) {
            const int *m = d.g + 3 * gi;
            pk[t] = (unsigned)(pmod(m[1], N) * L3 + pmod(m[2] - d.lo3, N)) | ((unsigned)pmod(m[0], N1) << 14);
        }
    }
    __syncthreads();
    if (tid < 64) {
        int n = 0;
        for (int b = 0; b < N1; b += 64) {
            const int p = b + tid;
            const bool on = p < N1 && (c1[p].x != 0.0 || c1[p].y != 0.0);
            const unsigned long long mask = __ballot(on);
            if (on) act[n + __popcll(mask & ((1ull << tid) - 1))] = p;
            n += __popcll(mask);
        }
        if (tid == 0) nact = n;
    }
    __syncthreads();
    const long nr = (long)N1 * N * N;
    const double *pi = d.phi + (long)i * nr, *pj = d.phi + (long)j * nr;
    const unsigned magic = 0xffffffffu / (unsigned)N1 + 1u;   // x / N1 = umulhi(x, magic) for x < 2^16, N1 > 1

    const int a0 = nact * blockIdx.z / gridDim.z, a1 = nact * (blockIdx.z + 1) / gridDim.z;
    for (int a = a0; a < a1; a += PL) {
        const int npl = min(PL, a1 - a);
        for (int task = grp; task < npl * N; task += NGRP) {
            const int pl = task / N, p2 = task - pl * N, p1 = act[a + pl];
            const double2 f = cmul(c1[p1], c2[p2]);
            double2 *dst = win_dyn + pl * wsize + p2 * L3;
            if (f.x == 0.0 && f.y == 0.0) {
                for (int t = s; t < L3; t += 4) dst[t] = make_double2(0.0, 0.0);
                continue;
            }
            const long off = ((long)p1 * N + p2) * N + Q * s;
            double2 x[Q];
#pragma unroll
            for (int n = 0; n < Q; n++) {
                const double2 c = c3[Q * s + n];
                const bool in = c.x != 0.0 || c.y != 0.0;
                x[n] = cscale(cmul(c, f), in ? pi[off + n] * pj[off + n] : 0.0);
            }
            quad_fft<Q>(x, twQ, twN, s);
#pragma unroll
            for (int k = 0; k < Q; k++) {
                const int t3 = pmod(4 * k + res - d.lo3, N);
                if (t3 < L3) dst[t3] = x[k];
            }
        }
        lds_sync();
        for (int task = grp; task < npl * L3; task += NGRP) {
            const int pl = task / L3;
            double2 *col = win_dyn + pl * wsize + (task - pl * L3);
            double2 y[Q];
#pragma unroll
            for (int n = 0; n < Q; n++) y[n] = col[(Q * s + n) * L3];
            quad_fft<Q>(y, twQ, twN, s);
#pragma unroll
            for (int k = 0; k < Q; k++) col[(4 * k + res) * L3] = y[k];
        }
        lds_sync();
        // TB vectors at a time (all 13 at once, or one after the other, spill or wait: 1.1 times
        // the time of a long list)
        constexpr int TB = MAXG <= 5 ? MAXG : 7;
#pragma unroll
        for (int t0 = 0; t0 < MAXG; t0 += TB) {
            double2 z[TB];
#pragma unroll
            for (int t = 0; t < TB; t++) z[t] = make_double2(0.0, 0.0);
#pragma unroll 1
            for (int pl = 0; pl < npl; pl++) {
                const unsigned p1 = (unsigned)act[a + pl];
                const double2 *w = win_dyn + pl * wsize;
#pragma unroll
                for (int t = 0; t < TB; t++) {
                    if (t0 + t >= MAXG) break;
                    const unsigned u = pk[t0 + t], st = (u >> 14) * p1;
                    const double2 e = tw1[N1 > 1 ? st - __umulhi(st, magic) * N1 : 0];
                    const double2 v = w[u & 0x3fffu];
                    z[t].x += v.x * e.x - v.y * e.y;
                    z[t].y += v.x * e.y + v.y * e.x;
                }
            }
#pragma unroll
            for (int t = 0; t < TB; t++) {
                if (t0 + t >= MAXG) break;
                double2 &s = acc[t0 + t];
                if constexpr (KEPT) {
                    add_kept(s.x, err[t0 + t].x, z[t].x);
                    add_kept(s.y, err[t0 + t].y, z[t].y);
                } else {
                    s = cadd(s, z[t]);
                }
            }
        }
        lds_sync();
    }
#pragma unroll
    for (int t = 0; t < MAXG; t++) {
        const int gi = gbase + t * NT;
        if (gi >= d.nlist) continue;
        if constexpr (KEPT) acc[t] = make_double2(kept(acc[t].x, err[t].x), kept(acc[t].y, err[t].y));
        if (d.part) d.part[((long)blockIdx.z * gridDim.x + blockIdx.x) * d.nlist + gi] = acc[t];
        else d.P[(long)blockIdx.x * d.ldp + gi] = cscale(acc[t], density_scale(d, gi));
    }
}

#define RP_DENSITY_LENGTHS(X) X(16) X(20) X(24) X(32) X(36) X(40) X(48)

}  // namespace

// Vectors of the list per thread: 4 or 5, whose sums keep their rounding errors,
// or 13 (the registers) for a longer list on up to 64 planes, sixteen groups of
// them; a list longer than the threads hold takes several workgroups per density.
static int vectors_per_thread(int N1, int nlist) { return nlist <= 1024 ? 4 : nlist <= 2560 || N1 > 64 ? 5 : 13; }

// workgroups that share a density's planes: enough for one workgroup per CU,
// each with four planes at least
static int density_split(int N1, int nv, int nlist)
{
    const int per = 512 * vectors_per_thread(N1, nlist), chunks = (nlist + per - 1) / per;
    return std::max(1, std::min(N1 / 4, 256 / std::max(1, nv * chunks)));
}

size_t density_part(const int fft[3], int nv, int nlist)
{
    const int nz = density_split(fft[0], nv, nlist);
    return nz > 1 ? (size_t)nz * nv * nlist : 0;
}

bool density_lanes(const int fft[3])
{
    if (fft[0] > 256 || fft[1] != fft[2]) return false;
#define RP_CASE(e) if (fft[1] == e) return true;
    RP_DENSITY_LENGTHS(RP_CASE)
#undef RP_CASE
    return false;
}

void launch_density(hipStream_t s, const Geometry &g, int nwan, const double *phi, const double *centre_dev,
                    const int *R_dev, const int *vec_dev, int nv, int nlist, const int *glist_dev,
                    const int *glist_host, bool zero_ok, long ldp, double2 *part, double2 *P, int *flag)
{
    if (nv == 0 || nlist == 0) return;
    DensityArgs d;
    d.N1 = g.fft[0];
    d.nwan = nwan;
    d.nlist = nlist;
    int lo = glist_host[2], hi = lo;
    for (int i = 1; i < nlist; i++) {
        lo = std::min(lo, glist_host[3 * i + 2]);
        hi = std::max(hi, glist_host[3 * i + 2]);
    }
    // the list's m3 window, or the whole axis where it wraps around
    const int N = g.fft[2];
    d.L3 = std::min(N, hi - lo + 1);
    d.lo3 = d.L3 < N ? lo : 0;
    d.zero_ok = zero_ok;
    for (int a = 0; a < 3; a++) d.q[a] = (double)g.iq[a] / g.kmesh[a];
    for (int a = 0; a < 9; a++) d.rec[a] = g.rec[a];
    d.scale = g.volume / ((double)g.fft[0] * g.fft[1] * g.fft[2]);
    d.phi = phi;
    d.centre = centre_dev;
    d.R = R_dev;
    d.vec = vec_dev;
    d.g = glist_dev;
    d.ldp = ldp;
    d.P = P;
    const int nz = density_split(g.fft[0], nv, nlist);
    d.part = nz > 1 ? part : nullptr;
    d.flag = flag;
    const int per = vectors_per_thread(g.fft[0], nlist);
    auto go = [&](auto kern, int per, int nt) {
        const size_t shm = sizeof(double2) * (size_t)(nt / 128) * N * d.L3;
        if (shm > 32768)
            (void)hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
        const unsigned chunks = (unsigned)((nlist + nt * per - 1) / (nt * per));
        hipLaunchKernelGGL(kern, dim3((unsigned)nv, chunks, (unsigned)nz), dim3(nt), shm, s, d);
    };
    switch (N) {
#define RP_CASE(e)                                                                                        \
    case e:                                                                                               \
        if (per == 4) go(k_density<e, 4, 256>, 4, 256);                                                   \
        else if (per == 5) go(k_density<e, 5, 512>, 5, 512);                                              \
        else go(k_density<e, 13, 512>, 13, 512);                                                          \
        break;
        RP_DENSITY_LENGTHS(RP_CASE)
#undef RP_CASE
    }
    if (nz > 1) {
        const long n = (long)nv * nlist;
        hipLaunchKernelGGL(k_density_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, d, nv, nz);
    }
}

}  // namespace rp
