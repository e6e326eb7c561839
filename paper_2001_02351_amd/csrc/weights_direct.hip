// Step a5 for a metal with every divided difference evaluated by itself: the
// weights of the split contractions at complex frequencies.
//
// These contractions round the weights to FP32, and the two-term form keeps
// 2^-17 of a weighted operand, so a weight that differs in its 14th digit now
// and then changes a last bit there and moves elements of chi by up to 5e-8 of
// their size (the three-term form: 4e-8, where few pairs make up chi).  The
// moment series of tetra.hip is the more accurate (1e-16 against up to 1e-13
// here) and the faster (14 112 pairs x 10 frequencies: 0.86 against 7.45 ms),
// but its weights change about one such rounding in a million (67 of 63
// million, six spectra of three widths, insulating and metallic); with this
// kernel chi stays the same in every bit.  Insulators have k_weights without
// its series for this, which has the same bits.  Real weights (imaginary axis)
// take the series: none of 32 million of their roundings changes.  FP64 takes
// it everywhere.
#include "tetra_dd.h"

namespace rp {

namespace {

// (1/|T|) int over {E_b < E_F < E_a} within T of lambda_v / (z - e): the
// region is tiled by clipping T first to E_b < E_F, then each piece to
// E_a > E_F; a piece S contributes (|S|/|T|) sum_j lambda_v(s_j) I_j^S(z),
// I_j^S the vertex integral of S on the transition energies at its corners
// (lambda_v is linear, so it is the barycentric combination of its corner
// values).
__device__ double2 clipped_vertex_integral(double2 zz, const double (&e)[4], const double (&eb)[4],
                                           const double (&ea)[4], double ef, int v)
{
    const double T[4][4] = {{1, 0, 0, 0}, {0, 1, 0, 0}, {0, 0, 1, 0}, {0, 0, 0, 1}};
    double phi1[4];
#pragma unroll
    for (int c = 0; c < 4; c++) phi1[c] = eb[c] - ef;
    double2 acc = make_double2(0.0, 0.0);
    auto inner = [&](const double (&r0)[4], const double (&r1)[4], const double (&r2)[4], const double (&r3)[4]) {
        const double ratio = fabs(det4(r0, r1, r2, r3));
        if (!(ratio > 0.0)) return;
        const double *R[4] = {r0, r1, r2, r3};
        double eS[4];
        double2 lS[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            eS[j] = R[j][0] * e[0] + R[j][1] * e[1] + R[j][2] * e[2] + R[j][3] * e[3];
            lS[j] = clog_d(make_double2(zz.x - eS[j], zz.y));
        }
        for (int j = 0; j < 4; j++) {
            const double lam = R[j][v];
            if (lam == 0.0) continue;
            double xs[5] = {eS[0], eS[1], eS[2], eS[3], eS[j]};
            double2 ls[5] = {lS[0], lS[1], lS[2], lS[3], lS[j]};
            sort5(xs, ls);
            const double2 d = dd4_sorted(zz, xs, ls);
            acc.x += ratio * lam * d.x;
            acc.y += ratio * lam * d.y;
        }
    };
    auto outer = [&](const double (&q0)[4], const double (&q1)[4], const double (&q2)[4], const double (&q3)[4]) {
        const double Q[4][4] = {{q0[0], q0[1], q0[2], q0[3]}, {q1[0], q1[1], q1[2], q1[3]},
                                {q2[0], q2[1], q2[2], q2[3]}, {q3[0], q3[1], q3[2], q3[3]}};
        double phi2[4];
#pragma unroll
        for (int j = 0; j < 4; j++)
            phi2[j] = ef - (Q[j][0] * ea[0] + Q[j][1] * ea[1] + Q[j][2] * ea[2] + Q[j][3] * ea[3]);
        clip_tet(Q, phi2, inner);
    };
    clip_tet(T, phi1, outer);
    return acc;
}

constexpr int kDThreads = 128;

// One thread per (pair, frequency).  The corner energies e_j of the 15
// distinct corners live in registers (the tetrahedron table indexes them with
// the same slot in every lane, which the compiler turns into register-relative
// moves) and the logarithms log(z - e_j) in LDS ([slot][thread]) with the two
// bands' corner energies: 60 KB per 128-thread block, two blocks per CU; each of the 24 tetrahedra sorts its five nodes
// (four corners, k's corner doubled) together with their logarithms and
// evaluates I_v(z) and I_v(z') (only I_v(z) when z' = z*).
//
// The Fermi level ef (hartree) cuts the tetrahedra.  With E_b < ef at
// all four corners of a tetrahedron and E_a > ef at all four, the insulating
// integral applies; with E_b >= ef or E_a <= ef at all four, the tetrahedron
// contributes nothing; otherwise clipped_vertex_integral tiles the part where
// E_b < ef < E_a.
__global__ void __launch_bounds__(kDThreads)
k_weights_direct(int K1, int K2, int K3, int q1, int q2, int q3, int nband, const double *E, const double *T, int o0,
                 int nO, int e0, int nE, int k0, long npair, int nfreq, const double2 *freq, double delta, double ef,
                 double2 *w)
{
    double eR[15];
    __shared__ double2 sL[15][kDThreads];
    __shared__ double sB[15][kDThreads];
    __shared__ double sA[15][kDThreads];
    const int tid = threadIdx.x;
    const long t = (long)blockIdx.x * blockDim.x + tid;
    if (t >= npair * nfreq) return;
    const int f = (int)(t / npair);
    const long p = t - (long)f * npair;
    const int b = o0 + (int)(p % nO);
    const int a = e0 + (int)((p / nO) % nE);
    const int k = k0 + (int)(p / ((long)nO * nE));
    const int n1 = k / (K2 * K3), n2 = (k / K3) % K2, n3 = k % K3;
    const double ha = 1.0 / kHartreeEv;
    const double2 om = make_double2(freq[f].x * ha, freq[f].y * ha);
    const double dl = delta * ha;
    const double2 z = make_double2(om.x, om.y + dl);
    const double2 zp = make_double2(-om.x, -om.y + dl);
    const int kq = (mesh_wrap(n1 + q1, K1) * K2 + mesh_wrap(n2 + q2, K2)) * K3 + mesh_wrap(n3 + q3, K3);
#pragma unroll
    for (int j = 0; j < 15; j++) {
        const int code = kTet.nbr[j];
        const int m1 = n1 + code / 9 - 1, m2 = n2 + (code / 3) % 3 - 1, m3 = n3 + code % 3 - 1;
        const int kv = (mesh_wrap(m1, K1) * K2 + mesh_wrap(m2, K2)) * K3 + mesh_wrap(m3, K3);
        const int kvq = (mesh_wrap(m1 + q1, K1) * K2 + mesh_wrap(m2 + q2, K2)) * K3 + mesh_wrap(m3 + q3, K3);
        const double eb = E[(long)kv * nband + b] * ha, ea = E[(long)kvq * nband + a] * ha;
        eR[j] = (E[(long)kvq * nband + a] - E[(long)kv * nband + b]) * ha;
        sB[j][tid] = eb;
        sA[j][tid] = ea;
    }
    // on the imaginary axis without broadening z' = z*, and since the
    // corner energies are real I_v(z*) = conj(I_v(z)): x = 2 Re sum I_v(z)/6
    const bool conj_pair = dl == 0.0 && om.x == 0.0;
    double2 x = make_double2(0.0, 0.0);
    for (int zi = 0; zi < (conj_pair ? 1 : 2); zi++) {
        const double2 zz = zi ? zp : z;
#pragma unroll
        for (int j = 0; j < 15; j++) sL[j][tid] = clog_d(make_double2(zz.x - eR[j], zz.y));
        for (int tt = 0; tt < 24; tt++) {
            double e4[4], b4[4], a4[4];
            bool all_in = true, none_b = true, none_a = true;
            int iv = 0;
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int sl = c_tetra.slot[tt][v];
                e4[v] = eR[sl];
                b4[v] = sB[sl][tid];
                a4[v] = sA[sl][tid];
                if (sl == kTet.self) iv = v;
                all_in = all_in && b4[v] < ef && a4[v] > ef;
                none_b = none_b && !(b4[v] < ef);
                none_a = none_a && !(a4[v] > ef);
            }
            if (none_b || none_a) continue;
            if (!all_in) {
                x = cadd(x, clipped_vertex_integral(zz, e4, b4, a4, ef, iv));
                continue;
            }
            double xs[5];
            double2 ls[5];
#pragma unroll
            for (int v = 0; v < 4; v++) {
                const int sl = c_tetra.slot[tt][v];
                xs[v] = eR[sl];
                ls[v] = sL[sl][tid];
            }
            xs[4] = eR[kTet.self];
            ls[4] = sL[kTet.self][tid];
            sort5(xs, ls);
            x = cadd(x, dd4_sorted(zz, xs, ls));
        }
    }
    if (conj_pair) x = make_double2(2.0 * x.x, 0.0);
    x = cscale(x, 1.0 / 6.0);
    double fac = 2.0 / (double)(K1 * K2 * K3);
    if (T) fac *= 1.0 - T[(long)kq * nband + a] * T[(long)k * nband + b];
    w[t] = cscale(x, fac);
}

}  // namespace

void launch_weights_direct(hipStream_t s, const int kmesh[3], const int iq[3], int nband, const double *E_eV,
                           const double *T, int o0, int o1, int e0, int e1, int k0, int k1, int nfreq,
                           const double2 *freq_eV, double delta_eV, double ef, double2 *w)
{
    const long npair = (long)(k1 - k0) * (e1 - e0) * (o1 - o0);
    const dim3 grid((unsigned)((npair * nfreq + kDThreads - 1) / kDThreads));
    hipLaunchKernelGGL(k_weights_direct, grid, dim3(kDThreads), 0, s, kmesh[0], kmesh[1], kmesh[2], iq[0], iq[1], iq[2],
                       nband, E_eV, T, o0, o1 - o0, e0, e1 - e0, k0, npair, nfreq, freq_eV, delta_eV, ef, w);
}

}  // namespace rp
