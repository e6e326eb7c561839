// Step a5: generalized-tetrahedron weights (Eqs. Xakqbk, tetrahedron, tak).
//
//   w_p(omega) = (2/Nk) (1 - T_{a,k+q} T_{b,k}) x_p(omega)
//   x_p(omega) = (1/6) sum_{T containing k} [ I_v(z) + I_v(z') ],
//   z = omega + i delta,  z' = -omega + i delta,
//
// where T runs over the 24 tetrahedra of the mesh that have k as a vertex
// (each mesh cell is cut into 6 tetrahedra around its (0,0,0)-(1,1,1)
// diagonal), v is k's vertex in T, and I_v(z) is the average over T of
// lambda_v / (z - e) for the linear interpolant e of the transition energies
// e = E_a(k+q) - E_b(k) at the four corners.  I_v(z) is the fourth divided
// difference of g(x) = (z-x)^3 log(z-x) with the node e_v doubled
// (Hermite-Genocchi).  With all four energies equal, x reduces to the
// textbook X(omega) of Eq. Xakqbk.
//
// Divided differences are evaluated top-down on sorted nodes: a set of
// nodes whose deviation from its median node is at most a quarter of that
// node's distance to z is summed as a Taylor series of g about the median
// node; any other set is split by the recurrence
// (g[x1..xn] - g[x0..x(n-1)]) / (xn - x0), whose denominator is then large
// enough that nothing cancels.  This replaces the degeneracy thresholds
// delta_a, delta_r the paper's tetrahedron routine takes.  Every series is
// centred on a node, so the only logarithms are log(z - e_j) at the 15
// distinct corners of the 24 tetrahedra around k: they are computed once per
// (pair, frequency) and kept in LDS, and each tetrahedron is pure arithmetic.
#include "tetra_dd.h"

namespace rp {

namespace {

// The part {E_b < E_F < E_a} of a tetrahedron T: T is clipped to E_b < E_F,
// then each piece to E_a > E_F.  A piece S contributes
// (|S|/|T|) sum_j lambda_v(s_j) I_j^S, I_j^S the vertex integral of S on the
// transition energies at its corners (lambda_v is linear, so it is the
// barycentric combination of its corner values).  The pieces, as their corner
// energies and the factors (|S|/|T|) lambda_v(s_j), are appended to (pc, n).
constexpr int kMaxPieces = 9;   // three of the first cut, three of each by the second
struct Piece {
    double e[4], lam[4];
};

__device__ void clipped_pieces(const double (&e)[4], const double (&eb)[4], const double (&ea)[4], double ef, int v,
                               Piece *pc, int &n)
{
    const double T[4][4] = {{1, 0, 0, 0}, {0, 1, 0, 0}, {0, 0, 1, 0}, {0, 0, 0, 1}};
    double phi1[4];
#pragma unroll
    for (int c = 0; c < 4; c++) phi1[c] = eb[c] - ef;
    auto inner = [&](const double (&r0)[4], const double (&r1)[4], const double (&r2)[4], const double (&r3)[4]) {
        const double ratio = fabs(det4(r0, r1, r2, r3));
        if (!(ratio > 0.0)) return;
        const double *R[4] = {r0, r1, r2, r3};
#pragma unroll
        for (int j = 0; j < 4; j++) {
            pc[n].e[j] = R[j][0] * e[0] + R[j][1] * e[1] + R[j][2] * e[2] + R[j][3] * e[3];
            pc[n].lam[j] = ratio * R[j][v];
        }
        n++;
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
}

constexpr int kWThreads = 256;
constexpr int kWPairs = 32;                       // pairs per workgroup
constexpr int kWLanes = kWThreads / kWPairs;      // threads per pair
constexpr int kWTets = 24 / kWLanes;              // tetrahedra per thread
constexpr int kWFreqs = 2 * kWLanes;              // frequencies per pass over the pairs
constexpr int kWMinFreqs = 2;                     // fewest frequencies per workgroup
constexpr int kMoments = 72;                      // 0.6^72 = 1.1e-16
constexpr double kSeriesRatio = 0.6;
constexpr int kCutPairs = 2;                      // pairs whose tetrahedra are cut at a time (one wave each)
static_assert(2 * kWFreqs <= 32, "a pass's frequencies, z and z', in the bits of a word");
static_assert(kWLanes == 8 && kWTets == 3, "eight threads per pair, three tetrahedra each");

template <int CTRL> __device__ __forceinline__ double dpp(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)hi << 32 | (unsigned)lo);
}

// sum over the eight threads of a pair, in a fixed order (quad_perm over
// lanes s ^ 1 and s ^ 2, then the mirrored half row: the quads hold equal sums)
__device__ __forceinline__ double sum8(double v)
{
    v += dpp<0xB1>(v);
    v += dpp<0x4E>(v);
    v += dpp<0x141>(v);
    return v;
}

// One workgroup per 32 pairs and a range of frequencies.
//
// All 24 tetrahedra of a pair together: with c the middle of the 15 corner
// energies, R half their spread and y = (e - c)/R,
//     sum_T I_v(z) = sum_m mu_m R^m / (z - c)^(m+1),   mu_m = sum_T <lambda_v y^m>_T
//     <lambda_v y^m>_T = 6 m!/(m+4)! h_m(y_0, .., y_3, y_v)
// (h_m the complete homogeneous symmetric polynomial; Hermite-Genocchi).  The
// moments mu_m do not depend on the frequency: eight threads per pair form 72
// of them from three tetrahedra each, and every frequency with
// R <= 0.6 |z - c| is one Horner sum of them to 1e-16.  Frequencies nearer to
// the pair's energies (9% of those of the 48^3 workload's z and z', none on
// the imaginary axis) go to a list, and one thread per (entry,
// tetrahedron) evaluates the divided difference from the entry's 15 logarithms
// log(z - e_j) in LDS.  No sum depends on which entries share a workgroup.
//
// The work is FP64 vector arithmetic and its latency.  With one thread per
// (pair, frequency) evaluating all 24 tetrahedra, 46% of the lanes active, the
// weights of 128 000 pairs x 20 real frequencies (48^3 workload) took 6.39 ms,
// now 1.70; 16 imaginary frequencies 1.33 ms, now 0.19; a metal's 14 112 pairs
// x 10 frequencies 7.45 ms, now 0.86; 3 072 pairs x 10 0.76 ms, now 0.20.
//
// Without SERIES (the split contractions of an insulator at complex
// frequencies, see weights_direct.hip for the reason) every entry goes to the
// list, with the bits of the one-thread form: 25^3 cRPA q-point 0.7 -> 0.34 ms
// of weights, the 48^3 launch 6.39 -> 5.75.
//
// METAL: the Fermi level ef (hartree) cuts the tetrahedra.  With E_b < ef at
// all four corners of a tetrahedron and E_a > ef at all four, the insulating
// integral applies; with E_b >= ef or E_a <= ef at all four, the tetrahedron
// contributes nothing; otherwise its part where E_b < ef < E_a is tiled by
// smaller tetrahedra (clipped_pieces), whose moments (for all frequencies at
// once) or integrals replace its own.
template <bool METAL, bool SERIES>
__global__ void __launch_bounds__(kWThreads, METAL ? 1 : 2)
k_weights(int K1, int K2, int K3, int q1, int q2, int q3, int nband, const double *E, const double *T,
          int o0, int nO, int e0, int nE, int k0, long npair, int nfreq, int fper, const double2 *freq,
          double delta, double ef, double2 *w)
{
    __shared__ double sE[15][kWPairs];
    __shared__ double sB[METAL ? 15 : 1][kWPairs];
    __shared__ double sA[METAL ? 15 : 1][kWPairs];
    __shared__ double sMu[SERIES ? kMoments : 1][kWPairs];
    __shared__ double sC[kWPairs], sR[kWPairs], sFac[kWPairs];
    __shared__ double2 sL[kWPairs][15];
    __shared__ double2 sVal[kWPairs * 24];
    // entries (frequency, pair, which of z and z') of uncut tetrahedra; METAL, a
    // pair with cut ones: bits 2 f, 2 f + 1 for z and z' of the pass's frequency f
    __shared__ int sQueue[kWPairs * kWFreqs];
    __shared__ int sNq, sSome[kWPairs];   // sSome: 0 nothing, 1 some, 2 whole tetrahedra only
    __shared__ unsigned sCut[kWPairs];
    __shared__ Piece sPc[METAL ? kCutPairs : 1][METAL ? 24 * kMaxPieces : 1];
    __shared__ int sNpc[kCutPairs];
    const int tid = threadIdx.x;
    const long p0 = (long)blockIdx.x * kWPairs;
    const int fa = blockIdx.y * fper, fb = min(nfreq, fa + fper);
    const double ha = 1.0 / kHartreeEv;
    const double dl = delta * ha;
    const int lane8 = tid & (kWLanes - 1), slot = tid / kWLanes;

    // corner energies (a pair past the end repeats the last one and is not stored)
    {
        const long p = min(p0 + slot, npair - 1);
        const int b = o0 + (int)(p % nO);
        const int a = e0 + (int)((p / nO) % nE);
        const int k = k0 + (int)(p / ((long)nO * nE));
        const int n1 = k / (K2 * K3), n2 = (k / K3) % K2, n3 = k % K3;
        for (int j = lane8; j < 15; j += kWLanes) {
            const int code = c_tetra.nbr[j];
            const int m1 = n1 + code / 9 - 1, m2 = n2 + (code / 3) % 3 - 1, m3 = n3 + code % 3 - 1;
            const int kv = (mesh_wrap(m1, K1) * K2 + mesh_wrap(m2, K2)) * K3 + mesh_wrap(m3, K3);
            const int kvq = (mesh_wrap(m1 + q1, K1) * K2 + mesh_wrap(m2 + q2, K2)) * K3 + mesh_wrap(m3 + q3, K3);
            const double eb = E[(long)kv * nband + b], ea = E[(long)kvq * nband + a];
            sE[j][slot] = (ea - eb) * ha;
            if constexpr (METAL) {
                sB[j][slot] = eb * ha;
                sA[j][slot] = ea * ha;
            }
        }
        if (lane8 == 0) {
            double fac = 2.0 / (double)(K1 * K2 * K3);
            if (T) {
                const int kq = (mesh_wrap(n1 + q1, K1) * K2 + mesh_wrap(n2 + q2, K2)) * K3 + mesh_wrap(n3 + q3, K3);
                fac *= 1.0 - T[(long)kq * nband + a] * T[(long)k * nband + b];
            }
            sFac[slot] = fac;
        }
    }
    __syncthreads();
    // moments: thread (slot, lane8) takes tetrahedra 3 lane8 .. 3 lane8 + 2
    if constexpr (SERIES) {
        double lo = sE[0][slot], hi = lo;
#pragma unroll
        for (int j = 1; j < 15; j++) {
            lo = fmin(lo, sE[j][slot]);
            hi = fmax(hi, sE[j][slot]);
        }
        const double c = 0.5 * (lo + hi), R = 0.5 * (hi - lo), ri = R > 0.0 ? 1.0 / R : 0.0;
        if (lane8 == 0) {
            sC[slot] = c;
            sR[slot] = R;
        }
        bool whole = true, some = true;   // every tetrahedron uncut / any of them contributes
        int kind[kWTets];                 // METAL: 0 nothing, 1 uncut, 2 cut
        if constexpr (METAL) {
            some = false;
#pragma unroll
            for (int i = 0; i < kWTets; i++) {
                bool all_in = true, none_b = true, none_a = true;
#pragma unroll
                for (int v = 0; v < 4; v++) {
                    const int sl = c_tetra.slot[kWTets * lane8 + i][v];
                    const double bb = sB[sl][slot], aa = sA[sl][slot];
                    all_in = all_in && bb < ef && aa > ef;
                    none_b = none_b && !(bb < ef);
                    none_a = none_a && !(aa > ef);
                }
                kind[i] = none_b || none_a ? 0 : all_in ? 1 : 2;
                whole = whole && kind[i] == 1;
                some = some || kind[i] != 0;
            }
            const unsigned long long group = 0xffull << (tid & 63 & ~(kWLanes - 1));
            whole = (__ballot(whole) & group) == group;
            some = (__ballot(some) & group) != 0;
        }
        if (lane8 == 0) sSome[slot] = whole ? 2 : some;
        if (whole) {
            double y[kWTets][5], P[kWTets][5];
#pragma unroll
            for (int i = 0; i < kWTets; i++)
#pragma unroll
                for (int v = 0; v < 5; v++) {
                    const int sl = v < 4 ? c_tetra.slot[kWTets * lane8 + i][v] : kTet.self;
                    y[i][v] = (sE[sl][slot] - c) * ri;
                    P[i][v] = 1.0;
                }
            for (int m = 0; m < kMoments; m++) {
                double h = 0.0;
#pragma unroll
                for (int i = 0; i < kWTets; i++) {
                    h += P[i][4];
                    // raise to degree m + 1: h_k(y_0..y_v) = h_k(y_0..y_{v-1}) + y_v h_{k-1}(y_0..y_v)
                    P[i][0] *= y[i][0];
#pragma unroll
                    for (int v = 1; v < 5; v++) P[i][v] = P[i][v - 1] + y[i][v] * P[i][v];
                }
                h = sum8(h);
                if (lane8 == 0) sMu[m][slot] = c_series.f[m + 4] * h;
            }
        } else if constexpr (METAL) {
            if (some) {
                Piece pc[kMaxPieces];
                double mu[kMoments];
#pragma unroll
                for (int m = 0; m < kMoments; m++) mu[m] = 0.0;
                for (int i = 0; i < kWTets; i++) {
                    double e4[4], b4[4], a4[4];
                    int iv = 0, n = 0;
#pragma unroll
                    for (int v = 0; v < 4; v++) {
                        const int sl = c_tetra.slot[kWTets * lane8 + i][v];
                        e4[v] = sE[sl][slot];
                        b4[v] = sB[sl][slot];
                        a4[v] = sA[sl][slot];
                        if (sl == kTet.self) iv = v;
                    }
                    if (kind[i] == 1) {
#pragma unroll
                        for (int v = 0; v < 4; v++) {
                            pc[0].e[v] = e4[v];
                            pc[0].lam[v] = v == iv ? 1.0 : 0.0;
                        }
                        n = 1;
                    } else if (kind[i] == 2) {
                        clipped_pieces(e4, b4, a4, ef, iv, pc, n);
                    }
                    for (int q = 0; q < n; q++) {
                        // sum_j lam_j h_m(s_0..s_3, s_j) with h_m(.., s_j) = h_m(s_0..s_3) + s_j h_{m-1}(.., s_j)
                        double y[4], P[4], H[4], lam[4];
#pragma unroll
                        for (int j = 0; j < 4; j++) {
                            y[j] = (pc[q].e[j] - c) * ri;
                            lam[j] = pc[q].lam[j];
                            P[j] = 1.0;
                            H[j] = 0.0;
                        }
#pragma unroll
                        for (int m = 0; m < kMoments; m++) {
#pragma unroll
                            for (int j = 0; j < 4; j++) {
                                H[j] = P[3] + y[j] * H[j];
                                mu[m] += lam[j] * H[j];
                            }
                            P[0] *= y[0];
#pragma unroll
                            for (int j = 1; j < 4; j++) P[j] = P[j - 1] + y[j] * P[j];
                        }
                    }
                }
#pragma unroll
                for (int m = 0; m < kMoments; m++) {
                    const double h = sum8(mu[m]);
                    if (lane8 == 0) sMu[m][slot] = c_series.f[m + 4] * h;
                }
            }
        }
    }
    __syncthreads();
    for (int fc = fa; fc < fb; fc += kWFreqs) {
        if (tid == 0) sNq = 0;
        if (tid < kWPairs) sCut[tid] = 0;
        __syncthreads();
        // the series: thread (pair, frequency)
        const int pr = tid & (kWPairs - 1);
        const long p = p0 + pr;
        const double c = SERIES ? sC[pr] : 0.0, R = SERIES ? sR[pr] : 0.0;
        for (int f = fc + tid / kWPairs; f < min(fb, fc + kWFreqs); f += kWLanes) {
            const double2 om = make_double2(freq[f].x * ha, freq[f].y * ha);
            // on the imaginary axis without broadening z' = z*, and since the
            // corner energies are real I_v(z*) = conj(I_v(z)): x = 2 Re sum I_v(z)/6
            const bool conj_pair = dl == 0.0 && om.x == 0.0;
            double2 x = make_double2(0.0, 0.0);
            int far = 0;   // bit zi: z (0) or z' (1) is left to the exact integrals
            if constexpr (!SERIES) {
                if (p < npair) far = conj_pair ? 1 : 3;
            } else if (p < npair && sSome[pr]) {
                for (int zi = 0; zi < (conj_pair ? 1 : 2); zi++) {
                    const double2 u = zi ? make_double2(-om.x - c, -om.y + dl) : make_double2(om.x - c, om.y + dl);
                    const double a2 = u.x * u.x + u.y * u.y;
                    if (!(R * R <= kSeriesRatio * kSeriesRatio * a2)) {
                        far |= 1 << zi;
                        continue;
                    }
                    const double2 ui = make_double2(u.x / a2, -u.y / a2), r = cscale(ui, R);
                    // terms until (R/|u|)^n < 1e-16
                    const float lr = -0.5f * __logf((float)(R * R / a2) + 1e-30f);
                    const int n = min(kMoments, (int)(36.9f / lr) + 2);
                    double2 s = make_double2(0.0, 0.0);
#pragma unroll 4
                    for (int m = n - 1; m >= 0; m--) {
                        const double t = s.x * r.x - s.y * r.y + sMu[m][pr];
                        s.y = s.x * r.y + s.y * r.x;
                        s.x = t;
                    }
                    x = cadd(x, cmul(s, ui));
                }
                if (conj_pair) x = make_double2(2.0 * x.x, 0.0);
            }
            if (far) {
                if (!METAL || sSome[pr] == 2) sQueue[atomicAdd(&sNq, 1)] = ((f - fc) * kWPairs + pr) * 4 + far;
                else atomicOr(&sCut[pr], (unsigned)far << 2 * (f - fc));
            }
            if (SERIES && p < npair) w[(long)f * npair + p] = cscale(x, sFac[pr] * (1.0 / 6.0));
        }
        __syncthreads();
        // the rest, 32 entries at a time: one thread per (entry, tetrahedron),
        // then one per entry adds its 24 values in order
        const int nq = sNq;
        for (int base = 0; base < nq; base += kWPairs) {
            const int n = min(kWPairs, nq - base);
            const bool on = slot < n;
            const int own = on ? sQueue[base + slot] : 0;
            double2 x = make_double2(0.0, 0.0);
            for (int zi = 0; zi < 2; zi++) {
                auto zof = [&](int item) {
                    const double2 v = freq[fc + (item >> 2) / kWPairs];
                    const double2 om = make_double2(v.x * ha, v.y * ha);
                    return zi ? make_double2(-om.x, -om.y + dl) : make_double2(om.x, om.y + dl);
                };
                for (int u = tid; u < n * 15; u += kWThreads) {
                    const int it = u / 15, j = u - it * 15, item = sQueue[base + it];
                    if (!(item >> zi & 1)) continue;
                    const double2 zz = zof(item);
                    sL[it][j] = clog_d(make_double2(zz.x - sE[j][(item >> 2) & (kWPairs - 1)], zz.y));
                }
                __syncthreads();
                for (int u = tid; u < n * 24; u += kWThreads) {
                    const int it = u / 24, tt = u - it * 24, item = sQueue[base + it];
                    if (!(item >> zi & 1)) continue;
                    double xs[5];
                    double2 ls[5];
#pragma unroll
                    for (int v = 0; v < 5; v++) {
                        const int sl = v < 4 ? c_tetra.slot[tt][v] : kTet.self;
                        xs[v] = sE[sl][(item >> 2) & (kWPairs - 1)];
                        ls[v] = sL[it][sl];
                    }
                    sort5(xs, ls);
                    sVal[u] = dd4_sorted(zof(item), xs, ls);
                }
                __syncthreads();
                if (lane8 == 0 && (own >> zi & 1))
                    for (int i = 0; i < 24; i++) x = cadd(x, sVal[slot * 24 + i]);
            }
            if (on && lane8 == 0) {
                const int pi = (own >> 2) & (kWPairs - 1), f = fc + (own >> 2) / kWPairs;
                if (dl == 0.0 && freq[f].x == 0.0) x = make_double2(2.0 * x.x, 0.0);   // z' = z*
                double2 *o = w + (long)f * npair + p0 + pi;
                if (SERIES) *o = cadd(*o, cscale(x, sFac[pi] * (1.0 / 6.0)));
                else *o = cscale(cscale(x, 1.0 / 6.0), sFac[pi]);
            }
            __syncthreads();
        }
        // METAL, pairs with cut tetrahedra, two at a time: 24 lanes of a wave
        // each cut a pair's tetrahedra into pieces, once for all frequencies;
        // then a wave takes a (pair, frequency) and its lanes the pieces' vertex
        // integrals (up to 864), the four of a piece side by side sharing its
        // four logarithms
        if constexpr (METAL) {
            const int wave = tid >> 6, lane = tid & 63;
            unsigned todo = (unsigned)__ballot(sCut[lane & (kWPairs - 1)] != 0);   // the same in every wave
            while (todo) {
                int pis[kCutPairs];
#pragma unroll
                for (int g = 0; g < kCutPairs; g++) {
                    pis[g] = todo ? __ffs(todo) - 1 : -1;
                    todo &= todo - 1;
                }
                __syncthreads();
                const int mine = wave == 0 ? pis[0] : wave == 1 ? pis[1] : -1;
                if (lane < 24 && mine >= 0) {
                    double e4[4], b4[4], a4[4];
                    bool all_in = true, none_b = true, none_a = true;
                    int iv = 0, n = 0;
                    Piece pc[kMaxPieces];
#pragma unroll
                    for (int v = 0; v < 4; v++) {
                        const int sl = c_tetra.slot[lane][v];
                        e4[v] = sE[sl][mine];
                        b4[v] = sB[sl][mine];
                        a4[v] = sA[sl][mine];
                        if (sl == kTet.self) iv = v;
                        all_in = all_in && b4[v] < ef && a4[v] > ef;
                        none_b = none_b && !(b4[v] < ef);
                        none_a = none_a && !(a4[v] > ef);
                    }
                    if (all_in) {
#pragma unroll
                        for (int v = 0; v < 4; v++) {
                            pc[0].e[v] = e4[v];
                            pc[0].lam[v] = v == iv ? 1.0 : 0.0;
                        }
                        n = 1;
                    } else if (!none_b && !none_a) {
                        clipped_pieces(e4, b4, a4, ef, iv, pc, n);
                    }
                    // place of this tetrahedron's pieces: the counts before it
                    int at = n;
#pragma unroll
                    for (int d = 1; d < 32; d <<= 1) {
                        const int o = __shfl_up(at, d);
                        if (lane >= d) at += o;
                    }
                    if (lane == 23) sNpc[wave] = at;
                    at -= n;
                    for (int i = 0; i < n; i++) sPc[wave][at + i] = pc[i];
                }
                __syncthreads();
                int turn = 0;
                for (int g = 0; g < kCutPairs; g++) {
                    const int pi = pis[g];
                    if (pi < 0) break;
                    const int units = 4 * sNpc[g];
                    for (int fi = 0; fi < kWFreqs; fi++) {
                        const unsigned far = sCut[pi] >> 2 * fi & 3u;
                        if (!far || (turn++ & (kWThreads / 64 - 1)) != wave) continue;
                        const int f = fc + fi;
                        const double2 om = make_double2(freq[f].x * ha, freq[f].y * ha);
                        const bool conj_pair = dl == 0.0 && om.x == 0.0;
                        // partial sums over lanes of units 64 h + lane + 256 j
                        double2 x[4];
#pragma unroll
                        for (int h = 0; h < 4; h++) x[h] = make_double2(0.0, 0.0);
                        for (int zi = 0; zi < 2; zi++) {
                            if (!(far >> zi & 1)) continue;
                            const double2 zz = zi ? make_double2(-om.x, -om.y + dl) : make_double2(om.x, om.y + dl);
                            for (int u = lane, h = 0; u < units; u += 64, h++) {
                                const Piece &pc = sPc[g][u >> 2];
                                const double lam = pc.lam[u & 3];
                                double xs[5];
                                double2 ls[5];
                                xs[4] = pc.e[u & 3];
                                ls[4] = clog_d(make_double2(zz.x - xs[4], zz.y));
                                ls[0] = make_double2(dpp<0x00>(ls[4].x), dpp<0x00>(ls[4].y));
                                ls[1] = make_double2(dpp<0x55>(ls[4].x), dpp<0x55>(ls[4].y));
                                ls[2] = make_double2(dpp<0xAA>(ls[4].x), dpp<0xAA>(ls[4].y));
                                ls[3] = make_double2(dpp<0xFF>(ls[4].x), dpp<0xFF>(ls[4].y));
                                if (lam == 0.0) continue;
#pragma unroll
                                for (int v = 0; v < 4; v++) xs[v] = pc.e[v];
                                sort5(xs, ls);
                                const double2 d = dd4_sorted(zz, xs, ls);
#pragma unroll
                                for (int t = 0; t < 4; t++) {
                                    if ((h & 3) != t) continue;
                                    x[t].x += lam * d.x;
                                    x[t].y += lam * d.y;
                                }
                            }
                        }
#pragma unroll
                        for (int h = 0; h < 4; h++)
#pragma unroll
                            for (int o = 1; o < 64; o <<= 1) {
                                x[h].x += __shfl_xor(x[h].x, o);
                                x[h].y += __shfl_xor(x[h].y, o);
                            }
                        if (lane == 0) {
                            double2 v = cadd(cadd(x[0], x[1]), cadd(x[2], x[3]));
                            if (conj_pair) v = make_double2(2.0 * v.x, 0.0);
                            double2 *o = w + (long)f * npair + p0 + pi;
                            *o = cadd(*o, cscale(v, sFac[pi] * (1.0 / 6.0)));
                        }
                    }
                }
            }
        }
        __syncthreads();
    }
}

// X at the mesh point (RP_W_SAMPLING), one thread per (pair, frequency).
__global__ void __launch_bounds__(256)
k_weights_sampling(int K1, int K2, int K3, int q1, int q2, int q3, int nband, const double *E, const double *T,
                   int o0, int nO, int e0, int nE, int k0, long npair, int nfreq, const double2 *freq, double delta,
                   double2 *w)
{
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
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
    const int kq = (mesh_wrap(n1 + q1, K1) * K2 + mesh_wrap(n2 + q2, K2)) * K3 + mesh_wrap(n3 + q3, K3);
    const double e = (E[(long)kq * nband + a] - E[(long)k * nband + b]) * ha;
    const double2 x = cadd(crecip(make_double2(om.x - e, om.y + dl)), crecip(make_double2(-om.x - e, -om.y + dl)));
    double fac = 2.0 / (double)(K1 * K2 * K3);
    if (T) fac *= 1.0 - T[(long)kq * nband + a] * T[(long)k * nband + b];
    w[t] = cscale(x, fac);
}

// ---- Fermi-surface weights of the intraband term (Eq. plasma) ----
//
// D_v = (1/|T|) int_T lambda_v delta(e - E) d^3k for the linear interpolant e
// of the corner energies over T.  The section {e = E} is a triangle (one
// corner on one side of E) or a quadrilateral (two on each side) with its
// corners on the edges that E separates.  In the reference tetrahedron (corner
// 0 at the origin, corner j at the j-th unit vector, volume 1/6) the delta
// turns the volume integral into a section integral over |grad e|, and the
// mean of the linear lambda_v over each triangle of the section is the mean of
// its corner values.
__device__ double fermi_corner(const double (&e)[4], int v, double E)
{
    int lo[4], hi[4], nl = 0, nh = 0;
#pragma unroll
    for (int c = 0; c < 4; c++) {
        if (e[c] < E) lo[nl++] = c;
        else hi[nh++] = c;
    }
    if (nl == 0 || nh == 0) return 0.0;
    const double gx = e[1] - e[0], gy = e[2] - e[0], gz = e[3] - e[0];
    const double gn = sqrt(gx * gx + gy * gy + gz * gz);
    double P[4][3], L[4];
    int np = 0;
    // the point of edge (i, j) where e = E, and lambda_v there
    auto edge = [&](int i, int j) {
        const double t = (E - e[i]) / (e[j] - e[i]);
#pragma unroll
        for (int d = 0; d < 3; d++) P[np][d] = (i == d + 1 ? 1.0 - t : 0.0) + (j == d + 1 ? t : 0.0);
        L[np] = (v == i ? 1.0 - t : 0.0) + (v == j ? t : 0.0);
        np++;
    };
    if (nl == 1) {
        edge(lo[0], hi[0]);
        edge(lo[0], hi[1]);
        edge(lo[0], hi[2]);
    } else if (nh == 1) {
        edge(lo[0], hi[0]);
        edge(lo[1], hi[0]);
        edge(lo[2], hi[0]);
    } else {
        // in cyclic order: consecutive corners share a face of T
        edge(lo[0], hi[0]);
        edge(lo[0], hi[1]);
        edge(lo[1], hi[1]);
        edge(lo[1], hi[0]);
    }
    auto area = [&](int a, int b, int c) {
        const double u0 = P[b][0] - P[a][0], u1 = P[b][1] - P[a][1], u2 = P[b][2] - P[a][2];
        const double w0 = P[c][0] - P[a][0], w1 = P[c][1] - P[a][1], w2 = P[c][2] - P[a][2];
        const double x = u1 * w2 - u2 * w1, y = u2 * w0 - u0 * w2, z = u0 * w1 - u1 * w0;
        return 0.5 * sqrt(x * x + y * y + z * z);
    };
    double sum = area(0, 1, 2) * (L[0] + L[1] + L[2]) / 3.0;
    if (np == 4) sum += area(0, 2, 3) * (L[0] + L[2] + L[3]) / 3.0;
    return 6.0 * sum / gn;
}

// One thread per (k, band a in [b0, b0 + nb)): the Fermi-surface weight
// D(k) = (1/(6 N_k)) sum over the 24 tetrahedra around k of k's corner weight,
// times (1 - T^2), times p p^T: contrib[t] = {xx, yy, zz, xy, xz, yz}.
__global__ void __launch_bounds__(256)
k_fermi_plasma(int K1, int K2, int K3, int nband, const double *__restrict__ E, const double *__restrict__ T,
               int b0, int nb, double ef, const double *__restrict__ p, double *__restrict__ contrib)
{
    const int nk = K1 * K2 * K3;
    const long t = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (long)nk * nb) return;
    const int k = (int)(t / nb), a = b0 + (int)(t - (long)k * nb);
    const int n1 = k / (K2 * K3), n2 = (k / K3) % K2, n3 = k % K3;
    const double ha = 1.0 / kHartreeEv;
    double e15[15];
#pragma unroll
    for (int j = 0; j < 15; j++) {
        const int code = kTet.nbr[j];
        const int kv = (mesh_wrap(n1 + code / 9 - 1, K1) * K2 + mesh_wrap(n2 + (code / 3) % 3 - 1, K2)) * K3 +
                       mesh_wrap(n3 + code % 3 - 1, K3);
        e15[j] = E[(long)kv * nband + a] * ha;
    }
    double D = 0.0;
#pragma unroll
    for (int tt = 0; tt < 24; tt++) {
        double e[4];
        int v = 0;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            e[c] = e15[kTet.slot[tt][c]];
            if (kTet.slot[tt][c] == kTet.self) v = c;
        }
        D += fermi_corner(e, v, ef);
    }
    D /= 6.0 * nk;
    if (T) D *= 1.0 - T[(long)k * nband + a] * T[(long)k * nband + a];
    const double px = p[3 * t], py = p[3 * t + 1], pz = p[3 * t + 2];
    double *o = contrib + 6 * t;
    o[0] = D * px * px;
    o[1] = D * py * py;
    o[2] = D * pz * pz;
    o[3] = D * px * py;
    o[4] = D * px * pz;
    o[5] = D * py * pz;
}

// out[q] = sum_t c[t][q], q < 6, in one block
__global__ void __launch_bounds__(256) k_sum6(long n, const double *__restrict__ c, double *__restrict__ out)
{
    __shared__ double red[6][256];
    const int tid = threadIdx.x;
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (long i = tid; i < n; i += 256)
#pragma unroll
        for (int q = 0; q < 6; q++) s[q] += c[6 * i + q];
#pragma unroll
    for (int q = 0; q < 6; q++) red[q][tid] = s[q];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (tid < w)
#pragma unroll
            for (int q = 0; q < 6; q++) red[q][tid] += red[q][tid + w];
        __syncthreads();
    }
    if (tid < 6) out[tid] = red[tid][0];
}

}  // namespace

void launch_weights(hipStream_t s, const int kmesh[3], const int iq[3], int nband,
                    const double *E_eV, const double *T, int o0, int o1, int e0, int e1,
                    int k0, int k1, int nfreq, const double2 *freq_eV, double delta_eV,
                    int mode, double ef_eV, double2 *w, bool direct)
{
    const long npair = (long)(k1 - k0) * (e1 - e0) * (o1 - o0);
    const long tot = npair * nfreq;
    if (tot == 0) return;
    if (mode == RP_W_SAMPLING) {
        hipLaunchKernelGGL(k_weights_sampling, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, kmesh[0], kmesh[1],
                           kmesh[2], iq[0], iq[1], iq[2], nband, E_eV, T, o0, o1 - o0, e0, e1 - e0, k0, npair, nfreq,
                           freq_eV, delta_eV, w);
        return;
    }
    // the split forms at complex frequencies: every difference by itself (weights_direct.hip says why)
    if (direct && mode == RP_W_TETRA_METAL) {
        launch_weights_direct(s, kmesh, iq, nband, E_eV, T, o0, o1, e0, e1, k0, k1, nfreq, freq_eV, delta_eV,
                              ef_eV / kHartreeEv, w);
        return;
    }
    // frequencies per workgroup: all of them where the pairs alone give two
    // workgroups per CU (each forms its pairs' moments once), else fewer, down
    // to two: the integrals of the near frequencies are the longest part
    const long blocks = (npair + kWPairs - 1) / kWPairs;
    const int want = (int)std::min<long>((nfreq + kWMinFreqs - 1) / kWMinFreqs, std::max<long>(1, 512 / blocks));
    const int fper = (nfreq + want - 1) / want;
    const dim3 grid((unsigned)blocks, (unsigned)((nfreq + fper - 1) / fper));
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(kWThreads), 0, s, kmesh[0], kmesh[1], kmesh[2], iq[0], iq[1], iq[2], nband,
                           E_eV, T, o0, o1 - o0, e0, e1 - e0, k0, npair, nfreq, fper, freq_eV, delta_eV,
                           ef_eV / kHartreeEv, w);
    };
    if (mode == RP_W_TETRA_METAL) go(k_weights<true, true>);
    else if (direct) go(k_weights<false, false>);
    else go(k_weights<false, true>);
}

void launch_fermi_plasma(hipStream_t s, const int kmesh[3], int nband, const double *E_eV, const double *T, int b0,
                         int b1, double ef_eV, const double *p, double *contrib, double *out)
{
    const long n = (long)kmesh[0] * kmesh[1] * kmesh[2] * (b1 - b0);
    if (n > 0)
        hipLaunchKernelGGL(k_fermi_plasma, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, kmesh[0], kmesh[1],
                           kmesh[2], nband, E_eV, T, b0, b1 - b0, ef_eV / kHartreeEv, p, contrib);
    hipLaunchKernelGGL(k_sum6, dim3(1), dim3(256), 0, s, n, contrib, out);
}

}  // namespace rp
