// The tetrahedra around a mesh point, the divided differences of their vertex
// integrals, and the clipping of a tetrahedron by a Fermi level: shared by the
// two weight kernels (tetra.hip, weights_direct.hip).
#pragma once
#include "fft_lds.h"

namespace rp {

namespace {

// The 24 tetrahedra around a mesh point (each mesh cell cut into 6 around its
// (0,0,0)-(1,1,1) diagonal): corners as slots into the 15 distinct
// neighbours, neighbour offsets as codes (d1+1)*9 + (d2+1)*3 + (d3+1).
struct TetraTable {
    int slot[24][4];
    int nbr[15];
    int self;   // slot of k itself (code 13)
    int ntet, nnbr;
};

constexpr TetraTable make_tetra_table()
{
    TetraTable tb{};
    int codes[24][4] = {};
    int cnt = 0;
    const int perms[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    for (int s = 0; s < 8; s++) {                 // k = cell corner + s
        const int so[3] = {(s >> 2) & 1, (s >> 1) & 1, s & 1};
        for (int pi = 0; pi < 6; pi++) {
            int corner[4][3] = {};
            for (int v = 1; v < 4; v++) {
                for (int d = 0; d < 3; d++) corner[v][d] = corner[v - 1][d];
                corner[v][perms[pi][v - 1]] = 1;
            }
            bool has = false;
            for (int v = 0; v < 4; v++)
                if (corner[v][0] == so[0] && corner[v][1] == so[1] && corner[v][2] == so[2]) has = true;
            if (!has) continue;
            for (int v = 0; v < 4; v++)
                codes[cnt][v] = (corner[v][0] - so[0] + 1) * 9 + (corner[v][1] - so[1] + 1) * 3 +
                                (corner[v][2] - so[2] + 1);
            cnt++;
        }
    }
    int n = 0;
    for (int t = 0; t < 24; t++)
        for (int v = 0; v < 4; v++) {
            int found = -1;
            for (int j = 0; j < n; j++)
                if (tb.nbr[j] == codes[t][v]) found = j;
            if (found < 0 && n < 15) {
                tb.nbr[n] = codes[t][v];
                found = n++;
            }
            tb.slot[t][v] = found;
        }
    for (int j = 0; j < n; j++)
        if (tb.nbr[j] == 13) tb.self = j;
    tb.ntet = cnt;
    tb.nnbr = n;
    return tb;
}

constexpr TetraTable kTet = make_tetra_table();
static_assert(kTet.ntet == 24 && kTet.nnbr == 15, "24 tetrahedra over 15 distinct corners expected");

__constant__ TetraTable c_tetra = kTet;

__device__ __forceinline__ double2 clog_d(double2 w)
{
    return make_double2(log(hypot(w.x, w.y)), atan2(w.y, w.x));
}

__device__ __forceinline__ double2 cdiv_real(double2 a, double d) { return make_double2(a.x / d, a.y / d); }

__device__ __forceinline__ double2 crecip(double2 w)
{
    double s = 1.0 / (w.x * w.x + w.y * w.y);
    return make_double2(w.x * s, -w.y * s);
}

// Series coefficients 6 / (m (m-1) (m-2) (m-3)) of the m-th Taylor term,
// m = 4 .. kSeriesMax - 1 (the m-th entry; entries below 4 unused).
constexpr int kSeriesMax = 4 + 96;
struct SeriesTable {
    double f[kSeriesMax];
};
constexpr SeriesTable make_series_table()
{
    SeriesTable t{};
    for (int m = 4; m < kSeriesMax; m++) t.f[m] = 6.0 / ((double)m * (m - 1) * (m - 2) * (m - 3));
    return t;
}
__constant__ SeriesTable c_series = make_series_table();

// sum_{m>=N} g^(m)(c)/m! * h_{m-N}(x_0-c, .., x_N-c) over the N+1 nodes
// x[a..a+N], about the node c = x[cm] with lw = log(z - c)
template <int N>
__device__ __forceinline__ double2 dd_series(double2 z, const double *x, int a, int cm, double2 lw)
{
    const double c = x[cm];
    const double2 w = make_double2(z.x - c, z.y);
    const double2 wi = crecip(w);
    double y[N + 1], P[N + 1];
#pragma unroll
    for (int i = 0; i <= N; i++) {
        y[i] = x[a + i] - c;
        P[i] = 1.0;
    }
    // Taylor coefficients of g(x) = (z-x)^3 log(z-x) about c, with w = z - c:
    // m=0: w^3 L, 1: -(3w^2 L + w^2), 2: (6wL + 5w)/2, 3: -(6L + 11)/6,
    // m>=4: 6 / (m(m-1)(m-2)(m-3)) w^-(m-3)
    double2 sum = make_double2(0.0, 0.0);
    const double2 w2 = cmul(w, w);
#pragma unroll
    for (int m = N; m < 4; m++) {
        if (m > N) {
            P[0] *= y[0];
#pragma unroll
            for (int i = 1; i <= N; i++) P[i] = P[i - 1] + y[i] * P[i];
        }
        double2 coef;
        if (m == 0) coef = cmul(cmul(w2, w), lw);
        else if (m == 1)
            coef = make_double2(-(3.0 * (w2.x * lw.x - w2.y * lw.y) + w2.x), -(3.0 * (w2.x * lw.y + w2.y * lw.x) + w2.y));
        else if (m == 2)
            coef = make_double2(0.5 * (6.0 * (w.x * lw.x - w.y * lw.y) + 5.0 * w.x),
                                0.5 * (6.0 * (w.x * lw.y + w.y * lw.x) + 5.0 * w.y));
        else coef = make_double2(-(6.0 * lw.x + 11.0) / 6.0, -lw.y);
        sum = make_double2(sum.x + coef.x * P[N], sum.y + coef.y * P[N]);
    }
    double2 wp = make_double2(1.0, 0.0);  // w^-(m-3)
    int quiet = 0;
    for (int m = 4; m < kSeriesMax; m++) {
        if (m > N) {
            // raise P to degree m - N: h_k(y_0..y_i) = h_k(y_0..y_{i-1}) + y_i h_{k-1}(y_0..y_i)
            P[0] *= y[0];
#pragma unroll
            for (int i = 1; i <= N; i++) P[i] = P[i - 1] + y[i] * P[i];
        }
        wp = cmul(wp, wi);
        const double fh = c_series.f[m] * P[N];
        const double2 t = make_double2(wp.x * fh, wp.y * fh);
        sum = cadd(sum, t);
        // stop after two consecutive terms below 1e-17 of the sum: the terms
        // shrink at least fourfold, and FP64 resolves 1.1e-16 of the sum
        const double tm = fabs(t.x) + fabs(t.y), sm = fabs(sum.x) + fabs(sum.y);
        if (tm <= 1e-17 * sm) {
            if (++quiet == 2) break;
        } else {
            quiet = 0;
        }
    }
    return sum;
}

// fourth divided difference of g over five sorted nodes x with lw[i] =
// log(z - x[i])
__device__ double2 dd4_sorted(double2 z, const double *x, const double2 *lw)
{
    // entry (a, n) = g[x_a .. x_{a+n}] at slot id(a,n) = 5n - n(n-1)/2 + a
    bool need[15], ser[15];
    double2 val[15];
#pragma unroll
    for (int i = 0; i < 15; i++) { need[i] = false; ser[i] = false; }
    need[14] = true;
    const double zy2 = z.y * z.y;
#pragma unroll
    for (int n = 4; n >= 1; n--) {
#pragma unroll
        for (int a = 0; a + n <= 4; a++) {
            const int id = 5 * n - n * (n - 1) / 2 + a;
            if (!need[id]) continue;
            const int cm = a + n / 2;
            const double dev = fmax(x[a + n] - x[cm], x[cm] - x[a]);
            const double dx = z.x - x[cm];
            if (16.0 * dev * dev <= dx * dx + zy2) {   // 4 dev <= |z - x_cm|
                ser[id] = true;
            } else {
                const int lid = 5 * (n - 1) - (n - 1) * (n - 2) / 2 + a;
                need[lid] = true;
                need[lid + 1] = true;
            }
        }
    }
#pragma unroll
    for (int n = 0; n <= 4; n++) {
#pragma unroll
        for (int a = 0; a + n <= 4; a++) {
            const int id = 5 * n - n * (n - 1) / 2 + a;
            if (!need[id]) continue;
            if (n == 0) {
                const double2 w = make_double2(z.x - x[a], z.y);
                val[id] = cmul(cmul(cmul(w, w), w), lw[a]);
            } else if (ser[id]) {
                if (n == 1) val[id] = dd_series<1>(z, x, a, a + n / 2, lw[a + n / 2]);
                else if (n == 2) val[id] = dd_series<2>(z, x, a, a + n / 2, lw[a + n / 2]);
                else if (n == 3) val[id] = dd_series<3>(z, x, a, a + n / 2, lw[a + n / 2]);
                else val[id] = dd_series<4>(z, x, a, a + n / 2, lw[a + n / 2]);
            } else {
                const int lid = 5 * (n - 1) - (n - 1) * (n - 2) / 2 + a;
                val[id] = cdiv_real(csub(val[lid + 1], val[lid]), x[a + n] - x[a]);
            }
        }
    }
    return val[14];
}

__device__ __forceinline__ int mesh_wrap(int n, int K) { return pmod(n, K); }

// ---- metallic cut: the part of a tetrahedron where E_b < E_F < E_a ----
//
// Points are barycentric coordinates with respect to the tetrahedron T.  A
// tetrahedron P is clipped to {phi < 0} for a linear phi given at its
// corners: one corner inside leaves a corner tetrahedron; two or three leave
// a triangular prism (bottom and top triangles joined by three lateral
// edges), cut into three tetrahedra.

__device__ __forceinline__ void lerp4(const double (&a)[4], const double (&b)[4], double s, double (&out)[4])
{
#pragma unroll
    for (int d = 0; d < 4; d++) out[d] = a[d] + s * (b[d] - a[d]);
}

template <typename Emit>
__device__ __forceinline__ void prism3(const double (&p0)[4], const double (&p1)[4], const double (&p2)[4],
                                       const double (&q0)[4], const double (&q1)[4], const double (&q2)[4], Emit &emit)
{
    emit(p0, p1, p2, q0);
    emit(p1, p2, q0, q1);
    emit(p2, q0, q1, q2);
}

template <typename Emit>
__device__ void clip_tet(const double (&P)[4][4], const double (&phi)[4], Emit &emit)
{
    int in[4], out[4], ni = 0, no = 0;
#pragma unroll
    for (int c = 0; c < 4; c++) {
        if (phi[c] < 0.0) in[ni++] = c;
        else out[no++] = c;
    }
    if (ni == 0) return;
    if (ni == 4) {
        emit(P[0], P[1], P[2], P[3]);
        return;
    }
    // the point where phi = 0 on the edge from inside corner a to outside corner b
    auto cut = [&](int a, int b, double (&q)[4]) { lerp4(P[a], P[b], phi[a] / (phi[a] - phi[b]), q); };
    double x0[4], x1[4], x2[4];
    if (ni == 1) {
        cut(in[0], out[0], x0);
        cut(in[0], out[1], x1);
        cut(in[0], out[2], x2);
        emit(P[in[0]], x0, x1, x2);
    } else if (ni == 3) {
        cut(in[0], out[0], x0);
        cut(in[1], out[0], x1);
        cut(in[2], out[0], x2);
        prism3(P[in[0]], P[in[1]], P[in[2]], x0, x1, x2, emit);
    } else {
        double y1[4], y2[4];
        cut(in[0], out[0], x1);
        cut(in[0], out[1], x2);
        cut(in[1], out[0], y1);
        cut(in[1], out[1], y2);
        prism3(P[in[0]], x1, x2, P[in[1]], y1, y2, emit);
    }
}

__device__ __forceinline__ double det4(const double (&a)[4], const double (&b)[4], const double (&c)[4],
                                       const double (&d)[4])
{
    // expansion along the first row
    auto m3 = [](double a0, double a1, double a2, double b0, double b1, double b2, double c0, double c1, double c2) {
        return a0 * (b1 * c2 - b2 * c1) - a1 * (b0 * c2 - b2 * c0) + a2 * (b0 * c1 - b1 * c0);
    };
    return a[0] * m3(b[1], b[2], b[3], c[1], c[2], c[3], d[1], d[2], d[3]) -
           a[1] * m3(b[0], b[2], b[3], c[0], c[2], c[3], d[0], d[2], d[3]) +
           a[2] * m3(b[0], b[1], b[3], c[0], c[1], c[3], d[0], d[1], d[3]) -
           a[3] * m3(b[0], b[1], b[2], c[0], c[1], c[2], d[0], d[1], d[2]);
}

// sorting network on five keys, carrying the logarithms
__device__ __forceinline__ void sort5(double (&xs)[5], double2 (&ls)[5])
{
#define RP_CSWAP(i, j)                                                                             \
    {                                                                                              \
        const bool sw_ = xs[j] < xs[i];                                                            \
        const double xi_ = xs[i], xj_ = xs[j];                                                     \
        const double2 li_ = ls[i], lj_ = ls[j];                                                    \
        xs[i] = sw_ ? xj_ : xi_;                                                                   \
        xs[j] = sw_ ? xi_ : xj_;                                                                   \
        ls[i] = sw_ ? lj_ : li_;                                                                   \
        ls[j] = sw_ ? li_ : lj_;                                                                   \
    }
    RP_CSWAP(0, 1) RP_CSWAP(3, 4) RP_CSWAP(2, 4) RP_CSWAP(2, 3) RP_CSWAP(0, 3)
    RP_CSWAP(0, 2) RP_CSWAP(1, 4) RP_CSWAP(1, 3) RP_CSWAP(1, 2)
#undef RP_CSWAP
}

}  // namespace

}  // namespace rp
