// Step a6 in FP64 (Eq. chi): chi_GG'(w) (+)= sum_p w_p(w) M_p(G) conj(M_p(G'))
// on FP64 matrix cores (v_mfma_f64_16x16x4f64).
//
// Each pair p contributes a rank-one term, so over a batch of pairs chi(w) is
// the complex product (M o w(w))^T conj(M) with the pair index as the
// contraction dimension.  Complex arithmetic uses four real products:
//   Re chi += Re(a) Re(b) + Im(a) Im(b),   Im chi += Im(a) Re(b) - Re(a) Im(b)
// with a = w_p M_p(G) and b = M_p(G').
//
// Tiling: a 256-thread block owns 64 rows G and 16 CB columns G' (CB = 2, 3, 4
// or 5) for two frequencies (the last block one, where they are odd); wave w owns 16 of the rows and all the
// columns, so that each weighted row value feeds CB column blocks.  What
// bounds it is the FP64 matrix-core rate: back-to-back 16x16x4 ops with their
// accumulators in ordinary registers reach 77.3 TFLOP/s on this card, and
// every FP64 vector op costs them about 3 cycles.  Hence at most 160
// accumulator registers and two waves per SIMD: one wave's LDS reads, weight
// products and barriers hide behind the other's matrix work, and the file is
// compiled with the accumulators in ordinary registers.  (A 64 x 64 tile for
// four frequencies on one wave per SIMD kept its 256 accumulators in AGPRs
// and moved all of them to and fro once per chunk: 48.8 TFLOP/s on 16 000
// pairs at N_G = 1500 and 20 frequencies, now 65.0; 58.8 of the Hermitian half.)
//
// The pair dimension is consumed in chunks of 16 pairs staged through LDS with
// two buffers: while the matrix cores work on one chunk, the next chunk's rows
// stream from HBM/L2 straight into the other buffer (global_load_lds, no
// staging registers).  Rows and pairs past the end are clamped to valid
// addresses: clamped rows are never stored and clamped pairs carry zero weight.
//
// Small N_G gives far fewer tiles than the 512 workgroups the chip holds; the
// pairs are then cut into slices (grid y), each slice writes an FP64 partial
// chi and k_chi_f64_sum adds them in slice order (see f64_shape).  A q-point of
// 12 288 pairs at N_G = 89 and 10 frequencies (16^3 grid, run_q) went from
// 13.95 to 6.84 ms with it, one of 27 648 at N_G = 300 and 16 (24^3, q -> 0)
// from 23.7 to 13.2 ms.
#include <type_traits>

#include "fft_lds.h"

namespace rp {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kT = 64;     // rows per tile
constexpr int kKC = 16;    // pairs per chunk

__device__ __forceinline__ d4 mfma64(double a, double b, d4 c)
{
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ void dma16(const void *src, void *lds)
{
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds, 16, 0, 0);
}

// Tiles of a matrix of n rows: 64 rows x tc columns each, row-major.  herm
// keeps those that hold an element on or above the diagonal: column tiles
// from rt * 64 / tc on.
__host__ __device__ __forceinline__ int first_ct(int rt, int tc, int herm) { return herm ? rt * kT / tc : 0; }

__device__ __forceinline__ void tile_of(int id, int nct, int tc, int herm, int &rt, int &ct)
{
    rt = 0;
    while (id >= nct - first_ct(rt, tc, herm)) {
        id -= nct - first_ct(rt, tc, herm);
        rt++;
    }
    ct = first_ct(rt, tc, herm) + id;
}

// herm: the weights are real (imaginary frequencies, no broadening), so chi
// is Hermitian: their imaginary parts (rounding residue) are dropped, only
// the elements on and above the diagonal are stored, each with its mirror
// image.  nslice > 1: slice y of the chunks goes to out + y * nfreq * ng^2
// (no mirror, no accumulation), else into chi = out.
template <int CB>
__global__ void __launch_bounds__(256, 2)
k_chi_f64(long npair, int ng, const double2 *__restrict__ M, int nfreq, const double2 *__restrict__ w,
          int accumulate, int herm, int nslice, double2 *__restrict__ out)
{
    constexpr int NW = 2, TC = 16 * CB;
    // [stage][pair][64 rows], [stage][pair][TC columns], then [stage][NW][pair] weights
    __shared__ double2 sA[2][kKC][kT];
    __shared__ double2 sB[2][kKC][TC];
    __shared__ double2 sw[2][NW][kKC];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int li = lane & 15, lk = lane >> 4;
    int rt, ct;
    tile_of(blockIdx.x, (ng + TC - 1) / TC, TC, herm, rt, ct);
    const int rt0 = rt * kT, ct0 = ct * TC;
    const int wr = wave * 16;
    const int f0 = blockIdx.z * NW;
    const long nchunk = (npair + kKC - 1) / kKC;
    const long c0 = nchunk * blockIdx.y / nslice, c1 = nchunk * (blockIdx.y + 1) / nslice;
    const bool live = rt0 + wr < ng;   // a wave whose rows all lie past the end only moves data

    // DMA assignment: wave w moves pairs 4w..4w+3 of both operands (columns
    // past the 64th, CB = 5, in a second piece)
    const int rowA = min(rt0 + lane, ng - 1);
    const int colB = min(ct0 + lane, ng - 1), colB2 = min(ct0 + 64 + lane, ng - 1);
    auto issue = [&](int stg, long c) {
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int pp = wave * 4 + t;
            const long p = min(c * kKC + pp, npair - 1);
            dma16(M + p * ng + rowA, &sA[stg][pp][0]);
            if (CB >= 4 || lane < TC) dma16(M + p * ng + colB, &sB[stg][pp][0]);
            if (CB == 5 && lane < TC - 64) dma16(M + p * ng + colB2, &sB[stg][pp][CB == 5 ? 64 : 0]);
        }
    };
    // weights: thread tid < NW*16 stages one value through a register
    const int wiw = tid / kKC, wpp = tid % kKC;
    auto wload = [&](long c) -> double2 {
        const long p = c * kKC + wpp;
        if (tid < NW * kKC && p < npair && f0 + wiw < nfreq) {
            const double2 v = w[(long)(f0 + wiw) * npair + p];
            return make_double2(v.x, herm ? 0.0 : v.y);
        }
        return make_double2(0.0, 0.0);
    };

    d4 accR[NW][CB], accI[NW][CB];
#pragma unroll
    for (int iw = 0; iw < NW; iw++)
#pragma unroll
        for (int cb = 0; cb < CB; cb++) {
            accR[iw][cb] = d4{0.0, 0.0, 0.0, 0.0};
            accI[iw][cb] = d4{0.0, 0.0, 0.0, 0.0};
        }

    if (c0 < c1) {
        issue(0, c0);
        const double2 w0 = wload(c0);
        if (tid < NW * kKC) sw[0][wiw][wpp] = w0;
    }
    auto chunks = [&](auto freqs) {
        constexpr int NF = decltype(freqs)::value;
        for (long c = c0; c < c1; c++) {
            const int stg = (int)((c - c0) & 1);
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            double2 wnext = make_double2(0.0, 0.0);
            if (c + 1 < c1) {
                issue(stg ^ 1, c + 1);
                wnext = wload(c + 1);
            }
            if (live) {
#pragma unroll
                for (int s = 0; s < kKC / 4; s++) {
                    const int pp = 4 * s + lk;
                    const double2 av = sA[stg][pp][wr + li];
                    double2 bv[CB];
#pragma unroll
                    for (int cb = 0; cb < CB; cb++) bv[cb] = sB[stg][pp][cb * 16 + li];
                    double2 a[NF];
#pragma unroll
                    for (int iw = 0; iw < NF; iw++) a[iw] = cmul(av, sw[stg][iw][pp]);
                    // first halves of the four products for all accumulators, then the
                    // second halves: dependent matrix-core ops are 2 NF CB instructions apart
#pragma unroll
                    for (int iw = 0; iw < NF; iw++)
#pragma unroll
                        for (int cb = 0; cb < CB; cb++) {
                            accR[iw][cb] = mfma64(a[iw].x, bv[cb].x, accR[iw][cb]);
                            accI[iw][cb] = mfma64(a[iw].y, bv[cb].x, accI[iw][cb]);
                        }
#pragma unroll
                    for (int iw = 0; iw < NF; iw++)
#pragma unroll
                        for (int cb = 0; cb < CB; cb++) {
                            accR[iw][cb] = mfma64(a[iw].y, bv[cb].y, accR[iw][cb]);
                            accI[iw][cb] = mfma64(-a[iw].x, bv[cb].y, accI[iw][cb]);
                        }
                }
            }
            // the other stage's weights: its readers finished before this chunk's barrier
            if (c + 1 < c1 && tid < NW * kKC) sw[stg ^ 1][wiw][wpp] = wnext;
        }
    };
    if (f0 + 1 < nfreq) chunks(std::integral_constant<int, 2>{});
    else chunks(std::integral_constant<int, 1>{});

    // result register r of lane (li, lk) holds row lk + 4 r, column li of a 16x16 block
    const long n2 = (long)ng * ng;
    const bool part = nslice > 1;
#pragma unroll
    for (int iw = 0; iw < NW; iw++) {
        if (f0 + iw >= nfreq) continue;
        double2 *C = out + ((part ? (long)blockIdx.y * nfreq : 0) + f0 + iw) * n2;
#pragma unroll
        for (int cb = 0; cb < CB; cb++)
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const int i = rt0 + wr + lk + 4 * r;
                const int j = ct0 + cb * 16 + li;
                if (i < ng && j < ng && (!herm || i <= j)) {
                    const double2 a = make_double2(accR[iw][cb][r], accI[iw][cb][r]);
                    const long idx = (long)i * ng + j;
                    C[idx] = accumulate && !part ? cadd(C[idx], a) : a;
                    if (herm && !part && i < j) {
                        const long jdx = (long)j * ng + i;
                        const double2 b = make_double2(a.x, -a.y);
                        C[jdx] = accumulate ? cadd(C[jdx], b) : b;
                    }
                }
            }
    }
}

// chi (+)= the slices' partial sums, in slice order; one thread per element.
// Bound by reading the partials, which the contraction has just left in the
// caches.  herm: an element below the diagonal takes its mirror image's.
__global__ void __launch_bounds__(256)
k_chi_f64_sum(int ng, int nfreq, int nslice, int accumulate, int herm, const double2 *__restrict__ part,
              double2 *__restrict__ chi)
{
    const long n2 = (long)ng * ng, n = n2 * nfreq;
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const long f = t / n2, e = t - f * n2;
    const int i = (int)(e / ng), j = (int)(e - (long)i * ng);
    const bool mirror = herm && i > j;
    const long src = f * n2 + (mirror ? (long)j * ng + i : e);
    double2 s = part[src];
    for (int k = 1; k < nslice; k++) s = cadd(s, part[k * n + src]);
    if (mirror) s.y = -s.y;
    chi[t] = accumulate ? cadd(chi[t], s) : s;
}

// Launch shape of one contraction: column blocks per tile and slices of the
// pairs.
struct F64Shape {
    int cb = 4, nslice = 1;
    unsigned tiles = 0;
};

unsigned f64_tiles(int ng, int cb, bool herm)
{
    const int tc = 16 * cb, nrt = (ng + kT - 1) / kT, nct = (ng + tc - 1) / tc;
    unsigned n = 0;
    for (int rt = 0; rt < nrt; rt++) n += (unsigned)(nct - first_ct(rt, tc, herm));
    return n;
}

// cb: the least time for the tiles formed, at the rates measured for each
// width (TFLOP/s executed on 16 000 pairs, N_G = 1500, 20 frequencies: 62, 64,
// 66 and 67 for 2, 3, 4 and 5 column blocks: the weight products and row reads
// are shared by more).  nslice: the chip holds 512 workgroups (two per CU); u
// tiles x frequency pairs take ceil(u s / 512) rounds of nchunk / s chunks,
// plus about six chunks' time per round to fill and store, plus the partial
// tiles written and read (about 0.0075 chunk times each).  The s of least cost
// is taken, with at least eight chunks per slice.  It depends on the sizes alone,
// never on the room an entry point has, so that all of them sum alike: the
// partial chi of all frequencies is at most kF64PartMax (16 slices of 20
// frequencies at N_G = 200 are 205 MB), that of one frequency at most what the
// frequencies and weights leave of the fixed workspace where they fit in it.
constexpr size_t kF64PartMax = (size_t)256 << 20;

F64Shape f64_shape(long npair, int ng, int nfreq, bool herm)
{
    const size_t fixed = align256(sizeof(double2) * nfreq) + align256(sizeof(double2) * (size_t)std::max(1L, npair) * nfreq);
    const size_t one_max = fixed <= kScratchBytes ? kScratchBytes - fixed : kF64PartMax;
    F64Shape best;
    constexpr double rate[] = {62.0, 64.0, 66.0, 67.0};
    double least = 1e300;
    for (int cb = 5; cb >= 2; cb--) {
        const double t = (double)f64_tiles(ng, cb, herm) * cb / rate[cb - 2];
        if (t < least) {
            least = t;
            best.cb = cb;
        }
    }
    best.tiles = f64_tiles(ng, best.cb, herm);
    const double u = 0.5 * best.tiles * nfreq;
    const long nchunk = (npair + kKC - 1) / kKC;
    double cost = 1e300;
    for (int s = 1; s <= 64 && (s == 1 || nchunk / s >= 8); s++) {
        const size_t one = sizeof(double2) * (size_t)s * ng * ng;
        if (s > 1 && (one * nfreq > kF64PartMax || one > one_max)) break;
        const double c = std::ceil(u * s / 512.0) * ((double)nchunk / s + 6.0) + (s > 1 ? 0.0075 * u * s : 0.0);
        if (c < cost) {
            cost = c;
            best.nslice = s;
        }
    }
    return best;
}

}  // namespace

size_t chi_f64_part_bytes(long npair, int ng, int nfreq, bool herm)
{
    const F64Shape sh = f64_shape(npair, ng, nfreq, herm);
    return sh.nslice > 1 ? sizeof(double2) * (size_t)sh.nslice * nfreq * ng * ng : 0;
}

void launch_chi_f64(hipStream_t s, long npair, int ng, const double2 *M, int nfreq, const double2 *w,
                    int accumulate, bool herm, void *part, size_t part_bytes, double2 *chi)
{
    F64Shape sh = f64_shape(npair, ng, nfreq, herm);
    // as many frequencies at a time as part holds (in twos, like the kernel's)
    const long n2 = (long)ng * ng;
    const size_t fit = part_bytes / (sizeof(double2) * (size_t)sh.nslice * n2);
    if (!fit) sh.nslice = 1;
    const int per = sh.nslice == 1 || fit >= (size_t)nfreq ? nfreq : fit > 1 ? (int)fit & ~1 : 1;
    for (int fa = 0; fa < nfreq; fa += per) {
        const int nf = std::min(per, nfreq - fa);
        double2 *x = chi + fa * n2, *out = sh.nslice > 1 ? (double2 *)part : x;
        const dim3 grid(sh.tiles, (unsigned)sh.nslice, (unsigned)((nf + 1) / 2));
        auto go = [&](auto kern) {
            hipLaunchKernelGGL(kern, grid, dim3(256), 0, s, npair, ng, M, nf, w + fa * npair, accumulate, (int)herm,
                               sh.nslice, out);
        };
        if (sh.cb == 5) go(k_chi_f64<5>);
        else if (sh.cb == 4) go(k_chi_f64<4>);
        else if (sh.cb == 3) go(k_chi_f64<3>);
        else go(k_chi_f64<2>);
        if (sh.nslice > 1) {
            const long n = nf * n2;
            hipLaunchKernelGGL(k_chi_f64_sum, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, ng, nf, sh.nslice,
                               accumulate, (int)herm, (const double2 *)part, x);
        }
    }
}

}  // namespace rp
