// Far field between well separated drops (the sum over the other drops'
// regular rules, Sec. 2.1, eq. reg_quadrature) by expansions in solid
// harmonics: each drop's sources as multipole moments about its centre, one
// translation per pair of drops into a local expansion about the target
// drop's centre, and one evaluation of that at the drop's targets.  The sums
// are those of the direct kernels, to a truncation below their rounding.
//
// All five kernels reduce to ten harmonic potentials.  With h = x0 - x,
// y = position relative to the expansion's centre, m_jk = u_j n_k + u_k n_j:
//   phi_k = sum f_k / r,  phi_3 = sum (y.f) / r:
//       S_i = phi_i - y0_k d_i phi_k + d_i phi_3          (h_i/r^3 = -d_i 1/r);
//   Phi_j = sum m_jk h_k / r^3,  Phi_3 = sum y_j m_jk h_k / r^3:
//       D_i = -(Phi_i - y0_j d_i Phi_j + d_i Phi_3)       (-6 h_i h_j h_k u_j n_k / r^5);
//   chi = sum sigma / r: S_L = chi, K* = -n0.grad chi;   lambda = sum sigma (h.n) / r^3 = L.
//
// Solid harmonics (m >= 0 kept; those of -m are (-1)^m times the conjugate):
//   R_n^m = rho^n P_n^m e^{im phi} / (n+m)!,   I_n^m = (n-m)! P_n^m e^{im phi} / rho^{n+1},
//   1/|x - y| = sum conj(R_n^m(y)) I_n^m(x),   M = sum q conj(R),
//   L_n^m = (-1)^n sum_{n'm'} M_{n'}^{m'} I_{n+n'}^{m+m'}(c_i - c_j),   phi(c_i + z) = sum conj(R_n^m(z)) L_n^m.
// The kernels run the recurrences of V = (-1)^m (n-m)! (n+m)! / (2m-1)!! R,
//   V_m^m = (x + iy)^m,   V_{n+1}^m = (2n+1) z V_n^m - (n^2 - m^2) rho^2 V_{n-1}^m,
// which need no division; the factor R / V (scale[]) goes into the moments and
// the evaluation's coefficients.  Lengths are divided by a power of two near
// the largest drop radius, so that the powers stay in range.
#include "expand.h"

#include <algorithm>
#include <cmath>
#include <map>
#include <utility>

#include "ehdbim.h"

namespace ehd {

hipError_t ensure(Expand::Buf& b, size_t bytes)
{
    if (bytes <= b.cap) return hipSuccess;
    if (b.p) (void)hipFree(b.p);
    b = Expand::Buf{};
    const hipError_t e = hipMalloc(&b.p, bytes);
    if (e == hipSuccess) b.cap = bytes;
    else b.p = nullptr;
    return e;
}

}  // namespace ehd

namespace {

typedef double dbl4 __attribute__((ext_vector_type(4)));

constexpr int kOrder = 40;                                   // largest order
// Translation classes: largest order, waves per block, lane sets of 64 lanes;
// a class's waves / sets waves split the source orders.
constexpr int kClassOrder[ehd::kExpClasses] = {14, 19, 29, 40};
constexpr int kClassWaves[ehd::kExpClasses] = {4, 4, 4, 8};
constexpr int kClassSets[ehd::kExpClasses] = {1, 2, 2, 4};
constexpr int kClassRows[ehd::kExpClasses] = {2, 2, 4, 4};   // consecutive degrees n per lane
__host__ __device__ constexpr int class_split(int k) { return kClassWaves[k] / kClassSets[k]; }
constexpr int kField = 17;                                   // source strengths
constexpr int kBasisPad = ((kOrder + 1) * (kOrder + 2) + 15) / 16 * 16;
constexpr int kSrcTile = 4;                                  // sources per stage of the moments
constexpr int kBasisLd = kSrcTile + 1;                       // their row in LDS (odd: the columns spread over the banks)
constexpr int kMomProducts = 512;                            // threads of the products
constexpr int kMomThreads = kMomProducts + 192;              // and of the basis: four sources, up to 48 orders
constexpr int kTiles = 3;                                    // column tiles of the evaluation: S (+ S_L), D (+ L), K*

__host__ __device__ constexpr int ncf(int N) { return (N + 1) * (N + 2) / 2; }
// first entry of column m (n = m..N) of a triangle
__host__ __device__ constexpr int col(int N, int m) { return m * (N + 1) - m * (m - 1) / 2; }
// the same with columns padded to fours (moments; order kOrder)
__host__ __device__ constexpr int pcol(int m)
{
    int s = 0;
    for (int k = 0; k < m; ++k) s += (kOrder + 1 - k + 3) / 4 * 4;
    return s;
}
constexpr int kMomLen = pcol(kOrder + 1);
// k-steps of the evaluation (two degrees of one order, re and im, per step)
__host__ __device__ constexpr int nksteps(int N)
{
    int s = 0;
    for (int m = 0; m <= N; ++m) s += (N + 1 - m + 1) / 2;
    return s;
}
constexpr int kColSteps = nksteps(kOrder);
// Translations: lanes (order m, kClassRows degrees) of a class, and its table of I_n^m,
// m <= 2N, n = m .. 2N + 8
__host__ __device__ constexpr int ngroups(int k)
{
    int s = 0;
    for (int m = 0; m <= kClassOrder[k]; ++m) s += (kClassOrder[k] + 1 - m + kClassRows[k] - 1) / kClassRows[k];
    return s;
}
__host__ __device__ constexpr int trow(int N, int m) { return m * (2 * N + 9) - m * (m - 1) / 2; }
constexpr int tlen(int N) { return trow(N, 2 * N + 1); }
static_assert(ngroups(0) <= 64 * kClassSets[0] && ngroups(1) <= 64 * kClassSets[1] && ngroups(2) <= 64 * kClassSets[2] &&
              ngroups(3) <= 64 * kClassSets[3], "one lane per group");

// ---------------------------------------------------------------------------
// Moments of the 17 source strengths f(3), sigma, sigma n(3), m_jk(6),
// y_j m_jk(3), y.f about the drop's centre, one block per (source chunk,
// drop).  Per stage of four sources, eight waves take the products basis x
// strengths on FP64 MFMA (16 basis functions x 16 strengths per tile, the
// tiles dealt to the waves; the seventeenth strength on the vector ALU) while
// three waves put the next stage's basis V_n^m into LDS (a thread per source
// and order, its chain over the degrees).  FP64 issue, on both units, bounds
// it.  part[drop][chunk][strength][basis].
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kMomThreads) void k_p2m(const ehd::ExpandDrop* __restrict__ drops,
                                                     const int2* __restrict__ orders, const double* __restrict__ src,
                                                     long long Spad, double iunit, int nchunk,
                                                     double* __restrict__ part)
{
    extern __shared__ double lds[];
    constexpr int ST = kSrcTile, LD = kBasisLd, NP = kMomProducts;
    const int d = blockIdx.y, N = orders[d].x;
    if (N < 0) return;
    const double c0 = drops[d].c[0], c1 = drops[d].c[1], c2 = drops[d].c[2];
    const long long ns = drops[d].ns;
    src += drops[d].soff;
    const int NB = (N + 1) * (N + 2), ntile = (NB + 15) / 16;
    double* const R = lds;                                   // [2][basis][source], rows of LD
    double* const rec = R + 2 * kBasisPad * LD;              // [2][14][ST]
    double* const q = rec + 2 * 14 * ST;                     // [2][kField][ST]
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int z = NB * LD + tid; z < 16 * ntile * LD; z += kMomThreads) R[z] = R[kBasisPad * LD + z] = 0.0;
    const long long per = ((ns + nchunk - 1) / nchunk + ST - 1) / ST * ST;
    const long long s0 = blockIdx.x * per, s1 = s0 + per < ns ? s0 + per : ns;
    const int nst = s1 > s0 ? (int)((s1 - s0 + ST - 1) / ST) : 0;
    constexpr int TW = (kBasisPad / 16 + 7) / 8, XW = (kBasisPad + NP - 1) / NP;
    dbl4 acc[TW];
    double ax[XW];
#pragma unroll
    for (int k = 0; k < TW; ++k) acc[k] = dbl4{0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < XW; ++k) ax[k] = 0.0;
    // roles: threads 0 .. 67 the strengths of a stage, 128 .. 183 the load of
    // the records (entry e: record e / ST of source e % ST), 512 .. its basis
    const int e_rec = tid - 128;
    const bool rec_role = e_rec >= 0 && e_rec < 14 * ST;
    const double* const rsrc = src + (long long)(rec_role ? e_rec / ST : 0) * Spad;
    // past the last source: its place without a strength (the basis of a place
    // far from the drop overflows, and infinity times no strength is NaN)
    const bool place = e_rec < 7 * ST;
    const long long slast = s1 - 1;
    double next = 0.0;
    for (int k = -2; k < nst; ++k) {
        // stage k + 2 loaded, stage k + 1 built, stage k multiplied
        const int kb = (k + 1) & 1, kc = k & 1;
        if (rec_role) {
            const long long s = s0 + (long long)(k + 2) * ST + e_rec % ST;
            const double v = rsrc[s < slast ? s : slast];
            next = s < s1 || place ? v : 0.0;
        }
        if (k >= -1) {
            const int s = tid % ST;
            const double* const rc = rec + kb * 14 * ST + s;
            auto at = [&](int r) { return rc[r * ST]; };
            const double x = (at(0) - c0) * iunit, y = (at(1) - c1) * iunit, z = (at(2) - c2) * iunit;
            if (tid < kField * ST) {
                const int f = tid / ST;
                double v;
                if (f < 3) v = at(7 + f);
                else if (f == 3) v = at(13);
                else if (f < 7) v = at(13) * at(f - 1);
                else if (f < 13) {
                    const int e = f - 7, i = e < 3 ? 0 : e < 5 ? 1 : 2, j = e < 3 ? e : e < 5 ? e - 2 : 2;
                    v = at(10 + i) * at(3 + j) + at(10 + j) * at(3 + i);
                } else if (f < 16) {
                    const int e = f - 13;
                    const double yu = x * at(10) + y * at(11) + z * at(12), yn = x * at(3) + y * at(4) + z * at(5);
                    v = yu * at(3 + e) + yn * at(10 + e);
                } else {
                    v = x * at(7) + y * at(8) + z * at(9);
                }
                q[(kb * kField + f) * ST + s] = v;
            }
            const int m = (tid - NP) / ST;
            if (tid >= NP && m <= N) {
                double dr = 1.0, di = 0.0, br = x, bi = y;   // (x + iy)^m by squaring
                for (int e = m; e; e >>= 1) {
                    if (e & 1) {
                        const double t = dr * br - di * bi;
                        di = dr * bi + di * br;
                        dr = t;
                    }
                    const double t = br * br - bi * bi;
                    bi = 2.0 * br * bi;
                    br = t;
                }
                // (n^2 - m^2) rho^2 V_{n-1} is carried, so that a step waits for
                // one FMA only: three waves hide no latency
                const double r2 = x * x + y * y + z * z, z2 = 2.0 * z;
                double hr = 0.0, hi = 0.0, a = (2 * m + 1) * z, w = 2 * m + 1, g = w, h = g * r2;
                double* o = R + kb * kBasisPad * LD + 2 * col(N, m) * LD + s;
#pragma unroll 2
                for (int n = m; n <= N; ++n, o += 2 * LD) {
                    o[0] = dr;
                    o[LD] = di;
                    const double tr = fma(a, dr, -hr), ti = fma(a, di, -hi);
                    hr = h * dr;
                    hi = h * di;
                    dr = tr;
                    di = ti;
                    a += z2;
                    w += 2.0;
                    g += w;
                    h = g * r2;
                }
            }
        }
        if (k >= 0 && wv < NP / 64) {
            const double* const Rk = R + kc * kBasisPad * LD;
            const double* const qk = q + kc * kField * ST;
            const double b = qk[(lane & 15) * ST + (lane >> 4)];
            const double* const a = Rk + (lane & 15) * LD + (lane >> 4);
            // no guards around the loads (clamped; the surplus is not stored),
            // so that they are issued together
            double av[TW];
#pragma unroll
            for (int t = 0; t < TW; ++t) av[t] = a[16 * min(wv + 8 * t, ntile - 1) * LD];
#pragma unroll
            for (int t = 0; t < TW; ++t)
                if (wv + 8 * t < ntile) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[t], b, acc[t], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < XW; ++t) {
                const double* const e = Rk + min(tid + t * NP, NB - 1) * LD;
#pragma unroll
                for (int s = 0; s < ST; ++s) ax[t] = fma(e[s], qk[16 * ST + s], ax[t]);
            }
        }
        // the records of stage k were last read a barrier ago
        if (rec_role) rec[kc * 14 * ST + e_rec] = next;
        __syncthreads();
    }
    if (wv >= NP / 64) return;
    double* const o = part + ((long long)d * nchunk + blockIdx.x) * kField * kBasisPad;
#pragma unroll
    for (int k = 0; k < TW; ++k) {
        const int t = wv + 8 * k;
        if (t < ntile)
            for (int r = 0; r < 4; ++r) o[(lane & 15) * kBasisPad + 16 * t + (lane >> 4) + 4 * r] = acc[k][r];
    }
#pragma unroll
    for (int k = 0; k < XW; ++k) {
        const int b = tid + k * NP;
        if (b < NB) o[16 * kBasisPad + b] = ax[k];
    }
}

// Moments of the NP potentials from pot0 on (phi 0..3, Phi 4..7, chi 8,
// lambda 9) from those of the strengths (the chunks added in order), one
// thread each: mom[drop][column-padded (m, n)][NP] (re, im), zero past the
// drop's order.  A dipole of strength v has
//   M_n^m = Mz_{n-1}^m + ((Mx + i My)_{n-1}^{m+1} - (Mx - i My)_{n-1}^{m-1}) / 2.
__global__ __launch_bounds__(256) void k_moments(const int2* __restrict__ orders, int nchunk, int NP, int pot0,
                                                 const double* __restrict__ scale, const double* __restrict__ part,
                                                 double* __restrict__ mom)
{
    const int d = blockIdx.y, N = orders[d].x, e = blockIdx.x * 256 + threadIdx.x;
    if (N < 0 || e >= kMomLen * NP) return;
    const double* const p0 = part + (long long)d * nchunk * kField * kBasisPad;
    auto get = [&](int f, int n, int m) {
        const bool neg = m < 0;
        const int k = neg ? -m : m;
        if (n < 0 || k > n) return make_double2(0.0, 0.0);
        const double* p = p0 + (long long)f * kBasisPad + 2 * (col(N, k) + n - k);
        double re = 0.0, im = 0.0;
#pragma unroll 4
        for (int c = 0; c < nchunk; ++c) {
            re += p[(long long)c * kField * kBasisPad];
            im -= p[(long long)c * kField * kBasisPad + 1];   // conj(R)
        }
        const double w = scale[n * (n + 1) / 2 + k];
        re *= w;
        im *= w;
        if (!neg) return make_double2(re, im);
        return (k & 1) ? make_double2(-re, im) : make_double2(re, -im);
    };
    auto dipole = [&](int fx, int fy, int fz, int n, int m) {
        const double2 z = get(fz, n - 1, m);
        const double2 xp = get(fx, n - 1, m + 1), yp = get(fy, n - 1, m + 1);
        const double2 xm = get(fx, n - 1, m - 1), ym = get(fy, n - 1, m - 1);
        return make_double2(z.x + 0.5 * ((xp.x - yp.y) - (xm.x + ym.y)), z.y + 0.5 * ((xp.y + yp.x) - (xm.y - ym.x)));
    };
    const int pot = pot0 + e % NP, c = e / NP;
    int m = 0, at = 0;
    for (;; ++m) {
        const int len = (kOrder + 1 - m + 3) / 4 * 4;
        if (c < at + len) break;
        at += len;
    }
    const int n = m + c - at;
    double2 v = make_double2(0.0, 0.0);
    if (n <= N && m <= N) {
        switch (pot) {
        case 0: case 1: case 2: v = get(pot, n, m); break;
        case 3: v = get(16, n, m); break;
        case 4: v = dipole(7, 8, 9, n, m); break;
        case 5: v = dipole(8, 10, 11, n, m); break;
        case 6: v = dipole(9, 11, 12, n, m); break;
        case 7: v = dipole(13, 14, 15, n, m); break;
        case 8: v = get(3, n, m); break;
        default: v = dipole(4, 5, 6, n, m); break;
        }
    }
    reinterpret_cast<double2*>(mom)[(long long)d * kMomLen * NP + e] = v;
}

// ---------------------------------------------------------------------------
// Translations: a block takes consecutive pairs of one target drop.  Lanes
// hold the local coefficients of one order m and R consecutive degrees n
// (two up to order 19, four above) for all potentials in registers over all of
// the block's pairs; the waves of
// a lane set split the source orders m'.  With a = I_{n+n'}^{m+m'} and
// b = (-1)^m' I_{n+n'}^{m-m'} (from LDS), M = p + i q:
//   M a + conj(M) b = (p s_r - q t_i, p s_i + q t_r),  s = a + b, t = a - b,
// and the R degrees' s and t shift by one as n' steps (R steps unrolled,
// so that the window stays in place): two table reads feed 4 R NP FMAs.  The
// moments are wave-uniform (scalar loads).  The potentials phi_3 and Phi_3
// move their origin with the pair: M_3 -= D.M, D = c_i - c_j.  While the block
// works on one pair, some of its waves' lanes build the next pair's table.
// FP64 FMA issue bounds it.  With ten potentials four degrees per lane spill,
// which costs more than it saves where the chains are short: 256 drops, orders
// up to 19 3.3 ms with two and 6.2 with four; above, 2.5 with four and 3.3 with
// two.
// lpart[slot][split][m, n][NP] (re, im), without the (-1)^n.
// ---------------------------------------------------------------------------
template <int CLS>
__device__ __forceinline__ void m2l_table(double2* T, const ehd::ExpandPair& P, int m)
{
    constexpr int NC = kClassOrder[CLS];
    const int N = P.order;
    if (m > 2 * N) return;
    const double x = P.D[0], y = P.D[1], z = P.D[2];
    const double i2 = 1.0 / (x * x + y * y + z * z);
    double2* const o = T + trow(NC, m) - m;
    double dr = sqrt(i2), di = 0.0;
    const double ux = -x * i2, uy = -y * i2, uz = z * i2;
    for (int k = 0; k < m; ++k) {                            // I_{k+1}^{k+1} = -(2k+1)(x + iy) I_k^k / r^2
        const double f = 2 * k + 1, t = f * (dr * ux - di * uy);
        di = f * (dr * uy + di * ux);
        dr = t;
    }
    // I_{n+1} = ((2n+1) z I_n - (n^2 - m^2) I_{n-1}) / r^2, the last product carried
    double hr = 0.0, hi = 0.0, a = (2 * m + 1) * uz, w = 2 * m + 1, g = w, h = g * i2;
#pragma unroll 2
    for (int n = m; n <= 2 * N + 8; ++n) {
        o[n] = make_double2(dr, di);
        const double tr = fma(a, dr, -hr), ti = fma(a, di, -hi);
        hr = h * dr;
        hi = h * di;
        dr = tr;
        di = ti;
        a += 2.0 * uz;
        w += 2.0;
        g += w;
        h = g * i2;
    }
}

template <int NP, int CLS>
__global__ __launch_bounds__(64 * kClassWaves[CLS], CLS < 2 ? 3 : 2) void k_m2l(const ehd::ExpandItem* __restrict__ items,
                                                               const ehd::ExpandPair* __restrict__ pairs,
                                                               const double* __restrict__ mom,
                                                               double* __restrict__ lpart)
{
    constexpr int NC = kClassOrder[CLS], SETS = kClassSets[CLS], SPL = class_split(CLS), R = kClassRows[CLS];
    constexpr int NT = 64 * kClassWaves[CLS];
    extern __shared__ double2 tab[];                         // [2][tlen(NC)]
    const ehd::ExpandItem it = items[blockIdx.x];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int set = wv % SETS, sp = wv / SETS;
    int m = 0, n0 = 0;                                       // this lane's order and first degree
    bool live = false;
    {
        int g = set * 64 + lane;
        for (; m <= NC; ++m) {
            const int k = (NC + 1 - m + R - 1) / R;
            if (g < k) { n0 = m + R * g; live = true; break; }
            g -= k;
        }
        if (!live) { m = 0; n0 = NC + 1; }
    }
    double acc[R][NP][2];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int k = 0; k < NP; ++k) acc[r][k][0] = acc[r][k][1] = 0.0;
    m2l_table<CLS>(tab, pairs[it.first], threadIdx.x);
    __syncthreads();
    for (int k = it.first; k < it.last; ++k) {
        const int ph = (k - it.first) & 1;
        if (k + 1 < it.last)                                 // the builders take turns
            m2l_table<CLS>(tab + (ph ^ 1) * tlen(NC), pairs[k + 1], (int)(threadIdx.x + 128 * (k - it.first)) & (NT - 1));
        const ehd::ExpandPair P = pairs[k];
        const int N = P.order;
        const double2* const T = tab + ph * tlen(NC);
        const double* const Mj = mom + (long long)P.j * kMomLen * NP * 2;
        if (n0 <= N) {
            for (int mp = sp + SPL * it.part; mp <= N; mp += SPL * it.parts) {
                const double* Mc = Mj + (long long)pcol(mp) * NP * 2;
                const int mb = m >= mp ? m - mp : mp - m;
                const double2* const ta = T + trow(NC, m + mp) - (m + mp);
                const double2* const tb = T + trow(NC, mb) - mb;
                // b = (-1)^m' I^{m-m'}, or (-1)^m conj(I^{m'-m}) for m' > m; none for m' = 0
                const double sb = mp == 0 ? 0.0 : ((m >= mp ? mp : m) & 1) ? -1.0 : 1.0;
                const double sc = m >= mp ? sb : -sb;
                double sr[R], si[R], tr[R], ti[R];
                auto entry = [&](int n, int w) {
                    const double2 a = ta[n], b = tb[n];
                    sr[w] = fma(sb, b.x, a.x);
                    tr[w] = fma(-sb, b.x, a.x);
                    si[w] = fma(sc, b.y, a.y);
                    ti[w] = fma(-sc, b.y, a.y);
                };
#pragma unroll
                for (int w = 0; w < R; ++w) entry(n0 + mp + w, w);
                for (int np = mp; np <= N; np += R) {
#pragma unroll
                    for (int u = 0; u < R; ++u) {
                        double p[NP], q[NP];
#pragma unroll
                        for (int e = 0; e < NP; ++e) {
                            p[e] = Mc[2 * e];
                            q[e] = Mc[2 * e + 1];
                        }
                        Mc += 2 * NP;
                        if constexpr (NP >= 4) {
                            p[3] -= P.D[0] * p[0] + P.D[1] * p[1] + P.D[2] * p[2];
                            q[3] -= P.D[0] * q[0] + P.D[1] * q[1] + P.D[2] * q[2];
                        }
                        if constexpr (NP >= 8) {
                            p[7] -= P.D[0] * p[4] + P.D[1] * p[5] + P.D[2] * p[6];
                            q[7] -= P.D[0] * q[4] + P.D[1] * q[5] + P.D[2] * q[6];
                        }
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const int w = (r + u) % R;
#pragma unroll
                            for (int e = 0; e < NP; ++e) {
                                acc[r][e][0] = fma(p[e], sr[w], fma(-q[e], ti[w], acc[r][e][0]));
                                acc[r][e][1] = fma(p[e], si[w], fma(q[e], tr[w], acc[r][e][1]));
                            }
                        }
                        entry(n0 + np + u + R, u);           // row 0's entry leaves the window
                    }
                }
            }
        }
        __syncthreads();
    }
    if (live) {
        double2* const o = reinterpret_cast<double2*>(lpart) +
                           ((long long)it.slot * SPL + sp) * ncf(NC) * NP + (long long)(col(NC, m) + n0 - m) * NP;
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (n0 + r <= NC)
#pragma unroll
                for (int e = 0; e < NP; ++e) o[r * NP + e] = make_double2(acc[r][e][0], acc[r][e][1]);
    }
}

// Local coefficients of a drop: the slots of every class and split added in a
// fixed order, one thread per coefficient; local[drop][m, n][NP].
struct LocalParts {
    const double2* p[ehd::kExpClasses];
};
__global__ __launch_bounds__(256) void k_local(const int2* __restrict__ orders, const int2* __restrict__ slots, int nd,
                                               int NP, LocalParts lp, double2* __restrict__ local)
{
    const int d = blockIdx.y, N = orders[d].y, e = blockIdx.x * 256 + threadIdx.x;
    if (N < 0 || e >= ncf(N) * NP) return;
    const int c = e / NP, pot = e % NP;
    int m = 0;
    while (c >= col(N, m + 1)) ++m;
    const int n = m + c - col(N, m);
    double2 s = make_double2(0.0, 0.0);
    for (int k = 0; k < ehd::kExpClasses; ++k) {
        const int NC = kClassOrder[k], spl = class_split(k);
        const int2 sl = slots[k * nd + d];
        if (n > NC) continue;
        const double2* p = lp.p[k] + (long long)sl.x * spl * ncf(NC) * NP + (long long)(col(NC, m) + n - m) * NP + pot;
        for (int u = 0; u < sl.y * spl; ++u) {
            const double2 v = p[(long long)u * ncf(NC) * NP];
            s.x += v.x;
            s.y += v.y;
        }
    }
    local[(long long)d * ncf(kOrder) * NP + e] = (n & 1) ? make_double2(-s.x, -s.y) : s;
}

// B operands of the evaluation from the local coefficients: per k-step (order
// m, degrees n and n + 1, each re and im) sixteen columns of each tile: values
// and gradients of the potentials as the header lists them.  Gradients by
// coefficients: d_z from L_{n+1}^m, d_x from (L_{n+1}^{m-1} - L_{n+1}^{m+1}) / 2,
// d_y from i (L_{n+1}^{m-1} + L_{n+1}^{m+1}) / 2.
__global__ __launch_bounds__(256) void k_l2c(const int2* __restrict__ orders, int NP, int pot0, unsigned tiles,
                                             const double* __restrict__ scale, const double2* __restrict__ local,
                                             double* __restrict__ cols)
{
    const int d = blockIdx.y, N = orders[d].y, e = blockIdx.x * 256 + threadIdx.x;
    if (N < 0 || e >= nksteps(N) * 64) return;
    const double2* const L = local + (long long)d * ncf(kOrder) * NP;
    auto get = [&](int pot, int n, int m) {
        const bool neg = m < 0;
        const int k = neg ? -m : m;
        if (pot < pot0 || pot >= pot0 + NP || n > N || k > n) return make_double2(0.0, 0.0);
        const double2 v = L[(col(N, k) + n - k) * NP + pot - pot0];
        if (!neg) return v;
        return (k & 1) ? make_double2(-v.x, v.y) : make_double2(v.x, -v.y);
    };
    const int ks = e >> 6, lane = e & 63, g = lane >> 4, c = lane & 15;
    int m = 0, at = 0;
    for (;; ++m) {
        const int len = (N + 1 - m + 1) / 2;
        if (ks < at + len) break;
        at += len;
    }
    const int n = m + 2 * (ks - at) + (g >> 1);
    const double w = n <= N ? (m ? 2.0 : 1.0) * scale[n * (n + 1) / 2 + m] : 0.0;
    for (int t = 0; t < kTiles; ++t) {
        if (!(tiles & (1u << t))) continue;
        double2 v = make_double2(0.0, 0.0);
        if (n <= N) {
            int pot, axis;                                   // axis -1: the value
            if (t == 2) { pot = 8; axis = c < 3 ? c : -2; }
            else if (c < 3) { pot = 4 * t + c; axis = -1; }
            else if (c < 15) { pot = 4 * t + (c - 3) / 3; axis = (c - 3) % 3; }
            else { pot = 8 + t; axis = -1; }
            if (axis == -1) v = get(pot, n, m);
            else if (axis == 2) v = get(pot, n + 1, m);
            else if (axis >= 0) {
                const double2 lo = get(pot, n + 1, m - 1), hi = get(pot, n + 1, m + 1);
                v = axis == 0 ? make_double2(0.5 * (lo.x - hi.x), 0.5 * (lo.y - hi.y))
                              : make_double2(-0.5 * (lo.y + hi.y), 0.5 * (lo.x + hi.x));
            }
        }
        cols[(((long long)d * kTiles + t) * kColSteps + ks) * 64 + lane] = (g & 1) ? (m ? w * v.y : 0.0) : w * v.x;
    }
}

// Evaluation at the targets: a wave takes 16 RT targets of one drop as RT MFMA
// row tiles (two; one where that would leave compute units idle); each lane runs the recurrence of V_n^m (re or im) of its target
// and hands the products to the matrix unit, whose B operands (k_l2c) stream
// from L2.  Bound by the matrix unit.  TM: column tiles present (bits).
template <unsigned TM, int RT>
__global__ __launch_bounds__(256) void k_l2p(const ehd::ExpandDrop* __restrict__ drops, const int2* __restrict__ orders,
                                             const int2* __restrict__ tblocks, const double* __restrict__ cols, double iunit, unsigned kinds,
                                             const double* __restrict__ tx, const double* __restrict__ tn, long long T,
                                             double* __restrict__ out)
{
    constexpr int LD = 16 * kTiles + 1;
    __shared__ double buf[4][16 * RT][LD];
    const int2 tb = tblocks[blockIdx.x];
    const int d = tb.x, N = orders[d].y;
    const ehd::ExpandDrop D = drops[d];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, g = lane >> 4;
    const bool im = g & 1, hi = g >> 1;
    double x[RT], y[RT], z[RT], r2[RT], dr[RT], di[RT];
    for (int k = 0; k < RT; ++k) {
        long long t = tb.y + wv * 16 * RT + 16 * k + (lane & 15);
        t = D.toff + (t < D.nt ? t : D.nt - 1);
        x[k] = (tx[t] - D.c[0]) * iunit;
        y[k] = (tx[T + t] - D.c[1]) * iunit;
        z[k] = (tx[2 * T + t] - D.c[2]) * iunit;
        r2[k] = x[k] * x[k] + y[k] * y[k] + z[k] * z[k];
        dr[k] = 1.0;
        di[k] = 0.0;
    }
    dbl4 acc[RT][kTiles];
    for (int k = 0; k < RT; ++k)
        for (int t = 0; t < kTiles; ++t) acc[k][t] = dbl4{0, 0, 0, 0};
    const double* B = cols + (long long)d * kTiles * kColSteps * 64 + lane;
    for (int m = 0; m <= N; ++m) {
        double p[RT], c[RT];                                 // R_{n-1}, R_n
        for (int k = 0; k < RT; ++k) {
            p[k] = 0.0;
            c[k] = im ? di[k] : dr[k];
        }
        for (int n = m; n <= N; n += 2) {
            double b[kTiles];
            for (int t = 0; t < kTiles; ++t)
                if (TM & (1u << t)) b[t] = B[(long long)t * kColSteps * 64];
            B += 64;
            const double a1 = 2 * n + 1, a2 = 2 * n + 3;
            const double g1 = (n - m) * (n + m), g2 = (n + 1 - m) * (n + 1 + m);
#pragma unroll
            for (int k = 0; k < RT; ++k) {
                const double n1 = a1 * z[k] * c[k] - g1 * r2[k] * p[k];
                const double n2 = a2 * z[k] * n1 - g2 * r2[k] * c[k];
                const double a = hi ? n1 : c[k];
#pragma unroll
                for (int t = 0; t < kTiles; ++t)
                    if (TM & (1u << t)) acc[k][t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b[t], acc[k][t], 0, 0, 0);
                p[k] = n1;
                c[k] = n2;
            }
        }
        for (int k = 0; k < RT; ++k) {
            const double t = dr[k] * x[k] - di[k] * y[k];
            di[k] = dr[k] * y[k] + di[k] * x[k];
            dr[k] = t;
        }
    }
    for (int k = 0; k < RT; ++k)
        for (int t = 0; t < kTiles; ++t)
            if (TM & (1u << t))
                for (int r = 0; r < 4; ++r) buf[wv][16 * k + g + 4 * r][16 * t + (lane & 15)] = acc[k][t][r];
    __syncthreads();
    const long long tl = tb.y + wv * 16 * RT + lane;
    if (lane >= 16 * RT || tl >= D.nt) return;
    const long long t = D.toff + tl;
    const double* v = buf[wv][lane];
    const double y0[3] = {(tx[t] - D.c[0]) * iunit, (tx[T + t] - D.c[1]) * iunit, (tx[2 * T + t] - D.c[2]) * iunit};
    // value - y0_k d_i(k) + d_i(3) of the vector potential in a tile
    auto vec = [&](const double* w, int i) {
        return w[i] - (y0[0] * w[3 + i] + y0[1] * w[6 + i] + y0[2] * w[9 + i]) + w[12 + i];
    };
    const double iu2 = iunit * iunit;
    if ((TM & 1u) && (kinds & EHD_STOKES_SL))
        for (int i = 0; i < 3; ++i) out[i * T + t] = vec(v, i) * iunit;
    if ((TM & 2u) && (kinds & EHD_STOKES_DL))
        for (int i = 0; i < 3; ++i) out[(3 + i) * T + t] = -vec(v + 16, i) * iu2;
    if ((TM & 1u) && (kinds & EHD_LAP_SL)) out[6 * T + t] = v[15] * iunit;
    if ((TM & 2u) && (kinds & EHD_LAP_DL)) out[7 * T + t] = v[31] * iu2;
    if ((TM & 4u) && (kinds & EHD_LAP_DLADJ))
        out[8 * T + t] = -(v[32] * tn[t] + v[33] * tn[T + t] + v[34] * tn[2 * T + t]) * iu2;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
// Costs of the plan, in cycles of one compute unit: per interaction of the
// direct sums (23.8 ms for 942 pairs of 2178 x 8450), per square of a
// translation's coefficients (8 ms for 64,000 pairs of mean order 15), per
// source and 16 basis functions of the moments (6.2 ms for 2.2 million sources
// at order 40), per target and k-step of the evaluation (1.4 ms for 558,000
// targets), and what the seven launches take on few drops, where no kernel
// fills the device (12 drops of p = 5 to 29: 0.7 ms against 0.3 saved).
// All kinds on 2 to 48 drops of p = 8, 16, 24, 32, 48 and mixed, volume
// fractions 0.1 and 0.01, both ways: the plan takes the faster one, or one
// within 5%, in each of 96 cases; it turns between 16 drops of p = 16 (direct
// 0.57 ms, expansions 0.68 to 0.78) and 24 (1.16 and 1.01, 0.75 sparse), and
// between 2 of p = 48 (0.35 and 0.41 to 0.52) and 4 (1.90 and 1.58, 0.62).  A
// single kind's direct sums cost a third to a half: next to the turn it loses
// up to 0.2 ms.
constexpr double kCostDirect = 0.8, kCostPair = 1.8, kCostMoment = 16.0, kCostEval = 3.5, kCostFixed = 256.0 * 1.2e6;
// Translation blocks per class to aim at (two to four rounds of the blocks
// that fit the device) and the most shares of the source orders.
constexpr int kClassBlocks[ehd::kExpClasses] = {2048, 2048, 1024, 512};
constexpr int kClassParts[ehd::kExpClasses] = {1, 2, 4, 8};
constexpr int kMaxDrops = 4096;        // more drops than this keep the direct sums (pair lists grow with the square)

// Smallest order whose truncation is below the direct sums' rounding: with
// rho the larger of (source radius) / (distance of the nearest target from
// the source's centre) and the same with the parts exchanged, the neglected
// terms of a potential are below rho^(N+1).  The Stokes double layer adds a
// dipole's and a gradient's derivative, (N+2)^2 together, and in Phi_3 the
// factor y, as large as the distance of the drops, which takes one power of
// rho back: (N+2)^2 rho^N <= 1e-14.  Evaluated in 80 bits where that is an
// equality, radii alike or 1 to 5, worst places: D 6e-15 (N = 6) to 9e-15 (24)
// of 6 / distance^2, the other kernels below 1.5e-15 of theirs; the direct sums
// of a distant pair, whose 2/r has one Newton step, are 3e-14 off in D.
// (4e-15 instead: orders half a one higher, 256 drops of p = 32 1% longer.)
// The rule is kept solved for rho.
struct OrderLimits {
    double rho[kOrder + 1];                                  // largest rho of each order
    OrderLimits()
    {
        for (int N = 0; N <= kOrder; ++N) rho[N] = N < 3 ? 0.0 : std::pow(1e-14 / ((N + 2.0) * (N + 2.0)), 1.0 / N);
    }
    int order(double r) const                                // smallest order for r, -1: none
    {
        if (!(r >= 0.0)) return -1;
        const double* const p = std::lower_bound(rho + 3, rho + kOrder + 1, r);
        return p == rho + kOrder + 1 ? -1 : (int)(p - rho);
    }
};

template <typename T>
hipError_t put(ehd::Expand::Buf& b, const std::vector<T>& v, hipStream_t st)
{
    hipError_t e = ehd::ensure(b, sizeof(T) * std::max<size_t>(v.size(), 1));
    if (e == hipSuccess && !v.empty()) e = hipMemcpyAsync(b.p, v.data(), sizeof(T) * v.size(), hipMemcpyHostToDevice, st);
    return e;
}

}  // namespace

namespace ehd {

hipError_t expand_plan(Expand& E, const std::vector<ExpandDrop>& drops, hipStream_t stream)
{
    E.on = false;
    const int nd = E.nd = (int)drops.size();
    if (nd < 2 || nd > kMaxDrops) return hipSuccess;
    double rmax = 0.0;
    for (const ExpandDrop& d : drops) rmax = std::max(rmax, std::max(d.rs, d.rt));
    if (!(rmax > 0.0) || !std::isfinite(rmax)) return hipSuccess;
    E.unit = std::exp2(std::ceil(std::log2(rmax)));
    if (!(E.unit > 1e-100) || !(E.unit < 1e100)) return hipSuccess;

    // nothing to gain where all pairs together are cheap
    double nts = 0.0, nss = 0.0, own = 0.0;
    for (const ExpandDrop& d : drops) {
        nts += (double)d.nt;
        nss += (double)d.ns;
        own += (double)d.nt * (double)d.ns;
    }
    if (!(kCostDirect * (nts * nss - own) > kCostFixed)) return hipSuccess;

    // pairs: expanded where separated and cheaper than the direct sum.  A plan
    // is made for every shape, so most pairs that stay direct are told by one
    // comparison: the order up to which a translation is cheaper than the
    // pair's sum follows from the node counts (few different ones), and with it
    // the least distance.  Whole rows fall by the farthest corner of the centres'
    // box (4000 drops of p = 4, nothing to expand: 400 ms with a search of the
    // order per pair).
    static const OrderLimits limits;
    std::vector<int> kind(nd);
    std::vector<std::pair<long long, long long>> kinds;      // (nt, ns)
    std::vector<double> smallest;                            // least source radius of a kind
    {
        std::map<std::pair<long long, long long>, int> seen;
        for (int d = 0; d < nd; ++d) {
            const auto at = seen.emplace(std::make_pair(drops[d].nt, drops[d].ns), (int)kinds.size());
            if (at.second) {
                kinds.push_back(at.first->first);
                smallest.push_back(drops[d].rs);
            }
            kind[d] = at.first->second;
            smallest[kind[d]] = std::min(smallest[kind[d]], drops[d].rs);
        }
    }
    auto m2l_cost = [](int N) { return kCostPair * (double)ncf(N) * ncf(N) + 2000.0; };
    double lo[3], hi[3];
    bool boxed = true;
    for (int c = 0; c < 3; ++c) {
        lo[c] = hi[c] = drops[0].c[c];
        for (const ExpandDrop& d : drops) {
            lo[c] = std::min(lo[c], d.c[c]);
            hi[c] = std::max(hi[c], d.c[c]);
            boxed = boxed && std::isfinite(d.c[c]);
        }
    }
    E.near.assign((size_t)nd * nd, 1);
    std::vector<int2> orders(nd, make_int2(-1, -1));
    std::vector<std::vector<ExpandPair>> lists(nd);
    std::vector<double> inv(kinds.size());                   // 1 / rho of a kind's largest order, 0: none
    double gain = 0.0;
    for (int i = 0; i < nd; ++i) {
        const ExpandDrop& A = drops[i];
        double least = HUGE_VAL, far2 = 0.0;
        for (size_t k = 0; k < kinds.size(); ++k) {
            const double direct = kCostDirect * (double)A.nt * (double)kinds[k].second;
            int N = kOrder;
            while (N >= 3 && !(m2l_cost(N) < direct)) --N;
            inv[k] = N < 3 ? 0.0 : 1.0 / limits.rho[N];
            if (inv[k] > 0.0) least = std::min(least, A.rt + smallest[k] * inv[k]);
        }
        for (int c = 0; c < 3; ++c) {
            const double d = std::max(A.c[c] - lo[c], hi[c] - A.c[c]);
            far2 += d * d;
        }
        if (least == HUGE_VAL || (boxed && far2 < least * least * (1.0 - 1e-9))) continue;
        for (int j = 0; j < nd; ++j) {
            const ExpandDrop& B = drops[j];
            const double q = inv[kind[j]];
            if (i == j || !(q > 0.0)) continue;
            const double dx = A.c[0] - B.c[0], dy = A.c[1] - B.c[1], dz = A.c[2] - B.c[2];
            const double d2 = dx * dx + dy * dy + dz * dz, need = std::max(A.rt + B.rs * q, B.rs + A.rt * q);
            if (!(d2 >= need * need * (1.0 - 1e-9))) continue;
            const double dist = std::sqrt(d2);
            if (!std::isfinite(dist) || !(dist - A.rt > 0.0) || !(dist - B.rs > 0.0) || dist < 0.25 * E.unit) continue;
            const int N = limits.order(std::max(B.rs / (dist - A.rt), A.rt / (dist - B.rs)));
            if (N < 0) continue;
            const double direct = kCostDirect * (double)A.nt * (double)B.ns, m2l = m2l_cost(N);
            if (m2l >= direct) continue;
            gain += direct - m2l;
            E.near[(size_t)i * nd + j] = 0;
            lists[i].push_back({j, N, {dx / E.unit, dy / E.unit, dz / E.unit}});
            orders[i].y = std::max(orders[i].y, N);
            orders[j].x = std::max(orders[j].x, N);
        }
    }
    int nsrc = 0;
    long long most = 0;
    for (int d = 0; d < nd; ++d) {
        if (orders[d].x >= 0) {
            ++nsrc;
            gain -= kCostMoment * (double)drops[d].ns * ((orders[d].x + 1) * (orders[d].x + 2) / 16);
            most = std::max(most, drops[d].ns);
        }
        if (orders[d].y >= 0) gain -= kCostEval * (double)drops[d].nt * nksteps(orders[d].y);
    }
    if (!(gain > kCostFixed)) {
        std::fill(E.near.begin(), E.near.end(), 1);
        return hipSuccess;
    }

    // work lists
    long long targets = 0;
    for (const ExpandDrop& d : drops) targets += d.nt;
    E.rowtiles = targets >= 65536 ? 2 : 1;                   // at least two blocks of 64 targets per compute unit
    std::vector<ExpandPair> pairs;
    std::vector<ExpandItem> items[kExpClasses];
    std::vector<int2> slots((size_t)kExpClasses * nd, make_int2(0, 0)), tblocks;
    long long total[kExpClasses] = {};
    auto cls = [](int N) {
        int k = 0;
        while (N > kClassOrder[k]) ++k;
        return k;
    };
    for (const auto& l : lists)
        for (const ExpandPair& p : l) ++total[cls(p.order)];
    for (int i = 0; i < nd; ++i) {
        for (int k = 0; k < kExpClasses; ++k) {
            const int first = (int)pairs.size();
            for (const ExpandPair& p : lists[i])
                if (cls(p.order) == k) pairs.push_back(p);
            const int n = (int)pairs.size() - first;
            if (!n) continue;
            // enough blocks for the device: a drop's pairs split evenly, and
            // where the class has few pairs also their source orders
            const int len = (int)std::max<long long>(1, total[k] / kClassBlocks[k]), cuts = (n + len - 1) / len;
            const int parts = (int)std::max<long long>(1, std::min<long long>(kClassParts[k], kClassBlocks[k] / (2 * total[k])));
            slots[(size_t)k * nd + i] = make_int2((int)items[k].size(), cuts * parts);
            for (int q = 0; q < cuts; ++q)
                for (int u = 0; u < parts; ++u)
                    items[k].push_back({i, first + (int)((long long)n * q / cuts), first + (int)((long long)n * (q + 1) / cuts),
                                        u, parts, (int)items[k].size()});
        }
        // every drop: one without expanded sources gets zeros
        for (long long t = 0; t < drops[i].nt; t += 64 * E.rowtiles) tblocks.push_back(make_int2(i, (int)t));
    }
    E.ntblocks = (int)tblocks.size();
    E.nchunk = (int)std::max<long long>(1, std::min<long long>({32, (1023 + nsrc) / nsrc, most / (16 * kSrcTile)}));
    // R / V = (-1)^m (2m-1)!! / ((n-m)! (n+m)!)
    std::vector<double> scale(ncf(kOrder));
    for (int m = 0; m <= kOrder; ++m) {
        double v = 1.0;
        for (int k = 1; k <= m; ++k) v *= -(2.0 * k - 1.0) / ((2.0 * k - 1.0) * (2.0 * k));
        for (int n = m; n <= kOrder; ++n) {
            if (n > m) v /= (double)(n - m) * (n + m);
            scale[n * (n + 1) / 2 + m] = v;
        }
    }

    hipError_t e = put(E.buf[Expand::DROPS], drops, stream);
    if (e == hipSuccess) e = put(E.buf[Expand::ORDERS], orders, stream);
    if (e == hipSuccess) e = put(E.buf[Expand::PAIRS], pairs, stream);
    for (int k = 0; k < kExpClasses; ++k) {
        if (e == hipSuccess) e = put(E.buf[Expand::ITEMS + k], items[k], stream);
        E.nitems[k] = (int)items[k].size();
        if (e == hipSuccess)
            e = ensure(E.buf[Expand::LPART + k],
                       sizeof(double2) * (size_t)class_split(k) * ncf(kClassOrder[k]) * 10 * items[k].size() + 16);
    }
    if (e == hipSuccess) e = put(E.buf[Expand::SLOTS], slots, stream);
    if (e == hipSuccess) e = put(E.buf[Expand::TBLOCKS], tblocks, stream);
    if (e == hipSuccess) e = put(E.buf[Expand::SCALE], scale, stream);
    if (e == hipSuccess) e = ensure(E.buf[Expand::MPART], sizeof(double) * (size_t)nd * E.nchunk * kField * kBasisPad);
    if (e == hipSuccess) e = ensure(E.buf[Expand::MOM], sizeof(double2) * (size_t)nd * kMomLen * 10);
    if (e == hipSuccess) e = ensure(E.buf[Expand::LOCAL], sizeof(double2) * (size_t)nd * ncf(kOrder) * 10);
    if (e == hipSuccess) e = ensure(E.buf[Expand::COLS], sizeof(double) * (size_t)nd * kTiles * kColSteps * 64);
    const hipError_t es = hipStreamSynchronize(stream);      // the host lists go out of scope
    if (e == hipErrorOutOfMemory) {                          // no room: the direct sums need none of it
        (void)hipGetLastError();
        E.release();
        std::fill(E.near.begin(), E.near.end(), 1);
        return es;
    }
    E.on = e == hipSuccess && es == hipSuccess;
    return e != hipSuccess ? e : es;
}

namespace {

template <int NP>
hipError_t launch_m2l(const Expand& E, hipStream_t st)
{
    hipError_t e = hipSuccess;
    auto go = [&](auto kernel, int k) {
        if (e != hipSuccess || !E.nitems[k]) return;
        const size_t lds = sizeof(double2) * 2 * tlen(kClassOrder[k]);
        if (lds > 65536) e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return;
        hipLaunchKernelGGL(kernel, dim3(E.nitems[k]), dim3(64 * kClassWaves[k]), lds, st,
                           E.at<ExpandItem>(Expand::ITEMS + k), E.at<ExpandPair>(Expand::PAIRS),
                           E.at<double>(Expand::MOM), E.at<double>(Expand::LPART + k));
    };
    go(k_m2l<NP, 3>, 3);
    go(k_m2l<NP, 2>, 2);
    go(k_m2l<NP, 1>, 1);
    go(k_m2l<NP, 0>, 0);
    return e;
}

}  // namespace

hipError_t expand_enqueue(const Expand& E, hipStream_t st, unsigned kinds, const double* src, long long Spad,
                          const double* tx, const double* tn, long long T, double* out)
{
    const double iu = 1.0 / E.unit;
    const bool S = kinds & EHD_STOKES_SL, D = kinds & EHD_STOKES_DL;
    const bool lap = kinds & (EHD_LAP_SL | EHD_LAP_DL | EHD_LAP_DLADJ);
    const int NP = (S && !D && !lap) || (D && !S && !lap) ? 4 : (!S && !D) ? 2 : 10;
    const int pot0 = NP == 10 ? 0 : NP == 2 ? 8 : S ? 0 : 4;
    const unsigned tiles = ((kinds & (EHD_STOKES_SL | EHD_LAP_SL)) ? 1u : 0u) |
                           ((kinds & (EHD_STOKES_DL | EHD_LAP_DL)) ? 2u : 0u) | ((kinds & EHD_LAP_DLADJ) ? 4u : 0u);
    const ExpandDrop* dr = E.at<ExpandDrop>(Expand::DROPS);
    const int2* orders = E.at<int2>(Expand::ORDERS);
    const double* scale = E.at<double>(Expand::SCALE);
    hipError_t e;
    const size_t lp2m = sizeof(double) * 2 * (kBasisPad * kBasisLd + (14 + kField) * kSrcTile);
    if ((e = hipFuncSetAttribute((const void*)k_p2m, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lp2m)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_p2m, dim3(E.nchunk, E.nd), dim3(kMomThreads), lp2m, st, dr, orders, src, Spad, iu, E.nchunk,
                       E.at<double>(Expand::MPART));
    hipLaunchKernelGGL(k_moments, dim3((kMomLen * NP + 255) / 256, E.nd), dim3(256), 0, st, orders, E.nchunk, NP, pot0,
                       scale, E.at<double>(Expand::MPART), E.at<double>(Expand::MOM));
    e = NP == 10 ? launch_m2l<10>(E, st) : NP == 4 ? launch_m2l<4>(E, st) : launch_m2l<2>(E, st);
    if (e != hipSuccess) return e;
    LocalParts lp;
    for (int k = 0; k < kExpClasses; ++k) lp.p[k] = E.at<double2>(Expand::LPART + k);
    hipLaunchKernelGGL(k_local, dim3((ncf(kOrder) * NP + 255) / 256, E.nd), dim3(256), 0, st, orders,
                       E.at<int2>(Expand::SLOTS), E.nd, NP, lp, E.at<double2>(Expand::LOCAL));
    hipLaunchKernelGGL(k_l2c, dim3((kColSteps * 64 + 255) / 256, E.nd), dim3(256), 0, st, orders, NP, pot0, tiles, scale,
                       E.at<double2>(Expand::LOCAL), E.at<double>(Expand::COLS));
    auto eval = [&](auto one, auto two) {
        auto go = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(E.ntblocks), dim3(256), 0, st, dr, orders, E.at<int2>(Expand::TBLOCKS),
                               E.at<double>(Expand::COLS), iu, kinds, tx, tn, T, out);
        };
        if (E.rowtiles == 2) go(two);
        else go(one);
    };
    switch (tiles) {
    case 1: eval(k_l2p<1, 1>, k_l2p<1, 2>); break;
    case 2: eval(k_l2p<2, 1>, k_l2p<2, 2>); break;
    case 3: eval(k_l2p<3, 1>, k_l2p<3, 2>); break;
    case 4: eval(k_l2p<4, 1>, k_l2p<4, 2>); break;
    case 5: eval(k_l2p<5, 1>, k_l2p<5, 2>); break;
    case 6: eval(k_l2p<6, 1>, k_l2p<6, 2>); break;
    default: eval(k_l2p<7, 1>, k_l2p<7, 2>); break;
    }
    return hipGetLastError();
}

}  // namespace ehd
