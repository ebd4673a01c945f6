// The radial pass: the radial factors (B_nl, Bh_nl) of every edge of a range
// of centers, evaluated once per call and read by the density and Jacobian
// kernels of the call (all bases but those whose kernels evaluate their own).  Evaluated inside those kernels, they
// were computed twice per edge, in tiles of a few edges that filled a wave
// badly and held the basis tables in the kernels' LDS; here the items
// (edge, degree) run flat over all lanes.
#include "soap_device.h"

#include <cmath>
#include <vector>

namespace soap {
using namespace dev;

namespace dev {

constexpr int NWR = 4, BSR = 64 * NWR;
constexpr int RAD_CB_MAX = 256; // centers per workgroup block
constexpr int RAD_EB = 128;     // most edges per pass over a block's edges
constexpr size_t RAD_TILE = 40 * 1024; // LDS bytes of a pass's results

// The center of edge e (rp[0] <= e < rp[ncb]): the last k with rp[k] <= e.
__device__ __forceinline__ int center_of(const int64_t *rp, int ncb, int64_t e) {
    int lo = 0, hi = ncb - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (rp[mid] <= e) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}
// |r_j - r_i|^2 of edge e of the block of centers c0...
template <typename PosT>
__device__ __forceinline__ double edge_r2(const Rows &R, const PosT *__restrict__ pos, const int64_t *rp, int64_t c0,
                                          int ncb, int64_t e) {
    const int64_t ci = c0 + center_of(rp, ncb, e);
    const int64_t i = R.centers ? (int64_t)R.centers[ci] : R.c_base + ci;
    const int64_t j = R.cols[e];
    const double x = (double)pos[3 * j] - (double)pos[3 * i], y = (double)pos[3 * j + 1] - (double)pos[3 * i + 1],
                 z = (double)pos[3 * j + 2] - (double)pos[3 * i + 2];
    return x * x + y * y + z * z;
}

// Doubles of the basis tables in LDS.  GTO: a' [l][NA], betaC [l][n][NA]
// (zero past n_max) and the exponential's table; compensated GTO: the same
// two as (value, remainder) pairs; Laplace form: the Chebyshev series
// [n][n+3][4] and B_n0(0) [n].
__host__ __device__ __forceinline__ size_t radial_table_doubles(const Params &P, int rbf, int na) {
    const size_t n = (size_t)P.n, lw = (size_t)P.lmax + 1;
    if (rbf == 0) return even(lw * na) + even(lw * n * na) + 128;
    if (rbf == 3) return 2 * lw * na + 2 * lw * n * na;
    return 4 * n * (n + 3) + even(n);
}
// edges per pass: their results stay within RAD_TILE (pair: bytes of one)
__host__ __device__ __forceinline__ int radial_tile_edges(const Params &P, int pair) {
    const int per = (P.n * (P.lmax + 1) | 1) * pair, e = (int)(RAD_TILE / (size_t)per);
    return e < 8 ? 8 : (e > RAD_EB ? RAD_EB : e);
}
__host__ __device__ __forceinline__ size_t radial_flat_lds_doubles(const Params &P, int rbf, int na, int pair) {
    const int EB = radial_tile_edges(P, pair);
    return even(RAD_CB_MAX + 1) + even(EB) + radial_table_doubles(P, rbf, na) +
           even(((size_t)EB * (P.n * (P.lmax + 1) | 1) * pair + 7) / 8);
}

// GTO (RBF 0), compensated GTO (3) and the polynomial Laplace form (2).  A
// workgroup takes blocks of cb consecutive centers, whose edges are
// contiguous: per pass of up to RAD_EB edges it leaves their squared lengths
// in LDS, then its threads take the items (degree, edge) - for the Laplace
// form (radial index, edge) - with the edge running fastest, so that the
// basis coefficients a wave reads are broadcast.  The results go through LDS:
// an edge's pairs leave as one contiguous run (204,662 edges, n_max 8, l_max 6:
// 96 us stored per item, 55 through an LDS tile).  An edge of length 0 has only
// its factors B_n0, its on-site term: the density step on the matrix cores takes
// the others as they are, and their gradients would enter its center's D.
template <typename PosT, typename ST, int NA, int RBF>
__global__ __launch_bounds__(BSR) void k_radial_flat(Params P, Rows R, const PosT *__restrict__ pos, int cb) {
    extern __shared__ __align__(16) double smem[];
    const int tid = threadIdx.x, n = P.n, lw = P.lmax + 1;
    Carver cv{smem};
    int64_t *rp = (int64_t *)cv.take(RAD_CB_MAX + 1);
    const int EB = radial_tile_edges(P, (int)sizeof(ST) * 2), per = n * lw, ldt = per | 1;
    double *r2 = cv.take(EB);
    auto *tile = (typename Pair<ST>::type *)cv.take(((size_t)EB * ldt * 2 * sizeof(ST) + 7) / 8); // [edge][n][l]
    double *A = nullptr, *B = nullptr, *e2 = nullptr;
    if constexpr (RBF == 0) {
        A = cv.take((size_t)lw * NA);
        B = cv.take((size_t)lw * n * NA);
        e2 = cv.take(128);
        for (int k = tid; k < lw * NA; k += BSR) {
            const int l = k / NA, q = k - l * NA;
            A[k] = q < n ? P.aprime[l * n + q] : 0.0;
        }
        for (int k = tid; k < lw * n * NA; k += BSR) {
            const int la = k / NA, q = k - la * NA;
            B[k] = q < n ? P.betaC[la * n + q] : 0.0;
        }
        for (int k = tid; k < 128; k += BSR) e2[k] = P.e2t[k];
    } else if constexpr (RBF == 3) {
        A = cv.take(2 * (size_t)lw * NA);
        B = cv.take(2 * (size_t)lw * n * NA);
        for (int k = tid; k < lw * NA; k += BSR) {
            const int l = k / NA, q = k - l * NA;
            A[2 * k] = q < n ? P.aprime[l * n + q] : 0.0;
            A[2 * k + 1] = q < n ? P.aprime_lo[l * n + q] : 0.0;
        }
        for (int k = tid; k < lw * n * NA; k += BSR) {
            const int la = k / NA, q = k - la * NA;
            B[2 * k] = q < n ? P.betaC[la * n + q] : 0.0;
            B[2 * k + 1] = q < n ? P.betaC_lo[la * n + q] : 0.0;
        }
    } else {
        // a neighbour at distance 0 adds the on-site term: B_n0 S_00 = c0_n
        A = cv.take(4 * (size_t)n * (n + 3));
        B = cv.take((size_t)n);
        for (int k = tid; k < 4 * n * (n + 3); k += BSR) A[k] = P.WN[k];
        for (int k = tid; k < n; k += BSR) B[k] = P.c0[k] * sqrt(4.0 * M_PI);
    }
    const int64_t origin = *P.rad_origin;
    for (int64_t c0 = (int64_t)blockIdx.x * cb; c0 < R.nc; c0 += (int64_t)gridDim.x * cb) {
        const int ncb = (int)((R.nc - c0) < cb ? (R.nc - c0) : cb);
        __syncthreads(); // the tables; the previous block's readers of rp
        for (int t = tid; t <= ncb; t += BSR) rp[t] = R.row_ptr[c0 + t];
        __syncthreads();
        for (int64_t eb = rp[0]; eb < rp[ncb]; eb += EB) {
            const int nE = (int)((rp[ncb] - eb) < EB ? (rp[ncb] - eb) : EB);
            if (eb != rp[0]) __syncthreads(); // the previous pass's readers of the tile
            for (int t = tid; t < nE; t += BSR) r2[t] = edge_r2(R, pos, rp, c0, ncb, eb + t);
            __syncthreads();
            const float inv_nE = 1.0f / (float)nE;
            const int items = (RBF == 2 ? n : lw) * nE;
            for (int it = tid; it < items; it += BSR) {
                const int q = qdiv(it, inv_nE), e = it - q * nE; // q: degree (Laplace form: radial index)
                const double d2 = r2[e];
                auto *o = tile + e * ldt;
                if constexpr (RBF == 0) {
                    // B = sum_k betaC e_k, Bh = sum_k betaC (-2 a'_k) e_k
                    double ex[NA], ea[NA];
#pragma unroll
                    for (int k = 0; k < NA; ++k) {
                        const double ap = A[q * NA + k];
                        ex[k] = exp_neg_tab(ap * d2, e2);
                        ea[k] = -2.0 * ap * ex[k];
                    }
                    const double *bc = B + (size_t)q * n * NA;
                    for (int a = 0; a < n; ++a) {
                        double b = 0.0, h = 0.0;
#pragma unroll
                        for (int k = 0; k < NA; ++k) {
                            b += bc[a * NA + k] * ex[k];
                            h += bc[a * NA + k] * ea[k];
                        }
                        o[a * lw + q] = d2 == 0.0 ? Pair<ST>::make(q == 0 ? b : 0.0, 0.0) : Pair<ST>::make(b, h);
                    }
                } else if constexpr (RBF == 3) {
#pragma clang fp contract(off)
                    // every exponential in double-double (a' as value and
                    // remainder), then compensated dot products (two-product
                    // and two-sum per term, the errors summed apart):
                    // B = sum_k betaC e_k, Bh = -2 sum_k (betaC a') e_k
                    dd ex[NA];
#pragma unroll
                    for (int k = 0; k < NA; ++k) {
                        const double ah = A[2 * (q * NA + k)], al = A[2 * (q * NA + k) + 1], xh = ah * d2;
                        ex[k] = dd_exp_neg(dd_fast_sum(xh, fma(ah, d2, -xh) + al * d2));
                    }
                    const double *bc = B + 2 * (size_t)q * n * NA;
                    for (int a = 0; a < n; ++a) {
                        double sb = 0.0, cb2 = 0.0, sh = 0.0, ch = 0.0;
#pragma unroll
                        for (int k = 0; k < NA; ++k) {
                            const double cx = bc[2 * (a * NA + k)], cy = bc[2 * (a * NA + k) + 1];
                            const dd m = dd_mul(dd{cx, cy}, dd{A[2 * (q * NA + k)], A[2 * (q * NA + k) + 1]});
                            const double pb = cx * ex[k].hi, ph = m.hi * ex[k].hi;
                            const dd tb = dd_two_sum(sb, pb), th = dd_two_sum(sh, ph);
                            sb = tb.hi;
                            sh = th.hi;
                            cb2 += (fma(cx, ex[k].hi, -pb) + tb.lo) + (cx * ex[k].lo + cy * ex[k].hi);
                            ch += (fma(m.hi, ex[k].hi, -ph) + th.lo) + (m.hi * ex[k].lo + m.lo * ex[k].hi);
                        }
                        const double b = sb + cb2, h = -2.0 * (sh + ch);
                        o[a * lw + q] = d2 == 0.0 ? Pair<ST>::make(q == 0 ? b : 0.0, 0.0) : Pair<ST>::make(b, h);
                    }
                } else {
                    // Laplace form: the P_j(u) = d^j/du^j sum_k WN_nk u^(k+2), u =
                    // r_cut - r, from their Chebyshev series (Clenshaw), then every degree:
                    //   f  = P_0 (1 - l(l+1) h/2) - s^2/r P_1 + s^2/2 P_2,  h = s^2/r^2,
                    //   f' = l(l+1) h/r P_0 + ((l(l+1)+2) h/2 - 1) P_1 + s^2/r P_2 - s^2/2 P_3
                    const double r = sqrt(d2);
                    const double tt = (P.rc - r) * P.inv_rc2 - 1.0, t2 = tt + tt;
                    const double *chp = A + (size_t)q * (n + 3) * 4;
                    double p[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        double b1 = 0.0, b2 = 0.0;
                        for (int i = n + 2; i >= 1; --i) {
                            const double nb1 = t2 * b1 - b2 + chp[4 * i + j];
                            b2 = b1;
                            b1 = nb1;
                        }
                        p[j] = tt * b1 - b2 + chp[j];
                    }
                    const double s2 = P.s2, hs2 = P.hs2, ir = r == 0.0 ? 0.0 : 1.0 / r, h = s2 * ir * ir;
                    double rl = 1.0; // r^-l
                    for (int l = 0; l < lw; ++l) {
                        double b, bh;
                        if (r == 0.0) {
                            b = l == 0 ? B[q] : 0.0;
                            bh = 0.0;
                        } else {
                            const double ll = (double)(l * (l + 1));
                            const double f = p[0] * (1.0 - 0.5 * ll * h) - s2 * ir * p[1] + hs2 * p[2];
                            const double fp = ll * h * ir * p[0] + (0.5 * (ll + 2.0) * h - 1.0) * p[1] +
                                              s2 * ir * p[2] - hs2 * p[3];
                            b = rl * f;
                            bh = rl * ir * (fp - (double)l * f * ir);
                        }
                        o[q * lw + l] = Pair<ST>::make(b, bh);
                        rl *= ir;
                    }
                }
            }
            __syncthreads();
            const float inv_per = 1.0f / (float)per;
            for (int k = tid; k < nE * per; k += BSR) {
                const int e = qdiv(k, inv_per);
                const typename Pair<ST>::type v = tile[e * ldt + k - e * per];
                store_pair<ST>(rad_row<ST>(P, eb + e - origin), k - e * per, v.x, v.y);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// The radial factors from a table: on each of rtab_k equal intervals of
// [0, r_cut] the polynomial through the factors at Chebyshev points, in t =
// 2 (r / h - k) - 1 on interval k.  Every B_nl and Bh_nl is a function smoothed
// by the Gaussians, so its j-th derivative is of order sigma^-j.
//
// Nothing but the factors themselves is rounded on the way to the records: h is
// a power of two, so that r / h, k and t are exact; the points are rounded to
// 2^-36 of an interval, so that their distances are exact as well; the values'
// transformation to monomial coefficients runs in double-double; and t takes
// the rounding error of r = sqrt(r^2).  (Coefficients formed in float64 at
// rounded points lost 20 to 100 ulp: the transformation's rows sum to over 100,
// and r / h amplifies a rounded r by the number of the interval.)
//
//   float64 records, h <= sigma / 20, degree 7: (B, Bh) coefficients of t^0..t^7
//   as 8 pairs.  Against 64-bit-mantissa arithmetic, relative to the largest
//   value on the interval: rms 8e-17 beyond the error of the points' values;
//   with the quadrature's values 2e-16 in the median, where the quadrature
//   itself has 3e-16 (sums of 64 terms; n_max 8, l_max 6).
//   float32 records, h <= sigma / 16, degree 6: t^0..t^2 as float64 pairs, t^3..t^6 as
//   float32 pairs.  The factor before its one rounding to float32 is off by 1e-12 to
//   4e-12 of the interval's largest value, the stored factor by the same 2.53e-8 rms
//   as that of the direct evaluation.  (Degree 4 with float32 from t^1 on, 48 bytes:
//   2e-9 and 5e-8 to 1e-6, worst next to a factor's zeros.)
// (3000-atom water, n_max 8, l_max 6: the quadrature's 64 nodes per edge took
// 435 us.)
// ---------------------------------------------------------------------------
template <typename ST> struct RadRecord;
template <> struct RadRecord<double> {
    static constexpr int D = 7;
    static constexpr double PER_SIGMA = 20.0; // intervals per sigma, at least
    double c[D + 1][2];
};
template <> struct RadRecord<float> {
    static constexpr int D = 6;
    static constexpr double PER_SIGMA = 16.0;
    static constexpr int ND = 3; // float64 coefficients
    double c[ND][2];
    float f[D + 1 - ND][2];
};
// In memory a record is NC chunks of 16 bytes, chunk c of an interval's records
// together: [interval][chunk][n lw], so that the lanes of a wave, which take
// consecutive factors of an edge, load consecutive chunks.
template <typename ST> constexpr int rad_chunks() { return sizeof(RadRecord<ST>) / 16; }
template <typename ST>
__device__ __forceinline__ RadRecord<ST> rad_load(const double2 *__restrict__ tab, int per, int64_t interval, int t) {
    double2 w[rad_chunks<ST>()];
    const double2 *p = tab + interval * (rad_chunks<ST>() * per) + t;
#pragma unroll
    for (int c = 0; c < rad_chunks<ST>(); ++c) w[c] = p[c * per];
    RadRecord<ST> q;
    __builtin_memcpy(&q, w, sizeof q);
    return q;
}
template <typename ST>
__device__ __forceinline__ void rad_store(const RadRecord<ST> &q, double2 *__restrict__ tab, int per, int64_t interval,
                                          int t) {
    double2 w[rad_chunks<ST>()];
    __builtin_memcpy(w, &q, sizeof q);
    for (int c = 0; c < rad_chunks<ST>(); ++c) tab[(interval * rad_chunks<ST>() + c) * per + t] = w[c];
}
__device__ __forceinline__ void rad_eval(const RadRecord<double> &q, double t, double &b, double &h) {
    b = q.c[7][0];
    h = q.c[7][1];
#pragma unroll
    for (int k = 6; k >= 0; --k) {
        b = __builtin_fma(b, t, q.c[k][0]);
        h = __builtin_fma(h, t, q.c[k][1]);
    }
}
__device__ __forceinline__ void rad_eval(const RadRecord<float> &q, double t, double &b, double &h) {
    const float tf = (float)t;
    float x = q.f[3][0], y = q.f[3][1];
#pragma unroll
    for (int k = 2; k >= 0; --k) {
        x = __builtin_fmaf(x, tf, q.f[k][0]);
        y = __builtin_fmaf(y, tf, q.f[k][1]);
    }
    b = (double)x;
    h = (double)y;
#pragma unroll
    for (int k = 2; k >= 0; --k) {
        b = __builtin_fma(b, t, q.c[k][0]);
        h = __builtin_fma(h, t, q.c[k][1]);
    }
}

// one record's coefficients from the values at its interval's D + 1 points
// (value p at v[p stride]); inv [k][p] (value, remainder): the points' values to
// the coefficient of t^k
template <int D>
__host__ __device__ __forceinline__ void rad_coefficients(const double *v, int64_t stride, const double *inv, double *c,
                                                          int cstride) {
    for (int k = 0; k <= D; ++k) {
        dd s{0.0, 0.0};
        for (int p = 0; p <= D; ++p) {
            const double *w = inv + 2 * (k * (D + 1) + p);
            s = dd_add(s, dd_mul(dd{w[0], w[1]}, dd{v[p * stride], 0.0}));
        }
        c[k * cstride] = s.hi;
    }
}

// the records from the factors at the intervals' points, vals [interval][point
// 0..D][n lw] (B, Bh)
template <typename ST>
__global__ __launch_bounds__(256) void k_radial_records(int64_t count, int per, const double2 *__restrict__ vals,
                                                        const double *__restrict__ inv,
                                                        double2 *__restrict__ out) {
    constexpr int D = RadRecord<ST>::D;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) {
        const int64_t iv = i / per;
        const double *v = (const double *)(vals + iv * (D + 1) * per + (i - iv * per));
        double c[D + 1][2];
        rad_coefficients<D>(v, 2 * (int64_t)per, inv, &c[0][0], 2);
        rad_coefficients<D>(v + 1, 2 * (int64_t)per, inv, &c[0][1], 2);
        RadRecord<ST> q;
        if constexpr (sizeof(ST) == 8) {
            for (int k = 0; k <= D; ++k)
                for (int j = 0; j < 2; ++j) q.c[k][j] = c[k][j];
        } else {
            constexpr int ND = RadRecord<ST>::ND;
            for (int k = 0; k <= D; ++k)
                for (int j = 0; j < 2; ++j) {
                    if (k < ND) q.c[k][j] = c[k][j];
                    else q.f[k - ND][j] = (float)c[k][j];
                }
        }
        rad_store(q, out, per, iv, (int)(i - iv * per));
    }
}

// A workgroup takes blocks of cb consecutive centers; per pass of up to
// RAD_TAB_EB edges it finds each edge's interval and t, then its threads take
// (edge, factor) with the factor running fastest: an edge's records and its
// pairs are contiguous.  An edge of length 0 has only its l = 0 factor B.
constexpr int RAD_TAB_EB = 256;
template <typename PosT, typename ST>
__global__ __launch_bounds__(BSR) void k_radial_table(Params P, Rows R, const PosT *__restrict__ pos, int cb) {
    __shared__ int64_t rp[RAD_CB_MAX + 1];
    __shared__ double tt[RAD_TAB_EB];
    __shared__ int iv[RAD_TAB_EB]; // -1 - interval for an edge of length 0
    const int tid = threadIdx.x, lw = P.lmax + 1, per = P.n * lw;
    const int64_t origin = *P.rad_origin;
    const double2 *tab = (const double2 *)P.rtab;
    const float inv_per = 1.0f / (float)per, inv_lw = 1.0f / (float)lw;
    for (int64_t c0 = (int64_t)blockIdx.x * cb; c0 < R.nc; c0 += (int64_t)gridDim.x * cb) {
        const int ncb = (int)((R.nc - c0) < cb ? (R.nc - c0) : cb);
        __syncthreads(); // the previous block's readers
        for (int t = tid; t <= ncb; t += BSR) rp[t] = R.row_ptr[c0 + t];
        __syncthreads();
        for (int64_t eb = rp[0]; eb < rp[ncb]; eb += RAD_TAB_EB) {
            const int nE = (int)((rp[ncb] - eb) < RAD_TAB_EB ? (rp[ncb] - eb) : RAD_TAB_EB);
            if (eb != rp[0]) __syncthreads(); // the previous pass's readers
            for (int t = tid; t < nE; t += BSR) {
                const double r2 = edge_r2(R, pos, rp, c0, ncb, eb + t), r = sqrt(r2);
                const double x = r * P.rtab_inv_h; // exact
                int k = (int)x; // r < r_cut; the last interval takes the rounding
                k = k < P.rtab_k ? k : P.rtab_k - 1;
                // sqrt(r2) = r + (r2 - r^2) / (2 r)
                const double dr2 = r > 0.0 ? __builtin_fma(-r, r, r2) / r : 0.0;
                tt[t] = __builtin_fma(dr2, P.rtab_inv_h, 2.0 * (x - (double)k) - 1.0);
                iv[t] = r == 0.0 ? -1 - k : k;
            }
            __syncthreads();
            for (int k0 = tid; k0 < nE * per; k0 += BSR) {
                const int e = qdiv(k0, inv_per), t = k0 - e * per;
                const int q = iv[e], k = q < 0 ? -1 - q : q;
                double b, h;
                rad_eval(rad_load<ST>(tab, per, k, t), tt[e], b, h);
                if (q < 0) {
                    b = t - qdiv(t, inv_lw) * lw == 0 ? b : 0.0;
                    h = 0.0;
                }
                store_pair<ST>(rad_row<ST>(P, eb + e - origin), t, b, h);
            }
        }
    }
}

// ---------------------------------------------------------------------------
// k_radial_quad: the polynomial basis by quadrature (the radial integral of
// Sec. 2.3, the sums over the basis and over the nodes swapped, G[n][q] =
// w_q r_q^2 g_n(r_q) 4 pi):
//   B_nl  = r^-l sum_q G_nq ii_l(x_q) g_q,
//   Bh_nl = (1/r) dB_nl/dr
//         = r^-l (1/r) sigma^-2 sum_q G_nq (r_q ii_{l+1}(x_q) - r ii_l(x_q)) g_q,
// x_q = r r_q / sigma^2, g_q = exp(-(r_q - r)^2 / (2 sigma^2)) (ii_l the
// exponentially scaled modified spherical Bessel function, the derivative
// from i_l' = i_{l+1} + (l/x) i_l), and for an edge of length 0 only the
// l = 0 factor, B_n0(0).  Output pairs [n][l] of the edge, for
// l <= l_max.
// A workgroup takes a block of cb consecutive centers, whose edges are
// contiguous; its waves take four edges at a time, round-robin, each lane
// finding its edge's center in the block's row offsets.  Per four edges the
// Bessel values of (edge, node) for 16 nodes at once go to the wave's LDS
// slab, then lane = (edge, l) accumulates all NA radial indices over those
// nodes (G broadcast from LDS).  The node sums run in node order, as in the
// in-kernel evaluation.
// ---------------------------------------------------------------------------
constexpr int RAD_EC = 4, RAD_QC = 16; // edges per wave pass; nodes per Bessel slab

__host__ __device__ __forceinline__ int radial_qpad(int Q) { return (Q + RAD_QC - 1) / RAD_QC * RAD_QC; }
// LDS doubles of k_radial_quad: the block's row offsets [RAD_CB_MAX + 1], G [NA][Qp], r_q [Qp], and
// per wave the Bessel slab [64][l_max + 2]
__host__ __device__ __forceinline__ size_t radial_quad_lds_doubles(const Params &P, int na) {
    const size_t qp = (size_t)radial_qpad(P.Q);
    return even(RAD_CB_MAX + 1) + even((size_t)na * qp) + even(qp) + NWR * even(64 * ((size_t)P.lmax + 2));
}

template <typename PosT, typename ST, int NA>
__global__ __launch_bounds__(BSR) void k_radial_quad(Params P, Rows R, const PosT *__restrict__ pos, int cb) {
    extern __shared__ __align__(16) double smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t origin = *P.rad_origin;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = P.n, Q = P.Q, Qp = radial_qpad(Q), lw = P.lmax + 1, tw = lw + 1;
    Carver cv{smem};
    int64_t *rp = (int64_t *)cv.take(RAD_CB_MAX + 1);
    double *G = cv.take((size_t)NA * Qp);
    double *rq = cv.take((size_t)Qp);
    double *slab = cv.take(0) + (size_t)wave * even(64 * (size_t)tw);
    for (int k = tid; k < NA * Qp; k += BSR) {
        const int a = k / Qp, q = k - a * Qp;
        G[k] = (a < n && q < Q) ? P.G[(size_t)a * Q + q] : 0.0;
    }
    for (int k = tid; k < Qp; k += BSR) rq[k] = k < Q ? P.rq[k] : 0.0;
    const int es = lane >> 4, sub = lane & 15; // edge slot; node (Bessel phase) or l (sum phase)
    double *mine = slab + (size_t)lane * tw;          // this lane's (edge, node) Bessel row
    const double *col = slab + (size_t)es * RAD_QC * tw; // this lane's edge, all 16 nodes
    const int l = sub < lw ? sub : lw - 1;
    for (int64_t c0 = (int64_t)blockIdx.x * cb; c0 < R.nc; c0 += (int64_t)gridDim.x * cb) {
        const int ncb = (int)((R.nc - c0) < cb ? (R.nc - c0) : cb);
        __syncthreads(); // the tables; the previous block's readers of rp
        for (int t = tid; t <= ncb; t += BSR) rp[t] = R.row_ptr[c0 + t];
        __syncthreads();
        const int64_t E1 = rp[ncb];
        for (int64_t eb = rp[0] + (int64_t)RAD_EC * wave; eb < E1; eb += (int64_t)RAD_EC * NWR) {
            const int64_t e = eb + es;
            const bool live = e < E1;
            double r = 0.0;
            if (live) r = sqrt(edge_r2(R, pos, rp, c0, ncb, e));
            double b[NA], h[NA];
#pragma unroll
            for (int a = 0; a < NA; ++a) b[a] = h[a] = 0.0;
            for (int q0 = 0; q0 < Qp; q0 += RAD_QC) {
                const int q = q0 + sub;
                if (live && q < Q) {
                    const double xq = rq[q];
                    const double gq = exp(-0.5 * (xq - r) * (xq - r) * P.inv_s2);
                    bessel_scaled_lds(lw, xq * r * P.inv_s2, gq, mine);
                } else {
                    for (int k = 0; k < tw; ++k) mine[k] = 0.0;
                }
                wave_sync();
#pragma unroll 2
                for (int qq = 0; qq < RAD_QC; ++qq) {
                    const double tl = col[qq * tw + l], d = rq[q0 + qq] * col[qq * tw + l + 1] - r * tl;
                    const double *g = G + q0 + qq;
#pragma unroll
                    for (int a = 0; a < NA; ++a) {
                        const double ga = g[(size_t)a * Qp];
                        b[a] += ga * tl;
                        h[a] += ga * d;
                    }
                }
                wave_sync(); // the slab is read before the next nodes overwrite it
            }
            if (live && sub < lw) {
                double sb = 1.0, sh = 0.0;
                if (r == 0.0) {
                    sb = l == 0 ? 1.0 : 0.0;
                } else {
                    const double ir = 1.0 / r;
                    double rl = 1.0;
                    for (int k = 0; k < l; ++k) rl *= ir;
                    sb = rl;
                    sh = rl * ir * P.inv_s2;
                }
                RadPair<ST> *o = rad_row<ST>(P, e - origin);
#pragma unroll
                for (int a = 0; a < NA; ++a)
                    if (a < n) store_pair<ST>(o, a * lw + l, b[a] * sb, h[a] * sh);
            }
        }
    }
}


} // namespace dev

static int radial_na(int n) { return n <= 4 ? 4 : (n <= 8 ? 8 : (n <= 12 ? 12 : 16)); }
template <typename T, typename ST, int NA> static const void *radial_kernel_n(int rbf) {
    if (rbf == 1) return (const void *)k_radial_quad<T, ST, NA>;
    if (rbf == 0) return (const void *)k_radial_flat<T, ST, NA, 0>;
    if (rbf == 2) return (const void *)k_radial_flat<T, ST, NA, 2>;
    if constexpr (sizeof(T) == 8) return (const void *)k_radial_flat<T, ST, NA, 3>; // float64 only
    return nullptr;
}
template <typename T, typename ST> static const void *radial_kernel_t(int rbf, int na) {
    switch (na) {
    case 4: return radial_kernel_n<T, ST, 4>(rbf);
    case 8: return radial_kernel_n<T, ST, 8>(rbf);
    case 12: return radial_kernel_n<T, ST, 12>(rbf);
    default: return radial_kernel_n<T, ST, 16>(rbf);
    }
}
static const void *radial_kernel(bool f64, bool ar64, int rbf, int na) {
    if (f64) return radial_kernel_t<double, double>(rbf, na);
    return ar64 ? radial_kernel_t<float, double>(rbf, na) : radial_kernel_t<float, float>(rbf, na);
}

size_t radial_bytes_per_edge(const Params &P, bool st64) { return (st64 ? 16 : 8) * (size_t)P.n * (P.lmax + 1); }

// direct: the factors from their definition, also where P has a table
static hipError_t launch_radial_from(const Params &P, const Rows &R, const void *pos, bool f64, bool ar64, double degree,
                                     bool direct, hipStream_t st) {
    if (R.nc <= 0) return hipSuccess;
    const int na = radial_na(P.n), pair = (f64 || ar64) ? 16 : 8;
    const bool table = P.rtab && !direct;
    const void *k = table ? (f64 ? (const void *)k_radial_table<double, double>
                                 : (ar64 ? (const void *)k_radial_table<float, double>
                                         : (const void *)k_radial_table<float, float>))
                          : radial_kernel(f64, ar64, P.rbf, na);
    if (!k) return hipErrorInvalidValue;
    const size_t lds =
        table ? 0 : 8 * (P.rbf == 1 ? radial_quad_lds_doubles(P, na) : radial_flat_lds_doubles(P, P.rbf, na, pair));
    int ncu = 256, dev_id = 0;
    (void)hipGetDevice(&dev_id);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev_id);
    // blocks of cb centers, one per workgroup: about one pass of edges, but at
    // least four workgroups per CU where the centers allow it (the quadrature,
    // whose waves take four edges at a time: 16)
    const bool quad = !table && P.rbf == 1;
    const int per_cu = quad ? 16 : 4;
    const int pass_edges = table ? RAD_TAB_EB : radial_tile_edges(P, pair);
    const int64_t pass = std::max<int64_t>(1, (int64_t)((double)pass_edges / std::max(1.0, degree)));
    int64_t cbl = (R.nc + (int64_t)per_cu * ncu - 1) / ((int64_t)per_cu * ncu);
    if (!quad) cbl = std::min(cbl, pass);
    int cb = (int)std::min<int64_t>(RAD_CB_MAX, cbl);
    const int64_t need = (R.nc + cb - 1) / cb;
    const int blocks = (int)std::min<int64_t>(need, (int64_t)ncu * 64);
    Params Pk = P;
    Rows Rk = R;
    void *args[] = {&Pk, &Rk, &pos, &cb};
    return hipLaunchKernel(k, dim3(blocks), dim3(BSR), args, lds, st);
}
hipError_t launch_radial(const Params &P, const Rows &R, const void *pos, bool f64, bool ar64, double degree,
                         hipStream_t st) {
    return launch_radial_from(P, R, pos, f64, ar64, degree, false, st);
}

// Most intervals of a table (doubling with 1 / sigma).  The quadrature is the slower one
// at any size of the table (whole step at 6144 intervals, 48 to 1500 atoms, n_max 2..12:
// 0.68 to 0.92 of its time; at 3072 0.68 to 0.91), so there the limit is on memory: 4096
// intervals of n_max 12, l_max 12 are 51 MB in float32 records and 82 MB in float64. The GTO
// exponentials (but for the compensated ones) cost less than records that don't stay in the L2: density step
// with the table over that without, 480 to 4096 centers, n_max 3..12: 192 and 384
// intervals 0.90 to 1.01, 768 0.96 to 1.02, 1536 0.95 to 1.05, 3072 1.00 to 1.14.
constexpr int RTAB_MAX_K = 4096, RTAB_MAX_K_GTO = 512;
double radial_table_inv_h(const Params &P, bool st64) {
    const double h = P.sigma / (st64 ? RadRecord<double>::PER_SIGMA : RadRecord<float>::PER_SIGMA);
    return std::exp2(-std::floor(std::log2(h)));
}
int radial_table_intervals(const Params &P, bool st64) {
    // the Laplace form is singular at r = 0; for GTO (rbf 0) the float64 records
    // (128 bytes a factor) cost more than the exponentials, the float32 ones less
    if (P.rbf == 2 || (P.rbf == 0 && st64)) return 0;
    const double k = std::ceil(P.rc * radial_table_inv_h(P, st64));
    return k <= (P.rbf == 0 ? RTAB_MAX_K_GTO : RTAB_MAX_K) ? std::max(1, (int)k) : 0;
}
size_t radial_table_bytes(const Params &P, bool st64) {
    const size_t rec = st64 ? sizeof(RadRecord<double>) : sizeof(RadRecord<float>);
    return rec * (size_t)radial_table_intervals(P, st64) * P.n * (P.lmax + 1);
}
// The points x[0..D] of an interval [-1, 1], and the pairs inv [k][p]: the inverse
// of their Vandermonde matrix by Gauss-Jordan elimination in extended precision.
static void radial_points(int D, long double *x, double *inv) {
    const int np = D + 1;
    std::vector<long double> M((size_t)np * 2 * np, 0.0L);
    for (int p = 0; p < np; ++p) x[p] = ldexpl(rintl(ldexpl(-cosl(M_PIl * (2 * p + 1) / (2 * np)), 36)), -36);
    for (int p = 0; p < np; ++p) {
        long double v = 1.0L;
        for (int k = 0; k < np; ++k, v *= x[p]) M[(size_t)p * 2 * np + k] = v;
        M[(size_t)p * 2 * np + np + p] = 1.0L;
    }
    for (int c = 0; c < np; ++c) {
        int piv = c;
        for (int r = c + 1; r < np; ++r)
            if (fabsl(M[(size_t)r * 2 * np + c]) > fabsl(M[(size_t)piv * 2 * np + c])) piv = r;
        for (int k = 0; k < 2 * np; ++k) std::swap(M[(size_t)c * 2 * np + k], M[(size_t)piv * 2 * np + k]);
        const long double d = 1.0L / M[(size_t)c * 2 * np + c];
        for (int k = 0; k < 2 * np; ++k) M[(size_t)c * 2 * np + k] *= d;
        for (int r = 0; r < np; ++r) {
            if (r == c) continue;
            const long double f = M[(size_t)r * 2 * np + c];
            for (int k = 0; k < 2 * np; ++k) M[(size_t)r * 2 * np + k] -= f * M[(size_t)c * 2 * np + k];
        }
    }
    for (int k = 0; k < np; ++k)
        for (int p = 0; p < np; ++p) {
            const long double v = M[(size_t)k * 2 * np + np + p];
            inv[2 * (k * np + p)] = (double)v;
            inv[2 * (k * np + p) + 1] = (double)(v - (long double)(double)v);
        }
}

// The table's values come from the float64 kernels above, over a "structure"
// whose neighbours sit at the intervals' points, RTAB_ROW of them per row of
// one center atom (GTO: compensated).
constexpr int RTAB_ROW = 8;
hipError_t build_radial_table(const Params &P, bool st64, void *tab) {
    const int K = radial_table_intervals(P, st64), D = st64 ? RadRecord<double>::D : RadRecord<float>::D, np = D + 1;
    const int per = P.n * (P.lmax + 1), pts = K * np;
    const long double h = 1.0L / (long double)radial_table_inv_h(P, st64);
    std::vector<long double> x(np);
    // one upload: inv [k][p], positions of the center (0) and the points, row
    // offsets, columns; then the values
    const size_t o_pos = 2 * (size_t)np * np;
    std::vector<double> up(o_pos + 3 * ((size_t)pts + 1), 0.0);
    radial_points(D, x.data(), up.data());
    double *pos = up.data() + o_pos;
    for (int k = 0; k < K; ++k)
        for (int p = 0; p < np; ++p) // exact: 12 bits of k, 37 of the point
            pos[3 * ((size_t)k * np + p + 1)] = (double)(((long double)k + (x[p] + 1.0L) / 2.0L) * h);
    const int nrow = (pts + RTAB_ROW - 1) / RTAB_ROW;
    const size_t o_row = up.size();
    up.resize(o_row + nrow + 1 + ((size_t)pts + nrow + 1) / 2, 0.0);
    int64_t *row = reinterpret_cast<int64_t *>(up.data() + o_row);
    for (int k = 0; k <= nrow; ++k) row[k] = std::min(pts, k * RTAB_ROW);
    int32_t *cols = reinterpret_cast<int32_t *>(row + nrow + 1); // then the rows' center atoms: 0
    for (int k = 0; k < pts; ++k) cols[k] = k + 1;
    double *dev = nullptr;
    const size_t up_bytes = 8 * up.size(), val_bytes = 16 * (size_t)pts * per;
    hipError_t e = hipMalloc((void **)&dev, up_bytes + 16 + val_bytes);
    if (e != hipSuccess) return e;
    double2 *vals = reinterpret_cast<double2 *>(dev + even(up.size()));
    e = hipMemcpy(dev, up.data(), up_bytes, hipMemcpyHostToDevice);
    if (e == hipSuccess) {
        Params Pp = P;
        if (Pp.rbf == 0) Pp.rbf = 3;
        Pp.rad = vals;
        Pp.rad_stride = 16 * (int64_t)per;
        Pp.rad_origin = reinterpret_cast<const int64_t *>(dev + o_row);
        Rows R{};
        R.n_atoms = pts + 1;
        R.nc = nrow;
        R.row_ptr = R.e_origin = Pp.rad_origin;
        R.cols = reinterpret_cast<const int32_t *>(dev + o_row + nrow + 1);
        R.centers = R.cols + pts;
        e = launch_radial_from(Pp, R, dev + o_pos, true, false, (double)RTAB_ROW, true, 0);
    }
    if (e == hipSuccess) {
        const int64_t count = (int64_t)K * per;
        const unsigned blocks = (unsigned)std::min<int64_t>((count + 255) / 256, 4096);
        if (st64)
            hipLaunchKernelGGL(k_radial_records<double>, dim3(blocks), dim3(256), 0, 0, count, per, vals, dev,
                               (double2 *)tab);
        else
            hipLaunchKernelGGL(k_radial_records<float>, dim3(blocks), dim3(256), 0, 0, count, per, vals, dev,
                               (double2 *)tab);
        e = hipGetLastError();
    }
    const hipError_t f = hipFree(dev); // waits for the kernels
    return e == hipSuccess ? f : e;
}

// the float64 records' arithmetic on the host: the points, and the coefficients of values there
extern "C" void soap_radial_record64(const double *vals, double *points, double *coef) {
    constexpr int D = RadRecord<double>::D;
    long double x[D + 1];
    double inv[2 * (D + 1) * (D + 1)];
    radial_points(D, x, inv);
    for (int p = 0; p <= D; ++p) points[p] = (double)x[p];
    rad_coefficients<D>(vals, 1, inv, coef, 1);
}

// dynamic LDS above the default limit for every variant (set_lds_limits)
hipError_t radial_set_lds_limit(int lim) {
    hipError_t e = hipSuccess;
    for (int v = 0; v < 3; ++v)
        for (int rbf = 0; rbf < 4; ++rbf)
            for (int na : {4, 8, 12, 16}) {
                const void *k = radial_kernel(v == 2, v == 1, rbf, na);
                if (k && e == hipSuccess)
                    e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, lim);
            }
    return e;
}

} // namespace soap
