// The density step of the Jacobian path on the matrix cores (built once per
// precision, DM_PART = 0, 1, 2, so that the parts compile in parallel).
//
// The coefficients c and the center derivative D = sum over edges of dc/dr_j,
//   dc_{a lm}/dr = Bh_al r S_lm + B_al grad S_lm  (solid harmonics S),
// take one product per entry for c and up to seven for D when they are summed
// entry by entry.  But r S_lm = r^2/(2l+1) grad S_lm + (a combination of degree
// l+1 harmonics with constant coefficients), and grad S_lm is one of degree l-1
// harmonics, so
//   D_{a lm} = T-_lm sum_e (B_al + Bh_al r^2/(2l+1)) S_{l-1}
//            + T+_lm sum_e Bh_al S_{l+1}
// with constant T-, T+: three sums per (a, lm) over the edges, each a product of
// radial factors by harmonics, and the constant combinations once per species.
// Per harmonic degree l' they are one matrix product over the row's edges:
// rows (B_l', B_{l'+1} + .., Bh_{l'-1}) x radial index, columns the 2l'+1
// harmonics, K the edges.
//
// One workgroup per center (persistent), chunks of up to W edges of one species:
//   staging: the radial pass's factors and the harmonics up to l_max + 1, columns m
//     over the waves, at the staging precision;
//   products: wave w owns the degrees l' = w, w + 4, ..., whose sums it keeps in
//     registers over the whole species run; four edges per product, aligned to
//     the run's start, so every sum is formed in the same order at any W;
//   species end: the sums to LDS (over the staging), D from them, c and D to the
//     scratch [c, Dx, Dy, Dz][lm][species n] for the output kernel and the edge
//     Jacobian kernel.
// What bounds it: the latency of these phases, at two workgroups per CU; the
// products themselves are 15 matrix instructions per edge at n_max 12, l_max 12
// (a tenth of its time).  3000-atom water, n_max 12, l_max 12: 0.71 ms against
// 1.48 in k_density.  Rows of a few edges per species leave the chunks nearly
// empty: CHNO (11 edges, 4 species) 0.31 against k_djs's 0.26.
#include "soap_device.h"

#ifndef DM_PART
#error "DM_PART must be defined"
#endif

namespace soap {
using namespace dev;
namespace dev {

__host__ __device__ __forceinline__ int dm_lp2(const Params &P) { return (P.lmax + 2) * (P.lmax + 2) | 1; }
__host__ __device__ __forceinline__ size_t dm_table_doubles(const Params &P) {
    const size_t ldN = (size_t)P.lmax + 2, n = (size_t)P.n, L = (size_t)P.L;
    // Nt, on-site terms, T+- (10 doubles and 6 16-bit words per lm)
    return even(ldN * ldN) + even(n) + 10 * L + even((6 * L + 3) / 4);
}
__host__ __device__ __forceinline__ size_t dm_stage_doubles(const Params &P, int W, int sb) {
    const size_t ly = (size_t)(P.lmax + 2) * (P.lmax + 2), lw = (size_t)P.lmax + 1;
    const size_t stage = even((ly * (W + 1) * sb + 7) / 8) + 2 * even((lw * desc_ldl(P.n, W) * sb + 7) / 8) + even(W);
    const size_t sums = 3 * (size_t)P.n * dm_lp2(P);
    return stage > sums ? even(stage) : even(sums);
}
__host__ __device__ __forceinline__ size_t dm_lds_doubles(const Params &P, int W, int sb) {
    return dm_table_doubles(P) + dm_stage_doubles(P, W, sb);
}

// NL: degrees l' per wave, ceil((l_max + 2) / 4); RT: 16-row tiles of the 3 n
// rows
template <typename T, typename ST, int NL, int RT>
__global__ __launch_bounds__(BSC, 2) void k_density_mx(Params P, Rows R, const T *__restrict__ pos, int W,
                                                       ST *__restrict__ c_scratch) {
    extern __shared__ __align__(16) double smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int S = P.S, n = P.n, lmax = P.lmax, lw = lmax + 1, L = P.L, ldN = lmax + 2, Sn = S * n, nL = n * L;
    const int LP2 = dm_lp2(P), LY = (lmax + 2) * (lmax + 2);
    constexpr int SB = sizeof(ST);
    Carver cv{smem};
    double *Nt = cv.take((size_t)ldN * ldN);
    double *c0 = cv.take((size_t)n);
    double *tm = cv.take(10 * (size_t)L); // [10][L]
    uint16_t *ti = (uint16_t *)cv.take((6 * (size_t)L + 3) / 4); // [6][L]
    const int WP = W + 1, ldl = desc_ldl(n, W);
    double *stage = cv.take(dm_stage_doubles(P, W, SB));
    double *X = stage; // the species' sums [3 n][LP2], over the staging
    Carver sv{stage};
    ST *Yl = (ST *)sv.take(((size_t)LY * WP * SB + 7) / 8);  // [lm'][W + 1]
    ST *Bl = (ST *)sv.take(((size_t)lw * ldl * SB + 7) / 8); // [l][n][W + 1]
    ST *Hl = (ST *)sv.take(((size_t)lw * ldl * SB + 7) / 8);
    double *r2s = sv.take((size_t)W);
    for (int k = tid; k < ldN * ldN; k += BSC) Nt[k] = P.Nt[k];
    for (int k = tid; k < n; k += BSC) c0[k] = P.c0[k];
    for (int k = tid; k < 10 * L; k += BSC) tm[k] = P.dtm[k];
    for (int k = tid; k < 6 * L; k += BSC) ti[k] = P.dti[k];
    // this lane's operands: A row 16 rt + (lane & 15) = which n + a of radial
    // factors, B column (lane & 15) of harmonics, K = edge lane >> 4 of four
    const int ro = lane & 15, kk = lane >> 4;
    double fB[RT], f0[RT], f1[RT];
    int oR[NL][RT], oY[NL][2];
    uint32_t live = 0; // bit j RT + rt: the row's degree exists
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int r = 16 * rt + ro, which = r < n ? 0 : (r < 2 * n ? 1 : 2), a = r - which * n;
        fB[rt] = which < 2 ? 1.0 : 0.0;
        f1[rt] = which == 1 ? 1.0 : 0.0;
        f0[rt] = which == 2 ? 1.0 : 0.0;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int lp = wave + 4 * j, ls = which == 0 ? lp : (which == 1 ? lp + 1 : lp - 1);
            const bool ok = r < 3 * n && ls >= 0 && ls <= lmax;
            oR[j][rt] = ok ? ls * ldl + a * WP : 0;
            live |= ok ? 1u << (j * RT + rt) : 0u;
        }
    }
#pragma unroll
    for (int j = 0; j < NL; ++j)
#pragma unroll
        for (int ct = 0; ct < 2; ++ct) {
            const int lp = wave + 4 * j <= lmax + 1 ? wave + 4 * j : 0, m = 16 * ct + ro;
            oY[j][ct] = (lp * lp + (m <= 2 * lp ? m : 2 * lp)) * WP;
        }
    double wl[NL]; // 1 / (2l + 1) of the middle rows' degree l = l' + 1
#pragma unroll
    for (int j = 0; j < NL; ++j) wl[j] = 1.0 / (double)(2 * (wave + 4 * j) + 3);
    const float inv_n = 1.0f / (float)n;
    const int64_t rad0 = *P.rad_origin;

    int64_t ci = blockIdx.x;
    const int64_t stride = gridDim.x;
    double gx = 0.0, gy = 0.0, gz = 0.0;
    int gs = -1;
    int64_t e0 = 0, e1 = 0;
    double3 pi = make_double3(0.0, 0.0, 0.0);
    int spec_i = 0;
    // the next up to W edges from cs on, one per lane (every wave)
    auto gather = [&](int64_t cs) {
        gx = gy = gz = 0.0;
        gs = -1;
        if (lane < W && cs + lane < e1) {
            const int64_t j = R.cols[cs + lane];
            gx = (double)pos[3 * j] - pi.x;
            gy = (double)pos[3 * j + 1] - pi.y;
            gz = (double)pos[3 * j + 2] - pi.z;
            gs = R.spec[j];
        }
    };
    auto fetch = [&]() {
        if (ci >= R.nc) return;
        const int64_t i = R.centers ? (int64_t)R.centers[ci] : R.c_base + ci;
        pi = make_double3((double)pos[3 * i], (double)pos[3 * i + 1], (double)pos[3 * i + 2]);
        spec_i = R.spec[i];
        e0 = R.row_ptr[ci];
        e1 = R.row_ptr[ci + 1];
        gather(e0);
    };
    fetch();
    while (ci < R.nc) {
        const int64_t cw = ci;
        const int spec_c = spec_i;
        ST *sc = c_scratch + cw * 4 * (size_t)L * Sn;
        dbl4 acc[NL][2][RT];
        auto clear = [&]() {
#pragma unroll
            for (int j = 0; j < NL; ++j)
#pragma unroll
                for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) acc[j][ct][rt] = dbl4{0.0, 0.0, 0.0, 0.0};
        };
        // c and D of species s: the combinations of its sums, or zeros
        auto put = [&](int s, bool sums) {
            for (int it = tid; it < nL; it += BSC) {
                const int lm = qdiv(it, inv_n), a = it - lm * n;
                double v[4] = {0.0, 0.0, 0.0, 0.0};
                if (sums) {
                    const double *x1 = X + (size_t)(n + a) * LP2, *x2 = X + (size_t)(2 * n + a) * LP2;
                    v[0] = X[(size_t)a * LP2 + lm];
                    const int p0 = ti[lm], p1 = ti[L + lm], p2 = ti[2 * L + lm];
                    const int q0 = ti[3 * L + lm], q1 = ti[4 * L + lm], q2 = ti[5 * L + lm];
                    v[1] = (tm[lm] * x1[p0 & 255] + tm[L + lm] * x1[p0 >> 8]) +
                           (tm[5 * L + lm] * x2[q0 & 255] + tm[6 * L + lm] * x2[q0 >> 8]);
                    v[2] = (tm[2 * L + lm] * x1[p1 & 255] + tm[3 * L + lm] * x1[p1 >> 8]) +
                           (tm[7 * L + lm] * x2[q1 & 255] + tm[8 * L + lm] * x2[q1 >> 8]);
                    v[3] = tm[4 * L + lm] * x1[p2 & 255] + tm[9 * L + lm] * x2[q2 & 255];
                }
                if (s == spec_c && lm == 0) v[0] += c0[a];
#pragma unroll
                for (int d = 0; d < 4; ++d) sc[((size_t)d * L + lm) * Sn + s * n + a] = (ST)v[d];
            }
        };
        // the end of species s: its sums to X, then c and D
        auto finish = [&](int s) {
            lds_barrier(); // the staging is read
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                const int lp = wave + 4 * j;
                if (lp > lmax + 1) continue; // uniform
#pragma unroll
                for (int ct = 0; ct < (j < 2 ? 1 : 2); ++ct) {
                    const int m = 16 * ct + ro;
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int r = 16 * rt + kk + 4 * i;
                            if (r < 3 * n && m <= 2 * lp) X[(size_t)r * LP2 + lp * lp + m] = acc[j][ct][rt][i];
                        }
                }
            }
            lds_barrier();
            put(s, true);
        };
        int cur = -1;
        clear();
        lds_barrier(); // the tables
        for (int64_t cs = e0; cs < e1;) {
            const int s = __builtin_amdgcn_readfirstlane(gs);
            const int nb = __popcll(__ballot(gs == s)), nb4 = (nb + 3) & ~3;
            if (s != cur) { // uniform: rows are sorted by species
                if (cur >= 0) {
                    finish(cur);
                    clear();
                }
                for (int z = cur + 1; z < s; ++z) put(z, false);
                cur = s;
            }
            lds_barrier(); // the previous chunk's readers of the staging (and of X)
            // ---- staging ----
            const bool mine = lane < nb;
            if (!mine) gx = gy = gz = 0.0; // edges of the next species, padding: no harmonic past l = 0, zero factors
            if (wave == 0 && lane < W) r2s[lane] = gx * gx + gy * gy + gz * gz;
            stage_radial<ST>(P, cs - rad0, nb, tid, Bl, Hl, ldl, WP);
            const int pad = nb4 - nb, per = n * lw;
            for (int k = tid; k < pad * per; k += BSC) {
                const int e = k / per, t = k - e * per, a = t / lw, l = t - a * lw, o = l * ldl + a * WP + nb + e;
                Bl[o] = (ST)0;
                Hl[o] = (ST)0;
            }
            // the harmonics up to l_max + 1: W lanes of edges, column groups over the rest
            {
                const int cgr = 64 / W, cg = lane / W, el = lane - cg * W;
                const double x = __shfl(gx, el), y = __shfl(gy, el), z = __shfl(gz, el);
                if (el < nb4) sh_cols_lane(x, y, z, Nt, ldN, lw + 1, Yl + el, WP, wave, NWC, cg, cgr);
            }
            const int64_t cn = cs + nb;
            if (cn < e1) gather(cn); // in flight through the products
            lds_barrier();
            // ---- products, four edges at a time ----
            for (int g = kk; g < nb4; g += 4) {
                const double r2 = r2s[g];
#pragma unroll
                for (int j = 0; j < NL; ++j) {
                    const int lp = wave + 4 * j;
                    if (lp > lmax + 1) continue; // uniform
                    const double w = r2 * wl[j];
                    double yv[2];
#pragma unroll
                    for (int ct = 0; ct < (j < 2 ? 1 : 2); ++ct) yv[ct] = (double)Yl[oY[j][ct] + g];
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) {
                        const double vb = (double)Bl[oR[j][rt] + g], vh = (double)Hl[oR[j][rt] + g];
                        double v = __builtin_fma(__builtin_fma(f1[rt], w, f0[rt]), vh, fB[rt] * vb);
                        v = (live >> (j * RT + rt)) & 1u ? v : 0.0;
#pragma unroll
                        for (int ct = 0; ct < (j < 2 ? 1 : 2); ++ct)
                            acc[j][ct][rt] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, yv[ct], acc[j][ct][rt], 0, 0, 0);
                    }
                }
            }
            cs = cn;
        }
        ci += stride;
        fetch(); // the next center's first edges before this center's stores
        if (cur >= 0) finish(cur);
        for (int z = cur + 1; z < S; ++z) put(z, false);
    }
}

} // namespace dev

#if DM_PART == 0
using DT = float;
using DS = float;
#elif DM_PART == 1
using DT = float;
using DS = double;
#else
using DT = double;
using DS = double;
#endif
#define DM_CAT2(a, b) a##b
#define DM_CAT(a, b) DM_CAT2(a, b)

template <int NL> static const void *dm_pick(int n) {
    const int rt = (3 * n + 15) / 16;
    return rt == 1 ? (const void *)k_density_mx<DT, DS, NL, 1>
                   : (rt == 2 ? (const void *)k_density_mx<DT, DS, NL, 2> : (const void *)k_density_mx<DT, DS, NL, 3>);
}
const void *DM_CAT(density_mx_, DM_PART)(int n, int lmax) {
    switch ((lmax + 5) / 4) {
    case 1: return dm_pick<1>(n);
    case 2: return dm_pick<2>(n);
    case 3: return dm_pick<3>(n);
    case 4: return dm_pick<4>(n);
    default: return nullptr;
    }
}

#if DM_PART == 0
static const void *dm_kernel(const Params &P, bool f64, bool ar64) {
    if (f64) return density_mx_2(P.n, P.lmax);
    return ar64 ? density_mx_1(P.n, P.lmax) : density_mx_0(P.n, P.lmax);
}

size_t density_mx_lds(const Params &P, int W, bool st64) { return 8 * dm_lds_doubles(P, W, st64 ? 8 : 4); }

int density_mx_blocks_per_cu(const Params &P, bool f64, bool ar64, size_t lds) {
    const void *k = dm_kernel(P, f64, ar64);
    int nb = 0;
    if (!k || hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 159 * 1024) != hipSuccess) return 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, BSC, lds) == hipSuccess ? nb : 0;
}

hipError_t launch_density_mx(const Params &P, const Rows &R, const void *pos, bool f64, bool ar64,
                             const DensityMxLaunch &cfg, void *c_scratch, hipStream_t st) {
    if (R.nc <= 0) return hipSuccess;
    Params Pk = P;
    Rows Rk = R;
    int W = cfg.W;
    void *args[] = {&Pk, &Rk, &pos, &W, &c_scratch};
    // persistent: as many workgroups as stay resident, each striding over the centers
    const int64_t blocks = std::min<int64_t>(R.nc, (int64_t)cfg.blocks);
    return hipLaunchKernel(dm_kernel(P, f64, ar64), dim3((unsigned)blocks), dim3(BSC), args, cfg.lds, st);
}
#endif

} // namespace soap
