// The edge Jacobian kernel: one workgroup per center, its waves working
// through the row in chunks of a few edges, in two phases per chunk.
//
//   J[i <- j] of an edge (i, j), species s, r = r_j - r_i:
//     (mu, s), mu < s:  K_l [U^mu_nl Bh_n'l r + V^mu_nl B_n'l]
//     (s, nu), nu > s:  K_l [Bh_nl r U^nu_n'l + B_nl V^nu_n'l]
//     (s, s), n' >= n:  both with mu = nu = s
//   (Eq. powerspectrum-derivative), U^nu_nl = sum_m S_lm c^nu_nlm and
//   V^nu_nl = sum_m grad S_lm c^nu_nlm.
//
//   1. U, V on the matrix cores: per degree a chain of 16x16x4 products, rows
//      (U, Vx, Vy, Vz) x 4 edges, K = m, columns 16 coefficients u = (species,
//      n).  A wave owns one column tile and the degrees of one parity, whose
//      coefficients it keeps in registers for the whole row.  The gradient
//      rows are formed as the products need them, each from two harmonics of
//      degree l-1 (the identities of stage_edges as a table): held in LDS they
//      would take three times the harmonics' space.
//   2. assembly: items (edge, species pair) over the waves; consecutive lanes
//      store consecutive values.
//
// What bounds it: U and V of an edge take 16 S n (l_max + 1) bytes of LDS
// until the edge is assembled, so the edges in flight on a CU are few at the
// large bases; the chunk is shared by all waves of the workgroup to have many
// waves per edge in flight.  The radial factors come from the radial pass
// (loaded one chunk ahead, before the stores of the current one: loads and
// stores retire in order), so no basis table takes LDS.  Stores of 16 bytes per
// lane over consecutive slots, 1 KB per wave and row, reach 5.3 TB/s in a pure
// store kernel, the 4-byte stores of 56 lanes of k_jacobian 4.7.
// 3000-atom water, n_max 12, l_max 12: 1.77 ms (4.0 TB/s) against k_jacobian's
// 2.86; CHNO, 4096 atoms, n_max 10, l_max 10: 0.65 against 0.80; polynomial n_max 8,
// l_max 6: 0.49 against 0.57.
#include "soap_device.h"

#include <cmath>

namespace soap {
using namespace dev;
namespace dev {

constexpr int EB_MAX_WAVES = 8;  // waves per workgroup
constexpr int EB_PF = 4;         // radial pairs prefetched per thread

// Table of the matrix-core rows in LDS and global memory: row comp (0: S,
// 1..3: dS/dx_comp) of harmonic lm is alpha Y[p] + beta Y[q]; alpha [4][Lp],
// beta [2][Lp] (x, y; the other rows take their q at the zero slot), Lp = L +
// 3, then (p | q << 8) [4][Lp] as 16-bit words.
__host__ __device__ __forceinline__ int eb_lp(const Params &P) { return P.L + 3; }
// row length of the staged harmonics: L values, a zero, odd
__host__ __device__ __forceinline__ int eb_ys(const Params &P) { return (P.L + 1) | 1; }
// LDS doubles for Q quads of edges per chunk, row blocks of RB edges
__host__ __device__ __forceinline__ size_t eb_lds_doubles(const Params &P, int Q, int RB, int ab) {
    const size_t EC = 4 * (size_t)Q, ldN = (size_t)P.lmax + 2, lw = (size_t)P.lmax + 1, lp = eb_lp(P);
    return 16 + even(ldN * ldN) + even(6 * lp) + even(lp) + even(EC * eb_ys(P)) +
           even((EC * 4 * P.S * P.n * lw * ab + 7) / 8) + even((EC * 2 * P.n * lw * ab + 7) / 8) + even(4 * (size_t)RB) +
           even((RB + 1) / 2) + even(((size_t)P.tri_lw + 1) / 2);
}

// VN consecutive values of the three rows of a block (fewer at a section's
// end), as one store per row: 4-byte alignment suffices
template <typename T, int VN> struct __attribute__((packed, aligned(4))) Run {
    T v[VN];
};
template <typename T, int VN>
__device__ __forceinline__ void store_rows(T *o, uint32_t Fe, int left, const T *x, const T *y, const T *z) {
    if (left >= VN) {
        Run<T, VN> r;
#pragma unroll
        for (int k = 0; k < VN; ++k) r.v[k] = x[k];
        *(Run<T, VN> *)o = r;
#pragma unroll
        for (int k = 0; k < VN; ++k) r.v[k] = y[k];
        *(Run<T, VN> *)(o + Fe) = r;
#pragma unroll
        for (int k = 0; k < VN; ++k) r.v[k] = z[k];
        *(Run<T, VN> *)(o + 2 * Fe) = r;
    } else {
#pragma unroll
        for (int k = 0; k < VN - 1; ++k)
            if (k < left) {
                o[k] = x[k];
                o[Fe + k] = y[k];
                o[2 * Fe + k] = z[k];
            }
    }
}

template <typename T> struct alignas(16) Quad {
    T u, x, y, z;
};

// HI: ceil((l_max + 1) / 2), the degrees of one parity; degree l = 2 i + h has
// i + 1 chunks of four m in either parity.
template <typename PosT, typename OutT, typename AT, int HI>
__global__ __launch_bounds__(64 * EB_MAX_WAVES, 4) void k_edge_blocks(Params P, Rows R, const PosT *__restrict__ pos,
                                                                     int Q, int RB, int split,
                                                                     const AT *__restrict__ c_scratch,
                                                                     typename EdgeBlocks<OutT, RBF_BUFFERED>::ptr jedge) {
    using AT2 = typename Pair<AT>::type;
    using AT4 = Quad<AT>;
    constexpr int NCH = HI * (HI + 1) / 2;
    constexpr int VN = 16 / sizeof(OutT); // values per lane and store
    extern __shared__ __align__(16) double smem[];
    const int S = P.S, n = P.n, lw = P.lmax + 1, L = P.L, Sn = S * n, ldN = lw + 1, tid = threadIdx.x;
    const int BS = blockDim.x, NW = BS >> 6, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int Fe = P.Fe, nl = n * lw, nnl = n * nl, tri_lw = P.tri_lw, EC = 4 * Q, YS = eb_ys(P), Lp = eb_lp(P);
    // `split` workgroups per center, each a run of whole chunks of its row
    const int64_t ci = blockIdx.x / split;
    const int part = blockIdx.x - (int)ci * split;
    int64_t e0 = R.row_ptr[ci], e1 = R.row_ptr[ci + 1];
    {
        const int64_t nch = (e1 - e0 + EC - 1) / EC, c0 = nch * part / split, c1 = nch * (part + 1) / split;
        e1 = c1 == nch ? e1 : e0 + c1 * EC;
        e0 += c0 * EC;
    }
    if (e1 <= e0) return;
    const int64_t ebase = *R.e_origin, rad0 = *P.rad_origin;

    Carver cv{smem};
    double *Kl = cv.take(16);
    double *Nt = cv.take((size_t)ldN * ldN);
    double *alpha = cv.take(6 * (size_t)Lp), *beta = alpha + 4 * Lp;
    uint16_t *pq = (uint16_t *)cv.take((size_t)Lp);
    double *Y = cv.take((size_t)EC * YS);                                        // [edge][lm], Y[L] = 0
    AT4 *UV = (AT4 *)cv.take(((size_t)EC * 4 * Sn * lw * sizeof(AT) + 7) / 8);   // [edge][u][l] = K_l (U, V)
    AT2 *G = (AT2 *)cv.take(((size_t)EC * 2 * nl * sizeof(AT) + 7) / 8);         // [edge][n][l] = (B, Bh)
    double *rgeo = cv.take(4 * (size_t)RB);
    int *rsp = (int *)cv.take((size_t)(RB + 1) / 2);
    uint32_t *dtab = (uint32_t *)cv.take(((size_t)tri_lw + 1) / 2);

    // this wave's part of the products: column tile, parity of the degrees, quad of edges
    const int NT = (Sn + 15) >> 4;
    const int wt = wave % NT, wr = wave / NT, h = wr & 1, wq = wr >> 1;
    const int comp = (lane & 15) >> 2, a_e = 4 * wq + (lane & 3), kk = lane >> 4, u = 16 * wt + (lane & 15);
    const int o_e = 4 * wq + (lane >> 4); // the edge of this lane's results
    const bool uok = u < Sn;
    AT bf[NCH]; // this tile's coefficients of the wave's degrees, [i][chunk]
    {
        const AT *cg = c_scratch + ci * 4 * (size_t)Sn * L + (uok ? u : 0); // component c of [c, Dx, Dy, Dz]
        int k = 0;
#pragma unroll
        for (int i = 0; i < HI; ++i) {
            const int l = 2 * i + h;
#pragma unroll
            for (int ch = 0; ch <= i; ++ch, ++k) {
                const int m = 4 * ch + kk;
                const bool ok = l < lw && m <= 2 * l && uok;
                const AT v = cg[(size_t)(ok ? l * l + m : 0) * Sn];
                bf[k] = ok ? v : (AT)0;
            }
        }
    }
    const int64_t ic = R.centers ? (int64_t)R.centers[ci] : R.c_base + ci;
    const double3 pi = make_double3((double)pos[3 * ic], (double)pos[3 * ic + 1], (double)pos[3 * ic + 2]);
    load_rows(rgeo, rsp, pos, R.spec, R.cols, e0, (int)((e1 - e0) < RB ? (e1 - e0) : RB), pi);
    if (tid < 16) Kl[tid] = M_PI * sqrt(8.0 / (double)(2 * tid + 1));
    for (int k = tid; k < ldN * ldN; k += BS) Nt[k] = P.Nt[k];
    for (int k = tid; k < 6 * Lp; k += BS) alpha[k] = P.jab[k];
    for (int k = tid; k < 4 * Lp; k += BS) pq[k] = P.jpq[k];
    for (int k = tid; k < EC; k += BS) Y[k * YS + L] = 0.0;
    for (int k = tid; k < tri_lw; k += BS) dtab[k] = P.dtab[k];
    const double *ap = alpha + comp * Lp + kk, *bp = beta + (comp == 2 ? Lp : 0) + kk, *Ya = Y + a_e * YS;
    const uint16_t *pp = pq + comp * Lp + kk;

    const float inv_lw = 1.0f / (float)lw, inv_nl = 1.0f / (float)nl;
    // harmonics of a chunk's edges: one (edge, column m) per thread
    auto stage_y = [&](int off, int nb) {
        for (int it = tid; it < nb * lw; it += BS) {
            const int e = qdiv(it, inv_lw), m = it - e * lw;
            const double *g = rgeo + 4 * (off + e);
            sh_col_y(m, m, lw, g[0], g[1], g[2], Nt, ldN, Y + e * YS, 1, 0);
        }
    };
    // radial pairs k of a chunk (edge-major); a zero-length edge gets zeros (a zero block)
    auto radial_at = [&](int64_t eb, int off, int k) {
        const int e = qdiv(k, inv_nl), t = k - e * nl;
        AT2 v = load_pair<AT>(rad_row<AT>(P, eb + e - rad0), t);
        if (rgeo[4 * (off + e) + 3] == 0.0) v.x = v.y = (AT)0;
        return v;
    };
    AT2 g[EB_PF];
    auto prefetch = [&](int64_t eb, int off, int nb) {
        const int cnt = nb * nl;
#pragma unroll
        for (int v = 0; v < EB_PF; ++v)
            if (v * BS < cnt) g[v] = radial_at(eb, off, v * BS + tid < cnt ? v * BS + tid : 0);
    };

    for (int64_t rb0 = e0; rb0 < e1; rb0 += RB) {
        const int rbn = (int)((e1 - rb0) < RB ? (e1 - rb0) : RB);
        if (rb0 != e0) { // (the barrier at the end of the last chunk: every wave is done with the block)
            load_rows(rgeo, rsp, pos, R.spec, R.cols, rb0, rbn, pi);
        }
        lds_barrier(); // the tables, the block's edges
        int nb = rbn < EC ? rbn : EC;
        stage_y(0, nb);
        prefetch(rb0, 0, nb);
        lds_barrier();
        for (int off = 0; off < rbn; off += EC) {
            const int64_t eb = rb0 + off;
            // this chunk's factors to LDS; more than the prefetched ones (large bases) from memory
            {
                const int cnt = nb * nl;
#pragma unroll
                for (int v = 0; v < EB_PF; ++v)
                    if (v * BS + tid < cnt) G[v * BS + tid] = g[v];
                for (int k = EB_PF * BS + tid; k < cnt; k += BS) G[k] = radial_at(eb, off, k);
            }
            const int noff = off + EC, nnb = noff < rbn ? ((rbn - noff) < EC ? rbn - noff : EC) : 0;
            if (nnb > 0) prefetch(eb + EC, noff, nnb);

            // ---- U, V ----
            {
                int k = 0;
#pragma unroll
                for (int i = 0; i < HI; ++i) {
                    const int l = 2 * i + h;
                    if (l < lw) { // uniform
                        const int b = l * l;
                        dbl4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                        for (int ch = 0; ch <= i; ++ch) {
                            const int o = pp[b + 4 * ch];
                            const double av = ap[b + 4 * ch] * Ya[o & 255] + bp[b + 4 * ch] * Ya[o >> 8];
                            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(av, (double)bf[k + ch], acc, 0, 0, 0);
                        }
                        if (uok && o_e < nb) {
                            const double K = Kl[l];
                            AT4 v;
                            v.u = (AT)(K * acc[0]);
                            v.x = (AT)(K * acc[1]);
                            v.y = (AT)(K * acc[2]);
                            v.z = (AT)(K * acc[3]);
                            UV[(o_e * Sn + u) * lw + l] = v;
                        }
                    }
                    k += i + 1;
                }
            }
            lds_barrier();
            // the next chunk's factors are waited for here, not behind the stores below
            if (nnb > 0) {
#pragma unroll
                for (int v = 0; v < EB_PF; ++v)
                    if (v * BS < nnb * nl) __asm__ volatile("" : "+v"(g[v].x), "+v"(g[v].y));
                stage_y(noff, nnb);
            }

            // ---- assembly: items (edge, other species), the diagonal pairs last ----
            for (int it = wave; it < nb * S; it += NW) {
                const int sg = it / nb, e = it - sg * nb;
                const int s = __builtin_amdgcn_readfirstlane(rsp[off + e]);
                int os = s + S - 1 - sg;
                os = os >= S ? os - S : os;
                const double *geo = rgeo + 4 * (off + e);
                const AT rx = (AT)geo[0], ry = (AT)geo[1], rz = (AT)geo[2];
                const AT2 *Be = G + e * nl;
                const AT4 *Ue = UV + ((size_t)e * Sn + os * n) * lw;
                OutT *o = jedge + (eb + e - ebase) * 3 * Fe;
                // slots of the section, VN consecutive ones per lane and store
                // (a lane owning some (n', l) and walking n needs a third
                // fewer LDS reads, but its shorter store runs cost more)
                if (os != s) { // (n, n', l): n of the lower species, n' of the higher
                    const bool up = os > s;
                    OutT *ob = o + (up ? s * nnl + tri_lw + (os - s - 1) * nnl : os * nnl);
                    for (int f0 = VN * lane; f0 < nnl; f0 += 64 * VN) {
                        int a = qdiv(f0, inv_nl), tt = f0 - a * nl, l = tt - qdiv(tt, inv_lw) * lw;
                        OutT vx[VN], vy[VN], vz[VN];
#pragma unroll
                        for (int v = 0; v < VN; ++v) {
                            const int al = a * lw + l;
                            const AT2 bb = Be[up ? al : tt];
                            const AT4 q = Ue[up ? tt : al];
                            const AT hu = bb.y * q.u;
                            vx[v] = (OutT)(hu * rx + bb.x * q.x);
                            vy[v] = (OutT)(hu * ry + bb.x * q.y);
                            vz[v] = (OutT)(hu * rz + bb.x * q.z);
                            // past the section's end the slot stays in range of the arrays (not stored)
                            if (v + 1 < VN && f0 + v + 1 < nnl) jac_next_slot(a, tt, l, nl, lw);
                        }
                        store_rows<OutT, VN>(ob + f0, Fe, nnl - f0, vx, vy, vz);
                    }
                } else { // (s, s): (n, n' >= n, l)
                    OutT *ob = o + s * nnl;
                    for (int f0 = VN * lane; f0 < tri_lw; f0 += 64 * VN) {
                        OutT vx[VN], vy[VN], vz[VN];
#pragma unroll
                        for (int v = 0; v < VN; ++v) {
                            const uint32_t d = dtab[f0 + v < tri_lw ? f0 + v : f0];
                            const int ta = d & 0xffff, tb = d >> 16; // n lw + l, n' lw + l
                            const AT2 A = Be[ta], B = Be[tb];
                            const AT4 qa = Ue[ta], qb = Ue[tb];
                            const AT hu = B.y * qa.u + A.y * qb.u;
                            vx[v] = (OutT)(hu * rx + (B.x * qa.x + A.x * qb.x));
                            vy[v] = (OutT)(hu * ry + (B.x * qa.y + A.x * qb.y));
                            vz[v] = (OutT)(hu * rz + (B.x * qa.z + A.x * qb.z));
                        }
                        store_rows<OutT, VN>(ob + f0, Fe, tri_lw - f0, vx, vy, vz);
                    }
                }
            }
            nb = nnb;
            lds_barrier(); // U, V and G are free; the next harmonics are in place
        }
    }
}

} // namespace dev

template <typename T, typename AT> static const void *eb_kernel_t(int hi) {
    switch (hi) {
    case 1: return (const void *)k_edge_blocks<T, T, AT, 1>;
    case 2: return (const void *)k_edge_blocks<T, T, AT, 2>;
    case 3: return (const void *)k_edge_blocks<T, T, AT, 3>;
    case 4: return (const void *)k_edge_blocks<T, T, AT, 4>;
    case 5: return (const void *)k_edge_blocks<T, T, AT, 5>;
    case 6: return (const void *)k_edge_blocks<T, T, AT, 6>;
    case 7: return (const void *)k_edge_blocks<T, T, AT, 7>;
    case 8: return (const void *)k_edge_blocks<T, T, AT, 8>;
    default: return nullptr;
    }
}
static const void *eb_kernel(bool f64, bool ar64, int lw) {
    const int hi = (lw + 1) / 2;
    if (f64) return eb_kernel_t<double, double>(hi);
    return ar64 ? eb_kernel_t<float, double>(hi) : eb_kernel_t<float, float>(hi);
}

bool eb_plan(const Params &P, bool f64, bool ar64, EdgeBlocksLaunch *out) {
    *out = EdgeBlocksLaunch{};
    const int nt = (P.S * P.n + 15) / 16, ab = (f64 || ar64) ? 8 : 4;
    const void *k = eb_kernel(f64, ar64, P.lmax + 1);
    int best = 0;
    // the most resident waves per CU, then the larger chunk and row block
    for (int Q : {2, 1})
        for (int RB : {128, 64}) {
            const int nw = 2 * Q * nt;
            const size_t lds = 8 * eb_lds_doubles(P, Q, RB, ab);
            int nb = 0;
            if (nw > EB_MAX_WAVES || lds > (size_t)159 * 1024) continue;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k, 64 * nw, lds) != hipSuccess) continue;
            if (nb * nw > best) {
                best = nb * nw;
                *out = EdgeBlocksLaunch{Q, RB, 64 * nw, lds};
            }
        }
    return best > 0;
}

hipError_t launch_edge_blocks(const Params &P, const Rows &R, const void *pos, bool f64, bool ar64,
                              const EdgeBlocksLaunch &cfg, double degree, const void *c_scratch, void *jedge,
                              hipStream_t st) {
    if (R.nc <= 0) return hipSuccess;
    Params Pk = P;
    // Few centers: several workgroups per center, each some of its chunks, until
    // about four workgroups per CU (what stays resident) have work (64-water
    // cluster, n_max 4, l_max 4: 41 us with one workgroup per center, 24 with
    // three); more centers gain nothing and load their tables again.
    int ncu = 256, dev_id = 0;
    (void)hipGetDevice(&dev_id);
    (void)hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev_id);
    const int64_t want = (4 * (int64_t)ncu) / R.nc, chunks = (int64_t)std::ceil(degree / (4.0 * cfg.Q));
    int Q = cfg.Q, RB = cfg.RB, split = (int)std::max<int64_t>(1, std::min(want, chunks));
    // a launch has fewer than 2^32 threads: more centers take several
    const int64_t most = (int64_t)UINT32_MAX / cfg.threads;
    const size_t per = (f64 || ar64 ? 8 : 4) * 4 * (size_t)P.S * P.n * P.L; // scratch of a center
    for (int64_t c0 = 0; c0 < R.nc; c0 += most) {
        Rows Rk = R;
        Rk.nc = std::min(most, R.nc - c0);
        Rk.row_ptr += c0;
        Rk.c_base += c0;
        if (Rk.centers) Rk.centers += c0;
        const void *cs = (const char *)c_scratch + per * (size_t)c0;
        void *args[] = {&Pk, &Rk, &pos, &Q, &RB, &split, &cs, &jedge};
        const hipError_t e = hipLaunchKernel(eb_kernel(f64, ar64, P.lmax + 1), dim3((unsigned)(Rk.nc * split)),
                                             dim3(cfg.threads), args, cfg.lds, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t eb_set_lds_limit(int lim) {
    hipError_t e = hipSuccess;
    for (int v = 0; v < 3; ++v)
        for (int lw = 1; lw <= LMAX + 1; lw += 2)
            if (e == hipSuccess)
                e = hipFuncSetAttribute(eb_kernel(v == 2, v == 1, lw), hipFuncAttributeMaxDynamicSharedMemorySize, lim);
    return e;
}

} // namespace soap
