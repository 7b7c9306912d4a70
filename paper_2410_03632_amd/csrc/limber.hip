// Limber approximations (first order and extended) and the non-linear correction.
//
//   C_ij(l) = N_t(l) (pi/2) sum_a wchi_a f_t(k)/k^2 dP[l][a] / chi_a^2 E_ij(l, a),  k = (l+1/2)/chi_a
//   E = K_i K_j                                      (order 1)
//   E = K_i K_j - nu^-2 (A_i K_j + K_i A_j),  A = sqrt(chi) (chi^2/2 Kt'' + chi^3/6 Kt''')   (order 2)
// with Kt = K / sqrt(chi) and nu = l + 1/2 (Sec. 2.2; the sign of the correction is the one of
// the Bessel expansion, see the header).  dP = P - P_sub is the caller's spectrum (or the
// difference non-linear minus linear of Sec. 3.2) at the Limber points.  FP64 throughout.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "internal.h"

namespace blast {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

struct LimbSel {
    int n_out;
    int16_t idx[kMaxEll];
};

__device__ inline void pair_decode(int p, int ng, int ns, uint32_t types, int &t, int &i, int &j) {
    const int ngg = (types & BLAST_GG) ? ng * (ng + 1) / 2 : 0;
    const int ngs = (types & BLAST_GS) ? ng * ns : 0;
    int q;
    int n, base;
    if (p < ngg) {
        t = BLAST_GG, q = p, n = ng, base = 0;
    } else if (p < ngg + ngs) {
        t = BLAST_GS, q = p - ngg;
        i = q / ns;
        j = ng + q % ns;
        return;
    } else {
        t = BLAST_SS, q = p - ngg - ngs, n = ns, base = ng;
    }
    int r = 0;
    while (q >= n - r) {
        q -= n - r;
        ++r;
    }
    i = base + r;
    j = base + r + q;
}

// The chi sum on FP64 matrix cores.  f_t / k^2 is (chi^2 / nu^2)^(shear legs of the pair), a product
// over the two legs, so with K'_i = K_i (times chi^2 for a shear bin), A'_i likewise and
// u_l(a) = wchi_a dP / chi_a^2 every type is one matrix per multipole,
//   Z_ij(l) = sum_a u_l(a) (K'_i - 2 nu^-2 A'_i)(a) K'_j(a),
//   C_ij(l) = N_t(l) (pi/2) nu^(-2 shear legs) (Z_ij + Z_ji) / 2,
// which for order 1 (no A') is symmetric by itself.  v_mfma_f64_16x16x4_f64: M and N are the bins,
// K the chi nodes; a lane's A and B operands hold the same (bin, node), so one LDS read of (K', A')
// serves both and every multipole of the wave.  Work-group = (16 output multipoles, cosmology),
// 4 waves of 4 multipoles; the chi nodes go by in chunks of 64 staged in LDS (the stencil of A'
// is summed while staging: 5 multiply-adds, where a separate pass wrote and re-read a (K, A) table).
// At full 3x2pt (10 + 5 bins, 96 multipoles, 256 nodes), batch 256: 86 us a call, of which the 1.6e6 MFMAs
// of 64 cycles take 41 and the 132 MB of inputs and outputs would take 28; the form with one
// thread per pair took 452 us plus 15 for its table.  LDS and registers are held to 26 KB and 80
// so that all six work-groups a CU gets there are resident (four resident: 125 us with the
// divisions of u and the stencil loads done per entry instead of once per thread and chunk, 110 with six).
constexpr int kLimbEll = 16, kLimbChunk = 64;

template <typename PT, int NBT, int ORDER>
__global__ __launch_bounds__(256, NBT == 1 ? 6 : 2) void limber_kernel(const PT *__restrict__ P, const PT *__restrict__ Psub,
                                                     const double *__restrict__ Kchi, const double *__restrict__ chi,
                                                     const double *__restrict__ wchi, const double *__restrict__ pref,
                                                     const double *__restrict__ ell, const double *__restrict__ lima,
                                                     const int *__restrict__ fds, int slot_gg, int slot_gs,
                                                     int slot_ss, int n_chi, int n_ell, int ng, int ns, uint32_t types,
                                                     int npairs, LimbSel sel, int accumulate, double *__restrict__ C) {
    constexpr int LE = kLimbEll, CH = kLimbChunk, NBP = 16 * NBT, KST = NBP + 1, UST = CH + 1, EW = LE / 4;
    constexpr int LPP = NBT == 1 ? 8 : 4;  // multipoles whose Z sit in LDS at a time
    constexpr size_t kIn = (size_t)(2 * CH * KST + LE * UST) * 8, kOut = (size_t)LPP * NBP * KST * 8;
    __shared__ __align__(16) unsigned char lds[kIn > kOut ? kIn : kOut];
    constexpr int NPR = NBP * (NBP + 1) / 2;
    __shared__ uint8_t pt[NPR], pi[NPR], pj[NPR];  // pairs: type, i, j
    double *Ks = (double *)lds, *As = Ks + CH * KST, *us = As + CH * KST;  // [node][bin], [multipole][node]
    double *Zs = (double *)lds;                                            // [multipole][i][j]
    const int io0 = blockIdx.x * LE, beta = blockIdx.y;
    const int nio = min(LE, sel.n_out - io0);
    const int nbins = ng + ns;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
    for (int p = threadIdx.x; p < npairs; p += 256) {
        int t = 0, i = 0, j = 0;
        pair_decode(p, ng, ns, types, t, i, j);
        pt[p] = (uint8_t)t, pi[p] = (uint8_t)i, pj[p] = (uint8_t)j;
    }
    // the wave's multipoles: output positions io0 + 4 e + wv
    double m2nu2[EW];
#pragma unroll
    for (int e = 0; e < EW; ++e) {
        const double nu = ell[sel.idx[io0 + min(4 * e + wv, nio - 1)]] + 0.5;
        m2nu2[e] = -2.0 / (nu * nu);
    }
    d4 acc[EW][NBT][NBT];
#pragma unroll
    for (int e = 0; e < EW; ++e)
#pragma unroll
        for (int i = 0; i < NBT; ++i)
#pragma unroll
            for (int j = 0; j < NBT; ++j) acc[e][i][j] = d4{0, 0, 0, 0};
    for (int a0 = 0; a0 < n_chi; a0 += CH) {
        __syncthreads();
        // a thread stages one chi node: wave wv the multipoles and bins wv, wv + 4, ...
        const int a = a0 + lane, ac = min(a, n_chi - 1);
        const double x2 = chi[ac] * chi[ac], q = wchi[ac] / x2;
#pragma unroll
        for (int e = 0; e < EW; ++e) {
            const int el = 4 * e + wv;
            double v = 0.0;
            if (el < nio && a < n_chi) {
                const size_t o = ((size_t)beta * n_ell + sel.idx[io0 + el]) * n_chi + a;
                double d = (double)P[o];
                if (Psub) d -= (double)Psub[o];
                v = q * d;
            }
            us[el * UST + lane] = v;
        }
        double la[5];
        const int s0 = ORDER == 2 ? fds[ac] : 0;
#pragma unroll
        for (int h = 0; h < 5; ++h) la[h] = ORDER == 2 ? lima[(size_t)ac * 5 + h] : 0.0;
#pragma unroll
        for (int u = 0; u < NBP / 4; ++u) {
            const int bin = 4 * u + wv;
            const double *row = Kchi + ((size_t)beta * nbins + min(bin, nbins - 1)) * n_chi;
            const double f = bin < ng ? 1.0 : x2;
            double k = 0.0, av = 0.0;
            if (bin < nbins && a < n_chi) {
                k = row[a] * f;
                if constexpr (ORDER == 2) {
#pragma unroll
                    for (int h = 0; h < 5; ++h) av = fma(la[h], row[s0 + h], av);
                    av *= f;
                }
            }
            Ks[lane * KST + bin] = k;
            if constexpr (ORDER == 2) As[lane * KST + bin] = av;
        }
        __syncthreads();
#pragma unroll 2
        for (int s = 0; s < CH / 4; ++s) {
            const int al = 4 * s + lk;
            double kv[NBT], av[NBT];
#pragma unroll
            for (int i = 0; i < NBT; ++i) {
                kv[i] = Ks[al * KST + 16 * i + lr];
                av[i] = ORDER == 2 ? As[al * KST + 16 * i + lr] : 0.0;
            }
#pragma unroll
            for (int e = 0; e < EW; ++e) {
                const double u = us[(4 * e + wv) * UST + al];
#pragma unroll
                for (int i = 0; i < NBT; ++i) {
                    const double x = u * (ORDER == 2 ? fma(m2nu2[e], av[i], kv[i]) : kv[i]);
#pragma unroll
                    for (int j = 0; j < NBT; ++j)
                        acc[e][i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, kv[j], acc[e][i][j], 0, 0, 0);
                }
            }
        }
    }
    // out through LDS, LPP multipoles at a time, so that the multipoles of a pair go out together
#pragma unroll
    for (int e0 = 0; e0 < EW; e0 += LPP / 4) {
        __syncthreads();
#pragma unroll
        for (int e = e0; e < e0 + LPP / 4; ++e) {
            double *Z = Zs + (size_t)(4 * (e - e0) + wv) * NBP * KST;
#pragma unroll
            for (int i = 0; i < NBT; ++i)
#pragma unroll
                for (int j = 0; j < NBT; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) Z[(16 * i + lk + 4 * r) * KST + 16 * j + lr] = acc[e][i][j][r];
        }
        __syncthreads();
        for (int q = threadIdx.x; q < npairs * LPP; q += 256) {
            const int e = q % LPP, p = q / LPP, io = io0 + 4 * e0 + e;
            if (io >= io0 + nio) continue;
            const int t = pt[p], i = pi[p], j = pj[p], l = sel.idx[io];
            const double *Z = Zs + (size_t)e * NBP * KST;
            const double z = ORDER == 2 ? 0.5 * (Z[i * KST + j] + Z[j * KST + i]) : Z[i * KST + j];
            const double nu = ell[l] + 0.5, in2 = 1.0 / (nu * nu);
            const double g = t == BLAST_GG ? 1.0 : (t == BLAST_GS ? in2 : in2 * in2);
            const int slot = t == BLAST_GG ? slot_gg : (t == BLAST_GS ? slot_gs : slot_ss);
            const double v = pref[slot * n_ell + l] * (0.5 * M_PI) * g * z;
            double *o = C + ((size_t)beta * npairs + p) * sel.n_out + io;
            *o = accumulate ? *o + v : v;
        }
    }
}

int npairs_for(int ng, int ns, uint32_t types) {
    return ((types & BLAST_GG) ? ng * (ng + 1) / 2 : 0) + ((types & BLAST_GS) ? ng * ns : 0) +
           ((types & BLAST_SS) ? ns * (ns + 1) / 2 : 0);
}

}  // namespace

blast_status limber(blast_plan *p, const blast_limber_args *a, hipStream_t s) {
    if (a->batch < 1) return set_error("batch must be >= 1"), BLAST_E_INVALID;
    if (a->p_dtype != 0 && a->p_dtype != 1) return set_error("p_dtype must be 0 (FP64) or 1 (FP32)"), BLAST_E_INVALID;
    if (!a->P || !a->K_chi || !a->C) return set_error("P, K_chi and C are required"), BLAST_E_INVALID;
    if (a->order != 1 && a->order != 2) return set_error("order must be 1 or 2"), BLAST_E_INVALID;
    if (a->order == 2 && !p->d_lima)
        return set_error("the extended Limber approximation needs at least 5 chi nodes"), BLAST_E_INVALID;
    const int ng = a->n_g, ns = a->n_s, nbins = ng + ns;
    if (ng < 0 || ns < 0 || nbins < 1 || nbins > kMaxBins)
        return set_error("need n_g, n_s >= 0 and 1 <= n_g + n_s <= %d", kMaxBins), BLAST_E_INVALID;
    if (a->types == 0 || (a->types & ~p->types))
        return set_error("types 0x%x not a non-empty subset of the plan's 0x%x", a->types, p->types), BLAST_E_INVALID;
    const int npairs = npairs_for(ng, ns, a->types);
    if (npairs < 1) return set_error("no bin pairs for these types and bins"), BLAST_E_INVALID;
    LimbSel sel{};
    if (a->n_ell_out == 0) {
        sel.n_out = p->n_ell;
        for (int i = 0; i < p->n_ell; ++i) sel.idx[i] = (int16_t)i;
    } else {
        if (a->n_ell_out < 0 || a->n_ell_out > p->n_ell || !a->ell_idx)
            return set_error("bad n_ell_out / ell_idx"), BLAST_E_INVALID;
        sel.n_out = a->n_ell_out;
        for (int i = 0; i < a->n_ell_out; ++i) {
            const int v = a->ell_idx[i];
            if (v < 0 || v >= p->n_ell || (i && v <= a->ell_idx[i - 1]))
                return set_error("ell_idx must be increasing indices into the plan's ell"), BLAST_E_INVALID;
            sel.idx[i] = (int16_t)v;
        }
    }
    const dim3 grid((unsigned)((sel.n_out + kLimbEll - 1) / kLimbEll), (unsigned)a->batch);
    auto launch = [&](auto ptag, auto nbt, auto order) {
        using PT = decltype(ptag);
        hipLaunchKernelGGL((limber_kernel<PT, decltype(nbt)::value, decltype(order)::value>), grid, dim3(256), 0, s,
                           (const PT *)a->P, (const PT *)a->P_sub, a->K_chi, p->d_chi, p->d_wchi, p->d_pref, p->d_ell,
                           p->d_lima, p->d_fds, p->slot[0], p->slot[1], p->slot[2], p->n_chi, p->n_ell, ng, ns, a->types,
                           npairs, sel, a->accumulate, a->C);
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    auto by_order = [&](auto ptag, auto nbt) {
        if (a->order == 2) launch(ptag, nbt, I2());
        else launch(ptag, nbt, I1());
    };
    auto by_bins = [&](auto ptag) {
        if (nbins <= 16) by_order(ptag, I1());
        else by_order(ptag, I2());
    };
    if (a->p_dtype == 0) by_bins(double());
    else by_bins(float());
    BLAST_HIP_TRY(hipGetLastError());
    return BLAST_OK;
}

}  // namespace blast
