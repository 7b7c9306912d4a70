// Contraction and R-quadrature of small batches: the basis streamed once, w kept in registers.
//
//   w[row][beta]          = sum_n Ttilde[a, b][row][n] c[beta][a, b][n]      (FP64 / FP32 MFMA, per b)
//   Y[beta][row][a][bin] += wR_b K_bin(R_b chi_a) w[row][beta]                (VALU, per b)
//
// At these batches the basis is all the traffic (7.25 GB in FP64 at full 3x2pt against 25 MB of P per
// cosmology) and one 16-column MFMA tile holds every cosmology, so the work is to keep reads of the
// basis in flight.  A wave owns one 16-row tile of one chi_a and walks the R nodes with a ring of
// 16-byte loads in registers (or half of them, next to a second wave); waves of a work-group share only the
// c rows (LDS, double buffered, loaded two nodes ahead) and the kernel weights (LDS, a chunk of nodes at a
// time), with one barrier per node that waits for no load of the basis.
//
// Measured (one MI355X, reads alone reach 6.2 TB/s): full 3x2pt in FP64, batch 1, 1.20 ms for 7.28 GB
// (6.0 TB/s; the contraction with w in memory and its R-quadrature took 1.47 + 0.06), in FP32, batch 8,
// 0.60 ms for 3.75 GB (6.2 TB/s; 0.73 + 0.12 before); 64 x 32 points of 60 rows in FP64, batch 1, 19 us
// for 64 MB (45 + 22 before), where the chain of loads, one node after the other, counts and not the rate.
//
// BT columns of the MFMA tile are cosmologies (4, 8 or 16); the 16 / BT copies of each cosmology's w
// that the tile then holds take a share of the bins each, so a lane keeps Y for 4 rows x NBL bins.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace blast {
namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t U4 __attribute__((ext_vector_type(4)));
typedef double d2v __attribute__((ext_vector_type(2)));


// R nodes whose kernel weights sit in LDS together
template <typename T, int BT, int NBL>
constexpr int stream_chunk() {
    return BT * (NBL * 16 / BT) * (int)sizeof(T) >= 2048 ? 8 : 16;
}

// LDS accesses done, then the barrier alone: __syncthreads would also wait for the loads in flight
__device__ inline void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// NC: blocks of 32 columns (nc_pad / 32); BT cosmologies per tile; NBL bins per lane; NPU: nodes held by
// the ring.
// ONCE: one cosmology tile, so that a basis tile is read once.
// TWO: two accumulator chains, K slices 0, 2 and 1, 3 of every four, as contract_quad_kernel<FP32> sums them.
// The launch sums ranges sp0 .. sp0 + nsp - 1 of the nsplit ranges of R nodes, range sp0 + i at Y + i * ysplit;
// from sp0 > 0 (FP64) on top of what is there.
// SW waves share a row tile: each takes every SW-th R node of the range, their Y are added through LDS at the
// end (half as many steps where the grid leaves SIMDs idle; 2 waves per tile, FP64: 75 x 29 points of 69 rows,
// batch 3 with 20 bins, 53 -> 36 us).
template <typename T, int NC, int BT, int NBL, int NPU, bool TWO, bool ONCE, int SW, int W>
__global__ __launch_bounds__(64 * W, SW > 1 && NBL == 16 ? 1 : 2) void stream_kernel(
    const T *__restrict__ basis, const T *__restrict__ c, int cld, const double *__restrict__ Kchi2,
    const double *__restrict__ wR, int batch, int nbins, int n_chi, int n_R, int rows_pad, RowTiles tiles, int nct,
    int nsplit, int sp0, int nsp, int units, int ybs, size_t ysplit, T *__restrict__ Y, T *__restrict__ w_out) {
    constexpr bool F64 = sizeof(T) == 8;
    constexpr int TW = W / SW, VEC = 16 / (int)sizeof(T), L = 8 / VEC;  // loads per block of 32 columns
    constexpr int ncp = 32 * NC, CST = ncp + VEC, GPR = ncp / VEC;
    constexpr int NBT = NBL * 16 / BT, KST = NBT + VEC, CB = stream_chunk<T, BT, NBL>();
    constexpr int CPT = (SW * BT * GPR + 64 * W - 1) / (64 * W);  // 16-byte pieces of c per thread and step
    // (the c rows' place also takes the Y of one row that waves of a tile add up)
    constexpr int CSZ = SW * BT * CST, RSZ = SW > 1 ? (W - TW) * 64 * NBL : 0;
    __shared__ __align__(16) T Cs[2 * CSZ > RSZ ? 2 * CSZ : RSZ];
    __shared__ __align__(16) T Ks[CB * BT * KST];

    const int per = (units + 7) / 8;
    const int unit = (int)(blockIdx.x % 8) * per + (int)(blockIdx.x / 8);
    if (unit >= units) return;  // uniform over the work-group
    const int groups = (tiles.n + TW - 1) / TW;
    // the cosmology tiles of a row group next to each other (they read the same basis tiles), then the
    // row groups of a chi node (they read the same c rows)
    const int ct = unit % nct, grp = (unit / nct) % groups;
    const int sp = sp0 + (unit / (nct * groups)) % nsp, a = unit / (nct * groups * nsp);
    const int b0 = (int)((long)n_R * sp / nsplit), b1 = (int)((long)n_R * (sp + 1) / nsplit);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int lr = lane & 15, lk = lane >> 4;
    // waves past the last tile repeat it and store nothing: a wave that left the loop's loads out would
    // make the compiler wait for every load in flight where the two paths meet
    const int wt = grp * TW + w % TW, h = w / TW;  // tile, first node of the wave
    const bool active = wt < tiles.n;
    const int rt = tiles.tile(__builtin_amdgcn_readfirstlane(min(wt, tiles.n - 1)));
    const int col = lr % BT, beta = ct * BT + col, bin0 = (lr / BT) * NBL;
    const int nb = min(BT, batch - ct * BT);
    const size_t NP = (size_t)n_chi * n_R;

    // the wave's tile of node b0, piece p of the lane at + p * PST, node b at + (b - b0) * nst
    constexpr int PST = F64 ? 4 : 64;
    const size_t nst = (size_t)rows_pad * ncp / VEC;
    // (FP64: MFMA row lk + 4 r, which lane group lk holds in register r, is row 4 lk + r of the tile, so that a
    // lane's four w are neighbours as they are on FP32)
    const U4 *pa = (const U4 *)basis + ((size_t)a * n_R + b0) * nst +
                   (F64 ? (size_t)(16 * rt + 4 * (lr & 3) + (lr >> 2)) * GPR + lk : (size_t)rt * GPR * 16 + lane);
    U4 A[NPU][NC][L];
    auto load_A = [&](int nu, int j, int b) {
        const U4 *q = pa + (size_t)(min(b, b1 - 1) - b0) * nst;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            // non-temporal where an instruction takes whole lines that nobody reads again (FP32, tiled, one
            // cosmology tile: 596 us instead of 703 at full 3x2pt, batch 8); the tiles of a larger batch read them
            // one soon after the other (batch 17: 938 us instead of 1265), and the row-major FP64 loads take
            // half a line each, whose other half must still be there for the next (1204 instead of 1380 at
            // batch 1)
            if constexpr (F64 || !ONCE) A[nu][j][l] = q[(j * L + l) * PST];
            else A[nu][j][l] = __builtin_nontemporal_load(q + (j * L + l) * PST);
        }
    };
    // c rows: thread's pieces of node b (rows past the batch and pieces past cld repeat valid ones: the
    // columns they feed are not stored, the basis columns they meet are zero)
    const T *pc[CPT];
    int oc[CPT], hc[CPT];
#pragma unroll
    for (int i = 0; i < CPT; ++i) {
        const int q = min((int)threadIdx.x + i * 64 * W, SW * BT * GPR - 1);
        const int r = q / GPR, v = q % GPR;
        hc[i] = r / BT;
        pc[i] = c + ((size_t)(ct * BT + min(r % BT, nb - 1)) * NP + (size_t)a * n_R) * cld + min(v, cld / VEC - 1) * VEC;
        oc[i] = r * CST + v * VEC;
    }
    U4 cr[CPT];
    auto load_c = [&](int b) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) cr[i] = *(const U4 *)(pc[i] + (size_t)min(b + hc[i], b1 - 1) * cld);
    };
    auto store_c = [&](int buf) {
#pragma unroll
        for (int i = 0; i < CPT; ++i)
            if (CPT * 64 * W == SW * BT * GPR || (int)threadIdx.x + i * 64 * W < SW * BT * GPR)
                *(U4 *)(&Cs[buf * CSZ + oc[i]]) = cr[i];
    };

    T y[4][NBL];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int q = 0; q < NBL; ++q) y[r][q] = (T)0;

    // weights of nodes b .. b + nn - 1 into LDS
    auto stage_weights = [&](int b, int nn) {
        // KU loads in flight per thread (clamped addresses, values masked)
        constexpr int KN = CB * BT * NBT, KPT = (KN + 64 * W - 1) / (64 * W), KU = KPT < 8 ? KPT : (F64 && NBL == 16 ? 4 : 8);
#pragma unroll
        for (int q0 = 0; q0 < KPT; q0 += KU) {  // (past the last weight: the last again, not stored)
            double kv[KU];
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const int q = min((int)threadIdx.x + (q0 + u) * 64 * W, KN - 1);
                const int bb = min(q % CB, nn - 1), bin = min((q / CB) % NBT, nbins - 1), cc = min(q / (CB * NBT), nb - 1);
                kv[u] = Kchi2[((size_t)(ct * BT + cc) * nbins + bin) * NP + (size_t)a * n_R + b + bb];
            }
            double wv = wR[b + min((int)threadIdx.x % CB, nn - 1)];
            // (keeps the loads out of the mask's branch, whose other side would leave them in flight)
#pragma unroll
            for (int u = 0; u < KU; ++u) asm volatile("" : "+v"(kv[u]), "+v"(wv));
#pragma unroll
            for (int u = 0; u < KU; ++u) {
                const int q = (int)threadIdx.x + (q0 + u) * 64 * W;
                if (KN % (64 * W * KU) != 0 && q >= KN) break;
                const int bb = q % CB, bin = (q / CB) % NBT, cc = q / (CB * NBT);
                Ks[(bb * BT + cc) * KST + bin] = bb < nn && bin < nbins && cc < nb ? (T)(wv * kv[u]) : (T)0;
            }
        }
    };

    load_c(b0);
    stage_weights(b0, min(CB, b1 - b0));  // ahead of the ring, whose loads they would wait for
    store_c(0);
    load_c(b0 + SW);
#pragma unroll
    for (int nu = 0; nu < NPU; ++nu)
#pragma unroll
        for (int j = 0; j < NC; ++j) load_A(nu, j, b0 + nu * SW + h);

    auto node = [&](auto nuc, int bs) {  // nodes bs .. bs + SW - 1, one per wave of a tile
        constexpr int nu = decltype(nuc)::value;
        const int i = (bs - b0) / SW, b = bs + h;
        lds_barrier();  // c(b) and the weights are in LDS; the last step's readers are done with the other buffer
        store_c((i + 1) & 1);
        load_c(bs + 2 * SW);
        __builtin_amdgcn_sched_barrier(0);
        const T *cs = &Cs[(i & 1) * CSZ + (h * BT + col) * CST + lk * VEC];
        using Acc = typename std::conditional<F64, d4, f4>::type;
        Acc acc = Acc{0, 0, 0, 0}, acc2 = Acc{0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            U4 cv[L];
#pragma unroll
            for (int l = 0; l < L; ++l) cv[l] = *(const U4 *)(cs + (j * L + l) * 4 * VEC);
#pragma unroll
            for (int l = 0; l < L; ++l) {
                if constexpr (F64) {
                    const d2v x = __builtin_bit_cast(d2v, A[nu][j][l]), z = __builtin_bit_cast(d2v, cv[l]);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[0], z[0], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[1], z[1], acc, 0, 0, 0);
                } else {
                    const f4 x = __builtin_bit_cast(f4, A[nu][j][l]), z = __builtin_bit_cast(f4, cv[l]);
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        Acc &to = TWO && (u & 1) ? acc2 : acc;
                        to = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u], z[u], to, 0, 0, 0);
                    }
                }
            }
            load_A(nu, j, b + NPU * SW);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (TWO) acc = acc + acc2;
        const bool in = SW == 1 || b < b1;  // (uniform) past the range: the last node again, which adds nothing
        if constexpr (SW > 1)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = in ? acc[r] : (T)0;
        // a lane holds w of rows 4 lk + r of the tile for its cosmology
        if (w_out && active && in && lr < BT && beta < batch) {
            T *wo = w_out + ((size_t)beta * NP + (size_t)a * n_R + b) * rows_pad + 16 * rt + 4 * lk;
            if constexpr (F64) {
                *(double2 *)wo = make_double2(acc[0], acc[1]);
                *(double2 *)(wo + 2) = make_double2(acc[2], acc[3]);
            } else {
                *(float4 *)wo = make_float4(acc[0], acc[1], acc[2], acc[3]);
            }
        }
        const T *ks = &Ks[(((b - b0) % CB) * BT + col) * KST + bin0];
#pragma unroll
        for (int q0 = 0; q0 < NBL; q0 += VEC) {
            const U4 kk = *(const U4 *)(ks + q0);
            const T *k = (const T *)&kk;
#pragma unroll
            for (int q = 0; q < VEC; ++q)
#pragma unroll
                for (int r = 0; r < 4; ++r) y[r][q0 + q] = fma(acc[r], k[q], y[r][q0 + q]);
        }
    };
    static_assert(CB % (NPU * SW) == 0, "whole rings per weights chunk");
    for (int bc = b0; bc < b1; bc += CB) {
        const int be = min(bc + CB, b1);
        if (bc > b0) {
            lds_barrier();  // the previous chunk's readers are done
            stage_weights(bc, be - bc);
        }
        int b = bc;  // whole rings, then the last steps of the range
        for (; b + (NPU - 1) * SW < be; b += NPU * SW) {
            node(std::integral_constant<int, 0>(), b);
            if constexpr (NPU > 1) node(std::integral_constant<int, 1>(), b + SW);
            if constexpr (NPU > 2) node(std::integral_constant<int, 2>(), b + 2 * SW);
            if constexpr (NPU > 3) node(std::integral_constant<int, 3>(), b + 3 * SW);
        }
        if constexpr (NPU > 1)
            if (b < be) node(std::integral_constant<int, 0>(), b);
        if constexpr (NPU > 2) {
            if (b + SW < be) node(std::integral_constant<int, 1>(), b + SW);
            if (b + 2 * SW < be) node(std::integral_constant<int, 2>(), b + 2 * SW);
        }
    }
    if constexpr (SW > 1) {
        // the tile's waves add up in the order of their first nodes, one row at a time
        T *red = Cs + ((size_t)(w % TW) * 64 + lane) * NBL;  // wave h of tile t at + ((h - 1) * TW + t) * 64 * NBL
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            lds_barrier();  // the readers of what lay here are done
            if (h > 0)
#pragma unroll
                for (int q = 0; q < NBL; ++q) red[(size_t)(h - 1) * TW * 64 * NBL + q] = y[r][q];
            lds_barrier();
            if (h == 0)
#pragma unroll
                for (int o = 0; o < SW - 1; ++o)
#pragma unroll
                    for (int q = 0; q < NBL; ++q) y[r][q] += red[(size_t)o * TW * 64 * NBL + q];
        }
        if (h > 0) return;
    }
    if (!active || beta >= batch) return;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * rt + 4 * lk + r;
        T *yp = Y + (size_t)(sp - sp0) * ysplit + (((size_t)beta * rows_pad + row) * n_chi + a) * ybs + bin0;
#pragma unroll
        for (int q0 = 0; q0 < NBL; q0 += VEC) {
            if (bin0 + q0 >= ybs) continue;
            U4 o;
            T *op = (T *)&o;
#pragma unroll
            for (int q = 0; q < VEC; ++q) op[q] = y[r][q0 + q];
            if constexpr (F64)
                if (sp0 > 0) {  // ranges one launch after the other: on top of the earlier ones' sum
                    const U4 old = *(const U4 *)(yp + q0);
                    o = __builtin_bit_cast(U4, __builtin_bit_cast(d2v, old) + __builtin_bit_cast(d2v, o));
                }
            *(U4 *)(yp + q0) = o;
        }
    }
}

template <typename T>
void launch(const StreamCall &k, hipStream_t s) {
    const blast_plan *p = k.plan;
    auto go4 = [&](auto nct_, auto btt, auto nblt, auto nput, auto twot, auto oncet, auto swt, auto wt) {
        constexpr int NC = decltype(nct_)::value, BT = decltype(btt)::value, NBL = decltype(nblt)::value;
        constexpr int NPU = decltype(nput)::value, SW = decltype(swt)::value, W = decltype(wt)::value, TW = W / SW;
        const int nct = (k.batch + BT - 1) / BT, groups = (k.tiles.n + TW - 1) / TW;
        const int nsp = k.apart ? k.nsplit : 1, units = p->n_chi * nsp * groups * nct;
        for (int sp0 = 0; sp0 < k.nsplit; sp0 += nsp)
            hipLaunchKernelGGL((stream_kernel<T, NC, BT, NBL, NPU, decltype(twot)::value, decltype(oncet)::value, SW, W>),
                               dim3((unsigned)((units + 7) / 8 * 8)), dim3(64 * W), 0, s, (const T *)k.basis,
                               (const T *)k.c, k.cld, k.K_chi2, p->d_wR, k.batch, k.nbins, p->n_chi, p->n_R,
                               p->rows_pad, k.tiles, nct, k.nsplit, sp0, nsp, units, k.ybs, k.ysplit, (T *)k.Y,
                               (T *)k.w_out);
    };
    auto go3 = [&](auto nct_, auto btt, auto nblt, auto nput, auto twot, auto oncet, auto swt) {
        using std::integral_constant;
        if constexpr (sizeof(T) == 4) {
            constexpr int BT = decltype(btt)::value;
            const int g = p->n_chi * ((k.batch + BT - 1) / BT), w4 = g * ((k.tiles.n + 3) / 4), w6 = g * ((k.tiles.n + 5) / 6);
            // 6 waves per work-group where that saves the busiest CU a work-group (results unchanged): 75 chi nodes,
            // 5 row tiles, 37 cosmologies 53.1 -> 46.5 us, 31 cosmologies of 128 nodes 58.7 -> 49.6; from three
            // work-groups per CU on the same or slower (540 of 12 tiles: 107.0 -> 107.9)
            if (w4 <= 512 && (w6 + 255) / 256 < (w4 + 255) / 256)
                return go4(nct_, btt, nblt, nput, twot, oncet, swt, integral_constant<int, 6>());
        }
        go4(nct_, btt, nblt, nput, twot, oncet, swt, integral_constant<int, 4>());
    };
    auto go2 = [&](auto nct_, auto btt, auto nblt, auto nput, auto twot, auto oncet) {
        using std::integral_constant;
        if constexpr (sizeof(T) == 8)
            if (k.node_waves == 2) return go3(nct_, btt, nblt, nput, twot, oncet, integral_constant<int, 2>());
        go3(nct_, btt, nblt, nput, twot, oncet, integral_constant<int, 1>());
    };
    // (only batches past the fused kernels' smallest take their two chains, and only batches past a tile more
    // than one: the widest tiles)
    auto go = [&](auto nct_, auto btt, auto nblt, auto nput) {
        if constexpr (sizeof(T) == 4 && decltype(nblt)::value == 16) {
            if (k.two_chains) return go2(nct_, btt, nblt, nput, std::true_type(), std::false_type());
            if (k.batch > decltype(btt)::value) return go2(nct_, btt, nblt, nput, std::false_type(), std::false_type());
        }
        go2(nct_, btt, nblt, nput, std::false_type(), std::true_type());
    };
    // rings as deep as the registers hold next to Y (256 per lane at two waves per SIMD)
    constexpr bool F64 = sizeof(T) == 8;
    auto by_shape = [&](auto nct_) {
        constexpr int NC = decltype(nct_)::value;
        using std::integral_constant;
        constexpr int R4 = NC <= 2 ? 4 : 2;                            // 4 cosmologies, 4 bins a lane
        constexpr int R8 = F64 ? (NC == 1 ? 4 : (NC == 4 ? 1 : 2)) : R4;  // 8 bins a lane
        constexpr int R16 = F64 ? (NC == 1 ? 2 : 1) : (NC == 1 ? 4 : 2);  // 16 bins a lane
        using B4 = integral_constant<int, 4>;
        using B8 = integral_constant<int, 8>;
        using B16 = integral_constant<int, 16>;
        const int bt = stream_tile(k.batch, k.nbins);
        if (bt == 4 && k.nbins <= 16) go(nct_, B4(), B4(), integral_constant<int, R4>());
        else if (bt == 4) go(nct_, B4(), B8(), integral_constant<int, R8>());
        else if (bt == 8 && k.nbins <= 16) go(nct_, B8(), B8(), integral_constant<int, R8>());
        else if (bt == 16) go(nct_, B16(), B16(), integral_constant<int, R16>());
        else go(nct_, B8(), B16(), integral_constant<int, R16>());
    };
    switch (p->nc_pad / 32) {
        case 1: by_shape(std::integral_constant<int, 1>()); break;
        case 2: by_shape(std::integral_constant<int, 2>()); break;
        case 3: by_shape(std::integral_constant<int, 3>()); break;
        default: by_shape(std::integral_constant<int, 4>()); break;
    }
}

}  // namespace

void stream_contract_quad(const StreamCall &k, bool f64, hipStream_t s) {
    if (f64) launch<double>(k, s);
    else launch<float>(k, s);
}

}  // namespace blast
