// Direction-split hop kernel: the fused hop of tm_hop.inc.h with a wave per hop.
//
// A block of eight waves computes 64 sites; wave d does hop d of all of them
// (d = 2 mu + (backward)), so the eight phases (load link and neighbour, wait,
// multiply) that one thread per site runs one after the other run side by
// side, in a quarter of the registers.  The waves leave their link products g
// (six complex per flavour) in LDS; the epilogue gives each thread the pair of
// elements (k, k + 6) the twist couples, for all flavours, and adds the eight
// products in the order of the one-thread kernel with the same operations, so
// both round alike.  Several right-hand sides: the block keeps its links in
// registers and walks pb.nrg right-hand sides, the next neighbours in flight
// during an epilogue (two LDS buffers, one barrier per right-hand side).
#pragma once

#include "tm_hop.inc.h"

namespace twm {

// Flavours per thread.  FP64 doublets put the two flavours of 32 sites into the
// halves of a wave (both load the same link), so a block takes the LDS (52 KiB)
// and the registers of the one-flavour kernel and two blocks share a compute
// unit where one did: R^-1 D of 12^3 x 24 in a solve 9.5 us against 13.2 with
// both flavours of 64 sites in a thread, 24^3 x 48 126 against 139.  In FP32,
// where two blocks fit either way, that costs more addresses and links per
// block than it gives (20^3 x 40 30 against 28, 12^3 x 24 6.0 against 6.9),
// half precision gains nothing where this kernel is used, and the twist on load
// needs both flavours of all twelve elements.
template <int P, int NF, bool TWL>
constexpr int split_nl()
{
    return split_sites(P, NF, TWL) < kSplitSites ? 1 : NF;
}

// The value of the lane 32 away (the other flavour of the site).
__device__ __forceinline__ uint32_t other_half(uint32_t a)
{
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    return (threadIdx.x & 32) ? r[0] : r[1];
}
__device__ __forceinline__ float other_half(float a) { return __uint_as_float(other_half(__float_as_uint(a))); }
__device__ __forceinline__ double other_half(double a)
{
    const uint32_t lo = other_half((uint32_t)__double2loint(a)), hi = other_half((uint32_t)__double2hiint(a));
    return __hiloint2double((int)hi, (int)lo);
}

// One LDS buffer: link products, hop factors (with the site scale in half
// precision, where each flavour has its own), the element maxima of the
// half-precision store and the reduction.
template <int P, int NF, bool TWL, bool RES>
struct SplitLds {
    using real = typename Prec<P>::real;
    static constexpr bool SC = Prec<P>::kScaled;
    static constexpr bool MX = SC || RES;        // a true residual may be rounded to half precision
    static constexpr int NL = split_nl<P, NF, TWL>();
    static constexpr int kFac = SC ? NL : 1;
    cx<real> g[8][NL][6][kSplitSites];
    real fac[8][kFac][kSplitSites];
    float mx[MX ? NL : 1][MX ? 6 : 1][MX ? kSplitSites : 1];
    double red[kSplitThreads / 64];
};

// Waves per SIMD the register allocation is held to (a block is two).
template <int P, int NF, bool TWL>
constexpr int split_waves()
{
    return P == TM_FP64 && (split_nl<P, NF, TWL>() == 2 || TWL) ? 2 : 4;
}
// Several rhs: two LDS buffers where they leave room for two blocks per
// compute unit (FP64's take 52 KiB each), else one and a second barrier per
// rhs.
template <int P>
constexpr bool split_two_buffers()
{
    return P != TM_FP64;
}

// Vector (rhs, flavour) of the flavour f a lane holds.
template <int P, int NF, bool TWL>
__device__ __forceinline__ uint32_t split_vec(int rhs, int f, int lane)
{
    return (uint32_t)(rhs * NF) + (uint32_t)(split_nl<P, NF, TWL>() == NF ? f : lane >> 5);
}

// One hop (direction MU, forward or backward) of one site and rhs for all
// flavours: its link products and factors to LDS.  The link comes in u with
// several rhs, and is loaded next to the neighbours otherwise.
template <int P, int NF, bool DAG, bool TWL, int RECON, bool LNT, bool MR, bool RES, int MU, bool FWD>
__device__ __forceinline__ void split_hop(SplitLds<P, NF, TWL, RES> &sh, cx<typename Prec<P>::real> (&u)[3][3],
                                          const HopProblem &pb, uint32_t nb, uint32_t cb, int rhs,
                                          typename Prec<P>::real sgn, int lane)
{
    using real = typename Prec<P>::real;
    constexpr int NL = split_nl<P, NF, TWL>();
    constexpr int SIG = (FWD != DAG) ? 1 : -1;   // D: 1 - g forward; D^+ swaps
    constexpr int D = 2 * MU + (FWD ? 0 : 1);
    constexpr bool WORDS = P == TM_FP16 && !TWL;
    constexpr int K0 = (!TWL && MU == 3 && SIG > 0) ? 6 : 0, N = (!TWL && MU == 3) ? 6 : 12;
    const uint32_t vh = pb.vh;
    [[maybe_unused]] cx<real> v[NL][12];
    [[maybe_unused]] uint32_t w[NL][12];
    real sc[NL];
#pragma unroll
    for (int f = 0; f < NL; f++) {
        const uint32_t vec = split_vec<P, NF, TWL>(rhs, f, lane);
        if constexpr (TWL) {
            SpinorIO<P>::template load<0, 12>(v[f], pb.in, vh, vec, nb);
            sc[f] = (real)1;
        } else if constexpr (WORDS) {
            SpinorIO<P>::template load_words<K0, N>(w[f], pb.in, vh, vec, nb, sc[f]);
        } else {
            SpinorIO<P>::template load_unscaled<K0, N>(v[f], pb.in, vh, vec, nb, sc[f]);
        }
    }
    if constexpr (!MR)
        LinkIO<P, RECON, LNT>::load(u, pb.gauge[FWD ? pb.out_parity : 1 - pb.out_parity], vh, MU, FWD ? cb : nb);
    if constexpr (TWL) apply_twist<real, NF>(v, pb.tw, true);
#pragma unroll
    for (int f = 0; f < NL; f++) {
        cx<real> g[2][3];
        if constexpr (WORDS) {
            f16x2 u2[3][3], hp[2][3], hs[2][3];
            link_pairs(u2, u);
            project_pairs<MU, SIG, !FWD>(hp, hs, w[f]);
#pragma unroll
            for (int c = 0; c < 3; c++) {
                g[0][c] = link_row_pairs<!FWD>(u2, hp[0], hs[0], c);
                g[1][c] = link_row_pairs<!FWD>(u2, hp[1], hs[1], c);
            }
        } else {
            cx<real> h[2][3];
            project<MU, SIG>(h, v[f] + ((TWL && MU == 3 && SIG > 0) ? 6 : 0));
#pragma unroll
            for (int c = 0; c < 3; c++) {
                g[0][c] = link_row<!FWD>(u, h[0], c);
                g[1][c] = link_row<!FWD>(u, h[1], c);
            }
        }
#pragma unroll
        for (int c = 0; c < 3; c++) {
            sh.g[D][f][c][lane] = g[0][c];
            sh.g[D][f][3 + c][lane] = g[1][c];
        }
        if (f < SplitLds<P, NF, TWL, RES>::kFac) sh.fac[D][f][lane] = ((MU == 3) ? (real)2 : (real)1) * (sgn * sc[f]);
    }
}

// Element k of vector vec at site cb.
template <int P, bool NT>
__device__ __forceinline__ cx<typename Prec<P>::real> load_elem(const SpinorPtr &s, uint32_t vh, uint32_t vec,
                                                                uint32_t cb, int k)
{
    if constexpr (P == TM_FP64) {
        const double2 c = lds_<NT>(at<double2>(SpinorIO<P>::row(s, vh, vec, k), cb * 16u));
        return mk(c.x, c.y);
    } else if constexpr (P == TM_FP32) {
        const float2 c = lds_<NT>(at<float2>(SpinorIO<P>::row(s, vh, vec, k >> 1), cb * 16u + (k & 1) * 8u));
        return mk(c.x, c.y);
    } else {
        const float sc = *at<float>(s.scale + (size_t)vec * vh, cb * 4u);
        const uint32_t c = lds_<NT>(at<uint32_t>(SpinorIO<P>::row(s, vh, vec, k >> 2), cb * 16u + (k & 3) * 4u));
        return mk(sc * half_to_f<P>(c & 0xffff), sc * half_to_f<P>(c >> 16));
    }
}
template <int P, bool NT>
__device__ __forceinline__ void store_elem(const SpinorPtr &s, uint32_t vh, uint32_t vec, uint32_t cb, int k,
                                           cx<typename Prec<P>::real> a, float inv)
{
    if constexpr (P == TM_FP64)
        sts_<NT>(at_w<double2>((void *)SpinorIO<P>::row(s, vh, vec, k), cb * 16u), make_double2(a.re, a.im));
    else if constexpr (P == TM_FP32)
        sts_<NT>(at_w<float2>((void *)SpinorIO<P>::row(s, vh, vec, k >> 1), cb * 16u + (k & 1) * 8u),
                 make_float2(a.re, a.im));
    else
        sts_<NT>(at_w<uint32_t>((void *)SpinorIO<P>::row(s, vh, vec, k >> 2), cb * 16u + (k & 3) * 4u),
                 SpinorIO<P>::pack1(a, inv));
}

// (lo, hi) <- R (lo, hi) or R^-1 (lo, hi) of the element pairs (k, k + 6)
template <typename T, int NF, int NL>
__device__ __forceinline__ void twist_pair(cx<T> (&v)[NL][2], const Twist &tw, bool inverse, int lane)
{
    const T ta = (T)tw.ta, b = (T)tw.b;
    const T s = inverse ? (T)-1 : (T)1;
    const T c = inverse ? (T)tw.c : (T)1;
    cx<T> o[NL][2];
#pragma unroll
    for (int f = 0; f < NL; f++) {
        const T t3 = (NL == NF ? f == 0 : lane < 32) ? ta : -ta;
#pragma unroll
        for (int e = 0; e < 2; e++) {
            cx<T> r = v[f][e] + (s * t3) * times_i(v[f][1 - e]);
            if constexpr (NL == 2) r = r + (s * b) * v[1 - f][e];
            if constexpr (NL < NF) r = r + (s * b) * mk(other_half(v[f][e].re), other_half(v[f][e].im));
            o[f][e] = c * r;
        }
    }
#pragma unroll
    for (int f = 0; f < NL; f++)
#pragma unroll
        for (int e = 0; e < 2; e++) v[f][e] = o[f][e];
}

// Partials that the last block of the same launch reads: exchanged and loaded
// at device scope (the L2 of each XCD would keep plain stores to itself), the
// exchange's result awaited before the block counts itself.  No cache
// write-back is needed, as a fence would do.
__device__ __forceinline__ void partial_put(double *p, double s)
{
    unsigned long long old = __hip_atomic_exchange((unsigned long long *)p, (unsigned long long)__double_as_longlong(s),
                                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __asm__ volatile("" : "+v"(old)::"memory");
}

// The reductions of a launch by its last block, in place of the finish launch.
// The blocks count themselves in groups of up to 64, the last of each group
// among the groups, so that no address takes more than 64 atomics; a wave or
// several add the partials of a vector, four loads of a lane in flight.
__device__ __forceinline__ void split_finish(const HopBatch &B)
{
    __shared__ int last;
    __shared__ double sums[8];
    if (threadIdx.x == 0) {
        CGFlags &f = *B.post.flags;
        const int ng = (B.total_blocks + kFinishGroup - 1) / kFinishGroup;
        const int g = ng == 1 ? 0 : (int)blockIdx.x % ng;
        const int size = ng == 1 ? B.total_blocks : B.total_blocks / ng + (g < B.total_blocks % ng);
        int *const done = &f.done_grp[g].n;
        last = 0;
        if (__hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == size - 1) {
            *done = 0;
            last = ng == 1 || __hip_atomic_fetch_add(&f.done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == ng - 1;
            if (last) f.done = 0;
        }
    }
    __syncthreads();
    if (!last) return;
    const int wave = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    int nv = 0;
    for (int i = 0; i < B.nprob; i++) nv += B.p[i].red.nvec;
    // waves per vector
    const int wpv = B.total_blocks <= kFinishGroup || nv > 4 ? 1 : nv > 2 ? 2 : nv == 2 ? 4 : 8;
    const int sub = wave % wpv;
    for (int k0 = 0; k0 < nv; k0 += 8 / wpv) {
        int i = 0, v = k0 + wave / wpv;
        while (i < B.nprob && v >= B.p[i].red.nvec) v -= B.p[i++].red.nvec;
        double s = 0.0;
        if (i < B.nprob) {
            const Reduce &rd = B.p[i].red;
            for (int b0 = sub * 64 + lane; b0 < rd.nblk; b0 += wpv * 256) {
                double a[4];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int b = b0 + j * wpv * 64;
                    a[j] = b < rd.nblk ? __longlong_as_double((long long)__hip_atomic_load(
                                             (unsigned long long *)&rd.partials[(long)v * rd.nblk + b],
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                                       : 0.0;
                }
                s += (a[0] + a[1]) + (a[2] + a[3]);
            }
        }
        s = wave_sum(s);
        if (wpv > 1) {   // one pass
            if (lane == 0) sums[wave] = s;
            __syncthreads();
            for (int w = 1; w < wpv && sub == 0; w++) s += sums[wave + w];
        }
        if (lane == 0 && sub == 0 && i < B.nprob) finish_apply(B.p[i].red, v, s);
    }
    __syncthreads();
    if (B.p[0].red.op == FIN_BETA || B.p[0].red.op == FIN_RELIABLE)
        cg_post(B.post, B.nprob, [&](int i) -> const Reduce & { return B.p[i].red; });
}

// MR: pb.nrg right-hand sides per block (else one).  RES (FP64): the result
// becomes the true residual pb.res - A, rounded to precision B.res_prec on its
// way out; the norm is that of the FP64 values.
template <int P, int NF, bool DAG, bool TWL, int RECON, bool LNT, bool MR, bool RES = false>
__global__ void __launch_bounds__(kSplitThreads, (split_waves<P, NF, TWL>())) hop_split_kernel(const HopBatch B)
{
    using real = typename Prec<P>::real;
    using Lds = SplitLds<P, NF, TWL, RES>;
    constexpr int NL = Lds::NL, NS = split_sites(P, NF, TWL);
    extern __shared__ __align__(16) unsigned char split_sh[];
    Lds *const shb = reinterpret_cast<Lds *>(split_sh);
    if (gated_off(B)) return;   // gated launch not needed this iteration

    const int lb = B.xcd_remap ? xcd_logical_block(blockIdx.x, B.total_blocks) : (int)blockIdx.x;
    int pi = 0;
    for (int i = 1; i < B.nprob; i++)
        if (lb >= B.p[i].blk_start) pi = i;
    const HopProblem &pb = B.p[pi];
    const int lbl = lb - pb.blk_start;
    const int sb = lbl / pb.ngrp;
    const int r0 = (lbl - sb * pb.ngrp) * pb.nrg;
    const int r1 = MR ? min(pb.nrhs, r0 + pb.nrg) : r0 + 1;
    const uint32_t vh = pb.vh;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = (int)(threadIdx.x & 63);
    const int nts = B.nt_streams;

    // the hop of this wave: neighbour, link (U, or U^+ for a backward hop) and factor
    const int mu = wave >> 1;
    const bool fwd = (wave & 1) == 0;
    const uint32_t jl = (uint32_t)sb * NS + (lane & (NS - 1));
    const bool valid = jl < vh;
    uint32_t nb = 0, cl = 0;
    real sgn = (real)1;
    cx<real> u[3][3];
    if (valid) {
        const uint32_t cb = cl = site_of(pb, jl);
        const uint32_t xh_n = (uint32_t)pb.X[0] >> 1;
        const uint32_t q0 = pb.dx.div(cb), q1 = pb.dy.div(q0), t = pb.dz.div(q1);
        const uint32_t xh = cb - q0 * xh_n, y = q0 - q1 * pb.X[1], z = q1 - t * pb.X[2];
        const int par = pb.out_parity;
        if (mu == 0) {
            // x = 2 xh + o: the neighbour's xh is the site's own in one direction
            const uint32_t o = (y + z + t + par) & 1;
            nb = cb - xh + (fwd ? (o ? (xh + 1 == xh_n ? 0 : xh + 1) : xh) : (o ? xh : (xh == 0 ? xh_n - 1 : xh - 1)));
        } else {
            const uint32_t c = mu == 1 ? y : mu == 2 ? z : t, L = (uint32_t)pb.X[mu];
            const uint32_t s = mu == 1 ? xh_n : mu == 2 ? xh_n * pb.X[1] : xh_n * pb.X[1] * pb.X[2];
            const bool edge = fwd ? c == L - 1 : c == 0;
            nb = fwd ? (edge ? cb - (L - 1) * s : cb + s) : (edge ? cb + (L - 1) * s : cb - s);
            if (mu == 3 && edge) sgn = (real)pb.tsign;
        }
        if constexpr (MR) LinkIO<P, RECON, LNT>::load(u, pb.gauge[fwd ? par : 1 - par], vh, mu, fwd ? cb : nb);
    }

    // the epilogue's elements: thread (site, k) holds k and k + 6 of every
    // flavour.  FP32 chunks hold two elements, so neighbouring lanes take the
    // two of a chunk and a wave's stores stay contiguous.
    int k, site;
    if constexpr (P == TM_FP32) {
        static_assert(NL == NF, "the flavours of a wave's halves come by whole elements");
        k = (int)(threadIdx.x >> 7) * 2 + (int)(threadIdx.x & 1);
        site = (int)(threadIdx.x & 127) >> 1;
    } else {
        k = wave;
        site = lane;
    }
    const uint32_t je = (uint32_t)sb * NS + (site & (NS - 1));
    const bool act = k < 6 && je < vh;
    const uint32_t cb = act ? site_of(pb, je) : 0;
    const int s = k >= 3, c = k - 3 * s;

    int r = r0;
    do {
        Lds &sh = shb[MR && split_two_buffers<P>() ? (r - r0) & 1 : 0];
        if constexpr (MR && !split_two_buffers<P>()) __syncthreads();
        if (valid) {
#define TM_SPLIT_HOP(MU, FWD) \
    split_hop<P, NF, DAG, TWL, RECON, LNT, MR, RES, MU, FWD>(sh, u, pb, nb, cl, r, sgn, lane)
            switch (wave) {
            case 0: TM_SPLIT_HOP(0, true); break;
            case 1: TM_SPLIT_HOP(0, false); break;
            case 2: TM_SPLIT_HOP(1, true); break;
            case 3: TM_SPLIT_HOP(1, false); break;
            case 4: TM_SPLIT_HOP(2, true); break;
            case 5: TM_SPLIT_HOP(2, false); break;
            case 6: TM_SPLIT_HOP(3, true); break;
            default: TM_SPLIT_HOP(3, false); break;
            }
#undef TM_SPLIT_HOP
        }
        __syncthreads();

        double nrm = 0.0;
        cx<real> A[NL][2];
        if (act) {
#pragma unroll
            for (int f = 0; f < NL; f++) {
                cx<real> lo = mk((real)0, (real)0), hi = mk((real)0, (real)0);
#pragma unroll
                for (int d = 0; d < 8; d++) {
                    const int m = d >> 1;
                    const bool pl = ((d & 1) == 0) != DAG;
                    const cx<real> gs = sh.g[d][f][k][site];
                    const real fc = sh.fac[d][f < Lds::kFac ? f : 0][site];
                    if (m == 3) {
                        if (pl)
                            acc_k<0>(hi, fc, gs);
                        else
                            acc_k<0>(lo, fc, gs);
                        continue;
                    }
                    acc_k<0>(lo, fc, gs);
                    // lower pair +- i s_m g: (i g1, i g0), (g1, -g0), (i g0, -i g1)
                    const cx<real> gh = m == 2 ? gs : sh.g[d][f][3 * (1 - s) + c][site];
                    const real sg = pl ? fc : -fc;
                    const real sf = s ? -sg : sg;
                    if (m == 0)
                        acc_k<2>(hi, sg, gh);
                    else if (m == 1)
                        acc_k<0>(hi, sf, gh);
                    else
                        acc_k<2>(hi, sf, gh);
                }
                A[f][0] = lo;
                A[f][1] = hi;
            }
            const int epi = B.epi;
            const real kk = (real)pb.k;
            if (epi == TM_EPI_TWINV || epi == TM_EPI_X_PLUS_K_TWINV_D) twist_pair<real, NF>(A, pb.tw, true, lane);
            if (epi >= TM_EPI_RX_PLUS_KD) {
                cx<real> X[NL][2];
#pragma unroll
                for (int f = 0; f < NL; f++)
#pragma unroll
                    for (int e = 0; e < 2; e++)
                        X[f][e] = (nts & kNtX) ? load_elem<P, true>(pb.x, vh, split_vec<P, NF, TWL>(r, f, lane), cb, k + 6 * e)
                                               : load_elem<P, false>(pb.x, vh, split_vec<P, NF, TWL>(r, f, lane), cb, k + 6 * e);
                if (epi == TM_EPI_RX_PLUS_KD) twist_pair<real, NF>(X, pb.tw, false, lane);
#pragma unroll
                for (int f = 0; f < NL; f++)
#pragma unroll
                    for (int e = 0; e < 2; e++) A[f][e] = X[f][e] + kk * A[f][e];
                if (epi == TM_EPI_TWINV_X_PLUS_KD) twist_pair<real, NF>(A, pb.tw, true, lane);
            }
            if constexpr (RES) {
#pragma unroll
                for (int f = 0; f < NL; f++)
#pragma unroll
                    for (int e = 0; e < 2; e++)
                        A[f][e] = load_elem<P, true>(pb.res, vh, split_vec<P, NF, TWL>(r, f, lane), cb, k + 6 * e) - A[f][e];
            } else if (pb.upd) {
                // CG residual update: out (holding r) = r - alpha A
                const real al = (real)pb.upd[r].alpha;
#pragma unroll
                for (int f = 0; f < NL; f++)
#pragma unroll
                    for (int e = 0; e < 2; e++)
                        A[f][e] = load_elem<P, false>(pb.out, vh, split_vec<P, NF, TWL>(r, f, lane), cb, k + 6 * e) - al * A[f][e];
            }
            if (pb.red.op != FIN_NONE) {
#pragma unroll
                for (int f = 0; f < NL; f++)
#pragma unroll
                    for (int e = 0; e < 2; e++)
                        nrm += (double)A[f][e].re * A[f][e].re + (double)A[f][e].im * A[f][e].im;
            }
        }

        // half-precision output: the site's scale is the maximum over its
        // elements, across the threads
        if (Lds::SC || (RES && B.res_prec != TM_FP32)) {
            if (act) {
#pragma unroll
                for (int f = 0; f < NL; f++)
                    sh.mx[f][k][site] = fmaxf(fmaxf(fabsf((float)A[f][0].re), fabsf((float)A[f][0].im)),
                                              fmaxf(fabsf((float)A[f][1].re), fabsf((float)A[f][1].im)));
            }
            __syncthreads();
        }
        if (act) {
#pragma unroll
            for (int f = 0; f < NL; f++) {
                const uint32_t vec = split_vec<P, NF, TWL>(r, f, lane);
                [[maybe_unused]] float inv = 0.f;
                if (Lds::SC || (RES && B.res_prec != TM_FP32)) {
                    float m = sh.mx[f][0][site];
#pragma unroll
                    for (int j = 1; j < 6; j++) m = fmaxf(m, sh.mx[f][j][site]);
                    inv = (m > 0.f) ? 1.0f / m : 0.f;
                    if (k == 0) *at_w<float>(pb.out.scale + (size_t)vec * vh, cb * 4u) = m;
                }
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    if constexpr (RES) {
                        const cx<float> t = mk((float)A[f][e].re, (float)A[f][e].im);
                        if (B.res_prec == TM_FP32)
                            store_elem<TM_FP32, false>(pb.out, vh, vec, cb, k + 6 * e, t, 0.f);
                        else if (B.res_prec == TM_FP16)
                            store_elem<TM_FP16, false>(pb.out, vh, vec, cb, k + 6 * e, t, inv);
                        else
                            store_elem<TM_BF16, false>(pb.out, vh, vec, cb, k + 6 * e, t, inv);
                    } else if (nts & kNtOut) {
                        store_elem<P, true>(pb.out, vh, vec, cb, k + 6 * e, A[f][e], inv);
                    } else {
                        store_elem<P, false>(pb.out, vh, vec, cb, k + 6 * e, A[f][e], inv);
                    }
                }
            }
        }

        if (pb.red.op != FIN_NONE) {
            const double t = block_sum<kSplitThreads>(nrm, sh.red);
            if (threadIdx.x == 0) {
                double *const q = &pb.red.partials[(long)r * pb.nsb + sb];
                if (B.finish_here)
                    partial_put(q, t);
                else
                    *q = t;
            }
        }
    } while (MR && ++r < r1);

    if constexpr (!TWL) {
        if (B.finish_here) split_finish(B);
    }
}

#define TM_SPLIT_RUN(P, NF, TWL, MR, RES, KERNEL)                                                            \
    do {                                                                                               \
        constexpr int bufs = MR && split_two_buffers<P>() ? 2 : 1;                                      \
        hipLaunchKernelGGL((KERNEL), dim3(B.total_blocks), dim3(kSplitThreads),                         \
                           bufs * sizeof(SplitLds<P, NF, TWL, RES>), st, B);                                 \
        return hipGetLastError();                                                                      \
    } while (0)
#define TM_SPLIT_CASE(P, NF, DAG, TWL, RECON, LNT, MR)                                                 \
    if (!res && nf == NF && dagger == DAG && twl == TWL && recon == RECON && lnt == LNT && mr == MR)   \
        TM_SPLIT_RUN(P, NF, TWL, MR, false, (hop_split_kernel<P, NF, DAG, TWL, RECON, LNT, MR>));
#define TM_SPLIT_CASES(P, NF, RECON)                                                                \
    TM_SPLIT_CASE(P, NF, 0, 0, RECON, true, false) TM_SPLIT_CASE(P, NF, 1, 0, RECON, true, false)   \
    TM_SPLIT_CASE(P, NF, 0, 0, RECON, false, false) TM_SPLIT_CASE(P, NF, 1, 0, RECON, false, false) \
    TM_SPLIT_CASE(P, NF, 0, 1, RECON, false, false) TM_SPLIT_CASE(P, NF, 1, 1, RECON, false, false)
#define TM_SPLIT_CASES_MR(P, NF, RECON)                                                            \
    TM_SPLIT_CASE(P, NF, 0, 0, RECON, false, true) TM_SPLIT_CASE(P, NF, 1, 0, RECON, false, true)
#define TM_SPLIT_CASE_RES(P, NF, RECON, LNT, MR)                                                       \
    if (res && nf == NF && dagger == 1 && twl == 0 && recon == RECON && lnt == LNT && mr == MR)        \
        TM_SPLIT_RUN(P, NF, false, MR, true, (hop_split_kernel<P, NF, true, false, RECON, LNT, MR, true>));
#define TM_SPLIT_CASES_RES(P, NF, RECON) \
    TM_SPLIT_CASE_RES(P, NF, RECON, true, false) TM_SPLIT_CASE_RES(P, NF, RECON, false, false)

#define TM_SPLIT_DEFINE(P)                                                                           \
    template <>                                                                                      \
    hipError_t launch_hop_split<P>(const HopBatch &B, int nf, int dagger, int twl, int recon,        \
                                   bool lnt, bool mr, bool res, hipStream_t st)                      \
    {                                                                                                \
        if (twl || mr) lnt = false;                                                                  \
        TM_SPLIT_CASES(P, 1, 12) TM_SPLIT_CASES(P, 2, 12)                                            \
        TM_SPLIT_CASES(P, 1, 18) TM_SPLIT_CASES(P, 2, 18)                                            \
        TM_SPLIT_CASES(P, 1, 8) TM_SPLIT_CASES(P, 2, 8)                                              \
        if constexpr (P == TM_FP64 || P == TM_FP32) {                                                \
            TM_SPLIT_CASES_MR(P, 1, 12)                                                              \
        }                                                                                            \
        if constexpr (P == TM_FP64) {                                                                \
            TM_SPLIT_CASES_RES(P, 1, 12) TM_SPLIT_CASES_RES(P, 2, 12)                                \
            TM_SPLIT_CASES_RES(P, 1, 18) TM_SPLIT_CASES_RES(P, 2, 18)                                \
            TM_SPLIT_CASES_RES(P, 1, 8) TM_SPLIT_CASES_RES(P, 2, 8)                                  \
            TM_SPLIT_CASE_RES(P, 1, 12, false, true)                                                 \
        }                                                                                            \
        return hipErrorInvalidConfiguration;                                                         \
    }

}  // namespace twm
