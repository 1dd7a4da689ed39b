// Gauge force of S = phi^+ (M^+ M)^-1 phi (M: the preconditioned operator of
// Eq. 2.2 or 2.3) from colour outer products of four spinor fields.
//
// With X = (M^+ M)^-1 phi, Y = M X, A = Y (asym) or R_ee^-+ Y (sym) on even
// sites and R_oo^-+ (D^+)_oe A on odd sites, B = X on even and R_oo^-1 D_oe X
// on odd sites, a link variation changes S by dS = 2 kappa^2 Re <A, dD B>.
// For the link U_mu(x) (boundary factor s):
//   G = 2 kappa^2 s sum_{flavour, spin} [ (1 - g_mu) A(x) B(x+mu)^+ + B(x) ((1 + g_mu) A(x+mu))^+ ]
// is the unconstrained gradient (dS = Re tr(G^+ dU)) and F = -1/2 T_A(U G^+)
// the traceless anti-Hermitian force (dS/dw^a = -2 tr(F T^a) for
// U -> exp(w^a T^a) U).  Because (1 -+ g_mu)/2 is a projector of rank two,
// sum_spin ((1 - g) A)_s B_s^+ = sum_j hA_j hB_j^+ with hA, hB the two-spin
// projections of A and B: each term is two 3x3 outer products.
#include "tm_fields.h"

namespace twm {

// two-spin projection of a full site vector v under (1 - SIG g_mu) (time: the
// kept spin pair, without the factor 2)
template <int MU, int SIG, typename T>
__device__ __forceinline__ void half_proj(const cx<T> *v, cx<T> (&h)[2][3])
{
#pragma unroll
    for (int c = 0; c < 3; c++) {
        if constexpr (MU == 0) {
            if constexpr (SIG > 0) {
                h[0][c] = v[c] + times_mi(v[9 + c]);
                h[1][c] = v[3 + c] + times_mi(v[6 + c]);
            } else {
                h[0][c] = v[c] + times_i(v[9 + c]);
                h[1][c] = v[3 + c] + times_i(v[6 + c]);
            }
        } else if constexpr (MU == 1) {
            if constexpr (SIG > 0) {
                h[0][c] = v[c] - v[9 + c];
                h[1][c] = v[3 + c] + v[6 + c];
            } else {
                h[0][c] = v[c] + v[9 + c];
                h[1][c] = v[3 + c] - v[6 + c];
            }
        } else if constexpr (MU == 2) {
            if constexpr (SIG > 0) {
                h[0][c] = v[c] + times_mi(v[6 + c]);
                h[1][c] = v[3 + c] + times_i(v[9 + c]);
            } else {
                h[0][c] = v[c] + times_i(v[6 + c]);
                h[1][c] = v[3 + c] + times_mi(v[9 + c]);
            }
        } else {
            const int o = (SIG > 0) ? 6 : 0;
            h[0][c] = v[o + c];
            h[1][c] = v[o + 3 + c];
        }
    }
}

// G += sum_j p_j q_j^+   (3x3 outer products)
template <typename T>
__device__ __forceinline__ void add_outer(cx<T> (&G)[3][3], const cx<T> (&p)[2][3], const cx<T> (&q)[2][3])
{
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) G[a][b] = G[a][b] + cmul(p[j][a], conjg(q[j][b]));
}

struct ForceArgs {
    int X[4];
    FastDiv dx, dy, dz;         // by Lx / 2, Ly, Lz
    uint32_t vh;
    double tsign;
    double k2x2;                // 2 kappa^2
    double coeff;
    int accumulate;
    const void *gauge[2];
    SpinorPtr Ae, Wo, Xe, Zo;   // A and B on even / odd sites
    void *F;
    void *G;                    // nullable
};

template <int P, int NF, int MU>
__device__ __forceinline__ void force_terms(cx<typename Prec<P>::real> (&G)[3][3], const ForceArgs &a,
                                            int par, uint32_t cb, uint32_t nb)
{
    using real = typename Prec<P>::real;
    const SpinorPtr &A_x = par == 0 ? a.Ae : a.Wo;
    const SpinorPtr &B_x = par == 0 ? a.Xe : a.Zo;
    const SpinorPtr &A_n = par == 0 ? a.Wo : a.Ae;
    const SpinorPtr &B_n = par == 0 ? a.Zo : a.Xe;
    // the time projectors keep one spin pair: half a site
    constexpr int N = MU == 3 ? 6 : 12, KP = MU == 3 ? 6 : 0, OP = MU == 3 ? 6 : 0;
#pragma unroll
    for (int f = 0; f < NF; f++) {
        cx<real> v[12], w[12];
        cx<real> hA[2][3], hB[2][3];
        // (1 - g) A(x) B(x+mu)^+
        SpinorIO<P>::template load<KP, N>(v + OP, A_x, a.vh, f, cb);
        SpinorIO<P>::template load<KP, N>(w + OP, B_n, a.vh, f, nb);
        half_proj<MU, 1>(v, hA);
        half_proj<MU, 1>(w, hB);
        add_outer(G, hA, hB);
        // B(x) ((1 + g) A(x+mu))^+
        SpinorIO<P>::template load<0, N>(v, A_n, a.vh, f, nb);
        SpinorIO<P>::template load<0, N>(w, B_x, a.vh, f, cb);
        half_proj<MU, -1>(v, hA);
        half_proj<MU, -1>(w, hB);
        add_outer(G, hB, hA);
    }
}

// A block of eight waves computes the links of 128 consecutive lexicographic
// sites: wave (parity, mu), 64 sites each.  The four directions of a site read
// its A and B while they are in L1, and both parities' 9-element records, which
// interleave in F, leave LDS as one contiguous stream.  (One thread per link
// in blocks of one parity and direction wrote 72 of every 144 bytes, each half
// from another XCD: at 16^3 x 32, FP32 doublet, 51.8 us; now 27, near the 22 us
// of its fields, links and F at the device copy's 5.2 TB/s.)
constexpr int kForceSites = 64, kForceThreads = 512;

// Records of the block from LDS to F (or G), nine complex per link.
template <typename FT>
__device__ __forceinline__ void force_write(FT *F, const FT *sh, uint32_t lex0, uint32_t n, long V, int accumulate)
{
    __syncthreads();
    for (int mu = 0; mu < 4; mu++) {
        FT *const q = F + ((long)mu * V + lex0) * 9;
        for (uint32_t i = threadIdx.x; i < n * 9; i += kForceThreads) {
            FT f = sh[mu * (2 * kForceSites * 9) + i];
            if (accumulate) {
                const FT o = q[i];
                f.x += o.x;
                f.y += o.y;
            }
            q[i] = f;
        }
    }
    __syncthreads();
}

template <int P, int NF, int RECON, typename FT>
__global__ void __launch_bounds__(kForceThreads, 2) force_kernel(const ForceArgs a)
{
    using real = typename Prec<P>::real;
    extern __shared__ __align__(16) unsigned char force_sh[];
    FT *const sh = reinterpret_cast<FT *>(force_sh);
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int par = wave >> 2, mu = wave & 3;
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t b0 = (uint32_t)xcd_logical_block(blockIdx.x, gridDim.x) * kForceSites;
    const uint32_t cb = b0 + lane;
    const bool valid = cb < a.vh;
    uint32_t l = 0;                     // record of this link in the block's 128 sites
    cx<real> G[3][3], M[3][3];
    if (valid) {
        const uint32_t xh_n = (uint32_t)a.X[0] >> 1;
        const uint32_t q0 = a.dx.div(cb), q1 = a.dy.div(q0), t = a.dz.div(q1);
        const uint32_t xh = cb - q0 * xh_n, y = q0 - q1 * a.X[1], z = q1 - t * a.X[2];
        const uint32_t o = (y + z + t + par) & 1;      // x = 2 xh + o
        l = 2 * lane + o;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) G[i][j] = mk((real)0, (real)0);
        real s = (real)a.k2x2;
        const uint32_t sy = xh_n, sz = xh_n * a.X[1], st = xh_n * a.X[1] * a.X[2];
        if (mu == 0) {
            force_terms<P, NF, 0>(G, a, par, cb, cb - xh + (o ? (xh + 1 == xh_n ? 0 : xh + 1) : xh));
        } else if (mu == 1) {
            force_terms<P, NF, 1>(G, a, par, cb, (int)y == a.X[1] - 1 ? cb - y * sy : cb + sy);
        } else if (mu == 2) {
            force_terms<P, NF, 2>(G, a, par, cb, (int)z == a.X[2] - 1 ? cb - z * sz : cb + sz);
        } else {
            force_terms<P, NF, 3>(G, a, par, cb, (int)t == a.X[3] - 1 ? cb - t * st : cb + st);
            s *= (real)2;                              // the time projector keeps 2 psi
            if ((int)t == a.X[3] - 1) s *= (real)a.tsign;
        }
        const real c = (real)a.coeff;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) G[i][j] = (s * c) * G[i][j];

        // F = -1/2 T_A(U G^+), T_A(M) = (M - M^+)/2 - tr(M - M^+)/6
        cx<real> u[3][3];
        LinkIO<P, RECON>::load(u, a.gauge[par], a.vh, mu, cb);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                cx<real> acc = cmul(u[i][0], conjg(G[j][0]));
                acc = acc + cmul(u[i][1], conjg(G[j][1]));
                acc = acc + cmul(u[i][2], conjg(G[j][2]));
                M[i][j] = acc;
            }
        const real trim = (M[0][0].im + M[1][1].im + M[2][2].im) / (real)3;   // Im tr M / 3
        FT *const F = sh + (mu * (2 * kForceSites) + l) * 9;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                // (M - M^+)/2 at (i, j) = (M_ij - conj(M_ji)) / 2
                real re = (real)0.5 * (M[i][j].re - M[j][i].re);
                real im = (real)0.5 * (M[i][j].im + M[j][i].im);
                if (i == j) im -= trim;
                FT f;
                f.x = re * (real)-0.5;
                f.y = im * (real)-0.5;
                F[i * 3 + j] = f;
            }
    }
    const long V = 2L * a.vh;
    const uint32_t n = 2 * min((uint32_t)kForceSites, a.vh - b0);
    force_write((FT *)a.F, sh, 2 * b0, n, V, a.accumulate);
    if (a.G) {
        if (valid) {
            FT *const Gs = sh + (mu * (2 * kForceSites) + l) * 9;
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++) {
                    FT gv;
                    gv.x = G[i][j].re;
                    gv.y = G[i][j].im;
                    Gs[i * 3 + j] = gv;
                }
        }
        force_write((FT *)a.G, sh, 2 * b0, n, V, a.accumulate);
    }
}

hipError_t force_launch(int prec, int nf, int force_prec, void *F, void *G, const void *gauge0,
                        const void *gauge1, int recon, SpinorPtr A[2], SpinorPtr Bv[2],
                        const int *X, uint32_t vh, double tsign, double coeff, int accumulate,
                        double kappa, hipStream_t st)
{
    ForceArgs a;
    for (int d = 0; d < 4; d++) a.X[d] = X[d];
    a.dx.set((uint32_t)X[0] / 2);
    a.dy.set((uint32_t)X[1]);
    a.dz.set((uint32_t)X[2]);
    a.vh = vh;
    a.tsign = tsign;
    a.k2x2 = 2.0 * kappa * kappa;
    a.coeff = coeff;
    a.accumulate = accumulate;
    a.gauge[0] = gauge0;
    a.gauge[1] = gauge1;
    a.Ae = A[0];
    a.Wo = A[1];
    a.Xe = Bv[0];
    a.Zo = Bv[1];
    a.F = F;
    a.G = G;
    const dim3 grid((vh + kForceSites - 1) / kForceSites);
#define TM_FK(P, NF, R, FT)                                                                     \
    if (prec == P && nf == NF && recon == R && force_prec == (sizeof(FT) == 16 ? TM_FP64 : TM_FP32)) { \
        hipLaunchKernelGGL((force_kernel<P, NF, R, FT>), grid, dim3(kForceThreads),              \
                           8 * kForceSites * 9 * sizeof(FT), st, a);                            \
        return hipGetLastError();                                                               \
    }
    TM_FK(TM_FP64, 1, 12, double2) TM_FK(TM_FP64, 2, 12, double2)
    TM_FK(TM_FP64, 1, 18, double2) TM_FK(TM_FP64, 2, 18, double2)
    TM_FK(TM_FP32, 1, 12, float2) TM_FK(TM_FP32, 2, 12, float2)
    TM_FK(TM_FP32, 1, 18, float2) TM_FK(TM_FP32, 2, 18, float2)
    TM_FK(TM_FP64, 1, 12, float2) TM_FK(TM_FP64, 2, 12, float2)
    TM_FK(TM_FP32, 1, 12, double2) TM_FK(TM_FP32, 2, 12, double2)
#undef TM_FK
    return hipErrorInvalidConfiguration;
}

}  // namespace twm
