// Thermophysical and transport properties over a whole field (paper
// Section 3.1, the Thermo class: Newton's method on the temperature
// polynomials; Section 3.2: these kernels are compute-bound, keep their
// coefficients in constant memory, and are split into segments to bound
// register use; Section 2: the transport model is Cantera's mixture-averaged
// one).  One thread per cell, cells in index order (SoA, coalesced); the transport
// of mechanisms beyond 16 species has kernels of its own, 16 cells per wave
// (transport_group_kernel).
//
// In the kernels with one thread per cell the coefficients are uniform across a
// wave, so every table read is a scalar load through the scalar cache (the
// counterpart of CUDA's constant memory); a cell's mole fractions and
// per-species reciprocals live in registers, sized by a compile-time bound
// KM >= K, and every species loop is unrolled over KM (guards against K are
// uniform branches).  Costs per cell with K species:
//   viscosity (Wilke)       K^2 pair terms of 3 fused multiply-adds
//   conductivity (Mathur)   K terms
//   diffusion               K (K - 1) / 2 pair polynomials and reciprocals
// Storage substitution (Section 3.2): the pair factors of Wilke's rule that
// depend only on molar masses are tabulated once per mechanism, and
// sqrt(mu_k/mu_j) is taken as s_k / s_j with s_k = T^(1/4) |P_k(ln T)| (the
// fitted square root itself), so no pow() and one square root pair per cell
// remain.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "host_common.h"
#include "quarters.h"

using chem_host::check_hip;
using chem_host::fail;
using chem_host::is_device_ptr;

namespace chem {
namespace {

constexpr int kThermoBlock = 256;
constexpr int kTrMaxK = 64;   // species the property kernels hold in registers
constexpr int kPoly = 5;      // coefficients of every ln T fit

// Mixture-averaged transport tables of a mechanism (device, contiguous).
// Wilke's factor times X_j, with t = s_k c1_kj / s_j and
// c1_kj = (W_j/W_k)^(1/4), c2_kj = 1/sqrt(8 (1 + W_k/W_j)), expands to
//   X_j c2 (1 + t)^2 = A_kj X_j + s_k (Bw_kj X_j/s_j + s_k C_kj X_j/s_j^2)
// with A = c2, Bw = 2 c1 c2, C = c1^2 c2: three fused multiply-adds per
// pair on per-cell vectors X, X/s, X/s^2 (all terms positive: no
// cancellation).
struct TrView {
    int32_t K;
    int32_t ld;          // row stride of every table: the kernel's bound KM (rows K .. KM-1 are padding)
    const double *P;     // ld x 5: viscosity fit, mu_k = (T^(1/4) P_k(ln T))^2 (padding: P = 1)
    const double *Q;     // ld x 5: conductivity fit, lam_k = T^(1/2) Q_k(ln T) (padding: Q = 1)
    const double *A;     // ld x ld at [k ld + j]: c2_kj (padding 0)
    const double *Bw;    // ld x ld: 2 c1_kj c2_kj
    const double *C;     // ld x ld: c1_kj^2 c2_kj
    const double *B;     // ld x ld x 5: diffusion fits, D_jk = T^(3/2) B_jk(ln T) / p (symmetric; padding B = 1)
    const double *invW;  // ld (padding 1)
};

// Reciprocals: the hardware estimate (relative error about 2^-24) refined
// by Newton steps, e -> e^2.  Two steps give the correctly rounded 1/x (all
// of 2^20 seeded x in [1e-12, 1e12] on gfx950); one step leaves about 10
// ulp (2.2e-15), used for the per-species and per-pair factors of the
// transport sums, where nothing cancels (in the group kernels for the pairs
// alone: there the second step of the per-species ones is 2 % of the time).
__device__ __forceinline__ double rcp_t(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
    return r;
}

__device__ __forceinline__ double rcp_1(double x)
{
    const double r = __builtin_amdgcn_rcp(x);
    return fma(fma(-x, r, 1.0), r, r);
}

// Powers of ln T shared by every fit of a cell.
struct LnPow {
    double x, x2, x3, x4;
};

__device__ __forceinline__ LnPow ln_powers(double x)
{
    const double x2 = x * x;
    return {x, x2, x2 * x, x2 * x2};
}

// c0 + c1 x + c2 x^2 + c3 x^3 + c4 x^4 with uniform (scalar) coefficients:
// every step multiplies a scalar by a per-cell power into a vector
// accumulator, one instruction each.  (Horner's rule would add a scalar to
// a product and costs a register move per step on this target, which takes
// one scalar operand per instruction.)
__device__ __forceinline__ double poly5(const double *c, const LnPow &p)
{
    double q = c[1] * p.x;
    q = fma(c[2], p.x2, q);
    q = fma(c[3], p.x3, q);
    q = fma(c[4], p.x4, q);
    return q + c[0];
}

// A cell's K mass fractions into registers, rows beyond K zero.  The loads
// are unconditional (rows past K - 1 read row K - 1 again), so all of them
// are in flight together; guarded loads would each wait for the last.
template <int KM>
__device__ __forceinline__ void load_rows(const double *__restrict__ Y, int64_t ldY, int64_t i, int K,
                                          double (&y)[KM])
{
#pragma unroll
    for (int k = 0; k < KM; k++) y[k] = Y[(int64_t)(k < K ? k : K - 1) * ldY + i];
#pragma unroll
    for (int k = 0; k < KM; k++)
        if (k >= K) y[k] = 0.0;
}

// yr_k = Y_k / W_k: the mixture sums below are in units of R (mass-specific
// h / R and cp / R); R enters once per cell, not once per species.
template <int KM>
__device__ __forceinline__ void load_yr(const double *__restrict__ Y, int64_t ldY, int64_t i, int K,
                                        const double *__restrict__ invW, double (&yr)[KM])
{
    load_rows<KM>(Y, ldY, i, K, yr);
#pragma unroll
    for (int k = 0; k < KM; k++)
        if (k < K) yr[k] *= invW[k];
}

// MODE bit 1: viscosity and conductivity; bit 2: diffusion coefficients.
// Every species loop unrolls and a cell's values stay in registers.
template <int KM, int MODE>
__global__ void __launch_bounds__(kThermoBlock) transport_kernel(TrView v, const double *__restrict__ T,
                                                                 const double *__restrict__ p,
                                                                 const double *__restrict__ Y, int64_t ldY,
                                                                 int64_t n, double *__restrict__ mu,
                                                                 double *__restrict__ lam,
                                                                 double *__restrict__ D, int64_t ldD)
{
    const int64_t i = (int64_t)blockIdx.x * kThermoBlock + threadIdx.x;
    if (i >= n) return;
    const int K = v.K;
    const double Tc = T[i];
    const LnPow lnT = ln_powers(log(Tc));
    const double sT = sqrt(Tc);

    // composition: y_k = max(Y_k, 0) / sum, X_k = (y_k / W_k) / sum_j (y_j / W_j);
    // X_j = 0 for the padding rows j >= K
    double X[KM], yv[KM];
    load_rows<KM>(Y, ldY, i, K, X);
    double ysum = 0.0;
#pragma unroll
    for (int k = 0; k < KM; k++) {
        X[k] = fmax(X[k], 0.0);
        ysum += X[k];
    }
    const double inv_y = rcp_t(ysum);
    double csum = 0.0;
#pragma unroll
    for (int k = 0; k < KM; k++) {
        yv[k] = X[k] * inv_y;
        X[k] = X[k] * inv_y * v.invW[k];
        csum += X[k];
    }
    const double inv_c = rcp_t(csum);
#pragma unroll
    for (int k = 0; k < KM; k++) X[k] *= inv_c;
    const int ld = KM;

    if constexpr (MODE & 1) {
        const double qT = sqrt(sT);
        double V[KM], Wv[KM];   // X_j / s_j and X_j / s_j^2
        double a1 = 0.0, a2 = 0.0;
#pragma unroll
        for (int k = 0; k < KM; k++) {
            const double r = rcp_1(qT * fabs(poly5(v.P + kPoly * k, lnT)));
            V[k] = X[k] * r;
            Wv[k] = V[k] * r;
            const double lk = sT * poly5(v.Q + kPoly * k, lnT);
            a1 = fma(X[k], lk, a1);
            a2 = fma(X[k], rcp_1(lk), a2);
        }
        lam[i] = 0.5 * (a1 + rcp_t(a2));
        double m = 0.0;
#pragma unroll
        for (int k = 0; k < KM; k++)
            if (k < K) {
                const double sk = qT * fabs(poly5(v.P + kPoly * k, lnT));
                const double *A = v.A + (int64_t)k * ld, *Bw = v.Bw + (int64_t)k * ld, *C = v.C + (int64_t)k * ld;
                double d0 = 0.0, d1 = 0.0, d2 = 0.0;
#pragma unroll
                for (int j = 0; j < KM; j++)
                    if (j < K) {   // skips the padding
                        d0 = fma(A[j], X[j], d0);
                        d1 = fma(Bw[j], V[j], d1);
                        d2 = fma(C[j], Wv[j], d2);
                    }
                const double den = fma(sk, fma(sk, d2, d1), d0);
                m = fma(X[k] * sk * sk, rcp_1(den), m);
            }
        mu[i] = m;
    }

    if constexpr (MODE & 2) {
        const double t32_p = Tc * sT * rcp_1(p[i]);
        // S_k = sum_{j != k} X_j / B_jk(ln T); pairs j < k once each
        double S[KM];
#pragma unroll
        for (int k = 0; k < KM; k++) S[k] = 0.0;
#pragma unroll
        for (int k = 0; k < KM; k++)
            if (k < K) {
                const double *B = v.B + (int64_t)k * ld * kPoly;
#pragma unroll
                for (int j = k + 1; j < KM; j++)
                    if (j < K) {
                        const double ib = rcp_1(poly5(B + kPoly * j, lnT));
                        S[j] = fma(X[k], ib, S[j]);
                        S[k] = fma(X[j], ib, S[k]);
                    }
                const double sk = S[k];
                D[(int64_t)k * ldD + i] = sk > 0.0 ? (1.0 - yv[k]) * t32_p * rcp_1(sk)
                                                   : t32_p * poly5(B + kPoly * k, lnT);
            }
    }
}

// ---------------------------------------------------------------------------
// Transport of the larger mechanisms: 16 cells per wave, species in groups of four.
// Lane 16 q + c holds cell c and, of every group g, species 4 g + q: the
// operand and result layout of the FP64 matrix instructions
//   16x16x4: D row 4 r + q in result r of lane (q, c), B row q in lane (q, c)
//   4x4x4:   D row q, B row q in lane (q, c)
// so the three contractions of the model run on them without a lane exchange:
//   fits          sum_c coef_c (ln T)^c        rows = species or pairs, K = 4, c = 0 as the initial value
//   Wilke sums    sum_j c2_kj (X_j, X_j/s'_j, X_j/s'_j^2)    rows = k, K = the species
//   with s'_k = s_k W_k^(-1/4): c1_kj s_k / s_j = s'_k / s'_j, one matrix for
//   all three sums
// and a wave's table reads are one LDS read per operand instead of a scalar
// load per coefficient.  The binary fits are evaluated once per pair: for groups
// G1 <= G2 one 16x16x4 gives the 16 pairs (4 G1 + q, 4 G2 + r), which enter the
// lane's own sum (species 4 G1 + q, weight X of 4 G2 + r) and four partial sums
// over q (species 4 G2 + r), reduced over the wave's quarters by lane swaps.
// What bounds them: the FP64 issue rate, which matrix and vector instructions
// share (64 multiply-adds per clock and CU either way; both together take the
// sum of their times): 35 species, 500,003 cells about 11,000 cycles of it per
// 16 cells, 300 us (920 before, one cell per lane with the coefficients as
// scalar loads: 27 KB of them per wave for the binary fits alone, through a 16 KB
// scalar cache, one wait after another); 20 species 131 us (164), 64 species
// 820 us (3503); 500 cells 14 us (138) at 35 species.  Two waves per SIMD asked
// for, so that results stay in vector registers (else they pass through the
// accumulation registers, +7 %); four cost spills (326 us).

// Tables of a mechanism of NG groups, in doubles: per group fits (P rows, P
// constants, Q rows, Q constants), 1/W and W^(-1/4); the Wilke matrix by (g, G)
// tiles of 4x4; the binary fits by (G1 <= G2) tiles of 16 rows.
constexpr int kFitLen = 40, kHeadLen = kFitLen + 8, kPairLen = 80;
__host__ __device__ constexpr int grp_head(int NG) { return kHeadLen * NG; }
__host__ __device__ constexpr int grp_wilke(int NG) { return 16 * NG * NG; }
__host__ __device__ constexpr int grp_pairs(int NG) { return kPairLen * (NG * (NG + 1) / 2); }

typedef double dx4 __attribute__((ext_vector_type(4)));

// Threads per block: the tables of 13 and more groups leave room for one block.
constexpr int grp_block(int NG) { return NG > 12 ? 512 : 256; }

// MODE bit 1: viscosity and conductivity; bit 2: diffusion coefficients.
template <int NG, int MODE>
__global__ void __launch_bounds__(grp_block(NG), 2) transport_group_kernel(const double *__restrict__ table, int K,
                                                                    const double *__restrict__ T,
                                                                    const double *__restrict__ p,
                                                                    const double *__restrict__ Y, int64_t ldY,
                                                                    int64_t n, double *__restrict__ mu,
                                                                    double *__restrict__ lam,
                                                                    double *__restrict__ D, int64_t ldD)
{
    extern __shared__ __align__(16) double tab[];
    constexpr int kBlock = grp_block(NG), kHead = grp_head(NG), kWilke = grp_wilke(NG), kPairs = grp_pairs(NG);
    constexpr int kFirst = kHead + (MODE & 1 ? kWilke : 0);   // head and Wilke matrix are contiguous
    for (int e = threadIdx.x; e < kFirst / 2; e += kBlock)
        ((double2 *)tab)[e] = ((const double2 *)table)[e];
    if constexpr (MODE & 2)
        for (int e = threadIdx.x; e < kPairs / 2; e += kBlock)
            ((double2 *)(tab + kFirst))[e] = ((const double2 *)(table + kHead + kWilke))[e];
    __syncthreads();
    const int ng = (K + 3) >> 2;
    const int64_t tiles = (n + 15) >> 4;

    for (int64_t t = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); t < tiles;
         t += (int64_t)gridDim.x * (kBlock / 64)) {
        // opaque: else the table reads, the same in every turn, move before
        // the loop and fill the registers
        int lane = threadIdx.x & 63;
        asm("" : "+v"(lane));
        const int c = lane & 15, q = lane >> 4;
        const int a4 = q * 4 + (lane & 3);   // this lane's element of a 4x4 operand
        const int64_t cell = t * 16 + c;
        const bool live = cell < n;
        const int64_t i = live ? cell : n - 1;   // the tail's idle lanes repeat the last cell
        // composition: y_k = max(Y_k, 0) / sum, X_k = (y_k / W_k) / sum_j (y_j / W_j), zero beyond K
        double X[NG];
#pragma unroll
        for (int g = 0; g < NG; g++) {
            const int k = 4 * g + q;
            X[g] = Y[(int64_t)(k < K ? k : K - 1) * ldY + i];
        }
        const double Tc = T[i];
        double ysum = 0.0;
#pragma unroll
        for (int g = 0; g < NG; g++) {
            X[g] = 4 * g + q < K ? fmax(X[g], 0.0) : 0.0;
            ysum += X[g];
        }
        const double inv_y = rcp_t(sum_quarters(ysum));
        double yv[MODE & 2 ? NG : 1], csum = 0.0;
#pragma unroll
        for (int g = 0; g < NG; g++) {
            const double y = X[g] * inv_y;
            if constexpr (MODE & 2) yv[g] = y;
            X[g] = y * tab[kFitLen * NG + 4 * g + q];
            csum += X[g];
        }
        const double inv_c = rcp_t(sum_quarters(csum));
#pragma unroll
        for (int g = 0; g < NG; g++) X[g] *= inv_c;

        const double x = log(Tc), sT = sqrt(Tc), x2 = x * x;
        const double xp = q == 0 ? x : q == 1 ? x2 : q == 2 ? x2 * x : x2 * x2;   // row q of the powers

        if constexpr (MODE & 1) {
            const double qT = sqrt(sT);
            double V[NG], Wv[NG];   // X / s' and X / s'^2
            double s[NG];
            const double *w4 = tab + (kFitLen + 4) * NG + q;
            double a1 = 0.0, a2 = 0.0;
#pragma unroll
            for (int g = 0; g < NG; g++) {
                const double *f = tab + kFitLen * g;
                s[g] = qT * fabs(__builtin_amdgcn_mfma_f64_4x4x4f64(f[a4], xp, f[16 + q], 0, 0, 0));
                const double r = rcp_t(s[g] * w4[4 * g]);
                V[g] = X[g] * r;
                Wv[g] = V[g] * r;
                const double lk = sT * __builtin_amdgcn_mfma_f64_4x4x4f64(f[20 + a4], xp, f[36 + q], 0, 0, 0);
                a1 = fma(X[g], lk, a1);
                a2 = fma(X[g], rcp_t(lk), a2);
            }
            a1 = sum_quarters(a1);
            a2 = sum_quarters(a2);
            double m = 0.0;
#pragma unroll
            for (int g = 0; g < NG; g++) {
                if (g >= ng) continue;
                const double *w = tab + kHead + g * NG * 16 + a4;
                double d0 = 0.0, d1 = 0.0, d2 = 0.0;
#pragma unroll
                for (int G = 0; G < NG; G++) {
                    const double a = w[G * 16];
                    d0 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, X[G], d0, 0, 0, 0);
                    d1 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, V[G], d1, 0, 0, 0);
                    d2 = __builtin_amdgcn_mfma_f64_4x4x4f64(a, Wv[G], d2, 0, 0, 0);
                }
                // X_k mu_k / (d0 + 2 s' d1 + s'^2 d2); rows beyond K: X = 0 over a unit matrix row
                const double sp = s[g] * w4[4 * g];
                const double den = fma(sp, fma(sp, d2, 2.0 * d1), d0);
                m = fma(X[g] * s[g] * s[g], rcp_t(den), m);
            }
            m = sum_quarters(m);
            if (live && q == 0) {
                lam[i] = 0.5 * (a1 + rcp_t(a2));
                mu[i] = m;
            }
        }

        if constexpr (MODE & 2) {
            const double t32_p = Tc * sT * rcp_t(p[i]);
            double S[NG];   // sum_{j != k} X_j / B_jk(ln T) of the lane's own species
#pragma unroll
            for (int g = 0; g < NG; g++) S[g] = 0.0;
#pragma unroll
            for (int G2 = 0; G2 < NG; G2++) {
                if (G2 >= ng) continue;
                // the group's four mole fractions in every lane
                const DPair h = swap_halves(X[G2], X[G2]), x01 = swap_quarters(h.a, h.a),
                            x23 = swap_quarters(h.b, h.b);
                const double Xr[4] = {x01.a, x01.b, x23.a, x23.b};
                double P[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int G1 = 0; G1 <= G2; G1++) {
                    const double *b = tab + kFirst + (G2 * (G2 + 1) / 2 + G1) * kPairLen;
                    const double2 c01 = *(const double2 *)(b + 64 + 4 * q), c23 = *(const double2 *)(b + 66 + 4 * q);
                    dx4 v = {c01.x, c01.y, c23.x, c23.y};
                    v = __builtin_amdgcn_mfma_f64_16x16x4f64(b[lane], xp, v, 0, 0, 0);
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const double ib = rcp_1(v[r]);
                        if (G1 < G2) {
                            S[G1] = fma(Xr[r], ib, S[G1]);
                            P[r] = fma(X[G1], ib, P[r]);
                        } else {
                            // a species' own fit takes no part (it may have no reciprocal)
                            P[r] = fma(X[G1], q == r ? 0.0 : ib, P[r]);
                        }
                    }
                }
                // quarter q keeps the sum of species 4 G2 + q
                const DPair p02 = swap_halves(P[0], P[2]), p13 = swap_halves(P[1], P[3]);
                const DPair s4 = swap_quarters(p02.a + p02.b, p13.a + p13.b);
                S[G2] += s4.a + s4.b;
            }
#pragma unroll
            for (int g = 0; g < NG; g++) {
                if (g >= ng) continue;
                double d = (1.0 - yv[g]) * t32_p * rcp_t(S[g]);
                if (!(S[g] > 0.0)) {   // a pure species: its own fit
                    const double *b = tab + kFirst + (g * (g + 1) / 2 + g) * kPairLen;
                    const double cf[kPoly] = {b[64 + 5 * q], b[5 * q], b[16 + 5 * q], b[32 + 5 * q], b[48 + 5 * q]};
                    d = t32_p * poly5(cf, ln_powers(x));
                }
                if (live && 4 * g + q < K) D[(int64_t)(4 * g + q) * ldD + i] = d;
            }
        }
    }
}

// Range boundaries of the mechanism's species: up to kMaxMid distinct T_mid
// values (ascending); a lane's choice of range for every species is fixed by
// which of them its T has reached.  nt < 0: more distinct values than that,
// the mixture coefficients are rebuilt at every temperature.
constexpr int kMaxMid = 4;
struct MidSet {
    int32_t nt;
    double t[kMaxMid];
};

__device__ __forceinline__ unsigned mid_pattern(const MidSet &ms, double T)
{
    unsigned b = 0;
#pragma unroll
    for (int q = 0; q < kMaxMid; q++)
        if (q < ms.nt && T >= ms.t[q]) b |= 1u << q;
    return b;
}

// Mixture polynomial coefficients at T (computation consolidation): with
// yr_k = Y_k / W_k and each species' range at T, in units of R,
//   cp  = sum_c M[c] T^c                                 (c = 0..4)
//   h   = T (M[0] + sum_c M[4+c] T^c) + M[9]             (c = 1..4)
// where M[0..4] = sum_k yr_k a1..a5, M[5..8] = sum_k yr_k a2/2..a5/5 and
// M[9] = sum_k yr_k a6 -- one pass over the species, after which every
// Newton step costs two quartics, whatever K.  The coefficients are
// uniform scalar loads: a wave wholly in one range takes one multiply-add
// per coefficient; a wave across T_mid takes both ranges with each lane's
// weight zero in the other (never a per-lane coefficient address, which
// would turn the loads into vector loads).
template <int KM>
__device__ __forceinline__ void mix_coeffs(const double *species, int K, const double (&yr)[KM], double T,
                                           double (&M)[10])
{
#pragma unroll
    for (int c = 0; c < 10; c++) M[c] = 0.0;
    constexpr int src[10] = {0, 1, 2, 3, 4, 7, 8, 9, 10, 5};
#pragma unroll
    for (int k = 0; k < KM; k++)
        if (k < K) {
            const double *s = species + k * kSpeciesLen;
            const double *lo = s + 1, *hi = s + 1 + kRangeLen;
            const bool low = T < s[0];
            // each lane's weight is zero in the other range; a range no lane
            // of the wave is in is skipped (a uniform branch)
            const double wl = low ? yr[k] : 0.0, wh = low ? 0.0 : yr[k];
            if (__any(low)) {
#pragma unroll
                for (int c = 0; c < 10; c++) M[c] = fma(wl, lo[src[c]], M[c]);
            }
            if (!__all(low)) {
#pragma unroll
                for (int c = 0; c < 10; c++) M[c] = fma(wh, hi[src[c]], M[c]);
            }
        }
}

__device__ __forceinline__ double mix_cp(const double (&M)[10], double T)
{
    return fma(fma(fma(fma(M[4], T, M[3]), T, M[2]), T, M[1]), T, M[0]);
}

__device__ __forceinline__ double mix_h(const double (&M)[10], double T)
{
    return fma(T, fma(fma(fma(fma(M[8], T, M[7]), T, M[6]), T, M[5]), T, M[0]), M[9]);
}

// Mixture h and cp of every cell at its temperature.
template <int KM>
__global__ void __launch_bounds__(kThermoBlock) h_cp_kernel(const double *__restrict__ species,
                                                            const double *__restrict__ invW, int K,
                                                            const double *__restrict__ T,
                                                            const double *__restrict__ Y, int64_t ldY, int64_t n,
                                                            double *__restrict__ h, double *__restrict__ cp)
{
    const int64_t i = (int64_t)blockIdx.x * kThermoBlock + threadIdx.x;
    if (i >= n) return;
    double yr[KM], M[10];
    load_yr<KM>(Y, ldY, i, K, invW, yr);
    const double Tc = T[i];
    mix_coeffs<KM>(species, K, yr, Tc, M);
    if (h) h[i] = kRu * mix_h(M, Tc);
    if (cp) cp[i] = kRu * mix_cp(M, Tc);
}

// Temperature from mixture enthalpy: Newton from the guess in T, each step
// T <- clamp(T - (h(T) - h) / cp(T), 200, 3500) K, done when the step is
// below tol; after max_iter steps without that, T = NaN and iters =
// max_iter + 1.  The mixture coefficients are rebuilt only when T crosses a
// range boundary.  cp is the mixture cp at the result.
template <int KM, bool EX>
__global__ void __launch_bounds__(kThermoBlock) t_from_h_kernel(const double *__restrict__ species,
                                                                const double *__restrict__ invW, int Kr, MidSet ms,
                                                                const double *__restrict__ h,
                                                                const double *__restrict__ Y, int64_t ldY,
                                                                int64_t n, double *__restrict__ T,
                                                                double *__restrict__ cp,
                                                                int32_t *__restrict__ iters, int max_iter,
                                                                double tol)
{
    const int64_t i = (int64_t)blockIdx.x * kThermoBlock + threadIdx.x;
    if (i >= n) return;
    const int K = EX ? KM : Kr;   // EX: exactly KM species, guards known at compile time
    double yr[KM], M[10];
    load_yr<KM>(Y, ldY, i, K, invW, yr);
    const double h0 = h[i] * (1.0 / kRu);
    double Tc = T[i];
    unsigned pat = mid_pattern(ms, Tc);
    int it = 0;
    bool done = false, rebuild = true;
    // one copy of the coefficient pass: built first, then again after a
    // step that crossed a range boundary (before the next step, or before cp)
    for (;;) {
        if (rebuild) mix_coeffs<KM>(species, K, yr, Tc, M);
        if (done || it == max_iter) break;
        it++;
        const double dT = -(mix_h(M, Tc) - h0) * rcp_t(mix_cp(M, Tc));
        Tc = fmin(fmax(Tc + dT, 200.0), 3500.0);
        const unsigned np = mid_pattern(ms, Tc);
        rebuild = ms.nt < 0 || np != pat;
        pat = np;
        done = fabs(dT) < tol;
    }
    T[i] = done ? Tc : __builtin_nan("");
    if (cp) cp[i] = done ? kRu * mix_cp(M, Tc) : __builtin_nan("");
    if (iters) iters[i] = done ? it : max_iter + 1;
}

unsigned blocks_for(int64_t n) { return (unsigned)((n + kThermoBlock - 1) / kThermoBlock); }

// Compile-time bounds of the species count: a call takes the smallest that
// holds K.  The transport kernels with one cell per lane serve up to 16
// species, the group kernels the rest, with their own list: 500,003 cells of 9
// species 44 us by lanes and 72 by groups, 14 species 90 and 101, 20 species 164
// and 131.  (Small calls are faster by groups at any count, 500 cells of 14
// species 27 and 10 us, but a cell's bits do not depend on the call's size.)
#define CHEM_TR_BOUNDS(X) X(9) X(12) X(16) X(20) X(24) X(36) X(48) X(64)
#define CHEM_TR_LANE_BOUNDS(X) X(9) X(12) X(16)
#define CHEM_TR_GROUPS(X) X(5) X(6) X(9) X(12) X(16)
constexpr int kTrLaneMaxK = 16;

// The cell-per-lane kernels' bound for K species (their tables' padded row count).
int tr_bound(int K)
{
#define CHEM_TR_BOUND(KM) \
    if (K <= KM) return KM;
    CHEM_TR_LANE_BOUNDS(CHEM_TR_BOUND)
#undef CHEM_TR_BOUND
    return -1;
}

// The group kernels' group count for K species.
int tr_groups(int K)
{
#define CHEM_TR_GROUP(NG) \
    if (K <= 4 * NG) return NG;
    CHEM_TR_GROUPS(CHEM_TR_GROUP)
#undef CHEM_TR_GROUP
    return -1;
}

// Doubles of the cell-per-lane tables at bound L: P, Q, A, Bw, C, B, invW.
size_t tr_table_len(int L) { return 10 * (size_t)L + 3 * (size_t)L * L + 5 * (size_t)L * L + L; }

template <int KM>
hipError_t launch_transport_km(const TrView &v, const double *T, const double *p, const double *Y, int64_t ldY,
                               int64_t n, double *mu, double *lam, double *D, int64_t ldD, hipStream_t st)
{
    const dim3 g(blocks_for(n)), b(kThermoBlock);
#define CHEM_TR_MODE(MODE) \
    hipLaunchKernelGGL((transport_kernel<KM, MODE>), g, b, 0, st, v, T, p, Y, ldY, n, mu, lam, D, ldD)
    if (mu && D)
        CHEM_TR_MODE(3);
    else if (mu)
        CHEM_TR_MODE(1);
    else
        CHEM_TR_MODE(2);
#undef CHEM_TR_MODE
    return hipGetLastError();
}

hipError_t launch_transport(const TrView &v, const double *T, const double *p, const double *Y, int64_t ldY,
                            int64_t n, double *mu, double *lam, double *D, int64_t ldD, hipStream_t st)
{
#define CHEM_TR_CASE(KM) \
    if (v.ld == KM) return launch_transport_km<KM>(v, T, p, Y, ldY, n, mu, lam, D, ldD, st);
    CHEM_TR_LANE_BOUNDS(CHEM_TR_CASE)
#undef CHEM_TR_CASE
    return hipErrorInvalidValue;
}

template <int NG, int MODE>
hipError_t launch_group_mode(const double *table, int K, const double *T, const double *p, const double *Y,
                             int64_t ldY, int64_t n, double *mu, double *lam, double *D, int64_t ldD,
                             hipStream_t st)
{
    constexpr int lds =
        8 * (grp_head(NG) + (MODE & 1 ? grp_wilke(NG) : 0) + (MODE & 2 ? grp_pairs(NG) : 0));
    if constexpr (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute((const void *)transport_group_kernel<NG, MODE>,
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        if (e != hipSuccess) return e;
    }
    // as many blocks as the chip holds, each over every grid-th piece
    constexpr int kBlock = grp_block(NG), per_cu = std::min(160 * 1024 / lds, 4), kCells = kBlock / 64 * 16;
    const int64_t blocks = std::min<int64_t>((n + kCells - 1) / kCells, 256 * per_cu);
    hipLaunchKernelGGL((transport_group_kernel<NG, MODE>), dim3((unsigned)blocks), dim3(kBlock), lds, st, table,
                       K, T, p, Y, ldY, n, mu, lam, D, ldD);
    return hipGetLastError();
}

hipError_t launch_transport_groups(const double *table, int K, const double *T, const double *p, const double *Y,
                                   int64_t ldY, int64_t n, double *mu, double *lam, double *D, int64_t ldD,
                                   hipStream_t st)
{
    const int ng = tr_groups(K);
#define CHEM_TR_CASE(NG)                                                                                        \
    if (ng == NG)                                                                                               \
        return mu && D ? launch_group_mode<NG, 3>(table, K, T, p, Y, ldY, n, mu, lam, D, ldD, st)               \
               : mu    ? launch_group_mode<NG, 1>(table, K, T, p, Y, ldY, n, mu, lam, D, ldD, st)               \
                       : launch_group_mode<NG, 2>(table, K, T, p, Y, ldY, n, mu, lam, D, ldD, st);
    CHEM_TR_GROUPS(CHEM_TR_CASE)
#undef CHEM_TR_CASE
    return hipErrorInvalidValue;
}

// Host tables of the cell-per-lane kernels (diff: K x K x 5, symmetric).
std::vector<double> lane_tables(int K, const std::vector<double> &W, const double *visc, const double *cond,
                                const double *diff)
{
    const int L = tr_bound(K);
    const size_t LL = (size_t)L * L;
    std::vector<double> t(tr_table_len(L), 0.0);
    double *P = t.data(), *Q = P + 5 * L, *A = Q + 5 * L, *Bw = A + LL, *C = Bw + LL, *B = C + LL;
    double *iw = B + 5 * LL;
    for (int k = 0; k < L; k++) {
        P[5 * k] = Q[5 * k] = 1.0;   // padding rows: finite, and weighted by X = 0
        iw[k] = 1.0;
        for (int j = 0; j < L; j++) B[((size_t)k * L + j) * 5] = 1.0;
    }
    for (int k = 0; k < K; k++) {
        for (int c = 0; c < 5; c++) {
            P[5 * k + c] = visc[5 * k + c];
            Q[5 * k + c] = cond[5 * k + c];
        }
        iw[k] = 1.0 / W[k];
        for (int j = 0; j < K; j++) {
            const double c1 = std::pow(W[j] / W[k], 0.25), c2 = 1.0 / std::sqrt(8.0 * (1.0 + W[k] / W[j]));
            A[(size_t)k * L + j] = c2;
            Bw[(size_t)k * L + j] = 2.0 * c1 * c2;
            C[(size_t)k * L + j] = std::sqrt(W[j] / W[k]) * c2;
            for (int c = 0; c < 5; c++) B[((size_t)k * L + j) * 5 + c] = diff[((size_t)k * K + j) * 5 + c];
        }
    }
    return t;
}

// Host tables of the group kernels, in the lanes' operand orders.  Padding
// species have the fit 1, weight 1 and a zero mole fraction.
std::vector<double> group_tables(int K, const std::vector<double> &W, const double *visc, const double *cond,
                                 const double *diff)
{
    const int NG = tr_groups(K);
    std::vector<double> t((size_t)grp_head(NG) + grp_wilke(NG) + grp_pairs(NG), 0.0);
    for (int g = 0; g < NG; g++)
        for (int i = 0; i < 4; i++) {
            const int k = 4 * g + i;
            double *f = t.data() + kFitLen * g, *w = t.data() + kFitLen * NG;
            for (int c = 0; c < 4; c++) {
                f[c * 4 + i] = k < K ? visc[5 * k + c + 1] : 0.0;
                f[20 + c * 4 + i] = k < K ? cond[5 * k + c + 1] : 0.0;
            }
            f[16 + i] = k < K ? visc[5 * k] : 1.0;
            f[36 + i] = k < K ? cond[5 * k] : 1.0;
            w[4 * g + i] = k < K ? 1.0 / W[k] : 1.0;
            w[4 * NG + 4 * g + i] = k < K ? std::pow(W[k], -0.25) : 1.0;
        }
    double *M = t.data() + grp_head(NG);
    for (int g = 0; g < NG; g++)
        for (int G = 0; G < NG; G++)
            for (int q = 0; q < 4; q++)
                for (int i = 0; i < 4; i++) {
                    const int k = 4 * g + i, j = 4 * G + q;
                    M[(g * NG + G) * 16 + q * 4 + i] =
                        k < K && j < K ? 1.0 / std::sqrt(8.0 * (1.0 + W[k] / W[j])) : 1.0;
                }
    double *b = M + grp_wilke(NG);
    for (int G2 = 0; G2 < NG; G2++)
        for (int G1 = 0; G1 <= G2; G1++, b += kPairLen)
            for (int q = 0; q < 4; q++)
                for (int r = 0; r < 4; r++) {
                    const int j = 4 * G1 + q, k = 4 * G2 + r;
                    const double *a = j < K && k < K ? diff + ((size_t)k * K + j) * 5 : nullptr;
                    for (int c = 0; c < 4; c++) b[c * 16 + q + 4 * r] = a ? a[c + 1] : 0.0;
                    b[64 + 4 * q + r] = a ? a[0] : 1.0;
                }
    return t;
}

hipError_t launch_h_cp(const DevMechView &m, const double *T, const double *Y, int64_t ldY, int64_t n, double *h,
                       double *cp, hipStream_t st)
{
#define CHEM_TH_CASE(KM)                                                                                 \
    if (m.K <= KM) {                                                                                          \
        hipLaunchKernelGGL((h_cp_kernel<KM>), dim3(blocks_for(n)), dim3(kThermoBlock), 0, st, m.species,     \
                           m.invW, m.K, T, Y, ldY, n, h, cp);                                                 \
        return hipGetLastError();                                                                             \
    }
    CHEM_TR_BOUNDS(CHEM_TH_CASE)
#undef CHEM_TH_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_t_from_h(const DevMechView &m, const MidSet &ms, const double *h, const double *Y, int64_t ldY,
                           int64_t n, double *T, double *cp, int32_t *iters, int max_iter, double tol,
                           hipStream_t st)
{
#define CHEM_TN_CASE(KM)                                                                                 \
    if (m.K <= KM) {                                                                                          \
        if (m.K == KM)                                                                                        \
            hipLaunchKernelGGL((t_from_h_kernel<KM, true>), dim3(blocks_for(n)), dim3(kThermoBlock), 0, st,  \
                               m.species, m.invW, m.K, ms, h, Y, ldY, n, T, cp, iters, max_iter, tol);        \
        else                                                                                                  \
            hipLaunchKernelGGL((t_from_h_kernel<KM, false>), dim3(blocks_for(n)), dim3(kThermoBlock), 0, st, \
                               m.species, m.invW, m.K, ms, h, Y, ldY, n, T, cp, iters, max_iter, tol);        \
        return hipGetLastError();                                                                             \
    }
    CHEM_TR_BOUNDS(CHEM_TN_CASE)
#undef CHEM_TN_CASE
    return hipErrorInvalidValue;
}

}  // namespace
}  // namespace chem

namespace {

int check_field(chem_mech m, int64_t n, int64_t ldY)
{
    if (!m) return fail(CHEM_EINVAL, "mechanism handle is NULL");
    if (n < 0) return fail(CHEM_EINVAL, "ncells must be >= 0");
    if (n > 0 && ldY < n) return fail(CHEM_EINVAL, "ldY must be >= ncells");
    if (m->host.K > chem::kTrMaxK)
        return fail(CHEM_EUNSUP, "the property kernels hold at most " + std::to_string(chem::kTrMaxK) + " species");
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess || cur != m->device)
        return fail(CHEM_EINVAL, "the current HIP device is not the mechanism's device");
    return CHEM_OK;
}

bool dev_or_null(const void *p) { return p == nullptr || is_device_ptr(p); }

}  // namespace

extern "C" {

int chem_set_transport(chem_mech m, const double *visc, const double *cond, const double *diff)
{
    if (!m) return fail(CHEM_EINVAL, "mechanism handle is NULL");
    if (!visc || !cond || !diff) return fail(CHEM_EINVAL, "visc, cond and diff must be host arrays");
    const int K = m->host.K;
    if (K > chem::kTrMaxK)
        return fail(CHEM_EUNSUP, "the property kernels hold at most " + std::to_string(chem::kTrMaxK) + " species");
    for (int e = 0; e < 5 * K; e++)
        if (!std::isfinite(visc[e]) || !std::isfinite(cond[e]))
            return fail(CHEM_EINVAL, "transport fits must be finite");
    for (int k = 0; k < K; k++)
        for (int j = 0; j < K; j++)
            for (int c = 0; c < 5; c++) {
                const double a = diff[((size_t)k * K + j) * 5 + c];
                if (!std::isfinite(a)) return fail(CHEM_EINVAL, "transport fits must be finite");
                if (a != diff[((size_t)j * K + k) * 5 + c])
                    return fail(CHEM_EINVAL, "the binary diffusion fits must be symmetric in the two species");
            }
    const std::vector<double> t = K <= chem::kTrLaneMaxK ? chem::lane_tables(K, m->W, visc, cond, diff)
                                                         : chem::group_tables(K, m->W, visc, cond, diff);
    int prev = 0;
    if (hipGetDevice(&prev) != hipSuccess) return fail(CHEM_EHIP, "hipGetDevice failed");
    int rc = check_hip(hipSetDevice(m->device), "hipSetDevice");
    void *blk = nullptr;
    if (rc == CHEM_OK && hipMalloc(&blk, t.size() * sizeof(double)) != hipSuccess) {
        (void)hipGetLastError();
        rc = fail(CHEM_ENOMEM, "transport table allocation failed");
    }
    if (rc == CHEM_OK)
        rc = check_hip(hipMemcpy(blk, t.data(), t.size() * sizeof(double), hipMemcpyHostToDevice),
                       "transport table copy");
    if (rc == CHEM_OK) {
        if (m->transport_block) {
            hipDeviceSynchronize();   // earlier calls may still read the old table
            hipFree(m->transport_block);
        }
        m->transport_block = blk;
    } else if (blk) {
        hipFree(blk);
    }
    hipSetDevice(prev);
    return rc;
}

int chem_mixture_h_cp(chem_mech m, const double *T, const double *Y, int64_t ldY, int64_t n, double *h,
                      double *cp, void *stream)
{
    int rc = check_field(m, n, ldY);
    if (rc != CHEM_OK || n == 0) return rc;
    if (!is_device_ptr(T) || !is_device_ptr(Y) || !dev_or_null(h) || !dev_or_null(cp))
        return fail(CHEM_EINVAL, "T, Y, h and cp must be device pointers (h and cp may be NULL)");
    return check_hip(chem::launch_h_cp(m->view, T, Y, ldY, n, h, cp, (hipStream_t)stream), "h/cp launch");
}

int chem_T_from_h(chem_mech m, const double *h, const double *Y, int64_t ldY, int64_t n, double *T, double *cp,
                  int32_t *iters, int32_t max_iter, double tol, void *stream)
{
    int rc = check_field(m, n, ldY);
    if (rc != CHEM_OK) return rc;
    if (max_iter < 1 || max_iter > 1000) return fail(CHEM_EINVAL, "max_iter must be in 1 .. 1000");
    if (!(tol > 0.0) || !std::isfinite(tol)) return fail(CHEM_EINVAL, "tol must be positive and finite");
    if (n == 0) return CHEM_OK;
    if (!is_device_ptr(h) || !is_device_ptr(Y) || !is_device_ptr(T) || !dev_or_null(cp) || !dev_or_null(iters))
        return fail(CHEM_EINVAL, "h, Y, T, cp and iters must be device pointers (cp and iters may be NULL)");
    // the distinct range boundaries of the species with two distinct ranges
    chem::MidSet ms{};
    std::vector<double> mids;
    for (int k = 0; k < m->host.K; k++) {
        const double *a = &m->host.nasa[k][0];
        bool two = false;
        for (int j = 0; j < 7; j++) two = two || a[3 + j] != a[10 + j];
        if (two) mids.push_back(a[1]);
    }
    std::sort(mids.begin(), mids.end());
    mids.erase(std::unique(mids.begin(), mids.end()), mids.end());
    ms.nt = mids.size() <= (size_t)chem::kMaxMid ? (int32_t)mids.size() : -1;
    for (int q = 0; q < chem::kMaxMid && q < (int)mids.size(); q++) ms.t[q] = mids[q];
    return check_hip(chem::launch_t_from_h(m->view, ms, h, Y, ldY, n, T, cp, iters, max_iter, tol,
                                           (hipStream_t)stream),
                     "T-from-h launch");
}

int chem_transport_field(chem_mech m, const double *T, const double *p, const double *Y, int64_t ldY, int64_t n,
                         double *mu, double *lam, double *D, int64_t ldD, void *stream)
{
    int rc = check_field(m, n, ldY);
    if (rc != CHEM_OK) return rc;
    if (!m->transport_block) return fail(CHEM_EINVAL, "no transport data: call chem_set_transport first");
    if ((mu == nullptr) != (lam == nullptr)) return fail(CHEM_EINVAL, "mu and lam are given together or not at all");
    if (!mu && !D) return fail(CHEM_EINVAL, "nothing to compute: mu/lam and D are all NULL");
    if (n == 0) return CHEM_OK;
    if (D && ldD < n) return fail(CHEM_EINVAL, "ldD must be >= ncells");
    if (!is_device_ptr(T) || !is_device_ptr(Y) || (D && !is_device_ptr(p)) || !dev_or_null(mu) ||
        !dev_or_null(lam) || !dev_or_null(D))
        return fail(CHEM_EINVAL, "T, p, Y, mu, lam and D must be device pointers");
    const int K = m->host.K;
    const double *t = (const double *)m->transport_block;
    if (K > chem::kTrLaneMaxK)
        return check_hip(chem::launch_transport_groups(t, K, T, p, Y, ldY, n, mu, lam, D, ldD, (hipStream_t)stream),
                         "transport launch");
    const int L = chem::tr_bound(K);
    const size_t LL = (size_t)L * L;
    chem::TrView v{K, L, t, t + 5 * L, t + 10 * L, t + 10 * L + LL, t + 10 * L + 2 * LL, t + 10 * L + 3 * LL,
                   t + 10 * L + 8 * LL};
    return check_hip(chem::launch_transport(v, T, p, Y, ldY, n, mu, lam, D, ldD, (hipStream_t)stream),
                     "transport launch");
}

}  // extern "C"
