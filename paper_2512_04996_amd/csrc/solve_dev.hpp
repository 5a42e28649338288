// solve_dev.hpp -- the closed-form rigid transform of Eq. 1 from its moments
// (float64, one lane), shared by the solve kernel (k_solve.hip) and the
// resident registration loop (k_loop.hip).
#pragma once

#include <math.h>

#include "vicp_internal.hpp"

namespace vicp {

namespace {

__host__ __device__ void svd3(double A[3][3], double U[3][3], double sig[3], double V[3][3])
{
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) V[i][j] = (i == j) ? 1.0 : 0.0;
    // one-sided Jacobi: rotate column pairs of A until they are orthogonal
    for (int sweep = 0; sweep < 16; ++sweep) {
        double worst = 0.0;
        for (int p = 0; p < 2; ++p) {
            for (int q = p + 1; q < 3; ++q) {
                double al = 0.0, be = 0.0, ga = 0.0;
                for (int r = 0; r < 3; ++r) {
                    al += A[r][p] * A[r][p];
                    be += A[r][q] * A[r][q];
                    ga += A[r][p] * A[r][q];
                }
                if (ga == 0.0) continue;
                const double rel = fabs(ga) / sqrt(al * be);
                worst = fmax(worst, rel);
                if (!(rel > 1e-15)) continue;
                const double zeta = (be - al) / (2.0 * ga);
                const double t = copysign(1.0, zeta) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
                const double c = 1.0 / sqrt(1.0 + t * t), s = c * t;
                for (int r = 0; r < 3; ++r) {
                    const double ap = A[r][p], aq = A[r][q];
                    A[r][p] = c * ap - s * aq;
                    A[r][q] = s * ap + c * aq;
                    const double vp = V[r][p], vq = V[r][q];
                    V[r][p] = c * vp - s * vq;
                    V[r][q] = s * vp + c * vq;
                }
            }
        }
        if (!(worst > 1e-15)) break;
    }
    for (int j = 0; j < 3; ++j) {
        double nrm = 0.0;
        for (int r = 0; r < 3; ++r) nrm += A[r][j] * A[r][j];
        sig[j] = sqrt(nrm);
    }
    // order by decreasing singular value (columns of A and V move together)
    for (int a = 0; a < 3; ++a)
        for (int b = a + 1; b < 3; ++b)
            if (sig[b] > sig[a]) {
                const double ts = sig[a];
                sig[a] = sig[b];
                sig[b] = ts;
                for (int r = 0; r < 3; ++r) {
                    double t = A[r][a];
                    A[r][a] = A[r][b];
                    A[r][b] = t;
                    t = V[r][a];
                    V[r][a] = V[r][b];
                    V[r][b] = t;
                }
            }
    for (int j = 0; j < 2; ++j)
        for (int r = 0; r < 3; ++r) U[r][j] = sig[j] > 0.0 ? A[r][j] / sig[j] : 0.0;
    if (sig[2] > 1e-13 * sig[0]) {
        for (int r = 0; r < 3; ++r) U[r][2] = A[r][2] / sig[2];
    } else {
        // complete the basis: the third left vector of a rank-2 H is free
        U[0][2] = U[1][0] * U[2][1] - U[2][0] * U[1][1];
        U[1][2] = U[2][0] * U[0][1] - U[0][0] * U[2][1];
        U[2][2] = U[0][0] * U[1][1] - U[1][0] * U[0][1];
    }
}

__host__ __device__ double det3(const double M[3][3])
{
    return M[0][0] * (M[1][1] * M[2][2] - M[1][2] * M[2][1]) - M[0][1] * (M[1][0] * M[2][2] - M[1][2] * M[2][0]) +
           M[0][2] * (M[1][0] * M[2][1] - M[1][1] * M[2][0]);
}

// Orthogonal polar factor of a well-conditioned 3x3 matrix by the scaled
// Newton iteration X <- (g X + X^{-T} / g) / 2 (Frobenius-norm scaling while
// far from convergence).  X starts as A / ||A||_F (the polar factor does not
// change), so every quantity is of order one and the scale g, which only
// speeds convergence, is computed in float32.  Returns false when X becomes
// singular or the iteration does not settle; the caller then uses the SVD.
__host__ __device__ bool polar3(const double A[3][3], double Q[3][3])
{
    // float64 only and compared within tolerance: fused multiply-adds allowed
    // (the float32 search keeps every rounding as written)
#pragma clang fp contract(fast)
    double X[3][3];
    double na = 0.0;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) na += A[i][j] * A[i][j];
    if (!(na > 0.0)) return false;
    const double inv = 1.0 / sqrt(na);
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) X[i][j] = A[i][j] * inv;
    bool scale = true;
    for (int it = 0; it < 24; ++it) {
        double C[3][3];   // cofactors: X^{-T} = C / det
        C[0][0] = X[1][1] * X[2][2] - X[1][2] * X[2][1];
        C[0][1] = X[1][2] * X[2][0] - X[1][0] * X[2][2];
        C[0][2] = X[1][0] * X[2][1] - X[1][1] * X[2][0];
        C[1][0] = X[0][2] * X[2][1] - X[0][1] * X[2][2];
        C[1][1] = X[0][0] * X[2][2] - X[0][2] * X[2][0];
        C[1][2] = X[0][1] * X[2][0] - X[0][0] * X[2][1];
        C[2][0] = X[0][1] * X[1][2] - X[0][2] * X[1][1];
        C[2][1] = X[0][2] * X[1][0] - X[0][0] * X[1][2];
        C[2][2] = X[0][0] * X[1][1] - X[0][1] * X[1][0];
        const double det = X[0][0] * C[0][0] + X[0][1] * C[0][1] + X[0][2] * C[0][2];
        if (!(det > 0.0)) return false;
        double nx = 0.0, nc = 0.0;
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) {
                nx += X[i][j] * X[i][j];
                nc += C[i][j] * C[i][j];
            }
        const double g = scale ? (double)sqrtf(sqrtf((float)nc) / ((float)det * sqrtf((float)nx))) : 1.0;
        const double a = 0.5 * g, b = 0.5 / (g * det);
        double diff = 0.0;
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) {
                const double v = a * X[i][j] + b * C[i][j];
                diff += (v - X[i][j]) * (v - X[i][j]);
                X[i][j] = v;
            }
        if (diff < 1e-4) scale = false;
        // quadratic convergence: after a step of size below 1e-8 the new
        // iterate is within rounding of the polar factor
        if (diff < 1e-16) {
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) Q[i][j] = X[i][j];
            return true;
        }
    }
    return false;
}

// 1/x in the float64 solve.  On the device: the hardware reciprocal refined
// by two Newton steps, a chain of five operations instead of the ten or so
// of a correctly rounded division (the result is within an ulp or two; the
// solve is compared within tolerance).  On the host: a division.
__host__ __device__ __forceinline__ double recip(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
#else
    return 1.0 / x;
#endif
}

// Roughly 1/sqrt(x), for a scale factor whose exact value does not matter.
__host__ __device__ __forceinline__ double rough_rsqrt(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_rsq(x);
#else
    return 1.0 / sqrt(x);
#endif
}

// True when the rotation part of Q (row-major 3x3) is orthogonal to 1e-12.
__host__ __device__ bool rot_orthogonal(const double* Q)
{
    double orth = 0.0;
    for (int i = 0; i < 3; ++i)
        for (int j = i; j < 3; ++j) {
            const double d = Q[i] * Q[j] + Q[3 + i] * Q[3 + j] + Q[6 + i] * Q[6 + j] - (i == j ? 1.0 : 0.0);
            orth = fmax(orth, fabs(d));
        }
    return orth < 1e-12;
}

// Orthogonal polar factor of A refined from a nearby rotation Q0 (the
// previous pose's rotation, orthogonal): with M = R^T A, the rotation
// increment exp([w]x) that makes M symmetric solves (tr(S) I - S) w =
// 2 axial(skew M) to first order, S = sym(M); it is applied as the Cayley
// rotation of w (exactly orthogonal), and the step repeats until |w| < 1e-8
// (the error then is at rounding: the convergence is cubic, two steps from
// the previous pose of an ICP iteration).  A is scaled by any positive
// factor (the polar factor does not change) to keep the products of order
// one.  Accepted only if the final S is positive definite (so R is the polar
// factor, not another stationary point); otherwise returns false.
__host__ __device__ bool polar_refine(const double A[3][3], double scale, const double Q0[3][3], double Q[3][3])
{
    // float64 only and compared within tolerance: fused multiply-adds allowed
    // (the float32 search keeps every rounding as written)
#pragma clang fp contract(fast)
    double R[3][3], An[3][3];
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            R[i][j] = Q0[i][j];
            An[i][j] = A[i][j] * scale;
        }
#pragma unroll 1
    for (int it = 0; it < 8; ++it) {
        double M[3][3];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) M[i][j] = R[0][i] * An[0][j] + R[1][i] * An[1][j] + R[2][i] * An[2][j];
        const double s00 = M[0][0], s11 = M[1][1], s22 = M[2][2];
        const double s01 = 0.5 * (M[0][1] + M[1][0]), s02 = 0.5 * (M[0][2] + M[2][0]), s12 = 0.5 * (M[1][2] + M[2][1]);
        const double k[3] = {M[2][1] - M[1][2], M[0][2] - M[2][0], M[1][0] - M[0][1]};   // 2 axial(skew M)
        // T = tr(S) I - S is symmetric: w = adj(T) k / det T
        const double t00 = s11 + s22, t11 = s00 + s22, t22 = s00 + s11;
        const double a00 = t11 * t22 - s12 * s12, a01 = s02 * s12 + s01 * t22, a02 = s01 * s12 + s02 * t11;
        const double a11 = t00 * t22 - s02 * s02, a12 = s01 * s02 + t00 * s12, a22 = t00 * t11 - s01 * s01;
        const double dT = t00 * a00 - s01 * a01 - s02 * a02;
        if (!(dT > 0.0)) return false;
        const double idT = recip(dT);
        const double w0 = (a00 * k[0] + a01 * k[1] + a02 * k[2]) * idT;
        const double w1 = (a01 * k[0] + a11 * k[1] + a12 * k[2]) * idT;
        const double w2 = (a02 * k[0] + a12 * k[1] + a22 * k[2]) * idT;
        const double ww = w0 * w0 + w1 * w1 + w2 * w2;
        // Cayley rotation of w with h = w / 2: I + f ([h]x + h h^T - |h|^2 I),
        // f = 2 / (1 + |h|^2)
        const double h0 = 0.5 * w0, h1 = 0.5 * w1, h2 = 0.5 * w2;
        const double f = 2.0 * recip(1.0 + 0.25 * ww);
        const double h01 = h0 * h1, h02 = h0 * h2, h12 = h1 * h2;
        const double D[3][3] = {{1.0 - f * (h1 * h1 + h2 * h2), f * (h01 - h2), f * (h02 + h1)},
                                {f * (h01 + h2), 1.0 - f * (h0 * h0 + h2 * h2), f * (h12 - h0)},
                                {f * (h02 - h1), f * (h12 + h0), 1.0 - f * (h0 * h0 + h1 * h1)}};
        double Rn[3][3];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) Rn[i][j] = R[i][0] * D[0][j] + R[i][1] * D[1][j] + R[i][2] * D[2][j];
        for (int i = 0; i < 3; ++i)
            for (int j = 0; j < 3; ++j) R[i][j] = Rn[i][j];
        if (ww < 1e-16) {
            // S positive definite: its leading minors are positive
            const bool pd = s00 > 0.0 && s00 * s11 - s01 * s01 > 0.0 &&
                            s00 * (s11 * s22 - s12 * s12) - s01 * (s01 * s22 - s12 * s02) +
                                    s02 * (s01 * s12 - s11 * s02) > 0.0;
            if (!pd) return false;
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) Q[i][j] = R[i][j];
            return true;
        }
    }
    return false;
}

// Moments about the centre c (sum p, sum q, sum p q^T, sum |p|^2, sum |q|^2,
// sum d, count); returns false (pose untouched)
// when H has rank < 2: its second singular value is below 1e-12 of the first
// or below the rounding floor of the one-pass sums, 1e-13 sqrt(sum|p|^2 sum|q|^2)
// (taken about c), so that a cross-covariance made of rounding noise (e.g.
// every correspondence on one target point) never yields a rotation.
// Rprev (row-major, may be null): the previous rotation, from which the polar
// factor is refined; prev_orth says it is known to be orthogonal (a previous
// solve's result), otherwise it is checked here.  In two halves: the rotation
// R (row-major; the refinement can be asked for alone, false also where it does
// not apply, and what follows it alone where it does not),
enum SolveStep { kSolveAll, kRefine, kAfterRefine };
template <SolveStep kStep>
__host__ __device__ __forceinline__ bool kabsch_rotation(const double* mom, const double* Rprev, bool prev_orth,
                                                         double* Rrow)
{
    // float64 only and compared within tolerance: fused multiply-adds allowed
    // (the float32 search keeps every rounding as written)
#pragma clang fp contract(fast)
    const double m = mom[18];
    if (!(m > 0.0)) return false;
    double pb[3], qb[3], H[3][3];
    const double im = recip(m);
    for (int a = 0; a < 3; ++a) {
        pb[a] = mom[a] * im;
        qb[a] = mom[3 + a] * im;
    }
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) H[a][b] = mom[6 + 3 * a + b] - m * pb[a] * qb[b];
    const double pq = mom[15] * mom[16];
    double R[3][3];
    // R = V U^T is the orthogonal polar factor of H^T (H^T = V S U^T =
    // (V U^T)(U S U^T)); when H is far above the rounding floor and det H is
    // clearly positive, no reflection fix is needed: the polar factor is
    // refined from the previous rotation, or else taken by the Newton polar
    // iteration.  The tests ||H|| > 1e6 floor and det H > 1e-6 ||H||^3 are
    // taken on squares (no square root on the way to the refinement).
    double Ht[3][3], nh = 0.0;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            Ht[i][j] = H[j][i];
            nh += H[i][j] * H[i][j];
        }
    const double dH = det3(Ht);
    const bool well = nh > 1e-14 * pq && dH > 0.0 && dH * dH > 1e-12 * nh * nh * nh;
    bool fast = false;
    if (kStep != kAfterRefine && well && Rprev && (prev_orth || rot_orthogonal(Rprev))) {
        const double Q0[3][3] = {{Rprev[0], Rprev[1], Rprev[2]}, {Rprev[3], Rprev[4], Rprev[5]},
                                 {Rprev[6], Rprev[7], Rprev[8]}};
        fast = polar_refine(Ht, rough_rsqrt(nh), Q0, R);
    }
    if (!fast) {
        if (kStep == kRefine) return false;
        if (!(well && polar3(Ht, R))) {
            const double floor_ = 1e-13 * sqrt(pq);
            double U[3][3], sig[3], V[3][3];
            svd3(H, U, sig, V);
            if (!(sig[0] > 0.0) || sig[1] <= 1e-12 * sig[0] || sig[1] <= floor_) return false;
            const double d = (det3(U) * det3(V) < 0.0) ? -1.0 : 1.0;
            for (int i = 0; i < 3; ++i)
                for (int j = 0; j < 3; ++j) R[i][j] = V[i][0] * U[j][0] + V[i][1] * U[j][1] + d * V[i][2] * U[j][2];
        }
    }
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) Rrow[3 * i + j] = R[i][j];
    return true;
}

// and its translation: t = qbar - R pbar with the means taken back from c.
__host__ __device__ __forceinline__ void kabsch_translation(const double* mom, const double c[3], const double* R,
                                                            double* t)
{
#pragma clang fp contract(fast)
    const double im = recip(mom[18]);
    for (int i = 0; i < 3; ++i) {
        const double rp = R[3 * i] * (mom[0] * im + c[0]) + R[3 * i + 1] * (mom[1] * im + c[1]) +
                          R[3 * i + 2] * (mom[2] * im + c[2]);
        t[i] = (mom[3 + i] * im + c[i]) - rp;
    }
}

__host__ __device__ __forceinline__ bool kabsch(const double* mom, const double c[3], double Rt[12],
                                                const double* Rprev, bool prev_orth)
{
    double R[9];
    if (!kabsch_rotation<kSolveAll>(mom, Rprev, prev_orth, R)) return false;
    for (int i = 0; i < 9; ++i) Rt[i] = R[i];
    kabsch_translation(mom, c, R, Rt + 9);
    return true;
}

}  // namespace

}  // namespace vicp
