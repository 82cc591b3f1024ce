// The part of a beamlet's setup that its ray-transfer matrix, its waist and
// the plane's distance alone decide: the complex curvature and amplitude on
// the plane.  Where all beamlets share the three (one matrix, one waist, a
// plane normal to the axis) the host evaluates it once and the setup kernel
// takes it as an argument (812 beamlets 9.4 -> 8.4 us, 51,468 15.6 -> 14.6); a
// batch has it from one thread per instance (441 instances: setup 170 -> 146
// us).  Compiled for host and device alike without contraction, from
// operations that IEEE 754 rounds alike on both (+ - * / sqrt), so every path
// gives the same bits.
#pragma once

#include <cmath>
#include <cstdint>

namespace gbd {
namespace terms {

struct cx {
    double re, im;
};
#define GBD_HD __host__ __device__ inline
GBD_HD cx add(cx a, cx b) { return cx{a.re + b.re, a.im + b.im}; }
GBD_HD cx sub(cx a, cx b) { return cx{a.re - b.re, a.im - b.im}; }
GBD_HD cx scl(cx a, double s) { return cx{a.re * s, a.im * s}; }
GBD_HD cx mul(cx a, cx b) {
#pragma clang fp contract(off)
    return cx{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
GBD_HD double absd(double x) { return x < 0.0 ? -x : x; }
GBD_HD cx inverse(cx b) {
#pragma clang fp contract(off)
    // Smith's algorithm: no overflow for widely scaled operands
    if (absd(b.re) >= absd(b.im)) {
        const double r = b.im / b.re, d = b.re + b.im * r;
        return cx{1.0 / d, -r / d};
    }
    const double r = b.re / b.im, d = b.re * r + b.im;
    return cx{r / d, -1.0 / d};
}
GBD_HD double modulus(cx z) {
#pragma clang fp contract(off)
    const double a = absd(z.re), b = absd(z.im), m = a > b ? a : b;
    if (m > 1e-140 && m < 1e140) return sqrt(z.re * z.re + z.im * z.im);
    if (!(m > 0.0)) return a + b;  // zero, or not a number
    const double r = (a > b ? b : a) / m;
    return m * sqrt(1.0 + r * r);
}
// principal square root (cut on the negative real axis; the sign of a zero
// imaginary part picks the side)
GBD_HD cx root(cx z) {
#pragma clang fp contract(off)
    const double m = modulus(z);
    if (m == 0.0) return cx{0.0, z.im};
    if (z.re >= 0.0) {
        const double t = sqrt(0.5 * (m + z.re));
        return cx{t, z.im / (2.0 * t)};
    }
    const double t = sqrt(0.5 * (m - z.re));
    return cx{absd(z.im) / (2.0 * t), copysign(t, z.im)};
}
// Eigenvalues admitted on the principal-root branch: the open lower half
// plane and the positive real axis (reached from 1 without crossing the cut).
GBD_HD bool on_branch(cx mu) {
    const double m = modulus(mu);
    const double tol = 1e-12 * m;
    if (!(m > 0.0)) return false;
    if (mu.im > tol) return false;
    if (mu.im >= -tol && mu.re <= 0.0) return false;
    return true;
}

}  // namespace terms

struct MatrixTerms {
    terms::cx q00, q01, q11;  // Q^-1 law's complex curvature on the plane, symmetrised
    terms::cx gamma;          // det(Mm)^(-1/2) from the eigenvalues' principal roots
    uint32_t on_branch;       // both eigenvalues on the principal branch
};

// M [4][4] a ray-transfer matrix, z the free space behind it; Q1^-1 =
// -i kappa I, kappa = lambda / (pi w0^2).
GBD_HD MatrixTerms matrix_terms(const double *M, double z, double lambda, double w0) {
#pragma clang fp contract(off)
    using namespace terms;
    const double kappa = lambda / (3.14159265358979323846 * w0 * w0);
    cx Mm[2][2], Nm[2][2];
    for (int r = 0; r < 2; r++)
        for (int c = 0; c < 2; c++) {
            const double A = M[4 * r + c], B = M[4 * r + c + 2], C = M[4 * (r + 2) + c], D = M[4 * (r + 2) + c + 2];
            Mm[r][c] = cx{A + z * C, -kappa * (B + z * D)};
            Nm[r][c] = cx{C, -kappa * D};
        }
    // complex-curvature law Q^-1 = Nm Mm^-1 (closed-form 2x2 inverse)
    const cx det = sub(mul(Mm[0][0], Mm[1][1]), mul(Mm[0][1], Mm[1][0]));
    const cx inv = inverse(det);
    const cx i00 = mul(Mm[1][1], inv), i11 = mul(Mm[0][0], inv), i01 = mul(scl(Mm[0][1], -1.0), inv),
             i10 = mul(scl(Mm[1][0], -1.0), inv);
    MatrixTerms t;
    t.q00 = add(mul(Nm[0][0], i00), mul(Nm[0][1], i10));
    t.q11 = add(mul(Nm[1][0], i01), mul(Nm[1][1], i11));
    t.q01 = scl(add(add(mul(Nm[0][0], i01), mul(Nm[0][1], i11)), add(mul(Nm[1][0], i00), mul(Nm[1][1], i10))), 0.5);
    const cx tr = add(Mm[0][0], Mm[1][1]);
    const cx disc = root(sub(mul(tr, tr), scl(det, 4.0)));
    const cx mu1 = scl(add(tr, disc), 0.5), mu2 = scl(sub(tr, disc), 0.5);
    t.on_branch = on_branch(mu1) && on_branch(mu2) ? 1u : 0u;
    t.gamma = inverse(mul(root(mu1), root(mu2)));
    return t;
}
#undef GBD_HD

}  // namespace gbd
