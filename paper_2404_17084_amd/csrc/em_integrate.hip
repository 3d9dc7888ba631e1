// Integration of the M4 kernel over each (particle, cell) pair, Sec. II-B.
//
// Far-field-subtracted form.  With lengths in units of h, the kernel mass in
// a cone of directions up to radius s is F(s) per steradian, F(s) -> 1/(4 pi)
// for s >= 2.  Writing F = 1/(4 pi) - F_c splits each vertex-pyramid integral
// into a solid-angle part and a remainder that vanishes beyond the support:
//     I(r0, R0, phi) = Omega/(4 pi) - [ Q(phi) - phi H(r0) ],
//     Q(phi) = r0 int_0^phi G_c(S(alpha)) dalpha,   H(r0) = r0 G_c(r0),
// where G_c' = F_c/s^2, G_c = 0 for s >= 2, and S(alpha) is the distance from
// the particle to the edge line's point at in-plane angle alpha.  Summed with
// the signs of the signed-cone decomposition, the solid-angle parts give the
// winding number of the cell about the particle (1 inside, 0 outside), so
//     f = [p inside] - (1/pi) sum_faces sigma_j { sum_edges sign(rho) [Q(l_b) - Q(l_a)] - pi H(r0) A_j },
// with A_j the signed angle the face's edges subtend at the foot point, and
// the per-edge Q difference taken along the edge (signed coordinate l from
// the foot g of the projection point on the edge line).  Walls with r0 >= 2
// and edges whose line lies beyond 2h contribute nothing to Q; such walls are
// skipped entirely.
//
// pi G_c as polynomials in s (exponents -1, 0, 2, 3, 4, 5):
//   s <= 1:      -1/(4s) + 7/20 - s^2/6 + 3 s^4/40 - s^5/40
//   1 <= s <= 2: -4/(15s) + 2/5 - s^2/3 + s^3/4 - 3 s^4/40 + s^5/120
//              = -(2 - s)^5 (s + 1) / (120 s)
// and the angular moments P_n = int S^n dalpha are evaluated in closed form
// from l (t = l/R0, S = sqrt(c^2 + l^2), c^2 = r0^2 + R0^2):
//   r0 P_-1 = atan2(r0 l, R0 S),  P_0 = atan2(l, R0),  P_2 = r0^2 P_0 + R0 l,
//   P_3 = (R0 l S + R0 c^2 a)/2 + r0^2 R0 a + r0^3 (r0 P_-1),  a = asinh(l/c),
//   P_4 = r0^4 P_0 + 2 r0^2 R0 l + R0^3 l + R0 l^3/3,
//   P_5 = R0 l (S^3/4 + 3 c^2 S/8) + 3 R0 c^4 a/8 + r0^2 P_3.
// The M4 piece radii s = 1, 2 split the edge at l_k = sqrt(k^2 - c^2).
#include <cmath>

#include "em_internal.h"
#include "em_boundary.h"
#include "em_fmath.h"
#include "em_wave.h"

namespace em {

namespace {

// Work counters of one thread (feed the algorithmic flop model).
struct Work {
    unsigned faces = 0, edges = 0, eterms = 0, moments = 0, quads = 0, angles = 0, qpoints = 0;
};

// pi * H(r0) = pi * r0 * G_c(r0)
template <typename R>
__device__ __forceinline__ R pi_H(R r0)
{
    if (r0 <= R(1)) {
        R r2 = r0 * r0;
        R r3 = r2 * r0;
        return R(0.35) * r0 - R(0.25) - r3 * R(1.0 / 6.0) + R(0.075) * r3 * r2 - R(0.025) * r3 * r3;
    }
    R u = R(2) - r0;
    R u2 = u * u;
    return -(u2 * u2 * u) * (r0 + R(1)) * R(1.0 / 120.0);
}

// pi r0 (G_shell - G_inner)(r0) = (r0 - 1)^5 (2 r0 + 1) / 60 (zero for r0 >= 1, where G_c is the shell polynomial)
template <typename R>
__device__ __forceinline__ R pi_dH(R r0)
{
    if (!(r0 < R(1))) return R(0);
    R u = r0 - R(1);
    R u2 = u * u;
    return u2 * u2 * u * (R(2) * r0 + R(1)) * R(1.0 / 60.0);
}

// angle atan(b/R0) - atan(a/R0) subtended at the foot point by the part [a, b] of the edge line
__device__ __forceinline__ float seg_angle(float R0, float a, float b, Work &wk)
{
    wk.angles++;
    return atan2_f32(R0 * (b - a), R0 * R0 + a * b);
}

// Transcendentals of the FP32 closed form at x >= 0 with S = sqrt(c^2 + x^2):
//   a = asinh(x/c), beta = P_0 - r0 P_-1 = atan(x/R0) - atan(r0 x/(R0 S)).
struct Trans {
    float x, S, a, beta;
};

__device__ __forceinline__ Trans trans(float r0, float R0, float c2, float c, float x, float S, Work &wk)
{
    wk.moments++;
    Trans t;
    t.x = x;
    t.S = S;
    t.a = log1p_f32(x * (1.0f + x * rcp_f32(S + c)) * rcp_f32(c));
    const float R02 = R0 * R0;
    t.beta = atan2_f32(x * R0 * (R02 + x * x), (S + r0) * (R02 * S + r0 * x * x));
    return t;
}

// Closed form of pi r0 int_0^alpha(x) [G_p(S) - G_p(r0)] dalpha for the piece
// polynomial pi G_p = g_-1/s + g_0 + g_2 s^2 + g_3 s^3 + g_4 s^4 + g_5 s^5:
//   -beta H_odd + r0 R0 T,  H_odd = g_-1 + g_3 r0^4 + g_5 r0^6,
//   T = g_2 x + g_3 P3' + g_4 (2 r0^2 x + R0^2 x + x^3/3)
//       + g_5 (x (S^3/4 + 3 c^2 S/8) + 3 c^4 a/8 + r0^2 P3'),
//   P3' = (x S + c^2 a)/2 + r0^2 a.
// FP32, the inner piece only (g_3 = 0).
__device__ __forceinline__ float core_inner(const Trans &t, float r0, float R0, float A, float c2)
{
    const float gm1 = -0.25f, g2 = -1.0f / 6.0f, g3 = 0.0f, g4 = 0.075f, g5 = -0.025f;
    const float x = t.x, S = t.S, a = t.a;
    const float Hodd = gm1 + g3 * A * A + g5 * A * A * A;
    const float P3r = 0.5f * (x * S + c2 * a) + A * a;
    const float T = g2 * x + g3 * P3r + g4 * (2.0f * A * x + R0 * R0 * x + x * x * x * (1.0f / 3.0f)) +
                    g5 * (x * (S * S * S * 0.25f + 0.375f * c2 * S) + 0.375f * c2 * c2 * a + A * P3r);
    return -t.beta * Hodd + r0 * R0 * T;
}

__constant__ float kGLx[4] = {0.1834346424956498f, 0.5255324099163290f, 0.7966664774136267f, 0.9602898564975363f};
__constant__ float kGLw[4] = {0.3626837833783620f, 0.3137066458778873f, 0.2223810344533745f, 0.1012285362903763f};

__device__ __forceinline__ float rcp32(float x) { return __builtin_amdgcn_rcpf(x); }

// shell piece by Gauss-Legendre:  pi r0 R0 int_a^b D_shell(R0^2 + l^2) dl,  a < b.
// 8 points per sub-interval, sub-intervals at most 0.8 dsing long (dsing: a
// lower bound of the distance from the part to the integrand's branch points
// l = +-ic), so the branch points stay outside the Bernstein ellipse of
// parameter 2.5 + sqrt(7.25) of every sub-interval and the truncation is far
// below the FP32 rounding of the term.
__device__ __forceinline__ float shell_quad(float r0, float R0, float c2, float dsing, float a, float b, Work &wk)
{
    const float V = 2.0f - r0;
    const float V2 = V * V, V4 = V2 * V2, V5 = V4 * V;
    const float rp1 = r0 + 1.0f;
    const float len = b - a;
    int nsub = (int)ceilf(len * rcp32(0.8f * dsing));
    nsub = nsub < 1 ? 1 : (nsub > 8 ? 8 : nsub);
    const float hl = 0.5f * len * rcp_f32((float)nsub);
    float tot = 0.0f;
    for (int k = 0; k < nsub; k++) {
        const float mid = a + (2.0f * (float)k + 1.0f) * hl;
        float acc = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; q++) {
            const float xq = (q & 1) ? -kGLx[q >> 1] : kGLx[q >> 1];
            const float l = mid + hl * xq;
            const float S = sqrt_f32(c2 + l * l);
            const float U = 2.0f - S;
            const float U2 = U * U;
            const float Sig = (((U + V) * U + V2) * U + V2 * V) * U + V4;
            const float num = rp1 * (r0 * Sig + V5) - r0 * U2 * U2 * U;
            acc += kGLw[q >> 1] * num * rcp32(S * (S + r0));
        }
        tot += acc * hl;
    }
    wk.quads += nsub;
    wk.qpoints += 8 * nsub;
    return tot * R0 * (1.0f / 120.0f);
}

// pi [Qt(l_b) - Qt(l_a)] for one directed edge (R0 > 0), lengths in units of h:
// the edge's whole share of pi int (G_c(S) - G_c(r0)) dalpha.  The signed edge
// interval is cut at the support crossings +-l2 and (when c < 1) the inner
// crossings +-l1 into parts beyond the support (-H times their angle), shell
// parts and an inner part, plus the piece correction dH times the angle of the
// shell parts when r0 < 1.
//
// FP32 form (distributions 0-2 of the mixed path): all cases are expressed as
// one fixed list of tasks - up to 4 angles, 3 closed-form points of the inner
// piece (|l_a|, |l_b| clamped, and l1) and 2 quadrature intervals of the shell
// piece - so that the lanes of a wavefront, which hold different particles, run
// each task type in the same code instead of one branch per geometric case.
__device__ __forceinline__ float sgnr(float x) { return x > 0.0f ? 1.0f : (x < 0.0f ? -1.0f : 0.0f); }

__device__ __forceinline__ float edge_term(float r0, float R0, float la, float lb, float, float Ht, float dH, Work &wk)
{
    const float A = r0 * r0;
    const float c2 = A + R0 * R0;
    // angle tasks: (a, b, weight)
    float aa0 = la, ab0 = lb, aw0 = 0.0f, aa1 = 0.0f, ab1 = 0.0f, aw1 = 0.0f;
    float aa2 = 0.0f, ab2 = 0.0f, aw2 = 0.0f, aa3 = 0.0f, ab3 = 0.0f, aw3 = 0.0f;
    // closed-form point weights at |ca|, |cb| and l1
    float wi0 = 0.0f, wi1 = 0.0f, wi2 = 0.0f;
    // quadrature intervals
    float qa0 = 0.0f, qb0 = 0.0f, qa1 = 0.0f, qb1 = 0.0f;
    bool q0 = false, q1 = false;
    float l2 = 0.0f, c = 1.0f, l1 = 0.0f, ca = la, cb = lb;
    if (!(c2 < 4.0f)) {
        aw0 = -Ht;  // the whole edge lies beyond the support
    } else {
        wk.eterms++;
        l2 = sqrt_f32(4.0f - c2);
        c = sqrt_f32(c2);
        ca = fmin(fmax(la, -l2), l2);
        cb = fmin(fmax(lb, -l2), l2);
        if (la < -l2) {
            aw0 = -Ht;
            ab0 = fmin(lb, -l2);
        }
        if (lb > l2) {
            aa1 = fmax(la, l2);
            ab1 = lb;
            aw1 = -Ht;
        }
        if (c2 >= 1.0f) {
            if (cb > ca) {
                q0 = true;
                qa0 = ca;
                qb0 = cb;
                aa2 = ca;
                ab2 = cb;
                aw2 = dH;
            }
        } else {
            l1 = sqrt_f32(1.0f - c2);
            // left shell part [max(ca, -l2), min(cb, -l1)]
            if (ca < -l1) {
                q0 = true;
                qa0 = ca;
                qb0 = fmin(cb, -l1);
                aa2 = ca;
                ab2 = qb0;
                aw2 = dH;
            }
            // right shell part [max(ca, l1), min(cb, l2)]
            if (cb > l1) {
                q1 = true;
                qa1 = fmax(ca, l1);
                qb1 = cb;
                aa3 = qa1;
                ab3 = cb;
                aw3 = dH;
            }
            // inner part [max(ca, -l1), min(cb, l1)]
            const float Ai = fmax(ca, -l1), Bi = fmin(cb, l1);
            if (Bi > Ai) {
                if (Bi == cb) wi1 += sgnr(cb);
                else wi2 += 1.0f;  // B = +l1
                if (Ai == ca) wi0 -= sgnr(ca);
                else wi2 += 1.0f;  // A = -l1: -sgn(A) core(l1) = +core(l1)
            }
        }
    }
    float tot = 0.0f;
    if (aw0 != 0.0f) tot += aw0 * seg_angle(R0, aa0, ab0, wk);
    if (aw1 != 0.0f) tot += aw1 * seg_angle(R0, aa1, ab1, wk);
    if (aw2 != 0.0f) tot += aw2 * seg_angle(R0, aa2, ab2, wk);
    if (aw3 != 0.0f) tot += aw3 * seg_angle(R0, aa3, ab3, wk);
    const float x0 = fabsf(ca), x1 = fabsf(cb);
    if (wi0 != 0.0f && x0 > 0.0f) {
        const Trans t = trans(r0, R0, c2, c, x0, x0 == l2 ? 2.0f : sqrt_f32(c2 + x0 * x0), wk);
        tot += wi0 * core_inner(t, r0, R0, A, c2);
    }
    if (wi1 != 0.0f && x1 > 0.0f) {
        const Trans t = trans(r0, R0, c2, c, x1, x1 == l2 ? 2.0f : sqrt_f32(c2 + x1 * x1), wk);
        tot += wi1 * core_inner(t, r0, R0, A, c2);
    }
    if (wi2 != 0.0f) {
        const Trans t = trans(r0, R0, c2, c, l1, 1.0f, wk);
        tot += wi2 * core_inner(t, r0, R0, A, c2);
    }
    if (q0) tot += shell_quad(r0, R0, c2, c2 >= 1.0f ? c : 1.0f, qa0, qb0, wk);
    if (q1) tot += shell_quad(r0, R0, c2, 1.0f, qa1, qb1, wk);
    return tot;
}

// ---------------------------------------------------------------- FP64 edge terms
// The parts of an edge [la, lb]: beyond the support [la, ca] + [cb, lb], shell
// [ca, ia] + [ib, cb], inner [ia, ib], every part oriented and possibly empty.
// Far edges (c >= 2) are all beyond (l2 = 0).
struct EdgeParts {
    double ca, cb, ia, ib;
    bool near, inner;
};

__device__ __forceinline__ EdgeParts edge_parts(bool live, double r0, double R0, double la, double lb)
{
    EdgeParts P;
    const double c2 = fma(R0, R0, r0 * r0);
    P.near = live && c2 < 4.0;
    P.inner = P.near && c2 < 1.0;
    const double l2 = P.near ? sqrt_f64(4.0 - c2) : 0.0;
    // min(max(x, lo), hi) of la <= lb: the median of three also when lo > hi
    P.ca = fmin(fmax(la, -l2), lb);
    P.cb = fmax(P.ca, fmin(l2, lb));
    P.ia = P.cb;
    P.ib = P.cb;
    if (P.inner) {
        const double l1 = sqrt_f64(1.0 - c2);
        P.ia = fmin(fmax(P.ca, -l1), P.cb);
        P.ib = fmax(P.ia, fmin(l1, P.cb));
    }
    return P;
}

// Length of the part [x, y]: the edge length from the edge record when the
// part is the whole edge (the difference of its ends would lose digits of a
// short edge far from the foot point), else the difference (a clipped end sits
// on a kernel sphere, where an end shift changes the integral only to second
// order).
__device__ __forceinline__ double part_len(double x, double y, double la, double lb, double Le)
{
    return (x == la && y == lb) ? Le : y - x;
}

// The angle of two parts [a1, b1], [a2, b2] at the foot point as the argument
// of the product of their complex numbers (R0^2 + a b) + i R0 (b - a) (the sum
// stays below pi).  Lengths below kFarLength.
__device__ __forceinline__ void angle_product(double R0, double a1, double b1, double a2, double b2, double &y,
                                              double &x)
{
    const double R02 = R0 * R0;
    const double x1 = fma(a1, b1, R02), y1 = R0 * (b1 - a1), x2 = fma(a2, b2, R02), y2 = R0 * (b2 - a2);
    x = fma(x1, x2, -(y1 * y2));
    y = fma(x1, y2, x2 * y1);
}

// The same for an edge that may reach further from the foot point (in units of
// h: a cell so much larger than the support): the product would overflow, so
// the numbers are scaled down first.
constexpr double kFarLength = 0x1p250;

__device__ __forceinline__ void angle_product_far(double R0, double a1, double b1, double a2, double b2, double &y,
                                                  double &x)
{
    const double R02 = R0 * R0;
    double x1 = fma(a1, b1, R02), y1 = R0 * (b1 - a1), x2 = fma(a2, b2, R02), y2 = R0 * (b2 - a2);
    const double s1 = fmax(fabs(x1), y1) > 0x1p480 ? 0x1p-540 : 1.0, s2 = fmax(fabs(x2), y2) > 0x1p480 ? 0x1p-540 : 1.0;
    x1 *= s1, y1 *= s1;
    x2 *= s2, y2 *= s2;
    x = fma(x1, x2, -(y1 * y2));
    y = fma(x1, y2, x2 * y1);
}

// Closed form of one piece over one edge part [a, a + L]: the integral along it
// of pi r0 [G_p(S) - G_p(r0)] dalpha for the piece polynomial pi G_p = g_-1/s +
// g_0 + g_2 s^2 + g_3 s^3 + g_4 s^4 + g_5 s^5, that is the difference between
// the part's ends of the antiderivative
//   -beta H_odd + r0 R0 T,  H_odd = g_-1 + g_3 r0^4 + g_5 r0^6,
//   T = g_2 x + g_3 P3' + g_4 (2 r0^2 x + R0^2 x + x^3/3)
//       + g_5 (x (S^3/4 + 3 c^2 S/8) + 3 c^4 a/8 + r0^2 P3'),
//   P3' = (x S + c^2 a)/2 + r0^2 a,  a = asinh(x/c),
//   beta = atan(x/R0) - atan(r0 x/(R0 S)),
// with every difference formed by a factor L instead of subtracting end values:
//   beta_b - beta_a = 2 atan2(R0 L, S_a S_b + a b + c^2 + r0 (S_a + S_b)),
//     numerator and denominator scaled by S_a S_b - a b where the sum S_a S_b +
//     a b would cancel ((S_a S_b)^2 - (a b)^2 = c^2 (a^2 + b^2 + c^2));
//   asinh(b/c) - asinh(a/c) = log(1 + L (1 + (a + b)/(S_a + S_b)) / (a + S_a)),
//     with a + S_a = c^2 / (S_a - a) for a < 0;
//   b S_b - a S_a = L (S_b + t),  t = a (a + b) / (S_a + S_b),
//   b S_b^3 - a S_a^3 = L (S_b^3 + t (S_a^2 + S_a S_b + S_b^2)),
//   b^3 - a^3 = L (a^2 + a b + b^2).
// The integrand is even in l, so a part with a + b < 0 is mirrored first.  One
// arctangent and one logarithm per part, where the ends taken apart cost two
// of each and every wall crossing a point of its own.
__device__ __forceinline__ double part_term(double r0, double R0, double a0, double L, bool shell)
{
    const double b0 = a0 + L;
    const bool mirror = a0 + b0 < 0.0;
    const double a = mirror ? -b0 : a0, b = mirror ? -a0 : b0;
    const double A = r0 * r0, R02 = R0 * R0;
    const double c2 = A + R02;
    const double Sa = sqrt_f64(fma(a, a, c2)), Sb = sqrt_f64(fma(b, b, c2));
    const double ab = a * b, SS = Sa * Sb, Ssum = Sa + Sb;
    const double rs = div_f64(1.0, Ssum);
    const bool neg = ab < 0.0;
    const double k = SS - ab, dx = fma(r0, Ssum, c2);
    const double yb = R0 * L * (neg ? k : 1.0);
    const double xb = neg ? fma(dx, k, c2 * (fma(a, a, fma(b, b, c2)))) : SS + ab + dx;
    const double Dbeta = 2.0 * atan2_f64(yb, xb);
    const double u = L * fma(a + b, rs, 1.0);
    const bool an = a < 0.0;
    // (c^2 may round to 0, the logarithm then is finite and multiplied by it)
    const double Da = log1p_ratio_f64(an ? u * (Sa - a) : u, max_f64(an ? c2 : a + Sa, 1e-290));
    const double t = a * (a + b) * rs;
    const double DxS = L * (Sb + t);
    const double DxS3 = L * fma(t, fma(Sa, Sa, fma(Sb, Sb, SS)), Sb * Sb * Sb);
    const double D3 = L * (fma(a, a, ab) + b * b);
    // the piece's coefficients (inner, or inner plus the step to the shell)
    const double sh = shell ? 1.0 : 0.0;
    const double gm1 = fma(sh, -1.0 / 60.0, -0.25), g2 = fma(sh, -1.0 / 6.0, -1.0 / 6.0), g3 = 0.25 * sh;
    const double g4 = fma(sh, -0.15, 0.075), g5 = fma(sh, 1.0 / 30.0, -0.025);
    const double Hodd = fma(A * A, fma(g5, A, g3), gm1);
    const double cD = fma(c2, Da, DxS);
    const double DP3 = fma(0.5, cD, A * Da);
    const double T5 = fma(0.25, DxS3, fma(0.375 * c2, cD, A * DP3));
    const double T4 = fma(fma(2.0, A, R02), L, D3 * (1.0 / 3.0));
    const double DT = fma(g2, L, fma(g3, DP3, fma(g4, T4, g5 * T5)));
    return fma(-Dbeta, Hodd, r0 * R0 * DT);
}

// The FP64 form of the edge's terms, one edge at a time (per-pair
// distributions, fixups, recomputed cells, table nodes); the task batches
// (k_integrate_queued64) spread the same terms over a wavefront.
__device__ __forceinline__ double edge_term(double r0, double R0, double la, double lb, double Le, double Ht,
                                            double dH, Work &wk)
{
    const EdgeParts P = edge_parts(true, r0, R0, la, lb);
    double tot = 0.0;
    if (la < P.ca || P.cb < lb) {
        double y, x;
        angle_product(R0, la, P.ca, P.cb, lb, y, x);
        if (!(fmax(R0, fmax(-la, lb)) < kFarLength)) angle_product_far(R0, la, P.ca, P.cb, lb, y, x);
        tot -= Ht * atan2_f64(y, x);
        wk.angles++;
    }
    if (P.near) {
        wk.eterms++;
        if (dH != 0.0 && (P.ca < P.ia || P.ib < P.cb)) {
            double y, x;
            angle_product(R0, P.ca, P.ia, P.ib, P.cb, y, x);
            tot += dH * atan2_f64(y, x);
            wk.angles++;
        }
#pragma unroll 1
        for (int q = 0; q < 3; q++) {  // shell, inner, shell
            const double x = q == 0 ? P.ca : (q == 1 ? P.ia : P.ib), y = q == 0 ? P.ia : (q == 1 ? P.ib : P.cb);
            if (y > x) {
                tot += part_term(r0, R0, x, part_len(x, y, la, lb, Le), q != 1);
                wk.moments++;
            }
        }
    }
    return tot;
}

constexpr double kInvPi = 0.318309886183790671537767526745;
constexpr float kInvPiF = 0.318309886183790671537767526745f;

// Error estimate of the FP32 terms of a pair in the mixed path: each term
// (an angle times its weight, an inner-part closed form, a Gauss-Legendre
// sub-interval) is taken to carry a relative error of up to 16 units of FP32
// rounding (a few for the inputs rounded from FP64, up to 5 for each
// transcendental, the rest for the arithmetic and the truncation of the
// sub-interval rule), the errors of different terms adding like a random walk:
// err = 16 * 2^-24 * sqrt(sum of squared terms) / pi, in units of f.
constexpr float kTermErr = 16.0f * 5.9604644775390625e-08f;

// Conditioning test of one edge in the mixed path: true for near-degenerate
// triangles that FP32 cannot resolve: the projection point within FP32
// rounding of the edge line, or the wall plane, the edge line's closest
// point or the edge itself within FP32 rounding of a piece radius (s = 1, 2)
// of the kernel, where the FP32 piece assignment is not reliable; also the
// particle within 2^-30 h of the edge line (c^2 < 2^-60), which keeps the FP32
// square roots and reciprocals away from denormal arguments.
__device__ __forceinline__ bool needs_fp64(double r0, double R0, double c2)
{
    const double e = 9.5367431640625e-07;  // 2^-20
    return (R0 * R0 < e * e * c2) || (c2 < 8.673617379884035e-19) || (fabs(r0 - 1.0) < e) ||
           (fabs(c2 - 1.0) < e) || (fabs(c2 - 4.0) < 4.0 * e);
}

// Raw f for one pair.  PREC = MAP_FP64 or MAP_MIXED.  Wall distance, foot
// point and edge projections are always FP64; in the mixed path the edge
// terms are FP32 (accumulated in FP64) unless the conditioning test sends the
// edge to the FP64 fixup pass.
template <int PREC>
__device__ __forceinline__ double pair_fraction(double px, double py, double pz, double h, int64_t cell,
                                                const int64_t *__restrict__ cfo, const int64_t *__restrict__ fvo,
                                                const double *__restrict__ plane, const EdgeRec *__restrict__ edges,
                                                Work &wk, uint64_t pair_k, unsigned *fix_count, uint64_t *fix_items,
                                                unsigned fix_cap, float &ev)
{
    using R = typename std::conditional<PREC == MAP_FP64, double, float>::type;
    const double invh = 1.0 / h;
    bool inside = true;
    int n_on = 0;
    double acc = 0.0;
    const int64_t f0 = cfo[cell], f1 = cfo[cell + 1];
    for (int64_t j = f0; j < f1; j++) {
        const double nx = plane[4 * j], ny = plane[4 * j + 1], nz = plane[4 * j + 2], cj = plane[4 * j + 3];
        const double d = cj - (nx * px + ny * py + nz * pz);
        wk.faces++;
        const bool in_j = d >= 0.0;
        inside = inside && in_j;
        n_on += d == 0.0 ? 1 : 0;
        const double r0d = fabs(d) * invh;
        if (!(r0d < 2.0)) continue;
        const R r0 = (R)r0d;
        const R Ht = pi_H<R>(r0);
        const R dH = pi_dH<R>(r0);
        double face = 0.0;
        const int64_t s0 = fvo[j], s1 = fvo[j + 1];
        for (int64_t s = s0; s < s1; s++) {
            const EdgeRec E = edges[s];
            const double wx = px - E.vx, wy = py - E.vy, wz = pz - E.vz;
            const double rho = E.mx * wx + E.my * wy + E.mz * wz;
            wk.edges++;
            if (rho == 0.0) continue;
            const double la = -(E.ex * wx + E.ey * wy + E.ez * wz) * invh;
            const double Le = E.L * invh, lb = la + Le;
            const double R0d = fabs(rho) * invh;
            if (PREC == MAP_MIXED && needs_fp64(r0d, R0d, r0d * r0d + R0d * R0d)) {
                const unsigned slot = atomicAdd(fix_count, 1u);
                if (slot < fix_cap) fix_items[slot] = (pair_k << 32) | (uint64_t)(uint32_t)s;
                continue;
            }
            const R t = edge_term(r0, (R)R0d, (R)la, (R)lb, (R)Le, Ht, dH, wk);
            face += (rho > 0.0) ? (double)t : -(double)t;
            if (PREC == MAP_MIXED) ev = fmaf((float)t, (float)t, ev);
        }
        acc += in_j ? face : -face;
    }
    return winding_term(inside, n_on, px, py, pz, cell, cfo, fvo, plane, edges) - acc * kInvPi;
}

// FP64 contribution of one edge to f (the fixup pass): the same terms as one
// iteration of the FP64 edge loop, with its wall's sign.
__device__ double edge_contribution_fp64(double px, double py, double pz, double h, const double *pl,
                                         const EdgeRec &E)
{
    Work wk;
    const double invh = 1.0 / h;
    const double d = pl[3] - (pl[0] * px + pl[1] * py + pl[2] * pz);
    const double r0 = fabs(d) * invh;
    if (!(r0 < 2.0)) return 0.0;
    const double wx = px - E.vx, wy = py - E.vy, wz = pz - E.vz;
    const double rho = E.mx * wx + E.my * wy + E.mz * wz;
    if (rho == 0.0) return 0.0;
    const double la = -(E.ex * wx + E.ey * wy + E.ez * wz) * invh;
    const double Le = E.L * invh;
    const double t = edge_term(r0, fabs(rho) * invh, la, la + Le, Le, pi_H<double>(r0), pi_dH<double>(r0), wk);
    const double face = (rho > 0.0) ? t : -t;
    return -(d >= 0.0 ? face : -face) * kInvPi;
}

// Adds a wavefront's sums to the work counters: lane q brings the q-th, so that
// the seven take one atomic instruction on one cache line (see next_tile_xcd).
__device__ __forceinline__ void add_counters(int lane, unsigned long long eterms, unsigned long long faces,
                                             unsigned long long edges, unsigned long long moments,
                                             unsigned long long quads, unsigned long long angles,
                                             unsigned long long qpoints, unsigned long long *counters)
{
    const int at[7] = {C_EDGE_TERMS, C_FACES, C_EDGES, C_MOMENTS, C_QUADS, C_ANGLES, C_QPOINTS};
    const unsigned long long v[7] = {eterms, faces, edges, moments, quads, angles, qpoints};
    unsigned long long mine = 0;
    int to = 0;
#pragma unroll
    for (int q = 0; q < 7; q++) {
        mine = lane == q ? v[q] : mine;
        to = lane == q ? at[q] : to;
    }
    if (mine != 0) atomicAdd(counter_copy(counters) + to, mine);
}

__device__ __forceinline__ unsigned long long wave_total(unsigned long long v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ void flush_work(const Work &wk, unsigned long long *counters)
{
    add_counters(threadIdx.x & 63, wave_total(wk.eterms), wave_total(wk.faces), wave_total(wk.edges),
                 wave_total(wk.moments), wave_total(wk.quads), wave_total(wk.angles), wave_total(wk.qpoints), counters);
}

struct FixList {
    unsigned *count;
    uint64_t *items;
    unsigned cap;
    float *err;  // mixed path: per-pair FP32 error estimates (or null)
};

// Appends the fixup item (pair k, slot) when the list has room; the count
// keeps growing past the capacity, which tells the host that items were lost.
__device__ __forceinline__ void push_fix(const FixList &fx, int64_t k, uint32_t slot)
{
    const unsigned i = atomicAdd(fx.count, 1u);
    if (i < fx.cap) fx.items[i] = ((uint64_t)k << 32) | (uint64_t)slot;
}

template <int PREC>
__device__ __forceinline__ double one_pair(int64_t k, const uint32_t *__restrict__ pair_p,
                                           const uint32_t *__restrict__ pair_c, const double *__restrict__ xyz,
                                           const double *__restrict__ h, const int64_t *__restrict__ cfo,
                                           const int64_t *__restrict__ fvo, const double *__restrict__ plane,
                                           const EdgeRec *__restrict__ edges, Work &wk, const FixList &fx)
{
    const int64_t a = pair_p[k];
    const int64_t c = pair_c[k];
    float ev = 0.0f;
    const double v = pair_fraction<PREC>(xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2], h[a], c, cfo, fvo, plane, edges,
                                         wk, (uint64_t)k, fx.count, fx.items, fx.cap, ev);
    if (PREC == MAP_MIXED && fx.err) fx.err[k] = kTermErr * kInvPiF * sqrt_f32(ev);
    return v;
}

template <int PREC>
__global__ void __launch_bounds__(256) k_integrate_flat(int64_t np, const uint32_t *__restrict__ pair_p,
                                                         const uint32_t *__restrict__ pair_c,
                                                         const double *__restrict__ xyz, const double *__restrict__ h,
                                                         const int64_t *__restrict__ cfo,
                                                         const int64_t *__restrict__ fvo,
                                                         const double *__restrict__ plane,
                                                         const EdgeRec *__restrict__ edges, double *__restrict__ f,
                                                         unsigned long long *counters, FixList fx)
{
    int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    Work wk;
    if (k < np) f[k] = one_pair<PREC>(k, pair_p, pair_c, xyz, h, cfo, fvo, plane, edges, wk, fx);
    flush_work(wk, counters);
}

// Persistent form: each wavefront takes tiles of 64*tile_waves consecutive
// (cell-ordered) pairs from a queue until the pairs run out.
template <int PREC, int WPE>
__global__ void __launch_bounds__(256, WPE) k_integrate_persistent(int64_t np, const uint32_t *__restrict__ pair_p,
                                                               const uint32_t *__restrict__ pair_c,
                                                               const double *__restrict__ xyz,
                                                               const double *__restrict__ h,
                                                               const int64_t *__restrict__ cfo,
                                                               const int64_t *__restrict__ fvo,
                                                               const double *__restrict__ plane,
                                                               const EdgeRec *__restrict__ edges,
                                                               double *__restrict__ f, unsigned long long *counters,
                                                               unsigned *tile_ctr, int tile_waves, FixList fx)
{
    const int lane = threadIdx.x & 63;
    const int64_t tile = 64 * (int64_t)tile_waves;
    const int64_t ntiles = (np + tile - 1) / tile;
    Work wk;
    for (;;) {
        unsigned t = 0;
        if (lane == 0) t = atomicAdd(tile_ctr, 1u);
        t = __shfl(t, 0, 64);
        if ((int64_t)t >= ntiles) break;
        const int64_t base = (int64_t)t * tile;
        for (int w = 0; w < tile_waves; w++) {
            const int64_t k = base + 64 * w + lane;
            if (k < np) f[k] = one_pair<PREC>(k, pair_p, pair_c, xyz, h, cfo, fvo, plane, edges, wk, fx);
        }
    }
    flush_work(wk, counters);
}

// Next tile of a persistent kernel of 4 wavefronts per workgroup in XCD-aware
// order, or -1 when none is left.  Workgroups are dispatched round-robin over
// the 8 XCDs, so workgroup b runs on XCD b mod 8; each XCD first takes the tiles
// of its own eighth of the (cell-ordered) pair list, so the tiles that share a
// cell's wall and edge records meet in one L2, then takes what is left in the
// other eighths.  A wavefront's first tile is fixed by its place in the grid,
// the later ones come from the eighths' counters (a cache line each): where there is a
// wavefront for every tile, none is touched.  (An atomic reaches memory one at a
// time per cache line: with a returning one per tile, wavefront and eighth on one
// line, and seven instructions per wavefront for the work counters, a call on
// 4,096 uniform particles took 1.27 ms, now 0.78; 32,768 clumpy ones 3.66, now
// 3.09.)  `probe` (-1 at the start) persists between calls.  Wave-uniform.  A pair's result does not depend on the
// wavefront that computes it.
__device__ __forceinline__ int64_t next_tile_xcd(unsigned *ctr, int64_t ntiles, int &probe, int lane)
{
    const int xcd = (int)(blockIdx.x & 7);
    const int64_t chunk = (ntiles + 7) / 8;
    if (probe < 0) {
        probe = 0;
        const int64_t lo = xcd * chunk, hi = lo + chunk < ntiles ? lo + chunk : ntiles;
        const int64_t t = lo + 4 * (int64_t)(blockIdx.x >> 3) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        if (t < hi) return t;
    }
    while (probe < 8) {
        const int y = (xcd + probe) & 7;
        const int64_t hi = (y + 1) * chunk < ntiles ? (y + 1) * chunk : ntiles;
        // the tiles that are no wavefront's first one
        const int64_t lo = y * chunk + 4 * (int64_t)(((int)gridDim.x - y + 7) / 8);
        if (lo < hi) {
            // (read first: at the end every wavefront looks at every eighth)
            unsigned *c = ctr + y * kXcdCtrStride;
            unsigned v = __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lo + (int64_t)__builtin_amdgcn_readfirstlane(v) < hi) {
                if (lane == 0) v = atomicAdd(c, 1u);
                v = __builtin_amdgcn_readfirstlane(v);
                if (lo + (int64_t)v < hi) return lo + (int64_t)v;
            }
        }
        probe++;
    }
    return -1;
}

// ---------------------------------------------------------------- queued tasks (mixed path)
// The edge terms split into independent tasks of three kinds: angles (one
// atan2), closed-form points (one trans + core) and shell quadrature
// sub-intervals (4 Gauss-Legendre points each, see run_quad).  In a wavefront of 64 pairs most
// lanes need only a few of the possible tasks at a given edge, so running
// every kind whenever any lane needs it leaves most lanes idle.  Here each
// lane classifies its edge and pushes its tasks, with their weights and the
// edge's sign, onto per-wavefront stacks in LDS; a stack holding 64 tasks is
// run by the whole wavefront at once, and every result is added to its
// pair's FP64 accumulator (LDS).  Lanes walk their cell's wall slots with one
// wave-uniform counter, so the pushes and runs are in uniform control flow.
constexpr int kQ = 128;  // stack capacity: below 64 pending before a push of at most 64

constexpr int kQA = 64;  // angle stack capacity: run before a push that would overflow it
struct WaveStacks {
    float ang[3][kQA];  // atan2 arguments of the angle (imaginary, real part), weight
    float pnt[4][kQ];   // inner parts: r0, signed R0 (sign = the term's sign), start a, length L
    float qd[4][kQ];    // shell sub-intervals: r0, signed R0, mid, half-length
    uint32_t qd_o[kQ];                // owner lanes (a word each: the sub-intervals are the most frequent tasks)
    uint8_t ang_o[kQA], pnt_o[kQ];
    double acc[64];
    double ev[64];  // sums of the squared FP32 task values per owner (error estimate)
};

// A task's value to its owner.  Both sums take the LDS double atomic, which
// issues in 8 clocks per wavefront (20 where owners repeat in pairs); the float
// one takes 193 (measured, all lanes on addresses of their own).
__device__ __forceinline__ void add_task(WaveStacks &W, int o, float v)
{
    const double d = (double)v;
    atomicAdd(&W.acc[o], d);
    atomicAdd(&W.ev[o], d * d);
}

__device__ __forceinline__ void run_angle(WaveStacks &W, int i)
{
    const int o = W.ang_o[i];
    const float v = W.ang[2][i] * atan2_f32(W.ang[0][i], W.ang[1][i]);
    add_task(W, o, v);
}

// Closed form of the inner piece (s <= 1) over one edge part [a, a + L],
// a >= -l1, a + L <= l1: the integral along it of pi r0 [G_inner(S) -
// G_inner(r0)] dalpha, that is the difference of the antiderivative
//     -beta H_odd + r0 R0 T
// (see core) between the part's ends, written so that every difference
// between the ends carries the factor L explicitly instead of subtracting
// two nearly equal end values (a part much shorter than h would lose most of
// its digits in FP32 otherwise):
//   beta_b - beta_a      = 2 atan2(R0 L, S_a S_b + a b + c^2 + r0 (S_a + S_b))
//                          (the solid angle of the triangle foot-v_a-v_b);
//   asinh(b/c) - asinh(a/c) = asinh(L (c^2 + S_a S_b - a b) / (c^2 (S_a + S_b)));
//   b S_b - a S_a         = L (S_b + a (a + b) / (S_a + S_b));
//   b S_b^3 - a S_a^3     = L (S_b^3 + a (a + b) (S_a^2 + S_a S_b + S_b^2) / (S_a + S_b));
//   b^3 - a^3             = L (a^2 + a b + b^2);
// S_a S_b +- a b is formed from (S_a S_b)^2 - (a b)^2 = c^2 (a^2 + b^2 + c^2)
// on the side where it would cancel.  L comes from the FP64 edge length when
// the part is the whole edge.
__device__ __forceinline__ void run_seg(WaveStacks &W, int i)
{
    const int o = W.pnt_o[i];
    const float r0 = W.pnt[0][i], sR0 = W.pnt[1][i], a = W.pnt[2][i], L = W.pnt[3][i];
    const float R0 = fabsf(sR0), w = sR0 < 0.0f ? -1.0f : 1.0f;
    const float b = a + L;
    const float A = r0 * r0, R02 = R0 * R0, c2 = fmaf(R0, R0, A);
    const float Sa = sqrt_f32(fmaf(a, a, c2)), Sb = sqrt_f32(fmaf(b, b, c2));
    const float ab = a * b, SS = Sa * Sb, Ssum = Sa + Sb;
    const float q = c2 * (fmaf(a, a, fmaf(b, b, c2)));  // (S_a S_b)^2 - (a b)^2
    float sp, sm;                                       // S_a S_b + a b, S_a S_b - a b
    if (ab > 0.0f) {
        sp = SS + ab;
        sm = q * rcp_f32(sp);
    } else {
        sm = SS - ab;
        sp = q * rcp_f32(sm);
    }
    const float rs = rcp_f32(Ssum);
    const float Dbeta = 2.0f * atan2_f32(R0 * L, fmaf(r0, Ssum, sp + c2));
    const float Z = L * (c2 + sm) * rcp_f32(c2 * Ssum);
    const float Da = log1p_f32(fmaf(Z * Z, rcp_f32(1.0f + sqrt_f32(fmaf(Z, Z, 1.0f))), Z));
    const float t = a * (a + b) * rs;
    const float DxS = L * (Sb + t);
    const float DxS3 = L * fmaf(t, Sb * Sb + SS + Sa * Sa, Sb * Sb * Sb);
    const float D3 = L * (fmaf(a, a, ab) + b * b);
    // inner piece: g_-1 = -1/4, g_2 = -1/6, g_3 = 0, g_4 = 3/40, g_5 = -1/40
    const float Hodd = -0.25f - 0.025f * A * A * A;
    const float DP3r = 0.5f * fmaf(c2, Da, DxS) + A * Da;
    const float DT = (-1.0f / 6.0f) * L + 0.075f * fmaf(2.0f * A + R02, L, D3 * (1.0f / 3.0f)) -
                     0.025f * (0.25f * DxS3 + 0.375f * c2 * fmaf(c2, Da, DxS) + A * DP3r);
    const float v = w * fmaf(-Dbeta, Hodd, r0 * R0 * DT);
    add_task(W, o, v);
}

// 4-point Gauss-Legendre nodes and weights on [-1, 1] (nodes in pairs +-x)
__constant__ float kGL4x[2] = {0.3399810435848563f, 0.8611363115940526f};
__constant__ float kGL4w[2] = {0.6521451548625461f, 0.3478548451374538f};

// One sub-interval of the shell integrand (the integrand of shell_quad) by
// 4-point Gauss-Legendre.  Sub-intervals are at most 0.4 times the distance
// to the integrand's branch points l = +-ic long (and at most 2 - r0), so
// the branch points lie outside the Bernstein ellipse of parameter
// 5 + sqrt(26) of every sub-interval; the Gauss-Legendre error theorem for
// analytic integrands then bounds the truncation by 1e-8 of the pair fraction
// per sub-interval over the whole (r0, c) range (measured: below 3e-10).
__device__ __forceinline__ void run_quad(WaveStacks &W, int i)
{
    const int o = (int)W.qd_o[i];
    const float r0 = W.qd[0][i], sR0 = W.qd[1][i], mid = W.qd[2][i], hl = W.qd[3][i];
    const float c2 = fmaf(sR0, sR0, r0 * r0), w = sR0 * hl * (1.0f / 120.0f);
    // the numerator (r0+1)(r0 Sigma + V^5) - r0 U^5 as a polynomial in U with
    // coefficients a0..a5 (a1..a4 = (r0+1) r0 V^(4-k), a0 = (r0+1)(V^5 + r0 V^4), a5 = -r0)
    const float V = 2.0f - r0;
    const float V2 = V * V, V3 = V2 * V, V4 = V2 * V2;
    const float t = (r0 + 1.0f) * r0;
    const float a0 = (r0 + 1.0f) * fmaf(r0, V4, V4 * V), a1 = t * V3, a2 = t * V2, a3 = t * V;
    float acc = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; q++) {
        const float xq = (q & 1) ? -kGL4x[q >> 1] : kGL4x[q >> 1];
        const float l = fmaf(hl, xq, mid);
        const float S = sqrt_f32(fmaf(l, l, c2));
        const float U = 2.0f - S;
        const float num = fmaf(fmaf(fmaf(fmaf(fmaf(-r0, U, t), U, a3), U, a2), U, a1), U, a0);
        acc = fmaf(kGL4w[q >> 1], num * rcp_f32(S * (S + r0)), acc);
    }
    const float v = w * acc;
    add_task(W, o, v);
}

template <int KIND>
__device__ __forceinline__ void run_one(WaveStacks &W, int i)
{
    if (KIND == 0) run_angle(W, i);
    else if (KIND == 1) run_seg(W, i);
    else run_quad(W, i);
}

// run the top 64 entries when 64 are pending (all = false), or all pending ones
template <int KIND>
__device__ __forceinline__ void run_stack(WaveStacks &W, int &count, int lane, bool all)
{
    if (count >= 64) {
        lds_sync_wave();
        run_one<KIND>(W, count - 64 + lane);
        count -= 64;
        lds_sync_wave();
    }
    if (all && count > 0) {
        lds_sync_wave();
        if (lane < count) run_one<KIND>(W, lane);
        count = 0;
        lds_sync_wave();
    }
}

__device__ __forceinline__ int64_t uniform64(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)(uint64_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ __forceinline__ int wave_max(int v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
    return v;
}

// A lane's current wall in the mixed task batches.
struct MixedWall {
    float r0 = 0.0f, nHt = 0.0f, dH = 0.0f;  // distance, -pi H, pi dH
    uint32_t sbit = 0;    // sign bit of the wall's terms (set: the particle is on its outer side)
    float c2_min = 0.0f;  // edges with a smaller c^2 go to the FP64 fixup pass (NaN: all of them, r0 asks for it)
    float r_len = 0.0f;   // reciprocal of the longest sub-interval of a shell part next to the inner piece; 0: the
                          // wall lies beyond the support, or the lane has none
};

// Work counters of a wavefront (scalars: the masks are there anyway).
struct WaveWork {
    unsigned eterms = 0, moments = 0, quads = 0, angles = 0;
};

__device__ __forceinline__ void flush_wave_work(Work &wk, WaveWork &ww, int lane, unsigned long long *counters)
{
    add_counters(lane, ww.eterms, wave_total(wk.faces), wave_total(wk.edges), ww.moments, ww.quads, ww.angles,
                 4ull * ww.quads, counters);
    wk = Work();
    ww = WaveWork();
}

// Lane masks: one bit per lane in a scalar register pair, so that logic on them is scalar.
__device__ __forceinline__ uint64_t mask_of(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// x with the sign bit flipped where sbit is set
__device__ __forceinline__ float flip_sign(float x, uint32_t sbit)
{
    return __uint_as_float(__float_as_uint(x) ^ sbit);
}
__device__ __forceinline__ double flip_sign(double x, uint32_t sbit)
{
    return __hiloint2double((int)((uint32_t)__double2hiint(x) ^ sbit), __double2loint(x));
}

// One step of the mixed task batches: this lane's edge E (record s of the edge
// table; live = the lane has a wall within the support and an edge at this
// step) is projected in FP64, classified in FP32 and its tasks are pushed;
// full stacks run as they fill.  Wave-uniform control flow; a lane that is not
// live goes through the same operations on undefined values and contributes
// nothing.
//
// Bound by vector issue.  On this chip an FP32 add, multiply or fused
// multiply-add and a 32-bit add or logical operation on registers or literals
// take 2 clocks per wavefront, comparisons, selects, minima, conversions, shifts,
// bit counts and all FP64 take 4, and reciprocals and square roots 8 (measured,
// single instructions in a loop).  So lane masks live in scalar registers, signs
// are bits, counts are floats, what depends on the wall alone is kept with the
// wall, and one coarse test stands before the exact conditioning test: 258 vector
// instructions a step where a form with lane predicates, counters in vector
// registers and float atomics took 290.  34.7e6 pairs of a clumpy cloud: 21.0 ->
// 16.9 ms, of which 2.4 ms are the atomics (add_task).
__device__ __forceinline__ void mixed_edge_step(WaveStacks &W, int lane, WaveWork &ww, int &nA, int &nP, int &nQ,
                                                uint64_t live, const EdgeRec &E, int32_t s, double px, double py,
                                                double pz, double invh, const MixedWall &wall, int64_t k,
                                                const FixList &fx, double &acc_in, float &ev_in)
{
    const float r0 = wall.r0;
    const double wx = px - E.vx, wy = py - E.vy, wz = pz - E.vz;
    const double rho = E.mx * wx + E.my * wy + E.mz * wz;
    const double lad = -(E.ex * wx + E.ey * wy + E.ez * wz) * invh;
    const double Ld = E.L * invh;
    const float R0 = (float)(fabs(rho) * invh);
    const float la = (float)lad, lb = (float)(lad + Ld);
    const float Le = (float)Ld;  // the edge's length from FP64: parts spanning the whole edge keep their digits
    const uint32_t sbit = ((uint32_t)__double2hiint(rho) ^ wall.sbit) & 0x80000000u;  // of the edge's terms
    const float R02 = R0 * R0, c2 = fmaf(r0, r0, R02);
    // The conditioning test (needs_fp64, here on FP32 values: the rounding of c^2
    // is 2^-24 relative, far inside the 2^-20 margins) and rho = 0, seldom true, behind a
    // coarse test that holds wherever they do: c^2 >= R0^2, so c^2 < c2_min or
    // R0^2 < 2^-40 c^2 gives R0^2 < c2_min + 2^-40 c^2; |c^2 - 1| < e or
    // |c^2 - 4| < 4 e gives |(c^2 - 1) (c^2 - 4)| < 13 e; rho = 0 gives R0 = 0
    // and c2_min > 0.
    constexpr float e = 9.5367431640625e-07f;  // 2^-20
    const uint64_t near_bad = live & (mask_of(!(R02 >= fmaf(c2, 9.094947017729282e-13f, wall.c2_min))) |
                                      mask_of(fabsf(fmaf(c2, c2 - 5.0f, 4.0f)) < 16.0f * e));
    if (near_bad != 0) {
        const bool bad = R02 < 9.094947017729282e-13f * c2 || c2 < wall.c2_min || wall.c2_min != wall.c2_min ||
                         fabsf(c2 - 1.0f) < e || fabsf(c2 - 4.0f) < 4.0f * e;
        if (lane_in(near_bad) && bad && rho != 0.0) {
            const unsigned slot = atomicAdd(fx.count, 1u);
            if (slot < fx.cap) fx.items[slot] = ((uint64_t)k << 32) | (uint64_t)(uint32_t)s;
        }
        live &= ~(near_bad & mask_of(bad || rho == 0.0));
    }
    // classification (the mixed form of edge_term).  The edge [la, lb] splits
    // into the parts beyond the support (|l| > l2), the shell parts and the
    // inner part (|l| < l1, when c < 1): [la, ca] + [cb, lb] beyond,
    // [ca, ia] + [ib, cb] shell, [ia, ib] inner, every part oriented and
    // possibly empty.  Far edges (c >= 2) are all beyond (l2 = 0).
    const uint64_t near = live & mask_of(c2 < 4.0f), inner = near & mask_of(c2 < 1.0f);
    const float l2 = lane_in(near) ? sqrt_f32(4.0f - c2) : 0.0f;
    const float l1 = lane_in(inner) ? sqrt_f32(1.0f - c2) : 0.0f;
    // clamps as medians of three (la <= lb, so min(max(x, lo), hi) is the
    // median of x, lo and hi also when lo > hi: one instruction each)
    const float ca = __builtin_amdgcn_fmed3f(la, -l2, lb);
    const float cb = __builtin_amdgcn_fmed3f(ca, l2, lb);
    const float ia = lane_in(inner) ? __builtin_amdgcn_fmed3f(ca, -l1, cb) : cb;
    const float ib = lane_in(inner) ? __builtin_amdgcn_fmed3f(ia, l1, cb) : cb;
    const uint64_t cut_a = mask_of(la < ca), cut_b = mask_of(cb < lb);      // (else ca = la, cb = lb)
    const uint64_t shell_a = near & mask_of(ca < ia), shell_b = near & mask_of(ib < cb);
    // Length of a part: the FP64-derived length when it is the whole edge, else
    // the FP32 difference (a clipped end sits on a kernel sphere, where an end
    // shift changes the integral only to second order)
    auto part_len = [&](bool whole, float x, float y) { return whole ? Le : y - x; };
    const float len_a = part_len(lane_in(~cut_a & mask_of(ia == lb)), ca, ia);  // shell parts [ca, ia] and [ib, cb]
    const float len_b = part_len(lane_in(~cut_b & mask_of(ib == la)), ib, cb);
    // angle terms: -H times the beyond parts' angle, dH times the shell
    // parts' angle.  The angle of two parts is the argument of the product of
    // their complex numbers (R0^2 + a b) + i R0 (b - a) (sum below pi).  One
    // angle per lane is taken here; a lane that has both pushes the shell
    // angle as a task.
    const uint64_t has_b = live & (cut_a | cut_b);
    const uint64_t has_s = (shell_a | shell_b) & mask_of(wall.dH != 0.0f);
    {
        // the parts [la, b1] and [a2, lb] (a lane without beyond parts has ca = la and cb = lb)
        const float b1 = lane_in(has_b) ? ca : ia, a2 = lane_in(has_b) ? cb : ib;
        const float x1 = fmaf(la, b1, R02), y1 = R0 * part_len(b1 == lb, la, b1);
        const float x2 = fmaf(lb, a2, R02), y2 = R0 * part_len(a2 == la, a2, lb);
        const float zx = fmaf(x1, x2, -(y1 * y2)), zy = fmaf(x2, y1, x1 * y2);
        const float w_in = flip_sign(lane_in(has_b) ? wall.nHt : (lane_in(has_s) ? wall.dH : 0.0f), sbit);
        const float v = lane_in(live) ? w_in * atan2_f32(zy, zx) : 0.0f;
        acc_in += (double)v;
        ev_in = fmaf(v, v, ev_in);
    }
    ww.eterms += __popcll(near);
    ww.angles += __popcll(has_b) + __popcll(has_s);
    {
        const uint64_t m = has_b & has_s;
        if (m != 0) {
            if (nA + __popcll(m) > kQA) run_stack<0>(W, nA, lane, true);
            const int slot = wave_push(m, nA);
            if (lane_in(m)) {
                const float x1 = fmaf(ca, ia, R02), y1 = R0 * len_a;
                const float x2 = fmaf(cb, ib, R02), y2 = R0 * len_b;
                W.ang[0][slot] = fmaf(x2, y1, x1 * y2);
                W.ang[1][slot] = fmaf(x1, x2, -(y1 * y2));
                W.ang[2][slot] = flip_sign(wall.dH, sbit);
                W.ang_o[slot] = (uint8_t)lane;
            }
            run_stack<0>(W, nA, lane, false);
        }
    }
    const float sR0 = flip_sign(R0, sbit);
    // inner part [ia, ib]: one closed-form task over the part (run_seg)
    {
        const uint64_t m = inner & mask_of(ib > ia);
        if (m != 0) {
            const int slot = wave_push(m, nP);
            ww.moments += __popcll(m);
            if (lane_in(m)) {
                W.pnt[0][slot] = r0;
                W.pnt[1][slot] = sR0;
                W.pnt[2][slot] = ia;
                W.pnt[3][slot] = part_len(ia == la && ib == lb, ia, ib);
                W.pnt_o[slot] = (uint8_t)lane;
            }
            run_stack<1>(W, nP, lane, false);
        }
    }
    // shell parts by quadrature: [ca, ia] and [ib, cb], each cut into 1 to 32
    // sub-intervals no longer than 0.4 times the distance to the branch points
    // l = +-ic of the integrand (c < 1: to the inner piece's sphere), nor than
    // V = 2 - r0: the shell integrand is of order V^4 on the edge, and a
    // sub-interval longer than V would let the polynomial in U = 2 - S grow far
    // beyond that inside the ellipse of analyticity that bounds the
    // Gauss-Legendre error
    float hl0 = 0.0f, hl1 = 0.0f, end0 = 0.0f, end1 = 0.0f;  // half-lengths, twice the numbers of sub-intervals
    if (lane_in(shell_a)) {
        const float r_len = lane_in(inner) ? wall.r_len : rcp_f32(fminf(0.4f * sqrt_f32(c2), 2.0f - r0));
        const float n = __builtin_amdgcn_fmed3f(ceilf(len_a * r_len), 1.0f, 32.0f);
        hl0 = 0.5f * len_a * rcp_f32(n);
        end0 = n + n;
    }
    if (lane_in(shell_b)) {
        const float n = __builtin_amdgcn_fmed3f(ceilf(len_b * wall.r_len), 1.0f, 32.0f);
        hl1 = 0.5f * len_b * rcp_f32(n);
        end1 = n + n;
    }
    // both parts' sub-intervals in one uniform loop: midpoints from + at hl, at = 1, 3, 5, ... below the part's end
    const float end = end0 + end1;
    for (float step = 1.0f;; step += 2.0f) {
        const uint64_t m = mask_of(step < end);
        if (m == 0) break;
        const int slot = wave_push(m, nQ);
        ww.quads += __popcll(m);
        if (lane_in(m)) {
            const float past = step - end0;
            const bool second = past > 0.0f;
            const float hl = second ? hl1 : hl0;
            W.qd[0][slot] = r0;
            W.qd[1][slot] = sR0;
            W.qd[2][slot] = fmaf(hl, second ? past : step, second ? ib : ca);
            W.qd[3][slot] = hl;
            W.qd_o[slot] = (uint32_t)lane;
        }
        run_stack<2>(W, nQ, lane, false);
    }
}

// The job of global tile t of a launch of several jobs (wave-uniform): the
// last job whose first tile is at or before t.
__device__ __forceinline__ int job_of_tile(const JobsArg &A, int64_t t)
{
    int lo = 0, hi = A.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (A.table[mid].wave_base <= t) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Field of the current job: the kernel argument itself for a one-job launch
// (kept in scalar registers as plain arguments would be), the device table
// entry otherwise.
#define JOB(field) (MULTI ? A.table[jj].field : A.one.field)

// Marker slot of a fixup item that asks for the winding weight of a pair whose
// particle lies on two or more of its cell's wall planes (an edge or a vertex
// of the cell; see em_boundary.h).
constexpr uint32_t kWindingSlot = 0xffffffffu;

// The states of two lanes that walked different walls of one pair: counts of
// walls whose plane holds the particle, and the top bit (outside of a wall).
__device__ __forceinline__ unsigned join_walls(unsigned a, unsigned b)
{
    return ((a & 0x7fffffffu) + (b & 0x7fffffffu)) | ((a | b) & 0x80000000u);
}

template <int WPE, bool MULTI>
__global__ void __launch_bounds__(256, WPE) k_integrate_queued(JobsArg A, unsigned *tile_ctr)
{
    __shared__ WaveStacks stacks[4];
    const int lane = threadIdx.x & 63;
    WaveStacks &W = stacks[threadIdx.x >> 6];
    int probe = -1;
    int cur = MULTI ? -1 : 0;
    Work wk;      // walls and edges, per lane
    WaveWork ww;  // the rest
    auto flush = [&](unsigned long long *counters) { flush_wave_work(wk, ww, lane, counters); };
    for (;;) {
        const int64_t t = next_tile_xcd(tile_ctr + kXcdCtr, A.n_tiles, probe, lane);
        if (t < 0) break;
        const int jj = MULTI ? job_of_tile(A, t) : 0;
        if (MULTI && jj != cur) {
            if (cur >= 0) flush(A.table[cur].counters);
            cur = jj;
        }
        const FixList fx = {JOB(fix_count), JOB(fix_items), JOB(fix_cap), nullptr};
        const EdgeRec *__restrict__ edges = JOB(edges);
        const double *__restrict__ plane = JOB(plane);
        const int64_t *__restrict__ fvo = JOB(fvo);
        const int sh = JOB(split), part = lane & ((1 << sh) - 1);  // 2^sh neighbouring lanes share a pair
        const int64_t k = (t - JOB(wave_base)) * (64 >> sh) + (lane >> sh);
        const bool active = k < JOB(np);
        double px = 0.0, py = 0.0, pz = 0.0, invh = 1.0;
        int32_t s = 0, s_end = 0, j = 0;
        if (active) {
            const int64_t a = JOB(pair_p)[k];
            const int64_t c = JOB(pair_c)[k];
            px = JOB(xyz)[3 * a];
            py = JOB(xyz)[3 * a + 1];
            pz = JOB(xyz)[3 * a + 2];
            invh = 1.0 / JOB(h)[a];
            const int64_t *__restrict__ cfo = JOB(cfo);
            const int64_t f0 = cfo[c], walls = cfo[c + 1] - f0, from = f0 + ((walls * part) >> sh);
            j = (int32_t)from - 1;
            s = (int32_t)fvo[from];
            s_end = (int32_t)fvo[f0 + ((walls * (part + 1)) >> sh)];
        }
        W.acc[lane] = 0.0;
        W.ev[lane] = 0.0;
        int32_t face_end = s;  // first slot past the current wall: the first step opens the cell's first wall
        const int n_steps = __builtin_amdgcn_readfirstlane(wave_max((int)(s_end - s)));
        const EdgeRec *ep = edges + s;
        int nA = 0, nP = 0, nQ = 0;
        double acc_in = 0.0;  // this lane's terms taken in place (not as tasks)
        float ev_in = 0.0f;   // the sum of their squares
        unsigned at_walls = 0;  // walls whose plane holds the particle; top bit: it is outside of a wall
        MixedWall wall;
        for (int it = 0; it < n_steps; it++, s++, ep++) {
            if (s == face_end) {
                wall.r_len = 0.0f;
                face_end = -1;
                if (s < s_end) {
                    j++;
                    face_end = (int32_t)fvo[j + 1];
                    const double *pl = plane + plane_at(j);
                    const double d = pl[3] - (pl[0] * px + pl[1] * py + pl[2] * pz);
                    wk.faces++;
                    const bool in_j = d >= 0.0;
                    at_walls = (at_walls + (d == 0.0)) | (in_j ? 0u : 0x80000000u);
                    const double r0d = fabs(d) * invh;
                    const float r0 = (float)r0d;
                    wall.sbit = in_j ? 0u : 0x80000000u;
                    wall.r0 = r0;
                    wall.nHt = -pi_H<float>(r0);
                    wall.dH = pi_dH<float>(r0);
                    wall.c2_min = fabsf(r0 - 1.0f) < 9.5367431640625e-07f ? NAN : 8.673617379884035e-19f;
                    if (r0d < 2.0) {
                        wall.r_len = rcp_f32(fminf(0.4f, 2.0f - r0));
                        wk.edges += face_end - s;
                    }
                }
            }
            const uint64_t live = mask_of(wall.r_len != 0.0f);
            double E[10];  // the edge record; some value or other in a lane without one
#pragma unroll
            for (int q = 0; q < 10; q++) asm volatile("" : "=v"(E[q]));
            if (lane_in(live)) {
                const double *from = reinterpret_cast<const double *>(ep);
#pragma unroll
                for (int q = 0; q < 10; q++) E[q] = from[q];
            }
            mixed_edge_step(W, lane, ww, nA, nP, nQ, live,
                            EdgeRec{E[0], E[1], E[2], E[3], E[4], E[5], E[6], E[7], E[8], E[9]}, s, px, py, pz, invh,
                            wall, k, fx, acc_in, ev_in);
        }
        run_stack<0>(W, nA, lane, true);
        run_stack<1>(W, nP, lane, true);
        run_stack<2>(W, nQ, lane, true);
        lds_sync_wave();
        double sum = W.acc[lane] + acc_in;
        float ev = ev_in + (float)W.ev[lane];
        for (int o = 1; o < 1 << sh; o <<= 1) {
            sum += __shfl_xor(sum, o, 64);
            ev += __shfl_xor(ev, o, 64);
            at_walls = join_walls(at_walls, __shfl_xor(at_walls, o, 64));
        }
        const bool inside = at_walls < 0x80000000u;
        if (active && part == 0) {
            const double v = (inside ? 1.0 : 0.0) - sum * kInvPi;
            JOB(f)[k] = v;
            if (JOB(S)) atomicAdd(JOB(S) + JOB(pair_p)[k], fixed52(v));
            float *const err = JOB(err);  // null when no estimate is wanted (the autotuner's timing runs)
            if (err) err[k] = kTermErr * kInvPiF * sqrt_f32(ev);
            if (inside && at_walls >= 2) push_fix(fx, k, kWindingSlot);
        }
        lds_sync_wave();
    }
    if (cur >= 0) flush(MULTI ? A.table[cur].counters : A.one.counters);
}

// FP64 form of the task batches: the beyond parts' angle (or the shell parts',
// in a lane without the former) is taken in place, a lane with both pushes the
// shell angle; every shell and inner part is one closed-form task (part_term),
// both pieces on one stack, since only their coefficients differ.
constexpr int kQP = 192;  // part stack capacity: below 64 pending before a step, run above 128 before its last push
struct WaveStacks64 {
    double ang[3][kQA];  // atan2 arguments of the angle (imaginary, real part), weight
    double pnt[4][kQP];  // parts: r0, signed R0 (sign = the term's sign), start a, length L
    double acc[64];
    uint8_t ang_o[kQA], pnt_o[kQP];  // owner lanes (pnt_o: plus kShellPart for a shell part)
};
constexpr int kShellPart = 64;

template <int KIND>
__device__ __forceinline__ void run_one64(WaveStacks64 &W, int i)
{
    if (KIND == 0) {
        atomicAdd(&W.acc[W.ang_o[i]], W.ang[2][i] * atan2_f64(W.ang[0][i], W.ang[1][i]));
    } else {
        const double sR0 = W.pnt[1][i];
        const int o = W.pnt_o[i];
        const double v = part_term(W.pnt[0][i], fabs(sR0), W.pnt[2][i], W.pnt[3][i], (o & kShellPart) != 0);
        atomicAdd(&W.acc[o & 63], sR0 < 0.0 ? -v : v);
    }
}

template <int KIND>
__device__ __forceinline__ void run_stack64(WaveStacks64 &W, int &count, int lane, bool all)
{
    if (count >= 64) {
        lds_sync_wave();
        run_one64<KIND>(W, count - 64 + lane);
        count -= 64;
        lds_sync_wave();
    }
    if (all && count > 0) {
        lds_sync_wave();
        if (lane < count) run_one64<KIND>(W, lane);
        count = 0;
        lds_sync_wave();
    }
}

// Bound by FP64 VALU issue: 0.20 vector instructions per SIMD and clock (a
// dense FMA stream reaches 0.235), 79 % of the lanes active; 10.2e6 pairs of a
// clumpy cloud take 8.7 ms, and took 20.2 ms with two closed-form points per part,
// an angle task per part and the library's double functions.  WPE:
// resident wavefronts per SIMD the register budget is cut for (3: 168 VGPRs;
// when it took 10.1 ms, 2 waves took 12.2, and a budget for 4, which spills 60 to
// 100 registers, 27.7).
template <int WPE, bool MULTI>
__global__ void __launch_bounds__(256, WPE) k_integrate_queued64(JobsArg A, unsigned *tile_ctr)
{
    __shared__ WaveStacks64 stacks[4];
    const int lane = threadIdx.x & 63;
    WaveStacks64 &W = stacks[threadIdx.x >> 6];
    int probe = -1;
    int cur = MULTI ? -1 : 0;
    Work wk;      // walls and edges, per lane
    WaveWork ww;  // the rest
    auto flush = [&](unsigned long long *counters) { flush_wave_work(wk, ww, lane, counters); };
    for (;;) {
        const int64_t t = next_tile_xcd(tile_ctr + kXcdCtr, A.n_tiles, probe, lane);
        if (t < 0) break;
        const int jj = MULTI ? job_of_tile(A, t) : 0;
        if (MULTI && jj != cur) {
            if (cur >= 0) flush(A.table[cur].counters);
            cur = jj;
        }
        const EdgeRec *__restrict__ edges = JOB(edges);
        const double *__restrict__ plane = JOB(plane);
        const int64_t *__restrict__ fvo = JOB(fvo);
        const int sh = JOB(split), part = lane & ((1 << sh) - 1);  // 2^sh neighbouring lanes share a pair
        const int64_t k = (t - JOB(wave_base)) * (64 >> sh) + (lane >> sh);
        const bool active = k < JOB(np);
        double px = 0.0, py = 0.0, pz = 0.0, invh = 1.0;
        int32_t s = 0, s_end = 0, j = 0;
        if (active) {
            const int64_t a = JOB(pair_p)[k];
            const int64_t c = JOB(pair_c)[k];
            px = JOB(xyz)[3 * a];
            py = JOB(xyz)[3 * a + 1];
            pz = JOB(xyz)[3 * a + 2];
            invh = 1.0 / JOB(h)[a];
            const int64_t *__restrict__ cfo = JOB(cfo);
            const int64_t f0 = cfo[c], walls = cfo[c + 1] - f0, from = f0 + ((walls * part) >> sh);
            j = (int32_t)from - 1;
            s = (int32_t)fvo[from];
            s_end = (int32_t)fvo[f0 + ((walls * (part + 1)) >> sh)];
        }
        const bool far = mask_of(invh > JOB(far_invh)) != 0;  // edges beyond kFarLength may be among the tile's
        W.acc[lane] = 0.0;
        int32_t face_end = s;
        const int n_steps = __builtin_amdgcn_readfirstlane(wave_max((int)(s_end - s)));
        const EdgeRec *ep = edges + s;
        int nA = 0, nP = 0;
        unsigned at_walls = 0;  // walls whose plane holds the particle; top bit: it is outside of a wall
        bool face_ok = false;
        uint32_t wall_sign = 0;
        double r0 = 0.0, nHt = 0.0, dH = 0.0;
        double acc_in = 0.0;  // this lane's angle terms taken in place
        for (int it = 0; it < n_steps; it++, s++, ep++) {
            if (s == face_end) {
                face_ok = false;
                face_end = -1;
                if (s < s_end) {
                    j++;
                    face_end = (int32_t)fvo[j + 1];
                    const double *pl = plane + plane_at(j);
                    const double d = pl[3] - (pl[0] * px + pl[1] * py + pl[2] * pz);
                    wk.faces++;
                    const bool in_j = d >= 0.0;
                    at_walls = (at_walls + (d == 0.0)) | (in_j ? 0u : 0x80000000u);
                    wall_sign = in_j ? 0u : 0x80000000u;
                    r0 = fabs(d) * invh;
                    face_ok = r0 < 2.0;
                    if (face_ok) wk.edges += face_end - s;
                    nHt = -pi_H<double>(r0);
                    dH = pi_dH<double>(r0);
                }
            }
            uint64_t live = mask_of(face_ok);
            double E[10];  // the edge record (EdgeRec's order); some value or other in a lane without one
#pragma unroll
            for (int q = 0; q < 10; q++) asm volatile("" : "=v"(E[q]));
            if (lane_in(live)) {
                const double *from = reinterpret_cast<const double *>(ep);
#pragma unroll
                for (int q = 0; q < 10; q++) E[q] = from[q];
            }
            const double wx = px - E[0], wy = py - E[1], wz = pz - E[2];
            const double rho = E[7] * wx + E[8] * wy + E[9] * wz;
            live &= mask_of(rho != 0.0);
            const double la = -(E[4] * wx + E[5] * wy + E[6] * wz) * invh;
            const double Le = E[3] * invh, lb = la + Le;
            const double R0 = fabs(rho) * invh;
            const uint32_t sbit = ((uint32_t)__double2hiint(rho) ^ wall_sign) & 0x80000000u;  // of the edge's terms
            const EdgeParts P = edge_parts(lane_in(live), r0, R0, la, lb);
            const uint64_t near = mask_of(P.near);
            const uint64_t cut_a = mask_of(la < P.ca), cut_b = mask_of(P.cb < lb);  // (else ca = la, cb = lb)
            const uint64_t shell_a = near & mask_of(P.ca < P.ia), shell_b = near & mask_of(P.ib < P.cb);
            const uint64_t has_b = live & (cut_a | cut_b);
            const uint64_t has_s = (shell_a | shell_b) & mask_of(dH != 0.0);
            ww.eterms += __popcll(near);
            ww.angles += __popcll(has_b) + __popcll(has_s);
            {
                // the parts [la, b1] and [a2, lb] (a lane without beyond parts has ca = la and cb = lb)
                const double b1 = lane_in(has_b) ? P.ca : P.ia, a2 = lane_in(has_b) ? P.cb : P.ib;
                double y, x;
                angle_product(R0, la, b1, a2, lb, y, x);
                if (far) angle_product_far(R0, la, b1, a2, lb, y, x);
                const double w = lane_in(has_b) ? nHt : (lane_in(has_s) ? dH : 0.0);
                const double v = flip_sign(w, sbit) * atan2_f64(y, x);
                acc_in += lane_in(live) ? v : 0.0;
            }
            {
                const uint64_t m = has_b & has_s;
                if (m != 0) {
                    if (nA + __popcll(m) > kQA) run_stack64<0>(W, nA, lane, true);
                    const int slot = wave_push(m, nA);
                    if (lane_in(m)) {
                        double y, x;
                        angle_product(R0, P.ca, P.ia, P.ib, P.cb, y, x);
                        W.ang[0][slot] = y;
                        W.ang[1][slot] = x;
                        W.ang[2][slot] = flip_sign(dH, sbit);
                        W.ang_o[slot] = (uint8_t)lane;
                    }
                }
            }
            auto push_part = [&](uint64_t m, double x, double len, int kind) {
                if (m == 0) return;
                const int slot = wave_push(m, nP);
                ww.moments += __popcll(m);
                if (lane_in(m)) {
                    W.pnt[0][slot] = r0;
                    W.pnt[1][slot] = flip_sign(R0, sbit);
                    W.pnt[2][slot] = x;
                    W.pnt[3][slot] = len;
                    W.pnt_o[slot] = (uint8_t)(lane + kind);
                }
            };
            const uint64_t ia_end = mask_of(P.ia == lb), ib_start = mask_of(P.ib == la);
            push_part(shell_a, P.ca, lane_in(~cut_a & ia_end) ? Le : P.ia - P.ca, kShellPart);
            push_part(near & mask_of(P.ia < P.ib), P.ia, part_len(P.ia, P.ib, la, lb, Le), 0);
            if (nP > kQP - 64) run_stack64<1>(W, nP, lane, false);
            push_part(shell_b, P.ib, lane_in(~cut_b & ib_start) ? Le : P.cb - P.ib, kShellPart);
            while (nP >= 64) run_stack64<1>(W, nP, lane, false);
        }
        run_stack64<0>(W, nA, lane, true);
        run_stack64<1>(W, nP, lane, true);
        lds_sync_wave();
        double sum = W.acc[lane] + acc_in;
        for (int o = 1; o < 1 << sh; o <<= 1) {
            sum += __shfl_xor(sum, o, 64);
            at_walls = join_walls(at_walls, __shfl_xor(at_walls, o, 64));
        }
        const bool inside = at_walls < 0x80000000u;
        if (active && part == 0) {
            const double v = (inside ? 1.0 : 0.0) - sum * kInvPi;
            JOB(f)[k] = v;
            if (JOB(S)) atomicAdd(JOB(S) + JOB(pair_p)[k], fixed52(v));
            if (inside && at_walls >= 2) push_fix(FixList{JOB(fix_count), JOB(fix_items), JOB(fix_cap), nullptr}, k, kWindingSlot);
        }
        lds_sync_wave();
    }
    if (cur >= 0) flush(MULTI ? A.table[cur].counters : A.one.counters);
}
#undef JOB

// ---------------------------------------------------------------- cell tiles
// A tile is up to 64 consecutive pairs of one cell (key = cell << 32 | tile
// index within the cell).  A wavefront integrating a tile shares the cell, so
// the cell's walls and edge records are wave-uniform: they are read with
// scalar loads into scalar registers, and the face/edge loops are uniform.
__global__ void k_tile_counts(int64_t n_cells, const int64_t *__restrict__ coff, int64_t *__restrict__ tcnt)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_cells) tcnt[i] = (coff[i + 1] - coff[i] + 63) / 64;
}

__global__ void k_tile_fill(int64_t n_cells, const int64_t *__restrict__ toff, uint64_t *__restrict__ tiles)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_cells) return;
    for (int64_t u = 0; u < toff[i + 1] - toff[i]; u++) tiles[toff[i] + u] = ((uint64_t)i << 32) | (uint64_t)u;
}

template <int PREC>
__global__ void __launch_bounds__(256) k_integrate_tiles(int64_t n_tiles, const uint64_t *__restrict__ tiles,
                                                          const int64_t *__restrict__ coff,
                                                          const uint32_t *__restrict__ pair_p,
                                                          const double *__restrict__ xyz,
                                                          const double *__restrict__ h,
                                                          const int64_t *__restrict__ cfo,
                                                          const int64_t *__restrict__ fvo,
                                                          const double *__restrict__ plane,
                                                          const EdgeRec *__restrict__ edges, double *__restrict__ f,
                                                          unsigned long long *counters, unsigned *tile_ctr, FixList fx)
{
    using R = typename std::conditional<PREC == MAP_FP64, double, float>::type;
    const int lane = threadIdx.x & 63;
    Work wk;
    for (;;) {
        unsigned t = 0;
        if (lane == 0) t = atomicAdd(tile_ctr, 1u);
        t = __builtin_amdgcn_readfirstlane(t);
        if ((int64_t)t >= n_tiles) break;
        const uint64_t key = tiles[t];
        const int64_t cell = uniform64((int64_t)(key >> 32));
        const int64_t start = uniform64(coff[cell] + 64 * (int64_t)(key & 0xffffffffu));
        const int64_t end = uniform64(coff[cell + 1]);
        const int64_t k = start + lane;
        const bool active = k < end;
        double px = 0.0, py = 0.0, pz = 0.0, hh = 1.0;
        if (active) {
            const int64_t a = pair_p[k];
            px = xyz[3 * a];
            py = xyz[3 * a + 1];
            pz = xyz[3 * a + 2];
            hh = h[a];
        }
        const double invh = 1.0 / hh;
        bool inside = true;
        int n_on = 0;
        double acc = 0.0;
        float ev = 0.0f;
        const int64_t f0 = uniform64(cfo[cell]), f1 = uniform64(cfo[cell + 1]);
        for (int64_t j = f0; j < f1; j++) {
            const double nx = plane[4 * j], ny = plane[4 * j + 1], nz = plane[4 * j + 2], cj = plane[4 * j + 3];
            const double d = cj - (nx * px + ny * py + nz * pz);
            wk.faces += active;
            const bool in_j = d >= 0.0;
            inside = inside && in_j;
            n_on += d == 0.0 ? 1 : 0;
            const double r0d = fabs(d) * invh;
            const int64_t s0 = uniform64(fvo[j]), s1 = uniform64(fvo[j + 1]);
            if (active && r0d < 2.0) {
                const R r0 = (R)r0d;
                const R Ht = pi_H<R>(r0);
                const R dH = pi_dH<R>(r0);
                double face = 0.0;
                for (int64_t s = s0; s < s1; s++) {
                    const EdgeRec &E = edges[s];
                    const double wx = px - E.vx, wy = py - E.vy, wz = pz - E.vz;
                    const double rho = E.mx * wx + E.my * wy + E.mz * wz;
                    wk.edges++;
                    if (rho == 0.0) continue;
                    const double la = -(E.ex * wx + E.ey * wy + E.ez * wz) * invh;
                    const double Le = E.L * invh, lb = la + Le;
                    const double R0d = fabs(rho) * invh;
                    if (PREC == MAP_MIXED && needs_fp64(r0d, R0d, r0d * r0d + R0d * R0d)) {
                        const unsigned slot = atomicAdd(fx.count, 1u);
                        if (slot < fx.cap) fx.items[slot] = ((uint64_t)k << 32) | (uint64_t)(uint32_t)s;
                        continue;
                    }
                    const R tv = edge_term(r0, (R)R0d, (R)la, (R)lb, (R)Le, Ht, dH, wk);
                    face += (rho > 0.0) ? (double)tv : -(double)tv;
                    if (PREC == MAP_MIXED) ev = fmaf((float)tv, (float)tv, ev);
                }
                acc += in_j ? face : -face;
            }
        }
        if (active) {
            f[k] = winding_term(inside, n_on, px, py, pz, cell, cfo, fvo, plane, edges) - acc * kInvPi;
            if (PREC == MAP_MIXED && fx.err) fx.err[k] = kTermErr * kInvPiF * sqrt_f32(ev);
        }
    }
    flush_work(wk, counters);
}

// FP64 values of flagged edges (fixup items, key = pair << 32 | face-vertex slot)
__global__ void k_fixup_values(int64_t n_fix, const uint64_t *__restrict__ keys, const uint32_t *__restrict__ pair_p,
                               const uint32_t *__restrict__ pair_c, const double *__restrict__ xyz,
                               const double *__restrict__ h, const int64_t *__restrict__ cfo,
                               const int64_t *__restrict__ fvo, const double *__restrict__ plane,
                               const EdgeRec *__restrict__ edges, double *__restrict__ vals,
                               unsigned long long *counters)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_fix) return;
    const uint64_t key = keys[i];
    const int64_t k = (int64_t)(key >> 32);
    const int64_t s = (int64_t)(key & 0xffffffffu);
    const int64_t a = pair_p[k], c = pair_c[k];
    if ((uint32_t)s == kWindingSlot) {
        // the kernel took the winding weight of the particle as 1
        vals[i] = cell_winding(xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2], c, cfo, fvo, plane, edges) - 1.0;
        atomicAdd(counter_copy(counters) + C_WINDING, 1ull);
        return;
    }
    // the face of slot s within the cell
    int64_t lo = cfo[c], hi = cfo[c + 1] - 1;
    while (lo < hi) {
        const int64_t mid = (lo + hi + 1) >> 1;
        if (fvo[mid] <= s) lo = mid;
        else hi = mid - 1;
    }
    vals[i] = edge_contribution_fp64(xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2], h[a], plane + 4 * lo, edges[s]);
}

// Adds the (key-sorted) fixup values of each pair, in key order, to f.
__global__ void k_fixup_apply(int64_t n_fix, const uint64_t *__restrict__ keys, const double *__restrict__ vals,
                              const uint32_t *__restrict__ pair_p, double *__restrict__ f,
                              unsigned long long *__restrict__ S)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_fix) return;
    const uint64_t k = keys[i] >> 32;
    if (i > 0 && (keys[i - 1] >> 32) == k) return;
    double sum = 0.0;
    for (int64_t j = i; j < n_fix && (keys[j] >> 32) == k; j++) sum += vals[j];
    const double old = f[k];
    f[k] = old + sum;
    atomicAdd(S + pair_p[k], fixed52(old + sum) - fixed52(old));
}

// Node values of the tabulated pyramid integral I(r0, R0, phi) (the variant of
// Sec. II-B that interpolates a pre-computed table): r0 = 2 i / (n0 - 1),
// R0 = 2 j / (n1 - 1), phi = (pi/2) k / (n2 - 1) (the last plane at
// pi/2 - 1e-12), from the FP64 closed form above:
//     I = Omega / (4 pi) - (1/pi) [pi (Q - phi H)](0 .. l),   l = R0 tan(phi),
// with the triangle's solid angle Omega = atan2(l R0 (R0^2 + l^2), (S + r0)(R0^2 S + r0 l^2)).
__global__ void k_table_build(int n0, int n1, int n2, double *__restrict__ tab64)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t total = (int64_t)n0 * n1 * n2;
    if (q >= total) return;
    const int k = (int)(q % n2);
    const int j = (int)((q / n2) % n1);
    const int i = (int)(q / ((int64_t)n1 * n2));
    const double r0 = 2.0 * i / (double)(n0 - 1);
    const double R0 = 2.0 * j / (double)(n1 - 1);
    const double phi = k == n2 - 1 ? 0.5 * M_PI - 1e-12 : 0.5 * M_PI * k / (double)(n2 - 1);
    double I = 0.0;
    if (r0 > 0.0 && R0 > 0.0 && phi > 0.0) {
        const double l = R0 * tan(phi);
        const double S = sqrt(r0 * r0 + R0 * R0 + l * l);
        const double om = atan2(l * R0 * (R0 * R0 + l * l), (S + r0) * (R0 * R0 * S + r0 * l * l));
        Work wk;
        const double e = edge_term(r0, R0, 0.0, l, l, pi_H<double>(r0), pi_dH<double>(r0), wk);
        I = om * (0.25 * kInvPi) - e * kInvPi;
    }
    tab64[q] = I;
}

// The node values as the reads take them (em_table.hip).
__global__ void k_table_pack(int n0, int n1, int n2, const double *__restrict__ tab64, TabNode *__restrict__ tab4)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t dj = n2, di = (int64_t)n1 * n2;
    if (q >= (int64_t)n0 * di) return;
    const int j = (int)((q / n2) % n1), i = (int)(q / di);
    const bool in = i + 1 < n0 && j + 1 < n1;
    tab4[q] = in ? TabNode{(float)tab64[q], (float)tab64[q + dj], (float)tab64[q + di], (float)tab64[q + di + dj]}
                 : TabNode{0.0f, 0.0f, 0.0f, 0.0f};
}

}  // namespace

// The listed cells' pairs in FP64, to the bit as pair_fraction<MAP_FP64>
// (the per-pair FP64 form): each workgroup takes chunks of up to 32 of a cell's
// pairs (kRecBlocks workgroups per cell, chunks round-robin), computes every
// (pair, edge) term of a chunk in parallel, then a thread per (pair, wall) adds
// the wall's edges in order and a thread per pair its walls in order, as
// pair_fraction does, so the result is the FP64 path's to the bit (cells of up to
// 64 walls and kRecTerms slots; larger ones take one thread per pair).  Bound by
// FP64 issue.  With a thread for all edges of a (pair, wall), where lanes wait for
// the wall of the most edges, 76,574 pairs of 729 cells took 141 us and 385 pairs
// of 9 cells 40; now 103 and 25.
constexpr int kRecPairs = 32, kRecBlocks = 4, kRecWalls = 64, kRecTerms = 2048;

__global__ void __launch_bounds__(256) k_recompute_cells(int64_t n_list, const uint32_t *__restrict__ cells,
                                                         const int64_t *__restrict__ coff,
                                                         const uint32_t *__restrict__ pair_p,
                                                         const double *__restrict__ xyz, const double *__restrict__ h,
                                                         const int64_t *__restrict__ cfo,
                                                         const int64_t *__restrict__ fvo,
                                                         const double *__restrict__ plane,
                                                         const EdgeRec *__restrict__ edges, double *__restrict__ f,
                                                         unsigned long long *__restrict__ S,
                                                         unsigned long long *counters)
{
    __shared__ double term[kRecTerms];               // of a (pair, slot), with the edge's sign
    __shared__ double wall[kRecPairs * kRecWalls];   // of a (pair, wall): its distance, then its sum
    __shared__ uint8_t side[kRecPairs * kRecWalls];  // of a (pair, wall): bit 0: distance >= 0, bit 1: 0
    __shared__ uint8_t wall_of[kRecTerms];           // of the cell's slots
    const int64_t q = blockIdx.x;
    if (q >= n_list) return;
    const int64_t c = cells[q];
    const int64_t f0 = cfo[c], nw = cfo[c + 1] - f0;
    const int64_t k0 = coff[c], np = coff[c + 1] - k0;
    const int64_t s0 = fvo[f0], ns = fvo[f0 + nw] - s0;
    if (nw > kRecWalls || ns > kRecTerms) {  // larger cells: one thread per pair
        for (int64_t k = k0 + (int64_t)blockIdx.y * blockDim.x + threadIdx.x; k < k0 + np;
             k += (int64_t)gridDim.y * blockDim.x) {
            const int64_t a = pair_p[k];
            Work wk;
            float ev = 0.0f;
            const double v = pair_fraction<MAP_FP64>(xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2], h[a], c, cfo, fvo,
                                                     plane, edges, wk, (uint64_t)k, nullptr, nullptr, 0u, ev);
            atomicAdd(S + a, fixed52(v) - fixed52(f[k]));
            f[k] = v;
        }
    } else {
        const int W = (int)nw, slots = (int)ns;
        for (int w = threadIdx.x; w < W; w += blockDim.x)
            for (int64_t sl = fvo[f0 + w]; sl < fvo[f0 + w + 1]; sl++) wall_of[sl - s0] = (uint8_t)w;
        const int per = slots > 0 ? min(kRecPairs, kRecTerms / slots) : kRecPairs;  // pairs of a chunk
        for (int64_t pb = (int64_t)blockIdx.y * per; pb < np; pb += (int64_t)gridDim.y * per) {
            const int nc = (int)(np - pb < per ? np - pb : per);
            __syncthreads();  // the previous chunk's sums are done
            for (int it = threadIdx.x; it < nc * W; it += blockDim.x) {
                const int p = it / W, w = it - p * W;
                const int64_t a = pair_p[k0 + pb + p];
                const double px = xyz[3 * a], py = xyz[3 * a + 1], pz = xyz[3 * a + 2];
                const int64_t j = f0 + w;
                const double nx = plane[4 * j], ny = plane[4 * j + 1], nz = plane[4 * j + 2], cj = plane[4 * j + 3];
                wall[it] = cj - (nx * px + ny * py + nz * pz);
            }
            __syncthreads();
            for (int it = threadIdx.x; it < nc * slots; it += blockDim.x) {
                const int p = it / slots, sl = it - p * slots;
                const int64_t a = pair_p[k0 + pb + p];
                const double invh = 1.0 / h[a];
                const double r0d = fabs(wall[p * W + wall_of[sl]]) * invh;
                double t = 0.0;
                if (r0d < 2.0) {
                    const EdgeRec E = edges[s0 + sl];
                    const double wx = xyz[3 * a] - E.vx, wy = xyz[3 * a + 1] - E.vy, wz = xyz[3 * a + 2] - E.vz;
                    const double rho = E.mx * wx + E.my * wy + E.mz * wz;
                    if (rho != 0.0) {
                        Work wk;
                        const double la = -(E.ex * wx + E.ey * wy + E.ez * wz) * invh;
                        const double Le = E.L * invh;
                        t = edge_term(r0d, fabs(rho) * invh, la, la + Le, Le, pi_H<double>(r0d), pi_dH<double>(r0d), wk);
                        t = (rho > 0.0) ? t : -t;
                    }
                }
                term[it] = t;
            }
            __syncthreads();
            for (int it = threadIdx.x; it < nc * W; it += blockDim.x) {
                const int p = it / W, w = it - p * W;
                const double d = wall[it];
                side[it] = (uint8_t)((d >= 0.0 ? 1 : 0) | (d == 0.0 ? 2 : 0));
                const int q0 = (int)(fvo[f0 + w] - s0), q1 = (int)(fvo[f0 + w + 1] - s0);
                double face = 0.0;
                for (int q = q0; q < q1; q++) face += term[p * slots + q];
                wall[it] = face;
            }
            __syncthreads();
            for (int p = threadIdx.x; p < nc; p += blockDim.x) {
                const int64_t k = k0 + pb + p, a = pair_p[k];
                bool inside = true;
                int n_on = 0;
                double acc = 0.0;
                for (int w = 0; w < W; w++) {
                    const uint8_t sd = side[p * W + w];
                    const bool in_j = (sd & 1) != 0;
                    inside = inside && in_j;
                    n_on += (sd >> 1) & 1;
                    const double face = wall[p * W + w];
                    acc += in_j ? face : -face;
                }
                const double v = winding_term(inside, n_on, xyz[3 * a], xyz[3 * a + 1], xyz[3 * a + 2], c, cfo, fvo,
                                              plane, edges) -
                                 acc * kInvPi;
                atomicAdd(S + a, fixed52(v) - fixed52(f[k]));
                f[k] = v;
            }
        }
    }
    if (threadIdx.x == 0 && blockIdx.y == 0) atomicAdd(counter_copy(counters) + C_FP64_PAIRS, (unsigned long long)np);
}

void launch_table_build(int n0, int n1, int n2, double *tab64, TabNode *tab4, hipStream_t s)
{
    const int64_t total = (int64_t)n0 * n1 * n2;
    const dim3 g((unsigned)((total + 255) / 256));
    hipLaunchKernelGGL(k_table_build, g, dim3(256), 0, s, n0, n1, n2, tab64);
    EM_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_table_pack, g, dim3(256), 0, s, n0, n1, n2, (const double *)tab64, tab4);
    EM_HIP(hipGetLastError());
}

void build_tiles(Workspace &ws, const DevInputs &in, PairSet &ps, hipStream_t s)
{
    const int64_t nc = in.n_cells;
    ps.n_tiles = 0;
    if (nc == 0 || ps.n_pairs == 0) return;
    int64_t *tcnt = ws.get<int64_t>(S_TILE_CNT, (size_t)nc);
    int64_t *toff = ws.get<int64_t>(S_TILE_OFF, (size_t)nc + 1);
    hipLaunchKernelGGL(k_tile_counts, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s, nc, ps.coff, tcnt);
    EM_HIP(hipGetLastError());
    scan_counts(ws, tcnt, toff, nc, s);
    int64_t nt = 0;
    read_back(ws, {{&nt, toff + nc, sizeof(int64_t)}}, s);
    uint64_t *tiles = ws.get<uint64_t>(S_TILES, (size_t)(nt > 0 ? nt : 1));
    hipLaunchKernelGGL(k_tile_fill, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, s, nc, (const int64_t *)toff,
                       tiles);
    EM_HIP(hipGetLastError());
    ps.tiles = tiles;
    ps.n_tiles = nt;
}

// The task-batch kernels (distribution 3) over one job (its entry passed by
// value) or several (the table in device memory, h_jobs its host copy): the
// tile space of a launch is the concatenation of the jobs' tiles.
static void launch_queued(const IntJob *h_jobs, const IntJob *d_jobs, int n_jobs, int precision,
                          const IntegrateTune &tune, unsigned *tile_ctr, bool zero_ctr, hipStream_t s)
{
    EM_CHECK(n_jobs >= 1 && h_jobs, MAP_EINVAL, "integration launch without jobs");
    EM_CHECK(n_jobs == 1 || d_jobs, MAP_EINVAL, "integration launch of several jobs without a device table");
    int64_t blocks64 = 0, tiles = 0;
    for (int i = 0; i < n_jobs; i++) {
        EM_CHECK(h_jobs[i].tile_base == blocks64 && h_jobs[i].wave_base == tiles && h_jobs[i].np > 0, MAP_EINVAL,
                 "integration job table: tile bases are not the running tile count");
        EM_CHECK(h_jobs[i].split == job_split(h_jobs[i].np, precision), MAP_EINVAL,
                 "integration job table: a job's split is not the one of its size");
        blocks64 += (h_jobs[i].np + 63) / 64;
        tiles += job_tiles(h_jobs[i]);
    }
    JobsArg A;
    A.table = d_jobs;
    A.n = n_jobs;
    A.n_tiles = tiles;
    A.one = h_jobs[0];
    if (zero_ctr) fill_zero_bytes(tile_ctr, kLaunchCtrs * sizeof(unsigned), s);
    const int block = 256;
    int64_t g = (int64_t)device_cu_count() * (tune.grid_per_cu > 0 ? tune.grid_per_cu : 8);
    const int64_t need = (tiles + (block / 64) - 1) / (block / 64);
    if (g > need) g = need;
    if (g < 1) g = 1;
    const bool multi = n_jobs > 1;
#define EM_LAUNCH_Q(...) hipLaunchKernelGGL((__VA_ARGS__), dim3((unsigned)g), dim3(block), 0, s, A, tile_ctr)
    if (precision == MAP_FP64 && tune.waves >= 3) {
        if (multi) EM_LAUNCH_Q(k_integrate_queued64<3, true>);
        else EM_LAUNCH_Q(k_integrate_queued64<3, false>);
    } else if (precision == MAP_FP64) {
        if (multi) EM_LAUNCH_Q(k_integrate_queued64<2, true>);
        else EM_LAUNCH_Q(k_integrate_queued64<2, false>);
    } else if (tune.waves >= 6 || tune.waves <= 0) {
        if (multi) EM_LAUNCH_Q(k_integrate_queued<6, true>);
        else EM_LAUNCH_Q(k_integrate_queued<6, false>);
    } else if (tune.waves >= 3) {
        if (multi) EM_LAUNCH_Q(k_integrate_queued<3, true>);
        else EM_LAUNCH_Q(k_integrate_queued<3, false>);
    } else {
        if (multi) EM_LAUNCH_Q(k_integrate_queued<2, true>);
        else EM_LAUNCH_Q(k_integrate_queued<2, false>);
    }
#undef EM_LAUNCH_Q
    EM_HIP(hipGetLastError());
}

void launch_integrate(const DevInputs &in, const EdgeRec *edges, const PairSet &ps, int precision,
                      const IntegrateTune &tune, double *f, float *err, double *S, int64_t *counters,
                      uint32_t *tile_ctr, uint64_t *fix_items, int64_t fix_cap, hipStream_t s)
{
    const int64_t np = ps.n_pairs;
    if (np == 0) return;
    if (tune.persistent != 3 && S) {  // the other distributions leave the sums to a pass of their own
        launch_integrate(in, edges, ps, precision, tune, f, err, nullptr, counters, tile_ctr, fix_items, fix_cap, s);
        launch_particle_sum(ps, f, S, s);
        return;
    }
    unsigned long long *cnt = reinterpret_cast<unsigned long long *>(counters);
    FixList fx;
    fx.count = tile_ctr + 1;
    fx.items = fix_items;
    fx.cap = (unsigned)(fix_cap > 0xffffffffLL ? 0xffffffffLL : fix_cap);
    fx.err = precision == MAP_MIXED ? err : nullptr;
    fill_zero_bytes(tile_ctr, kLaunchCtrs * sizeof(unsigned), s);
    const int block = 256;
    if (!tune.persistent) {
        const unsigned g = (unsigned)((np + block - 1) / block);
        if (precision == MAP_FP64)
            hipLaunchKernelGGL(k_integrate_flat<MAP_FP64>, dim3(g), dim3(block), 0, s, np, ps.pair_p, ps.pair_c, in.xyz,
                               in.h, in.cfo, in.fvo, in.plane, edges, f, cnt, fx);
        else
            hipLaunchKernelGGL(k_integrate_flat<MAP_MIXED>, dim3(g), dim3(block), 0, s, np, ps.pair_p, ps.pair_c,
                               in.xyz, in.h, in.cfo, in.fvo, in.plane, edges, f, cnt, fx);
        EM_HIP(hipGetLastError());
        return;
    }
    if (tune.persistent == 3) {
        IntJob J;
        J.np = np;
        J.split = job_split(np, precision);
        J.tile_base = J.wave_base = 0;
        J.pair_p = ps.pair_p;
        J.pair_c = ps.pair_c;
        J.far_invh = far_invh(in.box);
        J.xyz = in.xyz;
        J.h = in.h;
        J.cfo = in.cfo;
        J.fvo = in.fvo;
        J.plane = in.plane;
        J.edges = edges;
        J.f = f;
        J.err = fx.err;
        J.S = reinterpret_cast<unsigned long long *>(S);
        J.counters = cnt;
        J.fix_count = fx.count;
        J.fix_items = fx.items;
        J.fix_cap = fx.cap;
        launch_queued(&J, nullptr, 1, precision, tune, tile_ctr, false, s);
        return;
    }
    if (tune.persistent == 2 && ps.tiles) {
        int64_t g = (int64_t)device_cu_count() * (tune.grid_per_cu > 0 ? tune.grid_per_cu : 8);
        int64_t need = (ps.n_tiles + (block / 64) - 1) / (block / 64);
        if (g > need) g = need;
        if (g < 1) g = 1;
        if (precision == MAP_FP64)
            hipLaunchKernelGGL(k_integrate_tiles<MAP_FP64>, dim3((unsigned)g), dim3(block), 0, s, ps.n_tiles,
                               ps.tiles, ps.coff, ps.pair_p, in.xyz, in.h, in.cfo, in.fvo, in.plane, edges, f, cnt,
                               tile_ctr, fx);
        else
            hipLaunchKernelGGL(k_integrate_tiles<MAP_MIXED>, dim3((unsigned)g), dim3(block), 0, s, ps.n_tiles,
                               ps.tiles, ps.coff, ps.pair_p, in.xyz, in.h, in.cfo, in.fvo, in.plane, edges, f, cnt,
                               tile_ctr, fx);
        EM_HIP(hipGetLastError());
        return;
    }
    const int tw = tune.tile_waves > 0 ? tune.tile_waves : 1;
    int64_t tiles = (np + 64 * tw - 1) / (64 * tw);
    int64_t g = (int64_t)device_cu_count() * (tune.grid_per_cu > 0 ? tune.grid_per_cu : 8);
    int64_t need = (tiles + (block / 64) - 1) / (block / 64);
    if (g > need) g = need;
    if (g < 1) g = 1;
#define EM_LAUNCH_P(P, W)                                                                                         \
    hipLaunchKernelGGL((k_integrate_persistent<P, W>), dim3((unsigned)g), dim3(block), 0, s, np, ps.pair_p,      \
                       ps.pair_c, in.xyz, in.h, in.cfo, in.fvo, in.plane, edges, f, cnt, tile_ctr, tw, fx)
    const int w = tune.waves;
    if (precision == MAP_FP64) {
        if (w >= 4) EM_LAUNCH_P(MAP_FP64, 4);
        else if (w == 3) EM_LAUNCH_P(MAP_FP64, 3);
        else EM_LAUNCH_P(MAP_FP64, 2);
    } else {
        if (w >= 6) EM_LAUNCH_P(MAP_MIXED, 6);
        else if (w == 5) EM_LAUNCH_P(MAP_MIXED, 5);
        else EM_LAUNCH_P(MAP_MIXED, 4);
    }
#undef EM_LAUNCH_P
    EM_HIP(hipGetLastError());
}

void launch_integrate_jobs(const IntJob *h_jobs, const IntJob *d_jobs, int n_jobs, int precision,
                           const IntegrateTune &tune, unsigned *tile_ctr, hipStream_t s)
{
    launch_queued(h_jobs, d_jobs, n_jobs, precision, tune, tile_ctr, true, s);
}

void launch_recompute_cells(const DevInputs &in, const EdgeRec *edges, const PairSet &ps, const uint32_t *cells,
                            int64_t n_cells, double *f, double *S, int64_t *counters, hipStream_t s)
{
    if (n_cells <= 0) return;
    hipLaunchKernelGGL(k_recompute_cells, dim3((unsigned)n_cells, kRecBlocks), dim3(256), 0, s, n_cells,
                       cells, ps.coff, ps.pair_p, in.xyz, in.h, in.cfo, in.fvo, in.plane, edges, f,
                       reinterpret_cast<unsigned long long *>(S), reinterpret_cast<unsigned long long *>(counters));
    EM_HIP(hipGetLastError());
}

void launch_fixup(const DevInputs &in, const EdgeRec *edges, const PairSet &ps, const uint64_t *fix_keys,
                  int64_t n_fix, double *fix_vals, int64_t *counters, hipStream_t s)
{
    if (n_fix <= 0) return;
    hipLaunchKernelGGL(k_fixup_values, dim3((unsigned)((n_fix + 255) / 256)), dim3(256), 0, s, n_fix, fix_keys,
                       ps.pair_p, ps.pair_c, in.xyz, in.h, in.cfo, in.fvo, in.plane, edges, fix_vals,
                       reinterpret_cast<unsigned long long *>(counters));
    EM_HIP(hipGetLastError());
}

void launch_fixup_apply(const uint64_t *keys, const double *vals, int64_t n_fix, const uint32_t *pair_p, double *f,
                        double *S, hipStream_t s)
{
    if (n_fix <= 0) return;
    hipLaunchKernelGGL(k_fixup_apply, dim3((unsigned)((n_fix + 255) / 256)), dim3(256), 0, s, n_fix, keys, vals,
                       pair_p, f, reinterpret_cast<unsigned long long *>(S));
    EM_HIP(hipGetLastError());
}

}  // namespace em
