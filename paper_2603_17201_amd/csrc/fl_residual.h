// Sim3 reprojection residual, its hand-written backward, the float64 Sim3
// exponential and the Gauss-Newton step, plus per-event refinement of the
// loop Sim3 on the pairs a search accepted.
//
// The paper refines the loop Sim3 between its two projection searches
// (Sec. IV-C) and optimises poses with Jacobians it obtains by automatic
// differentiation (Sec. IV-F).  Here the residual of a matched pair is
//   p = sR X + t,  q = R_k p + t_k,  r = pi(q) - uv,
// its Jacobian with respect to a left perturbation xi = (omega, upsilon,
// sigma) of the Sim3 is written out by hand,
//   J = dpi/dq R_k [ -[p]x | I | p ],
// per-pair arithmetic is float32 and every sum is float64 with a fixed
// reduction order (thread, wave, block, then blocks in index order).
#pragma once

#include "fl_internal.h"

namespace fl {

constexpr int kResBlock = 256;
constexpr int kNAcc = kNAccPad;   // 7 gradient + 28 upper-triangle H + 1 count / loss

// ---------------------------------------------------------------------------
// float64 Sim3 algebra

struct Sim3d {
    double R[9];
    double t[3];
    double s;
};

// 1 / (i + 1), i < 72
struct RecipTable {
    double v[72];
    constexpr RecipTable() : v() {
        for (int i = 0; i < 72; ++i) v[i] = 1.0 / (double)(i + 1);
    }
};
__device__ constexpr RecipTable kRecip{};

// 1/x to within about one ulp: the hardware estimate r (relative error below
// 2^-22) and one step of third order, r (1 + e + e^2) with e = 1 - x r
// (cheaper on the serial path of a step than a correctly rounded division or
// two Newton steps).
__device__ __forceinline__ double recip(double x) {
    const double r = __builtin_amdgcn_rcp(x);
    const double e = fma(-x, r, 1.0);
    return fma(r, fma(e, e, e), r);
}

// The first NT terms of e^sigma = sum_k sigma^k / k! and of
// I_n(sigma) = integral_0^1 tau^n e^{sigma tau} d tau = sum_k sigma^k / (k! (n + k + 1)), n = 0..6.
template <int NT>
__device__ __forceinline__ void sigma_series(double sig, double* I, double& es) {
    double p[NT];
    p[0] = 1.0;
#pragma unroll
    for (int k = 1; k < NT; ++k) p[k] = p[k - 1] * sig * kRecip.v[k - 1];   // sigma^k / k!
    es = 0.0;
#pragma unroll
    for (int k = NT - 1; k >= 0; --k) es += p[k];
#pragma unroll
    for (int n = 0; n < 7; ++n) {
        double v = 0.0;
#pragma unroll
        for (int k = NT - 1; k >= 0; --k) v = fma(p[k], kRecip.v[n + k], v);
        I[n] = v;
    }
}

// Coefficients of the exponential of xi = (omega, upsilon, sigma):
// R = I + a W + b W^2 with W = [omega]x, s = e^sigma, and
// V = c0 I + c1 W + c2 W^2 = integral_0^1 e^{sigma tau} exp(tau W) d tau
// (closed form; series for small rotation angles), t = V upsilon.
struct ExpCoef {
    double a, b, c0, c1, c2, es;
};

__device__ __noinline__ ExpCoef sim3_exp_coef_full(double w0, double w1, double w2, double sig) {
    const double th2 = w0 * w0 + w1 * w1 + w2 * w2;
    const bool small = th2 < 1e-4;   // angle below 1e-2: the series need only th^2
    // th, sin th and cos th only where the series do not serve (taken inside
    // the branch, so that the common small-angle path does not wait for a
    // square root whose result it never uses)
    double th = 0.0, sn = 0.0, cs = 1.0;
    ExpCoef k;
    if (small) {
        // sin(th)/th and (1 - cos(th))/th^2 by their Taylor series: the next
        // terms are below th^8/9! < 3e-22 here
        const double t4 = th2 * th2;
        k.a = 1.0 - th2 * (1.0 / 6.0) + t4 * (1.0 / 120.0) - t4 * th2 * (1.0 / 5040.0);
        k.b = 0.5 - th2 * (1.0 / 24.0) + t4 * (1.0 / 720.0) - t4 * th2 * (1.0 / 40320.0);
    } else {
        th = sqrt(th2);
        sn = sin(th);
        cs = cos(th);
        k.a = sn / th;
        k.b = (1.0 - cs) / th2;
    }
    // I_n(sigma) for n = 0..6 and e^sigma = sum_k sigma^k / k! share one series
    double I[7];
    double es;
    const double asig = fabs(sig);
    if (asig < 2.5e-4) {
        sigma_series<5>(sig, I, es);   // remainder below 2.5e-4^5 / 5! < 1e-20
    } else if (asig < 4e-3) {
        sigma_series<7>(sig, I, es);   // below 4e-3^7 / 7! < 1e-20
    } else if (asig < 0.01) {
        sigma_series<9>(sig, I, es);   // below 0.01^9 / 9! < 3e-24
    } else if (fabs(sig) < 2.0) {
        double term = 1.0, e = 0.0;
        for (int n = 0; n < 7; ++n) I[n] = 0.0;
        for (int kk = 0; kk < 60; ++kk) {
            e += term;
#pragma unroll
            for (int n = 0; n < 7; ++n) I[n] += term * kRecip.v[n + kk];
            if (fabs(term) < 1e-18 * e) break;
            term *= sig * kRecip.v[kk];
        }
        es = e;
    } else {
        es = exp(sig);
        I[0] = expm1(sig) / sig;
        for (int m = 1; m < 7; ++m) I[m] = (es - (double)m * I[m - 1]) / sig;
    }
    k.es = es;
    k.c0 = I[0];
    if (small) {
        k.c1 = I[1] - th2 * (1.0 / 6.0) * I[3] + th2 * th2 * (1.0 / 120.0) * I[5];
        k.c2 = 0.5 * I[2] - th2 * (1.0 / 24.0) * I[4] + th2 * th2 * (1.0 / 720.0) * I[6];
    } else {
        const double den = sig * sig + th2;
        k.c1 = (es * (sig * sn - th * cs) + th) / (th * den);
        k.c2 = (k.c0 - (es * (sig * cs + th * sn) - sig) / den) / th2;
    }
    return k;
}

// The same coefficients, with the usual Gauss-Newton step (rotation angle
// below 1e-2, |sigma| below 1e-2) computed in line by the very same series
// and every other step by the out-of-line function above: the common case
// costs no call, and the code placed in line stays small enough not to push
// a kernel that holds many registers into spilling them.
__device__ __forceinline__ ExpCoef sim3_exp_coef(double w0, double w1, double w2, double sig) {
    const double th2 = w0 * w0 + w1 * w1 + w2 * w2;
    const double asig = fabs(sig);
    if (!(th2 < 1e-4 && asig < 0.01)) return sim3_exp_coef_full(w0, w1, w2, sig);
    ExpCoef k;
    const double t4 = th2 * th2;
    k.a = 1.0 - th2 * (1.0 / 6.0) + t4 * (1.0 / 120.0) - t4 * th2 * (1.0 / 5040.0);
    k.b = 0.5 - th2 * (1.0 / 24.0) + t4 * (1.0 / 720.0) - t4 * th2 * (1.0 / 40320.0);
    double I[7];
    double es;
    if (asig < 2.5e-4) sigma_series<5>(sig, I, es);
    else if (asig < 4e-3) sigma_series<7>(sig, I, es);
    else sigma_series<9>(sig, I, es);
    k.es = es;
    k.c0 = I[0];
    k.c1 = I[1] - th2 * (1.0 / 6.0) * I[3] + th2 * th2 * (1.0 / 120.0) * I[5];
    k.c2 = 0.5 * I[2] - th2 * (1.0 / 24.0) * I[4] + th2 * th2 * (1.0 / 720.0) * I[6];
    return k;
}

__device__ inline void hat_sq(double w0, double w1, double w2, double* W, double* W2) {
    W[0] = 0.0; W[1] = -w2; W[2] = w1;
    W[3] = w2; W[4] = 0.0; W[5] = -w0;
    W[6] = -w1; W[7] = w0; W[8] = 0.0;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j)
            W2[3 * i + j] = W[3 * i] * W[j] + W[3 * i + 1] * W[3 + j] + W[3 * i + 2] * W[6 + j];
}

// exp of a tangent xi = (omega, upsilon, sigma)
__device__ inline Sim3d sim3_exp(const double* xi) {
    const ExpCoef k = sim3_exp_coef(xi[0], xi[1], xi[2], xi[6]);
    double W[9], W2[9];
    hat_sq(xi[0], xi[1], xi[2], W, W2);
    Sim3d S;
    double V[9];
    for (int i = 0; i < 9; ++i) {
        const double I = (i % 4 == 0) ? 1.0 : 0.0;
        S.R[i] = I + k.a * W[i] + k.b * W2[i];
        V[i] = k.c0 * I + k.c1 * W[i] + k.c2 * W2[i];
    }
    for (int i = 0; i < 3; ++i) S.t[i] = V[3 * i] * xi[3] + V[3 * i + 1] * xi[4] + V[3 * i + 2] * xi[5];
    S.s = k.es;
    return S;
}

// log of a Sim3: omega from R (axis-angle, atan2 of the skew part's norm and
// the trace), sigma = ln s, upsilon solving V upsilon = t (Cramer's rule).
__device__ inline void sim3_log(const Sim3d& S, double* xi) {
    const double* R = S.R;
    const double v0 = 0.5 * (R[7] - R[5]), v1 = 0.5 * (R[2] - R[6]), v2 = 0.5 * (R[3] - R[1]);
    const double c = 0.5 * (R[0] + R[4] + R[8] - 1.0);
    const double sn = sqrt(v0 * v0 + v1 * v1 + v2 * v2);
    const double th = atan2(sn, c);
    double w0, w1, w2;
    if (sn > 1e-7 || c > 0.0) {
        // omega = th / sin(th) v; the series 1 + th^2/6 + 7 th^4/360 below 1e-4
        const double f = th < 1e-4 ? 1.0 + th * th * (1.0 / 6.0) + 7.0 * th * th * th * th / 360.0 : th / sn;
        w0 = f * v0;
        w1 = f * v1;
        w2 = f * v2;
    } else {
        // th near pi: the axis from the largest diagonal entry of (R + I) / 2
        int m = 0;
        if (R[4] > R[0]) m = 1;
        if (R[8] > R[4 * m]) m = 2;
        double ax[3];
        ax[m] = sqrt(fmax(0.0, 0.5 * (R[4 * m] + 1.0)));
        for (int j = 0; j < 3; ++j)
            if (j != m) ax[j] = 0.5 * (R[3 * m + j] + R[3 * j + m]) / (2.0 * ax[m]);
        w0 = th * ax[0];
        w1 = th * ax[1];
        w2 = th * ax[2];
    }
    const double sig = log(S.s);
    const ExpCoef k = sim3_exp_coef(w0, w1, w2, sig);
    double W[9], W2[9], V[9];
    hat_sq(w0, w1, w2, W, W2);
    for (int i = 0; i < 9; ++i) V[i] = k.c0 * ((i % 4 == 0) ? 1.0 : 0.0) + k.c1 * W[i] + k.c2 * W2[i];
    const double A0 = V[4] * V[8] - V[5] * V[7], A1 = V[5] * V[6] - V[3] * V[8], A2 = V[3] * V[7] - V[4] * V[6];
    const double det = V[0] * A0 + V[1] * A1 + V[2] * A2;
    const double id = 1.0 / det;
    const double* t = S.t;
    // upsilon = V^-1 t = adj(V) t / det(V)
    xi[3] = (A0 * t[0] + (V[2] * V[7] - V[1] * V[8]) * t[1] + (V[1] * V[5] - V[2] * V[4]) * t[2]) * id;
    xi[4] = (A1 * t[0] + (V[0] * V[8] - V[2] * V[6]) * t[1] + (V[2] * V[3] - V[0] * V[5]) * t[2]) * id;
    xi[5] = (A2 * t[0] + (V[1] * V[6] - V[0] * V[7]) * t[1] + (V[0] * V[4] - V[1] * V[3]) * t[2]) * id;
    xi[0] = w0;
    xi[1] = w1;
    xi[2] = w2;
    xi[6] = sig;
}

// S^-1 = (R^T, -R^T t / s, 1 / s)
__device__ inline Sim3d sim3_inv(const Sim3d& S) {
    Sim3d V;
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) V.R[3 * i + j] = S.R[3 * j + i];
    V.s = 1.0 / S.s;
    for (int i = 0; i < 3; ++i)
        V.t[i] = -(V.R[3 * i] * S.t[0] + V.R[3 * i + 1] * S.t[1] + V.R[3 * i + 2] * S.t[2]) * V.s;
    return V;
}

// A o B  (X -> A(B(X)))
__device__ inline Sim3d sim3_mul(const Sim3d& A, const Sim3d& B) {
    Sim3d C;
    for (int i = 0; i < 3; ++i) {
        for (int j = 0; j < 3; ++j)
            C.R[3 * i + j] = A.R[3 * i] * B.R[j] + A.R[3 * i + 1] * B.R[3 + j] + A.R[3 * i + 2] * B.R[6 + j];
        C.t[i] = A.s * (A.R[3 * i] * B.t[0] + A.R[3 * i + 1] * B.t[1] + A.R[3 * i + 2] * B.t[2]) + A.t[i];
    }
    C.s = A.s * B.s;
    return C;
}

__device__ inline Sim3d sim3_load(const double* p) {
    Sim3d S;
    for (int i = 0; i < 9; ++i) S.R[i] = p[i];
    for (int i = 0; i < 3; ++i) S.t[i] = p[9 + i];
    S.s = p[12];
    return S;
}

__device__ inline void sim3_store(const Sim3d& S, double* p) {
    for (int i = 0; i < 9; ++i) p[i] = S.R[i];
    for (int i = 0; i < 3; ++i) p[9 + i] = S.t[i];
    p[12] = S.s;
}

__device__ inline void sim3_to_f32(const Sim3d& S, fl_sim3* o) {
    for (int i = 0; i < 9; ++i) o->sR[i] = (float)(S.s * S.R[i]);
    for (int i = 0; i < 3; ++i) o->t[i] = (float)S.t[i];
    o->inv_s = (float)(1.0 / S.s);
    o->pad[0] = o->pad[1] = o->pad[2] = 0.0f;
}

// The part of the float32 form the residual reads (sR, t), for the steps
// inside a refinement; inv_s is filled in once at the end.
__device__ inline void sim3_to_f32_pose(const Sim3d& S, fl_sim3* o) {
    for (int i = 0; i < 9; ++i) o->sR[i] = (float)(S.s * S.R[i]);
    for (int i = 0; i < 3; ++i) o->t[i] = (float)S.t[i];
}

// Solve (H + lambda diag H) d = -g by an LDL^T factorisation (no square
// roots; one reciprocal per pivot); H given as its 28 upper entries row by
// row.  Returns false (d = 0) for a pivot that is not clearly positive.
// Right-looking, on the packed lower triangle (a[i(i+1)/2 + j] = H[i][j]):
// each pivot's column is scaled and its rank-1 product subtracted from the
// rest at once, with the forward substitution folded in, and the back
// substitution likewise updates every open right-hand side once an unknown is
// known.  It runs on one lane, so its dependency chain is its cost: per pivot
// one reciprocal, one multiply and one fused multiply-add deep, the updates
// themselves independent of one another.
__device__ inline bool solve7(const double* g, const double* Hu, double lambda, double* d) {
    double a[28];
    double dmax = 0.0;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j) a[i * (i + 1) / 2 + j] = Hu[j * 7 - j * (j - 1) / 2 + (i - j)];
        a[i * (i + 1) / 2 + i] *= (1.0 + lambda);
        dmax = fmax(dmax, fabs(a[i * (i + 1) / 2 + i]));
    }
    double y[7], Dinv[7], L[21];   // L[i(i-1)/2 + j] = L[i][j], j < i
#pragma unroll
    for (int i = 0; i < 7; ++i) y[i] = -g[i];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const double dj = a[j * (j + 1) / 2 + j];
        ok = ok && dj > 1e-14 * dmax;
        Dinv[j] = recip(dj);
#pragma unroll
        for (int i = j + 1; i < 7; ++i) L[i * (i - 1) / 2 + j] = a[i * (i + 1) / 2 + j] * Dinv[j];
#pragma unroll
        for (int i = j + 1; i < 7; ++i) {
            const double lij = L[i * (i - 1) / 2 + j];
#pragma unroll
            for (int k = j + 1; k <= i; ++k)
                a[i * (i + 1) / 2 + k] = fma(-lij, a[k * (k + 1) / 2 + j], a[i * (i + 1) / 2 + k]);
            y[i] = fma(-lij, y[j], y[i]);
        }
    }
    // L^T d = D^-1 y
#pragma unroll
    for (int i = 0; i < 7; ++i) y[i] *= Dinv[i];
#pragma unroll
    for (int i = 6; i >= 0; --i) {
        d[i] = y[i];
#pragma unroll
        for (int m = 0; m < i; ++m) y[m] = fma(-L[i * (i - 1) / 2 + m], d[i], y[m]);
    }
    if (!ok) {
#pragma unroll
        for (int i = 0; i < 7; ++i) d[i] = 0.0;
    }
    return ok;
}

// ---------------------------------------------------------------------------
// per-pair residual and Jacobian (float32)

struct PairTerm {
    float r0, r1, w, rho;
    float e;             // |r| (0 when not valid)
    float J[2][7];
    bool valid;
};

// INV: (A, tS) is the float32 form of S^-1 and the pair is a point of the
// current side observed on the loop side, p = S^-1 X; its Jacobian is still
// taken with respect to the left perturbation of S, under which
// S^-1 <- S^-1 exp(-xi):  J = dpi/dq R_k (-A) [ -[X]x | I | X ].
template <bool INV = false>
__device__ __forceinline__ void pair_term(const float* A, const float* tS, const float* T, float fx, float fy,
                                          float cx, float cy, float x, float y, float z, float uo, float vo,
                                          float delta, bool need_J, PairTerm& o) {
    const float p0 = A[0] * x + A[1] * y + A[2] * z + tS[0];
    const float p1 = A[3] * x + A[4] * y + A[5] * z + tS[1];
    const float p2 = A[6] * x + A[7] * y + A[8] * z + tS[2];
    float q0 = p0, q1 = p1, q2 = p2;
    if (T) {
        q0 = T[0] * p0 + T[1] * p1 + T[2] * p2 + T[9];
        q1 = T[3] * p0 + T[4] * p1 + T[5] * p2 + T[10];
        q2 = T[6] * p0 + T[7] * p1 + T[8] * p2 + T[11];
    }
    o.valid = q2 > 0.0f;
    if (!o.valid) {
        o.r0 = o.r1 = o.w = o.rho = o.e = 0.0f;
        return;
    }
    const float iz = __builtin_amdgcn_rcpf(q2);   // within 1 ulp
    o.r0 = fx * q0 * iz + cx - uo;
    o.r1 = fy * q1 * iz + cy - vo;
    const float e = sqrtf(o.r0 * o.r0 + o.r1 * o.r1);
    o.e = e;
    if (e <= delta) {
        o.w = 1.0f;
        o.rho = 0.5f * e * e;
    } else {
        o.w = delta * __builtin_amdgcn_rcpf(e);
        o.rho = delta * e - 0.5f * delta * delta;
    }
    if (!need_J) return;
    // M = dpi/dq R_k (2 x 3)
    const float a0 = fx * iz, a2 = -fx * q0 * iz * iz;
    const float b1 = fy * iz, b2 = -fy * q1 * iz * iz;
    float M[2][3];
    if (T) {
        for (int c = 0; c < 3; ++c) {
            M[0][c] = a0 * T[c] + a2 * T[6 + c];
            M[1][c] = b1 * T[3 + c] + b2 * T[6 + c];
        }
    } else {
        M[0][0] = a0; M[0][1] = 0.0f; M[0][2] = a2;
        M[1][0] = 0.0f; M[1][1] = b1; M[1][2] = b2;
    }
    for (int r = 0; r < 2; ++r) {
        float m0 = M[r][0], m1 = M[r][1], m2 = M[r][2];
        float a0 = p0, a1 = p1, a2 = p2;   // the point the perturbation acts on
        if (INV) {
            // row of -M A, acting on X
            const float b0 = -(m0 * A[0] + m1 * A[3] + m2 * A[6]);
            const float b1 = -(m0 * A[1] + m1 * A[4] + m2 * A[7]);
            const float b2 = -(m0 * A[2] + m1 * A[5] + m2 * A[8]);
            m0 = b0;
            m1 = b1;
            m2 = b2;
            a0 = x;
            a1 = y;
            a2 = z;
        }
        o.J[r][0] = a1 * m2 - a2 * m1;   // a x m: derivative along omega
        o.J[r][1] = a2 * m0 - a0 * m2;
        o.J[r][2] = a0 * m1 - a1 * m0;
        o.J[r][3] = m0;                  // upsilon
        o.J[r][4] = m1;
        o.J[r][5] = m2;
        o.J[r][6] = m0 * a0 + m1 * a1 + m2 * a2;   // sigma
    }
}

// acc[0..6] += w J^T r, acc[7..34] += w J^T J (upper, row by row): each
// pair's terms in float32 (as its residual and Jacobian are), accumulated
// over pairs in float64.
__device__ __forceinline__ void accumulate(const PairTerm& t, double* acc) {
    const float w = t.w, r0 = t.r0, r1 = t.r1;
#pragma unroll
    for (int i = 0; i < 7; ++i) acc[i] += (double)(w * fmaf(t.J[0][i], r0, t.J[1][i] * r1));
    int k = 7;
#pragma unroll
    for (int i = 0; i < 7; ++i)
#pragma unroll
        for (int j = i; j < 7; ++j) acc[k++] += (double)(w * fmaf(t.J[0][i], t.J[0][j], t.J[1][i] * t.J[1][j]));
}

// A float64 value of lane l (l wave-uniform).
__device__ __forceinline__ double readlane_f64(double x, int l) {
    const long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)v, l);
    const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// The value of lane l ^ H (H: a power of two), by lane permutations inside a
// row of 16 (quad_perm, row_ror:8, and for 4 row_half_mirror after the
// quads' reversal) and through LDS across rows.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const long long v = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
template <int H>
__device__ __forceinline__ double lane_xor_f64(double x) {
    if constexpr (H == 1) return dpp_f64<0xB1>(x);                       // quad_perm [1, 0, 3, 2]
    else if constexpr (H == 2) return dpp_f64<0x4E>(x);                  // quad_perm [2, 3, 0, 1]
    else if constexpr (H == 4) return dpp_f64<0x141>(dpp_f64<0x1B>(x));  // quad_perm [3, 2, 1, 0], row_half_mirror
    else if constexpr (H == 8) return dpp_f64<0x128>(x);                 // row_ror:8
    else return __shfl_xor(x, H);
}

// lo + its value in lane l ^ H in lanes whose bit H is clear, hi + its value
// there in the others.  Across rows the swap instructions of gfx950 hand both
// sums' operands over without a select (three instructions); inside a row the
// operands are selected and one permuted.
template <int H>
__device__ __forceinline__ double scatter_add(double lo, double hi) {
    if constexpr (H == 16 || H == 32) {
        const long long a = __double_as_longlong(lo), b = __double_as_longlong(hi);
        const auto swap = [](uint32_t x, uint32_t y) {
            if constexpr (H == 16) return __builtin_amdgcn_permlane16_swap(x, y, false, false);
            else return __builtin_amdgcn_permlane32_swap(x, y, false, false);
        };
        const auto l = swap((uint32_t)a, (uint32_t)b), h = swap((uint32_t)(a >> 32), (uint32_t)(b >> 32));
        return __longlong_as_double(((long long)h[0] << 32) | (long long)l[0]) +
               __longlong_as_double(((long long)h[1] << 32) | (long long)l[1]);
    } else {
        const bool up = (wave_lane() & H) != 0;
        return (up ? hi : lo) + lane_xor_f64<H>(up ? lo : hi);
    }
}

// One step of a reduce-scatter: of N values, lanes whose bit H is set keep the
// last N / 2, the others the first (N + 1) / 2 (w padded with a zero).
template <int N, int H>
__device__ __forceinline__ void reduce_scatter_step(double* w) {
    constexpr int K = (N + 1) / 2;
#pragma unroll
    for (int i = 0; i < K; ++i) w[i] = scatter_add<H>(w[i], K + i < N ? w[K + i] : 0.0);
}

// Block reduction of NV <= 64 doubles per thread, fixed order.  Inside a
// wave a butterfly reduce-scatter halves the values a lane carries at every
// step (63 exchanges for any NV instead of 6 NV), none of them through LDS,
// the cheapest first; the block then adds the wave totals in wave order.
// Result in s_out[0..NV).
template <int NV>
__device__ __forceinline__ void block_reduce(const double* v, double* s_red, double* s_out) {
    static_assert(NV <= 64, "at most 64 values");
    const int lane = wave_lane();
    const int wid = threadIdx.x / kWave;
    const int nw = blockDim.x / kWave;
    double w[64];
#pragma unroll
    for (int i = 0; i < 64; ++i) w[i] = i < NV ? v[i] : 0.0;
    reduce_scatter_step<64, 16>(w);
    reduce_scatter_step<32, 32>(w);
    reduce_scatter_step<16, 1>(w);
    reduce_scatter_step<8, 2>(w);
    reduce_scatter_step<4, 8>(w);
    reduce_scatter_step<2, 4>(w);
    // this lane's value
    const int i = (lane >> 4 & 1) * 32 + (lane >> 5) * 16 + (lane & 1) * 8 + (lane >> 1 & 1) * 4 + (lane >> 3 & 1) * 2 +
                  (lane >> 2 & 1);
    if (i < NV) s_red[wid * NV + i] = w[0];
    __syncthreads();
    if ((int)threadIdx.x < NV) {
        double s = 0.0;
        for (int q = 0; q < nw; ++q) s += s_red[q * NV + threadIdx.x];
        s_out[threadIdx.x] = s;
    }
    __syncthreads();
}

// Fixed-order sums of a wave for the refinement.  The four lanes of each quad
// first add their NV values pairwise in float32 (DPP quad permutations: lanes
// 2i and 2i + 1 swap halves and add, then lanes 4i + {0, 1} and 4i + {2, 3}
// swap quarters and add), so each lane keeps NV / 4 of the quad's sums; those
// are widened, and a reduce-scatter over the 16 quads adds them in float64.
// On return value `idx` of the wave's NV sums is v in the lane that got it
// (idx < 0: none).
constexpr int kSeg = 8;

template <int CTRL>
__device__ __forceinline__ float quad_perm_f32(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false));
}

template <int NV>
__device__ __forceinline__ double wave_reduce_quad(const float* v, int& idx) {
    static_assert(NV == 36, "nine values a lane after the quads");
    constexpr int H = NV / 2, Q = NV / 4;
    const int l = wave_lane();
    const bool odd = l & 1, hi = l & 2;
    // both lanes' sums of both halves, then the one to keep (a permuted add
    // each; selecting first costs waits between a select and its permutation)
    float h[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
        const float a = v[j] + quad_perm_f32<0xB1>(v[j]);   // quad_perm [1, 0, 3, 2]
        const float b = v[j + H] + quad_perm_f32<0xB1>(v[j + H]);
        h[j] = odd ? b : a;
    }
    double w[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const float a = h[j] + quad_perm_f32<0x4E>(h[j]);   // quad_perm [2, 3, 0, 1]
        const float b = h[j + Q] + quad_perm_f32<0x4E>(h[j + Q]);
        w[j] = (double)(hi ? b : a);
    }
    reduce_scatter_step<9, 16>(w);   // 5 left (4 in the upper lanes)
    reduce_scatter_step<5, 32>(w);   // 3 (2)
    reduce_scatter_step<3, 8>(w);    // 2 (1)
    reduce_scatter_step<2, 4>(w);    // 1
    const int n1 = l & 16 ? 4 : 5;                    // this lane's values after each step
    const int n2 = l & 32 ? n1 - 3 : 3;
    const int n3 = l & 8 ? n2 - 2 : min(n2, 2);
    const int at = (l & 16 ? 5 : 0) + (l & 32 ? 3 : 0) + (l & 8 ? 2 : 0) + (l & 4 ? 1 : 0);
    idx = (l & 4 ? 1 : 0) < n3 ? (odd ? H : 0) + (hi ? Q : 0) + at : -1;
    return w[0];
}

// The kSeg segments (or wave totals) of value c, NV values each, added
// pairwise.
static_assert(kSeg == 8, "a pairwise tree of 8");
template <int NV>
__device__ __forceinline__ double add_segments(const double* s_q, int c) {
    const double a = (s_q[c] + s_q[NV + c]) + (s_q[2 * NV + c] + s_q[3 * NV + c]);
    return a + ((s_q[4 * NV + c] + s_q[5 * NV + c]) + (s_q[6 * NV + c] + s_q[7 * NV + c]));
}

// Fixed-order float64 sum over the block: a wave butterfly (every lane ends
// with the same value: each stage adds the same two numbers in both lanes),
// then the wave totals in wave order.  s_w holds one double per wave.
__device__ __forceinline__ double block_sum_f64(double v, double* s_w) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (wave_lane() == 0) s_w[threadIdx.x / kWave] = v;
    __syncthreads();
    double sum = 0.0;
    for (int w = 0; w < (int)(blockDim.x / kWave); ++w) sum += s_w[w];
    return sum;
}

struct ResArgs {
    int32_t n;
    int32_t n_kf;
    const float* xyz;
    const float* uv;
    const int32_t* kf_idx;
    const float* kf_T;
    const fl_sim3* S;
    const double* xi;     // forward: S = exp(xi) S0 (S is then an output); backward: gradient with respect to xi
    const double* S0;
    fl_sim3* S_out;
    const double* scale;  // backward with xi: device factor of the gradient, may be null
    double* gxi;          // backward with xi: [7]
    float fx, fy, cx, cy;
    float delta;
    double grad_scale;
    float* r;
    float* w;
    double* loss;
    double* g;
    double* H;
    double* partial;      // [gridDim.x][kNAcc]
    uint32_t* done;       // one counter, zero on entry and on exit
};

__device__ __forceinline__ bool load_pair(const ResArgs& a, int i, float& x, float& y, float& z, float& uo,
                                          float& vo, const float*& T) {
    x = a.xyz[3 * (int64_t)i];
    y = a.xyz[3 * (int64_t)i + 1];
    z = a.xyz[3 * (int64_t)i + 2];
    uo = a.uv[2 * (int64_t)i];
    vo = a.uv[2 * (int64_t)i + 1];
    T = nullptr;
    if (a.kf_idx) {
        const int k = a.kf_idx[i];
        if (k < 0 || k >= a.n_kf) return false;
        if (a.kf_T) T = a.kf_T + 12 * (int64_t)k;
    } else if (a.kf_T) {
        T = a.kf_T;
    }
    return true;
}

// The block's NV sums (s_out) join the launch's: they go to the block's row
// of partials, and in the block that finishes last (true is returned there,
// in every thread) the rows are added into s_out, thread (c, seg) taking rows
// seg, seg + SEG, ... of value c and the segments in order.  The partials are
// stored and loaded at device scope and each block counts itself once its
// stores are complete, so no cache is written back or invalidated: a release
// fence per block wrote back the L2's dirty lines, the pairs' outputs among
// them.  s_seg holds kResBlock doubles.
template <int NV>
__device__ __forceinline__ bool finish_sums(const ResArgs& a, double* s_out, double* s_seg) {
    __shared__ int s_last;
    const int tid = threadIdx.x, nb = gridDim.x;
    if (nb > 1) {
        if (tid < NV)
            __hip_atomic_store(&a.partial[(int64_t)blockIdx.x * kNAcc + tid], s_out[tid], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's partials have arrived
        __syncthreads();
        if (tid == 0)
            s_last = __hip_atomic_fetch_add(a.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)nb - 1;
        __syncthreads();
        if (!s_last) return false;
        constexpr int SEG = kResBlock / NV;
        const int c = tid % NV, seg = tid / NV;
        if (seg < SEG) {
            double v = 0.0;
            const double* p = a.partial + c;
            int r = seg;
            for (; r + 7 * SEG < nb; r += 8 * SEG) {
                double x[8];
#pragma unroll
                for (int q = 0; q < 8; ++q)
                    x[q] = __hip_atomic_load(p + (int64_t)(r + q * SEG) * kNAcc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int q = 0; q < 8; ++q) v += x[q];
            }
            double x[7];
#pragma unroll
            for (int q = 0; q < 7; ++q)
                x[q] = r + q * SEG < nb ? __hip_atomic_load(p + (int64_t)(r + q * SEG) * kNAcc, __ATOMIC_RELAXED,
                                                            __HIP_MEMORY_SCOPE_AGENT) : 0.0;
#pragma unroll
            for (int q = 0; q < 7; ++q) v += x[q];
            s_seg[seg * NV + c] = v;
        }
        __syncthreads();
        if constexpr (NV == 1) {
            if (tid < kWave) {   // 256 segments
                double v = (s_seg[tid] + s_seg[tid + 64]) + (s_seg[tid + 128] + s_seg[tid + 192]);
#pragma unroll
                for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
                if (tid == 0) s_out[0] = v;
            }
        } else if (tid < NV) {
            double v = 0.0;
#pragma unroll
            for (int q = 0; q < SEG; ++q) v += s_seg[q * NV + tid];
            s_out[tid] = v;
        }
        if (tid == 0) *a.done = 0;
        __syncthreads();
    }
    return true;
}

__global__ __launch_bounds__(kResBlock) void residual_fwd_kernel(ResArgs a) {
    __shared__ double s_wave[kResBlock / kWave];
    __shared__ double s_out[1];
    __shared__ double s_seg[kResBlock];
    __shared__ fl_sim3 s_S;
    if (a.xi) {   // every block composes S for itself; block 0 hands it out
        if (threadIdx.x == 0) {
            sim3_to_f32(sim3_mul(sim3_exp(a.xi), sim3_load(a.S0)), &s_S);
            if (blockIdx.x == 0) *a.S_out = s_S;
        }
    } else if (threadIdx.x == 0) {
        s_S = *a.S;
    }
    __syncthreads();
    const fl_sim3 S = s_S;
    double loss = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += gridDim.x * blockDim.x) {
        float x, y, z, uo, vo;
        const float* T;
        PairTerm t;
        if (load_pair(a, i, x, y, z, uo, vo, T)) {
            pair_term(S.sR, S.t, T, a.fx, a.fy, a.cx, a.cy, x, y, z, uo, vo, a.delta, false, t);
        } else {
            t.valid = false;
            t.r0 = t.r1 = t.w = t.rho = 0.0f;
        }
        if (a.r) {
            a.r[2 * (int64_t)i] = t.r0;
            a.r[2 * (int64_t)i + 1] = t.r1;
        }
        if (a.w) a.w[i] = t.w;
        loss += (double)t.rho;
    }
    const double sum = block_sum_f64(loss, s_wave);
    if (threadIdx.x == 0) s_out[0] = sum;
    __syncthreads();
    if (finish_sums<1>(a, s_out, s_seg) && threadIdx.x == 0) *a.loss = s_out[0];
}

// scale J_l(xi)^T g by one wave (the definition at sim3_grad_xi_kernel below).
__device__ __forceinline__ void sim3_grad_xi_wave(const double* xi, const double* g, const double* scale, double* out);

template <bool INV>
__global__ __launch_bounds__(kResBlock) void residual_bwd_kernel(ResArgs a) {
    __shared__ double s_red[(kResBlock / kWave) * 35];
    __shared__ double s_out[35];
    __shared__ double s_seg[kResBlock];
    const fl_sim3 S = *a.S;
    double acc[35];
#pragma unroll
    for (int i = 0; i < 35; ++i) acc[i] = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += gridDim.x * blockDim.x) {
        float x, y, z, uo, vo;
        const float* T;
        if (!load_pair(a, i, x, y, z, uo, vo, T)) continue;
        PairTerm t;
        pair_term<INV>(S.sR, S.t, T, a.fx, a.fy, a.cx, a.cy, x, y, z, uo, vo, a.delta, true, t);
        if (t.valid) accumulate(t, acc);
    }
    block_reduce<35>(acc, s_red, s_out);
    if (!finish_sums<35>(a, s_out, s_seg)) return;
    if (a.gxi) {
        if (threadIdx.x < kWave) sim3_grad_xi_wave(a.xi, s_out, a.scale, a.gxi);
        return;
    }
    if (threadIdx.x < 7) a.g[threadIdx.x] = a.grad_scale * s_out[threadIdx.x];
    else if ((int)threadIdx.x < 35 && a.H) a.H[threadIdx.x - 7] = s_out[threadIdx.x];
}

__global__ void sim3_exp_mul_kernel(const double* __restrict__ xi, const double* __restrict__ S_in,
                                    double* __restrict__ S_out, fl_sim3* __restrict__ S32) {
    if (threadIdx.x != 0) return;
    const Sim3d E = sim3_exp(xi);
    const Sim3d S = sim3_mul(E, sim3_load(S_in));
    sim3_store(S, S_out);
    if (S32) sim3_to_f32(S, S32);
}

// Gradient with respect to the coordinates xi of S = exp(xi) S0, from the
// gradient g with respect to a left perturbation of S: exp(xi + d) equals
// exp(J_l(xi) d) exp(xi) to first order, so dL/dxi = J_l(xi)^T g, with the
// left Jacobian J_l(xi) = sum_k ad(xi)^k / (k + 1)!.  For xi = (w, u, sig)
// (omega, upsilon, sigma) the commutator of the 4x4 generators gives, in
// the rows and columns (omega, upsilon, sigma),
//   ad(xi) = [ [w]x        0          0 ]
//            [ [u]x   [w]x + sig I   -u ]
//            [ 0           0          0 ].
// Only J_l^T g is wanted, so the series runs on the vector: v_0 = g, v_k =
// ad(xi)^T v_{k-1} / (k + 1), 49 products a term where the matrix took 343.
// It is summed in float64 until a term's largest entry falls below 1e-18 of
// the sum's and the terms can only shrink from there (at most 64 terms; |w|
// <= pi and |sig| of order one converge in about 25).  out = scale * J_l^T g
// (scale: device, may be null).  One wave: lane c < 7 holds column c of
// ad(xi) and entry c of v (one lane with the matrices in scratch memory took
// 60 us; this takes 2).
__device__ __forceinline__ void sim3_grad_xi_wave(const double* xi, const double* g, const double* scale, double* out) {
    const int c = min(wave_lane(), 7);   // lanes past 6 carry zeros
    double x[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) x[i] = xi[i];
    // column c of ad(xi), by its row blocks: [w]x column, then [u]x column
    // (c < 3) or [w]x column + sig I (c < 6) or -u (c = 6), then 0
    auto hat_col = [](double a0, double a1, double a2, int j, double* h) {
        h[0] = j == 1 ? -a2 : j == 2 ? a1 : 0.0;
        h[1] = j == 0 ? a2 : j == 2 ? -a0 : 0.0;
        h[2] = j == 0 ? -a1 : j == 1 ? a0 : 0.0;
    };
    double W[3], U[3], A[6];
    hat_col(x[0], x[1], x[2], c < 3 ? c : c - 3, W);
    hat_col(x[3], x[4], x[5], c, U);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        A[i] = c < 3 ? W[i] : 0.0;
        A[3 + i] = c < 3 ? U[i] : c < 6 ? W[i] + (c - 3 == i ? x[6] : 0.0) : c == 6 ? -x[3 + i] : 0.0;
    }
    double v = c < 7 ? g[c] : 0.0, sum = v;
    // a bound of every |ad(xi)^T v| / |v|, largest entries: its largest column sum
    double norm = 0.0;
#pragma unroll
    for (int i = 0; i < 6; ++i) norm += fabs(A[i]);
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) norm = fmax(norm, __shfl_xor(norm, off));
    for (int k = 1; k < 64; ++k) {
        double n = 0.0;
#pragma unroll
        for (int r = 0; r < 6; ++r) n = fma(A[r], readlane_f64(v, r), n);   // row 6 of ad(xi) is 0
        v = n * (1.0 / (double)(k + 1));
        sum += v;
        double tmax = fabs(v), smax = fabs(sum);
#pragma unroll
        for (int off = 4; off > 0; off >>= 1) {
            tmax = fmax(tmax, __shfl_xor(tmax, off));
            smax = fmax(smax, __shfl_xor(smax, off));
        }
        if (readlane_f64(tmax, 0) <= 1e-18 * readlane_f64(smax, 0) && readlane_f64(norm, 0) < (double)(k + 2)) break;
    }
    if (wave_lane() < 7) out[wave_lane()] = (scale ? *scale : 1.0) * sum;
}

__global__ __launch_bounds__(64) void sim3_grad_xi_kernel(const double* __restrict__ xi, const double* g,
                                                          const double* __restrict__ scale, double* out) {
    sim3_grad_xi_wave(xi, g, scale, out);   // out may be g
}

// S_inv = S^-1 = (R^T, -R^T t / s, 1 / s) in float64, and its float32 form.
__global__ void sim3_inverse_kernel(const double* __restrict__ S_in, double* __restrict__ S_out,
                                    fl_sim3* __restrict__ S32) {
    if (threadIdx.x != 0) return;
    const Sim3d V = sim3_inv(sim3_load(S_in));
    if (S_out) sim3_store(V, S_out);
    if (S32) sim3_to_f32(V, S32);
}

__global__ void gn_step_kernel(const double* __restrict__ g, const double* __restrict__ H, double lambda,
                               double* __restrict__ S_io, fl_sim3* __restrict__ S32) {
    if (threadIdx.x != 0) return;
    double d[7];
    Sim3d S = sim3_load(S_io);
    if (solve7(g, H, lambda, d)) {
        S = sim3_mul(sim3_exp(d), S);
        sim3_store(S, S_io);
    }
    if (S32) sim3_to_f32(S, S32);
}

// ---------------------------------------------------------------------------
// Per-event refinement inside a batch, all Gauss-Newton steps in one launch.
// refine_blocks workgroups per event accumulate g and H over the event's
// accepted pairs (recorded by the search as point + observation + keyframe,
// held in registers across the steps), publish their partial sums as tagged
// rows and wait until every row of the step is tagged; every workgroup then
// sums the rows in the same order and solves the same 7x7 system, so all of
// them hold the bitwise-identical next Sim3 without a second exchange.  The
// wait only involves workgroups of the same event, which are co-resident (the
// whole grid is one workgroup per CU); its spin is bounded and a timeout is
// reported as n_matched = -1.

constexpr unsigned kSpinLimit = 1u << 22;

// One pair's terms of the refinement at S (its float32 form A, t), added to
// acc when the pair is in front of its keyframe: acc[0..6] w J^T r, acc[7..34]
// w J^T J (upper, row by row), acc[35] the pairs added.  The arithmetic of
// pair_term with fused multiply-adds throughout, the weight from the squared
// error and w J formed once (some 150 instructions a pair where separate
// products and sums took 250: two waves a SIMD issue them for 0.9 us a step
// instead of 1.3).  Both round at the size of the observation, which bounds the
// result: against float64 refinements of the same pairs the pose is off by 1.8
// to 3.0e-8 (relative, geometric means of 15 to 60 inputs of six kinds of
// event), with separate products it was by 1.9 to 3.3e-8.  INV as in
// pair_term: A, t are S^-1's, the pair is a point of the current side.
// No branch: a pair that is not there (has false) or whose depth is not positive
// adds zeros, whatever it holds: its residual, point and rows of the Jacobian
// are selected to zero, since an observation, a pose or an intrinsic that is
// not finite times a zero weight is not zero.  FIRST: acc is written, not
// added to.
template <bool INV, bool FIRST = false>
__device__ __forceinline__ void refine_pair_f32(const float* A, const float* t, const float* T, float fx, float fy,
                                                float cx, float cy, float x, float y, float z, float uo, float vo,
                                                float delta, float* acc, bool has = true) {
    const float p0 = fmaf(A[0], x, fmaf(A[1], y, fmaf(A[2], z, t[0])));
    const float p1 = fmaf(A[3], x, fmaf(A[4], y, fmaf(A[5], z, t[1])));
    const float p2 = fmaf(A[6], x, fmaf(A[7], y, fmaf(A[8], z, t[2])));
    const float q0 = fmaf(T[0], p0, fmaf(T[1], p1, fmaf(T[2], p2, T[9])));
    const float q1 = fmaf(T[3], p0, fmaf(T[4], p1, fmaf(T[5], p2, T[10])));
    const float q2 = fmaf(T[6], p0, fmaf(T[7], p1, fmaf(T[8], p2, T[11])));
    const bool in = has && q2 > 0.0f;
    const auto keep = [in](float v) { return in ? v : 0.0f; };
    const float iz = __builtin_amdgcn_rcpf(q2);   // within 1 ulp
    const float a0 = fx * iz, b1 = fy * iz;
    const float r0 = keep(fmaf(a0, q0, cx) - uo);
    const float r1 = keep(fmaf(b1, q1, cy) - vo);
    const float e2 = fmaf(r0, r0, r1 * r1);
    const float w = keep(e2 <= delta * delta ? 1.0f : delta * __builtin_amdgcn_rsqf(e2));   // within 1 ulp
    const float a2 = -a0 * (q0 * iz), b2 = -b1 * (q1 * iz);
    // the point the perturbation acts on
    const float x0 = keep(INV ? x : p0), x1 = keep(INV ? y : p1), x2 = keep(INV ? z : p2);
    float J[2][7], W[2][7];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const float d0 = r ? b1 : a0, d2 = r ? b2 : a2;
        float m0 = fmaf(d2, T[6], d0 * T[3 * r]);
        float m1 = fmaf(d2, T[7], d0 * T[3 * r + 1]);
        float m2 = fmaf(d2, T[8], d0 * T[3 * r + 2]);
        if (INV) {
            const float i0 = -fmaf(m0, A[0], fmaf(m1, A[3], m2 * A[6]));
            const float i1 = -fmaf(m0, A[1], fmaf(m1, A[4], m2 * A[7]));
            const float i2 = -fmaf(m0, A[2], fmaf(m1, A[5], m2 * A[8]));
            m0 = i0;
            m1 = i1;
            m2 = i2;
        }
        m0 = keep(m0);
        m1 = keep(m1);
        m2 = keep(m2);
        J[r][0] = fmaf(x1, m2, -(x2 * m1));
        J[r][1] = fmaf(x2, m0, -(x0 * m2));
        J[r][2] = fmaf(x0, m1, -(x1 * m0));
        J[r][3] = m0;
        J[r][4] = m1;
        J[r][5] = m2;
        J[r][6] = fmaf(m0, x0, fmaf(m1, x1, m2 * x2));
#pragma unroll
        for (int i = 0; i < 7; ++i) W[r][i] = w * J[r][i];
    }
    int k = 7;
#pragma unroll
    for (int i = 0; i < 7; ++i) {
        acc[i] = fmaf(W[0][i], r0, FIRST ? W[1][i] * r1 : fmaf(W[1][i], r1, acc[i]));
#pragma unroll
        for (int j = i; j < 7; ++j, ++k)
            acc[k] = fmaf(W[0][i], J[0][j], FIRST ? W[1][i] * J[1][j] : fmaf(W[1][i], J[1][j], acc[k]));
    }
    const float one = keep(1.0f);
    acc[35] = FIRST ? one : acc[35] + one;
}

// A pair's reprojection error at a float64 Sim3 (13 doubles: R, t, s), in
// float64 throughout; false when the pair is behind its keyframe.  The
// quantities that decide something (a Levenberg-Marquardt step's Huber loss,
// whether a pair is an inlier of a round) are evaluated this way: their
// float32 form carries ~1e-5 px of rounding per pair, enough to turn a
// near-tie either way.
__device__ __forceinline__ bool pair_error64(const double* S, const float* T, float fx, float fy, float cx, float cy,
                                             float x, float y, float z, float uo, float vo, double& e) {
    const double X = x, Y = y, Z = z, sc = S[12];
    double p[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i] = sc * (S[3 * i] * X + S[3 * i + 1] * Y + S[3 * i + 2] * Z) + S[9 + i];
    double q[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
        q[i] = (double)T[3 * i] * p[0] + (double)T[3 * i + 1] * p[1] + (double)T[3 * i + 2] * p[2] + (double)T[9 + i];
    if (!(q[2] > 0.0)) {
        e = 0.0;
        return false;
    }
    const double r0 = (double)fx * q[0] / q[2] + (double)cx - (double)uo;
    const double r1 = (double)fy * q[1] / q[2] + (double)cy - (double)vo;
    e = sqrt(r0 * r0 + r1 * r1);
    return true;
}

__device__ __forceinline__ double huber64(double e, double delta) {
    return e <= delta ? 0.5 * e * e : delta * e - 0.5 * delta * delta;
}

// Coefficient tables of the exponential's series, entry k of lane l's
// polynomial at [16 k + l]: lanes 0..6 I_l(sigma) = sum_k sigma^k / (k! (l + k
// + 1)), lane 7 e^sigma = sum_k sigma^k / k!, lanes 8 and 9 sin(th) / th and
// (1 - cos(th)) / th^2 in th^2, other lanes 0.  With |sigma| below 1e-2 and
// th^2 below 1e-4 nine (four) terms leave less than 0.01^9 / 9! < 3e-24.
constexpr int kExpTerms = 9;
struct ExpTable {
    double v[16 * kExpTerms];
    constexpr ExpTable() : v() {
        double f = 1.0;   // 1 / k!
        for (int k = 0; k < kExpTerms; ++k) {
            if (k > 0) f = f / (double)k;
            for (int l = 0; l < 7; ++l) v[16 * k + l] = f / (double)(l + k + 1);
            v[16 * k + 7] = f;
        }
        const double a[4] = {1.0, -1.0 / 6.0, 1.0 / 120.0, -1.0 / 5040.0};
        const double b[4] = {0.5, -1.0 / 24.0, 1.0 / 720.0, -1.0 / 40320.0};
        for (int k = 0; k < 4; ++k) {
            v[16 * k + 8] = a[k];
            v[16 * k + 9] = b[k];
        }
    }
};
__device__ constexpr ExpTable kExpTable{};

// S <- exp(d) S by the lanes of one wave, every lane holding the same step d:
// for the usual Gauss-Newton step (rotation angle and |sigma| below 1e-2) the
// lanes evaluate one series each (kExpTable, in LDS) and hand the ten values
// round, for any other step every lane evaluates the full coefficients; lane l < 13 then computes entry l of the
// product (R row-major, t, s) from the rows of exp(d) (R_d = I + a W + b W^2
// and V = c0 I + c1 W + c2 W^2 with W = [omega]x and W^2 = omega omega^T -
// |omega|^2 I) and from B, writes it to S64 (B may be S64) and its
// float32 pose to o32; with inv32 the lanes then write the float32 pose of the
// product's inverse (R^T / s, -R^T t / s).  What does not depend on the step
// is loaded beforehand (compose_inputs), beside the solve for it.
struct ComposeIn {
    double cf[kExpTerms], b[3], s;   // this lane's series, its column of B, the scale of B
};
__device__ __forceinline__ ComposeIn compose_inputs(const double* cf, const double* B) {
    const int l = wave_lane();
    ComposeIn in;
#pragma unroll
    for (int q = 0; q < kExpTerms; ++q) in.cf[q] = cf[16 * q + (l & 15)];
    const int o = l < 9 ? l % 3 : 9, st = l < 9 ? 3 : 1;   // a column of the rotation, or the translation
#pragma unroll
    for (int q = 0; q < 3; ++q) in.b[q] = B[o + st * q];
    in.s = B[12];
    return in;
}
__device__ __forceinline__ void compose_exp_lanes(const double* d, const ComposeIn& in, double* S64, fl_sim3* o32,
                                                  fl_sim3* inv32) {
    const int l = wave_lane();
    const double w0 = d[0], w1 = d[1], w2 = d[2], sig = d[6];
    const double th2 = w0 * w0 + w1 * w1 + w2 * w2;
    ExpCoef k;
    if (th2 < 1e-4 && fabs(sig) < 0.01) {
        const double x = l < 8 ? sig : th2;
        double v = in.cf[kExpTerms - 1];
#pragma unroll
        for (int q = kExpTerms - 2; q >= 0; --q) v = fma(v, x, in.cf[q]);
        const double I1 = readlane_f64(v, 1), I2 = readlane_f64(v, 2);
        k.c0 = readlane_f64(v, 0);
        k.c1 = fma(th2, fma(th2 * (1.0 / 120.0), readlane_f64(v, 5), (-1.0 / 6.0) * readlane_f64(v, 3)), I1);
        k.c2 = fma(th2, fma(th2 * (1.0 / 720.0), readlane_f64(v, 6), (-1.0 / 24.0) * readlane_f64(v, 4)), 0.5 * I2);
        k.es = readlane_f64(v, 7);
        k.a = readlane_f64(v, 8);
        k.b = readlane_f64(v, 9);
    } else {
        k = sim3_exp_coef_full(w0, w1, w2, sig);
    }
    // this lane's row i of R_d and V: lanes 0-8 entry (i, j) = (l / 3, l % 3)
    // of the rotation, lanes 9-11 row l - 9 of the translation
    const int i = l < 9 ? l / 3 : (l < 12 ? l - 9 : 0);
    const int j = l < 9 ? l % 3 : 0;
    const double wi = i == 0 ? w0 : (i == 1 ? w1 : w2);
    // row i of W: (0, -w2, w1), (w2, 0, -w0), (-w1, w0, 0)
    const double W0 = i == 0 ? 0.0 : (i == 1 ? w2 : -w1);
    const double W1 = i == 0 ? -w2 : (i == 1 ? 0.0 : w0);
    const double W2 = i == 0 ? w1 : (i == 1 ? -w0 : 0.0);
    const double Q0 = fma(wi, w0, i == 0 ? -th2 : 0.0);   // row i of W^2
    const double Q1 = fma(wi, w1, i == 1 ? -th2 : 0.0);
    const double Q2 = fma(wi, w2, i == 2 ? -th2 : 0.0);
    const double R0 = (i == 0 ? 1.0 : 0.0) + fma(k.b, Q0, k.a * W0);
    const double R1 = (i == 1 ? 1.0 : 0.0) + fma(k.b, Q1, k.a * W1);
    const double R2 = (i == 2 ? 1.0 : 0.0) + fma(k.b, Q2, k.a * W2);
    const double V0 = fma(k.c2, Q0, fma(k.c1, W0, i == 0 ? k.c0 : 0.0));
    const double V1 = fma(k.c2, Q1, fma(k.c1, W1, i == 1 ? k.c0 : 0.0));
    const double V2 = fma(k.c2, Q2, fma(k.c1, W2, i == 2 ? k.c0 : 0.0));
    const double s_new = k.es * in.s;
    const double rb = fma(R0, in.b[0], fma(R1, in.b[1], R2 * in.b[2]));
    const double vu = fma(V0, d[3], fma(V1, d[4], V2 * d[5]));
    const double v = l < 9 ? rb : l < 12 ? fma(k.es, rb, vu) : s_new;
    if (l < 13) S64[l] = v;
    if (l < 9) o32->sR[l] = (float)(s_new * v);
    else if (l < 12) o32->t[l - 9] = (float)v;
    if (inv32) {
        // the new entries are written before any lane reads them
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const double inv_s = 1.0 / s_new;
        if (l < 9) {
            inv32->sR[l] = (float)(inv_s * S64[3 * j + i]);
        } else if (l < 12) {
            inv32->t[i] = (float)(-(S64[i] * S64[9] + S64[3 + i] * S64[10] + S64[6 + i] * S64[11]) * inv_s);
        }
    }
}

constexpr int kRefKfLds = 128;   // keyframes of one event whose pose and intrinsics sit in LDS
constexpr int kRefMaxB = 64;     // workgroups per event
constexpr int kRefBlock = 512;   // threads of a refinement workgroup: 64 x 512 pairs at one per thread
// Accepted pairs of a thread in LDS, after the two or three in registers: ten
// events of 51,000 to 62,000 pairs each have 25 workgroups apiece, four to five
// pairs a thread.  Looked up in the search's lists again at every
// step, a step took 17,900 cycles, with them here 15,900.
constexpr int kRefLds = 2;
constexpr int kNAccLM = 37;      // the sums plus the Huber loss (slot 36)
// Each float64 partial travels as two 64-bit words, (high half << 32 | tag)
// and (low half << 32 | tag): a word is written and read in one piece, so a
// reader that sees the tag of the current launch and step in both words has
// the value, without a separate flag or any cache maintenance.  Rows are
// laid out for the larger (Levenberg-Marquardt) sum set.
constexpr int kRefWords = 80;    // 2 kNAccLM, padded
constexpr int kDeviceScope = 16;   // sc1 of the buffer loads and stores of the exchange
static_assert(kRefBlock / kWave == kSeg && kRefWords >= 2 * kNAccLM, "wave totals and segments alike, one a wave");
constexpr double kLmConverged = 1e-6;   // relative loss change that ends a round

// The refinement of each event in rounds.  Round 0 uses every accepted
// pair; a later round uses the pairs in front of their keyframe whose error
// at the round's starting Sim3 is within outlier_px.  A round is
// refine_iters evaluations of the sums.  Gauss-Newton (LM false) steps to
// S <- exp(d) S after every evaluation, d solving H d = -g.  Levenberg-
// Marquardt (LM true) evaluates the round's starting Sim3, then candidates
// exp(d) S_acc with (H + lambda diag H) d = -g at the accepted S_acc.  With
// rho the candidate's relative drop of the Huber loss below S_acc's: rho >
// 1e-6 takes it (lambda / 10, at least 1e-12), |rho| <= 1e-6 ends the round
// (converged; every workgroup holds the same sums, so all of them leave the
// round together), rho < -1e-6 drops it (lambda x 10, at most 1e16).
// lambda restarts at lm_lambda each round and the round ends at S_acc.
// ROUNDS false compiles the single-round kernel (no inlier tests).
template <bool LM, bool ROUNDS>
__global__ __launch_bounds__(kRefBlock) void refine_kernel(const BatchHdr* __restrict__ hp) {
    constexpr int NV = LM ? kNAccLM : kNAcc;
    constexpr int kRefCache = LM || ROUNDS ? 2 : 3;   // accepted pairs a thread keeps in registers across the steps
    static_assert(kRefCache == 2 || kRefCache == 3, "the calls below");
    __shared__ double s_w[kSeg * NV];        // the waves' sums
    __shared__ double s_q[kSeg * NV];        // segments of the event's rows
    __shared__ double s_out[NV];
    __shared__ double s_cf[16 * kExpTerms];
    __shared__ float s_kf[kRefKfLds * 16];   // per keyframe: T (12), fx, fy, cx, cy
    __shared__ float s_ikf[(LM || ROUNDS) ? 16 : kRefKfLds * 16];   // the same for the other direction's keyframes
    __shared__ double s_S64[13];
    __shared__ fl_sim3 s_S;
    __shared__ fl_sim3 s_Sinv;               // float32 form of S^-1 (two-sided refinement)
    __shared__ double s_Srs64[13];           // the round's starting Sim3 (inlier tests)
    __shared__ double s_acc[kNAcc];          // LM: g, H and count at S_acc
    __shared__ double s_Sacc[13];            // LM: S_acc
    __shared__ double s_lm[2];               // LM: loss at S_acc, lambda
    __shared__ float s_more[kRefLds][6][kRefBlock];   // each thread's pairs after those in registers
    __shared__ int s_segx[kRefBlock];        // the event's segments of accepted pairs: the pairs before each,
    __shared__ int s_segp[kRefBlock];        // and its place in the staging list less those
    __shared__ int s_segw[kRefBlock / kWave];
    __shared__ int s_fail;
    __shared__ int s_round_end;              // LM: the round converged at this step
    const BatchHdr& h = *hp;
    const int B = h.refine_blocks;
    const int n_units = h.n_events * B;
    const int iters = h.refine_iters;
    const int total = iters * (ROUNDS ? h.refine_rounds : 1);
    const float delta = h.huber_delta;
    const float tau = h.outlier_px;
    const int tid = threadIdx.x;
    const uint32_t epoch = *h.epoch;
    for (int i = tid; i < 16 * kExpTerms; i += blockDim.x) s_cf[i] = kExpTable.v[i];
    // An event's workgroups wait for each other, so they are spread evenly over
    // the XCDs (workgroup i is dispatched to XCD i mod 8): refinements in flight
    // together then fit whenever their workgroups do.  With one event's all on
    // one XCD, whose exchange is shorter (20 keyframes 72.1 -> 69.0 us), two such
    // launches would each hold CUs the other waits for.
    for (int unit = blockIdx.x; unit < n_units; unit += gridDim.x) {
        const int ev = unit / B, b = unit % B;
        const EventDesc ed = h.ev[ev];
        const int seg_n = h.refine_scan ? 0 : ed.seg_n;
        const MatchSeg sg = tid < seg_n ? h.match_seg[ed.seg_off + tid] : MatchSeg{0, 0};
        const int n_kf_ev = ed.kf_end - ed.kf_begin;
        const bool kf_lds = n_kf_ev <= kRefKfLds;
        if (tid < 13) s_S64[tid] = h.event_S[13 * (int64_t)ev + tid];
        if (tid == 0) s_fail = 0;
        if (kf_lds) {
            for (int i = tid; i < n_kf_ev * 16; i += blockDim.x) {
                const KfDesc& kd = h.kf[ed.kf_begin + (i >> 4)];
                const int f = i & 15;
                s_kf[i] = f < 12 ? kd.T[f] : f == 12 ? kd.fx : f == 13 ? kd.fy : f == 14 ? kd.cx : kd.cy;
            }
            // (threads without a pair read the first entry, which an event
            // without keyframes does not have)
            if (n_kf_ev == 0 && tid < 16) s_kf[tid] = 0.0f;
        }
        // two-sided refinement (Gauss-Newton only): the event's pairs of the
        // other direction and their keyframes
        const int n_inv = (LM || ROUNDS) ? 0 : ed.inv_n;
        const bool ikf_lds = h.inv_n_kf <= kRefKfLds;
        if (n_inv > 0 && ikf_lds) {
            for (int i = tid; i < h.inv_n_kf * 16; i += blockDim.x) {
                const int k = i >> 4, f = i & 15;
                s_ikf[i] = f < 12 ? h.inv_T[12 * k + f] : h.inv_cam[4 * k + f - 12];
            }
        }
        // The event's accepted pairs lie in the search workgroups' regions:
        // pair i is in the last segment with at most i pairs before it (a
        // segment past the last has all of them before it).  Three rounds of
        // seven independent reads find it, where a binary search would be a
        // chain of nine.
        const int incl = wave_incl_scan(sg.count);
        if (wave_lane() == kWave - 1) s_segw[tid / kWave] = incl;
        __syncthreads();
        int cnt = 0;
        {
            int before = incl - sg.count;
#pragma unroll
            for (int q = 0; q < kRefBlock / kWave; ++q) {
                before += q < tid / kWave ? s_segw[q] : 0;
                cnt += s_segw[q];
            }
            s_segx[tid] = before;
            s_segp[tid] = sg.start - before;   // place of pair i: i + this
        }
        __syncthreads();
        auto pair_at = [&](int i) -> const MatchRec& {
            static_assert(kRefBlock == 512, "three rounds of eight");
            int lo = 0;
#pragma unroll
            for (int step = 64; step >= 1; step /= 8) {
                int n = 0;
#pragma unroll
                for (int q = 1; q < 8; ++q) n += s_segx[lo + q * step] <= i;
                lo += n * step;
            }
            return h.match_stage[s_segp[lo] + i];
        };
        const bool use_list = !h.refine_scan && cnt <= ed.list_cap;
        // With the list, the event uses only as many workgroups as give each
        // thread one pair of each direction (every workgroup reads the same
        // counts, so all agree on Be); the others have nothing to add and
        // skip the event.
        const int per_dir = max(cnt, n_inv);
        const int Be = use_list ? max(1, min(B, (int)(((uint32_t)per_dir + blockDim.x - 1) / blockDim.x))) : B;
        if (b >= Be) {
            __syncthreads();
            continue;
        }
        const int stride = Be * blockDim.x;
        // this thread's first kRefCache accepted pairs, loaded once, and
        // whether each is an inlier of the current round
        float cx_[kRefCache], cy_[kRefCache], cz_[kRefCache], cu_[kRefCache], cv_[kRefCache];
        int ck_[kRefCache];
        bool in_[kRefCache];
#pragma unroll
        for (int r = 0; r < kRefCache; ++r) {
            const int i = b * blockDim.x + tid + r * stride;
            ck_[r] = -1;
            cx_[r] = cy_[r] = cz_[r] = cu_[r] = cv_[r] = 0.0f;
            in_[r] = true;
            if (use_list && i < cnt) {
                const MatchRec m = pair_at(i);
                cx_[r] = m.x;
                cy_[r] = m.y;
                cz_[r] = m.z;
                cu_[r] = m.u;
                cv_[r] = m.v;
                ck_[r] = m.kf;
            }
        }
        // (the next kRefLds in LDS, each thread its own)
#pragma unroll 1
        for (int r = 0; use_list && r < kRefLds && b * (int)blockDim.x + (kRefCache + r) * stride < cnt; ++r) {
            const int i = b * blockDim.x + tid + (kRefCache + r) * stride;
            if (i < cnt) {
                const MatchRec m = pair_at(i);
                s_more[r][0][tid] = m.x;
                s_more[r][1][tid] = m.y;
                s_more[r][2][tid] = m.z;
                s_more[r][3][tid] = m.u;
                s_more[r][4][tid] = m.v;
                s_more[r][5][tid] = __int_as_float(m.kf);
            }
        }
        // and its first pair of the other direction
        float ix_ = 0.0f, iy_ = 0.0f, iz_ = 0.0f, iu_ = 0.0f, iv_ = 0.0f;
        int ik_ = -1;
        if (b * (int)blockDim.x + tid < n_inv) {
            const int64_t g = ed.inv_off + (int64_t)b * blockDim.x + tid;
            ix_ = h.inv_xyz[3 * g];
            iy_ = h.inv_xyz[3 * g + 1];
            iz_ = h.inv_xyz[3 * g + 2];
            iu_ = h.inv_uv[2 * g];
            iv_ = h.inv_uv[2 * g + 1];
            const int k = h.inv_kf[g];
            ik_ = (k >= 0 && k < h.inv_n_kf) ? k : -1;
        }
        if (tid == 0) {   // (while the pairs arrive)
            const Sim3d S0 = sim3_load(s_S64);
            sim3_to_f32(S0, &s_S);
            if (n_inv > 0) sim3_to_f32_pose(sim3_inv(S0), &s_Sinv);
        }
        __syncthreads();
        // it: evaluation index (round it / iters); seq: exchanges done, which
        // picks the row buffer and the tag (a converged round skips the rest
        // of its evaluations, in every workgroup alike)
        for (int it = 0, seq = 0; it < total; ++it, ++seq) {
            const int rnd = it / iters, j = it - rnd * iters;
            const fl_sim3 S = s_S;
            // a round after the first keeps its inliers: a pair held in
            // registers is classified at the round's first evaluation (at the
            // round's starting Sim3); any other pair is tested against that
            // Sim3 at every step
            const bool bounded = ROUNDS && rnd > 0;
            const bool classify = bounded && j == 0;
            // Each thread adds its few pairs' terms in float32 (one pair per
            // thread when the list fits the workgroups, a couple of dozen at
            // most when the event's pairs are scanned); everything across
            // threads and workgroups is summed in float64.
            float accf[kNAcc];
            double lossd = 0.0;   // LM: the Huber loss of this thread's pairs, float64
            if (use_list) {
                // Straight-line code for the first pair, whose sums are written
                // rather than added to zeros; the others only where the
                // workgroup has them (a branch of a whole wave).
                auto cached = [&](auto R) {
                    constexpr int r = decltype(R)::value;
                    bool has = ck_[r] >= 0;
                    const int k = max(ck_[r], ed.kf_begin);
                    const float *T, *c;
                    if (kf_lds) {
                        T = &s_kf[16 * (k - ed.kf_begin)];
                        c = T + 12;
                    } else {
                        T = h.kf[k].T;
                        c = &h.kf[k].fx;
                    }
                    double e;
                    if (ROUNDS) {
                        if (classify && has)
                            in_[r] = pair_error64(s_Srs64, T, c[0], c[1], c[2], c[3], cx_[r], cy_[r], cz_[r], cu_[r],
                                                  cv_[r], e) && e <= (double)tau;
                        has = has && in_[r];
                    }
                    refine_pair_f32<false, r == 0>(S.sR, S.t, T, c[0], c[1], c[2], c[3], cx_[r], cy_[r], cz_[r], cu_[r],
                                                   cv_[r], delta, accf, has);
                    if (LM && has &&
                        pair_error64(s_S64, T, c[0], c[1], c[2], c[3], cx_[r], cy_[r], cz_[r], cu_[r], cv_[r], e))
                        lossd += huber64(e, (double)delta);
                };
                cached(std::integral_constant<int, 0>{});
                if (kRefCache > 1 && b * (int)blockDim.x + stride < cnt) cached(std::integral_constant<int, 1>{});
                if (kRefCache > 2 && b * (int)blockDim.x + 2 * stride < cnt)
                    cached(std::integral_constant<int, kRefCache - 1>{});
                for (int i = b * blockDim.x + tid + kRefCache * stride, r = 0; i < cnt; i += stride, ++r) {
                    MatchRec m;
                    if (r < kRefLds) {
                        m.x = s_more[r][0][tid];
                        m.y = s_more[r][1][tid];
                        m.z = s_more[r][2][tid];
                        m.u = s_more[r][3][tid];
                        m.v = s_more[r][4][tid];
                        m.kf = __float_as_int(s_more[r][5][tid]);
                    } else {
                        m = pair_at(i);
                    }
                    const KfDesc& kd = h.kf[m.kf];
                    double e;
                    if (bounded && !(pair_error64(s_Srs64, kd.T, kd.fx, kd.fy, kd.cx, kd.cy, m.x, m.y, m.z, m.u, m.v,
                                                  e) && e <= (double)tau))
                        continue;
                    refine_pair_f32<false>(S.sR, S.t, kd.T, kd.fx, kd.fy, kd.cx, kd.cy, m.x, m.y, m.z, m.u, m.v, delta, accf);
                    if (LM && pair_error64(s_S64, kd.T, kd.fx, kd.fy, kd.cx, kd.cy, m.x, m.y, m.z, m.u, m.v, e))
                        lossd += huber64(e, (double)delta);
                }
            } else {
                // no list (or it overflowed): scan the event's pairs keyframe by keyframe
#pragma unroll
                for (int i = 0; i < kNAcc; ++i) accf[i] = 0.0f;
                for (int k = ed.kf_begin; k < ed.kf_end; ++k) {
                    const KfDesc& kd = h.kf[k];
                    for (int64_t jj = b * blockDim.x + tid; jj < kd.n_pairs; jj += stride) {
                        const int64_t o = kd.pair_off + jj;
                        const uint8_t dec = h.out[0].decision[o];
                        if (dec != FL_ADD && dec != FL_FUSE) continue;
                        const int32_t lp = h.dense ? (int32_t)jj : h.pair_mp[o];
                        const int32_t bi = h.out[0].best_idx[o];
                        if (lp < 0 || lp >= kd.n_mp || bi < 0 || bi >= kd.n_kp) continue;
                        const int64_t gp = kd.mp_off + lp, kp = kd.kp_off + bi;
                        const float x = h.mp_xyz[3 * gp], y = h.mp_xyz[3 * gp + 1], z = h.mp_xyz[3 * gp + 2];
                        const float uo = h.kp_xy[2 * kp], vo = h.kp_xy[2 * kp + 1];
                        double e;
                        if (bounded && !(pair_error64(s_Srs64, kd.T, kd.fx, kd.fy, kd.cx, kd.cy, x, y, z, uo, vo, e) &&
                                         e <= (double)tau))
                            continue;
                        refine_pair_f32<false>(S.sR, S.t, kd.T, kd.fx, kd.fy, kd.cx, kd.cy, x, y, z, uo, vo, delta, accf);
                        if (LM && pair_error64(s_S64, kd.T, kd.fx, kd.fy, kd.cx, kd.cy, x, y, z, uo, vo, e))
                            lossd += huber64(e, (double)delta);
                    }
                }
            }
            if (n_inv > 0) {
                const fl_sim3 Si = s_Sinv;
                auto add_inverse = [&](int k, float x, float y, float z, float uo, float vo) {
                    const float* T = ikf_lds ? s_ikf + 16 * k : h.inv_T + 12 * (int64_t)k;
                    const float* c = ikf_lds ? T + 12 : h.inv_cam + 4 * (int64_t)k;
                    refine_pair_f32<true>(Si.sR, Si.t, T, c[0], c[1], c[2], c[3], x, y, z, uo, vo, delta, accf);
                };
                if (ik_ >= 0) add_inverse(ik_, ix_, iy_, iz_, iu_, iv_);
                for (int i = b * blockDim.x + tid + stride; i < n_inv; i += stride) {
                    const int64_t g = ed.inv_off + (int64_t)i;
                    const int k = h.inv_kf[g];
                    if (k < 0 || k >= h.inv_n_kf) continue;
                    add_inverse(k, h.inv_xyz[3 * g], h.inv_xyz[3 * g + 1], h.inv_xyz[3 * g + 2], h.inv_uv[2 * g],
                                h.inv_uv[2 * g + 1]);
                }
            }
            // the waves' sums, in float64 beyond a quad of threads
            {
                int idx;
                const double v = wave_reduce_quad<kNAcc>(accf, idx);
                if (idx >= 0) s_w[(tid / kWave) * NV + idx] = v;
                if (LM) {
                    double loss = lossd;
#pragma unroll
                    for (int off = 32; off > 0; off >>= 1) loss += __shfl_xor(loss, off);
                    if (wave_lane() == 0) s_w[(tid / kWave) * NV + 36] = loss;
                }
            }
            __syncthreads();
            if (Be > 1) {
                // Exchange of the Be partial sums of this step as tagged words
                // (device-coherent stores and loads of 16 bytes, the two words
                // of a value; each word carries its own tag).  Rows alternate
                // between two buffers by step: a workgroup writes step it + 2
                // only after it has read every row of step it + 1, which every
                // workgroup writes only after reading all rows of step it.
                const size_t slot = ((size_t)(seq & 1) * n_units + (size_t)ev * B);   // rows of this step: Be
                const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(
                    uniform_p(h.refine_rows + slot * kRefWords), 0, Be * kRefWords * 8, 0x00020000);
                const uint32_t tag = refine_tag(epoch, seq);
                const int w = __builtin_amdgcn_readfirstlane(tid / kWave), c = wave_lane();
                if (tid < NV) {
                    const uint64_t bits = (uint64_t)__double_as_longlong(add_segments<NV>(s_w, tid));
                    const v4u x = {tag, (uint32_t)(bits >> 32), tag, (uint32_t)bits};
                    __builtin_amdgcn_raw_buffer_store_b128(x, rows, 16 * tid, b * kRefWords * 8, kDeviceScope);
                }
                // Wave w loads rows w, w + kSeg, ..., lane c value c of each (a
                // row with a tag that is not yet the current one is loaded
                // again), and adds them in that order; then the segments are
                // added pairwise.  The order is the same in every workgroup, so
                // all of them solve for bitwise the same step.
                constexpr int kRowsPer = kRefMaxB / kSeg;
                v4u x[kRowsPer];
                uint32_t pending = 0;   // the same in every lane, like the branches on it
#pragma unroll
                for (int jr = 0; jr < kRowsPer; ++jr)
                    if (w + kSeg * jr < Be) pending |= 1u << jr;
                unsigned spins = 0;
                // the rows take about 1,600 cycles to arrive, and a load that
                // is on its way when they do costs as much again: the first is
                // sent 900 cycles on (20 keyframes: 9,500 cycles to here a step
                // without the pause, 8,850 with it)
                __builtin_amdgcn_s_sleep(14);
                while (pending) {
                    asm volatile("" ::: "memory");   // the rows change under this loop
#pragma unroll
                    for (int jr = 0; jr < kRowsPer; ++jr)
                        if (pending >> jr & 1u)
                            x[jr] = __builtin_amdgcn_raw_buffer_load_b128(rows, 16 * min(c, NV - 1),
                                                                          (w + kSeg * jr) * kRefWords * 8, kDeviceScope);
#pragma unroll
                    for (int jr = 0; jr < kRowsPer; ++jr)
                        if ((pending >> jr & 1u) && __ballot(x[jr].x != tag || x[jr].z != tag) == 0ull)
                            pending &= ~(1u << jr);
                    if (pending && ++spins > kSpinLimit) {
                        s_fail = 1;
                        break;
                    }
                }
                double a0 = 0.0, a1 = 0.0;
#pragma unroll
                for (int jr = 0; jr < kRowsPer; ++jr) {
                    if (w + kSeg * jr < Be) {
                        const double y = __longlong_as_double(((long long)x[jr].y << 32) | (long long)x[jr].w);
                        if (jr & 1) a1 += y; else a0 += y;
                    }
                }
                if (c < NV) s_q[w * NV + c] = a0 + a1;
                __syncthreads();
                if (s_fail) break;
            }
            if (tid < kWave) {
                // Wave 0, every lane alike: the event's sums, then the step,
                // which the lanes compose with S together.
                if (tid < NV) s_out[tid] = add_segments<NV>(Be > 1 ? s_q : s_w, tid);
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                __builtin_amdgcn_wave_barrier();
                bool round_end = j == iters - 1;
                double d[7];
                if (!LM) {
                    const ComposeIn in = compose_inputs(s_cf, s_S64);
                    if (solve7(s_out, s_out + 7, 0.0, d))
                        compose_exp_lanes(d, in, s_S64, &s_S, n_inv > 0 ? &s_Sinv : nullptr);
                } else {
                    // the evaluation just summed was at s_S64: the round's start
                    // (j = 0) or the last candidate
                    bool take = j == 0;
                    double lam = j == 0 ? (double)h.lm_lambda : s_lm[1];
                    if (j > 0) {
                        const double rho = s_lm[0] > 0.0 ? (s_lm[0] - s_out[36]) / s_lm[0] : 0.0;
                        take = rho > kLmConverged;
                        if (!take && rho >= -kLmConverged) round_end = true;   // converged
                        if (take) lam = fmax(lam * 0.1, 1e-12);
                        else if (!round_end) lam = fmin(lam * 10.0, 1e16);
                    }
                    if (take) {
                        if (tid < kNAcc) s_acc[tid] = s_out[tid];
                        if (tid < 13) s_Sacc[tid] = s_S64[tid];
                    }
                    if (tid == 0) {
                        if (take) s_lm[0] = s_out[36];
                        s_lm[1] = lam;
                    }
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    if (!round_end && solve7(s_acc, s_acc + 7, lam, d)) {
                        compose_exp_lanes(d, compose_inputs(s_cf, s_Sacc), s_S64, &s_S, nullptr);
                    } else {
                        if (tid < 13) s_S64[tid] = s_Sacc[tid];
                        if (tid < 9) s_S.sR[tid] = (float)(s_Sacc[12] * s_Sacc[tid]);
                        else if (tid < 12) s_S.t[tid - 9] = (float)s_Sacc[tid];
                    }
                }
                if (round_end) {
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    if (tid < 13) s_Srs64[tid] = s_S64[tid];   // the next round's starting Sim3
                }
                if (tid == 0) s_round_end = round_end;
            }
            __syncthreads();
            if (LM && s_round_end) it = (rnd + 1) * iters - 1;   // on to the next round
        }
        if (b == 0 && tid == 0) {
            if (!s_fail) {
                for (int i = 0; i < 13; ++i) h.event_S[13 * (int64_t)ev + i] = s_S64[i];
                if (h.event_S32_out) sim3_to_f32(sim3_load(s_S64), &h.event_S32_out[ev]);
            }
            if (h.event_n_matched)
                h.event_n_matched[ev] = s_fail ? -1 : (int32_t)(LM ? s_acc[35] : s_out[35]);
        }
        __syncthreads();
    }
    // The ADD conflicts of the search that precedes this launch: the search
    // workgroups' ADD regions go to workgroups from the last one down, so
    // workgroups with no refinement work (most of them for a single event)
    // take them while the others iterate.  The refinement reads accepted
    // pairs only, which an ADD and its relabelling as FUSE both are.
    if (h.resolve_in_refine) {
        // by the workgroups that have no share of any event, if that is most of
        // them: at the end of the others it would come on top of the steps
        const unsigned long long tag = (unsigned long long)epoch << 32;
        const int spare = (int)gridDim.x - n_units;
        const bool spare_only = 2 * spare >= (int)gridDim.x;
        const int r0 = spare_only ? (int)blockIdx.x - n_units : (int)(gridDim.x - 1 - blockIdx.x);
        for (int r = r0; r >= 0 && r < h.n_wg; r += spare_only ? spare : (int)gridDim.x) resolve_region_adds(h, r, tag);
    }
}

}  // namespace fl
